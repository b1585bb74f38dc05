"""On which streams ByPhase issues its calls, and which of them wait for which: recorded by stand-ins for the context and the
streams, without a GPU."""
import pytest
import torch

import paper_2006_08085_amd as D
from paper_2006_08085_amd.algorithms import ByPhase


class _Stream:
    raw = 100

    def __init__(self, log):
        _Stream.raw += 1
        self.cuda_stream, self.log = _Stream.raw, log

    def wait_stream(self, other):
        self.log.append(("wait", self.cuda_stream, other.cuda_stream))


class _Recorder:
    """A context that notes the stream of every call."""
    n, d, ld = 3, 5, 5

    def __init__(self, cuda):
        self.cuda, self.log = cuda, cuda.log

    def __getattr__(self, name):
        def call(*args, stream=None):
            self.log.append((name, self.cuda.current.cuda_stream if stream is None else stream))
        return call


class _Cuda:
    def __init__(self, monkeypatch):
        self.log = []
        self.current = _Stream(self.log)
        monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: self.current)
        monkeypatch.setattr(torch.cuda, "Stream", lambda device=None: _Stream(self.log))


def _by_phase(cuda, grad, overlap=True, cls=ByPhase, **kw):
    return cls(_Recorder(cuda), torch.zeros(3, 5), 0.1, grad, overlap=overlap, **kw)


@pytest.mark.parametrize("granularity", ["iteration", "phase"])
@pytest.mark.parametrize("switch_at", [0, 1, 2])
def test_the_phase_end_waits_on_the_stream_it_runs_on(monkeypatch, granularity, switch_at):
    cuda = _Cuda(monkeypatch)

    def grad(t, q, X, g):                      # leaves another stream current
        if t == switch_at:
            cuda.current = _Stream(cuda.log)

    bp = _by_phase(cuda, grad, granularity=granularity)
    bp.phase(3)
    comm, end = bp.comm.cuda_stream, cuda.current.cuda_stream
    assert cuda.log[-2:] == [("wait", end, comm), ("phase_end", end)]
    assert {s for name, s in (e for e in cuda.log if e[0].startswith("gossip"))} == {comm}
    cuda.log.clear()
    bp.phase(3)                                # the next phase starts behind the phase end, wherever that ran
    assert cuda.log[0] == ("wait", comm, end)


def test_without_overlap_the_gossip_follows_the_current_stream(monkeypatch):
    cuda = _Cuda(monkeypatch)

    def grad(t, q, X, g):
        cuda.current = _Stream(cuda.log)

    _by_phase(cuda, grad, overlap=False).phase(2)
    order = [e for e in cuda.log if e[0] in ("gossip_round", "accumulate", "phase_end")]
    first, second = order[0][1], order[2][1]
    assert first != second
    assert [s for name, s in order if name == "gossip_round"] == [first, first, second, second]
    assert not [e for e in cuda.log if e[0] == "wait"]


def test_a_phase_goes_through_iteration(monkeypatch):
    class Counting(ByPhase):
        seen = 0

        def iteration(self, R, eta=-1.0):
            self.seen += 1
            super().iteration(R, eta)

    bp = _by_phase(_Cuda(monkeypatch), lambda t, q, X, g: None, cls=Counting)
    bp.phase(4)
    assert bp.seen == 4 and bp.k == 1


class _RegisterTile(_Recorder):
    """A context whose graph the register-resident kernels serve: a phase's rounds are one call."""

    def kernel(self):
        return D.DETAG_KERNEL_REGISTER_TILE


@pytest.mark.parametrize("overlap", [True, False])
def test_the_rounds_of_a_phase_in_one_call(monkeypatch, overlap):
    cuda = _Cuda(monkeypatch)
    bp = ByPhase(_RegisterTile(cuda), torch.zeros(3, 5), 0.1, lambda t, q, X, g: None, overlap=overlap)
    now = cuda.current.cuda_stream
    for _ in range(2):
        cuda.log.clear()
        bp.phase(3)
        gossip = [e for e in cuda.log if e[0].startswith("gossip")]
        if overlap:                            # behind what made its inputs, and waited for by the phase end
            comm = bp.comm.cuda_stream
            assert comm != now and gossip == [("gossip_rounds", comm)]
            assert cuda.log[:2] == [("wait", comm, now), ("gossip_rounds", comm)]
            assert cuda.log[-2:] == [("wait", now, comm), ("phase_end", now)]
        else:
            assert gossip == [("gossip_rounds", now)] == cuda.log[:1]
