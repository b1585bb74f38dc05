"""On which streams ByPhase issues its calls, and which of them wait for which: recorded by stand-ins for the context and the
streams, without a GPU."""
import contextlib

import pytest
import torch

import paper_2006_08085_amd as D
from paper_2006_08085_amd import bench_by_phase
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


def test_what_the_measuring_tool_calls_iterations(monkeypatch):
    """A launch per round, also where phase() issues the rounds in one."""
    cuda = _Cuda(monkeypatch)
    bp = ByPhase(_RegisterTile(cuda), torch.zeros(3, 5), 0.1, lambda t, q, X, g: None)
    bench_by_phase.iterations(bp, 3)
    assert [e[0] for e in cuda.log if e[0].startswith("gossip")] == ["gossip_round"] * 6 and bp.k == 1


class _Failing:
    """A gradient that raises once, in iteration `at`."""

    def __init__(self, at):
        self.at = at

    def __call__(self, t, q, X, g):
        if t == self.at:
            self.at = None
            raise KeyError("no gradient")


@pytest.mark.parametrize("context,granularity,calls", [(_RegisterTile, "iteration", ["gossip_rounds"]),
                                                       (_Recorder, "iteration", ["gossip_round"] * 6),
                                                       (_RegisterTile, "phase", ["gossip_accel"] * 2)])
def test_a_phase_interrupted_by_its_first_gradient_is_not_gossiped_again(monkeypatch, context, granularity, calls):
    cuda = _Cuda(monkeypatch)
    bp = ByPhase(context(cuda), torch.zeros(3, 5), 0.1, _Failing(0), granularity=granularity)
    with pytest.raises(KeyError):
        bp.phase(3)
    bp.phase(3)
    assert [e[0] for e in cuda.log if e[0].startswith("gossip")] == calls and (bp.t, bp.k, bp.r) == (3, 1, 0)
    cuda.log.clear()
    bp.phase(3)
    assert [e[0] for e in cuda.log if e[0].startswith("gossip")] == calls


@pytest.mark.parametrize("at", [0, 1])
def test_an_interrupted_phase_ends_as_it_was_issued(monkeypatch, at):
    """Its rounds are issued for one R and eta, whatever the iterations that finish it ask for."""
    cuda = _Cuda(monkeypatch)
    bp = ByPhase(_RegisterTile(cuda), torch.zeros(3, 5), 0.1, _Failing(at))
    with pytest.raises(KeyError):
        bp.phase(3, 0.5)
    cuda.log.clear()
    for R, eta in ((4, 0.5), (3, 0.25)):
        with pytest.raises(RuntimeError, match="issued for"):
            bp.iteration(R, eta)
    assert not cuda.log and bp.t == at
    while bp.k == 0:
        bp.iteration(3, 0.5)
    assert bp.t == 3 and not [e for e in cuda.log if e[0].startswith("gossip")]
    bp.iteration(4, 0.25)


@pytest.mark.parametrize("context", [_RegisterTile, _Recorder])
@pytest.mark.parametrize("at", [0, 1, 3, 4])
def test_a_recording_that_fails_leaves_everything_as_it_was(monkeypatch, context, at):
    cuda = _Cuda(monkeypatch)
    monkeypatch.setattr(torch.cuda, "CUDAGraph", lambda: None)
    monkeypatch.setattr(torch.cuda, "graph", lambda graph: contextlib.nullcontext())
    bp = ByPhase(context(cuda), torch.zeros(3, 5), 0.1, _Failing(at))
    held = [id(t) for t in (*bp.xt, *bp.y, bp.G_k, bp.G_km1)]
    with pytest.raises(KeyError):
        bp.capture_two_phases(3)
    assert [id(t) for t in (*bp.xt, *bp.y, bp.G_k, bp.G_km1)] == held and (bp.t, bp.k, bp.r) == (0, 0, 0)
    cuda.log.clear()
    bp.phase(3)
    assert len([e for e in cuda.log if e[0].startswith("gossip")]) == (1 if context is _RegisterTile else 6)
    bp.grad = _Failing(3)
    with pytest.raises(KeyError):
        bp.phase(3)
    with pytest.raises(RuntimeError, match="in progress"):     # its gossip would be missing from the recording
        bp.capture_two_phases(3)
