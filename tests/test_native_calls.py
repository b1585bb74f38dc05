"""The native form of the hot path's calls takes plain arguments only and leaves the rest to ctypes, which words the refusals:
both ways accept the same and give the same."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2006_08085_amd as D
from paper_2006_08085_amd import binding, build


@pytest.fixture(scope="module", autouse=True)
def _built():
    build.ensure_built()
    assert binding.calls() is not None


def test_what_is_not_plain_is_left_to_ctypes():
    n, d, ld = 6, 100, 104
    ctx = D.detag_create(D.Topology.ring(), n, d, ld)
    f, t = ctx._native(), torch.zeros(n, ld)
    assert f.step(t, t, t, t, 0.1, 1, -1.0, 0) is None                 # not on a GPU
    assert f.step(1, None, "a", t, 0.1, 1, -1.0, 0) is None
    assert f.track(t) is None and f.accumulate(t, t, 1.0, 2) is None   # too few, too many
    assert f.mean(t, t) is None and f.consensus_error(t, None) is None and f.average_consensus("x", t) is None
    assert f.grad_softmax_bf16(t, t, t, t, 3, t, None) is None
    with pytest.raises(ValueError, match="X must be a GPU tensor"):
        ctx.step(t, t, t, t, 0.1, 1)
    with pytest.raises(ValueError, match="G_acc must be a GPU tensor"):
        ctx.accumulate(t, t)
    ctx.close()
    assert f.track(t, t, t) is None


@pytest.fixture
def sources(monkeypatch, tmp_path):
    """Copies of the sources of the native calls, and an empty place for what is built from them."""
    copies = [shutil.copy(f, tmp_path) for f in build.CALLS_SOURCES]
    monkeypatch.setattr(build, "CALLS_SOURCES", copies)
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(binding, "_calls", None)
    return copies


def _ctypes_serves():
    """The calls work, and word their refusals, without a native form."""
    assert binding.calls() is None
    ctx, t = D.detag_create(D.Topology.ring(), 6, 100, 104), torch.zeros(6, 104)
    with pytest.raises(ValueError, match="X must be a GPU tensor"):
        ctx.step(t, t, t, t, 0.1, 1)
    factors = D.Factors(ctx, 0)
    with pytest.raises(ValueError, match="Z must be a GPU tensor"):
        factors.average(t)
    assert ctx._native().step(t, t, t, t, 0.1, 1, -1.0, 0) is None
    ctx.close()


def test_without_the_native_form_ctypes_serves(sources):
    _ctypes_serves()


def test_a_native_form_of_other_sources_or_another_torch_is_not_loaded(sources, monkeypatch):
    built = build.calls_path()
    with open(built, "w") as f:
        f.write("loading this would raise")
    with open(sources[1], "a") as f:
        f.write("/* a declaration that changed */")
    assert build.calls_path() != built
    _ctypes_serves()
    monkeypatch.setattr(torch, "__version__", "0.0.1+other")
    assert "0.0.1_other" in build.calls_path()
    monkeypatch.setattr(binding, "_calls", None)
    _ctypes_serves()


def test_what_keeps_the_native_form_from_being_built_is_reported_and_no_error(sources, monkeypatch, capfd):
    with monkeypatch.context() as m:
        m.setattr(shutil, "which", lambda name: None)
        assert build.build_calls() is None
    with monkeypatch.context() as m:
        m.setitem(sys.modules, "torch", None)                          # not importable
        assert build.build_calls() is None and build.calls_path() is None
    with open(sources[0], "a") as f:
        f.write("#error another torch")
    assert build.build_calls() is None
    err = capfd.readouterr().err
    assert err.count("native calls not built") == 3 and "#error another torch" in err
    assert not [f for f in os.listdir(build.HERE) if f.endswith(".so")]


@pytest.mark.gpu
def test_both_ways_accept_the_same_and_give_the_same(monkeypatch):
    n, d, ld = 8, 300, 304
    dev = "cuda"
    ctx = D.detag_create(D.Topology.ring(), n, d, ld)
    g = torch.Generator(device=dev).manual_seed(1)
    X, Y, G, B = (torch.randn(n, ld, device=dev, generator=g) for _ in range(4))
    h, hw = torch.rand(d, device=dev, generator=g), torch.rand(n, ld, device=dev, generator=g)
    A, b = torch.randn(n, 16, d, device=dev, generator=g), torch.randn(n, 16, device=dev, generator=g)
    factors = D.Factors(ctx, 0)
    feats = torch.randn(n, 40, 32, device=dev, generator=g).bfloat16()
    labels = torch.zeros(n, 40, dtype=torch.int32, device=dev)
    batch = torch.arange(32, dtype=torch.int32, device=dev).repeat(n, 1)
    soft = D.detag_create(D.Topology.ring(), n, 2 * 33, 2 * 33)

    def everything(f=float, i=int):
        x, y, gr, o = (t.clone() for t in (X, Y, G, B))
        out = []
        ctx.step(x, y, gr, o, f(0.1), i(3))
        ctx.step(x, y, gr, o, 1, i(2), eta=f(0.25), variant=i(1))
        ctx.step_quadratic(x, y, gr, h, B, f(0.1), i(2), sigma=f(0.1), seed=i(5), step=i(2))
        ctx.step_quadratic(x, y, gr, hw, B, f(0.1), i(2), seed=-1, step=2 ** 32 + 3)
        ctx.grad_quadratic_diag(x, h, B, gr, sigma=f(0.2), seed=i(3), step=i(1))
        ctx.grad_quadratic_diag(x, hw, B, gr, noise=B, sigma=f(0.2))
        ctx.accumulate(gr, o, f(0.5))
        ctx.track(y, gr, o)
        ctx.dpsgd_step(x, gr, f(0.1))
        ctx.gossip_accel(x, i(3))
        ctx.gossip_round(x, y, y, f(0.1), stream=torch.cuda.current_stream().cuda_stream)
        ctx.gossip_rounds(x, y, i(2))
        ctx.gossip_rounds(x, None, i(2))
        out += [ctx.mean(x), ctx.consensus_error(x), ctx.mean(x, torch.zeros(d + 5, device=dev))[:d]]
        ctx.phase_end(x, x, y, gr, o, f(0.1))
        ctx.defacto_update(x, y, gr, f(0.1))
        factors.average(y)
        ctx.grad_lstsq(x, A, b, gr)
        xs, gs, loss = X[:, :66].contiguous(), torch.zeros(n, 66, device=dev), torch.zeros(n, device=dev)
        soft.grad_softmax_bf16(xs, feats, labels, batch, i(2), gs, loss)
        soft.grad_softmax_bf16(xs, feats, labels, batch, i(2), gs)
        torch.cuda.synchronize()
        return out + [x, y, gr, o, gs, loss]

    native = everything()
    other = torch.cuda.Stream()                                        # the current stream is looked up with every call
    with torch.cuda.stream(other):
        other.wait_stream(torch.cuda.default_stream())
        streamed = everything()
    odd = everything(f=np.float64)
    bad = torch.zeros(n, ld + 8, device=dev)[:, :ld]
    refusals = [(lambda: ctx.track(bad, G, B), "pitch"), (lambda: ctx.track(Y.double(), G, B), "must be torch.float32"),
                (lambda: ctx.track(Y[:4], G, B), "row-major"), (lambda: ctx.grad_lstsq(X, A[:, :, :-1], b, G), "shape"),
                (lambda: ctx.grad_quadratic_diag(X, h[::2], B, G), "contiguous float32"),
                (lambda: ctx.step_quadratic(X, Y, G, torch.zeros(1, 1, d, device=dev), B, 0.1, 1), "contiguous float32")]
    for call, words in refusals:
        with pytest.raises(ValueError, match=words):
            call()
    with pytest.raises(D.DetagError) as e:
        ctx.step(X, X, G, B, 0.1, 1)
    assert e.value.status == D.DETAG_EINVAL and "overlap" in e.value.message

    class Nothing:
        def __getattr__(self, name):
            return lambda *a: None

    monkeypatch.setattr(ctx, "_fast", Nothing())
    monkeypatch.setattr(soft, "_fast", Nothing())
    by_ctypes = everything()
    for one in (streamed, odd, by_ctypes):
        assert all(torch.equal(a, b) for a, b in zip(native, one))


THROWING = """
#include "py_calls.cpp"
extern "C" PyObject *throwing() {  // an entry point that runs out of memory, called as every other one is
  Calls c{};
  c.ctx = reinterpret_cast<detag_ctx *>(&c);
  return call(reinterpret_cast<PyObject *>(&c), nullptr, 0, 0, [](Args &) {
    return []() -> detag_status { throw std::bad_alloc(); };
  });
}
"""
CALLER = """
import ctypes, sys, threading, torch
throwing = ctypes.PyDLL(sys.argv[1]).throwing
throwing.restype = ctypes.py_object
for _ in range(3):
    try:
        throwing()
        sys.exit("no error")
    except MemoryError:
        pass
t = threading.Thread(target=lambda: [[] for _ in range(100000)])       # the interpreter lock is held again
t.start(), t.join()
print("went on")
"""


def test_an_exception_behind_an_entry_point_leaves_the_interpreter_whole(tmp_path):
    source, lib = tmp_path / "throwing.cpp", str(tmp_path / "throwing.so")
    source.write_text(THROWING)
    subprocess.run(build.calls_command(str(source), lib), check=True, capture_output=True)
    r = subprocess.run([sys.executable, "-c", CALLER, lib], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "went on" in r.stdout, (r.returncode, r.stderr[-2000:])
