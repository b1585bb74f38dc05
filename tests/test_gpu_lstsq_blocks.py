"""Least-squares gradient at the edges of its blocks: rows of less than one 16-byte piece per lane, around 1024 columns,
sample counts around a block's rows, both widths of the column blocks, odd pitches."""
import numpy as np
import pytest
import torch

import paper_2006_08085_amd as D
from oracle import objectives as OO
from workloads import generate as gen
from tests.gpu_util import DEV, SENTINEL, _built, padding_ok, to_dev, to_host  # noqa: F401
from tests.util import TOL_F32, amax, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,m,pad", [(1, 1, 1, 0), (3, 5, 2, 1), (2, 255, 63, 0), (2, 1023, 65, 2), (4, 1025, 64, 0), (5, 2050, 7, 3),
                                       (16, 8193, 130, 1), (64, 2049, 3, 0)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_blocks(n, d, m, pad, dtype):
    ld = d + pad
    X = gen.state(n, d, seed=1)
    if dtype == "bf16":
        X = OO.round_bf16(X)
    A, b = gen.lstsq_problem(n, m, d, seed=2, shift=0.5)
    topo = D.Topology.ring() if n > 1 else D.Topology.from_dense(np.ones((1, 1)))
    ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if dtype == "bf16" else D.DETAG_F32)
    G = to_dev(np.zeros((n, d)), ld)
    ctx.grad_lstsq(to_dev(X, ld, torch.bfloat16 if dtype == "bf16" else torch.float32), torch.from_numpy(A).to(DEV),
                   torch.from_numpy(b).to(DEV), G)
    ref = OO.grad_lstsq(X, A, b)
    # residuals are sums of d products of size |A| |x|, entries of G sums of m products of those
    S = max(amax(ref), amax(A) * np.sqrt(d) * amax(A) * amax(X))
    assert rel_err(to_host(G, d), ref, S) < TOL_F32
    assert padding_ok(G, d)


@pytest.mark.parametrize("d", [2, 3, 4, 6, 7, 258, 511, 770, 1027])
@pytest.mark.parametrize("m", [3, 65])  # one launch and two (both two beyond 1024 columns)
def test_the_last_columns_of_a_row(d, m):
    """A lane whose four columns do not all exist reads the row's last four: each product is counted once.  Small whole
    numbers, so that every sum is exact in any order."""
    n, rng = 3, np.random.default_rng(d * m)
    X, A, b = (rng.integers(-3, 4, shape).astype(np.float64) for shape in ((n, d), (n, m, d), (n, m)))
    ctx = D.detag_create(D.Topology.ring(), n, d, d)
    G = to_dev(np.zeros((n, d)), d)
    ctx.grad_lstsq(to_dev(X, d), *(torch.from_numpy(t.astype(np.float32)).to(DEV) for t in (A, b)), G)
    assert np.array_equal(to_host(G, d), OO.grad_lstsq(X, A, b))


def _alone(d):
    return D.detag_create(D.Topology.from_dense(np.ones((1, 1))), 1, d, d)


def test_more_rows_than_a_launch_has_threads_for():
    m = (1 << 26) + 8                                   # a wavefront per row: 2^32 threads and some
    A, b = torch.zeros(1, m, 1, device=DEV), torch.full((1, m), -1.0, device=DEV)
    A[0, :3, 0], A[0, -1, 0] = 1.0, 3.0
    X, G = torch.ones(1, 1, device=DEV), torch.zeros(1, 1, device=DEV)
    _alone(1).grad_lstsq(X, A, b, G)
    assert G.item() == 3 * 1.0 * 2.0 + 3.0 * 4.0        # A^T (A x - b), exact in fp32


def test_more_columns_than_a_launch_has_threads_for():
    d = (1 << 30) + 3                                   # four threads per column: 2^32 and some
    A, b = torch.zeros(1, 1, d, device=DEV), torch.full((1, 1), -2.0, device=DEV)
    A[0, 0, -2:] = torch.tensor([3.0, 4.0], device=DEV)
    A[0, 0, 1 << 29] = 5.0
    X, G = torch.zeros(1, d, device=DEV), torch.full((1, d), SENTINEL, device=DEV)
    _alone(d).grad_lstsq(X, A, b, G)
    assert torch.equal(G, 2.0 * A[0])                   # A^T (A x - b), exact in fp32


@pytest.mark.parametrize("n,d,m", [(1, 1, 1), (8, 1024, 64), (16, 1024, 64), (3, 1023, 63), (5, 64, 17), (64, 256, 5), (85, 129, 64), (7, 1021, 16)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_one_launch_gives_the_bits_of_two(n, d, m, dtype):
    """Problems of up to 64 samples and 1024 columns take one launch; the same rows among more samples, weighted by zero
    residuals, take two."""
    ld = d + 1
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X = to_dev(gen.state(n, d, seed=1), ld, tdt)
    A, b = (torch.from_numpy(t).to(DEV) for t in gen.lstsq_problem(n, m, d, seed=2, shift=0.5))
    topo = D.Topology.ring() if n > 1 else D.Topology.from_dense(np.ones((1, 1)))
    ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if dtype == "bf16" else D.DETAG_F32)
    G, G2 = to_dev(np.zeros((n, d)), ld), to_dev(np.zeros((n, d)), ld)
    ctx.grad_lstsq(X, A, b, G)
    # samples of zeros from the 65th on: exact zero residuals, which add exact zeros to every column
    A2, b2 = torch.zeros(n, 64 + 1, d, device=DEV), torch.zeros(n, 64 + 1, device=DEV)
    A2[:, :m], b2[:, :m] = A, b
    ctx.grad_lstsq(X, A2, b2, G2)
    assert torch.equal(G[:, :d], G2[:, :d])
    assert padding_ok(G, d) and padding_ok(G2, d)
    ref = OO.grad_lstsq(to_host(X, d), A.cpu().numpy(), b.cpu().numpy())
    S = max(amax(ref), amax(A.cpu().numpy()) * np.sqrt(d) * amax(A.cpu().numpy()) * amax(to_host(X, d)))
    assert rel_err(to_host(G, d), ref, S) < TOL_F32


@pytest.mark.parametrize("n,d,m", [(8, 1024, 64), (16, 500, 16), (3, 1023, 63), (5, 64, 17), (4, 65, 64), (8, 1025, 64)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_the_gradient_may_lie_over_the_state_or_the_targets(n, d, m, dtype):
    """Both are read before G is written: the bits of a call whose G lies apart."""
    ld = d + 1
    bf16 = dtype == "bf16"
    X = to_dev(gen.state(n, d, seed=1), ld, torch.bfloat16 if bf16 else torch.float32)
    A, b = (torch.from_numpy(t).to(DEV) for t in gen.lstsq_problem(n, m, d, seed=2, shift=0.5))
    ctx = D.detag_create(D.Topology.ring(), n, d, ld, D.DETAG_BF16 if bf16 else D.DETAG_F32)
    G = torch.zeros(n, ld, device=DEV)
    ctx.grad_lstsq(X, A, b, G)

    over_x = torch.empty(n, ld, device=DEV)
    x = over_x.view(torch.bfloat16).view(-1)[:n * ld].view(n, ld) if bf16 else over_x
    shifted = torch.empty(n * ld + 70, device=DEV)          # G starts 64 floats into X
    y = (shifted.view(torch.bfloat16) if bf16 else shifted)[:n * ld].view(n, ld)
    over_b = torch.empty(n, ld, device=DEV)
    for state, grad in ((x, over_x), (y, shifted[64:64 + n * ld].view(n, ld))):
        state.copy_(X)
        ctx.grad_lstsq(state, A, b, grad)
        assert torch.equal(grad[:, :d], G[:, :d])
    if m <= ld:
        targets = over_b.view(-1)[-n * m:].view(n, m)
        targets.copy_(b)
        ctx.grad_lstsq(X, A, targets, over_b)
        assert torch.equal(over_b[:, :d], G[:, :d])


@pytest.mark.parametrize("n,d,m", [(8, 1024, 64), (8, 257, 16), (8, 256, 16), (85, 129, 64), (4, 1025, 64)])
def test_a_recorded_call_gives_the_bits_of_the_others(n, d, m):
    """A recorded call goes to one launch up to 256 columns, others up to 1024."""
    ctx = D.detag_create(D.Topology.ring(), n, d, d)
    X, G = to_dev(gen.state(n, d, seed=1), d), torch.zeros(n, d, device=DEV)
    A, b = (torch.from_numpy(t).to(DEV) for t in gen.lstsq_problem(n, m, d, seed=2, shift=0.5))
    ctx.grad_lstsq(X, A, b, G)
    graph, recorded = torch.cuda.CUDAGraph(), torch.zeros(n, d, device=DEV)
    with torch.cuda.graph(graph):
        ctx.grad_lstsq(X, A, b, recorded)
    for k in range(3):
        recorded.zero_()
        X.mul_(1.0 if k == 0 else -0.5)
        graph.replay()
        ctx.grad_lstsq(X, A, b, G)
        torch.cuda.synchronize()
        assert torch.equal(recorded, G), k
