"""The LDS-resident kernels at the edges of their forms: the last matrix that counts as small and the first that does
not (n * ceil(d/4) = 2^19), ragged widths and odd pitches, worker counts around a full set of rows per lane, one weight
for the whole matrix and weights of its own, even and odd K, against the fp64 oracle on sampled columns."""
import numpy as np
import pytest
import torch

import paper_2006_08085_amd as D
from oracle import gossip as OG, noise as ON, objectives as OO, topology as OT
from workloads import generate as gen
from tests.gpu_util import DEV, SENTINEL, _built  # noqa: F401
from tests.util import TOL_BF16, TOL_F32, amax, rel_err

pytestmark = pytest.mark.gpu


def _graph(kind, n):
    if kind == "rr":
        return gen.edges_random_regular(n, 4, seed=n)
    if kind == "ring":
        return gen.edges_ring(n)
    if kind == "rr8":
        return np.array(sorted({tuple(sorted((i, (i + s) % n))) for i in range(n) for s in (1, 5, 7, 11)}))
    rng = np.random.default_rng(n)                       # a path and random edges, at most 8 neighbours
    e, deg = {(i, i + 1) for i in range(n - 1)}, np.full(n, 2)
    while len(e) < 2 * n:
        a, b = sorted(rng.integers(0, n, 2).tolist())
        if a != b and (a, b) not in e and deg[a] < 8 and deg[b] < 8:
            e.add((a, b)); deg[a] += 1; deg[b] += 1
    return np.array(sorted(e), dtype=np.int64)


def _matrix(n, d, ld, seed, dtype=torch.float32):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    t = torch.full((n, ld), SENTINEL, device=DEV)
    t[:, :d].normal_(generator=g)
    return t.to(dtype)


def _cols(t, cols):
    return t[:, torch.as_tensor(cols, device=DEV)].double().cpu().numpy()


@pytest.mark.parametrize("n,kind", [(3, "ring"), (5, "ring"), (8, "irregular"), (9, "rr"), (20, "ring"), (31, "irregular"),
                                    (64, "rr"), (65, "rr8"), (100, "irregular"), (129, "rr"), (256, "irregular"), (256, "rr")])
@pytest.mark.parametrize("extra,pad,dtype,K", [(0, 0, "f32", 3), (0, 3, "bf16", 4), (1, 2, "f32", 4), (2, 1, "bf16", 3), (7, 0, "f32", 5)])
def test_forms_and_edges(n, kind, extra, pad, dtype, K):
    # d: 4-column groups times n is 2^19 at most for extra = 0 (small: one or two rows per lane), more otherwise (four)
    d = (1 << 19) // n * 4 + 5 * extra
    ld = d + pad
    bf = dtype == "bf16"
    sd, tol = (torch.bfloat16, TOL_BF16) if bf else (torch.float32, TOL_F32)
    e = _graph(kind, n)
    W = OT.mixing_matrix(n, e, "metropolis")
    topo = D.Topology.ring() if kind == "ring" else D.Topology.from_edges(e, D.DETAG_W_METROPOLIS)
    ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if bf else D.DETAG_F32)
    assert ctx.kernel() == D.DETAG_KERNEL_LDS_TILE
    eta, alpha, sigma, seed = 0.35, 0.2, 0.1, 11
    rng = np.random.default_rng(5)
    cols = np.unique(np.concatenate([np.arange(min(d, 40)), np.arange(max(0, d - 300), d), rng.integers(0, d, 60)]))
    X, Y, Gn, Go, b = (_matrix(n, d, ld, k, sd if k < 2 else torch.float32) for k in range(5))
    h = torch.rand(ld, device=DEV)
    x, y, gn, go, bb, hh = (_cols(t, cols) for t in (X, Y, Gn, Go, b, h[None]))
    S = amax(x, y, gn, go)
    Z = X.clone()
    ctx.gossip_accel(Z, K, eta)
    assert rel_err(_cols(Z, cols), OG.accelerated_gossip(x, W, K, eta), S) < tol
    for variant, code in (("atc", D.DETAG_VARIANT_ATC), ("alg2", D.DETAG_VARIANT_ALG2)):
        Xs, Ys = X.clone(), Y.clone()
        ctx.step(Xs, Ys, Gn, Go, alpha, K, eta, code)
        xr, yr = OG.detag_step(x, y, gn, go, W, alpha, K, eta, variant)
        assert rel_err(_cols(Xs, cols), xr, S) < tol and rel_err(_cols(Ys, cols), yr, S) < tol, variant
    Xs, Ys, G = X.clone(), Y.clone(), Go.clone()
    ctx.step_quadratic(Xs, Ys, G, h, b, alpha, K, sigma=sigma, seed=seed, step=2, eta=eta)
    g = OO.grad_quadratic_diag(x, hh[0], bb, ON.normal_noise(seed, 2, n, cols), sigma)
    xr, yr = OG.detag_step(x, y, g, go, W, alpha, K, eta)
    assert rel_err(_cols(G, cols), g, amax(g)) < TOL_F32
    assert rel_err(_cols(Xs, cols), xr, S) < tol and rel_err(_cols(Ys, cols), yr, S) < tol
    Xp = X.clone()
    ctx.dpsgd_step(Xp, Gn, alpha)
    assert rel_err(_cols(Xp, cols), OG.dpsgd_step(x, gn, W, alpha), S) < tol
    for t in (Z, Xs, Ys, G, Xp):
        assert torch.equal(t[:, d:], torch.full_like(t[:, d:], SENTINEL))   # the padding is never written
    ctx.close()


@pytest.mark.parametrize("n,kind", [(12, "complete"), (64, "exponential"), (100, "complete"), (257, "rr"), (513, "asym"),
                                    (1000, "asym"), (1024, "asym"), (1025, "asym")])
@pytest.mark.parametrize("big,dtype,K", [(False, "f32", 3), (False, "bf16", 2), (True, "f32", 4), (True, "bf16", 3)])
def test_rounds_on_chip_beyond_the_family(n, kind, big, dtype, K):
    """More than 256 workers or 8 neighbours on the automatic path (1025 workers: one launch per round): the oracle, and
    the path with one launch per round."""
    d = (1 << 19) // n * 4 + 5 if big else 333
    ld = d + 3
    bf = dtype == "bf16"
    sd, tol = (torch.bfloat16, TOL_BF16) if bf else (torch.float32, TOL_F32)
    if kind == "complete":
        e = np.array([(i, j) for i in range(n) for j in range(i + 1, n)])
    elif kind == "exponential":
        e = np.array(sorted({tuple(sorted((i, (i + s) % n))) for i in range(n) for s in (1, 2, 4, 8, 16, 32)}))
    elif kind == "rr":
        e = _graph(kind, n)
    if kind == "asym":  # three neighbours with weights of their own (and no eigenvalues to compute at creation)
        W = sum(w * np.roll(np.eye(n), s, axis=1) for w, s in ((0.5, 0), (0.25, 1), (0.15, 7), (0.1, 200)))
        topo = D.Topology.from_dense(W)
    else:
        W, topo = OT.mixing_matrix(n, e, "metropolis"), D.Topology.from_edges(e, D.DETAG_W_METROPOLIS)
    ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if bf else D.DETAG_F32)
    assert ctx.kernel() == D.DETAG_KERNEL_PER_ROUND and not ctx.has_fused()
    eta, alpha = 0.35, 0.2
    rng = np.random.default_rng(5)
    cols = np.unique(np.concatenate([np.arange(20), np.arange(d - 40, d), rng.integers(0, d, 20)]))
    X, Y, Gn, Go = (_matrix(n, d, ld, k, sd if k < 2 else torch.float32) for k in range(4))
    x, y, gn, go = (_cols(t, cols) for t in (X, Y, Gn, Go))
    S = amax(x, y, gn, go)
    for path in (D.DETAG_PATH_AUTO, D.DETAG_PATH_PER_ROUND):
        ctx.set_path(path)
        Z, Xp = X.clone(), X.clone()
        ctx.gossip_accel(Z, K, eta)
        assert rel_err(_cols(Z, cols), OG.accelerated_gossip(x, W, K, eta), S) < tol
        ctx.dpsgd_step(Xp, Gn, alpha)
        assert rel_err(_cols(Xp, cols), OG.dpsgd_step(x, gn, W, alpha), S) < tol
        for variant, code in (("atc", D.DETAG_VARIANT_ATC), ("alg2", D.DETAG_VARIANT_ALG2)):
            Xs, Ys = X.clone(), Y.clone()
            ctx.step(Xs, Ys, Gn, Go, alpha, K, eta, code)
            xr, yr = OG.detag_step(x, y, gn, go, W, alpha, K, eta, variant)
            assert rel_err(_cols(Xs, cols), xr, S) < tol and rel_err(_cols(Ys, cols), yr, S) < tol, (path, variant)
            assert torch.equal(Xs[:, d:], torch.full_like(Xs[:, d:], SENTINEL))
    ctx.close()


@pytest.mark.parametrize("n,kind", [(7, "ring"), (12, "irregular"), (31, "irregular"), (100, "irregular"), (64, "rr"), (257, "irregular")])
@pytest.mark.parametrize("big", [False, True])
def test_an_infinity_reaches_only_its_neighbours(n, kind, big):
    """Padding of the neighbour tables must not name anybody else's row: after one round the columns of every worker that
    neither holds the infinity nor has it as a neighbour are what they are without it."""
    d = (1 << 19) // n * 4 + 8 if big else 200
    e = _graph(kind, n)
    W = OT.mixing_matrix(n, e, "metropolis")
    ctx = D.detag_create(D.Topology.from_edges(e, D.DETAG_W_METROPOLIS), n, d)
    Z = _matrix(n, d, d, 1)
    clean = Z.clone()
    ctx.gossip_accel(clean, 1, 0.3)
    for worker in (0, n // 2, int(np.argmax((W != 0).sum(1)))):
        bad = Z.clone()
        bad[worker, 5] = float("inf")
        ctx.gossip_accel(bad, 1, 0.3)
        untouched = torch.as_tensor(np.flatnonzero(W[worker] == 0), device=DEV)
        assert torch.equal(bad[untouched], clean[untouched])
        bad[:, 5] = clean[:, 5]
        assert torch.equal(bad, clean)


@pytest.mark.parametrize("n,kind", [(1, "alone"), (2, "ring"), (7, "ring"), (12, "rr"), (31, "irregular"), (64, "rr8"), (100, "irregular"),
                                    (129, "rr"), (256, "irregular"), (256, "rr"), (300, "rr"), (512, "asym")])
@pytest.mark.parametrize("big,dtype", [(False, "f32"), (True, "f32"), (False, "bf16")])
def test_dpsgd_is_the_step_of_one_launch_per_round(n, kind, big, dtype):
    """The same sum in the same order with the same roundings, so the same bits: workers close to each other (where a sum
    of neighbours instead of differences loses digits), values whose sum overflows, infinities."""
    d = min(1 << 17, (1 << 19) // n * 4) + 5 if big else 333
    sd = torch.bfloat16 if dtype == "bf16" else torch.float32
    if kind == "alone":
        topo = D.Topology.from_dense(np.ones((1, 1)))
    elif kind == "asym":
        topo = D.Topology.from_dense(sum(w * np.roll(np.eye(n), s, axis=1) for w, s in ((0.5, 0), (0.25, 1), (0.15, 7), (0.1, 200))))
    else:
        topo = D.Topology.ring() if kind == "ring" else D.Topology.from_edges(_graph(kind, n), D.DETAG_W_METROPOLIS)
    ctx = D.detag_create(topo, n, d, d, D.DETAG_BF16 if dtype == "bf16" else D.DETAG_F32)
    G = _matrix(n, d, d, 2)
    X = (1.0 + 1e-3 * _matrix(n, d, d, 1)).to(sd)
    X[:, 7] *= 1.5e38
    X[n // 2, 11] = float("inf")
    out = []
    for path in (D.DETAG_PATH_AUTO, D.DETAG_PATH_PER_ROUND):
        ctx.set_path(path)
        out.append(X.clone())
        ctx.dpsgd_step(out[-1], G, 0.1)
    got, want = out
    assert torch.isfinite(want[:, 7]).all()
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.nan_to_num(1.0), want.nan_to_num(1.0))
    ctx.close()


def test_more_elements_than_a_launch_has_threads_for():
    """2^36 elements and some in one bf16 matrix (137 GB) of more workers than the family serves: a lane has 16 of them, a
    grid counts 2^32 threads."""
    n, K, eta = 512, 2, 0.3
    d = (1 << 27) + 40
    if torch.cuda.mem_get_info()[0] < 2 * n * d + (8 << 30):
        pytest.skip("needs 146 GB of free GPU memory")
    W = sum(w * np.roll(np.eye(n), s, axis=1) for w, s in ((0.5, 0), (0.25, 1), (0.15, 7), (0.1, 200)))
    ctx = D.detag_create(D.Topology.from_dense(W), n, d, d, D.DETAG_BF16)
    Z = torch.zeros((n, d), dtype=torch.bfloat16, device=DEV)
    cols = np.concatenate([np.arange(40), (1 << 26) + np.arange(-20, 20), np.arange(d - 60, d)])
    at = torch.as_tensor(cols, device=DEV)
    Z[:, at] = _matrix(n, len(cols), len(cols), 1).to(torch.bfloat16)
    z = _cols(Z, cols)
    ctx.gossip_accel(Z, K, eta)
    got = _cols(Z, cols)
    Z[:, at] = 0
    rest = max(Z[i].abs().max().item() for i in range(0, n, 73))
    del Z
    torch.cuda.empty_cache()
    ctx.close()
    assert rel_err(got, OG.accelerated_gossip(z, W, K, eta), amax(z)) < TOL_BF16 and rest == 0


@pytest.mark.parametrize("n,kind", [(7, "ring"), (13, "irregular"), (64, "rr8"), (100, "irregular"), (200, "rr"), (300, "rr")])
@pytest.mark.parametrize("big,dtype", [(False, "f32"), (True, "f32"), (False, "bf16"), (True, "bf16")])
def test_where_the_rows_end_in_a_tile(n, kind, big, dtype):
    """Columns are independent: whatever number of columns the last tile has, each comes out as in a wider matrix, bit for
    bit, and nothing is written behind them."""
    base = (1 << 19) // n * 4 + 256 if big else 256
    ld, K, eta, alpha, sigma = base + 256, 3, 0.35, 0.2, 0.1
    sd = torch.bfloat16 if dtype == "bf16" else torch.float32
    topo = D.Topology.ring() if kind == "ring" else D.Topology.from_edges(_graph(kind, n), D.DETAG_W_METROPOLIS)
    state = [_matrix(n, ld, ld, k, sd if k < 2 else torch.float32) for k in range(5)]
    h = torch.rand(ld, device=DEV)

    def run(d):
        ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if dtype == "bf16" else D.DETAG_F32)
        X, Y, Gn, Go, b = state
        out = [X.clone() for _ in range(8)]
        ctx.gossip_accel(out[0], K, eta)
        ctx.dpsgd_step(out[1], Gn, alpha)
        out[3].copy_(Y), out[5].copy_(Y), out[7].copy_(Y)
        ctx.step(out[2], out[3], Gn, Go, alpha, K, eta, D.DETAG_VARIANT_ATC)
        ctx.step(out[4], out[5], Gn, Go, alpha, K, eta, D.DETAG_VARIANT_ALG2)
        G = Go.clone()
        if n <= 256:
            ctx.step_quadratic(out[6], out[7], G, h, b, alpha, K, sigma=sigma, seed=3, step=1, eta=eta)
        ctx.close()
        return out + [G]

    whole = run(base + 256)
    for more in (0, 1, 2, 3, 4, 5, 6, 7, 31, 33, 62, 130, 255):
        d = base + more
        before = [state[0], state[0], state[0], state[1], state[0], state[1], state[0], state[1], state[3]]
        for got, want, old in zip(run(d), whole, before):
            assert torch.equal(got[:, :d], want[:, :d]) and torch.equal(got[:, d:], old[:, d:]), more


def _weights(kind, n):
    if kind == "asym":
        return D.Topology.from_dense(sum(w * np.roll(np.eye(n), s, axis=1) for w, s in ((0.5, 0), (0.25, 1), (0.15, 7), (0.1, 200))))
    if kind == "star":
        return D.Topology.from_edges(np.array([(0, j) for j in range(1, n)]), D.DETAG_W_METROPOLIS)
    if kind == "complete":
        return D.Topology.from_edges(np.array([(i, j) for i in range(n) for j in range(i + 1, n)]), D.DETAG_W_METROPOLIS)
    return D.Topology.from_edges(_graph(kind, n), D.DETAG_W_METROPOLIS)


@pytest.mark.parametrize("n,kind,d,op,K,on_chip", [
    (257, "rr", 333, "gossip", 1, True), (257, "rr", 333, "step", 2, True), (257, "rr", 333, "dpsgd", 1, True),
    (64, "complete", 333, "step", 3, True), (100, "complete", 5000, "gossip", 1, True),
    (512, "asym", 333, "gossip", 1, True), (512, "asym", 333, "dpsgd", 1, True), (513, "asym", 333, "dpsgd", 1, False),
    (513, "asym", 333, "gossip", 2, False), (513, "asym", 333, "step", 2, False), (513, "asym", 333, "step", 3, True),
    (1000, "asym", 524, "gossip", 2, False), (1000, "asym", 525, "gossip", 2, True),
    (1024, "asym", 333, "step", 3, True), (1025, "asym", 333, "step", 3, False), (1025, "asym", 5000, "gossip", 3, False),
    (256, "star", 131_000, "step", 3, True), (257, "star", 131_000, "step", 3, False), (257, "star", 130_000, "step", 3, True)])
def test_route_of_contexts_that_report_one_launch_per_round(n, kind, d, op, K, on_chip):
    """On the automatic path such a context still runs on chip where that is the faster way.  Seen from outside: under
    capture, on a context whose scratch has never been allocated, only the on-chip route is recorded."""
    ctx = D.detag_create(_weights(kind, n), n, d, d)
    assert ctx.kernel() == D.DETAG_KERNEL_PER_ROUND
    X, Y, Gn, Go = (_matrix(n, d, d, k) for k in range(4))
    call = {"gossip": lambda x, y: ctx.gossip_accel(x, K, 0.3), "step": lambda x, y: ctx.step(x, y, Gn, Go, 0.1, K, 0.3),
            "dpsgd": lambda x, y: ctx.dpsgd_step(x, Gn, 0.1)}[op]
    Xr, Yr, refused = X.clone(), Y.clone(), None
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            Go.add_(0.0)                                # so that the recording holds some node
            try:
                call(Xr, Yr)
            except D.DetagError as e:
                refused = e
    assert (refused is None) == on_chip
    if on_chip:
        graph.replay()
    else:
        assert refused.status == D.DETAG_EINVAL and "detag_reserve_gossip" in refused.message
        torch.cuda.synchronize()
        assert torch.equal(Xr, X) and torch.equal(Yr, Y)
        call(Xr, Yr)
    call(X, Y)
    torch.cuda.synchronize()
    assert torch.equal(Xr, X) and torch.equal(Yr, Y)
    ctx.close()


@pytest.mark.parametrize("n,degree", [(257, 2), (257, 4), (300, 8), (512, 5), (513, 3), (1024, 4)])
@pytest.mark.parametrize("dtype,K", [("f32", 3), ("bf16", 2)])
def test_one_weight_beyond_256_workers(n, degree, dtype, K):
    """Lists of 16-bit offsets in registers, full and padded: every call against the oracle, and the same bits as one launch
    per round from the D-PSGD step (not from 513 workers on, which has no on-chip form)."""
    d = (1 << 19) // n * 4 + 5
    ld = d + 3
    bf = dtype == "bf16"
    sd, tol = (torch.bfloat16, TOL_BF16) if bf else (torch.float32, TOL_F32)
    w = 0.7 / degree
    W = 0.3 * np.eye(n) + sum(w * np.roll(np.eye(n), s, axis=1) for s in (1, n - 1, 7, 200, 97, 31, n - 60, 128)[:degree])
    ctx = D.detag_create(D.Topology.from_dense(W), n, d, ld, D.DETAG_BF16 if bf else D.DETAG_F32)
    eta, alpha = 0.35, 0.2
    cols = np.unique(np.concatenate([np.arange(40), np.arange(d - 70, d)]))
    X, Y, Gn, Go = (_matrix(n, d, ld, k, sd if k < 2 else torch.float32) for k in range(4))
    x, y, gn, go = (_cols(t, cols) for t in (X, Y, Gn, Go))
    S = amax(x, y, gn, go)
    Z, Xp = X.clone(), X.clone()
    ctx.gossip_accel(Z, K, eta)
    assert rel_err(_cols(Z, cols), OG.accelerated_gossip(x, W, K, eta), S) < tol
    ctx.dpsgd_step(Xp, Gn, alpha)
    assert rel_err(_cols(Xp, cols), OG.dpsgd_step(x, gn, W, alpha), S) < tol
    for variant, code in (("atc", D.DETAG_VARIANT_ATC), ("alg2", D.DETAG_VARIANT_ALG2)):
        Xs, Ys = X.clone(), Y.clone()
        ctx.step(Xs, Ys, Gn, Go, alpha, K, eta, code)
        xr, yr = OG.detag_step(x, y, gn, go, W, alpha, K, eta, variant)
        assert rel_err(_cols(Xs, cols), xr, S) < tol and rel_err(_cols(Ys, cols), yr, S) < tol, variant
        for t in (Z, Xp, Xs, Ys):
            assert torch.equal(t[:, d:], torch.full_like(t[:, d:], SENTINEL))
    ctx.set_path(D.DETAG_PATH_PER_ROUND)
    Xr = X.clone()
    ctx.dpsgd_step(Xr, Gn, alpha)
    assert torch.equal(Xp, Xr)
    ctx.close()


@pytest.mark.parametrize("n,kind", [(16, "rr"), (24, "rr8"), (100, "ring"), (64, "rr"), (64, "rr8"), (64, "irregular"),
                                    (128, "rr"), (128, "rr8"), (300, "irregular")])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_how_rows_are_requested_does_not_change_the_bits(n, kind, dtype):
    """How many rows' loads are in flight depends on the form, the state type, K and the threads of a block: the first columns
    of a matrix that takes four rows per lane, and the same columns alone, which take one or two."""
    topo = D.Topology.ring() if kind == "ring" else D.Topology.from_edges(_graph(kind, n), D.DETAG_W_METROPOLIS)
    wide, narrow = (1 << 19) // n * 4 + 1003, 1001
    ld, sd = wide + 2, torch.bfloat16 if dtype == "bf16" else torch.float32
    code = D.DETAG_BF16 if dtype == "bf16" else D.DETAG_F32
    X, Y, Gn, Go = (_matrix(n, wide, ld, k, sd if k < 2 else torch.float32) for k in range(4))
    for K in (1, 2, 3, 4, 5, 6):
        out = []
        for d in (wide, narrow):
            ctx = D.detag_create(topo, n, d, ld, code)
            z = X.clone()
            ctx.gossip_accel(z, K, 0.35)
            got = [z]
            for variant in (D.DETAG_VARIANT_ATC, D.DETAG_VARIANT_ALG2):
                x, y = X.clone(), Y.clone()
                ctx.step(x, y, Gn, Go, 0.2, K, 0.35, variant)
                got += [x, y]
            ctx.close()
            for t, before in zip(got, (X, X, Y, X, Y)):
                assert torch.equal(t[:, d:], before[:, d:])
            out.append([t[:, :narrow] for t in got])
        for k, (a, b) in enumerate(zip(*out)):
            assert torch.equal(a, b), (K, k)
