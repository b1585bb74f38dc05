"""Parity of DETAG_PATH_DENSE -- the K rounds of Algorithm 3 as one product with the matrix polynomial p_K(W^T) on
the matrix cores -- against the oracle, which takes the K rounds one after the other."""
import numpy as np
import pytest
import torch

import paper_2006_08085_amd as D
from oracle import gossip as OG
from oracle import objectives as OO
from oracle import topology as OT
from tests.util import TOL_BF16, TOL_F32, amax, rel_err
from workloads import generate as gen

pytestmark = pytest.mark.gpu

from tests.gpu_util import DEV, SENTINEL, _built, padding_ok, to_dev, to_host  # noqa: F401,E402


def _graph(n, graph):
    if graph == "asym":
        W = 0.5 * np.eye(n) + 0.5 * np.roll(np.eye(n), 1, axis=1)
        return D.Topology.from_dense(W), W, 0.3
    if graph == "ring":
        W = OT.mixing_matrix(n, gen.edges_ring(n))
        return D.Topology.ring(), W, (OT.eta_from_lambda(OT.spectrum(W)[2]) if n > 1 else 0.0)
    if graph == "torus88":
        W = OT.mixing_matrix(64, gen.edges_torus(8, 8))
        return D.Topology.torus(8, 8), W, OT.eta_from_lambda(OT.spectrum(W)[2])
    if graph == "star":                                         # a hub with n-1 neighbours: no on-chip round kernel
        e = np.array([(0, j) for j in range(1, n)])
    else:
        e = gen.edges_random_regular(n, 4, seed=n)
    W = OT.mixing_matrix(n, e, "metropolis")
    return D.Topology.from_edges(e, D.DETAG_W_METROPOLIS), W, OT.eta_from_lambda(OT.spectrum(W)[2])


CASES = [(5, "asym"), (1, "ring"), (2, "ring"), (17, "ring"), (33, "ring"), (64, "torus88"), (20, "star"), (100, "rr"),
         (130, "rr"), (256, "rr")]


@pytest.mark.parametrize("n,graph", CASES)
@pytest.mark.parametrize("K", [1, 5, 16])
def test_dense_gossip_and_step_f32(n, graph, K):
    d, ld = 150, 160               # two full 64-column tiles and a ragged one
    topo, W, eta = _graph(n, graph)
    ctx = D.detag_create(topo, n, d, ld)
    ctx.set_path(D.DETAG_PATH_DENSE)
    alpha = 0.05
    Z = gen.state(n, d, seed=K)
    Zd = to_dev(Z, ld)
    ctx.gossip_accel(Zd, K, eta)
    assert rel_err(to_host(Zd, d), OG.accelerated_gossip(Z, W, K, eta), amax(Z)) < TOL_F32
    assert padding_ok(Zd, d)
    X, Y, Gn, Go = (gen.state(n, d, s) for s in (1, 2, 3, 4))
    for variant, vcode in (("atc", D.DETAG_VARIANT_ATC), ("alg2", D.DETAG_VARIANT_ALG2)):
        Xd, Yd, Gnd, God = (to_dev(a, ld) for a in (X, Y, Gn, Go))
        ctx.step(Xd, Yd, Gnd, God, alpha, K, eta, vcode)
        Xr, Yr = OG.detag_step(X, Y, Gn, Go, W, alpha, K, eta, variant)
        S = amax(X, Y, Gn, Go)
        assert rel_err(to_host(Xd, d), Xr, S) < TOL_F32
        assert rel_err(to_host(Yd, d), Yr, S) < TOL_F32
        assert padding_ok(Xd, d) and padding_ok(Yd, d)
        assert np.array_equal(to_host(Gnd, d), Gn.astype(np.float32)) and np.array_equal(to_host(God, d), Go.astype(np.float32))


@pytest.mark.parametrize("n,graph", [(12, "rr"), (64, "torus88"), (256, "rr")])
@pytest.mark.parametrize("variant", ["atc", "alg2"])
def test_dense_step_bf16_state(n, graph, variant):
    d, ld, K, alpha = 200, 256, 8, 0.05
    topo, W, eta = _graph(n, graph)
    ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16)
    ctx.set_path(D.DETAG_PATH_DENSE)
    X, Y = (OO.round_bf16(gen.state(n, d, s)) for s in (1, 2))
    Gn, Go = (gen.state(n, d, s) for s in (3, 4))
    Xd, Yd = (to_dev(a, ld, torch.bfloat16) for a in (X, Y))
    Gnd, God = (to_dev(a, ld) for a in (Gn, Go))
    ctx.step(Xd, Yd, Gnd, God, alpha, K, eta, D.DETAG_VARIANT_ATC if variant == "atc" else D.DETAG_VARIANT_ALG2)
    Xr, Yr = OG.detag_step(X, Y, Gn, Go, W, alpha, K, eta, variant)
    S = amax(X, Y, Gn, Go)
    assert rel_err(to_host(Xd, d), Xr, S) < TOL_BF16
    assert rel_err(to_host(Yd, d), Yr, S) < TOL_BF16
    assert padding_ok(Xd, d) and padding_ok(Yd, d)
    Zd = to_dev(X, ld, torch.bfloat16)
    ctx.gossip_accel(Zd, K, eta)
    assert rel_err(to_host(Zd, d), OG.accelerated_gossip(X, W, K, eta), amax(X)) < TOL_BF16


def test_dense_long_K_near_one_eta():
    """The slack ring of the spectral-gap sweep (kappa = 0.01) at its phase length: the polynomial is
    evaluated in fp64 on the host, so the error does not grow with K as it does round by round."""
    n, d, ld = 16, 300, 320
    W = OT.slack(OT.mixing_matrix(n, gen.edges_ring(n)), 0.01)
    ctx = D.detag_create(D.Topology.ring(kappa=0.01), n, d, ld)
    ctx.set_path(D.DETAG_PATH_DENSE)
    eta = OT.eta_from_lambda(OT.spectrum(W)[2])
    K = ctx.phase_length()
    assert K > 40 and eta > 0.9
    Z = gen.state(n, d, seed=3)
    Zd = to_dev(Z, ld)
    ctx.gossip_accel(Zd, K)
    assert np.abs(to_host(Zd, d) - OG.accelerated_gossip(Z, W, K, eta)).max() < 2e-6 * amax(Z)


def test_dense_polynomial_cache_and_mean():
    """More (K, eta) pairs than the context keeps polynomials for, then the first again; equal values across the
    workers stay put and the worker mean is kept."""
    n, d, ld = 100, 130, 160
    topo, W, eta = _graph(n, "rr")
    ctx = D.detag_create(topo, n, d, ld)
    ctx.set_path(D.DETAG_PATH_DENSE)
    Z = gen.state(n, d, seed=9)
    for K, e in [(3, eta), (4, eta), (5, eta), (3, 0.0), (6, eta), (7, 0.1), (3, eta)]:
        Zd = to_dev(Z, ld)
        ctx.gossip_accel(Zd, K, e)
        out = to_host(Zd, d)
        assert rel_err(out, OG.accelerated_gossip(Z, W, K, e), amax(Z)) < TOL_F32
        assert np.abs(out.mean(0) - Z.mean(0)).max() < 2e-6 * amax(Z)
    C = np.tile(gen.state(1, d, seed=2), (n, 1))
    Cd = to_dev(C, ld)
    ctx.gossip_accel(Cd, 9)
    assert np.abs(to_host(Cd, d) - C).max() < 1e-6 * amax(C)


def test_dense_path_is_refused_above_256_workers():
    ctx = D.detag_create(D.Topology.ring(), 300, 64, 64)
    with pytest.raises(D.DetagError) as ei:
        ctx.set_path(D.DETAG_PATH_DENSE)
    assert ei.value.status == D.DETAG_EUNSUPPORTED


def test_config5_shape_bf16_short_run_dense():
    """The 256-worker workload (random 4-regular graph, Metropolis weights, bf16 X/Y, K=16) on the dense path,
    d reduced to 4,096 + 37 columns and 3 steps; the oracle rounds X and Y to bf16 after every step."""
    from workloads import CONFIGS
    cfg = CONFIGS[5]
    n, K, alpha = cfg.n, cfg.K, cfg.lr
    d, T = 4096 + 37, 3
    ld = D.padded_ld(d)
    e = gen.edges_random_regular(n, 4, seed=cfg.seed)
    W = OT.mixing_matrix(n, e, "metropolis")
    ctx = D.detag_create(D.Topology.from_edges(e, D.DETAG_W_METROPOLIS), n, d, ld, D.DETAG_BF16)
    ctx.set_path(D.DETAG_PATH_DENSE)
    eta = ctx.spectrum()["eta"]
    h, b = gen.quadratic_problem(n, d, seed=cfg.seed, b_std=cfg.extra["b_std"])
    hd = torch.zeros(ld); hd[:d] = torch.from_numpy(h); hd = hd.to(DEV)
    bd = to_dev(b, ld)
    Xd, Yd = (D.new_matrix(n, d, ld, dtype=torch.bfloat16) for _ in range(2))
    Ga, Gb = D.new_matrix(n, d, ld), D.new_matrix(n, d, ld)
    X = np.zeros((n, d)); Y = np.zeros((n, d)); Gold = np.zeros((n, d))
    for t in range(T):
        ctx.grad_quadratic_diag(Xd, hd, bd, Ga)
        ctx.step(Xd, Yd, Ga, Gb, alpha, K)
        Ga, Gb = Gb, Ga
        Gnew = OO.grad_quadratic_diag(X, h, b)
        Xn, Yn = OG.detag_step(X, Y, Gnew, Gold, W, alpha, K, eta)
        if t == 0:
            S1 = amax(X, Y, Gnew, Gold)
            assert rel_err(to_host(Xd, d), Xn, S1) < TOL_BF16
            assert rel_err(to_host(Yd, d), Yn, S1) < TOL_BF16
        X, Y, Gold = OO.round_bf16(Xn).astype(np.float64), OO.round_bf16(Yn).astype(np.float64), Gnew
    S = amax(X, Y, Gold)
    assert rel_err(to_host(Xd, d), X, S, floor=1.0) < TOL_BF16
    assert rel_err(to_host(Yd, d), Y, S, floor=1.0) < TOL_BF16


@pytest.mark.parametrize("n", [12, 17, 33, 64, 65, 100, 128, 129, 200, 256])
@pytest.mark.parametrize("d,ld", [(64, 64), (65, 65), (129, 160), (701, 704), (1025, 1025), (40001, 40001), (33000, 33024)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_resident_kernel_gives_the_bits_of_the_general_one(n, d, ld, dtype):
    """The kernel that holds P in registers against the general kernel, which serves contexts of fewer than 64
    columns: the same columns in slices of 63, around the edges of tiles of every width (64 to 512) and of a block's walk."""
    topo, W, eta = _graph(n, "rr")
    bf = dtype == "bf16"
    state = (lambda t: t.bfloat16()) if bf else (lambda t: t)
    g = torch.Generator(device=DEV).manual_seed(n + d)
    normal = lambda: torch.randn(n, ld, device=DEV, generator=g)  # noqa: E731
    X, Y, Gn, Go = state(normal()), state(normal()), normal(), normal()
    for t in (X, Y, Gn, Go):
        t[:, d:] = SENTINEL
    edges = sorted({0, d - 63} | {min(max(0, e - 31), d - 63) for e in (64, 128, 256, 512, 1024, 16384, 32768) if e < d + 31})

    def call(ctx, mode, x, y, gn, go):
        if mode == 0:
            ctx.gossip_accel(x, 3, eta)
        else:
            ctx.step(x, y, gn, go, 0.05, 3, eta, D.DETAG_VARIANT_ATC if mode == 1 else D.DETAG_VARIANT_ALG2)

    code = D.DETAG_BF16 if bf else D.DETAG_F32
    whole, narrow = D.detag_create(topo, n, d, ld, code), D.detag_create(topo, n, 63, ld, code)
    for ctx in (whole, narrow):
        ctx.set_path(D.DETAG_PATH_DENSE)
    for mode in (0, 1, 2):
        x, y = X.clone(), Y.clone()
        call(whole, mode, x, y, Gn, Go)
        assert padding_ok(x, d) and padding_ok(y, d)
        for c in edges:
            xs, ys = X.clone(), Y.clone()
            call(narrow, mode, xs[:, c:], ys[:, c:], Gn[:, c:], Go[:, c:])
            assert torch.equal(xs[:, c:c + 63], x[:, c:c + 63]) and torch.equal(ys[:, c:c + 63], y[:, c:c + 63]), (mode, c)


@pytest.mark.parametrize("n,d", [(20, 63), (20, 40000), (100, 700), (256, 700)])   # the general kernel, and P in registers
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_what_is_not_finite_stays_in_its_column(n, d, dtype):
    """An infinity or a NaN of one worker leaves nothing finite in its column of what depends on it, and the bits of every other
    column as they are without it."""
    topo, _, eta = _graph(n, "rr")
    ctx = D.detag_create(topo, n, d, d, D.DETAG_BF16 if dtype == "bf16" else D.DETAG_F32)
    ctx.set_path(D.DETAG_PATH_DENSE)
    g = torch.Generator(device=DEV).manual_seed(d)
    clean = [torch.randn(n, d, device=DEV, generator=g) for _ in range(4)]
    clean[:2] = [t.bfloat16() if dtype == "bf16" else t for t in clean[:2]]
    bad = [t.clone() for t in clean]
    bad[0][0, 5], bad[0][n - 1, 11], bad[1][n // 2, 20], bad[2][n - 1, 33] = float("inf"), -float("inf"), float("inf"), float("nan")
    for mode in (0, 1, 2):
        outs = []
        for x, y, gn, go in ([t.clone() for t in clean], [t.clone() for t in bad]):
            if mode == 0:
                ctx.gossip_accel(x, 3, eta)
                ctx.gossip_accel(y, 3, eta)
            else:
                ctx.step(x, y, gn, go, 0.05, 3, eta, D.DETAG_VARIANT_ATC if mode == 1 else D.DETAG_VARIANT_ALG2)
            outs.append((x, y))
        for k, spoiled in enumerate(([5, 11] if mode == 0 else [5, 11, 20], [20] if mode == 0 else [20, 33])):
            want, got = outs[0][k], outs[1][k]
            rows = torch.isfinite(got[:, spoiled]).any(0)
            if mode == 2 and k == 1:           # the gradients enter behind the rounds: one worker's entry
                assert not torch.isfinite(got[n - 1, 33]) and torch.equal(got[:n - 1, 33], want[:n - 1, 33])
                rows = rows[:1]
            assert not rows.any(), (mode, k, rows)
            others = [c for c in range(d) if c not in spoiled]
            assert torch.equal(got[:, others], want[:, others]), (mode, k)
