"""The calls a user of this library makes, as measurable cases.

listed() holds twelve of them, draw() gives more from the same ranges.  Every
case is one training iteration (or one diagnostic) on n simulated workers with
d parameters each, through the Python binding of the C entry points:

  quad     detag_step_quadratic: gradient query of the diagonal quadratic and one DeTAG phase in one call
  phase    detag_grad_quadratic_diag + detag_step, any graph, either form of the phase update
  dense    the same two calls on the matrix-core path
  dpsgd    detag_grad_quadratic_diag + detag_dpsgd_step, the D-PSGD baseline
  byphase  one phase of Algorithm 2 iteration by iteration (gossip rounds beside gradient queries, phase end)
  defacto  gradient query, exact average consensus, end of a round of Algorithm 1
  diag     worker mean and consensus distance
  lstsq    least-squares gradient + detag_step
  softmax  softmax-regression gradient on a bf16 mini-batch + detag_step

exact() restates each of them in 64 bits with plain torch.
"""
import math

import numpy as np
import torch

import paper_2006_08085_amd as D
from paper_2006_08085_amd import algorithms

DEV = "cuda"
DEFAULTS = dict(dtype="f32", sigma=0.1, variant="atc", tight=False, rows_h=False, K=8)


def _case(name, kind, graph, n, d, **kw):
    return dict(name=name, kind=kind, graph=graph, n=n, d=d, **dict(DEFAULTS, **kw))


def listed():
    return [
        # the smallest workload: 8 workers on a ring, least squares (64 x 1024 per worker), four gossip rounds
        _case("lstsq_ring8", "lstsq", "ring", 8, 1024, K=4, m=64),
        # ResNet-20-sized models of 16 workers on a ring, noisy quadratic: the spectral-gap experiment's shape
        _case("quad_ring16", "quad", "ring", 16, 272_474, K=6),
        # label-sorted CIFAR-10-shaped shards: 32 workers, softmax regression, batch of 128
        _case("softmax_ring32", "softmax", "ring", 32, 30_730, K=8, F=3072, C=10, S=1562, B=128),
        # ResNet-18-sized models of 64 workers on a torus: the headline workload
        _case("quad_torus64", "quad", "torus", 64, 11_173_962, K=8),
        # 256 workers on a random regular graph, bf16 state
        _case("quad_regular256_bf16", "quad", "regular4", 256, 1_048_576, K=16, dtype="bf16", sigma=0.0),
        # a user's own irregular network (Metropolis weights), pitch = d, Algorithm 2 as printed, one curvature per worker
        _case("alg2_irregular100_odd", "phase", "irregular", 100, 300_007, K=5, variant="alg2", tight=True, rows_h=True),
        # more workers than the on-chip kernels hold
        _case("phase_regular300", "phase", "regular4", 300, 100_000, K=8),
        # the polynomial form of the 256-worker phase
        _case("dense_regular256_bf16", "dense", "regular4", 256, 1_048_576, K=16, dtype="bf16", sigma=0.0),
        # the D-PSGD baseline on a mid-sized model, a network of its own, ragged width
        _case("dpsgd_irregular48", "dpsgd", "irregular", 48, 1_000_003),
        # Algorithm 2 iteration by iteration, gossip on a stream of its own
        _case("byphase_ring16", "byphase", "ring", 16, 272_474, K=6),
        # Algorithm 1: one round's averaging on a random regular graph of 64 workers
        _case("defacto_regular64", "defacto", "regular4", 64, 272_474, sigma=0.1),
        # what a run logs: worker mean and consensus distance of the headline state
        _case("diag_64", "diag", "torus", 64, 11_173_962),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, sizes log-uniform from the smallest to a good part of the largest listed."""
    kind = rng.choice(["quad", "quad", "quad", "phase", "phase", "dense", "dpsgd", "byphase", "defacto", "diag", "lstsq",
                       "softmax"])
    graph = rng.choice(["ring", "torus", "regular4", "irregular"])
    if graph == "torus":
        n = rng.choice([16, 32, 64, 36])
    elif graph == "ring":
        n = rng.choice([4, 8, 12, 16, 24, 32, 48, 64, 7, 20, 100])
    else:
        n = _log_int(rng, 12, 256)
    top = 3e8 if kind in ("quad", "diag") else 1e8
    if kind == "phase" and rng.random() < 0.4:  # networks whose rounds run one launch each
        graph, n, top = rng.choice([("regular4", rng.randint(257, 400)), ("exponential", rng.choice([32, 50, 64, 128]))]) + (2e7,)
    d = _log_int(rng, 1000, top / n)
    kw = dict(K=rng.randint(1, 16), dtype=rng.choice(["f32", "f32", "bf16"]), sigma=rng.choice([0.0, 0.1]),
              tight=rng.random() < 0.25, rows_h=rng.random() < 0.25)
    if kind == "phase":
        kw["variant"] = rng.choice(["atc", "alg2"])
    if kind in ("byphase", "lstsq", "softmax"):
        graph, n = "ring", rng.choice([4, 8, 16, 32])
        kw.update(dtype="f32", K=rng.randint(2, 8), rows_h=False)
    if kind == "byphase":
        d = _log_int(rng, 1000, 1_000_000)
    if kind == "lstsq":
        d = _log_int(rng, 200, 20_000)
        kw["m"] = _log_int(rng, 8, 512)
    if kind == "softmax":
        C = rng.randint(2, 10)
        F = 32 * _log_int(rng, 2, 128)
        d = C * F + C
        kw.update(F=F, C=C, S=rng.randint(300, 2000), B=32 * rng.randint(1, 8))
    c = _case("", kind, graph, n, d, **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# graphs and gossip matrices
# ---------------------------------------------------------------------------
def _torus_shape(n):
    return {16: (4, 4), 32: (4, 8), 64: (8, 8), 36: (6, 6)}[n]


def _edges(graph, n):
    rng = np.random.default_rng(n)
    e = set()
    add = lambda a, b: e.add((min(int(a), int(b)), max(int(a), int(b))))  # noqa: E731
    if graph == "ring":
        for i in range(n):
            add(i, (i + 1) % n)
    elif graph == "torus":
        r, c = _torus_shape(n)
        for v in range(n):
            add(v, (v // c + 1) % r * c + v % c)
            add(v, v // c * c + (v % c + 1) % c)
    elif graph == "regular4":  # two random Hamiltonian cycles without a common edge
        while len(e) != 2 * n:
            e.clear()
            for _ in range(2):
                p = rng.permutation(n)
                for a, b in zip(p, np.roll(p, 1)):
                    add(a, b)
    elif graph == "exponential":  # neighbours at distances 1, 2, 4, ...
        for i in range(n):
            s = 1
            while s <= n // 2:
                add(i, (i + s) % n)
                s *= 2
    else:  # a path plus random edges, at most 8 neighbours, 4 on average
        deg = np.zeros(n, int)
        for i in range(n - 1):
            add(i, i + 1)
            deg[i] += 1
            deg[i + 1] += 1
        while len(e) < 2 * n:
            a, b = rng.integers(0, n, 2)
            if a != b and (min(a, b), max(a, b)) not in e and deg[a] < 8 and deg[b] < 8:
                add(a, b)
                deg[a] += 1
                deg[b] += 1
    return np.array(sorted(e), dtype=np.int32)


def _topology(case):
    graph, n = case["graph"], case["n"]
    if graph == "ring":
        return D.Topology.ring()
    if graph == "torus":
        return D.Topology.torus(*_torus_shape(n))
    return D.Topology.from_edges(_edges(graph, n))


def _matrix(case):
    """W in 64 bits (symmetric): 1/(1+max degree of the two ends) per edge, the rest on the diagonal."""
    e, n = _edges(case["graph"], case["n"]), case["n"]
    deg = np.bincount(e.reshape(-1), minlength=n)
    W = np.zeros((n, n))
    for a, b in e:
        W[a, b] = W[b, a] = 1.0 / (1 + max(deg[a], deg[b]))
    W += np.diag(1.0 - W.sum(1))
    ev = np.linalg.eigvalsh(W)
    s = math.sqrt(1.0 - max(abs(ev[0]), abs(ev[-2])) ** 2)
    return torch.from_numpy(W).to(DEV), (1 - s) / (1 + s)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _alpha(case):
    return 0.01 if case["kind"] == "softmax" else 0.05 if case["kind"] == "lstsq" else 0.1


def _ld(case):
    return case["d"] if case["tight"] else D.padded_ld(case["d"])


def _inputs(case, seed):
    """Everything that comes from the seed: the state mid-run, the objective's data."""
    n, d, ld = case["n"], case["d"], _ld(case)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    sdt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(std, dtype=torch.float32, common=False):
        t = torch.zeros((n, ld), device=DEV)
        t[:, :d].normal_(0.0, std, generator=g)
        if common:  # workers that have been averaging: one model, small differences
            t[:, :d] += torch.empty(d, device=DEV).normal_(generator=g)
        return t.to(dtype)

    kind = case["kind"]
    s = {"X": normal(0.1, sdt, common=True), "seed": seed % 1000, "t": 0}
    if kind == "diag":
        return s
    if kind == "softmax":
        F, C, S, B = (case[k] for k in "FCSB")
        means = torch.empty(C, F, device=DEV).normal_(generator=g)
        pick = torch.randint(0, 2, (n, S), device=DEV, generator=g)
        lab = (torch.arange(n, device=DEV)[:, None] + pick) % C
        s["feats"] = torch.empty(n, S, F, device=DEV).normal_(generator=g).add_(means[lab]).to(torch.bfloat16)
        s["labels"] = lab.to(torch.int32)
        s["batch"] = torch.argsort(torch.rand(n, S, device=DEV, generator=g), 1)[:, :B].to(torch.int32).contiguous()
        s["X"].mul_(0.02)
    elif kind == "lstsq":
        m = case["m"]
        s["A"] = torch.empty(n, m, d, device=DEV).normal_(0.0, m ** -0.5, generator=g)
        s["b"] = torch.empty(n, m, device=DEV).normal_(generator=g) + torch.arange(n, device=DEV)[:, None] - (n - 1) / 2
    else:
        s["b"] = normal(1.0)
        h = torch.zeros((n, ld) if case["rows_h"] else (ld,), device=DEV)
        h[..., :d].uniform_(math.log(1e-3), 0.0, generator=g).exp_()
        h[..., d:] = 0
        s["h"] = h
    if kind not in ("dpsgd", "defacto"):
        s["Y"] = normal(0.05, sdt)
    if kind in ("quad", "phase", "dense", "lstsq", "softmax"):
        s["G"] = normal(0.05)  # the gradients of the iteration before
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    n, d, ld, kind = case["n"], case["d"], _ld(case), case["kind"]
    ctx = D.detag_create(_topology(case), n, d, ld, D.DETAG_BF16 if case["dtype"] == "bf16" else D.DETAG_F32)
    s.update(case=case, ctx=ctx, alpha=_alpha(case), K=case["K"],
             variant=D.DETAG_VARIANT_ALG2 if case["variant"] == "alg2" else D.DETAG_VARIANT_ATC)
    if kind in ("phase", "dense", "dpsgd", "lstsq", "softmax", "defacto"):
        s["Gnew"] = D.new_matrix(n, d, ld)
    if kind == "dense":
        ctx.set_path(D.DETAG_PATH_DENSE)
        ctx.reserve_gossip(D.DETAG_PATH_DENSE, case["K"])
    elif kind == "diag":
        s["xbar"] = torch.zeros(d, device=DEV)
        s["dist"] = torch.zeros(1, dtype=torch.float64, device=DEV)
    elif kind == "lstsq":
        ctx.reserve_gradient(m=case["m"])
    elif kind == "softmax":
        ctx.reserve_gradient(F=case["F"], C_classes=case["C"], B=case["B"])
        s["loss"] = torch.zeros(n, device=DEV)
    elif kind == "defacto":
        s["factors"] = D.Factors(ctx, 0)
        s["Xt"] = s["X"].clone()
    elif kind == "byphase":
        def grad(t, q, X, G):
            ctx.grad_quadratic_diag(X, s["h"], s["b"], G, sigma=case["sigma"], seed=s["seed"], step=t)
        s["bp"] = algorithms.ByPhase(ctx, s["X"], s["alpha"], grad, scale=1.0 / case["K"])
        s["bp"].Y.copy_(s.pop("Y"))
    return s


def run(s):
    case, ctx, kind = s["case"], s["ctx"], s["case"]["kind"]
    X, t = s["X"], s["t"]
    s["t"] = t + 1
    if kind == "quad":
        ctx.step_quadratic(X, s["Y"], s["G"], s["h"], s["b"], s["alpha"], s["K"], sigma=case["sigma"], seed=s["seed"], step=t,
                           variant=s["variant"])
        return X, s["Y"], s["G"]
    if kind == "diag":
        return ctx.mean(X, s["xbar"]), ctx.consensus_error(X, s["dist"])
    if kind == "byphase":
        s["bp"].phase(s["K"])
        return X, s["bp"].Y, s["bp"].G_km1  # the finished phase's gradients are the next one's g(k-1)
    G = s["Gnew"]
    if kind == "lstsq":
        ctx.grad_lstsq(X, s["A"], s["b"], G)
    elif kind == "softmax":
        ctx.grad_softmax_bf16(X, s["feats"], s["labels"], s["batch"], case["C"], G, s["loss"])
    else:
        ctx.grad_quadratic_diag(X, s["h"], s["b"], G, sigma=case["sigma"], seed=s["seed"], step=t)
    if kind == "dpsgd":
        ctx.dpsgd_step(X, G, s["alpha"])
        return X, G
    if kind == "defacto":
        s["factors"].average(s["Xt"])
        ctx.defacto_update(X, s["Xt"], G, s["alpha"])
        return X, s["Xt"]
    ctx.step(X, s["Y"], G, s["G"], s["alpha"], s["K"], variant=s["variant"])
    s["G"], s["Gnew"] = G, s["G"]
    return (X, s["Y"], G, s["loss"]) if kind == "softmax" else (X, s["Y"], G)


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# ---------------------------------------------------------------------------
def work(case):
    n, d, K, kind = case["n"], case["d"], case["K"], case["kind"]
    E, sb = n * d, 2 if case["dtype"] == "bf16" else 4
    deg = 2.0 * len(_edges(case["graph"], n)) / n
    rounds = 2.0 * K * E * (2 * deg + 4)
    h = 4 * (E if case["rows_h"] else d)
    grad = E * (4.0 + (40.0 if case["sigma"] else 0.0))  # Philox and Box-Muller are some 40 operations a value
    if kind == "diag":
        return {"bytes": E * sb + 4 * d + 8, "flops": 5.0 * E}
    if kind == "lstsq":
        m = case["m"]
        return {"bytes": 4 * n * m * d + 4 * n * m + 24 * E, "flops": 4.0 * n * m * d + rounds}
    if kind == "softmax":
        F, C, B = case["F"], case["C"], case["B"]
        return {"bytes": 2 * n * B * F + 8 * n * B + 24 * E, "flops": 4.0 * n * B * F * C + rounds}
    if kind == "dpsgd":
        return {"bytes": E * (2 * sb + 8) + h, "flops": grad + E * (2 * deg + 2)}
    if kind == "defacto":
        return {"bytes": E * (4 * sb + 4) + h, "flops": grad + 5.0 * E}
    if kind == "byphase":
        return {"bytes": 28 * E + h, "flops": K * (grad + 2 * E) + rounds}
    return {"bytes": E * (4 * sb + 12) + h, "flops": grad + rounds}


def tolerance(case):
    # bf16 state: one rounding at the store; a value at a tie goes either way.  fp32 state: sums of a few fp32 terms a
    # round, the reductions of the least-squares and softmax gradients in another order.
    if case["dtype"] == "bf16" and case["kind"] != "diag":
        return {"rel": 4e-3, "max": 3e-2}
    return {"rel": 2e-6, "max": 1e-4}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _philox(ctr, key):
    c0, c1, c2, c3 = ctr
    k0, k1 = key
    mask = 0xFFFFFFFF
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # wraps: the 64 product bits are what is wanted
        c0, c1, c2, c3 = ((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask
    return c0, c1, c2, c3


def _noise(n, lo, hi, seed, step):
    """Standard normals of workers 0..n-1 at columns lo..hi-1 (lo a multiple of 4): Philox-4x32-10 and Box-Muller."""
    q = torch.arange(lo // 4, (hi + 3) // 4, device=DEV, dtype=torch.int64).expand(n, -1)
    i = torch.arange(n, device=DEV, dtype=torch.int64)[:, None].expand_as(q)
    z0 = torch.zeros_like(q)
    u = [((r >> 9).double() + 0.5) * 2.0 ** -23 for r in _philox((q, z0, i, z0 + step), (seed, 0))]
    out = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        rad = torch.sqrt(-2.0 * torch.log(a))
        out += [rad * torch.cos(2 * math.pi * b), rad * torch.sin(2 * math.pi * b)]
    return torch.stack(out, -1).reshape(n, -1)[:, : hi - lo]


def _gossip(Z, W, K, eta):
    prev = cur = Z
    for _ in range(K):
        prev, cur = cur, (1 + eta) * (W @ cur) - eta * prev
    return cur


def exact(case, seed):
    s = _inputs(case, seed)
    n, d, ld, K, kind, alpha = case["n"], case["d"], _ld(case), case["K"], case["kind"], _alpha(case)
    if kind == "diag":
        xbar, dist = torch.empty(d, dtype=torch.float64, device=DEV), 0.0
        for lo in range(0, d, 1 << 20):
            x = s["X"][:, lo:min(d, lo + (1 << 20))].double()
            xbar[lo:lo + x.shape[1]] = m = x.mean(0)
            dist = dist + (x - m).square().sum()
        return xbar, dist.reshape(1)
    W, eta = _matrix(case)
    out = {k: torch.zeros((n, ld), dtype=torch.float64, device=DEV) for k in ("X", "Y", "G")}
    loss = None
    if kind == "lstsq":
        A = s["A"].double()
        r = (A * s["X"][:, None, :d].double()).sum(2) - s["b"].double()
        out["G"][:, :d] = (A * r[:, :, None]).sum(1)
        del A
    elif kind == "softmax":
        F, C, B = case["F"], case["C"], case["B"]
        loss = torch.zeros(n, dtype=torch.float64, device=DEV)
        for i in range(n):
            idx, x = s["batch"][i].long(), s["X"][i, :d].double()
            f, y = s["feats"][i, idx].double(), s["labels"][i, idx].long()
            lp = torch.log_softmax(f @ x[:C * F].reshape(C, F).T + x[C * F:], 1)
            at = torch.arange(B, device=DEV)
            loss[i] = -lp[at, y].mean()
            delta = lp.exp()
            delta[at, y] -= 1.0
            out["G"][i, :C * F] = (delta.T @ f / B).reshape(-1)
            out["G"][i, C * F:d] = delta.mean(0)
    step = 1 << 20
    for lo in range(0, d, step):
        hi = min(d, lo + step)
        c = slice(lo, hi)
        X = s["X"][:, c].double()
        if kind in ("lstsq", "softmax"):
            G = out["G"][:, c]
        else:
            G = s["h"][..., c].double() * (X - s["b"][:, c].double())
            for q in range(K if kind == "byphase" else 1):  # one query an iteration, averaged over the phase
                if case["sigma"]:
                    G = G + case["sigma"] / (K if kind == "byphase" else 1) * _noise(n, lo, hi, s["seed"], q)
            out["G"][:, c] = G
        if kind == "dpsgd":
            out["X"][:, c] = W @ X - alpha * G
        elif kind == "defacto":
            out["X"][:, c] = X.mean(0) - alpha * G
        elif kind == "byphase":
            Yg = _gossip(s["Y"][:, c].double(), W, K, eta)
            out["X"][:, c] = _gossip(X, W, K, eta) - alpha * Yg
            out["Y"][:, c] = Yg + G
        else:
            Y, Go = s["Y"][:, c].double(), s["G"][:, c].double()
            if case["variant"] == "alg2":
                Yg = _gossip(Y, W, K, eta)
                out["X"][:, c] = _gossip(X, W, K, eta) - alpha * Yg
                out["Y"][:, c] = Yg + G - Go
            else:
                out["X"][:, c] = _gossip(X - alpha * Y, W, K, eta)
                out["Y"][:, c] = _gossip(Y + G - Go, W, K, eta)
    if kind == "dpsgd":
        return out["X"], out["G"]
    if kind == "defacto":
        return out["X"], out["X"]
    return (out["X"], out["Y"], out["G"], loss) if kind == "softmax" else (out["X"], out["Y"], out["G"])
