"""The register-resident kernels on both sides of their block size (one wavefront up to 32,768 columns, four beyond) and of
the size from which they stream past the caches (80 MiB a call): columns are independent, so the same columns come out with
the same bits."""
import pytest
import torch

import paper_2006_08085_amd as D
from tests.gpu_util import DEV, SENTINEL, _built  # noqa: F401

pytestmark = pytest.mark.gpu


def _matrix(n, d, ld, seed, dtype=torch.float32):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    t = torch.full((n, ld), SENTINEL, device=DEV)
    t[:, :d] = torch.empty(d, n, device=DEV).normal_(generator=g).T  # the same values in the columns of every width
    return t.to(dtype)


def _all_calls(topo, n, d, dtype):
    ld, K, eta = D.padded_ld(d), 3, 0.35
    sd = torch.bfloat16 if dtype == "bf16" else torch.float32
    ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if dtype == "bf16" else D.DETAG_F32)
    assert ctx.kernel() == D.DETAG_KERNEL_REGISTER_TILE
    X, Y, Gn, Go, b = (_matrix(n, d, ld, k, sd if k < 2 else torch.float32) for k in range(5))
    h = _matrix(1, d, ld, 6)[0].abs()
    out = []
    for variant in (D.DETAG_VARIANT_ATC, D.DETAG_VARIANT_ALG2):
        x, y, g = X.clone(), Y.clone(), Go.clone()
        ctx.step(x, y, Gn, Go, 0.2, K, eta, variant)
        out += [x.clone(), y.clone()]
        x, y = X.clone(), Y.clone()
        ctx.step_quadratic(x, y, g, h, b, 0.2, K, sigma=0.1, seed=3, step=1, eta=eta, variant=variant)
        out += [x, y, g]
    z, p, r = X.clone(), X.clone(), X.clone()
    ctx.gossip_accel(z, K, eta)
    ctx.dpsgd_step(p, Gn, 0.2)
    ctx.gossip_round(X, Y, r, eta)
    ctx.close()
    for t in out + [z, p, r]:
        assert torch.equal(t[:, d:], torch.full_like(t[:, d:], SENTINEL))
    return [t[:, :d] for t in out + [z, p, r]]


@pytest.mark.parametrize("topo,n", [(D.Topology.ring(), 16), (D.Topology.torus(8, 8), 64)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_same_bits_on_both_sides_of_the_block_size_and_of_the_caches(topo, n, dtype):
    widths = (32_767, 32_768, 32_769, 5_242_880 // n, 5_242_880 // n + 70)
    runs = [_all_calls(topo, n, d, dtype) for d in widths]
    wide = runs[-1]
    for d, run in zip(widths, runs):
        for k, (got, want) in enumerate(zip(run, wide)):
            assert torch.equal(got[:, : min(d, widths[-1])], want[:, : min(d, widths[-1])]), (d, k)


@pytest.mark.parametrize("kind,n", [("ring", 4), ("ring", 12), ("ring", 16), ("torus44", 16), ("torus48", 32), ("ring", 48),
                                    ("ring", 64), ("torus88", 64)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [1, 63, 64, 65, 1000, 4097])
def test_two_wavefronts_to_a_phase_give_the_bits_of_one(kind, n, dtype, d):
    """Narrow contexts run the two sides of a phase in two wavefronts, wide ones in one: the first columns of both."""
    wide, ld, bf = 70001, 70016, dtype == "bf16"
    topo = D.Topology.ring() if kind == "ring" else D.Topology.torus(*{16: (4, 4), 32: (4, 8), 64: (8, 8)}[n])
    g = torch.Generator(device="cuda").manual_seed(n + d)
    normal = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    sdt = torch.bfloat16 if bf else torch.float32
    X, Y, G, B = normal(n, ld).to(sdt), normal(n, ld).to(sdt), normal(n, ld), normal(n, ld)
    X[1, 0] = float("inf")
    h = torch.rand(n, ld, device="cuda", generator=g)
    dts = D.DETAG_BF16 if bf else D.DETAG_F32
    one, two = D.detag_create(topo, n, wide, ld, dts), D.detag_create(topo, n, d, ld, dts)
    for variant in (D.DETAG_VARIANT_ATC, D.DETAG_VARIANT_ALG2):
        for K in (1, 4):
            for curvature in (None, h[0].contiguous(), h):
                out = []
                for ctx in (one, two):
                    x, y, gr = X.clone(), Y.clone(), G.clone()
                    if curvature is None:
                        ctx.step(x, y, gr, B, 0.1, K, 0.3, variant)
                    else:
                        ctx.step_quadratic(x, y, gr, curvature, B, 0.1, K, sigma=0.2, seed=7, step=3, eta=0.3, variant=variant)
                    out.append((x, y, gr))
                for a, b, before in zip(*out, (X, Y, G)):
                    assert torch.equal(a[:, :d].nan_to_num(), b[:, :d].nan_to_num())
                    assert torch.equal(a[:, :d].isnan(), b[:, :d].isnan())
                    assert torch.equal(b[:, d:].nan_to_num(), before[:, d:].nan_to_num())


def test_bf16_state_is_rounded_to_nearest_even():
    """Every exponent, ties, denormals, infinities and NaN through a store of bf16 state: y = 0 + g - 0."""
    exp = torch.arange(256, dtype=torch.int64)[:, None] << 23
    man = torch.tensor([0, 1, 0x7fff, 0x8000, 0x8001, 0xffff, 0x10000, 0x17fff, 0x18000, 0x18001, 0x7f7fff, 0x7f8000, 0x7fffff])
    bits = (exp + man).reshape(-1)
    bits = torch.cat([bits, bits + (1 << 31)])
    vals = torch.where(bits >= 1 << 31, bits - (1 << 32), bits).to(torch.int32).view(torch.float32)
    d = vals.numel()
    ctx = D.detag_create(D.Topology.ring(), 4, d, d, D.DETAG_BF16)
    g = vals.expand(4, d).contiguous().cuda()
    y, zero = torch.zeros(4, d, dtype=torch.bfloat16, device="cuda"), torch.zeros(4, d, device="cuda")
    ctx.track(y, g, zero)
    x, y2 = torch.zeros_like(y), torch.zeros_like(y)
    ctx.step(x, y2, g, zero, 0.0, 1, 0.0, D.DETAG_VARIANT_ALG2)     # the same through the register kernels
    want = vals.to(torch.bfloat16).float()
    for got in (y[0], y[3], y2[1]):
        got = got.float().cpu()
        assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.nan_to_num(7.0), want.nan_to_num(7.0))
