"""Which accesses stream past the caches depends on the size of a call and on whether its column tiles share cache lines
(the pitch, the base address): the bits of the result do not.  Sizes on both sides of the lines the kernels draw (32, 80,
128 and 192 MiB a call)."""
import numpy as np
import pytest
import torch

import paper_2006_08085_amd as D
from tests.gpu_util import DEV, SENTINEL, _built  # noqa: F401
from workloads import generate as gen

pytestmark = pytest.mark.gpu


def _topology(kind, n):
    if kind == "torus":
        return D.Topology.torus(8, 8)
    if kind == "path":  # rows of different weights
        return D.Topology.from_edges(np.array([(i, i + 1) for i in range(n - 1)], np.int32), D.DETAG_W_METROPOLIS)
    return D.Topology.from_edges(gen.edges_random_regular(n, 4, seed=1), D.DETAG_W_METROPOLIS)


def _place(values, ld, shift, dtype):
    n, d = values.shape
    flat = torch.full((n * ld + shift,), SENTINEL, device=DEV, dtype=dtype)
    t = flat[shift:].view(n, ld)
    t[:, :d] = values
    return t


def _all_calls(topo, n, d, ld, shift, dtype, values):
    K, eta = 3, 0.35
    ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if dtype == torch.bfloat16 else D.DETAG_F32)
    new = lambda k: _place(values[k], ld, shift, dtype if k < 2 else torch.float32)  # noqa: E731
    h = values[4][0].abs().contiguous()
    out = []
    for variant in (D.DETAG_VARIANT_ATC, D.DETAG_VARIANT_ALG2):
        x, y, gn, go = new(0), new(1), new(2), new(3)
        ctx.step(x, y, gn, go, 0.2, K, eta, variant)
        out += [x, y]
        if ctx.kernel() == D.DETAG_KERNEL_REGISTER_TILE or (ctx.has_fused() and variant == D.DETAG_VARIANT_ATC):
            x, y = new(0), new(1)
            ctx.step_quadratic(x, y, go, h, gn, 0.2, K, sigma=0.1, seed=3, step=1, eta=eta, variant=variant)
            out += [x, y, go]
    z, p, r = new(0), new(0), new(0)
    ctx.gossip_accel(z, K, eta)
    ctx.dpsgd_step(p, new(2), 0.2)
    ctx.gossip_round(new(0), new(1), r, eta)
    out += [z, p, r]
    ctx.set_path(D.DETAG_PATH_DENSE)
    for variant in (D.DETAG_VARIANT_ATC, D.DETAG_VARIANT_ALG2):
        x, y = new(0), new(1)
        ctx.step(x, y, new(2), new(3), 0.2, K, eta, variant)
        out += [x, y]
    ctx.set_path(D.DETAG_PATH_PER_ROUND)
    p = new(0)
    ctx.dpsgd_step(p, new(2), 0.2)
    out += [p, ctx.mean(new(0))[None], ctx.consensus_error(new(0))[None]]
    torch.cuda.synchronize()
    ctx.close()
    for t in out[:-2]:
        assert torch.equal(t[:, d:], torch.full_like(t[:, d:], SENTINEL))
    return [t[:, :d] for t in out]


@pytest.mark.parametrize("kind,n", [("torus", 64), ("rr", 64), ("rr", 20), ("rr", 200), ("path", 100)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_the_layout_does_not_change_the_bits(kind, n, dtype):
    topo = _topology(kind, n)
    for elements in (2_200_000, 4_000_000, 6_500_000, 9_500_000):
        d = elements // n + 3
        g = torch.Generator(device=DEV)
        g.manual_seed(d)
        values = [torch.empty(n, d, device=DEV).normal_(generator=g) for _ in range(5)]
        on_lines = _all_calls(topo, n, d, D.padded_ld(d), 0, dtype, values)
        for ld, shift in ((d + 1 - d % 2, 0), (D.padded_ld(d), 1)):
            for k, (got, want) in enumerate(zip(_all_calls(topo, n, d, ld, shift, dtype, values), on_lines)):
                assert torch.equal(got, want), (d, ld, shift, k)


@pytest.mark.parametrize("kind,n", [("path", 3), ("path", 14), ("rr", 20), ("path", 24), ("rr", 28)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_tiles_of_128_and_256_columns_beyond_the_caches(kind, n, dtype):
    """Few workers: whether a call at an odd pitch streams depends on the width of its tiles up to 480 MiB."""
    topo = _topology(kind, n)
    for elements in (18_000_000, 33_000_000):
        d = elements // n | 1
        g = torch.Generator(device=DEV)
        g.manual_seed(d)
        values = [torch.empty(n, d, device=DEV).normal_(generator=g) for _ in range(5)]
        on_lines = _all_calls(topo, n, d, D.padded_ld(d), 0, dtype, values)
        for k, (got, want) in enumerate(zip(_all_calls(topo, n, d, d, 0, dtype, values), on_lines)):
            assert torch.equal(got, want), (d, k)


@pytest.mark.parametrize("kind,n", [("ring", 4), ("ring", 8), ("ring", 16)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rings_at_odd_and_half_pitches(kind, n, dtype):
    """Register-resident calls: where rows may start for a call to stream depends on its form, up to 280 MiB."""
    for elements in (9_000_000, 18_000_000, 34_000_000):
        d = elements // n // 64 * 64 + 31
        g = torch.Generator(device=DEV)
        g.manual_seed(d)
        values = [torch.empty(n, d, device=DEV).normal_(generator=g) for _ in range(5)]
        on_lines = _all_calls(D.Topology.ring(), n, d, D.padded_ld(d), 0, dtype, values)
        for ld in (d, d + 1):
            for k, (got, want) in enumerate(zip(_all_calls(D.Topology.ring(), n, d, ld, 0, dtype, values), on_lines)):
                assert torch.equal(got, want), (d, ld, k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_row_walking_kernels_on_both_sides_of_128_mib(dtype):
    """Their loads stream from 104 or 128 MiB a call on: the same columns, alone and as part of a call beyond that."""
    n, few, many = 16, 1003, 1_200_003
    g = torch.Generator(device=DEV)
    g.manual_seed(2)
    values = [torch.empty(n, many, device=DEV).normal_(generator=g) for _ in range(5)]

    def calls(d):
        ld = d + 1
        ctx = D.detag_create(D.Topology.ring(), n, d, ld, D.DETAG_BF16 if dtype == torch.bfloat16 else D.DETAG_F32)
        new = lambda k: _place(values[k][:, :d], ld, 0, dtype if k < 2 else torch.float32)  # noqa: E731
        out = [new(4)]
        ctx.grad_quadratic_diag(new(0), values[3][0].abs().contiguous(), new(2), out[0], sigma=0.1, seed=3, step=1)
        x, y = new(0), new(1)
        ctx.step(x, y, new(2), new(3), 0.2, 0)
        out += [x, y]
        y = new(1)
        ctx.track(y, new(2), new(3))
        a = new(2)
        ctx.accumulate(a, new(3), 0.3)
        out += [y, a]
        x, xt, y, old = new(0), new(0), new(1), new(3)
        ctx.phase_end(x, xt, y, new(2), old, 0.2)
        out += [x, xt, y, old]
        x, xt, a = new(0), new(1), new(2)
        ctx.defacto_update(x, xt, a, 0.2)
        out += [x, xt, a]
        torch.cuda.synchronize()
        ctx.close()
        for t in out:
            assert torch.equal(t[:, d:], torch.full_like(t[:, d:], SENTINEL))
        return [t[:, :few] for t in out]

    for k, (got, want) in enumerate(zip(calls(many), calls(few))):
        assert torch.equal(got, want), k


@pytest.mark.parametrize("n", [20, 64, 100, 200])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_dense_gossip_that_streams(n, dtype):
    """Plain gossip on the dense path beyond 64 and 80 MiB: on lines it streams and walks its tiles in order, at an odd pitch
    it does neither."""
    d = (22_000_000 if dtype == torch.float32 else 44_000_000) // n | 1
    values = torch.empty(n, d, device=DEV).normal_(generator=torch.Generator(device=DEV).manual_seed(d))
    got = []
    for ld in (D.padded_ld(d), d):
        ctx = D.detag_create(_topology("rr", n), n, d, ld, D.DETAG_BF16 if dtype == torch.bfloat16 else D.DETAG_F32)
        ctx.set_path(D.DETAG_PATH_DENSE)
        z = _place(values, ld, 0, dtype)
        ctx.gossip_accel(z, 3, 0.35)
        torch.cuda.synchronize()
        ctx.close()
        assert torch.equal(z[:, d:], torch.full_like(z[:, d:], SENTINEL))
        got.append(z[:, :d])
    assert torch.equal(*got)
