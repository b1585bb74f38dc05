"""The on-chip sequence of the exact average consensus at the edges of its layouts (128, 64 and 32 columns to a wavefront for
up to 12, up to 24 and more workers), of its column tiles, and of the sizes from which it leaves its accesses to the caches."""
import numpy as np
import pytest
import torch

import paper_2006_08085_amd as D
from tests.gpu_util import SENTINEL, _built, padding_ok, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu


def _graph(n, rng):
    """A random tree with at most 7 children a node, and a few edges more."""
    e, deg = set(), np.zeros(n, int)
    for i in range(1, n):
        j = int(rng.choice(np.flatnonzero(deg[:i] < 7)))
        e.add((j, i))
        deg[i] += 1
        deg[j] += 1
    return np.array(sorted(e), np.int32)


@pytest.mark.parametrize("n", [2, 3, 8, 12, 13, 24, 25, 63, 64, 65, 130, 256])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_layouts_and_ragged_columns(n, dtype):
    rng = np.random.default_rng(n)
    topo = D.Topology.from_edges(_graph(n, rng))
    for d in (1, 3, 4, 31, 33, 66, 127, 130, 1029):
        for ld in (d, D.padded_ld(d) + 4):
            ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if dtype == torch.bfloat16 else D.DETAG_F32)
            f = D.Factors(ctx, int(rng.integers(n)))
            assert f.program().shape[0] > 0
            Z = to_dev(rng.standard_normal((n, d)) + 1.0, ld, dtype)
            z = to_host(Z, d)
            f.average(Z)
            got, want = to_host(Z, d), np.broadcast_to(z.mean(0), (n, d))
            # a row is a sum of up to 8 terms in each of R steps, a partial sum up to n times a value that counts 1/n in
            # the result; bf16 state rounds once more, to 8 bits
            bound = 8 * f.R * 2.0 ** -24 * np.abs(z).max() + (2.0 ** -8 * np.abs(want) if dtype == torch.bfloat16 else 0.0)
            assert np.all(np.abs(got - want) <= bound), (d, ld)
            assert padding_ok(Z, d)
            f.close()
            ctx.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_the_layout_of_the_rows_does_not_change_the_bits(dtype):
    n = 64
    topo = D.Topology.from_edges(_graph(n, np.random.default_rng(1)))
    for elements in (1_000_000, 9_000_000, 27_000_000, 52_000_000):  # both sides of 32 and 96 MiB
        d = elements // n + 5
        g = torch.Generator(device="cuda")
        g.manual_seed(d)
        values, runs = torch.empty(n, d, device="cuda").normal_(generator=g), []
        for ld, shift in ((D.padded_ld(d), 0), (d + 1 - d % 2, 0), (D.padded_ld(d), 1)):
            Z = torch.full((n * ld + shift,), SENTINEL, device="cuda", dtype=dtype)[shift:].view(n, ld)
            Z[:, :d] = values
            ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if dtype == torch.bfloat16 else D.DETAG_F32)
            f = D.Factors(ctx, 0)
            f.average(Z)
            torch.cuda.synchronize()
            assert torch.equal(Z[:, d:], torch.full_like(Z[:, d:], SENTINEL))
            runs.append(Z[:, :d])
            f.close()
            ctx.close()
        assert torch.equal(runs[0], runs[1]) and torch.equal(runs[0], runs[2]), d


@pytest.mark.parametrize("n", [3, 8, 9, 12, 13, 16, 20, 21, 24, 25, 28, 32, 33, 40])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_large_calls_of_few_workers_give_the_bits_of_small_ones(n, dtype):
    """The lanes to a row, and whether a wavefront copies its table to LDS, depend on the size of a call (16, 80 and 88 MiB) for
    up to 40 workers."""
    few, edges = 1003, np.array([(max(0, i - 2), i) for i in range(1, n)], np.int32)   # a deep tree: a long table
    for topo in (D.Topology.from_edges(_graph(n, np.random.default_rng(n))), D.Topology.from_edges(edges)):
        size = 2 if dtype == torch.bfloat16 else 4
        for mib in (17, 89):
            many = (mib << 20) // (n * size) + 3
            g = torch.Generator(device="cuda")
            g.manual_seed(n)
            values, runs = torch.empty(n, many, device="cuda").normal_(generator=g) + 1.0, []
            for d, ld in ((few, few), (many, D.padded_ld(many)), (many, many | 1)):
                Z = torch.full((n, ld), SENTINEL, device="cuda", dtype=dtype)
                Z[:, :d] = values[:, :d]
                want, largest = Z[:, :d].double().mean(0), Z[:, :d].double().abs().amax(0)
                ctx = D.detag_create(topo, n, d, ld, D.DETAG_BF16 if dtype == torch.bfloat16 else D.DETAG_F32)
                f = D.Factors(ctx, 0)
                assert f.program().shape[0] > 0
                f.average(Z)
                torch.cuda.synchronize()
                bound = 8 * f.R * 2.0 ** -24 * largest.max() + (2.0 ** -8 * want.abs() if dtype == torch.bfloat16 else 0.0)
                assert ((Z[:, :d].double() - want).abs() <= bound).all(), (d, ld)
                assert torch.equal(Z[:, d:], torch.full_like(Z[:, d:], SENTINEL))
                runs.append(Z[:, :d])
                f.close()
                ctx.close()
            assert torch.equal(runs[1], runs[2]) and torch.equal(runs[0], runs[1][:, :few]), mib
