"""The consensus distance where the number of its partial sums (one per 256 columns) is around a multiple of the threads, and
of the threads times the sums each of them keeps, that add them up."""
import pytest
import torch

import paper_2006_08085_amd as D
from tests.gpu_util import DEV, _built  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 2, 1023, 1024, 1025, 8191, 8192, 8193, 9217, 16385])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_number_of_partial_sums(blocks, dtype):
    n, d = 3, blocks * 256 - 100
    g = torch.Generator(device=DEV)
    g.manual_seed(blocks)
    X = torch.empty(n, d, device=DEV).normal_(generator=g).to(dtype)
    ctx = D.detag_create(D.Topology.ring(), n, d, d, D.DETAG_BF16 if dtype == torch.bfloat16 else D.DETAG_F32)
    x = X.double()
    want = (x - x.mean(0)).square().sum().item()
    out = torch.zeros(1, dtype=torch.float64, device=DEV)
    # every term is exact to a few ulps of fp64 and there are n * d of them
    assert abs(ctx.consensus_error(X).item() - want) <= 1e-12 * want
    assert ctx.consensus_error_static(X, out).item() == ctx.consensus_error(X).item()
    assert torch.allclose(ctx.mean(X), x.mean(0).float(), rtol=2.0 ** -23, atol=1e-30)
    ctx.close()
