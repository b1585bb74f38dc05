"""Softmax gradient at the edges of its blocks: one chunk of features, a short last chunk, more workers than chunks are
wanted for, batches that are not a multiple of the 64 samples a wavefront transposes at a time, few and many classes."""
import numpy as np
import pytest
import torch

import paper_2006_08085_amd as D
from oracle import objectives as OO
from workloads import generate as gen
from tests.gpu_util import DEV, _built, padding_ok, to_dev, to_host  # noqa: F401
from tests.util import TOL_F32, amax, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,S,F,C,B,pad", [(1, 40, 32, 2, 32, 0), (2, 90, 416, 10, 96, 1), (5, 70, 800, 5, 160, 3), (40, 64, 416, 9, 64, 0),
                                           (17, 300, 3072, 10, 256, 2), (3, 300, 4128, 4, 224, 0), (300, 33, 416, 3, 32, 5)])
def test_chunks_and_stages(n, S, F, C, B, pad):
    d = C * F + C
    ld = d + pad
    feats, labels = gen.softmax_problem(n, S, F, C, seed=3)
    fb = torch.from_numpy(feats).to(torch.bfloat16)
    idx = np.random.default_rng(1).integers(0, S, (n, B)).astype(np.int32)
    X = gen.state(n, d, seed=2, scale=0.05)
    topo = D.Topology.ring() if n > 1 else D.Topology.from_dense(np.ones((1, 1)))
    ctx = D.detag_create(topo, n, d, ld)
    G, loss = to_dev(np.zeros((n, d)), ld), torch.zeros(n, device=DEV)
    for _ in range(2):                                  # the second call finds the scratch used
        ctx.grad_softmax_bf16(to_dev(X, ld), fb.to(DEV), torch.from_numpy(labels).to(DEV), torch.from_numpy(idx).to(DEV), C, G, loss)
    ref, lref = OO.grad_softmax(X, fb.float().numpy(), labels, idx, F, C)
    assert rel_err(to_host(G, d), ref, amax(ref)) < TOL_F32
    assert np.abs(loss.cpu().numpy() - lref).max() < 1e-5 * np.abs(lref).max()
    assert padding_ok(G, d)


@pytest.mark.parametrize("n,S,F,C,B,pad", [(2, 70, 6144, 3, 64, 0), (2, 70, 6176, 3, 64, 1), (1, 300, 16416, 10, 256, 0), (20, 40, 9216, 7, 32, 2)])
def test_as_many_chunks_as_are_added_up_and_more(n, S, F, C, B, pad):
    """16, 17, 43 and 24 chunks: from 17 on a launch of its own adds their parts of the logits up."""
    test_chunks_and_stages(n, S, F, C, B, pad)
