"""The index lists on both sides of the row count up to which the compaction
sums the row counts itself, and the out-of-place block, whose expansion also
copies the identity path, against the in-place one."""
import numpy as np
import pytest
import torch

import oracle
from paper_1912_03203_amd import dynconv as dc
from paper_1912_03203_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dc.load()


@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (1, 5, 3), (2, 4, 130), (1, 4095, 2), (16, 256, 9), (17, 241, 9), (3, 1400, 5)])
@pytest.mark.parametrize("dilate", [0, 1, 3])
def test_lists(n, h, w, dilate):
    rng = inputs.rng_for(n + h + w)
    G = (rng.random(n * h * w) < 0.3).astype(np.uint8)
    A, D, nbr = oracle.indices(G, oracle.dilate(G, n, h, w, dilate), n, h, w)
    s = dc.Shape(n, h, w, 8)
    idx = dc.IndexBuffers.alloc(n * h * w)
    ws = torch.empty(dc.indices_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    dc.build_indices(torch.from_numpy(G).cuda(), s, dilate, idx, ws)
    torch.cuda.synchronize()
    P, Pd = (int(v) for v in idx.counts.cpu())
    assert (P, Pd) == (A.size, D.size)
    assert np.array_equal(idx.active[:P].cpu().numpy(), A)
    assert np.array_equal(idx.dilated[:Pd].cpu().numpy(), D)
    assert np.array_equal(idx.nbr[:9 * P].cpu().numpy().reshape(P, 9), nbr)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("n,h,w,c,e", [(1, 3, 5, 8, 16), (2, 19, 23, 40, 240), (1, 7, 7, 256, 1536)])
@pytest.mark.parametrize("density", [0.0, 0.3, None])
def test_block_out_of_place(dtype, n, h, w, c, e, density):
    rng = inputs.rng_for(c + e)
    dt = dc.NAME_TO_DTYPE[dtype]
    x = torch.from_numpy(inputs.blob_features(rng, n, h, w, c)).cuda().to(dt)
    blk = dc.BlockWeights.from_arrays(inputs.block_weights(rng, c, e, dtype=dtype), dt)
    s = dc.shape_of(x)
    idx = None
    if density is not None:
        idx = dc.IndexBuffers.alloc(n * h * w)
        mask = torch.from_numpy((rng.random(n * h * w) < density).astype(np.uint8)).cuda()
        dc.build_indices(mask, s, 1, idx, torch.empty(dc.indices_workspace_bytes(s), dtype=torch.uint8, device="cuda"))
    ws = torch.empty(dc.block_workspace_bytes(s, blk, dt), dtype=torch.uint8, device="cuda")
    y, z = torch.full_like(x, float("nan")), x.clone()
    keep = x.clone()
    dc.block_forward(x, y, blk, idx, ws)
    dc.block_forward(z, z, blk, idx, ws)
    torch.cuda.synchronize()
    assert torch.equal(x.view(torch.uint8), keep.view(torch.uint8))
    assert torch.equal(y.view(torch.uint8), z.view(torch.uint8))
