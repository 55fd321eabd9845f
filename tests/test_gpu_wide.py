"""The channel-parallel one-launch block kernel against the kernel chain, byte
for byte, where its tiling changes: chunks of 64 or 128 hidden channels (one,
several, a partial last one), 2, 4 or 8 tiles of needed positions (above 128
channels 2 or 4, and maps without such a cut), contraction tails, single rows,
columns and positions, empty, full and nearly full masks, more patches than one
grid dimension holds."""
import numpy as np
import pytest
import torch

from paper_1912_03203_amd import dynconv as dc
from paper_1912_03203_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dc.load()


CASES = [
    # dtype, (N, H, W, C, E), density, blocks
    ("f16", (1, 1, 1, 40, 16), 1.0, 1),          # one position, one chunk
    ("bf16", (2, 9, 41, 64, 64), 0.4, 2),        # a chunk of 64, strips of less than 40 columns
    ("f16", (2, 9, 13, 64, 80), 0.4, 2),         # one partial chunk of 128
    ("f16", (3, 14, 14, 64, 384), 0.3, 2),       # three chunks
    ("bf16", (300, 14, 14, 64, 208), 0.3, 1),    # 1,200 patches: k_block_fused
    ("f16", (2, 11, 7, 72, 16), 0.5, 2),         # several-chunk form with one chunk, contraction tail
    ("bf16", (3, 30, 29, 96, 144), 0.3, 2),      # 8 needed tiles, last chunk of 16
    ("f16", (2, 8, 8, 96, 128), 0.0, 2),         # no active position
    ("f16", (1, 6, 5, 104, 256), 1.0, 1),        # all active
    ("bf16", (2, 33, 40, 128, 272), 0.4, 1),     # wide image
    ("f16", (1, 3, 1000, 112, 144), 0.3, 1),     # 97-128 channels, 8 needed tiles
    ("f16", (5, 7, 7, 160, 960), 0.4, 2),        # 2 needed tiles
    ("bf16", (2, 16, 15, 160, 304), 0.4, 2),     # 4 needed tiles, chunks of 64
    ("f16", (1, 9, 1, 192, 80), 0.5, 1),         # less scratch on the chain
    ("f16", (1, 9, 1, 192, 208), 0.5, 1),        # one column, several chunks of 64
    ("bf16", (5, 14, 9, 192, 192), 0.4, 2),
    ("f16", (1, 100, 100, 160, 160), 0.9, 1),    # 4 needed tiles, all of them full
    ("bf16", (1, 60, 60, 192, 176), 0.9, 1),
    ("f16", (1, 112, 112, 160, 160), 0.9, 2),    # 160 and 192 channels without a cut: the chain
    ("bf16", (1, 48, 160, 192, 192), 0.6, 1),
    ("f16", (2, 20, 600, 160, 176), 0.9, 1),
    ("bf16", (1, 112, 112, 128, 144), 0.9, 1),   # 97-128 channels, 8 needed tiles, nearly full
    ("f16", (2, 5, 6, 32, 208), 0.4, 2),         # above the cell kernel's hidden width
    ("f32", (1, 7, 3, 8, 16), 0.5, 2),
    ("f32", (2, 16, 17, 32, 192), 0.4, 2),
    ("f32", (3, 12, 9, 64, 80), 0.4, 1),
    ("f32", (90, 32, 32, 16, 32), 0.4, 1),       # more than 256 patches: k_block_fused
]


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_%s" % (c[0], "x".join(map(str, c[1]))))
def test_stack_equals_the_kernel_chain(case, dense):
    dtype, (N, H, W, C, E), density, nb = case
    rng = inputs.rng_for(N * H * W + C + E)
    dt = dc.NAME_TO_DTYPE[dtype]
    x = torch.from_numpy(inputs.blob_features(rng, N, H, W, C)).cuda().to(dt)
    blocks = [dc.BlockWeights.from_arrays(inputs.block_weights(rng, C, E, dtype=dtype), dt) for _ in range(nb)]
    logits = torch.empty(N * H * W, device="cuda")
    dc.mask(x, blocks[0].w_mask, 0.0, logits=logits)
    for b in blocks:  # about the density in the first block; extremes in all
        b.b_mask = float("inf") if density == 1.0 else float("-inf") if density == 0.0 else float(
            inputs.percentile_bias(logits.cpu().numpy(), density))
    got = []
    for flags in (0, dc.STACK_UNFUSED):
        y = torch.full_like(x, float("nan"))
        masks = torch.full((nb, N * H * W), 9, dtype=torch.uint8, device="cuda")
        counts = torch.full((nb, 2), -1, dtype=torch.int32, device="cuda")
        dc.stack_forward(x, y, blocks, flags | (dc.STACK_DENSE if dense else 0), None if dense else masks,
                         None if dense else counts)
        torch.cuda.synchronize()
        got.append([t.cpu().view(torch.uint8).numpy() for t in (y, masks, counts)])
    for a, b, what in zip(got[0], got[1], ("output", "masks", "counts")):
        assert np.array_equal(a, b), what
    # the same, in place
    y = x.clone()
    dc.stack_forward(y, y, blocks, dc.STACK_DENSE if dense else 0)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().view(torch.uint8).numpy(), got[0][0])


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("c,e", [(40, 16), (96, 16), (160, 160), (32, 208)])
def test_more_patches_than_one_grid_dimension(c, e, dense):
    """Many tiny images: 8.5 M patches of 512 threads are more than the 2^32
    threads of one grid dimension.  Every image is one position, so the
    depthwise is its centre tap; compared with the kernel chain, byte for byte."""
    n, dt = 8_500_000, torch.float16
    g = torch.Generator(device="cuda").manual_seed(c)
    x = torch.randn(n, 1, 1, c, generator=g, device="cuda", dtype=dt)
    blk = dc.BlockWeights.from_arrays(inputs.block_weights(inputs.rng_for(c), c, e, dtype="f16"), dt)
    got = []
    for flags in (0, dc.STACK_UNFUSED):
        y = torch.full_like(x, float("nan"))
        counts = None if dense else torch.full((1, 2), -1, dtype=torch.int32, device="cuda")
        dc.stack_forward(x, y, [blk], flags | (dc.STACK_DENSE if dense else 0), None, counts)
        torch.cuda.synchronize()
        got.append((y, counts))
    assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16))
    if not dense:
        assert torch.equal(got[0][1], got[1][1]) and 0 < int(got[0][1][0, 0]) < n


def test_more_rows_than_one_grid_dimension():
    """70 M rows of one position: the index lists take one wave of 64 per row."""
    n = 70_000_000
    s = dc.Shape(n, 1, 1, 8)
    m = (torch.arange(n, device="cuda") % 3 == 0).to(torch.uint8)
    idx = dc.IndexBuffers.alloc(n)
    dc.build_indices(m, s, 1, idx, torch.empty(dc.indices_workspace_bytes(s), dtype=torch.uint8, device="cuda"))
    want = torch.arange(0, n, 3, device="cuda", dtype=torch.int32)
    p = want.numel()
    assert idx.counts.tolist() == [p, p]
    assert torch.equal(idx.active[:p], want) and torch.equal(idx.dilated[:p], want)
    nbr = idx.nbr[:9 * p].view(p, 9)
    assert torch.equal(nbr[:, 4], torch.arange(p, device="cuda", dtype=torch.int32))
    assert bool((nbr[:, [0, 1, 2, 3, 5, 6, 7, 8]] == -1).all())


@pytest.mark.parametrize("dtype,c,cp,e", [("bf16", 20, 16, 32), ("f16", 116, 64, 144), ("f32", 34, 24, 32),
                                          ("bf16", 232, 120, 256), ("f16", 312, 160, 160)])
def test_shuffle_units_equal_the_kernel_chain(dtype, c, cp, e):
    rng = inputs.rng_for(c)
    dt = dc.NAME_TO_DTYPE[dtype]
    x = torch.from_numpy(inputs.blob_features(rng, 3, 9, 11, c)).cuda().to(dt)
    br = [dc.BlockWeights.from_arrays(inputs.block_weights(rng, cp, e, dtype=dtype), dt, acts=(1, 0, 1))
          for _ in range(3)]
    got = []
    for flags in (0, dc.STACK_UNFUSED):
        y = torch.full_like(x, float("nan"))
        masks = torch.full((3, 3 * 9 * 11), 9, dtype=torch.uint8, device="cuda")
        counts = torch.full((3, 2), -1, dtype=torch.int32, device="cuda")
        dc.ShuffleStack(x, y, br, flags, masks, counts)()
        torch.cuda.synchronize()
        got.append([t.cpu().view(torch.uint8).numpy() for t in (y, masks, counts)])
    for a, b, what in zip(got[0], got[1], ("output", "masks", "counts")):
        assert np.array_equal(a, b), what
