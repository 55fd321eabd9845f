"""The pointwise and depthwise layers of a network where their launches change
shape: one 16 x 16 tile per wave against shared tiles, one chunk of the
contraction against several, 1, 2 or 4 output rows per depthwise task.  Against
the numpy fp64 definitions, within the storage rounding (2e-2 normwise for
16-bit, 1e-5 for fp32, as for the other layers)."""
import numpy as np
import pytest
import torch

from oracle import network as onet
from paper_1912_03203_amd import dynconv as dc
from paper_1912_03203_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dc.load()


def run(x, layers, dtype):
    dt = dc.NAME_TO_DTYPE[dtype]
    net = dc.NetworkWeights(layers, dt)
    xd = torch.from_numpy(x).cuda().to(dt)
    o = dc.network_output_shape(dc.shape_of(xd), net)
    y = torch.full((o.n, o.h, o.w, o.c), float("nan"), dtype=dt, device="cuda")
    dc.Network(xd, y, net)()
    torch.cuda.synchronize()
    return y.float().cpu().numpy().astype(np.float64)


def check(got, want, dtype):
    err = np.max(np.abs(got - want)) / np.max(np.abs(want))
    assert err <= (1e-5 if dtype == "f32" else 2e-2), err


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("n,h,w,c,o", [
    (1, 1, 1, 8, 8), (1, 7, 7, 40, 24), (1, 7, 7, 320, 1280), (1, 9, 5, 264, 40),  # a tile per wave
    (2, 60, 40, 32, 104),                                                          # the same, one step
    (9, 32, 32, 72, 40), (5, 40, 33, 264, 72), (3, 64, 40, 96, 200), (20, 14, 14, 520, 136)])
def test_conv1x1(dtype, n, h, w, c, o):
    rng = inputs.rng_for(c + o)
    x = inputs.round_to_storage(rng.standard_normal((n, h, w, c)), dtype)
    L = {"kind": "conv1x1", "w": inputs.round_to_storage(rng.normal(0, 0.05, (o, c)), dtype),
         "b": rng.normal(0, 0.1, o).astype(np.float32), "act": 1}
    want = np.maximum(x.reshape(-1, c).astype(np.float64) @ L["w"].astype(np.float64).T + L["b"], 0.0)
    check(run(x, [L], dtype), want.reshape(n, h, w, o), dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("n,h,w,c", [(1, 1, 1, 8), (2, 7, 9, 40), (40, 15, 14, 96), (64, 31, 17, 64), (300, 16, 9, 40)])
def test_depthwise_block(dtype, stride, n, h, w, c):
    """A block without expansion: depthwise (1, 2, 4 rows per task) and projection."""
    rng = inputs.rng_for(n + c)
    x = inputs.round_to_storage(rng.standard_normal((n, h, w, c)), dtype)
    L = {"kind": "block", "stride": stride, "acts": (2, 2, 0), "w1": None, "b1": None,
         "w2": inputs.round_to_storage(rng.normal(0, 0.3, (c, 9)), dtype), "b2": rng.normal(0, 0.1, c).astype(np.float32),
         "w3": inputs.round_to_storage(rng.normal(0, 0.2, (16, c)), dtype), "b3": rng.normal(0, 0.1, 16).astype(np.float32)}
    want = onet.dense_block(x.transpose(0, 3, 1, 2).astype(np.float64), L)
    check(run(x, [L], dtype), want.transpose(0, 2, 3, 1), dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("n,h,w,ci,o", [(1, 1, 1, 3, 8), (2, 3, 3, 3, 16), (1, 2, 40, 3, 32), (3, 33, 35, 3, 32),
                                        (2, 18, 67, 3, 72), (1, 9, 21, 1, 16), (1, 9, 21, 2, 16), (2, 9, 21, 4, 24)])
def test_conv3x3(dtype, stride, n, h, w, ci, o):
    """The stem's two read windows per lane (3 input channels), the border and
    the tensor's end, and the value-by-value gather of other widths."""
    rng = inputs.rng_for(h * w + ci)
    x = inputs.round_to_storage(rng.standard_normal((n, h, w, ci)), dtype)
    L = {"kind": "conv3x3", "w": inputs.round_to_storage(rng.normal(0, 0.2, (o, ci, 3, 3)), dtype),
         "b": rng.normal(0, 0.1, o).astype(np.float32), "stride": stride, "act": 2}
    want = onet.conv3x3(x.transpose(0, 3, 1, 2).astype(np.float64), L["w"], L["b"], stride, 2)
    check(run(x, [L], dtype), want.transpose(0, 2, 3, 1), dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("n,h,w", [(1, 1, 2), (1, 2, 1), (1, 1, 3), (3, 1, 1), (5, 2, 2), (7, 9, 9), (2, 4, 8), (4, 5, 15),
                                   (3, 3, 16), (6, 7, 17), (2, 1, 33), (2, 33, 1), (1, 64, 64)])
def test_stem_tiles_across_rows_and_images(dtype, stride, n, h, w):
    """Tiles of 16 positions that cross rows and images, windows that reach over
    the borders and over the tensor's first and last elements."""
    rng = inputs.rng_for(100 * h + w)
    x = inputs.round_to_storage(rng.standard_normal((n, h, w, 3)), dtype)
    L = {"kind": "conv3x3", "w": inputs.round_to_storage(rng.normal(0, 0.2, (40, 3, 3, 3)), dtype),
         "b": rng.normal(0, 0.1, 40).astype(np.float32), "stride": stride, "act": 0}
    want = onet.conv3x3(x.transpose(0, 3, 1, 2).astype(np.float64), L["w"], L["b"], stride, 0)
    check(run(x, [L], dtype), want.transpose(0, 2, 3, 1), dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("c", [8, 24, 32, 40, 64, 72, 96, 104, 128, 136, 224, 256, 264, 288, 512, 520])
def test_conv1x1_tile_rings(dtype, c):
    """One to seventeen contraction steps: rings as short as the contraction, the
    longest ring's full rounds and remainders; a partial last tile of outputs."""
    rng = inputs.rng_for(c)
    x = inputs.round_to_storage(rng.standard_normal((1, 5, 7, c)), dtype)
    L = {"kind": "conv1x1", "w": inputs.round_to_storage(rng.normal(0, 0.05, (88, c)), dtype),
         "b": rng.normal(0, 0.1, 88).astype(np.float32), "act": 0}
    want = x.reshape(-1, c).astype(np.float64) @ L["w"].astype(np.float64).T + L["b"]
    check(run(x, [L], dtype), want.reshape(1, 5, 7, 88), dtype)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("n,c,o", [(1024, 24, 64), (1025, 24, 64), (3072, 24, 64), (3073, 24, 64), (4096, 40, 64),
                                   (4097, 40, 64), (4096, 32, 72), (4096, 16, 16), (16 * 1024, 16, 16)])
def test_conv1x1_on_both_sides_of_the_tile_kernel(dtype, n, c, o):
    rng = inputs.rng_for(n + c)
    x = inputs.round_to_storage(rng.standard_normal((n, 1, 1, c)), dtype)
    L = {"kind": "conv1x1", "w": inputs.round_to_storage(rng.normal(0, 0.05, (o, c)), dtype),
         "b": rng.normal(0, 0.1, o).astype(np.float32), "act": 2}
    want = np.clip(x.reshape(-1, c).astype(np.float64) @ L["w"].astype(np.float64).T + L["b"], 0.0, 6.0)
    check(run(x, [L], dtype), want.reshape(n, 1, 1, o), dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("n,h,w,c", [(1, 3, 64, 8), (2, 9, 41, 32), (40, 21, 40, 40), (9, 30, 88, 96), (3, 5, 60, 144),
                                     (30, 27, 70, 32)])
def test_depthwise_weights_through_lds(dtype, stride, n, h, w, c):
    """Few weights per working lane: staged per workgroup, 1, 2 and 4 rows per task."""
    rng = inputs.rng_for(n * h + c)
    x = inputs.round_to_storage(rng.standard_normal((n, h, w, c)), dtype)
    L = {"kind": "block", "stride": stride, "acts": (2, 1, 0), "w1": None, "b1": None,
         "w2": inputs.round_to_storage(rng.normal(0, 0.3, (c, 9)), dtype), "b2": rng.normal(0, 0.1, c).astype(np.float32),
         "w3": inputs.round_to_storage(rng.normal(0, 0.2, (16, c)), dtype), "b3": rng.normal(0, 0.1, 16).astype(np.float32)}
    want = onet.dense_block(x.transpose(0, 3, 1, 2).astype(np.float64), L)
    check(run(x, [L], dtype), want.transpose(0, 2, 3, 1), dtype)
