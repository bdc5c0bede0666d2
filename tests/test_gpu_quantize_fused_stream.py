"""GPU parity of the quantize-fused streaming schedule (float32 input) against
lce_bitpack and lce_bconv2d_mfma and the oracle: rows of fewer words than a
wave's 64 and of several segments, column tiles, image boundaries inside a
tile, both padding values, strides, 1x1 filters as one row of pixels, several
tiles per workgroup, and the sign test's special values."""
import numpy as np
import pytest

from tests.layer_util import assert_match, dev, oracle_signs
from tests.test_gpu_mfma import oracle_run, sync_np
from workloads import Layer, make_layer_inputs

pytestmark = pytest.mark.gpu

LAYERS = [
    Layer("rows", 5, 14, 14, 256, 96, out="bitpacked", clamp=(-500, 3), input_kind="float"),
    Layer("short", 3, 7, 7, 512, 130, out="float", input_kind="float"),
    Layer("columns", 2, 9, 131, 64, 72, out="int32", input_kind="float"),
    Layer("one-word", 2, 17, 19, 32, 33, out="bitpacked", input_kind="float"),
    Layer("odd-words", 2, 13, 12, 96, 64, kh=5, kw=5, out="float", input_kind="float"),
    Layer("stride2", 3, 15, 22, 128, 100, stride=2, out="bitpacked", input_kind="float"),
    Layer("strided-above", 3, 13, 16, 640, 64, kh=2, kw=1, stride=3, out="int32",
          input_kind="float"),
    Layer("pointwise", 3, 11, 13, 1280, 100, kh=1, kw=1, out="bitpacked", input_kind="float"),
    Layer("valid", 2, 16, 40, 160, 64, padding="valid", out="bitpacked", input_kind="float"),
    Layer("several-tiles", 90, 14, 14, 64, 256, out="bitpacked", input_kind="float"),
]


@pytest.mark.parametrize("tile", [(0, 0), (2, 8), (4, 2)], ids=lambda t: f"{t[0]}x{t[1]}")
@pytest.mark.parametrize("pad_value", ["one", "zero"])
@pytest.mark.parametrize("layer", LAYERS, ids=lambda l: l.name)
def test_quantize_stream(layer, pad_value, tile):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_09398_amd as lce
    if tile == (4, 2) and layer.c_in >= 512:
        pytest.skip("the region of 512 pixels does not fit the LDS at this depth")
    inp = make_layer_inputs(layer, 41, 90, 0)
    x = inp.x_float
    x.flat[:6] = np.array([-0.0, 0.0, np.nan, -np.nan, -np.inf, np.inf], np.float32)
    kw = dict(stride=layer.strides, padding=layer.padding, pad_value=pad_value,
              clamp=layer.clamp, out_type=layer.out)
    if layer.out == "float":
        kw.update(multiplier=dev(inp.mult), bias=dev(inp.bias))
    elif layer.out == "bitpacked":
        kw.update(thresholds=dev(inp.thr))
    xd, wp = dev(x), lce.bitpack(dev(inp.w_float))
    wf = lce.mfma_weights(wp, layer.c_in)
    kernel = (layer.kh, layer.kw)
    lce.set_tuning(mfma_schedule="stream", mfma_tile_m=tile[0], mfma_tile_n=tile[1],
                   mfma_fs_wpc=1 if layer.name == "several-tiles" else 0)
    got = lce.quantize_bconv2d_mfma(xd, wf, layer.c_out, kernel, **kw)
    lce.set_tuning(**{k: 0 for k in lce.TUNING_KEYS})
    two = lce.bconv2d_mfma(lce.bitpack(xd), wf, layer.c_in, layer.c_out, kernel, **kw)
    torch.cuda.synchronize()
    assert torch.equal(got, two)
    assert_match(layer, sync_np(got),
                 oracle_run(layer, inp, oracle_signs(inp), 0 if pad_value == "zero" else 1),
                 f"{layer.name} {pad_value}")
