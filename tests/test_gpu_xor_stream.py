"""lce_bconv2d on shapes without a specialized XOR/POPCOUNT instance, forced onto
either of its routes and checked, by the schedule that ran, to have taken it:
the streaming matrix-core schedule on the packed filters as they are stored, over
every tile, and the generic XOR kernel.  All three kinds of output, bit for bit
against the oracle (float within one rounding): odd and even word counts, every
load width, both padding values, strides, VALID, 1x1, even and large windows,
filters that fill no block, and several tiles per workgroup."""
import numpy as np
import pytest

import oracle
from tests.layer_util import assert_match, clamp_of, dev, oracle_signs
from workloads import Layer, make_layer_inputs

pytestmark = pytest.mark.gpu

LAYERS = [
    Layer("cw7-s2", 3, 25, 31, 200, 136, stride=2, out="float"),
    Layer("cw7-bits", 2, 14, 13, 215, 75, out="bitpacked", clamp=(-500, 3)),
    Layer("cw12", 2, 21, 23, 384, 264, out="bitpacked", clamp=(-900, 800)),
    Layer("cw9", 3, 12, 17, 288, 100, out="int32"),
    Layer("cw10", 2, 13, 12, 320, 64, out="bitpacked"),
    Layer("cw1-7x7", 2, 40, 41, 30, 30, kh=7, kw=7, out="bitpacked"),
    Layer("cw2-4x4-s3", 2, 22, 20, 64, 40, kh=4, kw=4, stride=3, out="int32"),
    Layer("cw3-2x3", 4, 15, 20, 70, 320, kh=2, kw=3, out="float"),
    Layer("cw2-columns", 1, 5, 300, 64, 33, kh=2, kw=2, out="float", clamp=(0, 100)),
    Layer("pointwise", 3, 20, 21, 256, 500, kh=1, kw=1, out="bitpacked"),
    Layer("pointwise-odd", 3, 20, 21, 350, 30, kh=1, kw=1, out="int32"),
    Layer("pointwise-s2", 3, 20, 21, 128, 72, kh=1, kw=1, stride=2, out="bitpacked"),
    Layer("valid-5x5", 2, 20, 21, 220, 96, kh=5, kw=5, padding="valid", out="float"),
    Layer("valid-1x3", 2, 9, 40, 64, 20, kh=1, kw=3, padding="valid", out="bitpacked"),
    Layer("small", 1, 5, 6, 200, 33, out="int32"),
]
# (32-pixel blocks per wave, 32-filter blocks per workgroup); 0, 0: the planner's
TILES = [(0, 0), (2, 2), (2, 4), (2, 8), (4, 1), (4, 2), (4, 4), (4, 8)]
# regions of 512 pixels that do not fit the LDS: the XOR kernel takes them
TOO_LARGE = [("cw7-s2", (4, 1)), ("cw7-s2", (4, 2))]
FLIP = 7919


def run_and_check(layer, pad_value, want, **keys):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_09398_amd as lce
    inp = make_layer_inputs(layer, 51, 90, 0)
    x, w = lce.bitpack(dev(inp.x_float)), lce.bitpack(dev(inp.w_float))
    kw = dict(stride=layer.strides, padding=layer.padding, pad_value=pad_value,
              clamp=layer.clamp, out_type=layer.out,
              pad_correction=lce.pad_correction(w, layer.c_in))
    per_channel = None
    if layer.out == "float":
        kw.update(multiplier=dev(inp.mult), bias=dev(inp.bias))
    elif layer.out == "bitpacked":
        flip = np.arange(1, lce.packed_words(layer.c_out) + 1, dtype=np.int32) * FLIP
        co = np.arange(layer.c_out)
        per_channel = (flip[co // 32] >> (co % 32)) & 1
        kw.update(thresholds=dev(inp.thr), flip=dev(flip))
    ref = oracle.bconv2d(oracle_signs(inp), inp.w_sign, stride=layer.strides,
                         padding=layer.padding, clamp_range=clamp_of(layer), out=layer.out,
                         mult=inp.mult, bias=inp.bias, thr=inp.thr, flip=per_channel,
                         pad_value=0 if pad_value == "zero" else 1)
    with lce.tuning(**keys):
        got = lce.bconv2d(x, w, layer.c_in, **kw)
        assert lce.last_schedule() == want
    torch.cuda.synchronize()
    assert_match(layer, got.cpu().numpy(), ref, f"{layer.name} {pad_value} {keys}")


@pytest.mark.parametrize("pad_value", ["one", "zero"])
@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"{t[0]}x{t[1]}")
@pytest.mark.parametrize("layer", LAYERS, ids=lambda l: l.name)
def test_stored_filters_on_the_matrix_cores(layer, tile, pad_value):
    want = "xor-generic" if (layer.name, tile) in TOO_LARGE else "streaming-stored"
    run_and_check(layer, pad_value, want, xor_stream=1, mfma_tile_m=tile[0],
                  mfma_tile_n=tile[1])


@pytest.mark.parametrize("pad_value", ["one", "zero"])
@pytest.mark.parametrize("layer", LAYERS, ids=lambda l: l.name)
def test_generic_xor_kernel(layer, pad_value):
    run_and_check(layer, pad_value, "xor-generic", xor_stream=-1)


@pytest.mark.parametrize("layer", [
    Layer("rows", 90, 14, 14, 224, 256, out="bitpacked"),
    Layer("pointwise", 6, 53, 59, 64, 256, kh=1, kw=1, out="float"),
    Layer("columns", 1, 70, 310, 32, 72, kh=2, kw=3, out="int32"),
], ids=lambda l: l.name)
def test_several_tiles_per_workgroup(layer):
    """64-pixel tiles, one workgroup per CU: more tiles than workgroups."""
    assert layer.m > 64 * 256 * 1.02
    run_and_check(layer, "one", "streaming-stored", xor_stream=1, mfma_tile_m=2, mfma_tile_n=8,
                  mfma_fs_wpc=1)


def test_bits_past_the_channels_count_alike_on_both_routes():
    """Set bits past C_in, which the header rules out, count on both routes."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_09398_amd as lce
    layer = Layer("p", 2, 9, 13, 200, 64, out="int32")
    inp = make_layer_inputs(layer, 52, 90, 1)
    x, w = lce.bitpack(dev(inp.x_float)), lce.bitpack(dev(inp.w_float))
    x[..., -1] |= -1 << 8
    outs = []
    for route in (1, -1):
        with lce.tuning(xor_stream=route):
            outs.append(lce.bconv2d(x, w, 200, out_type="int32"))
    assert torch.equal(outs[0], outs[1])
