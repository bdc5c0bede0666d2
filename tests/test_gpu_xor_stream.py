"""lce_bconv2d on shapes without a specialized XOR/POPCOUNT instance: large
ones run the streaming matrix-core schedule on the packed filters as they are
stored, small ones the generic XOR kernel, which the tuning keys also force.
Both routes give the oracle's integers, for odd and even word counts, every
load width, both padding values, 1x1, even and large windows, and filters that
fill no block."""
import numpy as np
import pytest

import oracle
from tests.layer_util import assert_match, dev, oracle_signs
from tests.test_gpu_mfma import oracle_run, sync_np
from workloads import Layer, make_layer_inputs

pytestmark = pytest.mark.gpu

LAYERS = [
    Layer("cw7-s2", 24, 45, 61, 200, 136, stride=2, out="float"),
    Layer("cw12", 4, 21, 23, 384, 264, out="bitpacked", clamp=(-900, 800)),
    Layer("cw9", 3, 30, 17, 288, 200, out="int32"),
    Layer("cw1-7x7", 6, 40, 41, 30, 250, kh=7, kw=7, out="bitpacked"),
    Layer("cw3-2x3", 12, 30, 40, 70, 320, kh=2, kw=3, out="float"),
    Layer("pointwise", 12, 40, 41, 256, 500, kh=1, kw=1, out="bitpacked"),
    Layer("pointwise-odd", 12, 40, 41, 350, 300, kh=1, kw=1, out="int32"),
    Layer("valid-5x5", 8, 20, 21, 220, 96, kh=5, kw=5, padding="valid", out="float"),
    Layer("small", 1, 5, 6, 200, 33, out="int32"),
]


@pytest.mark.parametrize("pad_value", ["one", "zero"])
@pytest.mark.parametrize("layer", LAYERS, ids=lambda l: l.name)
def test_generic_shapes_both_routes(layer, pad_value):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_09398_amd as lce
    inp = make_layer_inputs(layer, 51, 90, 0)
    x, w = lce.bitpack(dev(inp.x_float)), lce.bitpack(dev(inp.w_float))
    kw = dict(stride=layer.strides, padding=layer.padding, pad_value=pad_value,
              clamp=layer.clamp, out_type=layer.out,
              pad_correction=lce.pad_correction(w, layer.c_in))
    if layer.out == "float":
        kw.update(multiplier=dev(inp.mult), bias=dev(inp.bias))
    elif layer.out == "bitpacked":
        kw.update(thresholds=dev(inp.thr),
                  flip=dev(np.arange(1, lce.packed_words(layer.c_out) + 1, dtype=np.int32) * 7919))
    got = lce.bconv2d(x, w, layer.c_in, **kw)
    with lce.tuning(xor_nb=1):
        forced = lce.bconv2d(x, w, layer.c_in, **kw)
    torch.cuda.synchronize()
    assert torch.equal(got, forced)
    if layer.out != "bitpacked":
        assert_match(layer, sync_np(got),
                     oracle_run(layer, inp, oracle_signs(inp), 0 if pad_value == "zero" else 1),
                     f"{layer.name} {pad_value}")
