"""The pixel-split schedule over large batches and few K stages, where a wave
that moves no filters of a stage must still wait for its own part of the input
region: every tile whose stages have fewer DMA instructions than waves (1 or 2
filter blocks over chunks of 2 or 4 words), over images enough that the region's
loads are slow, against the K split of the whole batch and the oracle on the
first and the last image."""
import numpy as np
import pytest

from tests.layer_util import assert_match, dev, oracle_signs
from workloads import Layer, make_layer_inputs

pytestmark = pytest.mark.gpu

LAYERS = [
    Layer("1x1", 2, 68, 138, 14, 32, kh=1, kw=1, out="int32"),
    Layer("3x1", 2, 100, 68, 41, 32, kh=3, kw=1, out="int32"),
    Layer("two-blocks", 2, 80, 90, 40, 64, kh=1, kw=1, out="bitpacked"),
    Layer("four-words", 2, 66, 70, 100, 30, kh=1, kw=1, out="bitpacked"),
    Layer("four-words-2x2", 2, 66, 70, 128, 20, kh=2, kw=2, out="int32"),
    Layer("float", 2, 68, 138, 33, 32, kh=1, kw=2, out="float"),
]


@pytest.mark.parametrize("pad_value", ["one", "zero"])
@pytest.mark.parametrize("layer", LAYERS, ids=lambda l: l.name)
def test_every_wave_waits_for_its_region(layer, pad_value):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    import paper_2011_09398_amd as lce
    inp = make_layer_inputs(layer, 61, 90, 0)
    few = lce.bitpack(dev(inp.x_float))
    n = 2_000_000 // (layer.h * layer.w) // 2 * 2
    x = few.repeat(n // 2, 1, 1, 1)
    # other images between the first two and the last two
    g = torch.Generator("cuda").manual_seed(7)
    x[2:-2] = x[2:-2].flatten()[torch.randperm(x[2:-2].numel(), device="cuda", generator=g)].view_as(x[2:-2])
    w = lce.bitpack(dev(inp.w_float))
    wf = lce.mfma_weights(w, layer.c_in)
    kw = dict(pad_value=pad_value, out_type=layer.out)
    if layer.out == "float":
        kw.update(multiplier=dev(inp.mult), bias=dev(inp.bias))
    elif layer.out == "bitpacked":
        kw.update(thresholds=dev(inp.thr))
    run = lambda: lce.bconv2d_mfma(x, wf, layer.c_in, layer.c_out, (layer.kh, layer.kw), **kw)
    with lce.tuning(mfma_schedule="ksplit"):
        want = run()
    ref = oracle.bconv2d(oracle_signs(inp), inp.w_sign, out=layer.out, mult=inp.mult,
                         bias=inp.bias, thr=inp.thr, pad_value=0 if pad_value == "zero" else 1)
    for tile in (0, 1, 2):
        for _ in range(3):
            with lce.tuning(mfma_schedule="pixel", mfma_tile_m=tile):
                got = run()
            torch.cuda.synchronize()
            assert torch.equal(got, want), f"{layer.name} {pad_value} tile {tile}"
    for images in (slice(0, 2), slice(-2, None)):
        assert_match(layer, got[images].cpu().numpy(), ref, layer.name)
