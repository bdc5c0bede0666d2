"""GPU parity of the streaming matrix-core schedule against the oracle.

int32 and bitpacked outputs bit for bit, float outputs within 1e-6 relative
(one fused multiply-add of an exact integer).  Shapes sit where the schedule
can go wrong: tiles of whole rows that cross image boundaries, column tiles
with a partial last one, several tiles per workgroup, 1x1 filters (the batch
as one row), two short rows per load and several loads per row, every word
count per load (4, 2, 1, by shape and by alignment), channels that fill no
word under both padding values, strides above the window, and filters that
fill no tile.
"""
import numpy as np
import pytest

import oracle
from tests.layer_util import assert_match, dev, oracle_signs
from tests.test_gpu_mfma import mfma_cases, mfma_run, oracle_run, sync_np
from workloads import Layer, make_layer_inputs

pytestmark = pytest.mark.gpu

# (32-pixel blocks per wave, 32-filter blocks per workgroup)
TILES = [(0, 0), (2, 2), (2, 4), (2, 8), (4, 1), (4, 2), (4, 4), (4, 8)]


@pytest.fixture(autouse=True)
def stream():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_09398_amd as lce
    lce.set_tuning(**{k: 0 for k in lce.TUNING_KEYS})
    lce.set_tuning(mfma_schedule="stream")
    yield lce


EDGES = [
    Layer("rows-cross-images", 5, 14, 14, 256, 96, out="bitpacked", clamp=(-500, 3)),
    Layer("rows-cross-two", 9, 3, 5, 64, 64, out="int32"),
    Layer("short-rows", 3, 7, 7, 512, 130, out="bitpacked"),
    Layer("columns", 2, 9, 131, 64, 72, out="float", clamp=(0, 576)),
    Layer("columns-bits", 1, 5, 300, 33, 40, out="bitpacked"),
    Layer("wide-words", 1, 6, 150, 256, 32, out="int32"),
    Layer("odd-words", 2, 17, 19, 96, 33, kh=5, kw=5, out="float"),
    Layer("partial-word", 2, 12, 13, 45, 64, out="bitpacked"),
    Layer("stride2", 3, 15, 22, 128, 100, stride=2, out="float"),
    Layer("stride-above-window", 3, 13, 16, 64, 64, kh=2, kw=1, stride=3, out="int32"),
    Layer("pointwise", 3, 11, 13, 200, 100, kh=1, kw=1, out="bitpacked"),
    Layer("pointwise-strided", 3, 11, 14, 64, 32, kh=1, kw=1, stride=2, out="float"),
    Layer("valid", 2, 16, 40, 160, 64, padding="valid", out="bitpacked"),
    Layer("one-pixel", 1, 1, 1, 32, 1, out="int32"),
]


@pytest.mark.parametrize("pad_value", ["one", "zero"])
@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"{t[0]}x{t[1]}")
@pytest.mark.parametrize("layer", EDGES, ids=lambda l: l.name)
def test_stream_edges(stream, layer, tile, pad_value):
    stream.set_tuning(mfma_tile_m=tile[0], mfma_tile_n=tile[1])
    inp = make_layer_inputs(layer, 31, 90, 0)
    ref = oracle_run(layer, inp, oracle_signs(inp), 0 if pad_value == "zero" else 1)
    assert_match(layer, sync_np(mfma_run(layer, inp, pad_value=pad_value)), ref,
                 f"{layer.name} {tile} {pad_value}")


@pytest.mark.parametrize("pad_value", ["one", "zero"])
@pytest.mark.parametrize("layer", mfma_cases(), ids=lambda l: l.name)
def test_stream_sweep(stream, layer, pad_value):
    inp = make_layer_inputs(layer, 11, 97, int(layer.name[2:]))
    ref = oracle_run(layer, inp, oracle_signs(inp), 0 if pad_value == "zero" else 1)
    assert_match(layer, sync_np(mfma_run(layer, inp, pad_value=pad_value)), ref,
                 f"{layer.name} {pad_value}")


@pytest.mark.parametrize("layer", [
    Layer("rows", 90, 14, 14, 64, 256, out="bitpacked"),
    Layer("columns", 1, 70, 310, 32, 250, out="int32"),
    Layer("pointwise", 7, 53, 59, 64, 256, kh=1, kw=1, out="float"),
], ids=lambda l: l.name)
def test_stream_several_tiles_per_workgroup(stream, layer):
    """More tiles than workgroups: each takes the next tile's region while the
    current one's products run.  (64-pixel tiles, one workgroup per CU.)"""
    assert layer.m > 64 * 256 * 1.02
    stream.set_tuning(mfma_tile_m=2, mfma_tile_n=8, mfma_fs_wpc=1)
    inp = make_layer_inputs(layer, 32, 90, 1)
    ref = oracle_run(layer, inp, oracle_signs(inp))
    for _ in range(2):
        assert_match(layer, sync_np(mfma_run(layer, inp)), ref, layer.name)


@pytest.mark.parametrize("offset", [1, 2])
@pytest.mark.parametrize("c_in", [64, 128])
def test_stream_input_alignment(stream, c_in, offset):
    """An input 4 or 8 bytes past a 16-byte boundary takes narrower loads; an
    output 4 bytes past an 8-byte one single-word stores."""
    import torch
    layer = Layer("a", 2, 10, 11, c_in, 128, out="bitpacked")
    inp = make_layer_inputs(layer, 33, 90, 2)
    words = stream.bitpack(dev(inp.x_float))
    room = torch.empty(words.numel() + 4, dtype=torch.int32, device="cuda")
    x = room[offset:offset + words.numel()].view(words.shape)
    x.copy_(words)
    wp = stream.bitpack(dev(inp.w_float))
    out_room = torch.empty(layer.m * 4 + 4, dtype=torch.int32, device="cuda")
    out = out_room[offset:offset + layer.m * 4].view(2, 10, 11, 4)
    stream.bconv2d_mfma(x, stream.mfma_weights(wp, c_in), c_in, 128, 3, out_type="bitpacked",
                        thresholds=dev(inp.thr), out=out)
    assert_match(layer, sync_np(out), oracle_run(layer, inp, oracle_signs(inp)), "alignment")


def test_stream_thresholds_and_flip(stream):
    """Infinite, NaN, huge and out-of-clamp thresholds, with a flip mask whose
    bits past C_out are set."""
    layer = Layer("t", 1, 9, 10, 40, 45, out="bitpacked", clamp=(-90, 100))
    inp = make_layer_inputs(layer, 34, 90, 3)
    thr = inp.thr.copy()
    thr[:10] = [np.inf, -np.inf, np.nan, 3e9, -3e9, 101, 100, -90, -89.5, 0.5]
    flip = np.array([0x2AAAAAAA, 0x7FFFFFFF], np.int32)
    per_channel = (flip[np.arange(45) // 32] >> (np.arange(45) % 32)) & 1
    ref = oracle.bconv2d(oracle_signs(inp), inp.w_sign, clamp_range=layer.clamp,
                         out="bitpacked", thr=thr, flip=per_channel)
    got = sync_np(mfma_run(layer, inp, thresholds=thr, flip=flip))
    assert_match(layer, got, ref, "thresholds and flip")


def test_stream_is_chosen_and_agrees(stream):
    """Layers that the library's own choice runs on this schedule (large batches;
    short and long K), and one of long shares that it leaves to another: equal to
    the K split and the pixel split, bit for bit."""
    import torch
    for n, h, c_in, c_out, k, chosen in ((256, 14, 256, 256, 3, True), (300, 28, 64, 256, 1, True),
                                         (150, 13, 96, 128, 5, True), (20, 14, 256, 64, 3, False)):
        g = torch.Generator("cuda").manual_seed(5)
        xp = stream.bitpack(torch.randn(n, h, h, c_in, device="cuda", generator=g))
        wp = stream.bitpack(torch.randn(c_out, k, k, c_in, device="cuda", generator=g))
        wf = stream.mfma_weights(wp, c_in)
        outs = []
        for sched, name in (("auto", "streaming" if chosen else "filter-stationary"),
                            ("stream", "streaming"), ("ksplit", "k-split"),
                            ("pixel", "pixel-split")):
            stream.set_tuning(mfma_schedule=sched)
            outs.append(stream.bconv2d_mfma(xp, wf, c_in, c_out, k, out_type="int32"))
            assert stream.last_schedule() == name, (n, h, c_in, c_out, k, sched)
        for o in outs[1:]:
            assert torch.equal(outs[0], o)


@pytest.mark.parametrize("out", ["int32", "bitpacked"])
@pytest.mark.parametrize("pad_value", ["one", "zero"])
@pytest.mark.parametrize("c_in", [45, 70, 100])
@pytest.mark.parametrize("sched", ["auto", "fs", "ksplit", "pixel", "stream"])
def test_input_bits_past_the_channels_count_nothing(stream, sched, c_in, pad_value, out):
    """The widened filters hold 0.0 there, so bits of x_packed past C_in do not
    reach any dot, whichever schedule runs (1, 2 and 4 words per region load)."""
    stream.set_tuning(mfma_schedule=sched)
    layer = Layer("p", 2, 9, 13, c_in, 64, out=out)
    inp = make_layer_inputs(layer, 35, 90, 4)
    words = stream.bitpack(dev(inp.x_float))
    words[..., -1] |= -1 << (c_in % 32)
    ref = oracle_run(layer, inp, oracle_signs(inp), 0 if pad_value == "zero" else 1)
    got = sync_np(mfma_run(layer, inp, pad_value=pad_value, x_packed=words))
    assert_match(layer, got, ref, f"{sched} {c_in} {pad_value}")
