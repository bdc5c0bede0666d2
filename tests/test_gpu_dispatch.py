"""Which schedule the library's own choice runs, on layers well to either side
of where the streaming schedule begins: large batches, long K and wide images on
it; small layers, and layers whose regions are mostly rows of few words, strided
columns or many loads, on the schedule that is faster there.  (Times in the
comments: streaming, chosen; microseconds on 256 CUs.)"""
import pytest

pytestmark = pytest.mark.gpu

STREAM, FS, KS, PX = "streaming", "filter-stationary", "k-split", "pixel-split"

# entry, n, h, w, c_in, c_out, kh, kw, stride, padding, out, schedule
CASES = [
    ("mfma", 256, 56, 56, 64, 64, 3, 3, 1, "same", "bitpacked", STREAM),
    ("mfma", 256, 14, 14, 256, 256, 3, 3, 1, "same", "bitpacked", STREAM),
    ("mfma", 256, 28, 28, 256, 512, 1, 1, 1, "same", "bitpacked", STREAM),
    ("mfma", 32, 64, 64, 256, 256, 5, 5, 1, "same", "float", STREAM),
    ("mfma", 2, 360, 640, 64, 64, 3, 3, 1, "same", "float", STREAM),
    ("quant", 128, 28, 28, 128, 128, 3, 3, 1, "same", "float", STREAM),
    ("xor", 64, 45, 61, 200, 136, 3, 3, 2, "same", "float", "streaming-stored"),
    ("xor", 256, 28, 28, 256, 512, 1, 1, 1, "same", "bitpacked", "streaming-stored"),
    ("mfma", 1, 56, 56, 64, 64, 3, 3, 1, "same", "bitpacked", FS),
    ("mfma", 162, 10, 11, 736, 564, 3, 1, 3, "valid", "bitpacked", KS),     # 62.8, 24.7
    ("mfma", 314, 31, 11, 416, 128, 2, 2, 3, "same", "bitpacked", KS),      # 46.8, 19.3
    ("mfma", 43, 62, 51, 448, 32, 2, 3, 3, "same", "int32", KS),            # 35.7, 17.1
    ("mfma", 202, 125, 4, 31, 640, 3, 1, 3, "same", "bitpacked", PX),       # 18.9, 10.9
    ("mfma", 100, 16, 13, 32, 75, 5, 5, 2, "same", "float", KS),            # 9.3, 5.7
    ("quant", 113, 26, 5, 384, 134, 7, 7, 2, "same", "float", KS),          # 56.0, 30.8
    ("xor", 379, 5, 83, 416, 32, 2, 2, 1, "same", "int32", "xor-generic"),  # 59.4, 41.8
    ("xor", 4, 20, 20, 64, 64, 3, 3, 1, "same", "float", "xor"),
    ("xor", 1, 5, 6, 200, 33, 3, 3, 1, "same", "int32", "xor-generic"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_schedule_of_the_library_s_choice(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are for 256 CUs")
    import paper_2011_09398_amd as lce
    entry, n, h, w, c_in, c_out, kh, kw, stride, padding, out, want = case
    words = lambda *shape: torch.zeros(shape, dtype=torch.int32, device="cuda")
    cw = lce.packed_words(c_in)
    filters = words(c_out, kh, kw, cw)
    per_channel = torch.zeros(c_out, device="cuda")
    args = dict(stride=stride, padding=padding, out_type=out)
    if out == "bitpacked":
        args.update(thresholds=per_channel)
    elif out == "float":
        args.update(multiplier=per_channel, bias=per_channel)
    if entry == "xor":
        lce.bconv2d(words(n, h, w, cw), filters, c_in, **args)
    elif entry == "mfma":
        lce.bconv2d_mfma(words(n, h, w, cw), lce.mfma_weights(filters, c_in), c_in, c_out,
                         (kh, kw), **args)
    else:
        lce.quantize_bconv2d_mfma(torch.zeros(n, h, w, c_in, device="cuda"),
                                  lce.mfma_weights(filters, c_in), c_out, (kh, kw), **args)
    assert lce.last_schedule() == want
