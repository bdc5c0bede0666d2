"""LceQuantize and LceDequantize where a row's words start anywhere in the
float stream: every pass and chunk edge, rows shorter than a word, longer than
a pass, and pointers at every 4-byte offset, against numpy and bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (rows, channels): one word per row and less, several, words past a pass of
# 1024 (33*47 words a row), a multiple of 32 (general path by alignment only)
SHAPES = [(1, 1), (5, 1), (4097, 3), (1, 31), (3000, 33), (777, 72), (40, 100), (3, 48257),
          (9, 4095), (2, 4097), (65, 64), (70001, 7), (1, 65537)]


# on either side of what picks a kernel: few channels and rows (bitpack), floats
# and channels (dequantize; rows of whole four floats, rows that cut them, rows
# longer than a workgroup's pass, two channels)
LARGE = [(40001, 12), (100001, 12), (449390, 7), (449389, 7), (1500000, 3), (101945, 72),
         (101944, 72), (863534, 17), (863533, 17), (2, 3670016), (3, 4900003), (2000001, 17),
         (16777217, 2)]


@pytest.mark.parametrize("rows,channels,offset",
                         [(r, c, o) for r, c in SHAPES for o in range(4)] +
                         [(r, c, o) for r, c in LARGE for o in (0, 1)])
def test_codec_edges(rows, channels, offset):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2011_09398_amd as lce
    rng = np.random.default_rng(rows * 7919 + channels)
    x = rng.standard_normal((rows, channels), dtype=np.float32)
    x.flat[:4] = np.array([-0.0, np.nan, -np.inf, np.inf], np.float32)[:min(4, x.size)]
    neg = np.zeros((rows, lce.packed_words(channels) * 32), np.uint8)
    neg[:, :channels] = x < 0
    want = np.packbits(neg, axis=1, bitorder="little").view(np.uint32)

    room = torch.full((x.size + 8,), -1.0, device="cuda")    # neighbours that would set bits
    xd = room[offset:offset + x.size].view(rows, channels)
    xd.copy_(torch.from_numpy(x))
    words = torch.full((want.size + 2,), 0x55555555, dtype=torch.int32, device="cuda")
    packed = lce.bitpack(xd, out=words[1:-1].view(rows, -1))
    torch.cuda.synchronize()
    got = words.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[1:-1].reshape(want.shape), want)
    assert got[0] == got[-1] == 0x55555555                    # nothing written around them

    back = torch.full((x.size + 8,), 7.0, device="cuda")
    y = lce.dequantize(packed, channels, out=back[offset:offset + x.size].view(rows, channels))
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), np.where(x < 0, np.float32(-1), np.float32(1)))
    outside = torch.cat([back[:offset], back[offset + x.size:]])
    assert bool((outside == 7.0).all())
