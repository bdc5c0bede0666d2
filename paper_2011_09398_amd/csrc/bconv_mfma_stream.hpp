// Streaming schedule of the matrix-core convolution (bconv_mfma.hpp has the
// arithmetic), for layers of many pixels, any K and any width.
//
// A workgroup (4 waves) takes tiles of 32*MB*(4/wf) pixels x 32*NB*wf filters
// one after another (persistent: about as many workgroups as fit the CUs).
// Each wave computes MB x NB blocks of 32x32 over all of K.
//   * A: the tile's input region is loaded into registers, widened once into
//     LDS (every word of every location), and read from there K step by K
//     step, one 1 KB operand per NB products (NB = 2 leaves the LDS at half
//     its rate).  The next tile's loads are issued before this tile's
//     products, so that they arrive behind them.
//   * B: the packed copy of the filters, a dword per lane, block and K step,
//     from L2 four K steps ahead, widened in registers.  A filter word is
//     widened once per MB products (7 ALU operations to MB * 32 cycles of the
//     matrix pipe), so no filter has to stay in registers and K is unbounded:
//     the filter-stationary schedule ends at 72 K steps, and its share of
//     pixels grows with the batch until its region no longer fits the LDS.
//   * The loop issues at most three ALU operations between two products: the
//     pipe takes one product per 32 cycles, and up to about six ALU
//     operations (5 cycles each, 8 where one waits for the other) hide behind
//     it; a group of fourteen between two K steps did not (K step 430 -> 320
//     cycles with one wave per SIMD; 256 is the pipe's rate).
//   * A tile is whole output rows where those fill it, else 32*k columns of
//     several rows, so that wide images stage 3 x 34 locations and not whole
//     rows, and the 32 pixels of a block are always consecutive in memory.
//   * Channels past C_in: their bits are 0 in both operands (masked off the
//     input's last word, where the widened filters of the other schedules hold
//     0.0), widen to +1.0 on both sides and add the same to every dot; that sum
//     is taken out at the end (or of the threshold).  So the packed filters
//     serve every C_in.
//
// Measured (us; the schedule that took the layer before, and this one):
// 56x56x64->64 batch 256 44.9 -> 21.5, 14x14x256 batch 256 42 -> 15.8,
// 7x7x512 batch 256 32.7 -> 16.8, 1x1 28x28x256->512 batch 256 58 -> 30,
// 5x5 64x64x256 batch 32 (float) 156 -> 79, 3x3 360x640x64 x2 (float) 48 -> 25;
// from float32 input 56x56x64->64 batch 256 (212 MB) 65 -> 48, 28x28x128 batch
// 128 with float output (103 MB) 28.5 -> 23, 14x14x256 batch 256 90 -> 27.
// What bounds it: 56x56x64 spends 13.5K of 37K cycles per wave in the
// products (the matrix pipes are busy 34% of the time), the rest in staging,
// output and waiting, where the scalar registers that the compiler spills (76
// there) are reloaded; with long K (5x5x256, busy 71%) it is the matrix pipe at
// the clock that random +-1 data leave it (about 8 PFLOP/s in a loop of products
// alone; here 5.4 with its 134 MB of output).
#pragma once

#include "bconv_mfma.hpp"

namespace lce {

struct StreamParams : MfmaGeom {
    int32_t tiles;                   // pixel tiles of the layer
    int32_t px;                      // output pixels per tile: th rows of tw columns
    int32_t th, tw, col_tiles;       // tw = OW (col_tiles = 1) or a multiple of 32
    int32_t wf;                      // waves side by side over filters (1, 2 or 4)
    int32_t ksteps;                  // KH*KW*CwE/2
    int32_t pad_sum;                 // what the padding channels add to every dot
    int32_t plane;                   // 16-byte elements per word plane of the A tile (odd)
    int32_t row_elems;               // elements (V words) of a region row: pw * Cw/V
    int32_t row_segs, row_pair;      // 64-lane segments per row; 1: a wave loads two rows at once
    int32_t units;                   // wave loads per region
    int32_t out8;                    // 1: pairs of output words may be stored as 8 bytes
    uint32_t w_bytes;                // OHWI filters: their size and one filter's
    int32_t w_row;
    uint32_t pad_fill[4];            // widened +1.0 codes of the last word's padding channels
    uint32_t tail;                   // bits of an input location's last word that are channels
    FastDiv div_ct, div_tw, div_oh;  // column tiles, tile columns, output rows of an image
    FastDiv div_g, div_segs;         // elements per location, segments per row
};

// wave loads of the region that a wave holds in flight
constexpr int stream_reg_u(int v) { return v == 0 ? 0 : v == 1 ? 8 : 4; }

// Where a tile lies: output row rr0 of the batch = row oy0 of image img0, column x0.
struct StreamTile {
    int rr0, x0, img0, oy0;
};

template <int V>
struct StreamRegion {
    uint32_t w[V == 0 ? 1 : stream_reg_u(V) * V];
    uint32_t out;                    // bit u: the lane's element of load u lies outside the image
};

// A lane's place in segment `seg` of a region row: element e = (column c,
// word group g), g fastest (so that a wave reads consecutive bytes).
template <int V>
__device__ __forceinline__ void stream_lane(const StreamParams &p, int lane, int seg, int &c,
                                            int &g, bool &ok) {
    const int e = seg * 64 + (p.row_pair ? lane & 31 : lane);
    ok = e < p.row_elems;
    c = (int)fast_div((uint32_t)e, p.div_g);
    g = e - c * (int)p.div_g.d;
}

// Input offset of the first element of the padded row that lies `r` rows below
// the tile's first one; false where that is no image row.
__device__ __forceinline__ bool stream_row(const StreamParams &p, const StreamTile &t, int r,
                                           int &base) {
    const int P = t.oy0 * p.sh + r;
    const int k = (int)fast_div((uint32_t)P, p.div_ph);
    const int y = P - k * p.ph - p.pt, img = t.img0 + k;
    base = (img * p.h + y) * p.w * p.cw * 4;
    return img < p.n && (unsigned)y < (unsigned)p.h;
}

// Wave loads u0 .. u0 + U - 1 of this wave: rows of the region (row_segs
// segments each, or two short rows at once), so that the row's place in the
// input is wave-uniform arithmetic and a lane only adds its own offset.
template <int V>
__device__ __forceinline__ void stream_load(const StreamParams &p, const StreamTile &t, int wave,
                                            int lane, int u0, StreamRegion<V> &ch) {
    const __amdgpu_buffer_rsrc_t xb = input_buffer(p);
    ch.out = 0;
    int c, g, voff;
    bool ok;
    auto place = [&](int seg) __attribute__((always_inline)) {
        stream_lane<V>(p, lane, seg, c, g, ok);
        const int xx = t.x0 * p.sw - p.pl + c;
        voff = ok && (unsigned)xx < (unsigned)p.w ? (xx * p.cw + V * g) * 4 : kBufOutside;
    };
    if (p.row_segs == 1) place(0);
#pragma unroll
    for (int u = 0; u < stream_reg_u(V); ++u) {
        const int unit = wave + 4 * (u0 + u);
        if (unit >= p.units) continue;
        int base, off = voff;
        if (p.row_pair) {
            int base1;
            const bool in0 = stream_row(p, t, 2 * unit, base);
            const bool in1 = stream_row(p, t, 2 * unit + 1, base1);
            off = (lane < 32 ? in0 : in1) ? off + (lane < 32 ? base : base1) : kBufOutside;
            // (an outside lane offset plus a row stays past every buffer)
            base = 0;
        } else {
            int r = unit;
            if (p.row_segs > 1) {
                r = (int)fast_div((uint32_t)unit, p.div_segs);
                place(unit - r * p.row_segs);
                off = voff;
            }
            if (!stream_row(p, t, r, base)) {
                off = kBufOutside;
                base = 0;
            }
        }
        if constexpr (V == 4) {
            const auto x = __builtin_amdgcn_raw_buffer_load_b128(xb, off, base, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) ch.w[4 * u + k] = x[k];
        } else if constexpr (V == 2) {
            const auto x = __builtin_amdgcn_raw_buffer_load_b64(xb, off, base, 0);
            ch.w[2 * u] = x[0];
            ch.w[2 * u + 1] = x[1];
        } else {
            ch.w[u] = __builtin_amdgcn_raw_buffer_load_b32(xb, off, base, 0);
        }
        if (p.pad_zero) ch.out |= off < 0 ? 1u << u : 0u;
    }
}

// Widen a wave's loads into the A tile: +1.0/-1.0 from the bits, 0.0 at
// padding locations under zero padding, where the padding channels of the
// last word stay +1.0 (they add the same to every dot).  TAIL: the input's bits
// past C_in are cleared.
template <int V, bool TAIL>
__device__ __forceinline__ void stream_widen(const StreamParams &p, const StreamRegion<V> &ch,
                                             u32x4 *atile, int wave, int lane, int u0) {
    int c, g, at;
    uint32_t tail;
    bool ok;
    auto place = [&](int seg) __attribute__((always_inline)) {
        stream_lane<V>(p, lane, seg, c, g, ok);
        at = V * g * p.plane + c;
        tail = TAIL && V * g + V == p.cw ? p.tail : ~0u;
    };
    if (p.row_segs == 1) place(0);
#pragma unroll
    for (int u = 0; u < stream_reg_u(V); ++u) {
        const int unit = wave + 4 * (u0 + u);
        if (unit >= p.units) break;
        int r = unit;
        if (p.row_pair) {
            r = 2 * unit + (lane >> 5);
        } else if (p.row_segs > 1) {
            r = (int)fast_div((uint32_t)unit, p.div_segs);
            place(unit - r * p.row_segs);
        }
        if (ok && r < p.tile_rows) {
            const bool zero = p.pad_zero && ((ch.out >> u) & 1u);
            const uint32_t fill = zero ? 0u : kFp4PlusOne;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const uint32_t w = k == V - 1 ? ch.w[V * u + k] & tail : ch.w[V * u + k];
                u32x4 o = widen_word(w, fill);
                if (k == V - 1 && zero && V * g + V == p.cw)
                    o = u32x4{p.pad_fill[0], p.pad_fill[1], p.pad_fill[2], p.pad_fill[3]};
                atile[at + r * p.pw + k * p.plane] = o;
            }
        }
    }
}

// LceQuantize fused into the staging: the input is float32, and a wave packs 64
// words (8 KiB) at a time, eight loads of 1 KiB each, consecutive lanes on
// consecutive 16 bytes.  A lane's four signs make a nibble (x < 0, the bitpack
// kernel's test), three DPP ORs the word of its eight lanes, and lane 8g + k
// keeps word 8k + g of the 64, widens it and writes it to the A tile.  (Giving a lane the 128 bytes of a word, as
// the other schedules do, touches 64 cache lines per load instruction: the
// 56x56x64->64 layer at batch 256, 205 MB in, 65 us there, 48 here.)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

__device__ __forceinline__ void stream_quantize(const StreamParams &p, const StreamTile &t,
                                                u32x4 *atile, int wave, int lane) {
    const __amdgpu_buffer_rsrc_t xb =
        buffer_of(p.x, (uint32_t)p.n * p.h * p.w * p.cw * 128u);
    const int k8 = lane & 7, g8 = lane >> 3;
    const int first = (t.x0 * p.sw - p.pl) * p.cw;       // the region row's first word in its image row
    const int row_words = p.w * p.cw;
    for (int unit = wave; unit < p.units; unit += 4) {
        const int r = (int)fast_div((uint32_t)unit, p.div_segs);
        const int e0 = (unit - r * p.row_segs) * 64;
        int base;
        const bool row_in = stream_row(p, t, r, base);   // (bytes of packed words; floats: 32 times)
        uint32_t word = 0;
        if (row_in) {
            f32x4_t v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int e = e0 + 8 * k + g8;
                const bool in = e < p.row_elems && (unsigned)(first + e) < (unsigned)row_words;
                const auto x = __builtin_amdgcn_raw_buffer_load_b128(
                    xb, in ? (first + e) * 128 + k8 * 16 : kBufOutside, base * 32, 0);
                v[k] = f32x4_t{__uint_as_float(x[0]), __uint_as_float(x[1]),
                               __uint_as_float(x[2]), __uint_as_float(x[3])};
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const f32x4_t f = v[k];
                uint32_t s = ((uint32_t)(f.x < 0.0f) | ((uint32_t)(f.y < 0.0f) << 1) |
                              ((uint32_t)(f.z < 0.0f) << 2) | ((uint32_t)(f.w < 0.0f) << 3))
                             << (4 * k8);
                s |= dpp_move<0xB1>(s);                  // quad_perm [1,0,3,2]
                s |= dpp_move<0x4E>(s);                  // quad_perm [2,3,0,1]
                s |= dpp_move<0x141>(s);                 // row_half_mirror
                word = k8 == k ? s : word;
            }
        }
        const int e = e0 + 8 * k8 + g8;
        if (e < p.row_elems) {
            const int c = (int)fast_div((uint32_t)e, p.div_g), j = e - c * p.cw;
            const bool in = row_in && (unsigned)(first + e) < (unsigned)row_words;
            atile[j * p.plane + r * p.pw + c] =
                widen_word(word, p.pad_zero && !in ? 0u : kFp4PlusOne);
        }
    }
}

// OUT: output kind.  MB x NB blocks of 32 pixels x 32 filters per wave; p.wf of the four waves
// side by side over filters, the others over pixels.  V: words per region load,
// 0 for a float32 input.  OHWI: p.wpk is the packed filter tensor itself
// ([C_out][taps][Cw]); a lane then reads its filter's own words (a 64-byte line
// serves eight K steps from the L1), and the word past an odd Cw, which belongs
// to the next tap, is cleared; every bit of an input word counts, as in the XOR
// kernels (the mask there measured 31.0 -> 32.8 us on 3x3/2 200->136).
template <int OUT, int MB, int NB, int V, bool OHWI = false>
__global__ __launch_bounds__(kMfmaThreads, MB * NB <= 4 ? 3 : 2) void bconv2d_mfma_stream_kernel(
    StreamParams p) {
    constexpr int RB = 4;                                // packed filters in flight (K steps)
    extern __shared__ __attribute__((aligned(16))) u32x4 smem[];
    fetch_arg_lines(p);
    const int tid = threadIdx.x;
    const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = p.wf == 1 ? wave : p.wf == 2 ? wave >> 1 : 0, wf = wave - wp * p.wf;
    const int bn = 32 * NB * p.wf;
    const int n_base = blockIdx.y * bn;
    const int f0 = n_base + wf * NB * 32;                // this wave's first filter
    const int PW = p.pw, plane = p.plane, cwh = p.cwe >> 1, ksteps = p.ksteps;
    u32x4 *atile = smem;
    float *thrs = reinterpret_cast<float *>(smem + p.cwe * plane);
    int *koff = reinterpret_cast<int *>(thrs + bn);      // [ksteps + 4]
    // the first region's loads, then the filters', then what the outputs need
    auto origin = [&](int t) __attribute__((always_inline)) {
        const int rg = (int)fast_div((uint32_t)t, p.div_ct);
        StreamTile o;
        o.rr0 = rg * p.th;
        o.x0 = (t - rg * p.col_tiles) * p.tw;
        o.img0 = (int)fast_div((uint32_t)o.rr0, p.div_oh);
        o.oy0 = o.rr0 - o.img0 * p.oh;
        return o;
    };
    int t = blockIdx.x;
    StreamTile tile = origin(t);
    StreamRegion<V> rch;
    if constexpr (V > 0) stream_load<V>(p, tile, wave, lane, 0, rch);
    const __amdgpu_buffer_rsrc_t wb =
        OHWI ? buffer_of(p.wpk, p.w_bytes) : filter_buffer(p, true);
    int col[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int co = f0 + 32 * i + l32;
        col[i] = OHWI ? min(co, p.cout - 1) * p.w_row + half * 4
                      : (half * p.coutp + min(co, p.coutp - 1)) * 4;
    }
    const int row8 = p.coutp * 8;
    // (OHWI, odd Cw: the second half's word of a tap's last pair does not exist)
    const bool odd = OHWI && (p.cw & 1);
    const uint32_t half_mask = odd && half ? 0u : ~0u;
    uint32_t bring[RB][NB];
    auto load_b = [&](int s, uint32_t (&d)[NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if constexpr (OHWI) {
                // (the whole offset in the lane's, which is what the buffer's
                // size is checked against)
                const int tap = odd ? (int)fast_div((uint32_t)s, p.div_cwh) : 0;
                d[i] = __builtin_amdgcn_raw_buffer_load_b32(wb, col[i] + s * 8 - tap * 4, 0, 0);
            } else {
                d[i] = __builtin_amdgcn_raw_buffer_load_b32(wb, col[i], s * row8, 0);
            }
        }
    };
    // the filter word of K step s as it was loaded
    auto filter_word = [&](uint32_t w, int s) __attribute__((always_inline)) {
        if constexpr (OHWI) {
            if (odd) {
                const int tap = (int)fast_div((uint32_t)s, p.div_cwh);
                return s - tap * cwh == cwh - 1 ? w & half_mask : w;
            }
        }
        return w;
    };
    uint32_t vmask;
    asm volatile("v_mov_b32 %0, 0x88888888" : "=v"(vmask));

#pragma unroll
    for (int r = 0; r < RB; ++r) load_b(min(r, ksteps - 1), bring[r]);
    float thr_raw = 0.0f;
    if constexpr (OUT == OUT_BITS) thr_raw = p.thr[min(n_base + min(tid, bn - 1), p.cout - 1)];
    // words past Cw: padding channels only, the same for every tile
    for (int e = plane * p.cw + tid; e < plane * p.cwe; e += kMfmaThreads)
        atile[e] = u32x4{kFp4PlusOne, kFp4PlusOne, kFp4PlusOne, kFp4PlusOne};
    float ep_a[NB], ep_b[NB];
    uint32_t flip_w[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int co = min(f0 + 32 * i + l32, p.cout - 1);
        ep_a[i] = OUT == OUT_FLOAT && p.mult ? p.mult[co] : 1.0f;
        ep_b[i] = OUT == OUT_FLOAT && p.bias ? p.bias[co] : 0.0f;
        flip_w[i] = 0;
        if constexpr (OUT == OUT_BITS) {
            const int fw = (f0 >> 5) + i;
            if (p.flip && fw < p.cwo) {
                const int nv = p.cout - 32 * fw;
                flip_w[i] = p.flip[fw] & (nv >= 32 ? ~0u : (1u << nv) - 1u);
            }
        }
    }
    // the A-tile offset of every K step (tap and word pair) from a window's
    // origin, in bytes; a few past the last one repeat it
    for (int s = tid; s < ksteps + 4; s += kMfmaThreads) {
        const int sc = min(s, ksteps - 1);
        const int tap = (int)fast_div((uint32_t)sc, p.div_cwh);
        const int ky = (int)fast_div((uint32_t)tap, p.div_kw);
        koff[s] = (2 * (sc - tap * cwh) * plane + ky * PW + tap - ky * p.kw) * 16;
    }
    // the window of each pixel block's lane: its A-tile offset where no image
    // boundary lies above it in the tile, and its output row in the tile
    uint32_t pix[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        const int q = min((wp * MB + b) * 32 + l32, p.px - 1);
        const int ty = (int)fast_div((uint32_t)q, p.div_tw);
        pix[b] = (uint32_t)(half * plane + ty * p.sh * PW + (q - ty * p.tw) * p.sw) |
                 (uint32_t)ty << 16;
    }

    if constexpr (OUT == OUT_BITS) {
        // the bound each dot is compared with, negated: the accumulators start
        // there, so that a finished value's sign is the output bit (kept within
        // +-(K + 1), where every partial sum is exact)
        if (tid < bn) {
            float T = n_base + tid < p.cout ? thr_to_dot_bound_f(thr_raw, p.lo, p.hi) : -INFINITY;
            const float kb = (float)(64 * ksteps);
            T = fminf(fmaxf(T, -kb), kb + 1.0f);
            thrs[tid] = -T - (float)p.pad_sum;
        }
    }
    for (;;) {
        // (the lane and wave indices pass through empty asm statements, so that the
        // compiler computes what depends on them anew for every tile instead of
        // keeping it in registers through the products)
        int lanev = lane, wavev = wave;
        asm volatile("" : "+v"(lanev), "+s"(wavev));
        // ---- the region of the tile
        if constexpr (V == 0) {
            stream_quantize(p, tile, atile, wavev, lanev);
        } else {
            stream_widen<V, !OHWI>(p, rch, atile, wavev, lanev, 0);
            for (int u0 = stream_reg_u(V); wavev + 4 * u0 < p.units; u0 += stream_reg_u(V)) {
                StreamRegion<V> ch;
                stream_load<V>(p, tile, wavev, lanev, u0, ch);
                stream_widen<V, !OHWI>(p, ch, atile, wavev, lanev, u0);
            }
        }
        // windows below an image boundary lie further down
        int a_base[MB];
#pragma unroll
        for (int b = 0; b < MB; ++b) a_base[b] = (int)(pix[b] & 0xFFFFu);
        if (p.n > 1 && tile.oy0 + p.th > p.oh) {
            const int gap = (p.ph - p.oh * p.sh) * PW;
#pragma unroll
            for (int b = 0; b < MB; ++b)
                a_base[b] += gap * (int)fast_div((uint32_t)tile.oy0 + (pix[b] >> 16), p.div_oh);
        }
        const int z = lds_barrier();                     // the A tile is complete
        // the next tile's region, in flight during this tile's products
        const StreamTile now = tile;
        t += (int)gridDim.x;
        const bool more = t < p.tiles;
        if (more) {
            tile = origin(t);
            if constexpr (V > 0) stream_load<V>(p, tile, wavev, lanev, 0, rch);
        }

        const float *thr_z = thrs + z;
        auto pin = []() __attribute__((always_inline)) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        };
        const int *ko = koff + z;
        const char *az = reinterpret_cast<const char *>(atile + z);
        int a_addr[MB];
#pragma unroll
        for (int b = 0; b < MB; ++b) a_addr[b] = a_base[b] * 16;
        mfma_v16f acc[MB][NB];
        u32x4 a[MB], bw[2][NB];
        int kcur = ko[1], knext;                         // offsets of steps s + 1 and s + 2
#pragma unroll
        for (int b = 0; b < MB; ++b) a[b] = *reinterpret_cast<const u32x4 *>(az + a_addr[b]);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            bw[0][i] = widen_word_vm(filter_word(bring[0][i], 0), kFp4PlusOne, vmask);
        // K step s with its filters widened in bc.  Between its products, in
        // pieces short enough to hide behind one: each pixel block's A is read
        // for step s + 1 after the block's last product, the filters of step
        // s + 1 are widened 32-bit word by word, and the ring slot of step s
        // (RI = s % RB) takes step s + RB or, past the last, the next tile's
        // step RI.
        auto step = [&](int s, auto ri_c, u32x4 (&bc)[NB], u32x4 (&bn_)[NB], auto first_c)
                        __attribute__((always_inline)) {
            constexpr bool first = decltype(first_c)::value;
            constexpr int RI = decltype(ri_c)::value;
            knext = ko[s + 2];
            uint32_t wn[NB];                             // the filter words of step s + 1
#pragma unroll
            for (int i = 0; i < NB; ++i) wn[i] = filter_word(bring[(RI + 1) % RB][i], s + 1);
            pin();
#pragma unroll
            for (int b = 0; b < MB; ++b) {
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    constexpr int kPer = 4 / MB;         // words widened per product
                    mfma_v16f c0v;
                    if constexpr (first) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) c0v[v] = 0.0f;
                        if constexpr (OUT == OUT_BITS) {
#pragma unroll
                            for (int qq = 0; qq < 4; ++qq) {
                                const float4 tq = *reinterpret_cast<const float4 *>(
                                    thr_z + (wf * NB + i) * 32 + 8 * qq + 4 * half);
                                c0v[4 * qq] = tq.x;
                                c0v[4 * qq + 1] = tq.y;
                                c0v[4 * qq + 2] = tq.z;
                                c0v[4 * qq + 3] = tq.w;
                            }
                        }
                    }
                    if constexpr (OUT == OUT_BITS)
                        acc[b][i] = mfma_fp4(bc[i], a[b], first ? c0v : acc[b][i]);
                    else
                        acc[b][i] = mfma_fp4(a[b], bc[i], first ? c0v : acc[b][i]);
                    if (i == NB - 1)
                        a[b] = *reinterpret_cast<const u32x4 *>(az + a_addr[b] + kcur);
#pragma unroll
                    for (int e = 0; e < kPer; ++e) {
                        const int j = (b * NB + i) * kPer + e, d = j & 3;
                        bn_[j >> 2][d] =
                            ((wn[j >> 2] << (3 - d)) & vmask) | kFp4PlusOne;
                    }
                    if (b == MB - 1 && i == NB - 1)
                        load_b(s + RB < ksteps ? s + RB : min(RI, ksteps - 1), bring[RI]);
                    pin();
                }
            }
            kcur = knext;
        };
        constexpr std::integral_constant<bool, true> yes{};
        constexpr std::integral_constant<bool, false> no{};
        constexpr std::integral_constant<int, 0> i0{};
        constexpr std::integral_constant<int, 1> i1{};
        constexpr std::integral_constant<int, 2> i2{};
        constexpr std::integral_constant<int, 3> i3{};
        step(0, i0, bw[0], bw[1], yes);
        int s = 1;
        for (; s + 4 <= ksteps; s += 4) {
            step(s, i1, bw[1], bw[0], no);
            step(s + 1, i2, bw[0], bw[1], no);
            step(s + 2, i3, bw[1], bw[0], no);
            step(s + 3, i0, bw[0], bw[1], no);
        }
        if (s < ksteps) step(s, i1, bw[1], bw[0], no);
        if (s + 1 < ksteps) step(s + 1, i2, bw[0], bw[1], no);
        if (s + 2 < ksteps) step(s + 2, i3, bw[1], bw[0], no);
        if (more) lds_barrier();                         // the A tile may be overwritten

        // ---- output.  Block b's 32 pixels are consecutive: its first, and
        // how many of them are real.
        asm volatile("" : "+v"(lanev));
        const int l32v = lanev & 31, halfv = lanev >> 5;
        int mb[MB], nv[MB];
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            const int qb = (wp * MB + b) * 32;
            if (p.col_tiles == 1) {
                mb[b] = now.rr0 * p.ow + qb;
                nv[b] = min(p.px - qb, p.m - mb[b]);
            } else {
                const int ty = (int)fast_div((uint32_t)qb, p.div_tw);
                const int x = now.x0 + qb - ty * p.tw;
                mb[b] = (now.rr0 + ty) * p.ow + x;
                nv[b] = qb < p.px && now.rr0 + ty < p.n * p.oh ? p.ow - x : 0;
            }
        }
        if constexpr (OUT == OUT_BITS) {
            uint32_t *out = reinterpret_cast<uint32_t *>(p.out) + (f0 >> 5);
            const bool two = NB == 2 && (f0 >> 5) + 1 < p.cwo;
#pragma unroll
            for (int b = 0; b < MB; b += 2) {
                // lanes below 32 store block b's pixels, the others block b + 1's
                const int m = (halfv ? mb[b + 1] : mb[b]) + l32v;
                const bool ok = l32v < (halfv ? nv[b + 1] : nv[b]) && f0 < p.cout;
                // (the signs shifted into words value by value, the blocks' words
                // side by side: each shift waits for the one before it)
                uint32_t word[NB], w[2][NB];
#pragma unroll
                for (int v = 15; v >= 0; --v)
#pragma unroll
                    for (int i = 0; i < NB; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const uint32_t u = __float_as_uint(acc[b + j][i][v]);
                            w[j][i] = v == 15 ? u >> 31 : __builtin_amdgcn_alignbit(w[j][i], u, 31);
                        }
#pragma unroll
                for (int i = 0; i < NB; ++i) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        w[j][i] = (w[j][i] | (w[j][i] << 8)) & 0x00FF00FFu;
                        w[j][i] = ((w[j][i] | (w[j][i] << 4)) & 0x0F0F0F0Fu) << (4 * halfv);
                    }
                    const auto sw = __builtin_amdgcn_permlane32_swap(w[0][i], w[1][i], false, false);
                    word[i] = (sw[0] | sw[1]) ^ flip_w[i];
                }
                if (ok) {
                    uint32_t *o = out + (size_t)m * p.cwo;
                    if (NB == 2 && two && p.out8) {
                        *reinterpret_cast<uint2 *>(o) = make_uint2(word[0], word[NB - 1]);
                    } else {
                        o[0] = word[0];
                        if (two) o[1] = word[NB - 1];
                    }
                }
            }
        } else {
            const float lof = (float)p.lo, hif = (float)p.hi, pad = (float)p.pad_sum;
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                const int mbu = __builtin_amdgcn_readfirstlane(mb[b]);
                const int nvu = __builtin_amdgcn_readfirstlane(min(max(nv[b], 0), 32));
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    // a buffer over the block's real pixels: stores past them are dropped
                    const int co = f0 + 32 * i + l32v, c4 = p.cout * 4;
                    const __amdgpu_buffer_rsrc_t ob = buffer_of(
                        reinterpret_cast<const float *>(p.out) +
                            (size_t)(uint32_t)mbu * (uint32_t)p.cout,
                        (uint32_t)nvu * (uint32_t)c4);
                    int vo = co < p.cout ? halfv * 4 * c4 + co * 4 : kBufOutside;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float d = acc[b][i][v] - pad;
                        uint32_t o;
                        if constexpr (OUT == OUT_FLOAT)
                            o = __float_as_uint(__builtin_fmaf(__builtin_amdgcn_fmed3f(d, lof, hif),
                                                               ep_a[i], ep_b[i]));
                        else
                            o = (uint32_t)min(max((int)d, p.lo), p.hi);
                        __builtin_amdgcn_raw_buffer_store_b32(o, ob, vo, 0, 0);
                        vo += (v & 3) == 3 ? 5 * c4 : c4;
                    }
                }
            }
        }
        if (!more) break;
    }
}

}  // namespace lce
