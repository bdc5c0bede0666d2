// Sign binarization + bitpacking (LceQuantize, arXiv 2011.09398 Section 3.2).
//
// Bit c%32 of word c/32 of a row is 1 iff x[row][c] < 0.0f (a 1 bit stands
// for -1.0, a 0 bit for +1.0); bits past the channel count are 0.
//
// The work is HBM-bound (4 bytes read per bit written), so the kernels are
// shaped for coalesced loads: in the fast path a wave reads 1 KiB of
// contiguous floats per instruction (one float4 per lane), each lane turns
// its four signs into a nibble, and three DPP row shifts OR the nibbles of
// eight neighbouring lanes into the 32-bit word they make up.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dpp.hpp"
#include "fastdiv.hpp"

namespace lce {

constexpr int kBitpackThreads = 256;
constexpr int kBitpackUnroll = 4;   // 1 KiB chunks in flight per wave

// Fast path: channels % 32 == 0 and x 16-byte aligned, so the tensor is a
// flat sequence of 32-float groups, each packing into one word.
// A chunk is 64 float4 = 256 floats = 8 words.
__global__ __launch_bounds__(kBitpackThreads) void bitpack32_kernel(
    const float4 *__restrict__ x, uint32_t *__restrict__ out, int64_t nwords) {
    const int lane = threadIdx.x & 63;
    const int64_t nvec = nwords * 8;            // float4 count
    const int64_t nchunks = (nwords + 7) / 8;
    const int64_t wave = ((int64_t)blockIdx.x * kBitpackThreads + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * kBitpackThreads) >> 6;
    const int shift = 4 * (lane & 7);
    for (int64_t c0 = wave * kBitpackUnroll; c0 < nchunks; c0 += nwaves * kBitpackUnroll) {
        float4 v[kBitpackUnroll];
#pragma unroll
        for (int u = 0; u < kBitpackUnroll; ++u) {
            const int64_t idx = (c0 + u) * 64 + lane;
            v[u] = idx < nvec ? x[idx] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < kBitpackUnroll; ++u) {
            uint32_t nib = (uint32_t)(v[u].x < 0.0f) | ((uint32_t)(v[u].y < 0.0f) << 1) |
                           ((uint32_t)(v[u].z < 0.0f) << 2) | ((uint32_t)(v[u].w < 0.0f) << 3);
            uint32_t s = nib << shift;
            s |= row_shr<1>(s);
            s |= row_shr<2>(s);
            s |= row_shr<4>(s);
            // Lane 8g+7 now holds the OR over lanes 8g..8g+7: word g of the chunk.
            const int64_t word = (c0 + u) * 8 + (lane >> 3);
            if ((lane & 7) == 7 && word < nwords) out[word] = s;
        }
    }
}

// Rows of one word and few channels: one thread per row, whose few loads lie in
// the lines that its neighbours' loads touch, with no barrier.
__global__ __launch_bounds__(kBitpackThreads) void bitpack_short_kernel(
    const float *__restrict__ x, uint32_t *__restrict__ out, int64_t rows, int channels) {
    const int64_t stride = (int64_t)gridDim.x * kBitpackThreads;
    for (int64_t r = (int64_t)blockIdx.x * kBitpackThreads + threadIdx.x; r < rows; r += stride) {
        const float *src = x + r * channels;
        uint32_t word = 0;
        for (int b = 0; b < channels; ++b) word |= (uint32_t)(src[b] < 0.0f) << b;
        out[r] = word;
    }
}

// Whether bitpack_short_kernel packs these rows faster than the general path
// (us short, general; rows x channels: 4096x7 2.4, 2.6; 65536x3 2.4, 3.3;
// 2000000x3 6.9, 8.3; 500000x6 4.4, 5.1, but 1000000x6 7.3, 6.0; 65536x12 3.0,
// 3.3, but 4096x12 2.8, 2.6 and 130000x8 3.7, 3.4).
inline bool bitpack_short(int64_t rows, int channels) {
    const int64_t floats = rows * channels;
    return channels <= 3 || (channels <= 7 && floats <= 3 << 20) ||
           (channels <= 12 && rows > 40000 && rows <= 100000);
}

// General path: any channel count and 4-byte alignment.  A row's words start
// anywhere in the float stream, so the signs are first packed as they lie in
// memory (16-byte loads, the fast path's nibbles) into LDS, and each output
// word is then cut out of that bit string: the floats are read once, 1 KiB per
// wave and instruction.  A workgroup takes `chunk` consecutive output words at
// a time, which cover at most 32*chunk consecutive floats.  (One thread per
// word, walking its own 32 floats, read 64 cache lines per instruction: 64
// images of 56x56x72, 60 MB, 124 us; this 12 us, 5.0 TB/s.)
// U: 16-byte loads in flight per thread: 2 where a pass has no more (64 rows of
// 33 channels: 2.3 us against 2.9 with 8, most of them nothing), else 8.
constexpr int kBitpackChunk = 1024;   // words per workgroup pass, at most

template <int U>
__global__ __launch_bounds__(kBitpackThreads) void bitpack_generic_kernel(
    const float *__restrict__ x, uint32_t *__restrict__ out, int64_t rows, int channels, int chunk,
    FastDiv div_cw) {
    __shared__ uint32_t bits[kBitpackChunk + 3];
    const int tid = threadIdx.x, lane = tid & 63;
    const int cw = (int)div_cw.d;
    const int64_t total = rows * (int64_t)cw, floats = rows * (int64_t)channels;
    // float index i sits at 16-byte unit (i + skew) / 4
    const int skew = (int)((reinterpret_cast<uintptr_t>(x) >> 2) & 3);
    const float4 *x4 = reinterpret_cast<const float4 *>(x - skew);
    const int shift = 4 * (lane & 7);
    for (int64_t w0 = (int64_t)blockIdx.x * chunk; w0 < total; w0 += (int64_t)gridDim.x * chunk) {
        const int n = (int)min((int64_t)chunk, total - w0);
        // the pass's first word: row r0, word j0; its first float, and the one
        // past its last
        const int64_t r0 = w0 / cw;
        const int j0 = (int)(w0 - r0 * cw);
        const int64_t first = r0 * channels + (int64_t)j0 * 32;
        const int rl = (int)fast_div((uint32_t)(j0 + n - 1), div_cw), jl = j0 + n - 1 - rl * cw;
        const int64_t end = (r0 + rl) * channels + min((int64_t)channels, (int64_t)jl * 32 + 32);
        const int64_t q0 = (first + skew) >> 2;                  // 16-byte units
        const int nq = (int)(((end + skew + 3) >> 2) - q0);
        for (int b = 0; b < nq; b += U * kBitpackThreads) {
            float4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = b + u * kBitpackThreads + tid;
                const int64_t f = ((q0 + i) << 2) - skew;        // the unit's first float
                v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (i < nq) {
                    if (f >= 0 && f + 4 <= floats) {
                        v[u] = x4[q0 + i];
                    } else {                                     // the tensor's ends
                        if (f >= 0 && f < floats) v[u].x = x[f];
                        if (f + 1 >= 0 && f + 1 < floats) v[u].y = x[f + 1];
                        if (f + 2 >= 0 && f + 2 < floats) v[u].z = x[f + 2];
                        if (f + 3 >= 0 && f + 3 < floats) v[u].w = x[f + 3];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = b + u * kBitpackThreads + tid;
                uint32_t s = ((uint32_t)(v[u].x < 0.0f) | ((uint32_t)(v[u].y < 0.0f) << 1) |
                              ((uint32_t)(v[u].z < 0.0f) << 2) | ((uint32_t)(v[u].w < 0.0f) << 3))
                             << shift;
                s |= row_shr<1>(s);
                s |= row_shr<2>(s);
                s |= row_shr<4>(s);
                if ((lane & 7) == 7 && (i >> 3) < kBitpackChunk + 2) bits[i >> 3] = s;
            }
        }
        __syncthreads();
        const int64_t origin = (q0 << 2) - skew;                 // the float at bit 0
        const int base = (int)(first - origin) - j0 * 32;        // row r0's bit position
        for (int i = tid; i < n; i += kBitpackThreads) {
            const int r = (int)fast_div((uint32_t)(j0 + i), div_cw), j = j0 + i - r * cw;
            const int at = base + r * channels + 32 * j;
            const int nb = min(32, channels - 32 * j);
            const uint32_t w = __builtin_amdgcn_alignbit(bits[(at >> 5) + 1], bits[at >> 5], at & 31);
            out[w0 + i] = nb == 32 ? w : w & ((1u << nb) - 1u);
        }
        __syncthreads();
    }
}

}  // namespace lce
