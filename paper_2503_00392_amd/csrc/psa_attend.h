// Per-block building blocks shared by the dense control kernel, the selection kernel and the metadata kernel:
// how one wave reads a 4 KiB (page, KV head) slice and what each lane holds, and the 16x16x16 matrix
// product with 16-bit operands that both attention kernels accumulate values with.
//
// Lane layout of a wave over one K or V slice [16 tokens][128 channels] of 2-byte elements:
//   rg = lane / 16  (row group 0..3),  cl = lane % 16  (channel slot: channels 8*cl .. 8*cl+7)
//   load i (0..3) fetches token row 4*i + rg, 16 bytes per lane, so one load instruction of the
//   wave covers rows 4*i .. 4*i+3 = 1 KiB of contiguous memory.
#pragma once

#include "psa_device.h"

namespace psa {

struct Slice {
    uint4 r[4];
};

__device__ __forceinline__ Slice load_slice(const uint8_t *slice_base, int lane) {
    Slice s;
    const uint8_t *p = slice_base + lane * 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) s.r[i] = ld16_stream(p + i * 1024);
    return s;
}

// Rows of a partly filled block beyond `valid` may hold anything (NaN included): make them zero.
__device__ __forceinline__ void zero_invalid_rows(Slice &v, int rg, int valid) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (4 * i + rg >= valid) v.r[i] = make_uint4(0, 0, 0, 0);
}

// D(16x16, fp32) += A(16x16) * B(16x16) on the matrix cores, 16-bit inputs.  Lane l supplies row l%16 of A
// and column l%16 of B, k values 4*(l/16) .. +3 of each; it receives column l%16 of D, rows 4*(l/16) .. +3.
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
template <int DT>
__device__ __forceinline__ f32x4_t mfma_16x16x16(const uint2 &a, const uint2 &b, f32x4_t c) {
    if constexpr (DT == 0) {
        return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4_t, a), __builtin_bit_cast(f16x4_t, b), c, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, a), __builtin_bit_cast(s16x4_t, b), c, 0, 0, 0);
    }
}

// p = hi + lo with both halves in the 16-bit type of the cache (round to nearest each): the bits of the asked-for half.
template <int DT>
__device__ __forceinline__ uint32_t half16(float p, bool low) {
    if constexpr (DT == 0) {
        const _Float16 h = (_Float16)p;
        return __builtin_bit_cast(uint16_t, low ? (_Float16)(p - (float)h) : h);
    } else {
        const __bf16 h = (__bf16)p;
        return __builtin_bit_cast(uint16_t, low ? (__bf16)(p - (float)h) : h);
    }
}

__device__ __forceinline__ uint32_t pick_word(const uint4 &v, int w) {
    return w == 0 ? v.x : (w == 1 ? v.y : (w == 2 ? v.z : v.w));
}

// One block of the value product: D[row][channel] += A[row][token] V[token][channel], eight 16x16x16 products, one per
// channel of the lane's eight.  Row 2 g of A holds the upper 16-bit halves of head g's weights, row 2 g + 1 the lower
// halves: the two share one product (sixteen rows are there anyway, and at most eight heads), lane (rg, *) ends up with
// both halves of heads 2 rg and 2 rg + 1 in registers 0, 1 and 2, 3 of each accumulator, to be added at the end.
// x: logits of head cl / 2 for the four tokens whose value rows the lane holds; the weights p = exp(x - ref), nothing
// where the head does not use the block (`on`; tokens beyond the request hold -inf), are added to l.
template <int DT>
__device__ __forceinline__ void add_weighted(f32x4_t (&acc)[8], const Slice &v, const float (&p)[4], bool low) {
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = half16<DT>(p[j], low);
    const uint2 a = make_uint2(w[0] | (w[1] << 16), w[2] | (w[3] << 16));
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const uint32_t w0 = pick_word(v.r[0], t >> 1), w1 = pick_word(v.r[1], t >> 1);
        const uint32_t w2 = pick_word(v.r[2], t >> 1), w3 = pick_word(v.r[3], t >> 1);
        const uint2 b = (t & 1) ? make_uint2((w0 >> 16) | (w1 & 0xffff0000u), (w2 >> 16) | (w3 & 0xffff0000u))
                                : make_uint2((w0 & 0xffffu) | (w1 << 16), (w2 & 0xffffu) | (w3 << 16));
        acc[t] = mfma_16x16x16<DT>(a, b, acc[t]);
    }
}
template <int DT>
__device__ __forceinline__ void add_values(f32x4_t (&acc)[8], float &l, const Slice &v, f32x4_t x, bool on, float ref, bool low) {
    float p[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = on ? exp2_fast(x[j] - ref) : 0.0f;
    l += (p[0] + p[1]) + (p[2] + p[3]);
    add_weighted<DT>(acc, v, p, low);
}
// The lane's sums of heads 2 rg and 2 rg + 1 (those below G), channels 8 cl .. 8 cl + 7, to rows[head][channel].
template <int G>
__device__ __forceinline__ void store_heads(const f32x4_t (&acc)[8], float (*rows)[kHeadDim], int rg, int cl) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (2 * rg + k < G) {
            f32x4_t *row = reinterpret_cast<f32x4_t *>(&rows[2 * rg + k][cl * 8]);
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                f32x4_t o;
#pragma unroll
                for (int t = 0; t < 4; ++t) o[t] = acc[4 * y + t][2 * k] + acc[4 * y + t][2 * k + 1];
                row[y] = o;
            }
        }
    }
}

}  // namespace psa
