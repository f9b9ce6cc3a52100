// The arithmetic of the stop rule (Algorithm 1, lines 12-18) and of the key product that feeds it, shared by the
// kernels that apply them: the selection kernel, where a wave folds chunks that other workgroups publish, and the
// one-workgroup-per-stream kernel of short contexts, where everything stays in LDS.  Both give the same bits.
#pragma once

#include "psa_device.h"

namespace psa {

// P_acc of Algorithm 1 lines 15-16 in the log2 domain: AS_acc / (AS_acc + AS_min * N_left).
__device__ __forceinline__ float p_acc(float Lacc, float Lmin, int n_left) {
    return 1.0f / (1.0f + (float)n_left * exp2_fast(Lmin - Lacc));
}

// Line 17's test.  P_acc is no number for a head whose logits are none: it passes no threshold of the caller's, but ends
// where a fixed budget of blocks below N ends, which is tested there alone (m = budget) and against kBudgetEps.
constexpr float kBudgetEps = -1.0f;
__device__ __forceinline__ float stop_threshold(float eps, int budget, int N) {     // (uniform: in a scalar register)
    const float t = budget > 0 && budget < N ? kBudgetEps : eps;
    return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(t)));
}
__device__ __forceinline__ bool passes_test(float P, float eps) { return fmaxf(P, 0.0f) > eps; }

// Scaled logits (log2 units) of one block against the heads of its group.  k: the block's key slice as four coalesced
// 1 KiB rows of lanes; qb: the B operand (column n = lane % 16 is head n, zero beyond the group).  Loading the slice in
// the operand's layout would touch sixteen 64-byte segments per instruction, so the wave turns it into that layout
// through its own patch of LDS (row = token, 17 16-byte words apart: no bank conflicts).  Row r of the A operand stands
// for token 4*(r%4) + r/4, so that lane (kq, n) ends up with head n's logits of tokens kq, 4+kq, 8+kq, 12+kq: the value
// pass wants the four tokens whose value rows ITS lane (kq, *) loads.  Tokens from `valid` on are -inf.
template <int DT>
__device__ __forceinline__ f32x4_t block_logits(const uint4 (&k)[4], const uint4 (&qb)[4], uint4 *stg, int lane, int valid) {
    const int n = lane & 15, kq = lane >> 4, arow = 4 * (n & 3) + (n >> 2);
    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) stg[(kk * 4 + kq) * 17 + n] = k[kk];
    lds_wave_sync();
    uint4 a[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) a[kk] = stg[arow * 17 + kk * 4 + kq];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) acc = mfma_16x16x32<DT>(a[kk], qb[kk], acc);
    f32x4_t sc;
#pragma unroll
    for (int x = 0; x < 4; ++x) sc[x] = (4 * x + kq < valid) ? acc[x] * kScaleLog2 : -INFINITY;
    return sc;
}

// The blocks' log2-sum-exp2 L_b per head, from logits in LDS (lg: rows of sixteen, one per (block, head)) to Lb (one
// value per row), by NT threads at once: kQuad threads per row, each its share of the row's four quarters.  (Reduced
// slice by slice as the products come, the chain of lane exchanges, exponentials and a logarithm took longer than the
// product itself, for every slice of a wave one after the other: 4.6 us for eight slices, 3.5 us this way.)
template <int G, int NT>
__device__ __forceinline__ void rows_lse(const float *lg, float *Lb, int rows, int tid) {
    constexpr int kQuad = G >= 8 ? 1 : (G == 4 ? 2 : 4), kShare = 4 / kQuad;
    for (int x = tid; x < rows * kQuad; x += NT) {
        const int row = x / kQuad, part = x % kQuad;
        const f32x4_t *src = reinterpret_cast<const f32x4_t *>(lg) + row * 4 + part * kShare;
        f32x4_t v[kShare];
        float mx = -INFINITY;
#pragma unroll
        for (int y = 0; y < kShare; ++y) {
            v[y] = src[y];
            mx = fmaxf(mx, fmaxf(fmaxf(v[y][0], v[y][1]), fmaxf(v[y][2], v[y][3])));
        }
        if constexpr (kQuad >= 2) mx = fmaxf(mx, dpp_f<0xB1>(mx));
        if constexpr (kQuad == 4) mx = fmaxf(mx, dpp_f<0x4E>(mx));
        float e[kShare];
#pragma unroll
        for (int y = 0; y < kShare; ++y)
            e[y] = (exp2_fast(v[y][0] - mx) + exp2_fast(v[y][1] - mx)) + (exp2_fast(v[y][2] - mx) + exp2_fast(v[y][3] - mx));
        float sum = e[0];
        if constexpr (kShare == 2) sum = e[0] + e[1];
        if constexpr (kShare == 4) sum = (e[0] + e[1]) + (e[2] + e[3]);
        if constexpr (kQuad >= 2) sum += dpp_f<0xB1>(sum);
        if constexpr (kQuad == 4) sum += dpp_f<0x4E>(sum);
        if (part == 0) Lb[row] = mx + log2_fast(sum);
    }
}

// A chunk's (log-sum-exp, minimum) of its nblk blocks' L_b per head, one wave.  Lane = (slot, head): 64/G slots each
// fold every (64/G)-th block, then a butterfly over the slots -- a fixed tree, so the result is reproducible; lse2 is
// symmetric, so every lane of a head ends with the same bits.
template <int G>
__device__ __forceinline__ void chunk_aggregate(const float *Lb, int nblk, int lane, float &aggL, float &aggMin) {
    constexpr int kSlots = 64 / G;
    const int g = lane % G;
    aggL = -INFINITY;
    aggMin = INFINITY;
    for (int i = lane / G; i < nblk; i += kSlots) {
        const float v = Lb[i * G + g];
        aggL = lse2(aggL, v);
        aggMin = fminf(aggMin, v);
    }
#pragma unroll
    for (int d = G; d < 64; d <<= 1) {
        aggL = lse2(aggL, __shfl_xor(aggL, d));
        aggMin = fminf(aggMin, __shfl_xor(aggMin, d));
    }
}

// Folds chunks j .. k-1 of a group of 64 / G consecutive chunks (the first is chunk `base` of the stream), one wave,
// lane = (chunk of the group, head).  In: L, M = the lane's chunk's words; (Cacc, Cmin) = the lane's head's state at
// the start of the group; stop = its stop so far; ready = whether the lane's chunk's block values can be had.
// A prefix scan over the chunks (steps of G lanes) gives every head's AS_acc and AS_min after every chunk of the group
// at once, hence P_acc at every chunk's end.  The chunks in which an open head passes the threshold are then visited in
// order (there are at most G stops per stream) for the head's exact stop, with a second prefix scan over that chunk's
// blocks; block_value(b, i) is value i = (block, head) of the chunk that starts at block b.
// Out: L, M = the state after the lane's chunk; returns the chunks of the group folded now: k, or less when every head
// has stopped (then all_stopped), or when it came to a chunk that is not `ready`.
// kScan: registers that hold one value per (block, head) of a chunk.
template <int G, int kScan, class BlockValue>
__device__ __forceinline__ int fold_group(float &L, float &M, float Cacc, float Cmin, unsigned long long &stop, int ready,
                                          int base, int j, int k, int N, int m, int KU, float eps, bool &all_stopped,
                                          BlockValue block_value) {
    const int lane = threadIdx.x & 63, g = lane % G, jl = lane / G;
    const unsigned long long head_lanes = (~0ull / ((1ull << G) - 1ull)) << g;   // the lanes of my head
    all_stopped = false;
#pragma unroll
    for (int d = G; d < 64; d <<= 1) {
        const float ol = __shfl_up(L, d), om = __shfl_up(M, d);
        if (lane >= d) { L = lse2(ol, L); M = fminf(om, M); }
    }
    L = lse2(Cacc, L);
    M = fminf(Cmin, M);
    const int b0 = (base + jl) * KU, n_end = min(b0 + KU, N);
    // a stop inside a chunk needs a position where the rule is tested (line 17 is reached every m blocks and
    // at the last block) and, P_acc being non-decreasing, a pass at the chunk's end
    const bool passes = ((n_end / m) * m > b0 || n_end == N) && passes_test(p_acc(L, M, N - n_end), eps);
    while (j < k) {
        const unsigned long long cand = __ballot(jl >= j && jl < k && stop == ~0ull && passes);
        if (cand == 0ull) return k;
        const int js = (__ffsll((long long)cand) - 1) / G;          // the first chunk in which an open head passes
        const bool scan = (cand >> (js * G + g)) & 1ull;            // does mine?
        if (__shfl(ready, js * G) == 0) return js;
        // That chunk's blocks' L_b, lane = (block, head), 64 values to a register and all registers asked for at
        // once; a prefix scan over the blocks of each head (steps of G lanes; the registers' scans side by side),
        // on top of the state after the chunk before, gives AS_acc and AS_min after every block, hence P_acc at
        // every position; the first tested position that passes is the stop.
        const int cb0 = (base + js) * KU, cnt = (min(cb0 + KU, N) - cb0) * G;
        float cl = js == 0 ? Cacc : __shfl(L, (js - 1) * G + g);
        float cm = js == 0 ? Cmin : __shfl(M, (js - 1) * G + g);
        bool found = false;
        float pl[kScan], pm[kScan];
#pragma unroll
        for (int u = 0; u < kScan; ++u) pm[u] = pl[u] = block_value(cb0, min(64 * u + lane, cnt - 1));
#pragma nounroll
        for (int d = G; d < 64; d <<= 1) {
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                const float ol = __shfl_up(pl[u], d), om = __shfl_up(pm[u], d);
                if (lane >= d) { pl[u] = lse2(ol, pl[u]); pm[u] = fminf(om, pm[u]); }
            }
        }
#pragma unroll
        for (int u = 0; u < kScan; ++u) {
            const float fl = lse2(cl, pl[u]), fm = fminf(cm, pm[u]);
            const int nn = cb0 + (64 * u + lane) / G + 1;
            const float P = p_acc(fl, fm, N - nn);
            const unsigned long long hits =
                __ballot(64 * u + lane < cnt && (nn % m == 0 || nn == N) && passes_test(P, eps)) & head_lanes;
            const int src = hits ? (__ffsll((long long)hits) - 1) : 0;
            const float Pf = __shfl(P, src);
            if (scan && !found && hits) {
                stop = ((unsigned long long)(cb0 + (64 * u + src) / G + 1) << 32) | __float_as_uint(Pf);
                found = true;
            }
            cl = __shfl(fl, 64 - G + g);       // my head's state after this register's last block
            cm = __shfl(fm, 64 - G + g);
        }
        j = js + 1;
        if (__ballot(stop == ~0ull) == 0ull) { all_stopped = true; return j; }
    }
    return k;
}

}  // namespace psa
