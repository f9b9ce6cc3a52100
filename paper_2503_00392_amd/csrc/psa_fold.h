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

// The rule is tested after every m-th block and after the last one (line 17); a fixed budget ends the blocks that count.
// In the chunk of blocks b0 .. b1 - 1 (b1: not beyond a budget) the last such position, b0 if there is none, and the first.
// Where m divides the chunk size and there is no budget, the last one is the chunk's end, whose state the chunk's word gives;
// else a second word per chunk and head covers the blocks up to that position ("split").
__device__ __forceinline__ int last_test(int b0, int b1, int m, int N) {
    const int t = b1 == N ? N : b1 / m * m;
    return t > b0 ? t : b0;
}
__device__ __forceinline__ int first_test(int b0, int m, int N) { return min(N, (b0 / m + 1) * m); }
__device__ __forceinline__ bool split_words(int KU, int m, int budget) { return budget > 0 || KU % m != 0; }
__device__ __forceinline__ int blocks_that_count(int N, int budget) { return budget > 0 ? min(N, budget) : N; }

// A group is 64 / G consecutive chunks, aligned, lane = (chunk of the group, head).  In: L, M = the lane's chunk's words;
// (Cacc, Cmin) = the lane's head's state at the start of the group.  Out: (L, M) = its AS_acc (log domain) and AS_min after
// the lane's chunk, by a prefix scan over the chunks (steps of G lanes); (E, F) = before it.  What stands in the lanes of later
// chunks does not matter, so the state after a chunk is a fixed expression of the chunk's place in its group, whichever chunks
// were published when a wave looked, and whichever wave looks.
template <int G>
__device__ __forceinline__ void group_states(float &L, float &M, float Cacc, float Cmin, float &E, float &F, int lane) {
#pragma unroll
    for (int d = G; d < 64; d <<= 1) {
        const float ol = __shfl_up(L, d), om = __shfl_up(M, d);
        if (lane >= d) { L = lse2(ol, L); M = fminf(om, M); }
    }
    L = lse2(Cacc, L);
    M = fminf(Cmin, M);
    E = __shfl_up(L, G);
    F = __shfl_up(M, G);
    if (lane < G) { E = Cacc; F = Cmin; }
}

// Whether the lane's head passes the threshold in the lane's chunk, blocks b0 .. b1 - 1, if it is open before it: P_acc is
// non-decreasing, so it does if it passes at the last position tested there; P is P_acc at that position.  (LT, MT): the
// chunk's second word, if there are any.
__device__ __forceinline__ bool chunk_passes(float L, float M, float E, float F, bool split, float LT, float MT, int b0, int b1,
                                             int N, int m, float eps, float &P) {
    const int t = last_test(b0, b1, m, N);
    if (split) { L = lse2(E, LT); M = fminf(F, MT); }
    P = p_acc(L, M, N - t);
    return t > b0 && passes_test(P, eps);
}

// The exact stop of the heads that pass in the chunk of blocks b0 .. b1 - 1, one wave: (cl, cm) = the state of head lane % G
// before it, Pt = its P_acc at the last tested position, block_value(i) = value i = (block, head) of the chunk's L_b.
// Lane = (block, head), 64 values to a register and all registers asked for at once; a prefix scan over the blocks of each
// head (steps of G lanes; the registers' scans side by side), on top of the state before, gives AS_acc and AS_min after every
// block, hence P_acc at every position; the first tested position that passes is the stop -- the last one, should rounding
// (another tree of sums than the chunk's word) let none pass.  kScan: registers that hold one value per (block, head).
template <int G, int kScan, class BlockValue>
__device__ __forceinline__ void stop_in_chunk(int b0, int b1, float cl, float cm, float Pt, int N, int m, float eps,
                                              BlockValue block_value, int &n, float &P_stop, int lane) {
    const int g = lane % G, cnt = (b1 - b0) * G;
    const unsigned long long head_lanes = (~0ull / ((1ull << G) - 1ull)) << g;   // the lanes of my head
    n = last_test(b0, b1, m, N);
    P_stop = Pt;
    if (first_test(b0, m, N) == n) return;     // (uniform)
    bool found = false;
    float pl[kScan], pm[kScan];
#pragma unroll
    for (int u = 0; u < kScan; ++u) pm[u] = pl[u] = block_value(min(64 * u + lane, cnt - 1));
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
        const int nn = b0 + (64 * u + lane) / G + 1;
        const float P = p_acc(fl, fm, N - nn);
        const unsigned long long hits =
            __ballot(64 * u + lane < cnt && (nn % m == 0 || nn == N) && passes_test(P, eps)) & head_lanes;
        const int src = hits ? (__ffsll((long long)hits) - 1) : 0;
        const float Pf = __shfl(P, src);
        if (!found && hits) {
            n = b0 + (64 * u + src) / G + 1;
            P_stop = Pf;
            found = true;
        }
        cl = __shfl(fl, 64 - G + g);       // my head's state after this register's last block
        cm = __shfl(fm, 64 - G + g);
    }
}
__device__ __forceinline__ unsigned long long stop_word(int n, float P) { return ((unsigned long long)n << 32) | __float_as_uint(P); }

// Folds chunks j .. k-1 of the stream's first group, whose words and block values are all at hand, one wave: the chunks in
// which an open head passes are visited in order (there are at most G stops per stream) for the head's exact stop.
// stop = the head's stop so far; block_value(b, i) is value i = (block, head) of the chunk that starts at block b.
// Returns the chunks folded now: k, or less when every head has stopped (then all_stopped).
template <int G, int kScan, class BlockValue>
__device__ __forceinline__ int fold_group(float L, float M, float LT, float MT, unsigned long long &stop, int j, int k, int N,
                                          int m, int KU, int budget, float eps, bool &all_stopped, BlockValue block_value, int lane) {
    const int nlim = blocks_that_count(N, budget), g = lane % G, jl = lane / G;
    all_stopped = false;
    float E, F, P;
    group_states<G>(L, M, -INFINITY, INFINITY, E, F, lane);
    const bool passes = chunk_passes(L, M, E, F, split_words(KU, m, budget), LT, MT, jl * KU, min(jl * KU + KU, nlim), N, m, eps, P);
    while (j < k) {
        const unsigned long long cand = __ballot(jl >= j && jl < k && stop == ~0ull && passes);
        if (cand == 0ull) return k;
        const int js = (__ffsll((long long)cand) - 1) / G, src = js * G + g;   // the first chunk in which an open head passes
        int n;
        float Ps;
        stop_in_chunk<G, kScan>(js * KU, min(js * KU + KU, nlim), __shfl(E, src), __shfl(F, src), __shfl(P, src), N, m, eps,
                                [&](int i) { return block_value(js * KU, i); }, n, Ps, lane);
        if ((cand >> src) & 1ull) stop = stop_word(n, Ps);
        j = js + 1;
        if (__ballot(stop == ~0ull) == 0ull) { all_stopped = true; return j; }
    }
    return k;
}

}  // namespace psa
