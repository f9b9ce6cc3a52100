// Ranking of a stream's blocks (Algorithm 1, line 6): criticality score descending, ties to the
// smaller logical block.  One workgroup per stream, everything in LDS and registers.
//
// Main path: a monotone bucket map + exact in-bucket ranking.
//   1. every thread holds K keys (order-preserving 32-bit images of the scores, inverted so that a
//      smaller key is a larger score) and the workgroup reduces their minimum and maximum;
//   2. bucket = floor((largest score - score) * scale) is monotone in the score, so bucket order is
//      rank order; an LDS counter per bucket and a workgroup scan give each bucket its output range;
//   3. the elements are laid out bucket by bucket ("slots"); an element's final rank is its bucket's base
//      plus the number of elements of the same bucket that precede it under (key, index) -- counted
//      exactly, so the result does not depend on the order in which the LDS atomics arrived.  The
//      counting goes slot by slot, every thread of the workgroup taking its share, so that neighbouring
//      lanes look at the same bucket.
// There are as many buckets as element slots, so a bucket holds about one element.  If one bucket
// holds more than kBucketLimit elements
// (near-identical scores) the quadratic in-bucket count would be slow, and the workgroup falls back
// to a bitonic network over 64-bit (key, index) words, eight to a thread: compare distances below 8 stay in
// registers, below 512 go through wave shuffles, the rest through LDS.  Both paths give the same total order.
//
// With few streams several workgroups share one stream: each counts all elements (cheap) and lays out and
// ranks its share of them (the expensive part, bound by LDS traffic).
//
// What bounds it is the chain of short steps between barriers, not data: hence two keys to a thread up to 2048 blocks,
// four up to 4096, eight beyond (a workgroup has 1024 threads at most); reductions along rows of lanes; counters of
// 16 bits, so that two workgroups of 8192 blocks fit a compute unit; and the request's row of the block table read at
// the start, so that the gather at the end finds it in the cache.  With eight keys to a thread throughout, 32-bit
// counters and reductions through LDS exchanges it took 11.9 us at 2048 blocks (64 streams), 8.0 now; 18.0 -> 13.4 at
// 8192 (32 streams), 40.5 -> 26.4 with 512 streams; where the time went: scores 0.9 us, range 0.5, counters 0.6, scan 0.4,
// shares 0.5, layout 0.4, count 0.9, gather and stores 0.4, the rest is the launch.
//
// The kernel also resets the stream's control block and chunk words for the progressive kernel,
// reports out-of-range contexts and block-table entries and, with a second tier, looks up which slices have slots.
// grid (workgroups per stream, S), Np / K threads, 8*Np + 512 bytes of dynamic LDS; Np = power of two >= max(512, max_blocks).
#include <limits.h>

#include "psa_host.h"

namespace psa {

constexpr int kBucketLimit = 192;


__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long v, int mask) {
    const int lo = __shfl_xor((int)(v & 0xffffffffull), mask);
    const int hi = __shfl_xor((int)(v >> 32), mask);
    return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

// The score a key stands for (with -0 read as +0).
__device__ __forceinline__ float score_of_key(uint32_t key) {
    const uint32_t asc = ~key;
    return __uint_as_float((asc & 0x80000000u) ? (asc & 0x7FFFFFFFu) : ~asc);
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }

// The network is the work of nthreads = Np / 8 threads, whole waves; the waves beyond them meet them at its barriers, two to
// every step that goes through LDS.  (With those running the network as well, on keys of nobody, a call with tied scores
// took 62.6 us at 2048 blocks and 8 streams.)
__device__ __forceinline__ void bitonic_barriers(int Np) {
    for (int k = 2; k <= Np; k <<= 1)
        for (int j = k >> 1; j >= 8 * 64; j >>= 1) { __syncthreads(); __syncthreads(); }
}
__device__ void bitonic_sort(unsigned long long (&e)[8], unsigned long long *lds_keys, int Np, int tid,
                             int nthreads) {
    for (int k = 2; k <= Np; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j >= 8) {
                const int tj = j >> 3;   // partner thread distance
                unsigned long long o[8];
                if (tj >= 64) {
#pragma unroll
                    for (int x = 0; x < 8; ++x) lds_keys[x * nthreads + tid] = e[x];
                    __syncthreads();
#pragma unroll
                    for (int x = 0; x < 8; ++x) o[x] = lds_keys[x * nthreads + (tid ^ tj)];
                    __syncthreads();
                } else {
#pragma unroll
                    for (int x = 0; x < 8; ++x) o[x] = shfl_xor_u64(e[x], tj);
                }
                const bool up = ((tid * 8) & k) == 0;        // ascending region of this merge
                const bool lower = (tid & tj) == 0;
                const bool keep_min = (lower == up);
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    const unsigned long long lo = e[x] < o[x] ? e[x] : o[x];
                    const unsigned long long hi = e[x] < o[x] ? o[x] : e[x];
                    e[x] = keep_min ? lo : hi;
                }
            } else {
                // partner inside the thread's own 8 keys
#define PSA_CE(A, B)                                                              \
    {                                                                             \
        const bool up = ((tid * 8 + (A)) & k) == 0;                               \
        const bool sw = (e[A] > e[B]) == up;                                      \
        const unsigned long long t0 = sw ? e[B] : e[A], t1 = sw ? e[A] : e[B];    \
        e[A] = t0;                                                                \
        e[B] = t1;                                                                \
    }
                if (j == 4) {
                    PSA_CE(0, 4) PSA_CE(1, 5) PSA_CE(2, 6) PSA_CE(3, 7)
                } else if (j == 2) {
                    PSA_CE(0, 2) PSA_CE(1, 3) PSA_CE(4, 6) PSA_CE(5, 7)
                } else {
                    PSA_CE(0, 1) PSA_CE(2, 3) PSA_CE(4, 5) PSA_CE(6, 7)
                }
#undef PSA_CE
            }
        }
    }
}

// K: keys per thread.  TIER: with a second tier (a parameter of the kernel otherwise costs registers: 14.8 us instead of 13.6
// at 8192 blocks).
template <int K, bool TIER>
__global__ __launch_bounds__(1024, 8) void order_kernel(KvView kv, DecodeWs ws, int G, int KU, int budget_blocks, int Np,
                                                      int force_bitonic, const int32_t *__restrict__ slot_of,
                                                      int32_t *__restrict__ order_out) {
    extern __shared__ unsigned long long lds_raw[];
    const int s = blockIdx.y, r = s / kv.num_kv_heads;
    const int part = blockIdx.x, nparts = gridDim.x;
    const int tid = threadIdx.x, nthreads = blockDim.x, lane = tid & 63, wave = tid >> 6;
    const int nwaves = nthreads >> 6;
    // what this thread needs from memory, requested before anything else: its K scores (loads of 8 or 16 bytes
    // where the row's length allows)
    const float *sc = ws.scores + (size_t)s * kv.max_blocks;
    const int32_t *table = kv.block_table + (size_t)r * kv.max_blocks;
    float scv[K];
    if (kv.max_blocks % K == 0) {
        typedef float vec_t __attribute__((ext_vector_type(K < 4 ? K : 4)));
        const vec_t *v = reinterpret_cast<const vec_t *>(sc + min(tid * K, kv.max_blocks - K));   // (clamped: no branch)
#pragma unroll
        for (int j = 0; j < K; ++j) scv[j] = v[j / 4][j % 4];
    } else {
#pragma unroll
        for (int j = 0; j < K; ++j) scv[j] = sc[min(tid * K + j, kv.max_blocks - 1)];
    }
    // ... and the request's row of the block table: whoever ranks a block gathers its page at the end, from the cache then
    bool bad_page = false;
    int page_at[K];
#pragma unroll
    for (int j = 0; j < K; ++j) page_at[j] = table[min(tid + j * nthreads, kv.max_blocks - 1)];
    // the scoring kernel clamps silently (it clears the error word); out-of-range inputs are reported here
    const int ctx = (tid == 0 && blockIdx.x == 0) ? ctx_clamped(kv, r, ws.header) : ctx_clamped_quiet(kv, r);
    const int N = (ctx + kPage - 1) / kPage;
#pragma unroll
    for (int j = 0; j < K; ++j) bad_page |= tid + j * nthreads < N && (unsigned)page_at[j] >= (unsigned)kv.num_pages;
    if (bad_page) set_error(ws.header, PSA_DEVERR_PAGE_RANGE);
    // ---- reset of the progressive kernel's per-stream state ------------------------------------
    if (tid == 0 && part == 0) {
        StreamCtl *c = &ws.ctl[s];
        // key chunks that may ever be handed out: all of them, or those a fixed budget of blocks covers
        const int nlim = budget_blocks > 0 ? min(N, budget_blocks) : N;
        const unsigned nch = (unsigned)((nlim + KU - 1) / KU);
        c->k_blocks = 0;
        c->key_progress = (unsigned long long)nch << 32;                                  // frontier 0
        for (int g = 0; g < 8; ++g) c->stop[g] = ~0ull;
    }
    if (part == 0) {
        unsigned long long *a = ws.agg + (size_t)s * ws.max_chunks * G;
        for (int i = tid; i < ws.max_chunks * G; i += nthreads) a[i] = kAggSentinel;      // nothing published yet
        unsigned long long *c = ws.carry + (size_t)s * ws.max_groups * G;
        for (int i = tid; i < ws.max_groups * G; i += nthreads) c[i] = kAggSentinel;
    }

    // LDS carve-up of the bucket path: 8*Np bytes + scratch
    uint32_t *skey = reinterpret_cast<uint32_t *>(lds_raw);                   // [Np] key by slot
    uint32_t *cnt = skey + Np;                                                // [Np / 2 + 4] bucket counts, then bases, two to a word
    uint16_t *base = reinterpret_cast<uint16_t *>(cnt);                       // base[b] .. base[b+1]: bucket b's slots
    uint16_t *slot = reinterpret_cast<uint16_t *>(cnt + Np / 2 + 4);          // [Np] logical block by slot
    uint32_t *scratch = reinterpret_cast<uint32_t *>(slot + Np);              // 64 words
    const int NB = Np;                                                        // one bucket per element slot

    uint32_t key[K];
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const int p = tid * K + j;
        key[j] = 0xFFFFFFFFu;
        if (p < N) {
            key[j] = descending_key(scv[j]);
            kmin = min(kmin, key[j]);
            kmax = max(kmax, key[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < K / 2; ++j) cnt[tid * (K / 2) + j] = 0u;
    if (tid < 16) scratch[48 + tid] = 0u;          // [48]: a bucket is too full; [56 + p]: where workgroup p's share begins
    // smallest and largest key: along the rows of lanes, over the wave's four rows, over the waves through LDS
    kmin = row_min16(kmin);
    kmax = row_max16(kmax);
    kmin = min(min(lane_value(kmin, 0), lane_value(kmin, 16)), min(lane_value(kmin, 32), lane_value(kmin, 48)));
    kmax = max(max(lane_value(kmax, 0), lane_value(kmax, 16)), max(lane_value(kmax, 32), lane_value(kmax, 48)));
    if (lane == 0) { scratch[wave] = kmin; scratch[16 + wave] = kmax; }
    lds_barrier();
    const int wl = lane & 15;                      // (at most sixteen waves)
    kmin = row_min16(wl < nwaves ? scratch[wl] : 0xFFFFFFFFu);
    kmax = row_max16(wl < nwaves ? scratch[16 + wl] : 0u);
    // Buckets are equal steps of the SCORE between the largest and the smallest one (not of its bit
    // pattern, which would crowd scores of small magnitude or mixed sign into a few buckets).  Every
    // operation below is monotone in the score, so a block that ranks before another never lands in a
    // later bucket; the exact order inside a bucket is settled by counting.
    const float smax = score_of_key(kmin), span = smax - score_of_key(kmax);
    const bool span_ok = span > 0.0f && span < INFINITY;       // false also for NaN: the fallback ranks then
    const float scale = span_ok ? (float)NB / span : 0.0f;
    int bkt[K], arrival[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        bkt[j] = 0; arrival[j] = 0;
        if (tid * K + j < N) {
            const float fb = (smax - score_of_key(key[j])) * scale;
            int b = fb >= (float)(NB - 1) ? NB - 1 : (int)fb;     // (a NaN compares false and converts to 0)
            b = b < 0 ? 0 : b;
            bkt[j] = b;
            arrival[j] = (int)((atomicAdd(&cnt[b >> 1], 1u << (16 * (b & 1))) >> (16 * (b & 1))) & 0xffffu);
            if (arrival[j] >= kBucketLimit) scratch[48] = 1u;
        }
    }
    lds_barrier();
    // exclusive scan of the bucket counts (K buckets per thread)
    uint32_t c8[K];
#pragma unroll
    for (int j = 0; j < K; ++j) c8[j] = (cnt[tid * (K / 2) + j / 2] >> (16 * (j & 1))) & 0xffffu;
    uint32_t mine = 0, e8[K];
#pragma unroll
    for (int j = 0; j < K; ++j) { e8[j] = mine; mine += c8[j]; }
    const uint32_t incl = wave_prefix_sum(mine);
    if (lane == 63) scratch[32 + wave] = incl;
    lds_barrier();
    const bool too_full = scratch[48] != 0u;
    const uint32_t t0 = row_sum16(wl < wave ? scratch[32 + wl] : 0u) + incl - mine;      // my first bucket's base
#pragma unroll
    for (int j = 0; j < K / 2; ++j) cnt[tid * (K / 2) + j] = (t0 + e8[2 * j]) | ((t0 + e8[2 * j + 1]) << 16);
    if (tid == 0) base[NB] = (uint16_t)N;
    // A workgroup's share of the ranking work is a run of whole buckets (the workgroups of a stream agree on the
    // buckets' ranges, not on the arrangement inside a bucket): share p starts with the first bucket that begins at
    // or after slot p * N / nparts.  Whoever holds the bucket that slot falls into notes where the next one begins.
    const int share = (N + nparts - 1) / nparts;       // (share 0 starts at slot 0; nparts <= 4)
    for (int p = 1; p < nparts; ++p) {
        const uint32_t target = (uint32_t)min(p * share, N);
        if (t0 < target && target <= t0 + mine) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const uint32_t lo = t0 + e8[j], hi = lo + c8[j];          // bucket's slots [lo, hi)
                if (lo < target && target <= hi) scratch[56 + p] = hi;
            }
        }
    }
    lds_barrier();

    int32_t *ord = ws.order + (size_t)s * kv.max_blocks;
    int32_t *rpage = ws.ranked_page + (size_t)s * kv.max_blocks;
    int32_t *oout = order_out ? order_out + (size_t)s * kv.max_blocks : nullptr;

    // With a second tier, a block whose slice has a slot is read from the slot: ranked_page then holds ~slot (< 0).
    auto location = [&](int page) {
        if constexpr (!TIER) return page;
        const int slot = slot_of[kv.slice_base + (long long)page * kv.num_kv_heads + s % kv.num_kv_heads];
        return slot >= 0 ? ~slot : page;
    };
    if (!too_full && !force_bitonic) {
        // every workgroup of the stream builds its share of the slot table: the elements of a bucket side by side, in
        // arrival order (which may differ between the workgroups; the exact count below does not depend on it) ...
        const int first = (int)scratch[56 + part];
        const int last = part == nparts - 1 ? N : (int)scratch[56 + part + 1];
        const int mine = last - first;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const uint32_t at = (uint32_t)base[bkt[j]] + (uint32_t)arrival[j];
            if (tid * K + j < N && at >= (uint32_t)first && at < (uint32_t)last) {
                slot[at] = (uint16_t)(tid * K + j);
                skey[at] = key[j];
            }
        }
        lds_barrier();
        // ... and ranks its own share of the SLOTS, all threads taking part: thread t takes slots first + t,
        // first + t + nthreads, ...  Neighbouring lanes hold neighbouring slots, that is the same bucket or the
        // next, so a wave's reads of the bucket's members are mostly the same addresses.  The final rank of a
        // slot's element is its bucket's base plus the number of the bucket's members that precede it under
        // (key, block index).
        for (int q0 = 0; q0 < mine; q0 += 2 * nthreads) {         // two slots per thread and turn
            uint32_t mk[2], me[2], b0[2], cn[2], before[2], cmax = 0;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int q = q0 + tid + j * nthreads;
                mk[j] = 0; me[j] = 0; b0[j] = 0; cn[j] = 0; before[j] = 0;
                if (q < mine) {
                    mk[j] = skey[first + q];
                    me[j] = slot[first + q];
                    const float fb = (smax - score_of_key(mk[j])) * scale;     // the bucket, exactly as it was computed above
                    int b = fb >= (float)(NB - 1) ? NB - 1 : (int)fb;
                    b = b < 0 ? 0 : b;
                    b0[j] = base[b];
                    cn[j] = (uint32_t)base[b + 1] - b0[j];
                    cmax = max(cmax, cn[j]);
                }
            }
            for (uint32_t i = 0; i < cmax; ++i) {
                uint32_t ko[2], so[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {              // reads past a bucket's end stay inside the table
                    const uint32_t at = min(b0[j] + i, (uint32_t)(Np - 1));
                    ko[j] = skey[at];
                    so[j] = slot[at];
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const bool precedes = ko[j] < mk[j] || (ko[j] == mk[j] && so[j] < me[j]);
                    before[j] += (i < cn[j] && precedes) ? 1u : 0u;
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (q0 + tid + j * nthreads < mine) {
                    const uint32_t rank = b0[j] + before[j];
                    ord[rank] = (int)me[j];
                    rpage[rank] = location(clamp_page_quiet(table[me[j]], kv.num_pages));
                    if (oout) oout[rank] = (int)me[j];
                }
            }
        }
    } else if (part == 0) {     // (uniform over the workgroup) the fallback is one workgroup's work
        __syncthreads();   // everyone is done with the bucket arrays before LDS is reused
        const int holders = Np / 8;
        if (K < 8 && __builtin_amdgcn_readfirstlane(tid) >= holders) {
            bitonic_barriers(Np);
            return;
        }
        unsigned long long e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int p = tid * 8 + j;
            e[j] = p < N ? (((unsigned long long)descending_key(sc[p]) << 32) | (unsigned)p) : ~0ull;
        }
        bitonic_sort(e, lds_raw, Np, tid, holders);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int p = tid * 8 + j;
            if (p < N) {
                const int b = (int)(e[j] & 0xffffffffull);
                ord[p] = b;
                rpage[p] = location(clamp_page_quiet(table[b], kv.num_pages));
                if (oout) oout[p] = b;
            }
        }
        if (oout)
            for (int p = N + tid; p < kv.max_blocks; p += holders) oout[p] = -1;
        return;
    }
    if (oout && part == 0)
        for (int p = N + tid; p < kv.max_blocks; p += nthreads) oout[p] = -1;
}

template <bool TIER>
static hipError_t launch_order_t(dim3 grid, const KvView &kv, const DecodeWs &ws, int G, const DecodePlan &plan, int budget, int Np,
                                 const int32_t *slot_of, int32_t *order_out, hipStream_t st) {
    const size_t lds = (size_t)Np * 8 + 512;
    const int KU = plan.chunk_blocks, bitonic = plan.force_bitonic;
    if (Np <= 2048) {
        order_kernel<2, TIER><<<grid, Np / 2, lds, st>>>(kv, ws, G, KU, budget, Np, bitonic, slot_of, order_out);
    } else if (Np == 4096) {
        order_kernel<4, TIER><<<grid, Np / 4, lds, st>>>(kv, ws, G, KU, budget, Np, bitonic, slot_of, order_out);
    } else {
        static OncePerDevice once;
        const hipError_t e = allow_dynamic_lds(once, order_kernel<8, TIER>, kMaxBlocks * 8 + 512);
        if (e != hipSuccess) return e;
        order_kernel<8, TIER><<<grid, Np / 8, lds, st>>>(kv, ws, G, KU, budget, Np, bitonic, slot_of, order_out);
    }
    return hipGetLastError();
}

hipError_t launch_order(const KvView &kv, const DecodeWs &ws, int G, const DecodePlan &plan, int budget_blocks,
                        const int32_t *slot_of, int32_t *order_out, hipStream_t st) {
    const int S = kv.batch * kv.num_kv_heads;
    int Np = 512;
    while (Np < kv.max_blocks) Np <<= 1;
    // with few streams, up to 4 workgroups share a stream's ranking
    int parts = 256 / (S > 0 ? S : 1);
    parts = parts < 1 ? 1 : (parts > 4 ? 4 : parts);
    if (Np < 2048) parts = 1;
    return slot_of ? launch_order_t<true>(dim3(parts, S), kv, ws, G, plan, budget_blocks, Np, slot_of, order_out, st)
                   : launch_order_t<false>(dim3(parts, S), kv, ws, G, plan, budget_blocks, Np, slot_of, order_out, st);
}

}  // namespace psa
