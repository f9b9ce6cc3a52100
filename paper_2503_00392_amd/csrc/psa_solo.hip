// A whole decode step in one launch for short contexts: one workgroup per (request, KV head) scores, ranks, reads keys,
// applies the stop rule, reads values and merges, with everything it hands from step to step in LDS.
//
// What bounds a short request is not memory but the chain of dependent launches: the general path's kernels (five, when
// this was measured) take 28 us one after the other at 1024 tokens (8 streams), 35 at 4096, of which each spends 4 to 9 us on
// being started, on its first loads and on draining, and the selection kernel another 4 on passing words between workgroups.
// One workgroup of sixteen waves has no one to wait for: a barrier replaces a launch, LDS replaces the workspace.
// 1024 tokens, 8 streams, G = 4: 28.0 -> 14.4 us; 256 streams: 38.2 -> 19.7; 2048 tokens: 30.8 -> 18.4 and 47.9 -> 28.1;
// 4096 tokens, 256 streams: 60.4 -> 44.0.  What bounds it then is what one compute unit can have in flight between the
// barriers: with 8 streams its waves wait for 58 to 70 % of their time and its vector ALUs are busy 27 to 37 % (by counters).
// Reading keys a step ahead, or four value slices instead of two, ran out of registers and was 5 to 20 % slower.
//
// The results are bit for bit those of the general path: the same products (scores on the matrix cores where that forms
// them there), the same chunks of 32 ranked blocks with the same trees of sums (psa_fold.h), the same value units summed by
// four waves each, the same merge.
#include "psa_attend.h"
#include "psa_fold.h"
#include "psa_host.h"

namespace psa {

constexpr int kSoloChunk = 32;                             // ranked blocks per chunk and value unit, as in the general path
constexpr int kSoloUnits = kSoloBlocks / kSoloChunk;       // 8: one group of the fold at every G
constexpr int kSoloWaves = 16;
constexpr int kSoloStep = 64;                              // ranked blocks whose keys are read between two looks at the rule

template <int G>
struct SoloShared {
    union {
        uint4 stage[kSoloWaves][16 * 17];                  // per wave: one key slice in transposition
        float acc[kSoloWaves][G][kHeadDim];                // per wave: numerator of its blocks of a value unit
    };
    uint4 qb[4][64];                                       // B operand of the key product, by lane
    __attribute__((aligned(16))) float lg[kSoloStep][G][kPage];   // logits of the step's blocks
    float partial[kSoloUnits][G][kHeadDim];                // per value unit: numerator
    float ref[kSoloUnits][G], den[kSoloUnits][G];          // ... its reference and its sum of weights
    float l[kSoloWaves][G];
    float Lb[kSoloBlocks][G];                              // per ranked block: log2-sum-exp2
    float aggL[kSoloUnits][G], aggMin[kSoloUnits][G];      // per chunk
    float testL[kSoloUnits][G], testMin[kSoloUnits][G];    // the same up to the last tested position (see last_test)
    __attribute__((aligned(16))) uint32_t key[kSoloBlocks];   // ranking key by logical block
    int page[kSoloBlocks];                                 // by logical block
    int order[kSoloBlocks];                                // logical block by rank
    unsigned long long stop[G];
    int finished;
};

// Bits of the sticky error word for everything this call's tables and lengths hold, found by one workgroup of its own:
// a workgroup that only looks at its own request could not clear the word before the others write it.
__device__ __forceinline__ void solo_report(const KvView &kv, int32_t *header) {
    // A wave takes four requests at a time, a lane every 64th block: all their loads are in flight at once (one entry per
    // thread and turn, in the grid's last workgroup, made a call of 1024 requests of one KV head 155 us long; 101 now).
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int bits = 0;
    for (int r0 = 4 * wave; r0 < kv.batch; r0 += 4 * kSoloWaves) {
        int raw[4], page[4][kSoloBlocks / 64];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = min(r0 + u, kv.batch - 1);
            raw[u] = kv.ctx_lens[r];
#pragma unroll
            for (int k = 0; k < kSoloBlocks / 64; ++k)
                page[u][k] = kv.block_table[(size_t)r * kv.max_blocks + min(64 * k + lane, kv.max_blocks - 1)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ctx = max(0, min(raw[u], kv.max_blocks * kPage)), N = (ctx + kPage - 1) / kPage;
            if (raw[u] != ctx) bits |= PSA_DEVERR_CTX_RANGE;
#pragma unroll
            for (int k = 0; k < kSoloBlocks / 64; ++k)
                if (64 * k + lane < N && (unsigned)page[u][k] >= (unsigned)kv.num_pages) bits |= PSA_DEVERR_PAGE_RANGE;
        }
    }
    const int page_bad = __syncthreads_or(bits & PSA_DEVERR_PAGE_RANGE), ctx_bad = __syncthreads_or(bits & PSA_DEVERR_CTX_RANGE);
    if (tid == 0) {
        header[0] = 0;
        header[1] = (page_bad ? PSA_DEVERR_PAGE_RANGE : 0) | (ctx_bad ? PSA_DEVERR_CTX_RANGE : 0);
    }
}

// grid (1 + S), 1024 threads; the first workgroup writes the error word.  MFMA: scores on the matrix cores.
template <int DT, int G, int SCORER, bool MFMA>
__global__ __launch_bounds__(kSoloThreads) void solo_kernel(KvView kv, DecodeWs ws, const uint8_t *__restrict__ q,
                                                    const uint8_t *__restrict__ meta, float eps, int m, int budget,
                                                    float *__restrict__ out, int32_t *__restrict__ n_selected,
                                                    float *__restrict__ mass_est, int32_t *__restrict__ blocks_read,
                                                    float *__restrict__ lse_out, int32_t *__restrict__ order_out,
                                                    float *__restrict__ scores_out, int32_t *__restrict__ traffic_out) {
    extern __shared__ __attribute__((aligned(16))) unsigned char solo_lds[];
    SoloShared<G> &sh = *reinterpret_cast<SoloShared<G> *>(solo_lds);
    if (blockIdx.x == 0) { solo_report(kv, ws.header); return; }       // (first, so that it is over before the last stream)
    const int s = (int)blockIdx.x - 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rg = lane >> 4, cl = lane & 15;
    const int r = s / kv.num_kv_heads, h = s % kv.num_kv_heads;
    const int32_t *table = kv.block_table + (size_t)r * kv.max_blocks;
    const uint8_t *qh = q + (size_t)(r * kv.num_q_heads + h * G) * kRowBytes;     // the group's queries
    // everything the workgroup needs first, asked for at once: pages, queries in both layouts, the length
    const int lb = 16 * wave + cl;                             // block whose page this lane holds (lanes 0..15, repeated)
    int page_of_lane = table[min(lb, kv.max_blocks - 1)];
    uint4 qw[MFMA ? 4 : G];                                    // (MFMA: the lane's part of the B operand, head cl)
#pragma unroll
    for (int g = 0; g < (MFMA ? 4 : G); ++g) {
        if constexpr (MFMA) {
            qw[g] = ld16(qh + (size_t)min(cl, G - 1) * kRowBytes + (4 * g + rg) * 16);
            if (cl >= G) qw[g] = make_uint4(0, 0, 0, 0);
        } else {
            qw[g] = ld16(qh + (size_t)g * kRowBytes + cl * 16);
        }
    }
    if (tid < 256) {                                           // (see load_queries of the selection kernel)
        const int kk = tid >> 6, n = tid & 15, kq = (tid & 63) >> 4;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (n < G) v = ld16(qh + (size_t)n * kRowBytes + (4 * kk + kq) * 16);
        sh.qb[kk][tid & 63] = v;
    }
    const int ctx = ctx_clamped_quiet(kv, r);
    const int N = (ctx + kPage - 1) / kPage;                   // <= max_blocks <= kSoloBlocks
    page_of_lane = lb < N ? clamp_page_quiet(page_of_lane, kv.num_pages) : 0;

    // ---- scores (line 5): wave w takes blocks 16 w .. 16 w + 15 -----------------------------------------------------
    if (16 * wave < N) {
        auto put = [&](int blk, float cs) {
            sh.key[blk] = descending_key(cs);
            if (scores_out) scores_out[(size_t)s * kv.max_blocks + blk] = cs;
        };
        if constexpr (MFMA) {
            // one product over the blocks' records, row = block, as score_mfma_kernel forms it: whole rows are loaded (four
            // to an instruction) and turned into the operand's layout through the wave's patch, the minima first
            uint4 a[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = min(4 * (i & 3) + rg, N - 1 - 16 * wave);     // (clamped: the loads need no branch)
                const size_t record = (size_t)__shfl(page_of_lane, j) * kv.num_kv_heads + h;
                a[i] = ld16_stream(meta + record * kMetaBytes + (i >> 2) * 256 + cl * 16);
            }
            const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
            f32x4_t part[8];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int i = 0; i < 4; ++i) sh.stage[wave][(4 * i + rg) * 17 + cl] = a[4 * half + i];
                lds_wave_sync();
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    uint32_t w[4] = {qw[kk].x, qw[kk].y, qw[kk].z, qw[kk].w};
                    if constexpr (SCORER == 0) {
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            const uint32_t neg = ((w[x] >> 15) & 0x00010001u) * 0xFFFFu;
                            w[x] &= half ? ~neg : neg;
                        }
                    }
                    part[4 * half + kk] = mfma_16x16x32<DT>(sh.stage[wave][cl * 17 + 4 * kk + rg],
                                                            make_uint4(w[0], w[1], w[2], w[3]), zero);
                }
                lds_wave_sync();
            }
            const f32x4_t d = sum_tree(part);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const float cs = row_max16(cl < G ? d[x] : -INFINITY) * (SCORER == 1 ? 0.5f * kScale : kScale);
                const int blk = 16 * wave + 4 * rg + x;
                if (cl == 0 && blk < N) put(blk, cs);
            }
        } else {
            // sixteen lanes to a block, four blocks a step, packed dots
            constexpr int kRecord = SCORER == 2 ? 256 : kMetaBytes;
            uint4 lo[4], hi[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int j = min(4 * it + rg, N - 1 - 16 * wave);     // (clamped: the loads need no branch)
                const uint8_t *mp = meta + ((size_t)__shfl(page_of_lane, j) * kv.num_kv_heads + h) * kRecord + cl * 16;
                lo[it] = ld16_stream(mp);
                hi[it] = SCORER == 2 ? make_uint4(0, 0, 0, 0) : ld16_stream(mp + 256);
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const uint32_t a[4] = {lo[it].x, lo[it].y, lo[it].z, lo[it].w};
                const uint32_t b[4] = {hi[it].x, hi[it].y, hi[it].z, hi[it].w};
                float cs = -INFINITY;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const uint32_t w[4] = {qw[g].x, qw[g].y, qw[g].z, qw[g].w};
                    float p = 0.0f;
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const uint32_t neg = ((w[x] >> 15) & 0x00010001u) * 0xFFFFu;   // 0xFFFF in each negative half
                        p = dot2<DT>(a[x], SCORER ? w[x] : (w[x] & neg), p);
                    }
                    if constexpr (SCORER != 2) {
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            const uint32_t neg = ((w[x] >> 15) & 0x00010001u) * 0xFFFFu;
                            p = dot2<DT>(b[x], SCORER ? w[x] : (w[x] & ~neg), p);
                        }
                    }
                    p = row_sum16(p);
                    cs = fmaxf(cs, p * (SCORER == 1 ? 0.5f * kScale : kScale));
                }
                const int blk = 16 * wave + 4 * it + rg;
                if (cl == 0 && blk < N) put(blk, cs);
            }
        }
        if (lane < 16 && lb < N) sh.page[lb] = page_of_lane;
    }
    if (tid < G) sh.stop[tid] = ~0ull;
    if (tid < kSoloBlocks && tid >= N) sh.key[tid] = 0xFFFFFFFFu;      // (precedes nothing)
    lds_barrier();

    // ---- ranking (line 6): four threads to a block, each counts a quarter of the blocks that precede it ------------
    {
        const int e = tid >> 2, part = tid & 3;
        if (e < N) {
            const uint32_t mine = sh.key[e];
            int before = 0;
            for (int j = part * 4; j < N; j += 16) {
                const uint4 o = *reinterpret_cast<const uint4 *>(&sh.key[j]);
                before += (o.x < mine || (o.x == mine && j < e)) ? 1 : 0;
                before += (o.y < mine || (o.y == mine && j + 1 < e)) ? 1 : 0;
                before += (o.z < mine || (o.z == mine && j + 2 < e)) ? 1 : 0;
                before += (o.w < mine || (o.w == mine && j + 3 < e)) ? 1 : 0;
            }
            before += __shfl_xor(before, 1);
            before += __shfl_xor(before, 2);
            if (part == 0) sh.order[before] = e;
        }
    }
    lds_barrier();
    if (order_out)
        for (int x = tid; x < kv.max_blocks; x += 1024) order_out[(size_t)s * kv.max_blocks + x] = x < N ? sh.order[x] : -1;

    // ---- keys and the stop rule (lines 7-18), 64 ranked blocks at a time ----------------------------------------
    const int nlim = budget > 0 ? min(N, budget) : N;
    const int nch = (nlim + kSoloChunk - 1) / kSoloChunk;      // chunks that may ever be folded
    eps = stop_threshold(eps, budget, N);
    float *logits = ws.logits + (size_t)s * kv.max_blocks * (kPage * G);
    int nread = 0;                                             // key slices read (traffic accounting)
    if (nch > 0) {
        int walked = 0;
        for (int b0 = 0; b0 < min(N, nch * kSoloChunk); b0 += kSoloStep) {
            const int nblk = min(kSoloStep, min(N, nch * kSoloChunk) - b0);
            nread = b0 + nblk;
            {
                uint4 ka[4][4], qb[4];                         // (qb from LDS every step: registers are short here)
                int blk[4];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) qb[kk] = sh.qb[kk][lane];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    blk[u] = sh.order[b0 + min(wave + kSoloWaves * u, nblk - 1)];      // (clamped: no branch around a load)
                    const uint8_t *kp = kv.k_pool + ((size_t)sh.page[blk[u]] * kv.num_kv_heads + h) * kSliceBytes + lane * 16;
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) ka[u][kk] = ld16_stream(kp + kk * 1024);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = wave + kSoloWaves * u;
                    if (i < nblk) {
                        const f32x4_t sc = block_logits<DT>(ka[u], qb, sh.stage[wave], lane, min(kPage, ctx - blk[u] * kPage));
                        if (cl < G) *reinterpret_cast<f32x4_t *>(&sh.lg[i][cl][4 * rg]) = sc;
                    }
                }
            }
            lds_barrier();
            rows_lse<G, 1024>(&sh.lg[0][0][0], &sh.Lb[b0][0], nblk * G, tid);
            for (int x = tid * 4; x < nblk * G * kPage; x += 4096)
                *reinterpret_cast<f32x4_t *>(logits + (size_t)b0 * G * kPage + x) =
                    *reinterpret_cast<const f32x4_t *>(&sh.lg[0][0][0] + x);
            lds_barrier();
            if (wave < kSoloStep / kSoloChunk && wave * kSoloChunk < nblk) {
                float aggL, aggMin;
                const int c = b0 / kSoloChunk + wave;
                chunk_aggregate<G>(&sh.Lb[c * kSoloChunk][0], min(kSoloChunk, nblk - wave * kSoloChunk), lane, aggL, aggMin);
                if (lane < G) { sh.aggL[c][lane] = aggL; sh.aggMin[c][lane] = aggMin; }
                if (split_words(kSoloChunk, m, budget)) {
                    const int c0 = c * kSoloChunk;
                    chunk_aggregate<G>(&sh.Lb[c0][0], last_test(c0, min(c0 + kSoloChunk, nlim), m, N) - c0, lane, aggL, aggMin);
                    if (lane < G) { sh.testL[c][lane] = aggL; sh.testMin[c][lane] = aggMin; }
                }
            }
            lds_barrier();
            if (wave == 0) {
                int ln = lane;                                 // (opaque: what derives from it is not kept from before the loop)
                asm volatile("" : "+v"(ln));
                const int g = ln % G, jl = ln / G, k = (b0 + nblk + kSoloChunk - 1) / kSoloChunk;
                const float L = jl < k ? sh.aggL[jl][g] : -INFINITY, M = jl < k ? sh.aggMin[jl][g] : INFINITY;
                const bool split = split_words(kSoloChunk, m, budget) && jl < k;
                const float LT = split ? sh.testL[jl][g] : -INFINITY, MT = split ? sh.testMin[jl][g] : INFINITY;
                unsigned long long stop = sh.stop[g];          // lane = (chunk, head)
                bool all = false;
                walked = fold_group<G, (kSoloChunk * G + 63) / 64>(L, M, LT, MT, stop, walked, k, N, m, kSoloChunk, budget, eps, all,
                                                                    [&](int b, int i) { return (&sh.Lb[b][0])[i]; }, ln);
                if (ln < G) sh.stop[ln] = stop;
                if (ln == 0) sh.finished = all || walked >= nch;
            }
            lds_barrier();
            if (sh.finished) break;
        }
    }
    // ---- values (lines 10-12): four waves to a unit of 32 ranked blocks, as in the general path's chunks ----------
    const unsigned long long my_stop = sh.stop[lane % G];      // head lane % G's
    const int n_mine = (my_stop != ~0ull && (int)(my_stop >> 32) <= N) ? (int)(my_stop >> 32) : N;
    int nmax = n_mine;
#pragma unroll
    for (int d = 1; d < G; d <<= 1) nmax = max(nmax, __shfl_xor(nmax, d));
    nmax = __builtin_amdgcn_readfirstlane(nmax);
    const int hd = cl >> 1, n_hd = __shfl(n_mine, hd);         // the head whose weights the lane supplies (see add_weighted)
    const int units = (nmax + kSoloChunk - 1) / kSoloChunk;
    __syncthreads();                                           // (the logits are in memory, the LDS patches are free)
    for (int u0 = 0; u0 < units; u0 += 4) {
        const int unit = u0 + (wave >> 2), w4 = wave & 3, start = unit * kSoloChunk;
        const int nblk = min(kSoloChunk, N - start), maxcnt = min(nblk, nmax - start);
        if (maxcnt > 0) {                                      // (uniform over the wave)
            const int jmax = (maxcnt - w4 + 3) / 4;            // the wave's blocks: w4, w4 + 4, ...
            const int mycnt = min(nblk, max(0, n_mine - start)), hdcnt = min(nblk, max(0, n_hd - start));
            float Lc = -INFINITY;                              // the unit's reference, of head lane % G first
            for (int i = lane / G; i < mycnt; i += 64 / G) Lc = fmaxf(Lc, sh.Lb[start + i][lane % G]);
#pragma unroll
            for (int d = G; d < 64; d <<= 1) Lc = fmaxf(Lc, __shfl_xor(Lc, d));
            Lc = __shfl(Lc, hd);
            const float *lg = logits + (size_t)start * (kPage * G) + (size_t)(hd < G ? hd : 0) * kPage + 4 * rg;
            f32x4_t acc[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            float l = 0.0f;
            constexpr int kDepth = 2;
            for (int j0 = 0; j0 < jmax; j0 += kDepth) {
                Slice v[kDepth];
                f32x4_t x[kDepth];
                int valid[kDepth], blk[kDepth];
#pragma unroll
                for (int u = 0; u < kDepth; ++u) {
                    blk[u] = w4 + 4 * min(j0 + u, jmax - 1);
                    const int b = sh.order[start + blk[u]];
                    v[u] = load_slice(kv.v_pool + ((size_t)sh.page[b] * kv.num_kv_heads + h) * kSliceBytes, lane);
                    x[u] = *reinterpret_cast<const f32x4_t *>(lg + (size_t)blk[u] * (kPage * G));
                    valid[u] = min(kPage, ctx - b * kPage);
                }
#pragma unroll
                for (int u = 0; u < kDepth; ++u) {
                    if (j0 + u < jmax) {
                        if (valid[u] < kPage) zero_invalid_rows(v[u], rg, valid[u]);
                        add_values<DT>(acc, l, v[u], x[u], hd < G && blk[u] < hdcnt, Lc, cl & 1);
                    }
                }
            }
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            store_heads<G>(acc, sh.acc[wave], rg, cl);
            if (rg == 0 && hd < G && !(cl & 1)) {
                sh.l[wave][hd] = l;
                if (w4 == 0) sh.ref[unit][hd] = Lc;
            }
        }
        lds_barrier();
        if (unit < units) {
            const int w0 = wave & ~3;
            for (int x = tid & 255; x < G * kHeadDim; x += 256) {
                const int g = x / kHeadDim, ch = x % kHeadDim;
                sh.partial[unit][g][ch] =
                    (sh.acc[w0][g][ch] + sh.acc[w0 + 1][g][ch]) + (sh.acc[w0 + 2][g][ch] + sh.acc[w0 + 3][g][ch]);
                if (ch == 0) sh.den[unit][g] = (sh.l[w0][g] + sh.l[w0 + 1][g]) + (sh.l[w0 + 2][g] + sh.l[w0 + 3][g]);
            }
        }
        lds_barrier();
    }
    // ---- merge (line 19), in the general path's order of sums -----------------------------------------------
    for (int x = tid; x < G * kHeadDim; x += 1024) {
#pragma clang fp contract(off)
        const int g = x / kHeadDim, ch = x % kHeadDim;
        const unsigned long long st = sh.stop[g];
        const bool stopped = st != ~0ull && (int)(st >> 32) <= N;
        const int n = stopped ? (int)(st >> 32) : N, nun = (n + kSoloChunk - 1) / kSoloChunk;
        float M = -INFINITY;
        for (int u = 0; u < nun; ++u) M = fmaxf(M, sh.ref[u][g]);
        float t = 0.0f, d[kSoloUnits];
#pragma unroll
        for (int u = 0; u < kSoloUnits; ++u) {
            d[u] = 0.0f;
            if (u < nun) {
                const float mi = sh.ref[u][g];
                const float w = (mi == -INFINITY || M == -INFINITY) ? 0.0f : exp2_fast(mi - M);
                d[u] = sh.den[u][g] * w;
                const float a = sh.partial[u][g][ch] * w;
                t += a;
            }
        }
        const float den = ((d[0] + d[4]) + (d[2] + d[6])) + ((d[1] + d[5]) + (d[3] + d[7]));
        const size_t qi = (size_t)r * kv.num_q_heads + h * G + g;
        out[qi * kHeadDim + ch] = den > 0.0f ? t / den : 0.0f;
        if (ch == 0) {
            n_selected[qi] = n;
            mass_est[qi] = stopped ? __uint_as_float((uint32_t)st) : (N > 0 ? 1.0f : 0.0f);
            if (lse_out) lse_out[qi] = den > 0.0f ? (M + log2_fast(den)) * kLn2 : -INFINITY;
        }
    }
    if (tid == 0) {
        if (blocks_read) blocks_read[s] = nmax;
        if (traffic_out) { traffic_out[2 * s] = nread; traffic_out[2 * s + 1] = nmax; }
    }
}

template <int DT, int G, int SCORER, bool MFMA = false>
static hipError_t launch_solo_t(const KvView &kv, const DecodeArgs &a, const DecodeWs &ws, hipStream_t st) {
    static OncePerDevice once;
    const hipError_t e = allow_dynamic_lds(once, solo_kernel<DT, G, SCORER, MFMA>, sizeof(SoloShared<G>));
    if (e != hipSuccess) return e;
    const unsigned S = (unsigned)(kv.batch * kv.num_kv_heads);
    solo_kernel<DT, G, SCORER, MFMA><<<S + 1, kSoloThreads, sizeof(SoloShared<G>), st>>>(
        kv, ws, (const uint8_t *)a.q, (const uint8_t *)a.meta, a.threshold, a.check_granularity, a.budget_blocks, a.out,
        a.n_selected, a.mass_est, a.blocks_read, a.lse_out, a.order_out, a.scores_out, a.traffic_out);
    return hipGetLastError();
}

template <int DT, int G>
static hipError_t launch_solo_g(const KvView &kv, const DecodeArgs &a, const DecodeWs &ws, hipStream_t st) {
    if constexpr (G >= 8) {
        if (score_on_matrix_cores(G, kv.num_kv_heads, a.scorer))
            return a.scorer == 1 ? launch_solo_t<DT, G, 1, true>(kv, a, ws, st) : launch_solo_t<DT, G, 0, true>(kv, a, ws, st);
    } else if (a.scorer == 0) {
        return launch_solo_t<DT, G, 0>(kv, a, ws, st);
    }
    return a.scorer == 2 ? launch_solo_t<DT, G, 2>(kv, a, ws, st) : launch_solo_t<DT, G, 1>(kv, a, ws, st);
}

hipError_t launch_solo(const KvView &kv, int dtype, int G, const DecodeArgs &a, const DecodeWs &ws, hipStream_t st) {
#define PSA_CASE(DT, GG) \
    if (dtype == DT && G == GG) return launch_solo_g<DT, GG>(kv, a, ws, st);
    PSA_CASE(0, 1) PSA_CASE(0, 2) PSA_CASE(0, 4) PSA_CASE(0, 8)
    PSA_CASE(1, 1) PSA_CASE(1, 2) PSA_CASE(1, 4) PSA_CASE(1, 8)
#undef PSA_CASE
    return hipErrorInvalidValue;
}

}  // namespace psa
