// Progressive selection and attention (Algorithm 1, lines 7-18): walks every stream's ranked blocks, computes the
// exact scaled logits q.k/sqrt(d) of each block from its key slice, decides on the GPU where every query head stops, and
// multiplies the selected blocks' weights with their value slices.
//
// Terms.  "Stream": one (request, KV head) pair -- one ranking, G query heads.  "Chunk": CB
// consecutive ranked blocks, the unit of work of a workgroup.
//
// One workgroup (4 waves) per (chunk, stream), in a one-dimensional grid with the streams varying
// fastest: the hardware hands workgroups out in that order, so each stream's chunks start in rank
// order, interleaved over the streams, and a compute unit takes the next one the moment a slot is free
// (four fit).  A workgroup
//   1. returns at once if its chunk lies beyond the stream's blocks or beyond the limit the fold has set
//      (the stream is closed, or cannot go that far any more);
//   2. fetches the chunk's page numbers and waits (napping about a microsecond between looks at one
//      progress word, a bounded number of times) until the chunk is inside the read-ahead window --
//      chunks read beyond the fold's frontier are at most max(window, frontier/4), 256 at most, which
//      bounds the keys read beyond the stop -- or the limit falls below it (with a second tier, a
//      chunk that has slices in host memory waits until the fold is one chunk away, unless it lies
//      inside the depth hint: the host link is too slow to read ahead over it);
//   3. reads the chunk's key slices (each wave keeps 4 slices = 16 KiB in flight, loaded as coalesced
//      1 KiB rows and turned into the matrix-operand layout through a patch of LDS), computes the
//      scaled logits of all G heads as a 16-token x 16-head x 128-channel product on the matrix
//      cores (heads beyond G are zero columns), keeps them in LDS until the chunk is done, and then reduces
//      every block's log-sum-exp L_b (= log AS of line 10) at once;
//   4. publishes the chunk's (log-sum-exp, minimum) of L_b per head as one 64-bit word per head;
//   5. waits for the words of the chunks before it and finds how many of its blocks every head uses -- a head stops in the
//      first chunk at whose last tested position P_acc exceeds the threshold, and if that is this one, at a block that a
//      prefix scan over the chunk's L_b finds (words that do not come, it makes itself: see settle_chunk);
//   6. reads those value slices, and leaves the chunk's part of the output (reference, sum of weights, numerator) for the
//      final merge.
// Keys and values in one kernel: the logits stay in LDS.  In a kernel of its own the value pass had them written to memory
// and read back (6 % of the keys' bytes at G = 4, 12 % at G = 8, and writes cost this kernel several times their bytes), and
// it could not begin before the last stream's fold had ended, nor the launch gap be hidden; here the values of the streams
// that stop early are read while the deep ones are still folding.  Two kernels -> one (median of repeated calls, all builds
// in turn on one machine, here and below): 32K tokens, batch 8 103.2 -> 88.4 us a call, four layers at 128K 758 -> 684, 64
// ragged requests at G = 8 1555 -> 1361, everything selected (64K, batch 16) 848 -> 761, one request of 4K tokens 32.1 ->
// 29.0.  A slot is held while a workgroup waits for the fold, which is why this lost in an earlier form with fewer resident
// workgroups: four fit a compute unit with two value slices in flight per wave (128 registers); three with four slices were
// 4 % slower at G = 8, and no faster elsewhere.  Value slices asked for before the fold's answer, where the stream was
// likely to need them, made no difference.
// From the last key to the published word a chunk takes 0.9 us, and 3.2 us from its first load on an idle chip; with
// the reduction inside the loop over the slices, and the words after all stores, these were 1.0 us (3 us under load)
// and 4.6 us.  A call at 32K tokens, batch 8, went from 112.5 to 109.7 us, at 4K, batch 31, from 58.1 to 54.1.
// The wait of step 2 is a courtesy: when the looks run out the workgroup simply reads its chunk.  The wait of step 5 is for the
// words of chunks of the same stream that come before, whose workgroups have smaller indexes.  Within one launch those have
// always started: the hardware starts workgroups in the order of their indexes (within each of the chip's partitions), so the
// one with the smallest index that is not done waits for none that has not.  Beside another launch that does not hold: the
// waiting workgroups of one call can fill a partition while the next chunk of the other is queued behind them, and the other
// way round.  So nobody relies on it: when the looks of step 5 run out, the workgroup reads the missing chunks itself and makes
// their words and, at the end of a group, the carry.  Every workgroup that has started then ends without any that has not, in
// whatever order they are started.
// THE FOLD applies lines 12-17 chunk by chunk, strictly in rank order, to steer the reading: AS_acc, AS_min and P_acc at the
// last tested position of each published chunk after the frontier say in which chunk every head stops.  One wave per stream
// does it, in workgroups of its own at the head of the grid (so they start first): it looks at the words of the next chunks,
// folds what is published, moves the frontier, tells the readers how far the stream can still go (stop_bound), and looks
// again.  Once every head has stopped (or the blocks ran out) it closes the stream: the chunks beyond what it used are never
// read.  Chunks are folded in groups (see fold_stream); the workgroup of a group's last chunk leaves the state after it in a
// carry word per head, from which the next group's workgroups go on by themselves in step 5.  They had waited for the fold
// to pass their chunk and to hand out the stops before, which it found from the L_b in memory: a chunk's way from its word
// to its values was then the fold's look, its arithmetic, a load of the L_b, two stores one after the other, and the
// workgroup's look and load of the stops -- 3.7 to 5.2 us on an idle chip and 7.5 in the median of a busy one.  One request
// of 4K tokens 29.0 -> 26.8 us a call, 32K tokens, batch 8 88.4 -> 84.7, four layers at 128K 684 -> 672, 64 ragged requests
// at G = 8 1361 -> 1331, two tiers 522 -> 502.  (With every waiting workgroup looking at its group's words all the time,
// instead of at one word until the fold has come to the group, everything selected at 64K, batch 16, took 820 us instead of
// 766.)
//
// Communication between workgroups: every shared word is read and written with relaxed agent-scope
// atomics (coherent accesses); a writer waits for its data stores to complete before it stores the
// word that announces them (the chunk words, the progress word), and a reader looks at the announcing
// word before it issues the loads that depend on it.  Accesses to one cache line are served one at a
// time (tens of nanoseconds each), which is why one thread per workgroup touches the stream's control
// block.  The chunks' partial outputs and the heads' stops are plain stores: their reader is the next kernel.
//
// The fold is one scan in rank order and every reduction has a fixed shape, so results are bitwise
// reproducible although the scheduling is dynamic.
#include "psa_attend.h"
#include "psa_fold.h"
#include "psa_host.h"

namespace psa {

// ---- agent-scope atomics ---------------------------------------------------------------------
__device__ __forceinline__ int ld_relaxed(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_relaxed(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_relaxed(const float *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(unsigned long long *p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(float *p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every word one wave writes and another reads inside this kernel travels through the relaxed
// agent-scope atomics above (cache-coherent accesses), never through plain loads and stores, so no
// cache write-back or invalidation is ever needed.  What remains is ORDER: a wave's earlier
// stores must have completed before the store that announces them is issued.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ unsigned long long pack2(float a, float b) {
    return ((unsigned long long)__float_as_uint(b) << 32) | __float_as_uint(a);
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }


constexpr int kKeyDepth = 4;         // key slices a wave keeps in flight
constexpr int kValueDepth = 2;       // value slices a wave keeps in flight
constexpr int kSelectThreads = 256;  // 4 waves; four such workgroups fit a CU (registers, LDS at G = 8)

// Tokens of stream s's request, clamped like everywhere else.
__device__ __forceinline__ int stream_ctx(const KvView &kv, int s) {
    const int ctx = kv.ctx_lens[s / kv.num_kv_heads];
    return ctx < 0 ? 0 : (ctx > kv.max_blocks * kPage ? kv.max_blocks * kPage : ctx);
}

__device__ __forceinline__ int window_of(int window, int frontier) {
    const int w = max(window, frontier >> 2);
    return w > kMaxWindowChunks ? kMaxWindowChunks : w;
}

__device__ __forceinline__ void nap(int tries) {
    // about half a microsecond, then about one: long enough that the pollers of one stream stay below
    // what one cache line serves, short enough that an opening window is noticed at once
    __builtin_amdgcn_s_sleep(20);
    if (tries > 1) __builtin_amdgcn_s_sleep(20);
}

// MAXB: blocks of a chunk at most, 32 or kMaxChunkBlocks (the size of the patch that holds a chunk's logits).
template <int G, int MAXB>
struct SelectShared {
    uint4 qb[4][64];                       // B operand of the QK^T product of the workgroup's stream, by lane
    float Lb[MAXB][G];                     // per-block log2-sum-exp2
    int page[MAXB];
    int valid[MAXB];
    int entry[MAXB];                       // second tier: the block's entry in the staging buffer, -1 = none (its wave's own)
    int go;                                // after the wait for the window: 1 = read the chunk, 0 = the stream closed
    unsigned long long kp0;                // the stream's progress word as the workgroup first saw it
    uint4 stage[kSelectThreads / 64][16 * 17];   // per wave: one key slice, rows padded to 272 bytes; later its numerators
    // the chunk's logits: position 4 r + j of a (block, head) row holds token 4 j + r
    __attribute__((aligned(16))) float lg[MAXB][G][kPage];
    int cnt[G];                                      // blocks of the chunk each head uses (-1: nobody needs the chunk)
    int next;                                        // the chunk to read next (see settle_chunk), -1 = none
    float st_l[kSelectThreads / 64][G], st_ref[G];   // value phase: per wave the sum of its weights, the reference
};

// How far a stream can still go, in chunks, given what the fold knows after n blocks.  AS_acc only grows and AS_min only
// shrinks as more blocks are folded, so for any n* >= n
//     P_acc(n*) >= AS_acc(n) / (AS_acc(n) + AS_min(n) (N - n*)),
// and the right-hand side exceeds eps as soon as N - n* < (AS_acc(n) / AS_min(n)) (1 - eps) / eps: the head stops at the
// first tested position from there on, whatever the blocks in between hold.  Lane g < G carries head g (stop_end > 0: it has
// stopped in the chunk that ends there; lanes >= G need nothing); the result, the largest need of the group plus one chunk
// to spare against rounding, is the same in every lane.  Keys beyond it are never worth reading.
template <int G>
__device__ __forceinline__ int stop_bound(float Lacc, float Lmin, int stop_end, int n, int N, int m, int KU, float odds) {
    const int lane = threadIdx.x & 63;
    int need = 0;
    if (lane < G) {
        if (stop_end > 0) {
            need = stop_end;
        } else {
            // blocks that may be left over when the test first passes: fewer than ratio * odds (taken a little
            // low, and one lower still: the bound must hold in binary32)
            const float room = exp2_fast(Lacc - Lmin) * odds * 0.999f - 1.0f;
            int nstar = room >= (float)N ? 0 : N - (int)fmaxf(room, 0.0f);     // (NaN compares false: N, no bound)
            nstar = max(nstar, n + 1);
            nstar = (int)min((long long)N, ((long long)nstar + m - 1) / m * m);   // the next tested position
            need = nstar;
        }
    }
#pragma unroll
    for (int d = 1; d < 8; d <<= 1) need = max(need, __shfl_xor(need, d));
    need = uniform(__shfl(need, 0));
    return (need + KU - 1) / KU + 1;
}

// The progress word of a stream (see StreamCtl).
__device__ __forceinline__ unsigned long long progress_word(int lim, int grant, int walked) {
    return ((unsigned long long)(unsigned)lim << 32) | ((unsigned)grant << 16) | (unsigned)walked;
}
__device__ __forceinline__ int progress_frontier(unsigned long long kp) { return (int)(kp & 0xffffull); }
__device__ __forceinline__ int progress_grant(unsigned long long kp) { return (int)((kp >> 16) & 0xffffull); }
__device__ __forceinline__ int progress_limit(unsigned long long kp) { return (int)(kp >> 32); }
// The read-ahead window of a stream when `closed` of the S streams have finished: the launch's total of chunks in
// flight (window per stream x S) shared by the streams still open.
__device__ __forceinline__ int granted(int window, int S, int closed) {
    return min(kMaxWindowChunks, (int)(((long long)window * S) / max(1, S - closed)));
}

// =================================================================================================
// The fold (Algorithm 1 lines 12-18 in rank order, a chunk at a time): one wave per stream, from the kernel's first moment
// until the stream closes.
//
// Chunks are folded a GROUP at a time: 64 / G consecutive chunks, aligned, lane = (chunk of the group, head), kLook groups
// to a look; a look's loads are in flight together.  A sequential walk, chunk by chunk on G lanes, cost a deep stream 0.3 us
// per chunk -- more than reading the chunk costs the rest of the machine.
// The expression that gives the state after a chunk is fixed by the chunk's place in its group (see group_states): the
// fold is reproducible bit for bit although its timing is not, and the chunks' own workgroups find the same bits.
//
// The wave waits for nothing but chunks whose workgroups are in this kernel's grid, and those end without it: they wait for
// the window and for chunks before them, each a bounded number of looks; so it always ends.  A count of looks bounds it all
// the same (kFoldPatience: about half a second in which neither this stream moves nor another one closes), after which the
// stream is closed as it stands and PSA_DEVERR_STALLED is raised.  With more streams than folding waves (4 * kMaxFoldGroups)
// a wave folds several streams, one after the other, and the grid hands out the chunks in the same order: all chunks of the
// streams that are folded first, then those of the next.  A chunk whose fold has not begun would otherwise hold its slot
// until its looks run out, thousands of them all slots there are, while the chunks the folds wait for have not started (4096
// streams of 512 blocks, all selected: 860 ms and PSA_DEVERR_STALLED).
// =================================================================================================
constexpr int kFoldPatience = 1 << 19;
constexpr int kMaxFoldGroups = 128;            // workgroups of four folding waves at most: they must leave the
                                               // compute units room for the chunks they wait for

template <int G>
__device__ void fold_stream(const KvView &kv, const DecodeWs &ws, int s, float eps, int m, int KU, int budget, int window) {
    constexpr int CPG = 64 / G;                // chunks per group
    constexpr int kLook = CPG >= 32 ? 1 : 32 / CPG;   // groups per look: 32 chunks, 64 with one head
    const int lane = threadIdx.x & 63, g = lane % G, jl = lane / G;     // my head, my chunk of the group
    const unsigned long long head_lanes = (~0ull / ((1ull << G) - 1ull)) << g;   // the lanes of my head
    StreamCtl *ctl = &ws.ctl[s];
    const int N = (stream_ctx(kv, s) + kPage - 1) / kPage;
    const unsigned long long *agg = ws.agg + (size_t)s * ws.max_chunks * G;
    const float2 *tested = ws.agg_tested + (size_t)s * ws.max_chunks * G;
    const bool split = split_words(KU, m, budget);
    // chunks that may ever be folded: all of them, or those a fixed budget of blocks covers (the limit in the
    // progress word is for the readers of keys and may be tighter: see stop_bound)
    const int nlim = blocks_that_count(N, budget), nch = (nlim + KU - 1) / KU;
    if (nch == 0) {                            // an empty request: the ranking kernel left it closed
        if (lane == 0) atomicAdd(&ws.header[kClosedStreams], 1);
        return;
    }
    eps = stop_threshold(eps, budget, N);
    const int S = kv.batch * kv.num_kv_heads;
    const float odds = eps > 0.0f ? (1.0f - eps) / eps : INFINITY;      // (1 - eps) / eps of the stop test
    float Cacc = -INFINITY, Cmin = INFINITY;   // my head's (L_acc, L_min) at the start of the group
    float P_end = 0.0f;                        // my head's P_acc at the last position tested in the chunk it stops in
    int stop_end = 0;                          // blocks up to the end of the chunk my head stops in, 0 = still open
    int base = 0, walked = 0;                  // the group's first chunk; chunks folded so far
    int closed = 0, lim_now = nch;             // streams seen closed at the last look; the limit last published
    int looks = 0, seen = 0;                   // looks in vain since the stream moved or another one closed
    bool finished = false;
    while (!finished) {
        // the groups' words, and (in flight at the same time) how many streams have closed
        unsigned long long v[kLook];
#pragma unroll
        for (int u = 0; u < kLook; ++u) {
            const int ci = base + u * CPG + jl;
            v[u] = (ci < nch) ? ld_relaxed(&agg[(size_t)ci * G + g]) : kAggSentinel;
        }
        const int closed_now = uniform(ld_relaxed(&ws.header[kClosedStreams]));
        const int before = walked;
        float Lw = Cacc, Mw = Cmin;            // my head's state at the frontier (for stop_bound)
#pragma unroll
        for (int u = 0; u < kLook; ++u) {
            const unsigned long long pub = __ballot(v[u] != kAggSentinel);
            const int k = ((pub == ~0ull) ? 64 : (__ffsll((long long)~pub) - 1)) / G;     // leading published chunks
            const int j = walked - base;                                                   // of which folded before
            if (finished || k <= j) break;
            float L = __uint_as_float((uint32_t)(v[u] & 0xffffffffull)), M = __uint_as_float((uint32_t)(v[u] >> 32)), E, F, P;
            float LT = -INFINITY, MT = INFINITY;
            if (split) {                       // (written before the chunk's word)
                const size_t at = (size_t)min(base + jl, nch - 1) * G + g;
                LT = ld_relaxed(&tested[at].x);
                MT = ld_relaxed(&tested[at].y);
            }
            group_states<G>(L, M, Cacc, Cmin, E, F, lane);
            const int b0 = (base + jl) * KU;
            const bool passes = chunk_passes(L, M, E, F, split, LT, MT, b0, min(b0 + KU, nlim), N, m, eps, P);
            const unsigned long long mine = __ballot(jl >= j && jl < k && stop_end == 0 && passes) & head_lanes;
            if (mine != 0ull) {
                const int src = __ffsll((long long)mine) - 1;
                stop_end = min((base + src / G + 1) * KU, N);
                P_end = __shfl(P, src);
            }
            if (__ballot(stop_end == 0) == 0ull) {                // every head has stopped: up to the last one's chunk
                int last = stop_end;
#pragma unroll
                for (int d = 1; d < G; d <<= 1) last = max(last, __shfl_xor(last, d));
                walked = uniform((last + KU - 1) / KU);
                finished = true;
            } else {
                walked = base + k;
                if (walked >= nch) finished = true;
                Lw = __shfl(L, (k - 1) * G + g);
                Mw = __shfl(M, (k - 1) * G + g);
                if (k < CPG) break;            // (a later group's words wait for this one's)
                if (!finished) {
                    Cacc = Lw;
                    Cmin = Mw;
                    base += CPG;
                }
            }
        }
        if (walked == before) {
            // Nothing new.  While the wait lasts, tell the readers if other streams have closed meanwhile, which
            // widens this one's window.
            if (++looks > kFoldPatience) {
                if (lane == 0) set_error(ws.header, PSA_DEVERR_STALLED);
                break;
            }
            if (closed_now != seen) { seen = closed_now; looks = 0; }
            if (closed_now != closed && walked > 0) {
                closed = closed_now;
                if (lane == 0) st_relaxed(&ctl->key_progress, progress_word(lim_now, granted(window, S, closed), walked));
            }
            __builtin_amdgcn_s_sleep(8);
            continue;
        }
        closed = closed_now;
        looks = 0;
        if (finished) break;
        // The frontier opens the window for waiting workgroups; the limit tells them how far the stream can still go.
        // The window: the launch's total of chunks in flight is shared by the streams still open, so the last,
        // deepest streams are read as wide as the whole batch was (a window sized for all streams leaves the
        // machine idle once most of them have closed).
        lim_now = min(nch, stop_bound<G>(Lw, Mw, stop_end, walked * KU, N, m, KU, odds));
        if (lane == 0) st_relaxed(&ctl->key_progress, progress_word(lim_now, granted(window, S, closed), walked));
    }
    // every head has stopped, or the blocks ran out: close the stream (limit = frontier).  A fixed budget is the one position
    // tested, so the stops are known here, and its chunks have nothing to settle.
    if (budget > 0 && lane < G && stop_end > 0) ctl->stop[lane] = stop_word(nlim, P_end);
    if (lane == 0) {
        st_relaxed(&ctl->key_progress, progress_word(walked, 0, walked));
        atomicAdd(&ws.header[kClosedStreams], 1);
    }
}

// Physical page and valid-token count of each ranked block of chunk c of stream s -> LDS.  Issued before
// the workgroup looks at the window, so that the loads overlap its wait.
template <int G, int MAXB>
__device__ __forceinline__ void stage_pages(SelectShared<G, MAXB> &sh, const KvView &kv, const DecodeWs &ws, int CB,
                                            int s, int c, int tid) {
    const int ctx = stream_ctx(kv, s);
    const int N = (ctx + kPage - 1) / kPage;
    const int nblk = min(CB, N - c * CB);
    const size_t row0 = (size_t)s * kv.max_blocks + c * CB;
    if (tid < nblk) {
        const int page = ws.ranked_page[row0 + tid];
        // (the ranking kernel wrote a page of the pool, or with a second tier possibly ~slot; anything else
        // is taken for page 0 rather than for an address)
        sh.page[tid] = (kv.slot_pool != nullptr && page < 0) ? page : clamp_page_quiet(page, kv.num_pages);
        sh.valid[tid] = min(kPage, ctx - ws.order[row0 + tid] * kPage);
    }
}

// B operand of the QK^T product of stream s -> LDS (every wave of the workgroup reads it from there): column
// n = lane%16 is query head n (zero beyond the group), k block kq = lane/16; for step kk the lane holds
// channels 8*(4*kk + kq) .. +7.  (The caller's next barrier makes it visible.)
template <int G, int MAXB>
__device__ __forceinline__ void load_queries(SelectShared<G, MAXB> &sh, const KvView &kv, const uint8_t *__restrict__ q,
                                             int s) {
    const int tid = threadIdx.x;
    if (tid < 256) {
        const int kk = tid >> 6, ln = tid & 63, n = ln & 15, kq = ln >> 4;
        const int r = s / kv.num_kv_heads, h = s % kv.num_kv_heads;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (n < G) v = ld16(q + ((size_t)(r * kv.num_q_heads + h * G + n) * kHeadDim + (4 * kk + kq) * 8) * 2);
        sh.qb[kk][ln] = v;
    }
}

// =================================================================================================
// Key work of one workgroup: chunk c of stream s.  Ends with the chunk published (wave 0 stores the chunk's
// words, which the stream's folding wave is looking at).
// =================================================================================================
// What a chunk publishes, per head, in every lane of wave 0 (head lane % G): (log-sum-exp, minimum) of its L_b, and the
// same up to its last tested position where that is not its end.
struct Published { float L, M, LT, MT; };

// kBatch: key slices a wave keeps in flight.
template <int DT, int G, int MAXB, int kBatch>
__device__ __forceinline__ Published process_chunk(SelectShared<G, MAXB> &sh, const KvView &kv, const DecodeWs &ws, int m, int CB,
                                                   int budget, int s, int c, int tid) {
    const int lane = tid & 63, wave = tid >> 6;
    const int h = s % kv.num_kv_heads;
    const int ctx = stream_ctx(kv, s);
    const int N = (ctx + kPage - 1) / kPage;
    const int start = c * CB;
    const int nblk = min(CB, N - start);
    // (the chunk's pages and valid-token counts are in LDS already: stage_pages)
    // B operand of the QK^T product (see load_queries): the same for every chunk of the stream
    const int n = lane & 15, kq = lane >> 4;
    uint4 qb[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qb[kk] = sh.qb[kk][lane];
    // ---- keys: wave w takes blocks w, w + 4, ..., each a 4 KiB slice read as four coalesced 1 KiB loads.  A operand
    //      of the product: row n = token n of the block, same channel assignment as the queries. ------------------
    auto issue = [&](int i, uint4 (&dst)[4]) {
        const uint8_t *kp = key_slice(kv, sh.page[i], h) + lane * 16;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) dst[kk] = ld16_stream(kp + kk * 1024);
    };
    auto consume = [&](int i, const uint4 (&k)[4]) {
        // (second tier with a staging buffer: a slice that came over the host link is kept for the update)
        if (kv.staging != nullptr) {
            const int entry = sh.page[i] >= 0 ? stage_key_slice(kv, sh.page[i], h, k, lane) : -1;
            if (lane == 0) sh.entry[i] = entry;
        }
        const f32x4_t sc = block_logits<DT>(k, qb, sh.stage[wave], lane, sh.valid[i]);
        if (n < G) *reinterpret_cast<f32x4_t *>(&sh.lg[i][n][4 * kq]) = sc;
    };
    constexpr int kWaves = kSelectThreads / 64;
    if (kBatch > 1 && nblk == 32) {
        // A whole chunk of 32 blocks, eight per wave: a rolling window.  kBatch slices are in flight; the oldest is
        // worked on and its registers go to the next load at once, so the wave never stands with nothing in
        // flight between rounds.
        uint4 ka[kBatch][4];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) issue(wave + kWaves * u, ka[u]);
#pragma unroll
        for (int k = 0; k < 32 / kWaves; ++k) {
            consume(wave + kWaves * k, ka[k % kBatch]);
            if (k + kBatch < 32 / kWaves) issue(wave + kWaves * (k + kBatch), ka[k % kBatch]);
        }
    } else {
        for (int i0 = wave; i0 < nblk; i0 += kWaves * kBatch) {
            uint4 ka[kBatch][4];
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (i0 + kWaves * u < nblk) issue(i0 + kWaves * u, ka[u]);
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (i0 + kWaves * u < nblk) consume(i0 + kWaves * u, ka[u]);
        }
    }
    lds_barrier();
    // ---- the blocks' log-sum-exp L_b per head, from the logits in LDS, all threads of the workgroup at once ----------
    rows_lse<G, kSelectThreads>(&sh.lg[0][0][0], &sh.Lb[0][0], nblk * G, tid);
    lds_barrier();
    if (wave != 0) return Published{};

    // ---- publish: the chunk's (log-sum-exp, minimum) of its blocks' L_b per head ------------------------------------
    Published own;
    chunk_aggregate<G>(&sh.Lb[0][0], nblk, lane, own.L, own.M);
    unsigned long long w = pack2(own.L, own.M);
    if (w == kAggSentinel) w = kAggSentinel - 1;     // a NaN pair that happens to look like "not published"
    own.LT = -INFINITY;
    own.MT = INFINITY;
    if (split_words(CB, m, budget)) {                // the same up to the chunk's last tested position, in memory before the word
        const int upto = last_test(start, min(start + nblk, blocks_that_count(N, budget)), m, N) - start;
        chunk_aggregate<G>(&sh.Lb[0][0], upto, lane, own.LT, own.MT);
        float2 *t = ws.agg_tested + ((size_t)s * ws.max_chunks + c) * G + lane;
        if (lane < G) { st_relaxed(&t->x, own.LT); st_relaxed(&t->y, own.MT); }
        stores_done();
    }
    // The G words need no order among themselves: a chunk counts as published when all of them are there.
    if (lane < G) st_relaxed(&ws.agg[((size_t)s * ws.max_chunks + c) * G + lane], w);
    return own;
}

// The first of chunks from .. to - 1 whose words (agg: the stream's) are not all there, -1 if they are.  One wave.
template <int G>
__device__ __forceinline__ int first_unpublished(const unsigned long long *agg, int from, int to, int lane) {
    for (int i0 = from * G; i0 < to * G; i0 += 64) {
        const unsigned long long w = i0 + lane < to * G ? ld_relaxed(&agg[i0 + lane]) : 0;
        const unsigned long long missing = __ballot(w == kAggSentinel);
        if (missing != 0ull) return (i0 + __ffsll((long long)missing) - 1) / G;
    }
    return -1;
}

// Looks (about a microsecond each) at a frontier that stands still before a workgroup reads what is missing: spin_limit, and no
// more than this many unless slices come over the host link, where a chunk can take milliseconds.  A launch that has the chip to
// itself reads nothing twice even with 64; launches beside others, of 2 to 4 streams, read no more than one after the
// other (8 requests of 32K tokens on each of 3 streams: 203 us a round, 264 in turn).
constexpr int kPatience = 1 << 10;

// (No fixed budget.)  How many of chunk c's blocks every head uses (sh.cnt), and the stops of the heads that stop in it:
// wave 0 waits for the words of the group's chunks before this one and for the group's carry, and finds what the fold finds;
// the group's last chunk leaves the next group's carry.  `own`: what the chunk published.  Nobody needs the workgroup's own
// chunk, `mine`, if every head stops before it, which the words or the closed stream say.
// sh.next: -1 once `mine` is settled, else the chunk this workgroup is to read next.  When the looks have brought nothing,
// the workgroup reads the chunks before its own whose words are missing, the first one first, settles each (c < mine until
// then), and comes back to its own.  Whatever a chunk leaves in memory is the same bits whoever works on it, so it does not
// matter that the chunk's own workgroup is under way, or comes later.
template <int G, int MAXB>
__device__ __forceinline__ void settle_chunk(SelectShared<G, MAXB> &sh, const KvView &kv, const DecodeWs &ws, const Published &own,
                                             float eps, int m, int CB, int spin_limit, int s, int c, int mine, int lane) {
    constexpr int CPG = 64 / G, kScan = (MAXB * G + 63) / 64;
    const int g = lane % G, jl = lane / G;
    const unsigned long long head_lanes = (~0ull / ((1ull << G) - 1ull)) << g;
    const int N = (stream_ctx(kv, s) + kPage - 1) / kPage;
    const int group = c / CPG, base = group * CPG, cj = c - base, start = c * CB, end = min(start + CB, N);
    const unsigned long long *words = ws.agg + (size_t)s * ws.max_chunks * G, *agg = words + base * G;
    const float2 *tested = ws.agg_tested + ((size_t)s * ws.max_chunks + base) * G;
    unsigned long long *carry = ws.carry + ((size_t)s * ws.max_groups + group) * G;
    const int patience = kv.slot_pool != nullptr ? spin_limit : min(spin_limit, kPatience);
    unsigned long long v = 0, cw = 0;
    bool close = group == 0;
    for (int looks = 0, seen = -1;;) {
        const unsigned long long kp = ld_relaxed(&ws.ctl[s].key_progress);
        if (jl < cj && close) v = ld_relaxed(&agg[lane]);
        if (group > 0 && close) cw = ld_relaxed(&carry[g]);
        if (close && __ballot(v == kAggSentinel || cw == kAggSentinel) == 0ull) break;
        const int fr = uniform(progress_frontier(kp)), lim = uniform(progress_limit(kp));
        if (mine >= lim) {
            if (lane < G) sh.cnt[lane] = -1;
            if (lane == 0) sh.next = -1;
            return;
        }
        if (fr != seen) { seen = fr; looks = 0; }
        const bool tired = looks > patience;
        if (tired) {
            const int missing = first_unpublished<G>(words, fr, c, lane);
            if (missing >= 0) {
                if (lane == 0) sh.next = missing;
                return;
            }
            looks = 0;
        }
        // Until the fold has come to the group, one word says so; then the words themselves.
        const bool was = close;
        close = fr >= base || tired;
        if (close && !was) continue;
        // a fifth of a microsecond, and the same again for every eight chunks the fold has to go: the pollers of one stream
        // share cache lines
        for (int i = c - fr; i >= 0; i -= 8) __builtin_amdgcn_s_sleep(8);
        looks += 1 + (max(0, c - fr) >> 3);
    }
    float L = jl == cj ? own.L : (jl < cj ? __uint_as_float((uint32_t)(v & 0xffffffffull)) : -INFINITY);
    float M = jl == cj ? own.M : (jl < cj ? __uint_as_float((uint32_t)(v >> 32)) : INFINITY);
    const bool split = split_words(CB, m, 0);
    float LT = own.LT, MT = own.MT;
    if (split && jl < cj) {
        LT = ld_relaxed(&tested[lane].x);
        MT = ld_relaxed(&tested[lane].y);
    }
    const float Cacc = group > 0 ? __uint_as_float((uint32_t)(cw & 0xffffffffull)) : -INFINITY;
    const float Cmin = group > 0 ? __uint_as_float((uint32_t)(cw >> 32)) : INFINITY;
    float E, F, P;
    group_states<G>(L, M, Cacc, Cmin, E, F, lane);
    const int b0 = (base + jl) * CB;
    const bool passes = jl <= cj && chunk_passes(L, M, E, F, split, LT, MT, b0, min(b0 + CB, N), N, m, eps, P);
    const unsigned long long hits = __ballot(passes) & head_lanes;
    const int first = hits != 0ull ? (__ffsll((long long)hits) - 1) / G : CPG;
    const bool gone = first < cj || (group > 0 && cw == kCarryStopped), here = !gone && first == cj;
    int cnt = gone ? 0 : end - start;
    if (__ballot(here) != 0ull) {
        const int src = cj * G + g;
        int n;
        float Ps;
        stop_in_chunk<G, kScan>(start, end, __shfl(E, src), __shfl(F, src), __shfl(P, src), N, m, eps,
                                [&](int i) { return (&sh.Lb[0][0])[i]; }, n, Ps, lane);
        if (here) {
            cnt = n - start;
            if (lane < G) ws.ctl[s].stop[lane] = stop_word(n, Ps);      // (for the final merge)
        }
    }
    if (cj == CPG - 1 && end < N && jl == cj) {                         // the lanes that hold the state after the group
        unsigned long long w = pack2(L, M);
        if (w >= kCarryStopped) w = kCarryStopped - 1;                  // (a NaN pair that looks like one of the two)
        st_relaxed(&carry[G + g], gone || here ? kCarryStopped : w);
    }
    if (lane < G) sh.cnt[lane] = cnt;
    const int missing = c < mine ? first_unpublished<G>(words, c + 1, mine, lane) : -1;
    if (lane == 0) sh.next = c == mine ? -1 : (missing >= 0 ? missing : mine);
}

// =================================================================================================
// The chunk's values (lines 10-12), by the workgroup that holds its logits: the heads that are still open use all of it, and
// those that stop in it their stop's share (sh.cnt).  The four waves stream independently: wave w takes blocks w, w+4, ...
// of the chunk, and nothing is shared until the sums at the end.
//   weights   p = exp(logit - L), L = per head the largest log-sum-exp of a block the head uses: a reference every wave
//             knows beforehand, so nothing is rescaled on the way and the four waves' sums simply add up.  (p <= 1, and
//             the largest weight is at least 1/16: the weights keep their precision as 16-bit halves.)
//   numerator D[head][channel] += P[head][token] V[token][channel]: eight 16x16x16 products per block, the weights
//             split into hi + lo 16-bit halves that sit in neighbouring rows (see add_weighted).  The k index of both
//             operands is the token: lane (rg, *) holds the value rows rg, 4+rg, 8+rg, 12+rg -- the rows its four loads
//             fetched -- and the key product left the logits so that the 16 bytes at [block][head][4 rg] are those
//             same four tokens: one read of LDS, no transposition.
// Output per chunk and head: (L, sum of p, numerator[128]) for the final merge.
// =================================================================================================
constexpr int kWholeChunk = 32;      // blocks of a chunk in the default plan: the size with a fixed schedule
template <int DT, int G, int MAXB>
__device__ __forceinline__ void attend_chunk(SelectShared<G, MAXB> &sh, const KvView &kv, const DecodeWs &ws, int s, int c,
                                             int tid) {
    const int lane = tid & 63, wave = uniform(tid >> 6), rg = lane >> 4, cl = lane & 15;
    const int h = s % kv.num_kv_heads;
    const int mycnt = sh.cnt[lane % G];                        // blocks of the chunk that head lane % G uses
    int maxcnt = mycnt;
#pragma unroll
    for (int d = 1; d < G; d <<= 1) maxcnt = max(maxcnt, __shfl_xor(maxcnt, d));
    maxcnt = uniform(maxcnt);
    if (maxcnt <= 0) return;
    const int jmax = (maxcnt - wave + 3) / 4;                  // blocks of this wave (may be <= 0)
    const int hd = cl >> 1;                                    // the head whose weights the lane supplies (see add_weighted)
    const int lg_lane = (hd < G ? hd : 0) * kPage + 4 * rg;
    const int hdcnt = __shfl(mycnt, hd);
    Slice v[kValueDepth];
    auto issue = [&](int j, auto slot) __attribute__((always_inline)) {
        constexpr int u = decltype(slot)::value;
        v[u] = load_slice(value_slice(kv, uniform(sh.page[wave + 4 * j]), h), lane);
    };
    f32x4_t acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    float l = 0.0f, Lc = -INFINITY;
    auto reference = [&]() __attribute__((always_inline)) {    // of head lane % G first: every wave computes the same bits
        for (int i = lane / G; i < mycnt; i += 64 / G) Lc = fmaxf(Lc, sh.Lb[i][lane % G]);
#pragma unroll
        for (int d = G; d < 64; d <<= 1) Lc = fmaxf(Lc, __shfl_xor(Lc, d));
        Lc = __shfl(Lc, hd);
    };
    auto consume = [&](int j, auto slot) __attribute__((always_inline)) {
        constexpr int u = decltype(slot)::value;
        const int blk = wave + 4 * j;
        if (kv.staging != nullptr) {                           // (second tier: see stage_value_slice)
            const int entry = uniform(sh.entry[blk]);
            if (entry >= 0) stage_value_slice(kv, entry, uniform(sh.page[blk]), h, v[u].r, lane);
        }
        const int valid = uniform(sh.valid[blk]);
        if (valid < kPage) zero_invalid_rows(v[u], rg, valid);
        // tokens beyond `valid` hold -inf logits; blocks beyond the head's stop, and heads beyond the group, weigh nothing
        const bool on = hd < G && blk < hdcnt;
        const f32x4_t x = *reinterpret_cast<const f32x4_t *>(&sh.lg[blk][0][0] + lg_lane);
        add_values<DT>(acc, l, v[u], x, on, Lc, cl & 1);
    };
    if (maxcnt == kWholeChunk) {                               // eight blocks for every wave: a rolling window, as for the keys
        static_for<kValueDepth>([&](auto u) { issue(u, u); });
        reference();
        static_for<kWholeChunk / 4>([&](auto j) {
            const std::integral_constant<int, j % kValueDepth> slot;
            consume(j, slot);
            if (j + kValueDepth < kWholeChunk / 4) issue(j + kValueDepth, slot);
            __builtin_amdgcn_sched_barrier(0);                 // (steps that are interleaved run out of registers)
        });
    } else {
        static_for<kValueDepth>([&](auto u) { if (u < jmax) issue(u, u); });
        reference();
        for (int j0 = 0; j0 < jmax; j0 += kValueDepth) {
            static_for<kValueDepth>([&](auto u) {
                if (j0 + u < jmax) {
                    consume(j0 + u, u);
                    if (j0 + kValueDepth + u < jmax) issue(j0 + kValueDepth + u, u);
                }
            });
        }
    }
    // the exp-sum over the four row groups, then the four waves through LDS (one reference: plain sums)
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    float (*st_acc)[G][kHeadDim] = reinterpret_cast<float (*)[G][kHeadDim]>(&sh.stage[0][0]);
    store_heads<G>(acc, st_acc[wave], rg, cl);
    if (rg == 0 && hd < G && !(cl & 1)) {
        sh.st_l[wave][hd] = l;
        if (wave == 0) sh.st_ref[hd] = Lc;
    }
    lds_barrier();
    float *dst = ws.partial + ((size_t)s * ws.max_chunks + c) * G * kPartialStride;
    for (int idx = tid; idx < G * kHeadDim; idx += 256) {
        const int g = idx / kHeadDim, ch = idx % kHeadDim;
        dst[g * kPartialStride + 4 + ch] =
            (st_acc[0][g][ch] + st_acc[1][g][ch]) + (st_acc[2][g][ch] + st_acc[3][g][ch]);
        if (ch == 0) {
            dst[g * kPartialStride] = sh.st_ref[g];
            dst[g * kPartialStride + 1] = (sh.st_l[0][g] + sh.st_l[1][g]) + (sh.st_l[2][g] + sh.st_l[3][g]);
        }
    }
}

struct SelectArgs {
    KvView kv;
    const uint8_t *q;
    DecodeWs ws;
    float eps;
    int m, CB, budget, window, spin_limit;
    const int32_t *depth_hint;
};

// The kernel's arguments, anew from where they were passed.
__device__ __forceinline__ SelectArgs args_anew() {
    typedef const __attribute__((address_space(4))) uint32_t *Words;
    Words from = (Words)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(from));
    uint32_t copy[sizeof(SelectArgs) / 4];
#pragma unroll
    for (unsigned i = 0; i < sizeof(SelectArgs) / 4; ++i) copy[i] = from[i];
    SelectArgs a;
    __builtin_memcpy(&a, copy, sizeof(a));
    return a;
}

// The workgroup's chunk, c, is not settled (see settle_chunk): reads the chunks that are asked for until it is.  Hardly ever
// needed, so nothing of it may cost the way that all others take: it has the kernel's arguments anew, for every step, and the
// thread's index, or their values and what derives from them would be kept in registers, which are short.
template <int DT, int G, int MAXB>
__device__ __forceinline__ void catch_up(SelectShared<G, MAXB> &sh, int s, int c) {
    for (int at = uniform(sh.next); at >= 0; at = uniform(sh.next)) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        lds_barrier();                          // (everyone has read sh.next, and is done with the chunk before)
        Published own;
        {
            const SelectArgs a = args_anew();
            const int N = (stream_ctx(a.kv, s) + kPage - 1) / kPage;
            stage_pages<G, MAXB>(sh, a.kv, a.ws, a.CB, s, at, tid);
            if (tid == 0) atomicAdd(&a.ws.ctl[s].k_blocks, min(a.CB, N - at * a.CB));
            lds_barrier();
            own = process_chunk<DT, G, MAXB, 1>(sh, a.kv, a.ws, a.m, a.CB, a.budget, s, at, tid);
        }
        {
            const SelectArgs a = args_anew();
            if (tid < 64) settle_chunk<G, MAXB>(sh, a.kv, a.ws, own, a.eps, a.m, a.CB, a.spin_limit, s, at, c, tid);
        }
        lds_barrier();
    }
}

// =================================================================================================
// grid = folders + S * max_chunks workgroups of 256 threads.  The first `folders` = min(ceil(S / 4), kMaxFoldGroups)
// workgroups are the folds, one wave per stream (they start first and stay until their streams close); then one
// workgroup per (chunk, stream), streams fastest -- with more streams than folding waves, the streams of one turn of
// those waves after the other.
// =================================================================================================
template <int DT, int G, int MAXB>
__global__ __launch_bounds__(kSelectThreads, G * MAXB > 256 ? 2 : 4) void select_kernel(SelectArgs args) {
    const KvView &kv = args.kv;
    const DecodeWs &ws = args.ws;
    const uint8_t *__restrict__ q = args.q;
    const int32_t *depth_hint = args.depth_hint;
    const float eps = args.eps;
    const int m = args.m, CB = args.CB, budget = args.budget, window = args.window, spin_limit = args.spin_limit;
    __shared__ SelectShared<G, MAXB> sh;
    const int S = kv.batch * kv.num_kv_heads;
    const int folders = min((S + 3) / 4, kMaxFoldGroups);
    if ((int)blockIdx.x < folders) {
        for (int fs = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6); fs < S; fs += 4 * folders)
            fold_stream<G>(kv, ws, fs, eps, m, CB, budget, window > 0 ? window : 1);
        return;
    }
    // Workgroups go to the chip's eight partitions by index, round robin.  With the streams in the same order in
    // every batch of S workgroups, and S a multiple of eight, all chunks of a stream would land on one partition:
    // the last, deepest streams would then be read by an eighth of the machine.  So the streams' order rotates by
    // one from chunk to chunk (when S is even; an odd S rotates by itself).
    int b = (int)blockIdx.x - folders, s0 = 0, ns = S;                 // streams s0 .. s0 + ns - 1 are this turn's
    if (S > 4 * folders) {
        const int turn = b / (4 * folders * ws.max_chunks);
        b -= turn * (4 * folders * ws.max_chunks);
        s0 = turn * 4 * folders;
        ns = min(4 * folders, S - s0);
    }
    const int c = b / ns;
    const int s = s0 + (b % ns + ((ns & 1) ? 0 : c)) % ns;
    // One round trip for everything a workgroup needs to know first: the stream's progress word (asked for before
    // anything else), its length, its queries, its chunk's pages.  Most workgroups of a launch belong to chunks
    // beyond their stream's stop and leave right here; the faster they do, the sooner the slots they hold go to
    // chunks that matter.
    unsigned long long kp_first = 0;
    if (threadIdx.x == 0) kp_first = ld_relaxed(&ws.ctl[s].key_progress);
    const int N = (stream_ctx(kv, s) + kPage - 1) / kPage;
    if (c * CB >= N) return;
    load_queries<G, MAXB>(sh, kv, q, s);
    stage_pages<G, MAXB>(sh, kv, ws, CB, s, c, threadIdx.x);
    if (threadIdx.x == 0) sh.kp0 = kp_first;
    lds_barrier();
    if (c >= progress_limit(sh.kp0)) return;          // closed, out of reach, or beyond a block budget
    // Second tier: a chunk with slices that are not cached is read over the host link, where reading ahead
    // of the stop costs far more than waiting does: such a chunk is read when it is expected to be needed
    // (inside the hint) or when the fold is about to reach it.
    const bool tiered = kv.slot_pool != nullptr;
    if (threadIdx.x == 0) {
        bool from_host = false;
        if (tiered)
            for (int i = 0; i < min(CB, N - c * CB); ++i) from_host |= sh.page[i] >= 0;
        // chunks read beyond the fold's frontier are at most the window: wait until this one is inside
        // it, or the stream closes before it
        const int hinted = hinted_chunks(depth_hint, s, N, CB);
        int go = 1;
        for (int tries = 0;; ++tries) {
            const unsigned long long kp = tries == 0 ? sh.kp0 : ld_relaxed(&ws.ctl[s].key_progress);
            const int fr = progress_frontier(kp), grant = progress_grant(kp), lim = progress_limit(kp);
            const int win = max(window_of(window, fr), grant);      // (the fold grants more once streams have closed)
            if (c >= lim) { go = 0; break; }       // closed, or a block budget ends before this chunk
            // with a hint: everything up to it plus a margin (a sixteenth and two chunks: the depth of a
            // decode step differs a little from the previous step's) at once; past that, a window that
            // starts at 8 chunks and doubles with the distance the hint fell short by
            const int padded = hinted + (hinted >> 4) + 2;
            int reach = hinted > 0 ? max(padded, fr + min(max(8, 2 * (fr - hinted)), win)) : fr + win;
            if (from_host) reach = min(reach, max(hinted, fr + 2));
            if (c < reach || tries >= spin_limit) break;
            nap(tries);
        }
        sh.go = go;
    }
    lds_barrier();
    if (!sh.go) return;
    if (threadIdx.x == 0) atomicAdd(&ws.ctl[s].k_blocks, min(CB, N - c * CB));     // traffic accounting
    const Published own = process_chunk<DT, G, MAXB, kKeyDepth>(sh, kv, ws, m, CB, budget, s, c, threadIdx.x);
    if (budget > 0) {                          // used by every head: the values wait for nothing
        if (threadIdx.x < G) sh.cnt[threadIdx.x] = min(CB, min(N, budget) - c * CB);
        if (threadIdx.x == 0) sh.next = -1;
    } else if (threadIdx.x < 64) {
        settle_chunk<G, MAXB>(sh, kv, ws, own, eps, m, CB, spin_limit, s, c, c, threadIdx.x);
    }
    lds_barrier();
    if (__builtin_expect(sh.next >= 0, 0)) catch_up<DT, G, MAXB>(sh, s, c);
    attend_chunk<DT, G, MAXB>(sh, kv, ws, s, c, threadIdx.x);
}

template <int DT, int G>
static hipError_t launch_select_t(const KvView &kv, const void *q, const DecodeWs &ws, float eps, int m,
                                  int budget, const DecodePlan &plan, hipStream_t st) {
    const unsigned S = (unsigned)(kv.batch * kv.num_kv_heads);
    const unsigned folders = (S + 3) / 4 < (unsigned)kMaxFoldGroups ? (S + 3) / 4 : (unsigned)kMaxFoldGroups;
    const unsigned grid = folders + S * (unsigned)plan.max_chunks;
    const SelectArgs args = {kv, (const uint8_t *)q, ws, eps, m, plan.chunk_blocks, budget, plan.window_chunks, plan.spin_limit,
                             plan.depth_hint};
    if (plan.chunk_blocks <= 32)
        select_kernel<DT, G, 32><<<grid, kSelectThreads, 0, st>>>(args);
    else
        select_kernel<DT, G, kMaxChunkBlocks><<<grid, kSelectThreads, 0, st>>>(args);
    return hipGetLastError();
}

hipError_t launch_select(const KvView &kv, int dtype, int G, const void *q, const DecodeWs &ws, float eps,
                         int m, int budget, const DecodePlan &plan, hipStream_t st) {
#define PSA_CASE(DT, GG) \
    if (dtype == DT && G == GG) return launch_select_t<DT, GG>(kv, q, ws, eps, m, budget, plan, st);
    PSA_CASE(0, 1) PSA_CASE(0, 2) PSA_CASE(0, 4) PSA_CASE(0, 8)
    PSA_CASE(1, 1) PSA_CASE(1, 2) PSA_CASE(1, 4) PSA_CASE(1, 8)
#undef PSA_CASE
    return hipErrorInvalidValue;
}

}  // namespace psa
