// Host side of psa_decode_attention: workspace layout, launch plan and the kernel sequence
//   score (Algorithm 1 line 5) -> order (line 6) -> select (lines 7-18) -> finalize (line 19),
// all enqueued on one stream with no host involvement in between -- or, for short contexts, one kernel that does it all.
#include "psa_host.h"

namespace psa {

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Compute units of the current device (256 on MI355X); read once.
int compute_units() {
    static int cached = 0;
    if (cached == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cached = n;
    }
    return cached;
}

DecodePlan make_plan(const psa_kv_desc *d, const psa_tuning *t) {
    DecodePlan p;
    const int S = d->batch * d->num_kv_heads;
    p.chunk_blocks = (t && t->chunk_blocks) ? t->chunk_blocks : 32;
    if (t && t->window_chunks > 0) {
        p.window_chunks = t->window_chunks;
    } else {
        // about 96 MiB of key slices inside the streams' windows together (the chip holds 1024 workgroups of this
        // kernel, one 128 KiB chunk each; three quarters of that measured best: the fold widens the windows of the
        // streams that stay open longest), 2 to 24 chunks per stream
        const long long per_stream = (96ll << 20) / ((long long)(S > 0 ? S : 1) * p.chunk_blocks * kSliceBytes);
        p.window_chunks = per_stream < 2 ? 2 : (per_stream > 24 ? 24 : (int)per_stream);
    }
    p.spin_limit = (t && t->spin_limit > 0) ? t->spin_limit : (1 << 14);
    p.max_chunks = (d->max_blocks_per_seq + p.chunk_blocks - 1) / p.chunk_blocks;
    if (p.max_chunks < 1) p.max_chunks = 1;
    p.force_bitonic = t ? t->force_bitonic : 0;
    p.depth_hint = t ? t->depth_hint : nullptr;
    p.events = t ? static_cast<hipEvent_t *>(t->phase_events) : nullptr;
    // One launch for short contexts, where the chain of launches is what a call costs (psa_solo.hip).  One compute unit does
    // a stream's work there.  Up to 128 blocks that is the better bargain with any number of streams (one launch against the
    // chain, 2048 tokens, G = 4): where the rule selects little, 17 us against 26 to 30 with 1 to 8 streams, 31 against 52
    // with 256; where nearly everything is selected, 61 against 77 with 256 streams, but 32 against 26 with one, 30 against
    // 28 with 8, 35 against 31 with 32 (at 1536 tokens the two are even there).  Above 128 blocks a stream that selects
    // nearly all its blocks wants more than one unit, unless there are streams for most of the chip: at 256 blocks 63 us
    // against 32 with 8 streams, 99 against 103 with 192; at 192 blocks 53 against 53 with 128.  Hence three streams for
    // four blocks.
    // (The chain was five kernels then.  With four, G = 4, 2048 tokens: little selected 16 us against 24 with 8 streams, 22
    // against 27 with 32, 24 against 33 with 128; all selected 25 against 24, 35 against 26, 39 against 39; 256 blocks, 192
    // streams 56 against 55 and 97 against 93.  A stream's share is not known beforehand, so the line stays.)
    // Whoever tunes the general path, times its phases or brings a second tier gets the general path.  So does a call of more
    // streams than one grid of workgroups of 1024 threads can have (fewer than 2^32 threads).
    const bool tuned = t && (t->window_chunks > 0 || t->spin_limit > 0 || t->force_bitonic || t->phase_events ||
                             (t->chunk_blocks && t->chunk_blocks != 32));
    const int mb = d->max_blocks_per_seq;
    p.solo = !d->tier && !tuned && mb <= kSoloBlocks && (mb <= 128 || 4 * S >= 3 * mb) && (S + 1ll) * kSoloThreads < (1ll << 32);
    return p;
}

struct WsLayout {
    size_t header, ctl, scores, order, ranked_page, agg, logits, agg_tested, carry, partial, total;
};

static WsLayout layout(const psa_kv_desc *d, const DecodePlan &p) {
    const size_t S = (size_t)d->batch * d->num_kv_heads;
    const size_t G = (size_t)(d->num_q_heads / d->num_kv_heads);
    const size_t MB = (size_t)d->max_blocks_per_seq;
    WsLayout L;
    size_t at = 0;
    L.header = at;      at = align_up(at + 512, 256);
    L.ctl = at;         at = align_up(at + S * sizeof(StreamCtl), 256);
    L.scores = at;      at = align_up(at + S * MB * 4, 256);
    L.order = at;       at = align_up(at + S * MB * 4, 256);
    L.ranked_page = at; at = align_up(at + S * MB * 4, 256);
    L.agg = at;         at = align_up(at + S * p.max_chunks * G * 8, 256);
    L.partial = at;     at = align_up(at + S * p.max_chunks * G * kPartialStride * 4, 256);
    // one launch: the logits; the general path: two small tables
    L.logits = at;
    L.agg_tested = at;
    L.carry = align_up(at + S * p.max_chunks * G * 8, 256);
    // The size is what it was when every path kept its logits here, block by block sums beside them, and had a work list: what
    // fits the static array is drawn in it, and calls that were refused there for their size stay refused.
    at = align_up(at + S * MB * kPage * G * 4, 256);
    at = align_up(at + S * MB * G * 4, 256);
    L.total = align_up(at + S * p.max_chunks * 4, 256);
    return L;
}

size_t decode_workspace_bytes_plan(const psa_kv_desc *d, const DecodePlan &p) { return layout(d, p).total; }

// num_pages == 0: the kernels read a bad table entry as page 0, which does not exist then (the pools may be NULL), so no
// kernel that reads slices is launched.  Every request comes out empty; those with tokens have table entries outside the
// pool, which the error word says.  Workgroup 0 finds the word, the others write the outputs (each may be NULL but `out`).
__global__ __launch_bounds__(256) void no_pages_kernel(KvView kv, int32_t *header, float *out, int32_t *n_selected, float *mass_est,
                                                       int32_t *blocks_read, float *lse, int32_t *order, int32_t *traffic) {
    if (blockIdx.x == 0) {
        int page_bad = 0, ctx_bad = 0;
        for (int r = threadIdx.x; r < kv.batch; r += 256) {
            const int ctx = ctx_clamped_quiet(kv, r);
            page_bad |= ctx > 0;
            ctx_bad |= ctx != kv.ctx_lens[r];
        }
        page_bad = __syncthreads_or(page_bad);
        ctx_bad = __syncthreads_or(ctx_bad);
        if (threadIdx.x == 0) {
            header[0] = 0;
            header[1] = (page_bad ? PSA_DEVERR_PAGE_RANGE : 0) | (ctx_bad ? PSA_DEVERR_CTX_RANGE : 0);
        }
        return;
    }
    const long long heads = (long long)kv.batch * kv.num_q_heads, S = (long long)kv.batch * kv.num_kv_heads;
    const long long first = (long long)(blockIdx.x - 1) * 256 + threadIdx.x, step = (long long)(gridDim.x - 1) * 256;
    for (long long i = first; i < heads * kHeadDim; i += step) out[i] = 0.0f;
    for (long long i = first; i < heads; i += step) {
        if (n_selected) n_selected[i] = 0;
        if (mass_est) mass_est[i] = 0.0f;
        if (lse) lse[i] = -INFINITY;
    }
    for (long long i = first; i < S; i += step) {
        if (blocks_read) blocks_read[i] = 0;
        if (traffic) traffic[2 * i] = traffic[2 * i + 1] = 0;
    }
    if (order)
        for (long long i = first; i < S * kv.max_blocks; i += step) order[i] = -1;
}

hipError_t launch_no_pages(const KvView &kv, const DecodeArgs &a, int32_t *header, hipStream_t st) {
    no_pages_kernel<<<1 + 1024, 256, 0, st>>>(kv, header, a.out, a.n_selected, a.mass_est, a.blocks_read, a.lse_out, a.order_out,
                                              a.traffic_out);
    return hipGetLastError();
}

hipError_t launch_decode(const psa_kv_desc *d, const DecodeArgs &a, const DecodePlan &plan, void *wsp,
                         hipStream_t st) {
    const KvView kv = make_view(d);
    const WsLayout L = layout(d, plan);
    uint8_t *base = static_cast<uint8_t *>(wsp);
    DecodeWs ws;
    ws.header = reinterpret_cast<int32_t *>(base + L.header);
    ws.ctl = reinterpret_cast<StreamCtl *>(base + L.ctl);
    ws.scores = reinterpret_cast<float *>(base + L.scores);
    ws.order = reinterpret_cast<int32_t *>(base + L.order);
    ws.ranked_page = reinterpret_cast<int32_t *>(base + L.ranked_page);
    ws.agg = reinterpret_cast<unsigned long long *>(base + L.agg);
    ws.logits = reinterpret_cast<float *>(base + L.logits);
    ws.agg_tested = reinterpret_cast<float2 *>(base + L.agg_tested);
    ws.carry = reinterpret_cast<unsigned long long *>(base + L.carry);
    ws.partial = reinterpret_cast<float *>(base + L.partial);
    ws.max_chunks = plan.max_chunks;
    const int G = d->num_q_heads / d->num_kv_heads;
    ws.max_groups = (plan.max_chunks * G + 63) / 64;
    if (kv.batch == 0) return hipSuccess;
    hipEvent_t *ev = plan.events;
    hipError_t e;
    if (kv.num_pages == 0) {
        if (ev) (void)hipEventRecord(ev[0], st);
        e = launch_no_pages(kv, a, ws.header, st);
        for (int i = 1; ev && i < 6; ++i) (void)hipEventRecord(ev[i], st);
        return e;
    }
    if (plan.solo) return launch_solo(kv, d->dtype, G, a, ws, st);
    if (ev) (void)hipEventRecord(ev[0], st);
    if ((e = launch_score(kv, d->dtype, G, a.scorer, a.q, a.meta, ws, a.scores_out, st)) != hipSuccess) return e;
    if (ev) (void)hipEventRecord(ev[1], st);
    const int32_t *slot_of = d->tier ? make_tier_view(d->tier).slot_of : nullptr;
    if ((e = launch_order(kv, ws, G, plan, a.budget_blocks, slot_of, a.order_out, st)) != hipSuccess) return e;
    if (ev) (void)hipEventRecord(ev[2], st);
    if ((e = launch_select(kv, d->dtype, G, a.q, ws, a.threshold, a.check_granularity, a.budget_blocks, plan, st)) != hipSuccess)
        return e;
    if (ev) (void)hipEventRecord(ev[3], st);
    if (ev) (void)hipEventRecord(ev[4], st);      // (no kernel in between: the selection reads the values as well)
    e = launch_finalize(kv, ws, G, plan.chunk_blocks, a.out, a.n_selected, a.mass_est, a.blocks_read, a.lse_out,
                        a.traffic_out, st);
    if (ev) (void)hipEventRecord(ev[5], st);
    return e;
}

}  // namespace psa
