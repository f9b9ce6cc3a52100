// Value pass and final merge of one PSA decode step (Algorithm 1, lines 10-12 and 19).
//
// By the time these kernels run, the selection kernel has fixed every query head's stop n_g and
// left the exact scaled logits of the ranked blocks in the workspace.  What remains is plain
// attention over each head's own prefix: softmax numerators from the stored logits, times the value
// slices of the selected blocks -- every workgroup independent, no waiting, and only blocks
// actually selected are read.
//   attend_kernel    per value unit (chunk, stream) on the work list the selection kernel wrote:
//                    p = exp(logit - reference), partial numerator sum_t p_t v_t per head (on the
//                    matrix cores, the weights as a sum of two 16-bit halves) and exp-sum
//   finalize_kernel  merges a head's chunks (the online-softmax merge of line 11, all at once):
//                    out_g = sum over the chunks of the head's own prefix of the partial numerators,
//                    over the sum of the partial exp-sums, both rescaled to one reference maximum
#include "psa_attend.h"
#include "psa_host.h"

namespace psa {

// Blocks a head uses, from its stop (n, P_acc) as the selection kernel left it: n, or N when it never stopped.
__device__ __forceinline__ int stop_blocks(unsigned long long st, int N) {
    return (st != ~0ull && (int)(st >> 32) <= N) ? (int)(st >> 32) : N;
}

// =================================================================================================
// One workgroup per entry of the work list the selection kernel left (value unit = chunk c of stream s);
// the grid is sized for the most there can be, and a workgroup beyond the list's end returns after one
// round trip.  256 threads.  The four waves stream independently: wave w takes blocks w, w+4, ... of the unit,
// four value slices (16 KiB) in flight at a time, and nothing is shared until the final merge.
// What bounds it: with many units the memory (5.8 TB/s, logits included, on 16 requests of 64K tokens whose blocks are
// nearly all selected, 374 us before and after), with few the chain of loads before the first slice: entry, then
// everything about the unit at once, then slices.  (With the stops, the block values and the slices asked for one
// after the other, two slices in flight, 12 requests of up to 24K tokens took 12.1 us; 9.2 now.)  Four slices need 152
// registers, hence three workgroups per CU; three slices at four workgroups spilled and were slower throughout, as was
// a grid of resident workgroups that walks the list (31.4 us against 26.4 at 32K tokens, batch 8).
//   weights   p = exp(logit - L), L = per head the largest log-sum-exp of a block the head uses (the selection
//             kernel left one per block): a reference every wave knows beforehand, so nothing is rescaled
//             on the way and the four waves' sums simply add up.  (p <= 1, and the largest weight is at least
//             1/16: the weights keep their precision as 16-bit halves.)
//   numerator D[head][channel] += P[head][token] V[token][channel]: eight 16x16x16 products per block, the weights
//             split into hi + lo 16-bit halves that sit in neighbouring rows (see add_weighted; in products of their
//             own the two halves took sixteen).  The k
//             index of both operands is the token: lane (rg, *) holds the value rows rg, 4+rg, 8+rg, 12+rg
//             -- the rows its four loads fetched -- and the selection kernel stored the logits so that the
//             16 bytes at [block][head][4 rg] are those same four tokens: one load, no transposition.
// Output per unit and head: (L, sum of p, numerator[128]) for the final merge.
// =================================================================================================
constexpr int kValueDepth = 4;      // value slices a wave keeps in flight
constexpr int kUnitBlocks = 32;     // blocks of a unit in the default plan: the size with a fixed schedule

template <int DT, int G>
__global__ __launch_bounds__(256, 3) void attend_kernel(KvView kv, DecodeWs ws, int CB) {
    __shared__ __attribute__((aligned(16))) float st_acc[4][G][kHeadDim];
    __shared__ float st_l[4][G];
    __shared__ float st_ref[G];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), rg = lane >> 4, cl = lane & 15;
    // (the list's length and the entry are asked for together; an entry beyond the length is not used)
    const int item = ws.value_items[blockIdx.x];
    const int count = ws.header[kValueCount];
    if ((int)blockIdx.x >= count) return;
    const int s = __builtin_amdgcn_readfirstlane(item / ws.max_chunks), c = __builtin_amdgcn_readfirstlane(item % ws.max_chunks);
    const int h = s % kv.num_kv_heads, start = c * CB;
    const size_t row0 = (size_t)s * kv.max_blocks + start;
    const int room = min(CB, kv.max_blocks - start);          // rows of the tables that belong to the unit
    // Everything about the unit is asked for at once: the heads' stops, the length, the wave's blocks (wave, wave + 4,
    // ...: lane j has the page and the logical index of the j-th), the blocks' log-sum-exps.
    const unsigned long long stop = ws.ctl[s].stop[lane % G];
    const int mine = min(wave + 4 * (lane & 15), room - 1);
    int pg = ws.ranked_page[row0 + mine];
    const int od = ws.order[row0 + mine];
    constexpr int kRef = G * kUnitBlocks / 64 > 0 ? G * kUnitBlocks / 64 : 1;     // loads for the values of 32 blocks
    const float *bl = ws.block_lse + row0 * G;
    float lse[kRef];
#pragma unroll
    for (int k = 0; k < kRef; ++k) lse[k] = bl[min(64 * k + lane, room * G - 1)];
    const int ctx = ctx_clamped_quiet(kv, s / kv.num_kv_heads);
    const int N = (ctx + kPage - 1) / kPage;
    const int nblk = min(CB, N - start);
    // blocks of this chunk that head lane % G uses: those before its stop; and the most any head of the group uses
    const int mycnt = min(nblk, max(0, stop_blocks(stop, N) - start));
    int maxcnt = mycnt;
#pragma unroll
    for (int d = 1; d < G; d <<= 1) maxcnt = max(maxcnt, __shfl_xor(maxcnt, d));
    maxcnt = __builtin_amdgcn_readfirstlane(maxcnt);
    if (maxcnt <= 0) return;    // no head of the group reaches this chunk
    const int jmax = (maxcnt - wave + 3) / 4;           // blocks of this wave (may be <= 0)
    if (!(kv.slot_pool != nullptr && pg < 0)) pg = clamp_page_quiet(pg, kv.num_pages);   // (a page of the pool, or ~slot)
    const float *lg = ws.logits + row0 * (kPage * G);
    const int hd = cl >> 1;                             // the head whose weights the lane supplies (see add_weighted)
    const int lg_lane = (hd < G ? hd : 0) * kPage + 4 * rg;
    const int hdcnt = __shfl(mycnt, hd);

    Slice v[kValueDepth];
    f32x4_t x[kValueDepth];
    auto issue = [&](int j, auto slot) __attribute__((always_inline)) {
        constexpr int u = decltype(slot)::value;
        v[u] = load_slice(value_slice(kv, __builtin_amdgcn_readlane(pg, j), h), lane);
        x[u] = load_stream(lg + (wave + 4 * j) * (kPage * G) + lg_lane);
    };
    f32x4_t acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    float l = 0.0f, Lc = -INFINITY;
    // Reference exponent per head: the largest block log-sum-exp among the blocks the head uses (log2 units).  Lane =
    // (block, head) pairs, 64 / G blocks per load, then a butterfly over the lanes of a head: every lane l ends with
    // the reference of head l % G, and takes its own head's from there.  Every wave computes the same bits.
    auto reference = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kRef; ++k)
            if ((64 * k + lane) / G < mycnt && 64 * k + lane < kUnitBlocks * G) Lc = fmaxf(Lc, lse[k]);
        for (int i = kUnitBlocks + lane / G; i < mycnt; i += 64 / G) Lc = fmaxf(Lc, bl[(size_t)i * G + lane % G]);
#pragma unroll
        for (int d = G; d < 64; d <<= 1) Lc = fmaxf(Lc, __shfl_xor(Lc, d));
        Lc = __shfl(Lc, hd);
    };
    auto consume = [&](int j, auto slot) __attribute__((always_inline)) {
        constexpr int u = decltype(slot)::value;
        const int blk = wave + 4 * j;
        if (kv.staging != nullptr) {               // (second tier: see stage_key_slice)
            const int loc = __builtin_amdgcn_readlane(pg, j);
            if (loc >= 0) stage_value_slice(kv, loc, h, v[u].r, lane);
        }
        const int valid = ctx - __builtin_amdgcn_readlane(od, j) * kPage;
        if (valid < kPage) zero_invalid_rows(v[u], rg, valid);
        // tokens beyond `valid` hold -inf logits; blocks beyond the head's stop, and heads beyond the
        // group, weigh nothing
        const bool on = hd < G && blk < hdcnt;
        add_values<DT>(acc, l, v[u], x[u], on, Lc, cl & 1);      // (a head that uses no block of the unit is never `on`)
    };
    if (maxcnt == kUnitBlocks) {
        // Eight blocks for every wave: a rolling window, the oldest slice is worked on and its registers go to the next
        // load at once.
        static_for<kValueDepth>([&](auto u) { issue(u, u); });
        reference();
        static_for<kUnitBlocks / 4>([&](auto j) {
            const std::integral_constant<int, j % kValueDepth> slot;
            consume(j, slot);
            if (j + kValueDepth < kUnitBlocks / 4) issue(j + kValueDepth, slot);
            __builtin_amdgcn_sched_barrier(0);           // (steps that are interleaved run out of registers)
        });
    } else {
        static_for<kValueDepth>([&](auto u) { if (u < jmax) issue(u, u); });      // (rows beyond jmax may hold anything)
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
    store_heads<G>(acc, st_acc[wave], rg, cl);
    if (rg == 0 && hd < G && !(cl & 1)) {
        st_l[wave][hd] = l;
        if (wave == 0) st_ref[hd] = Lc;
    }
    lds_barrier();
    float *dst = ws.partial + ((size_t)s * ws.max_units + c) * G * kPartialStride;
    for (int idx = tid; idx < G * kHeadDim; idx += 256) {
        const int g = idx / kHeadDim, ch = idx % kHeadDim;
        dst[g * kPartialStride + 4 + ch] =
            (st_acc[0][g][ch] + st_acc[1][g][ch]) + (st_acc[2][g][ch] + st_acc[3][g][ch]);
        if (ch == 0) {
            dst[g * kPartialStride] = st_ref[g];
            dst[g * kPartialStride + 1] = (st_l[0][g] + st_l[1][g]) + (st_l[2][g] + st_l[3][g]);
        }
    }
}

constexpr int kUnitLanes = 16;   // value units merged side by side by one workgroup

// =================================================================================================
// grid (S*G), 512 threads = 16 unit lanes x 32 channel quads; unit lane j takes units j, j+16, ...
// in ascending order, and the 16 lanes are then added in a fixed order.
__global__ __launch_bounds__(512) void finalize_kernel(KvView kv, DecodeWs ws, int G, int VU,
                                                       float *__restrict__ out,
                                                       int32_t *__restrict__ n_selected,
                                                       float *__restrict__ mass_est,
                                                       int32_t *__restrict__ blocks_read,
                                                       float *__restrict__ lse_out,
                                                       int32_t *__restrict__ traffic_out) {
    __shared__ float red[8];
    __shared__ float wgt[kMaxBlocks / 4];        // per-unit rescale factor (value units are >= 4 blocks)
    __shared__ __attribute__((aligned(16))) float num_part[kUnitLanes][kHeadDim];
    const int s = blockIdx.x / G, g = blockIdx.x % G, tid = threadIdx.x;
    const int cq = tid & 31, uj = tid >> 5;
    const int r = s / kv.num_kv_heads, h = s % kv.num_kv_heads;
    int ctx = kv.ctx_lens[r];
    ctx = ctx < 0 ? 0 : (ctx > kv.max_blocks * kPage ? kv.max_blocks * kPage : ctx);
    const int N = (ctx + kPage - 1) / kPage;
    const StreamCtl *ctl = &ws.ctl[s];
    const unsigned long long st = ctl->stop[g];
    int n = N;
    float P = N > 0 ? 1.0f : 0.0f;
    if (st != ~0ull && (int)(st >> 32) <= N) { n = (int)(st >> 32); P = __uint_as_float((uint32_t)st); }
    const int nun = (n + VU - 1) / VU;
    const float *src = ws.partial + ((size_t)s * ws.max_units * G + g) * kPartialStride;
    const size_t stride = (size_t)G * kPartialStride;

    // reference maximum over the units
    float M = -INFINITY;
    for (int i = tid; i < nun; i += 512) { const float mi = src[i * stride]; wgt[i] = mi; M = fmaxf(M, mi); }
    // (over the wave with lane exchanges, over the eight waves through LDS: two barriers instead of ten)
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) M = fmaxf(M, __shfl_xor(M, d));
    if ((tid & 63) == 0) red[tid >> 6] = M;
    __syncthreads();
    M = fmaxf(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])), fmaxf(fmaxf(red[4], red[5]), fmaxf(red[6], red[7])));
    __syncthreads();
    // per-unit weights and the denominator
    float den = 0.0f;
    for (int i = tid; i < nun; i += 512) {
        const float mi = wgt[i];
        const float w = (mi == -INFINITY || M == -INFINITY) ? 0.0f : exp2_fast(mi - M);
        wgt[i] = w;
        den += src[i * stride + 1] * w;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) den += __shfl_xor(den, d);          // (a fixed tree: reproducible)
    if ((tid & 63) == 0) red[tid >> 6] = den;
    __syncthreads();
    den = ((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7]));
    // numerator: channels 4*cq .. 4*cq+3, units uj, uj+16, ...; four loads in flight per thread
    float4 num = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int i0 = uj; i0 < nun; i0 += 4 * kUnitLanes) {
        float4 a[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = i0 + k * kUnitLanes;
            a[k] = (i < nun) ? *reinterpret_cast<const float4 *>(src + i * stride + 4 + 4 * cq)
                             : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = i0 + k * kUnitLanes;
            const float w = (i < nun) ? wgt[i] : 0.0f;
            num.x = fmaf(a[k].x, w, num.x); num.y = fmaf(a[k].y, w, num.y);
            num.z = fmaf(a[k].z, w, num.z); num.w = fmaf(a[k].w, w, num.w);
        }
    }
    *reinterpret_cast<float4 *>(&num_part[uj][4 * cq]) = num;
    __syncthreads();
    if (tid < kHeadDim) {
        float t = 0.0f;
#pragma unroll
        for (int j = 0; j < kUnitLanes; ++j) t += num_part[j][tid];
        const size_t qi = (size_t)r * kv.num_q_heads + h * G + g;
        out[qi * kHeadDim + tid] = den > 0.0f ? t / den : 0.0f;
        if (tid == 0) {
            n_selected[qi] = n;
            mass_est[qi] = P;
            if (lse_out) lse_out[qi] = den > 0.0f ? (M + log2_fast(den)) * kLn2 : -INFINITY;
            if (g == 0) {
                int mx = 0;
                for (int x = 0; x < G; ++x) {
                    const unsigned long long sx = ctl->stop[x];
                    const int nx = (sx != ~0ull && (int)(sx >> 32) <= N) ? (int)(sx >> 32) : N;
                    mx = max(mx, nx);
                }
                if (blocks_read) blocks_read[s] = mx;
                if (traffic_out) { traffic_out[2 * s] = ctl->k_blocks; traffic_out[2 * s + 1] = mx; }
            }
        }
    }
}

template <int DT, int G>
static hipError_t launch_attend_t(const KvView &kv, const DecodeWs &ws, const DecodePlan &plan, hipStream_t st) {
    const unsigned grid = (unsigned)(kv.batch * kv.num_kv_heads) * (unsigned)plan.max_chunks;
    attend_kernel<DT, G><<<grid, 256, 0, st>>>(kv, ws, plan.chunk_blocks);
    return hipGetLastError();
}

hipError_t launch_attend(const KvView &kv, int dtype, int G, const DecodeWs &ws, const DecodePlan &plan,
                         hipStream_t st) {
#define PSA_CASE(DT, GG) \
    if (dtype == DT && G == GG) return launch_attend_t<DT, GG>(kv, ws, plan, st);
    PSA_CASE(0, 1) PSA_CASE(0, 2) PSA_CASE(0, 4) PSA_CASE(0, 8)
    PSA_CASE(1, 1) PSA_CASE(1, 2) PSA_CASE(1, 4) PSA_CASE(1, 8)
#undef PSA_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_finalize(const KvView &kv, const DecodeWs &ws, int G, int VU, float *out,
                           int32_t *n_selected, float *mass_est, int32_t *blocks_read, float *lse_out,
                           int32_t *traffic_out, hipStream_t st) {
    finalize_kernel<<<kv.batch * kv.num_kv_heads * G, 512, 0, st>>>(kv, ws, G, VU, out, n_selected, mass_est,
                                                                    blocks_read, lse_out, traffic_out);
    return hipGetLastError();
}

}  // namespace psa
