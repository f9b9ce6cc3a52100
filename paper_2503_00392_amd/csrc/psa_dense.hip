// Dense control: exact paged decode attention (softmax(q K^T / sqrt d) V over every block),
// split over the context, with fp32 online softmax; a second kernel merges the splits.
#include "psa_attend.h"
#include "psa_fold.h"
#include "psa_host.h"

namespace psa {

constexpr int kMaxSplits = 1024;   // splits of a request at most: their weights are an array in the merge's LDS
constexpr int kDenseStride = 132;  // M, l, error bits (head 0), pad, acc[128]

// grid (nsplit, S); 256 threads.  Wave w of the workgroup takes blocks b0+w, b0+w+4, ... and carries its own
// online softmax over them, both products on the matrix cores:
//   logits  D[token][head] = K[token][channel] Q[channel][head]: four 16x16x32 steps (see block_logits); lane (kq, n) =
//           (lane/16, lane%16) ends up with the logits of head n/2 for tokens kq, 4+kq, 8+kq, 12+kq -- the token rows its
//           value loads fetch;
//   values  D[head][channel] += P[head][token] V[token][channel]: eight 16x16x16 products per block (one per
//           channel of the lane's eight), the weights split into two 16-bit halves in neighbouring rows (see
//           add_weighted); lane (kq, cl) accumulates heads 2kq and 2kq+1 of channels 8cl..8cl+7.
// The running maximum of a head is shared by the wave (two exchanges per block); the four waves are merged
// once at the end.
// Bound by memory: 5.9 -> 6.1 TB/s on 6 ragged requests of up to 64K tokens (146.6 -> 141.7 us a call, each time within
// 0.1), 256 requests of up to 2048 143 -> 128 us, 8 of up to 30000 29.2 -> 27.0.  Whole rows of keys are loaded and turned
// into the operand's layout in LDS, which alone gave 145.5, 134.5 and 28.4: loaded in that layout, an instruction touched
// half a cache line of sixteen tokens and could not be marked read-once.  The next block's keys are under way while a block
// is worked on, with three workgroups to a compute unit: with two (as many registers as the compiler likes) 140.6, 129.5 and
// 30.0, with four 144.7 on the first.
template <int DT, int G>
__global__ __launch_bounds__(256, 3) void dense_split_kernel(KvView kv, const uint8_t *__restrict__ q,
                                                          float *__restrict__ partial,
                                                          int blocks_per_split, int32_t *header) {
    const int s = blockIdx.y, split = blockIdx.x, nsplit = gridDim.x;
    const int r = s / kv.num_kv_heads, h = s % kv.num_kv_heads;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rg = lane >> 4, cl = lane & 15;
    // the call's error word: cleared here, set by the merge kernel from what the workgroups found (a launch of its own for
    // the clearing cost 5 us)
    if (split == 0 && s == 0 && tid < 64) header[tid] = 0;
    const int raw_ctx = kv.ctx_lens[r], ctx = ctx_clamped_quiet(kv, r);
    int err = raw_ctx != ctx ? PSA_DEVERR_CTX_RANGE : 0;
    const int N = (ctx + kPage - 1) / kPage;
    // every request is cut into the same number of splits, each over its own length: ragged batches stay balanced
    const int bps = min(blocks_per_split, (N + nsplit - 1) / nsplit);
    const int b0 = split * bps;
    const int b1 = min(N, b0 + bps);

    // B operand of the logits: columns 2 g and 2 g + 1 = head g (zero beyond the group), channels 8*(4kk + rg) .. +7 in
    // step kk; the two lanes of a head supply the two halves of its weights (see add_weighted)
    const int hd = cl >> 1;
    uint4 qb[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        qb[kk] = make_uint4(0, 0, 0, 0);
        if (hd < G) qb[kk] = ld16(q + ((size_t)(r * kv.num_q_heads + h * G + hd) * kHeadDim + (4 * kk + rg) * 8) * 2);
    }
    __shared__ uint4 stage[4][16 * 17];                  // per wave: a key slice on its way into the operand's layout
    float m = -INFINITY, l = 0.0f;                       // head hd: running maximum (whole wave), exp-sum (this row group)
    f32x4_t acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    const int32_t *table = kv.block_table + (size_t)r * kv.max_blocks;
    int pages = 0;                                       // lane j: page of the wave's block j of 64
    auto slice_of = [&](int b, int i) __attribute__((always_inline)) {      // where block b, the wave's i-th, lies in the pools
        if ((i & 63) == 0) {
            const int bl = b + 4 * lane, page = table[min(bl, b1 - 1)];
            pages = clamp_page_quiet(page, kv.num_pages);
            if (pages != page) err |= PSA_DEVERR_PAGE_RANGE;
        }
        return ((size_t)__builtin_amdgcn_readlane(pages, i & 63) * kv.num_kv_heads + h) * kSliceBytes;
    };
    size_t off = 0;
    Slice k;
    if (b0 + wave < b1) {
        off = slice_of(b0 + wave, 0);
        k = load_slice(kv.k_pool + off, lane);
    }
    for (int b = b0 + wave, i = 0; b < b1; b += 4, ++i) {
        const Slice kc = k;
        Slice v = load_slice(kv.v_pool + off, lane);
        if (b + 4 < b1) {                                // (the next keys are under way while these are worked on)
            off = slice_of(b + 4, i + 1);
            k = load_slice(kv.k_pool + off, lane);
        }
        const int valid = min(kPage, ctx - b * kPage);
        const f32x4_t sc = block_logits<DT>(kc.r, qb, stage[wave], lane, valid);
        if (valid < kPage) zero_invalid_rows(v, rg, valid);
        float bm = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
        bm = fmaxf(bm, __shfl_xor(bm, 16));
        bm = fmaxf(bm, __shfl_xor(bm, 32));
        const float mn = fmaxf(m, bm);                   // finite: every block below N has a valid token
        const float alpha = exp2_fast(m - mn);
        float p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) p[j] = exp2_fast(sc[j] - mn);
        l = l * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
        m = mn;
        // the accumulators hold heads 2rg and 2rg + 1: rescale each by its head's factor, where a maximum has moved
        if (__ballot(alpha != 1.0f)) {
            const float a0 = __shfl(alpha, 4 * rg), a1 = __shfl(alpha, 4 * rg + 2);
#pragma unroll
            for (int t = 0; t < 8; ++t) { acc[t][0] *= a0; acc[t][1] *= a0; acc[t][2] *= a1; acc[t][3] *= a1; }
        }
        add_weighted<DT>(acc, v, p, cl & 1);
    }
    // the exp-sum over the four row groups
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);

    // merge the 4 waves through LDS
    __shared__ __attribute__((aligned(16))) float st_acc[4][G][kHeadDim];
    __shared__ float st_m[4][G], st_l[4][G];
    __shared__ int st_err[4];
    store_heads<G>(acc, st_acc[wave], rg, cl);
    if (rg == 0 && hd < G && !(cl & 1)) { st_m[wave][hd] = m; st_l[wave][hd] = l; }
    const bool bad_ctx = __ballot(err & PSA_DEVERR_CTX_RANGE) != 0ull, bad_page = __ballot(err & PSA_DEVERR_PAGE_RANGE) != 0ull;
    if (lane == 0) st_err[wave] = (bad_ctx ? PSA_DEVERR_CTX_RANGE : 0) | (bad_page ? PSA_DEVERR_PAGE_RANGE : 0);
    __syncthreads();
    float *dst = partial + ((size_t)s * nsplit + split) * G * kDenseStride;
    if (tid == 0) dst[2] = __int_as_float(st_err[0] | st_err[1] | st_err[2] | st_err[3]);
    for (int idx = tid; idx < G * kHeadDim; idx += 256) {
        const int g = idx / kHeadDim, ch = idx % kHeadDim;
        float M = fmaxf(fmaxf(st_m[0][g], st_m[1][g]), fmaxf(st_m[2][g], st_m[3][g]));
        float lsum = 0.0f, a = 0.0f;
        if (M != -INFINITY) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float sc = exp2_fast(st_m[w][g] - M);
                lsum += st_l[w][g] * sc;
                a += st_acc[w][g][ch] * sc;
            }
        }
        dst[g * kDenseStride + 4 + ch] = a;
        if (ch == 0) { dst[g * kDenseStride] = M; dst[g * kDenseStride + 1] = lsum; }
    }
}

// grid (S*G); 512 threads = 4 split lanes x 128 channels.  Split lane j takes splits j, j+4, ... in
// ascending order (loads issued four deep, no branches); the 4 lanes are then added in a fixed order.
__global__ __launch_bounds__(512) void dense_combine_kernel(const float *__restrict__ partial, int nsplit,
                                                            int G, int num_kv_heads, int num_q_heads,
                                                            float *__restrict__ out,
                                                            float *__restrict__ lse, int32_t *header) {
    __shared__ float red[8];
    __shared__ float wgt[kMaxSplits];           // rescale factor of every split
    __shared__ float num_part[4][kHeadDim];
    __shared__ float den_part[4];
    const int s = blockIdx.x / G, g = blockIdx.x % G, tid = threadIdx.x;
    const int ch = tid & 127, sl = tid >> 7;
    const int r = s / num_kv_heads, h = s % num_kv_heads;
    const float *src = partial + ((size_t)s * nsplit * G + g) * kDenseStride;
    const size_t stride = (size_t)G * kDenseStride;
    float M = -INFINITY;
    int err = 0;
    for (int i = tid; i < nsplit; i += 512) {
        const float mi = src[i * stride];
        wgt[i] = mi;
        M = fmaxf(M, mi);
        if (g == 0) err |= __float_as_int(src[i * stride + 2]);
    }
    if (err) set_error(header, err);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) M = fmaxf(M, __shfl_xor(M, d));
    if ((tid & 63) == 0) red[tid >> 6] = M;
    __syncthreads();
    M = fmaxf(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])), fmaxf(fmaxf(red[4], red[5]), fmaxf(red[6], red[7])));
    for (int i = tid; i < nsplit; i += 512) {
        const float mi = wgt[i];
        wgt[i] = (mi == -INFINITY || M == -INFINITY) ? 0.0f : exp2_fast(mi - M);
    }
    __syncthreads();
    float num = 0.0f, den = 0.0f;
    for (int i0 = sl; i0 < nsplit; i0 += 16) {
        float a[4], l[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = min(i0 + 4 * k, nsplit - 1);          // clamped: the loads need no branch
            a[k] = src[i * stride + 4 + ch];
            l[k] = src[i * stride + 1];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float w = (i0 + 4 * k < nsplit) ? wgt[i0 + 4 * k] : 0.0f;
            num = fmaf(a[k], w, num);
            den = fmaf(l[k], w, den);
        }
    }
    num_part[sl][ch] = num;
    if (ch == 0) den_part[sl] = den;
    __syncthreads();
    if (tid < kHeadDim) {
        const float n = (num_part[0][tid] + num_part[1][tid]) + (num_part[2][tid] + num_part[3][tid]);
        const float dsum = (den_part[0] + den_part[1]) + (den_part[2] + den_part[3]);
        const size_t qi = (size_t)r * num_q_heads + h * G + g;
        out[qi * kHeadDim + tid] = dsum > 0.0f ? n / dsum : 0.0f;
        if (lse && tid == 0) lse[qi] = dsum > 0.0f ? (M + log2_fast(dsum)) * kLn2 : -INFINITY;
    }
}

// ---- host side ----------------------------------------------------------------------------------
int dense_num_splits(const psa_kv_desc *d) {
    const int S = d->batch * d->num_kv_heads;
    // aim at ~8 workgroups per CU over the whole grid, at least 8 blocks (64 KiB of K+V) per split
    int want = (2048 + S - 1) / S;
    int max_by_len = (d->max_blocks_per_seq + 7) / 8;
    int n = want < max_by_len ? want : max_by_len;
    if (n > kMaxSplits) n = kMaxSplits;
    return n < 1 ? 1 : n;
}

size_t dense_workspace_bytes(const psa_kv_desc *d) {
    const size_t S = (size_t)d->batch * d->num_kv_heads;
    const int G = d->num_q_heads / d->num_kv_heads;
    return 256 + S * dense_num_splits(d) * G * kDenseStride * sizeof(float);
}

template <int DT, int G>
static hipError_t launch_dense_t(const KvView &kv, const void *q, float *out, float *lse, void *ws,
                                 int nsplit, hipStream_t st) {
    int32_t *header = reinterpret_cast<int32_t *>(ws);
    float *partial = reinterpret_cast<float *>(reinterpret_cast<uint8_t *>(ws) + 256);
    const int S = kv.batch * kv.num_kv_heads;
    const int bps = (kv.max_blocks + nsplit - 1) / nsplit;
    dense_split_kernel<DT, G><<<dim3(nsplit, S), 256, 0, st>>>(kv, (const uint8_t *)q, partial, bps, header);
    dense_combine_kernel<<<S * G, 512, 0, st>>>(partial, nsplit, G, kv.num_kv_heads, kv.num_q_heads, out, lse, header);
    return hipGetLastError();
}

hipError_t launch_dense(const psa_kv_desc *d, const void *q, float *out, float *lse, void *ws,
                        hipStream_t st) {
    const KvView kv = make_view(d);
    const int G = d->num_q_heads / d->num_kv_heads;
    const int nsplit = dense_num_splits(d);
    if (kv.num_pages == 0) {
        DecodeArgs a{};
        a.out = out;
        a.lse_out = lse;
        return launch_no_pages(kv, a, reinterpret_cast<int32_t *>(ws), st);
    }
#define PSA_CASE(DT, GG) \
    if (d->dtype == DT && G == GG) return launch_dense_t<DT, GG>(kv, q, out, lse, ws, nsplit, st);
    PSA_CASE(0, 1) PSA_CASE(0, 2) PSA_CASE(0, 4) PSA_CASE(0, 8)
    PSA_CASE(1, 1) PSA_CASE(1, 2) PSA_CASE(1, 4) PSA_CASE(1, 8)
#undef PSA_CASE
    return hipErrorInvalidValue;
}

}  // namespace psa
