// Final merge of one PSA decode step (Algorithm 1, line 19).
//
// By the time this kernel runs, the selection kernel has fixed every query head's stop n_g and left, per chunk and head,
// (reference, sum of weights, numerator[128]).  finalize_kernel merges a head's chunks (the online-softmax merge of
// line 11, all at once): out_g = sum over the chunks of the head's own prefix of the partial numerators, over the sum of
// the partial exp-sums, both rescaled to one reference maximum.
#include "psa_host.h"

namespace psa {

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
    // Blocks the fold has gone over: all that any head uses, unless it gave up (PSA_DEVERR_STALLED); beyond them the chunks'
    // outputs may be another call's.
    const int folded = min(N, (int)(ctl->key_progress & 0xffffull) * VU);
    int n = folded;
    float P = N > 0 ? 1.0f : 0.0f;
    if (st != ~0ull && (int)(st >> 32) <= folded) { n = (int)(st >> 32); P = __uint_as_float((uint32_t)st); }
    const int nun = (n + VU - 1) / VU;
    const float *src = ws.partial + ((size_t)s * ws.max_chunks * G + g) * kPartialStride;
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
                    const int nx = (sx != ~0ull && (int)(sx >> 32) <= folded) ? (int)(sx >> 32) : folded;
                    mx = max(mx, nx);
                }
                if (blocks_read) blocks_read[s] = mx;
                if (traffic_out) { traffic_out[2 * s] = ctl->k_blocks; traffic_out[2 * s + 1] = mx; }
            }
        }
    }
}

hipError_t launch_finalize(const KvView &kv, const DecodeWs &ws, int G, int VU, float *out,
                           int32_t *n_selected, float *mass_est, int32_t *blocks_read, float *lse_out,
                           int32_t *traffic_out, hipStream_t st) {
    finalize_kernel<<<kv.batch * kv.num_kv_heads * G, 512, 0, st>>>(kv, ws, G, VU, out, n_selected, mass_est,
                                                                    blocks_read, lse_out, traffic_out);
    return hipGetLastError();
}

}  // namespace psa
