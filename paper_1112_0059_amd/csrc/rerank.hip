// FP8 candidate pass support and exact re-rank (float descriptors).
//
//   k_fp8_rowprep   per reference: power-of-two scale, E8M0 exponent, seed
//   k_fp8_pack      references -> FP8 A-fragment tiles
//   k_fp8_qprep     queries -> FP8 codes of -q * 2^e_q and E8M0 2^(1-e_q)
//   k_cand_merge    per query: 4k best candidates over the half/slice lists (the
//                   shared-list variants find theirs in refine.hip)
//   k_rerank        per query (one wave): exact FP32 squared distances of the
//                   candidates, the k+1 nearest by (distance, index), and
//                   Algorithm 2's per-class updates dist_C - dist_B
//   k_img_reduce    per image: per-class sums of the updates (FP64, in an order
//                   the image's size alone fixes), and the argmin
//
// Every step depends only on the image's own descriptors, so an image's
// result is the same whatever batch it is classified in.
#include "wave_select.h"

namespace lnbnn {

// Largest e with m * 2^e <= 448 (OCP e4m3 maximum), for m > 0; 0 for m == 0.
// Clamped so that the E8M0 exponents built from it stay inside 1..254.
static __device__ __forceinline__ int fp8_exponent(float m)
{
    if (!(m > 0.0f)) return 0;
    int ex;
    (void)frexpf(m, &ex);                 // m < 2^ex
    int e = 8 - ex;                       // m * 2^e < 256 <= 448
    if (ldexpf(m, e + 1) <= 448.0f) e += 1;
    return max(-120, min(120, e));
}

// pack two floats into two OCP e4m3 codes (round to nearest even)
static __device__ __forceinline__ uint32_t fp8x2(float a, float b)
{
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false) & 0xffffu;
}

// Seed (squared norm) and E8M0 exponent of every row.  A reference with a NaN or
// an infinity, or whose squared norm overflows, is packed like a padding row (seed
// +inf, zero codes), which no key passes: a NaN key would hide the other rows of
// its tile, whose smallest key it makes NaN.
__global__ void k_fp8_rowprep(const float *__restrict__ refs, int64_t n_refs, int64_t n_pad,
                              int32_t *__restrict__ rsc, float *__restrict__ seed)
{
    for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < n_pad;
         row += (int64_t)gridDim.x * blockDim.x) {
        if (row >= n_refs) {
            rsc[row] = 127;
            seed[row] = __builtin_inff();
            continue;
        }
        const float4 *p = reinterpret_cast<const float4 *>(refs + row * kDim);
        float m = 0.0f;
        bool finite = true;
        for (int c = 0; c < kDim / 4; ++c) {
            const float4 v = p[c];
            m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
            finite = finite && isfinite(v.x) && isfinite(v.y) && isfinite(v.z) && isfinite(v.w);
        }
        const int e = finite ? fp8_exponent(m) : 0;
        // ||r~||^2 of the dequantised values r~ = fp8(r * 2^e) * 2^-e
        float s = 0.0f;
        for (int c = 0; c < kDim / 4; ++c) {
            const float4 v = p[c];
            const uint32_t lo = fp8x2(ldexpf(v.x, e), ldexpf(v.y, e));
            const uint32_t hi = fp8x2(ldexpf(v.z, e), ldexpf(v.w, e));
            const int w = (int)(lo | (hi << 16));
            const float r0 = ldexpf(__builtin_amdgcn_cvt_f32_fp8(w, 0), -e);
            const float r1 = ldexpf(__builtin_amdgcn_cvt_f32_fp8(w, 1), -e);
            const float r2 = ldexpf(__builtin_amdgcn_cvt_f32_fp8(w, 2), -e);
            const float r3 = ldexpf(__builtin_amdgcn_cvt_f32_fp8(w, 3), -e);
            s = fmaf(r0, r0, s);
            s = fmaf(r1, r1, s);
            s = fmaf(r2, r2, s);
            s = fmaf(r3, r3, s);
        }
        rsc[row] = 127 - e;
        seed[row] = finite && isfinite(s) ? s : __builtin_inff();
    }
}

// Fragment u = ((tile * 2 + s) * 2 + half) * 64 + lane: 16 codes of row
// 32*tile + (lane & 31), K elements 64*s + 32*(lane >> 5) + 16*half + 0..15.
__global__ void k_fp8_pack(const float *__restrict__ refs, int64_t n_refs, int64_t n_frag,
                           const int32_t *__restrict__ rsc, const float *__restrict__ seed,
                           uint4 *__restrict__ frag)
{
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < n_frag;
         u += (int64_t)gridDim.x * blockDim.x) {
        const int lane = (int)(u & 63);
        const int half = (int)((u >> 6) & 1);
        const int s = (int)((u >> 7) & 1);
        const int64_t tile = u >> 8;
        const int64_t row = tile * kTileRows + (lane & 31);
        uint4 out = make_uint4(0u, 0u, 0u, 0u);
        if (row < n_refs && seed[row] < __builtin_inff()) {
            const int e = 127 - rsc[row];
            const float4 *p = reinterpret_cast<const float4 *>(refs + row * kDim + 64 * s + 32 * (lane >> 5) + 16 * half);
            uint32_t w[4];
            for (int c = 0; c < 4; ++c) {
                const float4 v = p[c];
                w[c] = fp8x2(ldexpf(v.x, e), ldexpf(v.y, e)) | (fp8x2(ldexpf(v.z, e), ldexpf(v.w, e)) << 16);
            }
            out = make_uint4(w[0], w[1], w[2], w[3]);
        }
        frag[u] = out;
    }
}

// Queries: codes of -q * 2^e_q in natural K order and the E8M0 exponent of
// 2^(1 - e_q), so the candidate pass accumulates -2 q~.r~.
__global__ void k_fp8_qprep(const BatchDesc *bd, uint4 *__restrict__ q8, int32_t *__restrict__ qsc)
{
    const int64_t n_q = bd->n_q;
    const float *q = static_cast<const float *>(bd->q);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_q; i += (int64_t)gridDim.x * blockDim.x) {
        const float4 *p = reinterpret_cast<const float4 *>(q + i * kDim);
        float m = 0.0f;
        for (int c = 0; c < kDim / 4; ++c) {
            const float4 v = p[c];
            m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
        }
        const int e = fp8_exponent(m);
        for (int c = 0; c < kDim / 16; ++c) {
            uint32_t w[4];
            for (int j = 0; j < 4; ++j) {
                const float4 v = p[4 * c + j];
                w[j] = fp8x2(-ldexpf(v.x, e), -ldexpf(v.y, e)) | (fp8x2(-ldexpf(v.z, e), -ldexpf(v.w, e)) << 16);
            }
            q8[i * (kDim / 16) + c] = make_uint4(w[0], w[1], w[2], w[3]);
        }
        qsc[i] = 128 - e;
    }
}

// One wave per query: the n_cand best (key, index) pairs over the n_lists
// sorted candidate lists of kp_stride entries each (together at least n_cand;
// entries past a list's real rows have index -1).  The lists are taken rank by
// rank, 64 of them at a time, until a rank adds nothing.  With one thread per
// query this merge was a chain of n_cand x n_lists dependent loads on a few
// workgroups: 1.52 ms for 1,999 descriptors of 64 lists, now 45 us.
__global__ __launch_bounds__(256) void k_cand_merge(RerankArgs a)
{
    constexpr int CAP = 192;        // 4 * 32 candidates + 64
    __shared__ uint64_t s_sel[4][WaveSelect<CAP>::kSize];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n_q = a.bd->n_q;
    for (int64_t q = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(wave); q < n_q; q += (int64_t)gridDim.x * 4) {
        const int64_t base = ((int64_t)min(lane, a.n_lists - 1) * a.q_cap + q) * a.kp_stride;
        const bool in = lane < a.n_lists;
        // a list's last key is NaN: its stage wait gave up
        const bool marked = in && __builtin_isnan(a.part_d[base + a.kp_stride - 1]);
        if (__builtin_amdgcn_ballot_w64(marked) != 0 && lane == 0) *a.status = kStatusWaitGaveUp;
        WaveSelect<CAP> sel(s_sel[wave], a.n_cand, ~0ull);
        for (int p = 0; p < a.kp_stride; ++p) {
            const int i = a.part_i[base + p];
            if (!sel.add(pair_of(a.part_d[base + p], i), in && i >= 0, lane)) break;
        }
        sel.cut(lane);
        for (int j = lane; j < a.n_cand; j += 64) a.cand[q * a.n_cand + j] = j < sel.n ? pair_index(sel.buf[j]) : -1;
        wave_lds_fence();
    }
}

static __device__ __forceinline__ bool pair_less(float d0, int i0, float d1, int i1)
{
    return d0 < d1 || (d0 == d1 && (uint32_t)i0 < (uint32_t)i1);
}

// One wave per query.  Lane j holds candidates j and j + 64 (n_cand <= 128)
// and computes each one's squared distance in FP32, directly as
// sum_t (q_t - r_t)^2 in dimension order; the candidates are ranked by
// (distance, index); the k+1 smallest are the neighbours.  The holder of
// rank j < k emits Algorithm 2's update for its class if no lower rank has
// that class: dist_C - dist_B, formed in FP64 from the two FP32 distances
// (exactly).
__global__ __launch_bounds__(256) void k_rerank(RerankArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t n_q = a.bd->n_q;
    const int k = a.k;
    const int nc = a.n_cand > 64 ? 2 : 1;       // candidate slots per lane
    const float *qf32 = static_cast<const float *>(a.bd->q);
    int32_t *nbr_idx = a.bd->nbr_idx;
    float *nbr_dist = a.bd->nbr_dist;
    for (int64_t q = blockIdx.x * 4 + (threadIdx.x >> 6); q < n_q; q += (int64_t)gridDim.x * 4) {
        float d[2];
        int idx[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int j = lane + 64 * c;
            d[c] = __builtin_inff();
            idx[c] = 0x7fffffff;
            if (j >= a.n_cand) continue;
            const int r = a.cand[q * a.n_cand + j];
            if (r < 0 || r >= a.n_refs) continue;
            const float4 *qr = reinterpret_cast<const float4 *>(qf32 + q * kDim);
            const float4 *rr = reinterpret_cast<const float4 *>(a.ref_f32 + (int64_t)r * kDim);
            float s = 0.0f;
            for (int t = 0; t < kDim / 4; ++t) {
                const float4 x = qr[t], y = rr[t];
                float e = x.x - y.x;
                s = fmaf(e, e, s);
                e = x.y - y.y;
                s = fmaf(e, e, s);
                e = x.z - y.z;
                s = fmaf(e, e, s);
                e = x.w - y.w;
                s = fmaf(e, e, s);
            }
            d[c] = s;
            idx[c] = r;
        }
        int rank[2] = {0, 0};
        for (int c2 = 0; c2 < nc; ++c2) {
            for (int i = 0; i < 64; ++i) {
                const float di = __shfl(d[c2], i);
                const int ii = __shfl(idx[c2], i);
#pragma unroll
                for (int c = 0; c < 2; ++c) rank[c] += pair_less(di, ii, d[c], idx[c]) ? 1 : 0;
            }
        }
        const unsigned long long m0 = __builtin_amdgcn_ballot_w64(rank[0] == k);
        const unsigned long long m1 = __builtin_amdgcn_ballot_w64(nc > 1 && rank[1] == k);
        // the holder of rank k (always one with valid lists; lane 0 otherwise)
        const int src = m0 ? (int)__builtin_ctzll(m0) : m1 ? (int)__builtin_ctzll(m1) : 0;
        const float db = m0 ? __shfl(d[0], src) : __shfl(d[1], src);
        int cls[2];
        bool first[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            // a slot without a real candidate (only possible when the lists
            // are invalid, e.g. after a stage wait gave up) never reads a label
            const bool real = idx[c] >= 0 && idx[c] < a.n_refs;
            first[c] = c < nc && rank[c] < k && real;
            cls[c] = first[c] ? a.labels[idx[c]] : -1;
        }
        for (int c2 = 0; c2 < nc; ++c2) {
            for (int i = 0; i < 64; ++i) {
                const int ri = __shfl(rank[c2], i);
                const int ci = __shfl(cls[c2], i);
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    if (ri < rank[c] && ci == cls[c]) first[c] = false;
            }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (c >= nc) break;
            if (rank[c] < k) {
                a.upd_cls[q * k + rank[c]] = first[c] ? cls[c] : -1;
                a.upd_delta[q * k + rank[c]] = (double)d[c] - (double)db;
            }
            if (nbr_idx && rank[c] <= k) {
                nbr_idx[q * (k + 1) + rank[c]] = idx[c];
                nbr_dist[q * (k + 1) + rank[c]] = d[c];
            }
        }
    }
}

// One workgroup per image: totals[c] = sum of the updates of class c over the
// image's descriptors; argmin with the lowest class on ties.  Classes with no
// update stay 0.
//
// A group of G lanes takes a contiguous share of the image's descriptors in
// order, one lane per neighbour rank (a descriptor updates a class at most
// once, so the lanes of a group never collide), and adds to sums of its own in
// LDS; the groups' sums are then added in group order.  The order of every sum
// depends on the image's descriptor count and k alone, so an image's totals are
// the same in any batch.  Classes beyond the LDS window take another pass.
//
// Before, every thread owned a class and walked all the image's updates: 2.48 ms
// for eight images of 500-4,000 descriptors (k = 10), one workgroup each, now
// 32 us.
template <int G>
__global__ __launch_bounds__(512) void k_img_reduce(RerankArgs a)
{
    constexpr int GROUPS = 512 / G;
    constexpr int WINDOW = 8192 / GROUPS;           // classes per pass
    constexpr int AHEAD = 4;                        // descriptors loaded ahead of their sums
    __shared__ double s_sum[GROUPS][WINDOW];
    __shared__ double s_bv[512];
    __shared__ int s_bc[512];
    const int tid = threadIdx.x, group = tid / G, j = tid % G;
    const int64_t n_img = a.bd->n_img;
    double *totals = static_cast<double *>(a.bd->totals);
    const int k = a.k;
    for (int64_t img = blockIdx.x; img < n_img; img += gridDim.x) {
        const int64_t q0 = a.offsets[img], n = a.offsets[img + 1] - q0;
        const int64_t share = (n + GROUPS - 1) / GROUPS;
        const int64_t g0 = q0 + min(n, group * share), g1 = q0 + min(n, (group + 1) * share);
        double best = __builtin_inf();
        int bc = 0x7fffffff;
        for (int c0 = 0; c0 < a.n_classes; c0 += WINDOW) {
            for (int i = tid; i < GROUPS * WINDOW; i += 512) (&s_sum[0][0])[i] = 0.0;
            __syncthreads();
            for (int64_t q = g0; q < g1; q += AHEAD) {
                int c[AHEAD];
                double d[AHEAD];
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    const bool in = q + u < g1 && j < k;
                    const int64_t o = (in ? q + u : q0) * k + (in ? j : 0);
                    const int cls = a.upd_cls[o];
                    d[u] = a.upd_delta[o];
                    c[u] = in && cls >= c0 && cls < c0 + WINDOW ? cls - c0 : -1;
                }
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    if (c[u] >= 0) s_sum[group][c[u]] += d[u];
                    wave_lds_fence();
                }
            }
            __syncthreads();
            const int c = c0 + tid;
            if (tid < WINDOW && c < a.n_classes) {
                double sum = 0.0;
                for (int g = 0; g < GROUPS; ++g) sum += s_sum[g][tid];
                totals[img * a.n_classes + c] = sum;
                if (sum < best) {
                    best = sum;
                    bc = c;
                }
            }
            __syncthreads();
        }
        s_bv[tid] = best;
        s_bc[tid] = bc;
        __syncthreads();
        for (int off = 256; off > 0; off >>= 1) {
            if (tid < off) {
                const double ov = s_bv[tid + off];
                const int oc = s_bc[tid + off];
                if (ov < s_bv[tid] || (ov == s_bv[tid] && oc < s_bc[tid])) {
                    s_bv[tid] = ov;
                    s_bc[tid] = oc;
                }
            }
            __syncthreads();
        }
        if (tid == 0) a.bd->cls[img] = s_bc[0] == 0x7fffffff ? 0 : s_bc[0];
        __syncthreads();
    }
}

hipError_t launch_fp8_index(const float *refs, int64_t n_refs, int64_t n_pad, uint4 *frag, float *seed,
                            int32_t *rsc, hipStream_t s)
{
    k_fp8_rowprep<<<grid_for(n_pad, 256, 65536), 256, 0, s>>>(refs, n_refs, n_pad, rsc, seed);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t n_frag = (n_pad / kTileRows) * 4 * 64;
    k_fp8_pack<<<grid_for(n_frag, 256, 65536), 256, 0, s>>>(refs, n_refs, n_frag, rsc, seed, frag);
    return hipGetLastError();
}

hipError_t launch_fp8_qprep(const BatchDesc *bd, int64_t q_cap, uint4 *q8, int32_t *qsc, hipStream_t s)
{
    k_fp8_qprep<<<grid_for(q_cap, 256, 16384), 256, 0, s>>>(bd, q8, qsc);
    return hipGetLastError();
}

hipError_t launch_cand_merge(const RerankArgs &a, int64_t q_cap, hipStream_t s)
{
    k_cand_merge<<<grid_for(q_cap, 4, 65536), 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_rerank(const RerankArgs &a, int64_t q_cap, int64_t img_cap, hipStream_t s)
{
    k_rerank<<<grid_for(q_cap, 4, 65536), 256, 0, s>>>(a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.k <= 16)
        k_img_reduce<16><<<grid_for(img_cap, 1, 16384), 512, 0, s>>>(a);
    else
        k_img_reduce<32><<<grid_for(img_cap, 1, 16384), 512, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace lnbnn
