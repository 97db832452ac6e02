// HIP kernels of the local NBNN hot path for gfx950 (MI355X), apart from
// the distance kernel itself (dist_topk.h, instantiated by dist_inst.hip):
//
// K0  pack        references -> MFMA A-fragment tiles + accumulator seeds
// K2  finish      merge of the per-slice lists, background distance,
//                 per-class update of the image totals (Algorithm 2 body); the
//                 shared-list variants finish in refine.hip
// K3  argmin      per-image decision (Algorithm 2, return line)
// plus the variant table and the dispatch to the K1 instances.  (The FP8
// packing, candidate merge, exact re-rank and per-image reduction live in
// rerank.hip.)
#include <algorithm>

#include "dist_topk.h"

namespace lnbnn {

// ---------------------------------------------------------------------------
// K0: packing of u8 references.
//
// k_pack_u8 (16-bit formats): fragment u = (tile * kSteps + s) * 64 + lane
// holds the eight K elements lane `lane` supplies at step s for row 32*tile +
// (lane & 31).
// ---------------------------------------------------------------------------
template <class Op>
__global__ void k_pack_u8(const uint8_t *__restrict__ refs, int64_t n_refs, int64_t n_frag,
                          uint4 *__restrict__ frag)
{
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < n_frag;
         u += (int64_t)gridDim.x * blockDim.x) {
        const int lane = (int)(u & 63);
        const int s = (int)((u >> 6) % Op::kSteps);
        const int64_t tile = (u >> 6) / Op::kSteps;
        const int64_t src = tile * kTileRows + (lane & 31);
        const bool ok = src < n_refs;
        frag[u] = Op::pack_frag(refs + (ok ? src : 0) * Op::kRow, ok, s, lane >> 5);
    }
}

// INT8 rows: fragments and seeds in one pass.  Packed row r holds reference
// perm[r] (padding where perm[r] < 0).  G lanes share a row, one 16-byte chunk
// each (lane c: K elements 16c..16c+15, fragment half c & 1 of step c >> 1), so a
// row is read as one contiguous run, once.  Seeds: floor(||s||^2 / 2) + sum(s)
// with s = r - 128 (stored as the int32 bit pattern), 2^30 on padding rows.
template <class Op, int G>
__global__ __launch_bounds__(256) void k_pack_i8(const uint8_t *__restrict__ refs, int64_t n_pad,
                                                 uint4 *__restrict__ frag, int32_t *__restrict__ seed,
                                                 const int32_t *__restrict__ perm)
{
    constexpr int C = Op::kRow / 16;
    const int c = threadIdx.x % G;
    for (int64_t row = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / G; row < n_pad;
         row += (int64_t)gridDim.x * blockDim.x / G) {
        const int32_t src = perm[row];
        int32_t sq = 0, sum = 0;
        if (c < C) {
            const uint4 v = Op::pack_frag(refs + (int64_t)(src < 0 ? 0 : src) * Op::kRow, src >= 0, c >> 1, c & 1);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sq = __builtin_amdgcn_sdot4((int)w[i], (int)w[i], sq, false);
                sum = __builtin_amdgcn_sdot4((int)w[i], 0x01010101, sum, false);
            }
            frag[((row / kTileRows) * Op::kSteps + (c >> 1)) * 64 + (row & 31) + 32 * (c & 1)] = v;
        }
#pragma unroll
        for (int o = 1; o < G; o <<= 1) {
            sq += __shfl_xor(sq, o);
            sum += __shfl_xor(sum, o);
        }
        if (c == 0) seed[row] = src >= 0 ? (sq >> 1) + sum : Op::kPadSeed;
    }
}

// Parity of ||r - 128||^2 per reference row: the same as the parity of the
// row's byte sum, since x^2 and x have the same parity and 128 is even; that
// is the xor of the bytes' low bits.  Sixteen lanes per row (one 16-byte chunk
// each), so rows are read as contiguous runs.
__global__ __launch_bounds__(256) void k_row_parity(const uint8_t *__restrict__ refs, int64_t n_refs, int dim,
                                                    uint8_t *__restrict__ out)
{
    const int c = threadIdx.x & 15;
    for (int64_t row = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 4; row < n_refs;
         row += ((int64_t)gridDim.x * blockDim.x) >> 4) {
        uint32_t x = 0;
        if (c < dim / 16) {
            const uint4 v = reinterpret_cast<const uint4 *>(refs + row * dim)[c];
            x = v.x ^ v.y ^ v.z ^ v.w;
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) x ^= __shfl_xor(x, o);
        x ^= x >> 16;
        x ^= x >> 8;
        if (c == 0) out[row] = (uint8_t)(x & 1u);
    }
}

__global__ __launch_bounds__(256) void k_check_labels(const int32_t *__restrict__ labels, int32_t n, int32_t n_classes,
                                                      int32_t *__restrict__ first_bad)
{
    int bad = n;
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        if (labels[i] < 0 || labels[i] >= n_classes) bad = min(bad, (int)i);
    if (bad < n) atomicMin(first_bad, bad);
}

__global__ void k_set_i32(int32_t *p, int32_t v) { *p = v; }

// Odd rows of each 256-row block.
__global__ __launch_bounds__(256) void k_parity_blocks(const uint8_t *__restrict__ par, int64_t n_refs,
                                                       int32_t *__restrict__ block_odd)
{
    __shared__ int s_n[4];
    const int64_t row = blockIdx.x * (int64_t)256 + threadIdx.x;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(row < n_refs && par[row]);
    if ((threadIdx.x & 63) == 0) s_n[threadIdx.x >> 6] = (int)__builtin_popcountll(m);
    __syncthreads();
    if (threadIdx.x == 0) block_odd[blockIdx.x] = s_n[0] + s_n[1] + s_n[2] + s_n[3];
}

// In-place exclusive prefix sums of v[0, n), the total into v[n].  One workgroup.
__global__ __launch_bounds__(1024) void k_prefix(int32_t *__restrict__ v, int64_t n)
{
    __shared__ int s_w[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int base = 0;
    for (int64_t at = 0; at < n; at += 1024) {
        const int64_t i = at + threadIdx.x;
        const int x = i < n ? v[i] : 0;
        int inc = x;
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(inc, o);
            if (lane >= o) inc += y;
        }
        if (lane == 63) s_w[wave] = inc;
        __syncthreads();
        int before = 0, all = 0;
        for (int w = 0; w < 16; ++w) {
            before += w < wave ? s_w[w] : 0;
            all += s_w[w];
        }
        if (i < n) v[i] = base + before + inc - x;
        base += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) v[n] = base;
}

// The packed order: even rows from 0, odd rows from even_pad, padding between.
__global__ __launch_bounds__(256) void k_parity_perm(const uint8_t *__restrict__ par, int64_t n_refs, int64_t n_blocks,
                                                     const int32_t *__restrict__ block_odd, int64_t even_pad,
                                                     int64_t n_pad, int32_t *__restrict__ perm)
{
    __shared__ int s_n[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row = blockIdx.x * (int64_t)256 + threadIdx.x;
    const bool odd = row < n_refs && par[row];
    const unsigned long long m = __builtin_amdgcn_ballot_w64(odd);
    if (lane == 0) s_n[wave] = (int)__builtin_popcountll(m);
    __syncthreads();
    int64_t before = block_odd[blockIdx.x];          // odd rows before this one
    for (int w = 0; w < wave; ++w) before += s_n[w];
    before += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
    if (row < n_refs) perm[odd ? even_pad + before : row - before] = (int32_t)row;
    if (blockIdx.x == 0) {
        const int64_t n_odd = block_odd[n_blocks];
        for (int64_t r = n_refs - n_odd + threadIdx.x; r < even_pad; r += 256) perm[r] = -1;
        for (int64_t r = even_pad + n_odd + threadIdx.x; r < n_pad; r += 256) perm[r] = -1;
    }
}

// Accumulator seed ||r||^2 (an exact integer in FP32), +inf on padding rows
// so they never enter a neighbour list.
__global__ void k_seed_u8(const uint8_t *__restrict__ refs, int64_t n_refs, int64_t n_pad,
                          float *__restrict__ seed)
{
    for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < n_pad;
         row += (int64_t)gridDim.x * blockDim.x) {
        if (row >= n_refs) {
            seed[row] = __builtin_inff();
            continue;
        }
        const uint4 *p = reinterpret_cast<const uint4 *>(refs + row * kDim);
        uint32_t acc = 0;
#pragma unroll
        for (int c = 0; c < kDim / 16; ++c) {
            uint4 v = p[c];
            uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    uint32_t x = (w[i] >> (8 * b)) & 0xffu;
                    acc += x * x;
                }
        }
        seed[row] = (float)acc;
    }
}

// ---------------------------------------------------------------------------
// K2: finish.  One thread per query: merge the n_lists sorted partial
// lists into the k+1 best (d', index) pairs, then apply Algorithm 2's update:
// dist_B is the (k+1)-th distance, and each class met among the first k
// neighbours, at its first (= nearest) occurrence, adds dist_C - dist_B to
// the image total.  Exact modes add exact integers with 64-bit atomics, so
// totals do not depend on the order of the atomics.
// ---------------------------------------------------------------------------
static __device__ __forceinline__ bool pair_less(float d0, int i0, float d1, int i1)
{
    return d0 < d1 || (d0 == d1 && (uint32_t)i0 < (uint32_t)i1);
}

// Reference of a packed row.  A row outside the packed set cannot occur; the
// guards keep a defect visible as a wrong answer instead of a wild read.
static __device__ __forceinline__ int reference_of(const FinishArgs &a, int row)
{
    if (row < 0 || row >= a.n_rows) return -1;
    const int i = a.perm ? a.perm[row] : row;
    return i < a.n_refs ? i : -1;
}

__global__ __launch_bounds__(256) void k_finish(FinishArgs a)
{
    const int64_t n_q = a.bd->n_q;
    const int64_t n_img = a.bd->n_img;
    unsigned long long *totals = static_cast<unsigned long long *>(a.bd->totals);
    const int kp = a.k + 1;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n_q;
         q += (int64_t)gridDim.x * blockDim.x) {
        int heads[kMaxLists];
        bool marked = false;            // a list's last key is NaN: its stage wait gave up
        for (int l = 0; l < a.n_lists; ++l) {
            heads[l] = 0;
            const float last = a.part_d[((int64_t)l * a.q_cap + q) * a.kp_stride + a.kp_stride - 1];
            marked = marked || __builtin_isnan(last);
        }
        if (marked) *a.status = kStatusWaitGaveUp;
        float dd[kMaxKP];
        int ii[kMaxKP];
        for (int p = 0; p < kp; ++p) {
            float bd = __builtin_inff();
            int bi = -1, bl = 0;
            for (int l = 0; l < a.n_lists; ++l) {
                if (heads[l] >= kp) continue;
                const int64_t o = ((int64_t)l * a.q_cap + q) * a.kp_stride + heads[l];
                const float d = a.part_d[o];
                const int i = a.part_i[o];
                if (pair_less(d, i, bd, bi)) {
                    bd = d;
                    bi = i;
                    bl = l;
                }
            }
            heads[bl] += 1;
            dd[p] = bd;
            ii[p] = reference_of(a, bi);
        }
        // ||q - shift||^2 turns the key back into the squared distance
        const uint4 *qr = reinterpret_cast<const uint4 *>(static_cast<const uint8_t *>(a.bd->q) + q * a.dim);
        uint32_t qq = 0;
        for (int c = 0; c < a.dim / 16; ++c) {
            const uint4 v = qr[c];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            for (int i = 0; i < 4; ++i)
                for (int b = 0; b < 4; ++b) {
                    const int32_t x = (int32_t)((w[i] >> (8 * b)) & 0xffu) - a.q_shift;
                    qq += (uint32_t)(x * x);
                }
        }
        // image of query q: last m with offsets[m] <= q
        int64_t lo = 0, hi = n_img - 1;
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (a.offsets[mid] <= q) lo = mid; else hi = mid - 1;
        }
        const int64_t img = lo;
        const int db = (int)dd[a.k];
        int lab[kMaxKP];
        for (int j = 0; j < a.k; ++j) {
            const int c = ii[j] >= 0 ? a.labels[ii[j]] : 0;
            lab[j] = c;
            bool first = true;
            for (int jj = 0; jj < j; ++jj) first = first && (lab[jj] != c);
            if (first) {
                const long long delta = (long long)((int)dd[j] - db);
                atomicAdd(totals + img * a.n_classes + c, (unsigned long long)delta);
            }
        }
        int32_t *nbr_idx = a.bd->nbr_idx;
        float *nbr_dist = a.bd->nbr_dist;
        if (nbr_idx) {
            for (int p = 0; p < kp; ++p) {
                nbr_idx[q * kp + p] = ii[p];
                nbr_dist[q * kp + p] = dd[p] + (float)qq;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// K3: argmin over classes, lowest class on ties.  One wave per image.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_argmin(const BatchDesc *bd, int32_t n_classes)
{
    const long long *totals = static_cast<const long long *>(bd->totals);
    int32_t *out_class = bd->cls;
    const int lane = threadIdx.x & 63;
    const int64_t n_img = bd->n_img;
    for (int64_t img = blockIdx.x * 4 + (threadIdx.x >> 6); img < n_img; img += (int64_t)gridDim.x * 4) {
        const long long *t = totals + img * n_classes;
        long long best = 0x7fffffffffffffffLL;
        int bc = 0x7fffffff;
        for (int c = lane; c < n_classes; c += 64) {
            const long long v = t[c];
            if (v < best) {
                best = v;
                bc = c;
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            const long long ov = __shfl_xor(best, off);
            const int oc = __shfl_xor(bc, off);
            if (ov < best || (ov == best && oc < bc)) {
                best = ov;
                bc = oc;
            }
        }
        if (lane == 0) out_class[img] = bc;
    }
}

// [rows][stride] array: entries [r][0, bd->n_q) set to v.
__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t stride, int64_t rows, const BatchDesc *bd)
{
    const int64_t n = bd->n_q;
    for (int64_t r = blockIdx.y; r < rows; r += gridDim.y)
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
            p[r * stride + i] = v;
}

// ---------------------------------------------------------------------------
// Original NBNN totals (Algorithm 1): totals[img][C] = sum over the image's
// descriptors d of ||d - NN_C(d)||^2.  cls_min holds the smallest INT8 key
// of every (class, query); the squared distance is that key plus
// ||q - 128||^2.  A workgroup takes 32 classes of an image: each wave every 4th
// of them, lanes over the image's queries (64-bit sums, exact), four loads in
// flight; the norms are summed by each workgroup again, which reads 128 bytes
// per query next to the classes' 128.  One workgroup per image left 8 images on
// 8 CUs.
// ---------------------------------------------------------------------------
constexpr int kTotalsClasses = 32;

__global__ __launch_bounds__(256) void k_nbnn_totals(NbnnArgs a)
{
    __shared__ long long s_nrm[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n_img = a.bd->n_img;
    const uint8_t *qb = static_cast<const uint8_t *>(a.bd->q);
    unsigned long long *totals = static_cast<unsigned long long *>(a.bd->totals);
    const int groups = (a.n_classes + kTotalsClasses - 1) / kTotalsClasses;
    for (int64_t u = blockIdx.x; u < n_img * groups; u += gridDim.x) {
        const int64_t img = u / groups;
        const int c0 = (int)(u - img * groups) * kTotalsClasses, c1 = min(c0 + kTotalsClasses, a.n_classes);
        const int64_t q0 = a.offsets[img], q1 = a.offsets[img + 1];
        long long nrm = 0;
        // eight lanes per query, one 16-byte chunk each
        for (int64_t i = q0 * 8 + tid; i < q1 * 8; i += 256) {
            const uint4 v = reinterpret_cast<const uint4 *>(qb)[i];
            const uint32_t w[4] = {v.x ^ 0x80808080u, v.y ^ 0x80808080u, v.z ^ 0x80808080u, v.w ^ 0x80808080u};
            int32_t sq = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) sq = __builtin_amdgcn_sdot4((int)w[j], (int)w[j], sq, false);
            nrm += sq;
        }
        for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off);
        if (lane == 0) s_nrm[wave] = nrm;
        __syncthreads();
        nrm = s_nrm[0] + s_nrm[1] + s_nrm[2] + s_nrm[3];
        for (int c = c0 + wave; c < c1; c += 4) {
            const int32_t *m = a.cls_min + (int64_t)c * a.q_cap;
            long long sum = 0;
            for (int64_t q = q0 + lane; q < q1; q += 256) {
                int32_t x[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = q + 64 * j < q1 ? m[q + 64 * j] : 0;
                sum += (long long)x[0] + x[1] + x[2] + x[3];
            }
            for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
            if (lane == 0) totals[img * a.n_classes + c] = (unsigned long long)(sum + nrm);
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_begin(BeginArgs a)
{
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) *a.dst = a.bd;
        if (threadIdx.x == 0 && a.status) *a.status = 0;
        for (int64_t i = threadIdx.x; i < a.n_off; i += 256) a.dst_off[i] = a.off[i];
    }
    unsigned long long *t = static_cast<unsigned long long *>(a.bd.totals);
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < a.n_zero; i += (int64_t)gridDim.x * 256) t[i] = 0ull;
}

__global__ void k_fill_u64(unsigned long long *p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

// ---------------------------------------------------------------------------
// Variant table and dispatch
// ---------------------------------------------------------------------------
static const Variant kVariants[] = {
    // nt, mt, waves, buffers, qt, pl
    {1, 2, 4, 4, 32, 0},   // 0
    {2, 2, 4, 4, 32, 0},   // 1
    {2, 4, 4, 2, 32, 0},   // 2
    {2, 2, 4, 2, 32, 0},   // 3
    {2, 4, 8, 4, 32, 0},   // 4
    {2, 2, 8, 8, 32, 0},   // 5
    {1, 4, 8, 4, 32, 0},   // 6
    {2, 4, 4, 3, 32, 0},   // 7
    {2, 8, 8, 4, 32, 0},   // 8  (4 KB tiles only: INT8, FP8)
    {2, 4, 8, 8, 32, 0},   // 9  (4 KB tiles only: INT8, FP8)
    {2, 8, 8, 3, 32, 0},   // 10 (160-element INT8 rows only)
    {1, 8, 8, 3, 32, 0},   // 11 (8-bit formats: INT8 rows of 128 or 160, FP8 lists up to 40)
    {2, 8, 4, 3, 32, 0},   // 12 (FP8 lists of 64: one wave per SIMD)
    {2, 8, 8, 4, 16, 0},   // 13 (16x16 blocks, INT8 rows of 128)
    {2, 4, 8, 4, 16, 0},   // 14 (16x16 blocks, FP16 / BF16)
    {4, 8, 8, 4, 16, 0},   // 15 (16x16 blocks, INT8 rows of 128, lists up to 6)
    {2, 8, 8, 4, 32, 1},   // 16 (pair lists, 4 KB tiles: INT8, FP8 lists up to 40)
    {2, 4, 8, 4, 32, 1},   // 17 (pair lists, FP16 / BF16)
    {2, 8, 4, 3, 32, 1},   // 18 (pair lists, FP8 lists of 40 and 64: one wave per SIMD)
    {2, 8, 8, 3, 32, 1},   // 19 (pair lists, 160-element INT8 rows)
    {2, 4, 8, 4, 32, 1},   // 20 (pair lists + next-tile prefetch, FP16 / BF16)
    {2, 8, 8, 4, 32, 1},   // 21 (pair lists without next-tile prefetch: INT8, FP8)
    {2, 8, 8, 4, 32, 0},   // 22 (w8_nt2_mt8_nb4 without next-tile prefetch: INT8, FP8)
    {2, 8, 8, 2, 32, 1},   // 23 (pair lists, FP16 / BF16, 8-tile stages in two buffers)
    {2, 4, 8, 3, 32, 1},   // 24 (pair lists, FP16 / BF16, 4-tile stages three deep)
    {4, 8, 8, 4, 16, 1},   // 25 (16x16 blocks, shared lists: INT8 rows of 128, FP8 lists up to 40)
    {4, 4, 8, 4, 16, 1},   // 26 (16x16 blocks, shared lists: FP16 / BF16)
    {4, 8, 8, 4, 16, 1},   // 27 (25 without next-tile prefetch: FP8)
    {8, 8, 8, 4, 16, 1},   // 28 (25 with two halves of query tiles per wave: INT8 rows of 128, lists up to 11)
};
static const char *kVariantNames[] = {"w4_nt1_mt2_nb4", "w4_nt2_mt2_nb4", "w4_nt2_mt4_nb2", "w4_nt2_mt2_nb2",
                                      "w8_nt2_mt4_nb4", "w8_nt2_mt2_nb8", "w8_nt1_mt4_nb4", "w4_nt2_mt4_nb3",
                                      "w8_nt2_mt8_nb4", "w8_nt2_mt4_nb8", "w8_nt2_mt8_nb3", "w8_nt1_mt8_nb3",
                                      "w4_nt2_mt8_nb3", "q16_w8_nt2_mt8_nb4", "q16_w8_nt2_mt4_nb4",
                                      "q16_w8_nt4_mt8_nb4", "pl_w8_nt2_mt8_nb4", "pl_w8_nt2_mt4_nb4",
                                      "pl_w4_nt2_mt8_nb3", "pl_w8_nt2_mt8_nb3", "plpf_w8_nt2_mt4_nb4",
                                      "plnp_w8_nt2_mt8_nb4", "np_w8_nt2_mt8_nb4", "pl_w8_nt2_mt8_nb2",
                                      "pl_w8_nt2_mt4_nb3", "plq16_w8_nt4_mt8_nb4", "plq16_w8_nt4_mt4_nb4",
                                      "plq16np_w8_nt4_mt8_nb4", "plq16_w8_nt8_mt8_nb4"};
static constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

int num_variants() { return kNumVariants; }
Variant variant(int v) { return kVariants[v]; }
const char *variant_name(int v) { return (v >= 0 && v < kNumVariants) ? kVariantNames[v] : "?"; }

int kp_bucket(int kp, int fmt)
{
    if (fmt == FMT_I8N) return kp == 1 ? 1 : 0;   // one running minimum per class
    if (fmt == FMT_F16 || fmt == FMT_BF16 || fmt == FMT_I8 || fmt == FMT_I8L) {
        static const int b[] = {2, 6, 11, 16, 21, 33};
        for (int x : b)
            if (kp <= x) return x;
    } else if (fmt == FMT_FP8) {
        static const int b[] = {4, 8, 20, 40, 64};   // per-half candidate lists (>= 2k)
        for (int x : b)
            if (kp <= x) return x;
    }
    return 0;
}

bool variant_supports(int v, int fmt, int kp)
{
    if (v < 0 || v >= kNumVariants) return false;
    const int b = kp_bucket(kp, fmt);
    if (b == 0) return false;
    // 5 KB tiles (160-element INT8 rows) split evenly over the waves only
    // in these stage shapes
    if (fmt == FMT_I8L) return v == 11 || ((v == 2 || v == 7 || v == 10) && b <= 16) || (v == 19 && b <= 33);
    if (v == 10 || v == 19) return false;
    // pair lists: one list per query
    if (v == 16) return (fmt == FMT_I8 || fmt == FMT_I8N || fmt == FMT_FP8) && b <= 40;
    if (v == 17) return (fmt == FMT_F16 || fmt == FMT_BF16) && b <= 33;
    if (v == 20) return (fmt == FMT_F16 || fmt == FMT_BF16) && b <= 16;
    if (v == 21) return (fmt == FMT_FP8 && b <= 40) || fmt == FMT_I8;
    if (v == 22) return (fmt == FMT_FP8 && b <= 20) || (fmt == FMT_I8 && b <= 16);
    if (v == 23 || v == 24) return (fmt == FMT_F16 || fmt == FMT_BF16) && b <= 33;
    if (v == 25) return (fmt == FMT_I8 && b <= 33) || (fmt == FMT_FP8 && b <= 40);
    if (v == 27) return fmt == FMT_FP8 && b <= 40;
    if (v == 28) return (fmt == FMT_I8 || fmt == FMT_I8N) && b <= 11;
    if (v == 26) return (fmt == FMT_F16 || fmt == FMT_BF16) && b <= 33;
    if (v == 18) return fmt == FMT_FP8 && b > 20;
    // 16x16 output blocks: INT8 (128-element rows) and the 16-bit formats
    if (v == 13) return (fmt == FMT_I8 || fmt == FMT_I8N) && b <= 16;
    if (v == 14) return (fmt == FMT_F16 || fmt == FMT_BF16) && b <= 16;
    if (v == 15) return (fmt == FMT_I8 || fmt == FMT_I8N) && b <= 6;
    if (v == 12) return fmt == FMT_FP8 && b > 40;
    // one query tile per wave with 8-tile stages: the 4 KB-tile formats
    if (v == 11) return fmt == FMT_I8 || fmt == FMT_I8N || (fmt == FMT_FP8 && b <= 40);
    // the deep stage variants need the 4 KB tiles of the 8-bit formats
    if ((v == 8 || v == 9) && (fmt == FMT_F16 || fmt == FMT_BF16)) return false;
    // 64-entry lists take a SIMD's whole register file: one wave per SIMD
    if (fmt == FMT_FP8 && b > 40) return v == 0;
    if (fmt == FMT_FP8) return v == 0 || v == 6 || ((v == 1 || v == 4 || v == 5 || v >= 8) && b <= 20);
    return kVariants[v].nt == 1 || b <= 16;
}

// Every compiled K1 instance set: dist_kernel_<tag>_<kp>(v) returns the
// kernel of variant v, or nullptr when v is not built for that list length.
#define LNBNN_DECLARE_INSTANCE(tag, op, fmt, kp) void *dist_kernel_##tag##_##kp(int v);
LNBNN_DIST_INSTANCES(LNBNN_DECLARE_INSTANCE)
#undef LNBNN_DECLARE_INSTANCE

static void *dist_kernel(int v, int fmt, int kp)
{
    if (!variant_supports(v, fmt, kp)) return nullptr;
    const int b = kp_bucket(kp, fmt);
#define LNBNN_PICK_INSTANCE(tag, op, f, k) \
    if (fmt == f && b == k) return dist_kernel_##tag##_##k(v);
    LNBNN_DIST_INSTANCES(LNBNN_PICK_INSTANCE)
#undef LNBNN_PICK_INSTANCE
    return nullptr;
}

hipError_t launch_dist_topk(int v, int fmt, int kp, const DistArgs &a, int grid, hipStream_t s)
{
    void *fn = dist_kernel(v, fmt, kp);
    if (!fn) return hipErrorInvalidValue;
    DistArgs args = a;
    void *params[] = {&args};
    return hipLaunchKernel(fn, dim3(grid), dim3(kVariants[v].waves * 64), params, 0, s);
}

int dist_topk_blocks_per_cu(int v, int fmt, int kp)
{
    void *fn = dist_kernel(v, fmt, kp);
    if (!fn) return 0;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, kVariants[v].waves * 64, 0) != hipSuccess) return 0;
    return n;
}

// ---------------------------------------------------------------------------
// Host launchers of the small kernels
// ---------------------------------------------------------------------------
int grid_for(int64_t n, int block, int cap)
{
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

hipError_t launch_pack_u8(const uint8_t *refs, int64_t n_refs, int64_t n_pad, int fmt, uint4 *frag,
                          float *seed, hipStream_t s)
{
    const int64_t n_tiles = n_pad / kTileRows;
    if (fmt == FMT_F16) {
        const int64_t n_frag = n_tiles * OpF16::kSteps * 64;
        k_pack_u8<OpF16><<<grid_for(n_frag, 256, 65536), 256, 0, s>>>(refs, n_refs, n_frag, frag);
    } else if (fmt == FMT_BF16) {
        const int64_t n_frag = n_tiles * OpBF16::kSteps * 64;
        k_pack_u8<OpBF16><<<grid_for(n_frag, 256, 65536), 256, 0, s>>>(refs, n_refs, n_frag, frag);
    } else {
        return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (seed) {
        k_seed_u8<<<grid_for(n_pad, 256, 65536), 256, 0, s>>>(refs, n_refs, n_pad, seed);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_pack_i8(const uint8_t *refs, int64_t n_pad, int dim, uint4 *frag, int32_t *seed, hipStream_t s,
                          const int32_t *perm)
{
    if (dim == kDim)
        k_pack_i8<OpI8, 8><<<grid_for(n_pad * 8, 256, 65536), 256, 0, s>>>(refs, n_pad, frag, seed, perm);
    else if (dim == kDimLoc)
        k_pack_i8<OpI8L, 16><<<grid_for(n_pad * 16, 256, 65536), 256, 0, s>>>(refs, n_pad, frag, seed, perm);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_check_labels(const int32_t *labels, int64_t n, int32_t n_classes, int32_t *first_bad, hipStream_t s)
{
    k_set_i32<<<1, 1, 0, s>>>(first_bad, (int32_t)n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_check_labels<<<grid_for(n, 1024, 4096), 256, 0, s>>>(labels, (int32_t)n, n_classes, first_bad);
    return hipGetLastError();
}

hipError_t launch_parity_count(const uint8_t *par, int64_t n_refs, int32_t *block_odd, hipStream_t s)
{
    const int64_t n_blocks = (n_refs + 255) / 256;
    k_parity_blocks<<<(unsigned)n_blocks, 256, 0, s>>>(par, n_refs, block_odd);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_prefix<<<1, 1024, 0, s>>>(block_odd, n_blocks);
    return hipGetLastError();
}

hipError_t launch_parity_perm(const uint8_t *par, int64_t n_refs, const int32_t *block_odd, int64_t even_pad,
                              int64_t n_pad, int32_t *perm, hipStream_t s)
{
    const int64_t n_blocks = (n_refs + 255) / 256;
    k_parity_perm<<<(unsigned)n_blocks, 256, 0, s>>>(par, n_refs, n_blocks, block_odd, even_pad, n_pad, perm);
    return hipGetLastError();
}

hipError_t launch_begin(const BeginArgs &a, hipStream_t s)
{
    k_begin<<<grid_for(a.n_zero, 256, 1024), 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, int64_t n, hipStream_t s)
{
    k_fill_u64<<<grid_for(n, 256, 4096), 256, 0, s>>>(p, n);
    return hipGetLastError();
}

hipError_t launch_finish(const FinishArgs &a, int64_t q_cap, hipStream_t s)
{
    k_finish<<<grid_for(q_cap, 256, 16384), 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_argmin(const BatchDesc *bd, int64_t img_cap, int32_t n_classes, hipStream_t s)
{
    k_argmin<<<grid_for(img_cap, 4, 16384), 256, 0, s>>>(bd, n_classes);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, int64_t stride, int64_t rows, const BatchDesc *bd,
                           hipStream_t s)
{
    dim3 grid(grid_for(n, 256, 1024), (unsigned)std::min<int64_t>(std::max<int64_t>(rows, 1), 1024));
    k_fill_i32<<<grid, 256, 0, s>>>(p, v, stride, rows, bd);
    return hipGetLastError();
}

hipError_t launch_nbnn_totals(const NbnnArgs &a, int64_t img_cap, hipStream_t s)
{
    const int64_t groups = (a.n_classes + kTotalsClasses - 1) / kTotalsClasses;
    k_nbnn_totals<<<grid_for(img_cap * groups, 1, 16384), 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_row_parity(const uint8_t *refs, int64_t n_refs, int dim, uint8_t *out, hipStream_t s)
{
    k_row_parity<<<grid_for(n_refs * 16, 256, 65536), 256, 0, s>>>(refs, n_refs, dim, out);
    return hipGetLastError();
}

}  // namespace lnbnn
