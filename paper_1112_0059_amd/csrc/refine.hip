// Second half of the shared-list search: from each query's best tiles (the
// lists k_dist_topk leaves) to its best rows.
//
//   k_refine<Op>      per query (one wave): merge of the query's partial lists
//                     of (key, tile), recomputation of the rows of the k + 1
//                     best tiles on the matrix cores, the k + 1 best rows by
//                     (key, row), and Algorithm 2's class updates
//   k_refine<OpFP8>   the same up to the FP8 candidates (the 4k best rows), for
//                     the exact re-rank in rerank.hip
//
// The tiles are recomputed with the instruction and the operand order of the
// 32x32 distance kernels, so an FP8 key has the same bits there and here; the
// keys of the exact formats are exact integers anyway.
//
// What bounds it: reading n_need tiles (4-8 KB each) per query, mostly from L2
// and the infinity cache.  The 63 other columns of each output block are
// wasted, which costs nothing next to the reads.  Two tiles are computed per
// step, so that their 64 rows fill the 64 lanes, one row each.
#include "dist_topk.h"
#include "wave_select.h"

namespace lnbnn {

// One tile's accumulators with the query in every column.
template <class Op>
static __device__ __forceinline__ typename Op::acc_t tile_values(const RefineArgs &r, int64_t tile,
                                                                 const uint4 (&b)[Op::kSteps][Op::kBU], int sb, int lane,
                                                                 int h)
{
    TileRegs<Op> t;
    tile_load<Op>(r.frag + tile * (Op::kSteps * Op::kAU * 64), reinterpret_cast<const float4 *>(r.seed) + tile * 8,
                  r.row_scale + (Op::kScaled ? tile * kTileRows : 0), lane, h, t);
    typename Op::acc_t acc = __builtin_bit_cast(typename Op::acc_t, t.sd);
#pragma unroll
    for (int s = 0; s < Op::kSteps; ++s) acc = Op::mma(t.av[s], b[s], acc, t.sa, sb);
    return acc;
}

// The query's partial lists: slots slot0 .. slot0 + n_lists - 1 (see the walk
// of k_dist_topk: whole blocks have one, a remaining block one per slice or
// run piece).
static __device__ __forceinline__ int query_slots(const SlotMap &m, const Walk &w, int64_t q, int64_t *slot0)
{
    const int64_t blk = q / m.block, first_rem = (int64_t)w.full_rounds * m.grid;
    if (blk < first_rem) {
        *slot0 = blk;
        return 1;
    }
    const int64_t b = blk - first_rem;
    if (w.rem_slices > 0) {
        *slot0 = first_rem + b * w.rem_slices;
        return w.rem_slices;
    }
    const int64_t w0 = b * m.n_tiles / w.slice_tiles, w1 = ((b + 1) * m.n_tiles - 1) / w.slice_tiles;
    *slot0 = first_rem + b + w0;
    return (int)(w1 - w0 + 1);
}

// Image of query q (wave-uniform): the last m with offsets[m] <= q, 64 probes at
// a time.
static __device__ __forceinline__ int64_t image_of(const int64_t *offsets, int64_t n_img, int64_t q, int lane)
{
    int64_t lo = 0, hi = n_img;
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + 63) >> 6, m = lo + lane * step;
        const bool le = m < hi && offsets[m] <= q;
        const int c = (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(le));
        lo += (c > 0 ? c - 1 : 0) * step;
        hi = min(hi, lo + step);
    }
    return lo;
}

// Selects the query's best rows into sel.buf (sorted, sel.n of them).
template <class Op, int CAP>
static __device__ __forceinline__ void best_rows(const RefineArgs &r, const float *part_d, const int32_t *part_i, int kp,
                                                 const Walk &walk, int64_t q, const void *q_src, WaveSelect<CAP> &sel,
                                                 int *tiles, int32_t *status, int lane)
{
    const int h = lane >> 5;
    int64_t slot0;
    const int nl = query_slots(r.map, walk, q, &slot0);
    const int64_t ql = q % r.map.block;
    const int need_rows = sel.need;
    // the n_need best tiles by (key, tile)
    int n_tiles = 0;
    float tau = __builtin_inff();
    bool marked = false;            // a list's last key is NaN: its stage wait gave up
    for (int l = lane; l < nl; l += 64) marked |= __builtin_isnan(part_d[((slot0 + l) * r.map.block + ql) * kp + kp - 1]);
    if (__builtin_amdgcn_ballot_w64(marked) != 0 && lane == 0) atomicOr(status, kStatusWaitGaveUp);
    if (nl == 1) {
        const int64_t base = (slot0 * r.map.block + ql) * kp;
        const bool in = lane < r.n_need;
        const int t = in ? part_i[base + lane] : -1;
        if (in) tau = part_d[base + lane];
        n_tiles = (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(t >= 0));
        if (t >= 0) tiles[lane] = t;
        tau = __shfl(tau, r.n_need - 1);
        wave_lds_fence();
    } else {
        // lists are sorted: rank by rank over all of them, until a rank adds nothing
        sel.need = r.n_need;
        for (int p = 0; p < r.n_need; ++p) {
            bool more = false;
            for (int l0 = 0; l0 < nl; l0 += 64) {
                const int l = l0 + lane;
                const int64_t o = ((slot0 + min(l, nl - 1)) * r.map.block + ql) * kp + p;
                const int t = part_i[o];
                more |= sel.add(part_d[o], t, l < nl && t >= 0, lane);
            }
            if (!more) break;
        }
        sel.cut(lane);
        n_tiles = sel.n;
        if (lane < n_tiles) tiles[lane] = (int)sel.buf[lane].y;
        if (n_tiles == r.n_need) tau = __builtin_bit_cast(float, sel.buf[n_tiles - 1].x);
        wave_lds_fence();
    }
    // their rows: n_need tiles hold a row of key <= tau each, so if no more rows
    // than that are needed, no row above tau is
    sel = WaveSelect<CAP>(sel.buf, need_rows,
                          n_tiles == r.n_need && need_rows <= r.n_need && !__builtin_isnan(tau) ? tau : __builtin_inff());
    uint4 b[Op::kSteps][Op::kBU];
    int sb;
    Op::load_b(q_src, r.q_scale, q, true, h, b, sb);
    for (int t = 0; t < n_tiles; t += 2) {
        const int ta = __builtin_amdgcn_readfirstlane(tiles[t]);
        const int tb = __builtin_amdgcn_readfirstlane(tiles[min(t + 1, n_tiles - 1)]);
        const typename Op::acc_t va = tile_values<Op>(r, ta, b, sb, lane, h);
        const typename Op::acc_t vb = tile_values<Op>(r, tb, b, sb, lane, h);
        // lane c + 16 j + 32 h takes register c of tile j
        const int c = lane & 15;
        const bool second = lane & 16;
        typename Op::gate_t v = va[0];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const typename Op::gate_t x = second ? vb[i] : va[i];
            v = c == i ? x : v;
        }
        const int tile = second ? tb : ta;
        const int row = tile * kTileRows + 8 * (c >> 2) + 4 * h + (c & 3);
        const bool real = Op::kParity ? v < (typename Op::gate_t)(1 << 29) : (float)v < __builtin_inff();
        sel.add(Op::tile_key(v, Op::kParity && tile >= r.odd_tile0), row, real && (!second || t + 1 < n_tiles), lane);
    }
    sel.cut(lane);
}

// Exact formats: neighbours, background distance and class updates of one query
// per wave.  Exact integers are added with 64-bit atomics, so totals do not
// depend on the order of the atomics.
template <class Op>
__global__ __launch_bounds__(256) void k_refine(RefineArgs r, FinishArgs a)
{
    constexpr int CAP = 128;        // kMaxKP + 64 or more
    __shared__ uint2 s_sel[4][CAP];
    __shared__ int s_tiles[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n_q = a.bd->n_q, n_img = a.bd->n_img;
    const Walk walk = a.bd->walk;
    const int kp = a.k + 1;
    int32_t *nbr_idx = a.bd->nbr_idx;
    float *nbr_dist = a.bd->nbr_dist;
    // Neighbouring queries belong to the same image: with few classes their
    // atomics all go to the same totals and wait for each other, so workgroups
    // take groups of four queries from `spread` distant parts of the batch in
    // turn (two classes, 144,000 descriptors: 1.15 -> 0.82 ms).  With many
    // classes the totals are many, and neighbours, which share tiles, are better
    // kept together (256 classes, 288,000 descriptors: 1.96 ms, spread 2.59 ms).
    const int64_t spread = max(1, 64 / a.n_classes);
    const int64_t part = ((n_q + 3) / 4 + spread - 1) / spread;
    for (int64_t u = blockIdx.x; u < part * spread; u += gridDim.x) {
        const int64_t q = ((u % spread) * part + u / spread) * 4 + __builtin_amdgcn_readfirstlane(wave);
        if (q >= n_q) continue;
        WaveSelect<CAP> sel(s_sel[wave], kp, __builtin_inff());
        best_rows<Op, CAP>(r, a.part_d, a.part_i, a.kp_stride, walk, q, a.bd->q, sel, s_tiles[wave], a.status, lane);
        // rank `lane` of the list; fewer than k + 1 rows only after a stage wait gave up
        const bool have = lane < sel.n && lane < kp;
        const uint2 e = sel.buf[have ? lane : 0];
        const float key = __builtin_bit_cast(float, e.x);
        int idx = -1;
        if (have) idx = a.perm ? a.perm[e.y] : (int)e.y;
        const int lab = lane < a.k && idx >= 0 ? a.labels[idx] : -1;
        const int db = __shfl((int)key, a.k);
        bool first = lab >= 0;
        for (int j = 0; j < a.k; ++j) {
            const int before = __builtin_amdgcn_readlane(lab, j);
            if (j < lane && before == lab) first = false;
        }
        const int64_t img = image_of(a.offsets, n_img, q, lane);
        if (first && sel.n == kp)
            atomicAdd(a.totals + img * a.n_classes + lab, (unsigned long long)(long long)((int)key - db));
        if (nbr_idx) {
            // ||q - shift||^2 turns the key back into the squared distance
            uint32_t qq = 0;
            if (lane * 4 < a.dim) {
                const uint32_t w = reinterpret_cast<const uint32_t *>(static_cast<const uint8_t *>(a.bd->q) + q * a.dim)[lane];
                for (int i = 0; i < 4; ++i) {
                    const int32_t x = (int32_t)((w >> (8 * i)) & 0xffu) - a.q_shift;
                    qq += (uint32_t)(x * x);
                }
            }
            for (int o = 32; o > 0; o >>= 1) qq += __shfl_xor(qq, o);
            if (lane < kp) {
                nbr_idx[q * kp + lane] = idx;
                nbr_dist[q * kp + lane] = have ? key + (float)qq : __builtin_inff();
            }
        }
        wave_lds_fence();
    }
}

// FP8: the n_cand best rows by (key, row), one query per wave.
__global__ __launch_bounds__(256) void k_refine_fp8(RefineArgs r, RerankArgs a)
{
    constexpr int CAP = 192;        // 4 * 32 candidates + 64
    __shared__ uint2 s_sel[4][CAP];
    __shared__ int s_tiles[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n_q = a.bd->n_q;
    const Walk walk = a.bd->walk;
    for (int64_t q = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(wave); q < n_q; q += (int64_t)gridDim.x * 4) {
        WaveSelect<CAP> sel(s_sel[wave], a.n_cand, __builtin_inff());
        best_rows<OpFP8, CAP>(r, a.part_d, a.part_i, a.kp_stride, walk, q, r.q, sel, s_tiles[wave], a.status, lane);
        for (int j = lane; j < a.n_cand; j += 64) a.cand[q * a.n_cand + j] = j < sel.n ? (int)sel.buf[j].y : -1;
        wave_lds_fence();
    }
}

hipError_t launch_refine(int fmt, const RefineArgs &r, const FinishArgs &a, int64_t q_cap, hipStream_t s)
{
    const int grid = grid_for(q_cap, 4, 65536);
    switch (fmt) {
    case FMT_F16: k_refine<OpF16><<<grid, 256, 0, s>>>(r, a); break;
    case FMT_BF16: k_refine<OpBF16><<<grid, 256, 0, s>>>(r, a); break;
    case FMT_I8: k_refine<OpI8><<<grid, 256, 0, s>>>(r, a); break;
    case FMT_I8L: k_refine<OpI8L><<<grid, 256, 0, s>>>(r, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_refine_fp8(const RefineArgs &r, const RerankArgs &a, int64_t q_cap, hipStream_t s)
{
    k_refine_fp8<<<grid_for(q_cap, 4, 65536), 256, 0, s>>>(r, a);
    return hipGetLastError();
}

}  // namespace lnbnn
