// Second half of the shared-list search: from each query's best tiles (the
// lists k_dist_topk leaves) to its best rows.
//
//   k_refine<Op>      per query (one wave): merge of the query's partial lists
//                     of (key, tile), recomputation of the rows of the k + 1
//                     best tiles, the k + 1 best rows by (key, row), and
//                     Algorithm 2's class updates
//   k_refine_fp8<Op>  the same up to the FP8 candidates (the 4k best rows), for
//                     the exact re-rank in rerank.hip
//
// A wave recomputes two tiles per step, one row per lane.  INT8 and 16-bit rows
// are dotted with the query on the vector units (v_dot4 / v_dot2; the query sits
// in scalar registers): their keys are exact integers in any order.  An FP8 key
// must have the bits the distance kernel gave it, so it comes from that kernel's
// instruction and operand order, with the query in every column of the block.
//
// What bounds it: reading n_need tiles (4-8 KB each) per query from L2 and the
// infinity cache, and the instructions of the selection.
#include "dist_topk.h"
#include "wave_select.h"

namespace lnbnn {

// The query as the row arithmetic of its format wants it, and one row's key
// part per lane: rows() takes two tiles, lane l row row_in(l) of the first one
// or, where second(l), of the second.
template <class Op>
struct RowDot;

// one row per lane: lanes 0-31 the first tile
struct RowPerLane {
    static __device__ __forceinline__ bool second(int lane) { return lane & 32; }
    static __device__ __forceinline__ int row_in(int lane) { return lane & 31; }
};

// The N dwords of a query (a wave-uniform address) into scalar registers.  A
// scalar load drops the two low bits of its address, and a caller's u8 rows may
// start at any byte: such a query is loaded one dword per lane and read lane by
// lane.
template <int N>
static __device__ __forceinline__ void load_query(const uint8_t *p, int lane, uint32_t (&w)[N])
{
    static_assert(N <= 64, "one dword per lane");
    if (((uintptr_t)p & 3) == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = load_uniform(reinterpret_cast<const uint32_t *>(p), i);
    } else {
        uint32_t x = 0;
        if (lane < N) __builtin_memcpy(&x, p + 4 * lane, 4);
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = (uint32_t)__builtin_amdgcn_readlane((int)x, i);
    }
}

// INT8: D = seed + sum of s * u in 32-bit integers, u = 127 - q as in load_b.
template <int S, int FMT>
struct RowDot<OpI8T<S, FMT>> : RowPerLane {
    using Op = OpI8T<S, FMT>;
    uint32_t u[8 * S];
    __device__ __forceinline__ RowDot(const RefineArgs &, const void *q_src, int64_t q, int lane)
    {
        load_query(static_cast<const uint8_t *>(q_src) + q * Op::kRow, lane, u);
#pragma unroll
        for (int i = 0; i < 8 * S; ++i) u[i] ^= 0x7f7f7f7fu;
    }
    __device__ __forceinline__ int rows(const RefineArgs &r, int ta, int tb, int lane, int *row) const
    {
        const int tile = second(lane) ? tb : ta;
        *row = tile * kTileRows + row_in(lane);
        const uint4 *f = r.frag + (int64_t)tile * (S * 64) + (lane & 31);
        uint4 v[2 * S];
#pragma unroll
        for (int c = 0; c < 2 * S; ++c) v[c] = f[(c >> 1) * 64 + 32 * (c & 1)];
        int d = reinterpret_cast<const int32_t *>(r.seed)[*row];
#pragma unroll
        for (int c = 0; c < 2 * S; ++c) {
            d = __builtin_amdgcn_sdot4((int)v[c].x, (int)u[4 * c + 0], d, false);
            d = __builtin_amdgcn_sdot4((int)v[c].y, (int)u[4 * c + 1], d, false);
            d = __builtin_amdgcn_sdot4((int)v[c].z, (int)u[4 * c + 2], d, false);
            d = __builtin_amdgcn_sdot4((int)v[c].w, (int)u[4 * c + 3], d, false);
        }
        return d;
    }
};

// 16-bit formats: d' = seed + sum of r * (-2 q) in FP32, exact integers.
template <class O>
struct RowDot16 : RowPerLane {
    uint32_t u[64];                 // pairs of -2 q in the operand format
    // Sixteen lanes convert eight elements each and the pairs are read lane by
    // lane.  Converted from scalar registers, by every lane alike, the 128
    // elements were most of a query's instructions: 128,000 descriptors against
    // 300 references, k = 1, 223 us then and 175 now.
    __device__ __forceinline__ RowDot16(const RefineArgs &, const void *q_src, int64_t q, int lane)
    {
        uint2 raw;
        __builtin_memcpy(&raw, static_cast<const uint8_t *>(q_src) + q * kDim + 8 * (lane & 15), 8);
        const uint4 w = O::cvt8(raw, -2.0f);
        const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int i = 0; i < 64; ++i) u[i] = (uint32_t)__builtin_amdgcn_readlane((int)x[i & 3], i >> 2);
    }
    static __device__ __forceinline__ float dot2(uint32_t x, uint32_t y, float c)
    {
        if constexpr (O::kFmt == FMT_F16) {
            typedef _Float16 h2 __attribute__((ext_vector_type(2)));
            return __builtin_amdgcn_fdot2(__builtin_bit_cast(h2, x), __builtin_bit_cast(h2, y), c, false);
        } else {
            typedef __bf16 b2 __attribute__((ext_vector_type(2)));
            return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b2, x), __builtin_bit_cast(b2, y), c, false);
        }
    }
    __device__ __forceinline__ float rows(const RefineArgs &r, int ta, int tb, int lane, int *row) const
    {
        const int tile = second(lane) ? tb : ta;
        *row = tile * kTileRows + row_in(lane);
        const uint4 *f = r.frag + (int64_t)tile * (8 * 64) + (lane & 31);
        float d = r.seed[*row];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint4 v[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = f[(4 * half + (c >> 1)) * 64 + 32 * (c & 1)];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                d = dot2(v[c].x, u[4 * (8 * half + c) + 0], d);
                d = dot2(v[c].y, u[4 * (8 * half + c) + 1], d);
                d = dot2(v[c].z, u[4 * (8 * half + c) + 2], d);
                d = dot2(v[c].w, u[4 * (8 * half + c) + 3], d);
            }
        }
        return d;
    }
};
template <> struct RowDot<OpF16> : RowDot16<OpF16> { using RowDot16<OpF16>::RowDot16; };
template <> struct RowDot<OpBF16> : RowDot16<OpBF16> { using RowDot16<OpBF16>::RowDot16; };

// FP8: the block instruction of the distance kernel that made the lists, with
// the query in every column.  The two block shapes sum in different orders
// (two chained sums of 64 products, or one of 128) and their keys may differ in
// the last place; a listed key bounds the rows' keys only where both come
// from one of them.
template <class Op>
struct RowDotFP8 {
    static constexpr int kAcc = Op::kAccN;          // a lane's registers of a tile
    uint4 b[Op::kSteps][Op::kBU];
    int sb;
    __device__ __forceinline__ RowDotFP8(const RefineArgs &r, const void *q_src, int64_t q, int lane)
    {
        Op::load_b(q_src, r.q_scale, q, true, lane / Op::kQT, b, sb);
    }
    __device__ __forceinline__ typename Op::acc_t block(const RefineArgs &r, int64_t tile, int lane) const
    {
        TileRegs<Op> t;
        tile_load<Op>(r.frag + tile * (Op::kSteps * Op::kAU * 64), reinterpret_cast<const float4 *>(r.seed) + tile * 8,
                      r.row_scale + tile * kTileRows, lane, lane / Op::kQT, t);
        typename Op::acc_t acc = t.sd;
#pragma unroll
        for (int s = 0; s < Op::kSteps; ++s) acc = Op::mma(t.av[s], b[s], acc, t.sa, sb);
        return acc;
    }
    // lane c + kAcc j + kQT h takes register c of tile j
    static __device__ __forceinline__ bool second(int lane) { return lane & kAcc; }
    static __device__ __forceinline__ int row_in(int lane)
    {
        const int c = lane & (kAcc - 1);
        return Op::kRowStride * (c >> 2) + 4 * (lane / Op::kQT) + (c & 3);
    }
    __device__ __forceinline__ float rows(const RefineArgs &r, int ta, int tb, int lane, int *row) const
    {
        const typename Op::acc_t va = block(r, ta, lane), vb = block(r, tb, lane);
        const int c = lane & (kAcc - 1);
        float v = va[0];
#pragma unroll
        for (int i = 0; i < kAcc; ++i) {
            const float x = second(lane) ? vb[i] : va[i];
            v = c == i ? x : v;
        }
        *row = (second(lane) ? tb : ta) * kTileRows + row_in(lane);
        return v;
    }
};
template <> struct RowDot<OpFP8> : RowDotFP8<OpFP8> { using RowDotFP8<OpFP8>::RowDotFP8; };
template <> struct RowDot<OpFP8Q> : RowDotFP8<OpFP8Q> { using RowDotFP8<OpFP8Q>::RowDotFP8; };

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
                                                 int *tiles, float *keys, int32_t *status, int lane)
{
    int64_t slot0;
    const int nl = query_slots(r.map, walk, q, &slot0);
    const int64_t ql = q % r.map.block;
    const int need_rows = sel.need;
    // the n_need best tiles by (key, tile)
    int n_tiles = 0;
    float tau = __builtin_inff();
    bool marked = false;            // a list's last key is NaN: its stage wait gave up
    for (int l = lane; l < nl; l += 64) marked |= __builtin_isnan(part_d[((slot0 + l) * r.map.block + ql) * kp + kp - 1]);
    if (__builtin_amdgcn_ballot_w64(marked) != 0 && lane == 0) *status = kStatusWaitGaveUp;
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
                more |= sel.add(pair_of(part_d[o], t), l < nl && t >= 0, lane);
            }
            if (!more) break;
            if (p == 0 && sel.n >= sel.need) sel.cut(lane);   // a bound for the other ranks
        }
        sel.cut(lane);
        n_tiles = sel.n;
        if (lane < n_tiles) tiles[lane] = pair_index(sel.buf[lane]);
        if (n_tiles == r.n_need) tau = pair_key(sel.buf[n_tiles - 1]);
        wave_lds_fence();
    }
    // their rows: n_need tiles hold a row of key <= tau each, so if no more rows
    // than that are needed, no row above tau is
    const bool bounded = n_tiles == r.n_need && need_rows <= r.n_need && !__builtin_isnan(tau);
    sel = WaveSelect<CAP>(sel.buf, need_rows, bounded ? pair_of(tau, 0x7fffffff) : ~0ull);
    const RowDot<Op> dot(r, q_src, q, lane);
    // the 64 rows of tiles t and t + 1, one per lane; +inf where there is none
    auto rows = [&](int t, int *row) -> float {
        const int ta = __builtin_amdgcn_readfirstlane(tiles[t]);
        const int tb = __builtin_amdgcn_readfirstlane(tiles[min(t + 1, n_tiles - 1)]);
        const typename Op::gate_t v = dot.rows(r, ta, tb, lane, row);
        const bool second = RowDot<Op>::second(lane);
        const int par = Op::kParity && (second ? tb : ta) >= r.odd_tile0;
        const bool real = Op::kParity ? v < (typename Op::gate_t)(1 << 29) : (float)v < __builtin_inff();
        return real && (!second || t + 1 < n_tiles) ? Op::tile_key(v, par) : __builtin_inff();
    };
    if (!bounded && n_tiles > 4 && need_rows <= 48) {
        // A small index (fewer tiles than needed) gives no bound, and then every
        // row would go through the buffer.  The need-th smallest of the 64
        // lanes' smallest keys bounds the rows' (64 groups of rows, each with a
        // row no larger).
        float low = __builtin_inff();
        for (int t = 0; t < n_tiles; t += 2) {
            int row;
            const float key = rows(t, &row);
            keys[t * 32 + lane] = key;
            low = __builtin_fminf(low, key);
        }
        sel.add(pair_of(low, lane), low < __builtin_inff(), lane);
        sel.cut(lane);
        sel = WaveSelect<CAP>(sel.buf, need_rows, sel.bound == ~0ull ? ~0ull : pair_of(pair_key(sel.bound), 0x7fffffff));
        wave_lds_fence();
        for (int t = 0; t < n_tiles; t += 2) {
            const float key = keys[t * 32 + lane];
            const int tile = tiles[min(t + (RowDot<Op>::second(lane) ? 1 : 0), n_tiles - 1)];
            sel.add(pair_of(key, tile * kTileRows + RowDot<Op>::row_in(lane)), key < __builtin_inff(), lane);
        }
    } else {
        for (int t = 0; t < n_tiles; t += 2) {
            int row;
            const float key = rows(t, &row);
            sel.add(pair_of(key, row), key < __builtin_inff(), lane);
        }
    }
    sel.cut(lane);
}

// Exact formats: neighbours, background distance and class updates, one query
// at a time per wave.  Exact integers are added, so totals do not depend on the
// order of the additions.
//
// Neighbouring queries belong to the same image, so with one atomic per update
// they wait for each other at the same few totals: 144,000 descriptors of two
// classes took 1.15 ms, 0.82 ms with the queries dealt from distant images.  So
// where a wave has several queries (n_run consecutive ones) and the classes fit
// its LDS table, it sums an image's updates there and adds the sums when the
// image ends.
constexpr int kTableClasses = 256;

template <class Op>
__global__ __launch_bounds__(256) void k_refine(RefineArgs r, FinishArgs a)
{
    constexpr int CAP = 128;        // kMaxKP + 64 or more
    __shared__ uint64_t s_sel[4][WaveSelect<CAP>::kSize];
    __shared__ int s_tiles[4][64];
    __shared__ float s_keys[4][34 * kTileRows];
    __shared__ long long s_table[4][kTableClasses];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n_q = a.bd->n_q, n_img = a.bd->n_img;
    const Walk walk = a.bd->walk;
    const int kp = a.k + 1;
    unsigned long long *totals = static_cast<unsigned long long *>(a.bd->totals);
    int32_t *nbr_idx = a.bd->nbr_idx;
    float *nbr_dist = a.bd->nbr_dist;
    const int64_t n_waves = (int64_t)gridDim.x * 4;
    const int64_t n_run = (n_q + n_waves - 1) / n_waves;
    const bool table = n_run > 1 && a.n_classes <= kTableClasses;
    long long *tab = s_table[wave];
    if (table)
        for (int c = lane; c < a.n_classes; c += 64) tab[c] = 0;
    int64_t img = -1, img_end = 0;  // image of the last query, and the query it ends before
    auto flush = [&]() {
        wave_lds_fence();
        for (int c = lane; c < a.n_classes; c += 64) {
            const long long v = tab[c];
            if (v != 0) atomicAdd(totals + img * a.n_classes + c, (unsigned long long)v);
            tab[c] = 0;
        }
        wave_lds_fence();
    };
    const int64_t q0 = ((int64_t)blockIdx.x * 4 + wave) * n_run, q1 = min(q0 + n_run, n_q);
    for (int64_t q = q0; q < q1; ++q) {
        WaveSelect<CAP> sel(s_sel[wave], kp, ~0ull);
        best_rows<Op, CAP>(r, a.part_d, a.part_i, a.kp_stride, walk, q, a.bd->q, sel, s_tiles[wave], s_keys[wave], a.status, lane);
        // rank `lane` of the list; fewer than k + 1 rows only after a stage wait gave up
        const bool have = lane < sel.n && lane < kp;
        const uint64_t e = sel.buf[have ? lane : 0];
        const float key = pair_key(e);
        int idx = -1;
        if (have) idx = a.perm ? a.perm[pair_index(e)] : pair_index(e);
        const int lab = lane < a.k && idx >= 0 ? a.labels[idx] : -1;
        const int db = __shfl((int)key, a.k);
        bool first = lab >= 0 && sel.n == kp;
        for (int j = 0; j < a.k; ++j) {
            const int before = __builtin_amdgcn_readlane(lab, j);
            if (j < lane && before == lab) first = false;
        }
        if (q >= img_end) {
            if (table && img >= 0) flush();
            img = image_of(a.offsets, n_img, q, lane);
            img_end = a.offsets[img + 1];
        }
        const long long delta = (int)key - db;
        // the updates of one query are of different classes
        if (first && table) tab[lab] += delta;
        if (first && !table) atomicAdd(totals + img * a.n_classes + lab, (unsigned long long)delta);
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
    if (table && img >= 0) flush();
}

// FP8: the n_cand best rows by (key, row), one query per wave.  Op: the block
// shape of the lists.
template <class Op>
__global__ __launch_bounds__(256) void k_refine_fp8(RefineArgs r, RerankArgs a)
{
    constexpr int CAP = 192;        // 4 * 32 candidates + 64
    __shared__ uint64_t s_sel[4][WaveSelect<CAP>::kSize];
    __shared__ int s_tiles[4][64];
    __shared__ float s_keys[4][48 * kTileRows];     // lists of up to 48 tiles (k <= 12) take the bounded pass
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n_q = a.bd->n_q;
    const Walk walk = a.bd->walk;
    for (int64_t q = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(wave); q < n_q; q += (int64_t)gridDim.x * 4) {
        WaveSelect<CAP> sel(s_sel[wave], a.n_cand, ~0ull);
        best_rows<Op, CAP>(r, a.part_d, a.part_i, a.kp_stride, walk, q, r.q, sel, s_tiles[wave], s_keys[wave], a.status, lane);
        for (int j = lane; j < a.n_cand; j += 64) a.cand[q * a.n_cand + j] = j < sel.n ? pair_index(sel.buf[j]) : -1;
        wave_lds_fence();
    }
}

hipError_t launch_refine(int fmt, const RefineArgs &r, const FinishArgs &a, int64_t q_cap, hipStream_t s)
{
    // One query per wave up to 2,048 (nothing gains on the shortest path there),
    // then at least four, on at most 2,048 workgroups.  30 KB of LDS let five of
    // them run on a CU, so that is a round and a half.  Two-class sweep, 144,000
    // descriptors, this kernel alone: 776 us, one round of 1,280 850, four rounds
    // of shorter runs 723; but beside other indexes' sweeps those four rounds
    // cost the call 2.45 ms against 2.25.
    const int grid = grid_for(q_cap, q_cap <= 2048 ? 4 : 16, 2048);
    switch (fmt) {
    case FMT_F16: k_refine<OpF16><<<grid, 256, 0, s>>>(r, a); break;
    case FMT_BF16: k_refine<OpBF16><<<grid, 256, 0, s>>>(r, a); break;
    case FMT_I8: k_refine<OpI8><<<grid, 256, 0, s>>>(r, a); break;
    case FMT_I8L: k_refine<OpI8L><<<grid, 256, 0, s>>>(r, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_refine_fp8(int qt, const RefineArgs &r, const RerankArgs &a, int64_t q_cap, hipStream_t s)
{
    const int grid = grid_for(q_cap, 4, 65536);
    if (qt == 16)
        k_refine_fp8<OpFP8Q><<<grid, 256, 0, s>>>(r, a);
    else
        k_refine_fp8<OpFP8><<<grid, 256, 0, s>>>(r, a);
    return hipGetLastError();
}

}  // namespace lnbnn
