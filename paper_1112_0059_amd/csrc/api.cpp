// C ABI of the local NBNN library: index residency, batch planning, the
// launch sequence (direct or replayed from a hipGraph), timing and the
// project autotuner.  See include/lnbnn.h for the contract of every entry
// point.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <sstream>

#include "runtime.h"

using namespace lnbnn;

namespace lnbnn {

static thread_local std::string g_err;

int set_err(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

int hip_err(hipError_t e, const char *what)
{
    if (e == hipErrorOutOfMemory) return set_err(LNBNN_ENOMEM, "%s: %s", what, hipGetErrorString(e));
    return set_err(LNBNN_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

// LNBNN_FAULT=alloc|launch makes the named site fail with LNBNN_EDEVICE, so
// error paths can be exercised without breaking the device.
bool fault_injected(const char *site)
{
    const char *f = getenv("LNBNN_FAULT");
    return f && strcmp(f, site) == 0;
}

// LNBNN_LOG=1: one line on stderr per notable event.
bool log_enabled()
{
    const char *e = getenv("LNBNN_LOG");
    return e && *e && strcmp(e, "0") != 0;
}

void log_line(const char *fmt, ...)
{
    if (!log_enabled()) return;
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    fprintf(stderr, "[lnbnn] %s\n", buf);
}

// LNBNN_HBM_BUDGET: bytes, with an optional K / M / G suffix; 0 when unset
// or malformed.
static int64_t env_budget()
{
    const char *e = getenv("LNBNN_HBM_BUDGET");
    if (!e || !*e) return 0;
    char *end = nullptr;
    const double v = strtod(e, &end);
    if (end == e || !(v > 0)) return 0;
    double mul = 1;
    if (*end == 'K' || *end == 'k') mul = 1024.0;
    else if (*end == 'M' || *end == 'm') mul = 1024.0 * 1024;
    else if (*end == 'G' || *end == 'g') mul = 1024.0 * 1024 * 1024;
    else if (*end) return 0;
    return (int64_t)(v * mul);
}

static std::mutex g_stream_mu;
static std::map<int, std::vector<hipStream_t>> g_streams;   // device -> streams no index holds

int stream_acquire(int device, hipStream_t *out)
{
    {
        std::lock_guard<std::mutex> lock(g_stream_mu);
        auto &v = g_streams[device];
        if (!v.empty()) {
            *out = v.back();
            v.pop_back();
            return LNBNN_OK;
        }
    }
    // a blocking stream stays ordered after work on the NULL stream
    LN_HIP(hipStreamCreate(out));
    return LNBNN_OK;
}

void stream_release(int device, hipStream_t s)
{
    std::lock_guard<std::mutex> lock(g_stream_mu);
    g_streams[device].push_back(s);
}

struct KeptBlock {
    int device;
    void *p;
    size_t bytes;
};
static std::mutex g_kept_mu;
static std::vector<KeptBlock> g_kept;                       // oldest first
static size_t g_kept_bytes = 0;
static std::unordered_map<void *, KeptBlock> g_given;       // buffers in use
static thread_local bool t_keep_frees = true;               // false: this thread's dfree goes to the driver

static void drop_kept_locked(size_t down_to)
{
    size_t n = 0;
    while (n < g_kept.size() && g_kept_bytes > down_to) {
        (void)hipFree(g_kept[n].p);
        g_kept_bytes -= g_kept[n++].bytes;
    }
    g_kept.erase(g_kept.begin(), g_kept.begin() + n);
}

static hipError_t dmalloc(void **p, size_t bytes)
{
    if (fault_injected("alloc")) return hipErrorOutOfMemory;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(g_kept_mu);
    // the smallest kept block that fits and is no larger by more than a page:
    // what callers account for is what they asked for
    size_t best = g_kept.size();
    for (size_t i = 0; i < g_kept.size(); ++i)
        if (g_kept[i].device == dev && g_kept[i].bytes >= bytes && g_kept[i].bytes <= bytes + 4096 &&
            (best == g_kept.size() || g_kept[i].bytes < g_kept[best].bytes))
            best = i;
    if (best < g_kept.size()) {
        *p = g_kept[best].p;
        g_kept_bytes -= g_kept[best].bytes;
        g_given[*p] = g_kept[best];
        g_kept.erase(g_kept.begin() + best);
        return hipSuccess;
    }
    e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && !g_kept.empty()) {
        (void)hipGetLastError();
        drop_kept_locked(0);
        e = hipMalloc(p, bytes);
    }
    if (e == hipSuccess) g_given[*p] = KeptBlock{dev, *p, bytes};
    return e;
}

void dfree(void *p)
{
    if (!p) return;
    std::lock_guard<std::mutex> lock(g_kept_mu);
    auto it = g_given.find(p);
    if (it == g_given.end() || !t_keep_frees) {
        if (it != g_given.end()) g_given.erase(it);
        (void)hipFree(p);
        return;
    }
    g_kept.push_back(it->second);
    g_kept_bytes += it->second.bytes;
    g_given.erase(it);
    drop_kept_locked(kKeptBytes);
}

// Stream-ordered allocation; the kept buffers make room for it too.
static hipError_t dmalloc_async(void **p, size_t bytes, hipStream_t s)
{
    hipError_t e = hipMallocAsync(p, bytes, s);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    {
        std::lock_guard<std::mutex> lock(g_kept_mu);
        drop_kept_locked(0);
    }
    return hipMallocAsync(p, bytes, s);
}

// Bytes kept on a device: free for the next index, though the driver counts
// them as used.
static size_t kept_bytes(int device)
{
    std::lock_guard<std::mutex> lock(g_kept_mu);
    size_t n = 0;
    for (const KeptBlock &b : g_kept) n += b.device == device ? b.bytes : 0;
    return n;
}

int64_t row_bytes(int dtype, int dim) { return dtype == LNBNN_U8 ? dim : (int64_t)dim * 4; }

int mode_fmt(int mode)
{
    switch (mode) {
    case LNBNN_EXACT_F16: return FMT_F16;
    case LNBNN_EXACT_BF16: return FMT_BF16;
    case LNBNN_FP8_RERANK: return FMT_FP8;
    case LNBNN_EXACT_I8: return FMT_I8;
    case LNBNN_FP8_RERANK_2K: return FMT_FP8;
    case LNBNN_NBNN_I8: return FMT_I8N;
    }
    return -1;
}

bool is_fp8_mode(int mode) { return mode == LNBNN_FP8_RERANK || mode == LNBNN_FP8_RERANK_2K; }

int index_fmt(const lnbnn_index *ix, int mode)
{
    const int f = mode_fmt(mode);
    return f == FMT_I8 && ix->dim == kDimLoc ? FMT_I8L : f;
}

Workspace::~Workspace()
{
    void *ps[] = {q, offsets, bd, part_d, part_i, totals, totals_f64, cls, nbr_idx, nbr_dist,
                  q8, qsc, cand, upd_cls, upd_delta};
    for (void *p : ps)
        dfree(p);
    if (h_status) (void)hipHostFree(h_status);
}

int64_t Workspace::bytes() const
{
    return qbytes_cap + (2 * img_cap + 2) * 8 + img_cap * (int64_t)sizeof(BatchDesc) + part_cap * 8 +
           nbr_cap * 8 + img_cap * 4 + q8_cap * (kDim + 4) + cand_cap * 4 + upd_cap * 12;
}

// The FP8 modes re-rank 4k candidates per query (at least k + 1), the best
// 4k FP8 keys of the union of the distance kernel's lists; lanes l and l+32
// see disjoint halves of every reference tile and keep separate lists.
// LNBNN_FP8_RERANK keeps 4k keys per half (up to the 64-entry lists, k <=
// 16), so the union holds the FP8 top 4k and the candidates are exactly
// them, whatever the launch plan.  LNBNN_FP8_RERANK_2K keeps 2k per half:
// faster (shorter lists), and the union still holds the FP8 top 2k.
// The original NBNN mode keeps one running minimum per class.
int fp8_candidates(int k) { return 4 * k; }
int dist_list_len(int mode, int k)
{
    if (mode == LNBNN_FP8_RERANK) return std::min(4 * k, 64);
    if (mode == LNBNN_FP8_RERANK_2K) return 2 * k;
    if (mode == LNBNN_NBNN_I8) return 1;
    return k + 1;
}

// (Re)allocate *p for `need` elements.  A buffer being replaced goes to the
// index's retired list instead of hipFree, which would synchronise the
// whole device (and break a graph being captured on another thread); the
// retired buffers are freed with the index.
static int grow(lnbnn_index *ix, void **p, int64_t need, size_t elem)
{
    if (*p) {
        std::lock_guard<std::mutex> lock(ix->retired_mu);
        ix->retired.push_back(*p);
        *p = nullptr;
    }
    LN_HIP(dmalloc(p, (size_t)std::max<int64_t>(need, 1) * elem));
    return LNBNN_OK;
}

int64_t cap_bucket(int64_t n, int64_t lo)
{
    int64_t b = lo;
    while (b < n) b *= 2;
    return b;
}

int32_t wait_spin_limit()
{
    const char *e = getenv("LNBNN_WAIT_SPINS");
    if (!e || !*e) return 1 << 20;
    const long v = strtol(e, nullptr, 10);
    return (int32_t)std::max(0L, std::min(v, (long)(1 << 30)));
}

int status_check(Workspace &ws)
{
    if (*(volatile int32_t *)ws.h_status != kStatusWaitGaveUp) return LNBNN_OK;
    // the word holds a failure until it is reported
    *(volatile int32_t *)ws.h_status = 0;
    return set_err(LNBNN_EDEVICE,
                   "the distance kernel gave up a bounded wait for an LDS stage (results of the call are invalid)");
}

int begin_batch(const lnbnn_index *ix, int mode, const BatchDesc &bd, const int64_t *off, BatchDesc *dst,
                int64_t *dst_off, int32_t *status, hipStream_t s)
{
    BeginArgs a;
    a.bd = bd;
    a.dst = dst;
    a.dst_off = dst_off;
    a.n_off = bd.n_img + 1;
    a.n_zero = is_fp8_mode(mode) || mode == LNBNN_NBNN_I8 ? 0 : bd.n_img * ix->n_classes;
    a.status = status;
    if (a.n_off <= kBeginOffsets) {
        std::copy(off, off + a.n_off, a.off);
    } else {
        LN_HIP(hipMemcpyAsync(dst_off, off, (size_t)a.n_off * 8, hipMemcpyHostToDevice, s));
        a.n_off = 0;
    }
    LN_HIP(launch_begin(a, s));
    return LNBNN_OK;
}

void drop_graphs(std::map<GraphKey, GraphEntry> &graphs)
{
    for (auto &kv : graphs)
        if (kv.second.exec) (void)hipGraphExecDestroy(kv.second.exec);
    graphs.clear();
}

static void drop_graphs(lnbnn_index *ix) { drop_graphs(ix->graphs); }

// Marks the end of a call's use of the index's workspace on stream s.
static hipError_t ws_mark(lnbnn_index *ix, hipStream_t s)
{
    if (s == ix->own_stream) {
        ix->ws_use = lnbnn_index::WsUse::own;
        return hipSuccess;
    }
    ix->ws_use = lnbnn_index::WsUse::event;
    return hipEventRecord(ix->ws_free, s);
}

// Orders stream s after the last use of the index's workspace.
static int ws_order(lnbnn_index *ix, hipStream_t s)
{
    if (ix->ws_use == lnbnn_index::WsUse::none) return LNBNN_OK;
    if (ix->ws_use == lnbnn_index::WsUse::own) {
        if (s == ix->own_stream) return LNBNN_OK;
        LN_HIP(hipEventRecord(ix->ws_free, ix->own_stream));
    }
    LN_HIP(hipStreamWaitEvent(s, ix->ws_free, 0));
    return LNBNN_OK;
}

// Waits for the last use of the index's workspace.
static int ws_sync(lnbnn_index *ix)
{
    if (ix->ws_use == lnbnn_index::WsUse::own) LN_HIP(hipStreamSynchronize(ix->own_stream));
    if (ix->ws_use == lnbnn_index::WsUse::event) LN_HIP(hipEventSynchronize(ix->ws_free));
    return LNBNN_OK;
}

// Wait for the work that may still use a workspace before its buffers are
// replaced: the index's own workspace is last used by the work before the
// ws_free event; a serving slot's grows only when the slot is created, with
// no work on it yet.  (No device-wide synchronisation: another thread may be
// capturing a graph on a serving stream, and that call is refused then.)
static int quiesce_ws(lnbnn_index *ix, const Workspace &ws)
{
    return &ws == &ix->ws ? ws_sync(ix) : LNBNN_OK;
}

int ensure_ws(lnbnn_index *ix, Workspace &ws, int64_t q_cap, int64_t img_cap, int64_t part, int64_t nbr,
              int64_t qbytes, bool need_f64)
{
    const bool ok = q_cap <= ws.q_cap && img_cap <= ws.img_cap && part <= ws.part_cap &&
                    nbr <= ws.nbr_cap && qbytes <= ws.qbytes_cap && (!need_f64 || ws.totals_f64);
    if (ok && ws.bd) return LNBNN_OK;
    // buffers may be in use by earlier asynchronous work
    int rc;
    if ((rc = quiesce_ws(ix, ws))) return rc;
    if (&ws == &ix->ws) drop_graphs(ix);
    const int64_t nc = ix->n_classes;
    img_cap = std::max(img_cap, ws.img_cap);
    if (img_cap > ws.img_cap || !ws.bd) {
        if ((rc = grow(ix, (void **)&ws.offsets, 2 * img_cap + 2, 8))) return rc;
        if ((rc = grow(ix, (void **)&ws.bd, img_cap + 1, sizeof(BatchDesc)))) return rc;
        if ((rc = grow(ix, (void **)&ws.totals, img_cap * nc, 8))) return rc;
        if ((rc = grow(ix, (void **)&ws.cls, img_cap, 4))) return rc;
        if (ws.totals_f64 || need_f64)
            if ((rc = grow(ix, (void **)&ws.totals_f64, img_cap * nc, 8))) return rc;
        ws.img_cap = img_cap;
    }
    if (need_f64 && !ws.totals_f64)
        if ((rc = grow(ix, (void **)&ws.totals_f64, ws.img_cap * nc, 8))) return rc;
    if (part > ws.part_cap) {
        if ((rc = grow(ix, (void **)&ws.part_d, part, 4))) return rc;
        if ((rc = grow(ix, (void **)&ws.part_i, part, 4))) return rc;
        ws.part_cap = part;
    }
    if (nbr > ws.nbr_cap) {
        if ((rc = grow(ix, (void **)&ws.nbr_idx, nbr, 4))) return rc;
        if ((rc = grow(ix, (void **)&ws.nbr_dist, nbr, 4))) return rc;
        ws.nbr_cap = nbr;
    }
    if (qbytes > ws.qbytes_cap) {
        if ((rc = grow(ix, &ws.q, qbytes, 1))) return rc;
        ws.qbytes_cap = qbytes;
    }
    if (!ws.status) {
        LN_HIP(hipHostMalloc((void **)&ws.h_status, sizeof(int32_t), hipHostMallocDefault));
        *ws.h_status = 0;
        LN_HIP(hipHostGetDevicePointer((void **)&ws.status, ws.h_status, 0));
    }
    ws.q_cap = std::max(ws.q_cap, q_cap);
    return LNBNN_OK;
}

int ensure_fp8_ws(lnbnn_index *ix, Workspace &ws, int64_t q_cap, int n_cand, int k)
{
    const int64_t cand = q_cap * n_cand, upd = q_cap * k;
    if (q_cap <= ws.q8_cap && cand <= ws.cand_cap && upd <= ws.upd_cap && ws.q8) return LNBNN_OK;
    int rc;
    if ((rc = quiesce_ws(ix, ws))) return rc;
    if (&ws == &ix->ws) drop_graphs(ix);
    if (q_cap > ws.q8_cap || !ws.q8) {
        if ((rc = grow(ix, (void **)&ws.q8, q_cap * (kDim / 16), 16))) return rc;
        if ((rc = grow(ix, (void **)&ws.qsc, q_cap, 4))) return rc;
        ws.q8_cap = q_cap;
    }
    if (cand > ws.cand_cap || !ws.cand) {
        if ((rc = grow(ix, (void **)&ws.cand, cand, 4))) return rc;
        ws.cand_cap = cand;
    }
    if (upd > ws.upd_cap || !ws.upd_cls) {
        if ((rc = grow(ix, (void **)&ws.upd_cls, upd, 4))) return rc;
        if ((rc = grow(ix, (void **)&ws.upd_delta, upd, 8))) return rc;
        ws.upd_cap = upd;
    }
    return LNBNN_OK;
}

static int blocks_per_cu(lnbnn_index *ix, int v, int fmt, int kpb)
{
    auto key = std::make_tuple(v, fmt, kpb);
    {
        std::lock_guard<std::mutex> lock(ix->plan_mu);
        auto it = ix->occupancy.find(key);
        if (it != ix->occupancy.end()) return it->second;
    }
    int n = dist_topk_blocks_per_cu(v, fmt, kpb);
    if (n < 1) n = 1;
    std::lock_guard<std::mutex> lock(ix->plan_mu);
    ix->occupancy[key] = n;
    return n;
}

// A variant that can run the mode's format and list length, and keeps the
// mode's candidate rule: the union-of-halves FP8 rule is defined on one list
// per row half, so pair-list variants do not serve it.
static bool variant_serves(int v, int mode, int fmt, int kp)
{
    if (!variant_supports(v, fmt, kp)) return false;
    return !(variant(v).pl && mode == LNBNN_FP8_RERANK_2K);
}

// Variant with per-lane-group lists of rows for an exact search of a small index,
// or -1 where lists of tiles are faster.  k_refine costs every query about the same
// (1 ns and more in a large batch at k = 1), while row lists cost it an insertion
// path that grows with the references seen, and that is latency where a batch does
// not fill the chip.  So the line lies at a number of references that falls with the
// list length and rises with the batch.  Rows against tiles, microseconds a call
// (references x descriptors):
//   FP16  k = 1:  3,000 x 128,000 196 / 232; 6,000 x 64,000 187 / 225, x 128,000 291 / 290
//         k = 2:  600 x 30,000 92 / 110, 3,000 169 / 168
//         k = 5:  1,000 x 64,000 155 / 180, x 30,000 131 / 129; 2,000 x 128,000 305 / 316
//         k = 10: 1,000 x 64,000 240 / 269; 2,000 x 128,000 496 / 499
//         k = 15: 1,000 x 128,000 489 / 590; 600 x 64,000 280 / 320
//   INT8  k = 1:  1,000 x 30,000 65 / 81; 1,000 x 128,000 125 / 143, 3,000 214 / 167
//         k = 10: 300 x 128,000 205 / 284, 600 276 / 284; 300 x 64,000 148 / 166
//         k = 15: 300 x 128,000 288 / 300, 600 385 / 355
// Lists of 21 and 33 stay on tiles (FP16, k = 32, 1,000 x 128,000: 1,106 us, every
// tile recomputed for every query, against 1,270).
static int row_list_variant(int fmt, int kp, int b, int64_t n_refs, int64_t n_q)
{
    const bool q1 = n_q >= 1000, q20 = n_q >= 20000, q50 = n_q >= 50000, q100 = n_q >= 100000;
    int64_t most = 0;           // references
    if (fmt == FMT_F16 || fmt == FMT_BF16) {
        if (b <= 2) most = q100 ? 4500 : q50 ? 6400 : 3200;
        else if (kp == 3) most = q50 ? 1500 : q20 ? 3200 : 0;
        else if (b <= 6) most = q100 ? 2100 : q50 ? 1500 : q20 ? 700 : 0;
        else if (b <= 11) most = q50 ? 1100 : 0;
        else if (b <= 16) most = q100 ? 1100 : q50 ? 700 : 0;
        return n_refs > most ? -1 : b <= 2 && !q100 ? 6 : 2;
    }
    if (b <= 2) most = q100 ? 1100 : q1 ? 3200 : 0;
    else if (b <= 11) most = q100 ? 640 : q50 ? 320 : 0;
    else if (b <= 16) most = q100 ? 320 : 0;
    return n_refs > most ? -1 : q100 ? 2 : 11;
}

// max_lists = 1: the caller's buffers hold one list per query and no more.
static int default_variant(int mode, int fmt, int kp, bool over, int64_t n_refs, int64_t n_tiles, int64_t n_q,
                           int max_lists, int cu_count)
{
    const int b = kp_bucket(kp, fmt);
    if (!is_fp8_mode(mode) && fmt != FMT_I8N && max_lists > 1) {
        const int v = row_list_variant(fmt, kp, b, n_refs, n_q);
        if (v >= 0) return v;
    }
    // Shared lists of tiles wherever the rule allows them.  16x16 blocks (64
    // queries per wave on four query tiles) beat 32x32 pair lists at every batch
    // size measured: INT8, one image of 2,251 descriptors against 15.36M
    // references 4.27 ms against 4.35, 32 images against 2.27M 10.96 against
    // 11.3, the two-class sweep 2.83 against 3.01; FP16, k = 20, 20.3 against
    // 22.0; original NBNN 11.6 against 12.4.  FP8 keeps the 32x32 form, whose keys
    // the re-rank's candidates are defined by.
    if (fmt == FMT_I8 || fmt == FMT_I8N) {
        // Two query halves per wave (blocks of 1,024 queries) read a tile from
        // LDS once for twice the queries: 128 images against 15.36M references
        // 388 ms against 424, 32 against 2.27M 9.9 against 10.5, original NBNN
        // 9.4 against 10.4.  Not where the larger blocks pad more than that
        // gains (one image of 2,251: 4.68 ms against 4.08), nor, with lists
        // (two starts per lane), where a block's pieces are short: 48,000
        // descriptors against 1.2M references (6,900 tiles a piece) 5.9 ms
        // either way, against 0.6M 3.3 against 3.2.
        const int64_t b512 = (n_q + 511) / 512, b1024 = (n_q + 1023) / 1024;
        const int64_t piece = b1024 < cu_count ? n_tiles * b1024 / cu_count : n_tiles;
        const bool halves = b1024 * 200 <= b512 * 106 && variant_supports(28, fmt, kp);
        // (Algorithm 1 on fewer than 64 tiles, too few to cut for idle CUs: 600
        // references, 64,000 descriptors 74 us with halves, 63 without)
        if (fmt == FMT_I8N) return halves && n_tiles >= 64 ? 28 : 15;
        return halves && piece >= 8192 ? 28 : 25;
    }
    if (fmt == FMT_I8L) return 19;
    if (fmt == FMT_F16 || fmt == FMT_BF16) return 26;
    // the union-of-halves rule keeps per-half lists of rows, whose insertions are
    // most of its time over short slices: one query tile per wave (no spills)
    // beats two, 24.2 ms against 30.1 for 48,000 descriptors over 2.27M
    // references, k = 10 (make_plan takes two where the slices are long)
    if (mode == LNBNN_FP8_RERANK_2K) return b <= 40 ? 11 : 0;
    // an FP8 index of no more tiles than the list holds: every tile would be
    // recomputed for every query, so short lists of rows are the better ones
    // (600 references, 64,000 descriptors, k = 5: 379 us against 516) where
    // two lists per query fit
    if (b <= 20 && n_tiles <= kp && max_lists > 1) return 0;
    // 44-64 entries (k = 11..16): one wave per SIMD, 77 ms against 253 on
    // per-half lists for 18,000 descriptors over 15.36M references, k = 16;
    // beyond k = 16 the rule itself is that of per-half lists
    return b <= 40 ? 16 : !over ? 18 : 0;
}

// Most rounds of (block, slice) items worth trying for `rem` blocks: few blocks
// fill a grid almost evenly in one (13 blocks: 19 slices, 247 of 256), and each
// further round only adds lists.
static int64_t cut_rounds(int64_t rem, int64_t grid)
{
    return std::max<int64_t>(1, std::min<int64_t>(8, (16 * rem + grid - 1) / grid));
}

int make_plan(lnbnn_index *ix, int mode, int k, int64_t q_cap, int64_t n_q, int max_lists, Plan *out)
{
    const int kp = dist_list_len(mode, k);
    const bool over = mode == LNBNN_FP8_RERANK && fp8_candidates(k) > kp;   // lists shorter than 4k
    const int fmt = index_fmt(ix, mode);
    const int kpb = kp_bucket(kp, fmt);
    if (kpb == 0) return set_err(LNBNN_EINVAL, "k + 1 = %d is not supported by mode %d", kp, mode);
    lnbnn_tuning tu{-1, 0, 0};
    {
        std::lock_guard<std::mutex> lock(ix->plan_mu);
        auto it = ix->pinned.find({mode, kpb});
        if (it != ix->pinned.end() && q_cap >= it->second.min_q) tu = it->second.t;
    }
    const int64_t n_tiles = ix->rows[fmt] / kTileRows;
    const int v = tu.variant >= 0 ? tu.variant
                                  : default_variant(mode, fmt, kp, over, ix->n_refs, n_tiles, n_q, max_lists,
                                                    ix->cu_count);
    if (!variant_serves(v, mode, fmt, kp))
        return set_err(LNBNN_EINVAL, "variant %d cannot serve mode %d with k + 1 = %d", v, mode, kp);
    const Variant var = variant(v);
    const int64_t qb = (int64_t)var.waves * var.qt * var.nt;
    const int bpc = blocks_per_cu(ix, v, fmt, kpb);
    int64_t resident = (int64_t)ix->cu_count * bpc;
    if (tu.max_workgroups > 0) resident = std::min<int64_t>(resident, tu.max_workgroups);
    auto up8 = [](int64_t t) { return std::max<int64_t>(8, (t + 7) / 8 * 8); };
    Plan p;
    p.variant = v;
    p.fmt = fmt;
    p.kpb = kpb;
    p.pl = var.pl;
    p.block = (int)qb;
    p.max_lists = max_lists;
    p.q_cap = q_cap;
    if (p.pl || fmt == FMT_I8N) {
        // Shared lists (and the original NBNN, whose pieces combine by atomic
        // minima): whole blocks in full rounds of the grid, then the R
        // remaining blocks, cut into slices or equal runs (see k_dist_topk).
        // Every piece costs its tiles and the start of a fresh list, about
        // kStart tiles' time (nearly every tile inserts until 64 k tiles are
        // seen; the original NBNN has no list, only its queries to load and
        // its minima to flush: 6,000 references of two classes, 100,000
        // descriptors 188 us at 128 tiles, 131 at 64, 126 at 32, where batches of
        // 200,000 lose 4 %).  K rounds of (block, slice) items: K x (tiles per
        // slice + start).  Runs: one piece, or two where a block ends inside, per
        // workgroup, whatever R is; but each workgroup then reads other tiles
        // at any time, and the L2 and the infinity cache serve nobody twice
        // (kRunCost).  Without a cut a batch just past a multiple of 256 blocks
        // ran one more whole round: 563 blocks of 512 queries over 15.36M
        // references took 526 ms instead of 431 ms.
        const double kStart = fmt == FMT_I8N ? 64 : 128;
        constexpr double kRunCost = 1.08;
        const int64_t n_qb = std::max<int64_t>(1, (n_q + qb - 1) / qb);
        const int64_t grid = resident, full = n_qb / grid, rem = n_qb % grid;
        int64_t slices = rem > 0 ? 1 : 0, tiles = n_tiles, pieces = rem;
        if (rem > 0 && max_lists > 1) {
            // Up to an eighth of the grid in blocks: a sweep of few tiles is
            // nothing but list start, cut or not (each tile inserts, about three
            // tiles' time), and its latency is all there is: 2,000 descriptors
            // against 3,000 FP16 references, k = 10, 76 us in slices of 8 of the 96
            // tiles, 160 in one sweep.  With more blocks the second list of every
            // query costs more than that gains (INT8, 64,000 descriptors, 2,000
            // references, k = 10: 191 us whole, 247 in two slices).
            // 16 tiles are too few to be worth it (INT8, 300 references, 12,000
            // descriptors, k = 5: 68 us whole, 74 in two).
            const bool few = fmt != FMT_I8N && rem * 8 <= grid && n_tiles > 16;
            auto piece = [&](double t) { return t + (few ? std::min(2 * t, kStart) : kStart); };
            double best = few ? piece((double)n_tiles) : (double)n_tiles;
            for (int64_t rounds = 1; rounds <= cut_rounds(rem, grid); ++rounds) {
                // as many slices as fill the rounds, or as a query may have lists
                // (three blocks in at most 64 lists each: 192 of 256 workgroups)
                const int64_t most = std::min<int64_t>(rounds * grid / rem, max_lists);
                const int64_t t = up8((n_tiles + most - 1) / most);
                const int64_t n = (n_tiles + t - 1) / t;
                const double cost = (double)((rem * n + grid - 1) / grid) * piece((double)t);
                if (n > 1 && cost < best) {
                    best = cost;
                    slices = n;
                    tiles = t;
                    pieces = rem * n;
                }
            }
            const int64_t run = up8((rem * n_tiles + grid - 1) / grid);
            if (run < n_tiles && (n_tiles - 1) / run + 2 <= max_lists && ((double)run + 2 * kStart) * kRunCost < best) {
                slices = 0;
                tiles = run;
                pieces = rem + (rem * n_tiles + run - 1) / run;
            }
        }
        const bool cut = rem > 0 && tiles < n_tiles;
        p.grid = (int)grid;
        p.walk.full_rounds = (int)full;
        p.walk.rem_slices = (int)slices;
        p.walk.slice_tiles = (int)tiles;
        p.lists = cut ? (full * grid + pieces) * qb : std::max<int64_t>(n_q, 1);
        p.n_slices = (int)((n_tiles + tiles - 1) / tiles);
        p.n_lists = 1;
        p.chunk_tiles = (int)(tu.chunk_tiles > 0 ? std::min<int64_t>(tu.chunk_tiles, n_tiles) : n_tiles);
        *out = p;
        return LNBNN_OK;
    }
    // One list per lane group: the reference set is split into equal slices
    // only when the query blocks alone cannot keep every workgroup slot busy
    // twice over; each split costs one more partial list per lane group (the
    // merge takes at most kMaxLists lists per query).  The split is the one
    // whose (query block, slice) items fill the resident workgroups most
    // evenly: estimated time = rounds of items x (tiles per slice + a start-up
    // cost per item), fewest slices on a tie.  It depends on the capacity
    // bucket alone, and for the default shape of the union-of-halves FP8 rule
    // (whose candidates are those of the slices' lists) on blocks of 512
    // queries, one workgroup per CU, whatever shape runs it.
    const int groups = 64 / var.qt;                      // lists per query and slice
    const bool by512 = mode == LNBNN_FP8_RERANK_2K && kpb <= 20 && tu.variant < 0;
    const int64_t slice_qb = by512 ? 512 : qb;
    const int64_t resident_wg = resident;
    if (by512) {
        resident = ix->cu_count;
        if (tu.max_workgroups > 0) resident = std::min<int64_t>(resident, tu.max_workgroups);
    }
    const int64_t n_qb = std::max<int64_t>(1, (q_cap + slice_qb - 1) / slice_qb);
    auto slice_tiles = [&](int64_t s) { return up8((n_tiles + s - 1) / s); };
    int64_t tps = slice_tiles(1);
    if (n_qb < 2 * resident) {
        constexpr int64_t kItemStartTiles = 32;
        double best = 1e300;
        for (int64_t s = 1; s <= kMaxLists / groups; ++s) {
            const int64_t t = slice_tiles(s);
            if ((n_tiles + t - 1) / t != s) continue;          // the same split as a smaller s
            const int64_t rounds = (n_qb * s + resident - 1) / resident;
            const double cost = (double)rounds * (double)(t + kItemStartTiles);
            if (cost < best) {
                best = cost;
                tps = t;
            }
        }
    }
    const int64_t S = (n_tiles + tps - 1) / tps;
    p.n_slices = (int)S;
    p.n_lists = (int)S * groups;
    p.walk.n_slices = (int)S;
    p.walk.tiles_per_slice = (int)tps;
    int64_t item_qb = qb, grid_wg = resident_wg;
    // The union-of-halves rule: two query tiles per wave read a tile once for
    // twice the queries and win where the lists have settled, over long slices.
    // Lists of up to 8 (k <= 4): 48,000 descriptors, k = 1, slices of 8,900 tiles
    // 12.2 ms against 17.1, k = 3 14.9 against 18.8; one image, 15,000 tiles 5.6
    // against 7.9.  Lists of 20, whose insertions cost more: slices of 60,000
    // tiles 96 ms against 119, 48,000 tiles 36.5 against 39.6, but 8,900 tiles
    // 28.6 against 22.7.  And for lists of up to 4 where whole slices of 512
    // queries fill the chip anyway (45,500 descriptors over 97,000 references,
    // k = 1, three indexes in turn: 0.79 against 0.89 a call, though alone 1.23
    // against 1.09).  One tile elsewhere: its items are twice as many (one
    // image, slices of 2,200 tiles, k = 1: 0.85 against 1.38).  Same slices and
    // lists either way.
    const int64_t settled = kpb <= 8 ? 4096 : 24576;
    if (by512 && (tps >= settled || (kpb <= 4 && n_qb * S >= ix->cu_count))) {
        p.variant = 8;
        item_qb = slice_qb;
        p.block = (int)item_qb;
        grid_wg = (int64_t)ix->cu_count * blocks_per_cu(ix, p.variant, fmt, kpb);
        if (tu.max_workgroups > 0) grid_wg = std::min<int64_t>(grid_wg, tu.max_workgroups);
    }
    p.grid = (int)std::max<int64_t>(1, std::min<int64_t>((q_cap + item_qb - 1) / item_qb * S, grid_wg));
    // By default an item sweeps its whole slice with its lists in registers;
    // a tuned chunk length makes workgroups that own several items walk the
    // slice chunk by chunk instead (lists saved between chunks), which keeps
    // the workgroups of an XCD on the same references at the same time.
    p.chunk_tiles = tu.chunk_tiles > 0 ? (int)std::min<int64_t>(tu.chunk_tiles, tps) : (int)tps;
    *out = p;
    return LNBNN_OK;
}

int64_t batch_elems(const lnbnn_index *ix, const Plan &p, int64_t q_cap)
{
    // the original NBNN mode keeps its per-class minima in part_i
    if (p.fmt == FMT_I8N) return (int64_t)ix->n_classes * q_cap;
    if (p.pl) return p.lists * p.kpb;
    return (int64_t)p.n_lists * q_cap * p.kpb;
}

int64_t work_elems(const lnbnn_index *ix, const Plan &p, int64_t q_cap)
{
    if (!p.pl || p.fmt == FMT_I8N) return batch_elems(ix, p, q_cap);
    // whole blocks have one list per query; the remaining ones, fewer than a
    // grid, at most cut_rounds rounds of (block, slice) items or one piece per
    // block and workgroup, and at most max_lists per block
    if (p.max_lists <= 1) return std::max<int64_t>(q_cap, 1) * p.kpb;
    auto lists = [&](int64_t block) {
        const int64_t n_qb = std::max<int64_t>(1, (q_cap + block - 1) / block);
        const int64_t rem = std::min<int64_t>(n_qb, p.grid);
        const int64_t pieces = std::max<int64_t>(cut_rounds(rem, p.grid) * p.grid, rem + p.grid);
        return (n_qb / p.grid * p.grid + std::min<int64_t>(pieces, rem * p.max_lists)) * block;
    };
    // INT8 batches of other sizes may take the shape with larger blocks, where
    // the list length has it
    return std::max(lists(p.block), p.fmt == FMT_I8 && variant_supports(28, p.fmt, p.kpb) ? lists(1024) : 0) * p.kpb;
}

int enqueue_batch(lnbnn_index *ix, const Plan &p, const BatchIO &io, hipStream_t s, hipEvent_t *kev)
{
    if (fault_injected("launch")) return set_err(LNBNN_EDEVICE, "injected launch failure");
    const bool fp8 = p.fmt == FMT_FP8;
    // every buffer the launches write must hold what this plan writes
    const Workspace *w = io.ws;
    const bool nbnn = p.fmt == FMT_I8N;
    if (!w || io.q_cap > w->q_cap || io.img_cap > w->img_cap || batch_elems(ix, p, io.q_cap) > w->part_cap ||
        !w->status)
        return set_err(LNBNN_EINVAL, "internal: workspace smaller than the plan");
    if (fp8 && (io.q_cap > w->q8_cap || io.q_cap * fp8_candidates(io.k) > w->cand_cap ||
                io.q_cap * io.k > w->upd_cap))
        return set_err(LNBNN_EINVAL, "internal: FP8 workspace smaller than the plan");
    if (fp8)
        LN_HIP(launch_fp8_qprep(io.bd, io.q_cap, io.q8, io.qsc, s));
    else if (nbnn)
        LN_HIP(launch_fill_i32(io.part_i, 0x7fffffff, io.q_cap, io.q_cap, ix->n_classes, io.bd, s));
    DistArgs a{};
    a.q = fp8 ? static_cast<const void *>(io.q8) : nullptr;
    a.q_scale = io.qsc;
    a.bd = io.bd;
    a.frag = ix->frag[p.fmt];
    a.seed = ix->seed[p.fmt];
    // never read by the unscaled formats; any valid address keeps the
    // kernel's pointer arithmetic defined
    a.row_scale = ix->row_scale ? ix->row_scale : reinterpret_cast<const int32_t *>(a.seed);
    a.odd_tile0 = ix->odd_tile0;
    a.n_tiles = ix->rows[p.fmt] / kTileRows;
    a.chunk_tiles = p.chunk_tiles;
    a.q_cap = io.q_cap;
    a.part_d = io.part_d;
    a.part_i = io.part_i;
    a.status = w->status;
    a.spin_limit = wait_spin_limit();
    a.tile_class = nbnn ? ix->tile_class : nullptr;
    a.cls_min = nbnn ? io.part_i : nullptr;
    if (kev) LN_HIP(hipEventRecord(kev[0], s));
    LN_HIP(launch_dist_topk(p.variant, p.fmt, p.kpb, a, p.grid, s));
    if (kev) LN_HIP(hipEventRecord(kev[1], s));
    RefineArgs t{};
    t.q = a.q;
    t.q_scale = a.q_scale;
    t.frag = a.frag;
    t.seed = a.seed;
    t.row_scale = a.row_scale;
    t.odd_tile0 = a.odd_tile0;
    t.n_need = dist_list_len(io.mode, io.k);
    t.map = SlotMap{a.n_tiles, p.block, p.grid};
    if (fp8) {
        RerankArgs r{};
        r.bd = io.bd;
        r.offsets = io.offsets;
        r.ref_f32 = ix->ref_f32;
        r.labels = ix->labels;
        r.n_refs = ix->n_refs;
        r.n_lists = p.n_lists;
        r.kp_stride = p.kpb;
        r.n_cand = fp8_candidates(io.k);
        r.k = io.k;
        r.n_classes = ix->n_classes;
        r.q_cap = io.q_cap;
        r.part_d = io.part_d;
        r.part_i = io.part_i;
        r.cand = io.cand;
        r.upd_cls = io.upd_cls;
        r.upd_delta = io.upd_delta;
        r.status = w->status;
        if (p.pl)
            LN_HIP(launch_refine_fp8(variant(p.variant).qt, t, r, io.q_cap, s));
        else
            LN_HIP(launch_cand_merge(r, io.q_cap, s));
        LN_HIP(launch_rerank(r, io.q_cap, io.img_cap, s));
    } else if (nbnn) {
        NbnnArgs n{};
        n.bd = io.bd;
        n.offsets = io.offsets;
        n.cls_min = io.part_i;
        n.q_cap = io.q_cap;
        n.n_classes = ix->n_classes;
        LN_HIP(launch_nbnn_totals(n, io.img_cap, s));
        LN_HIP(launch_argmin(io.bd, io.img_cap, ix->n_classes, s));
    } else {
        FinishArgs f{};
        f.q_shift = p.fmt == FMT_I8 || p.fmt == FMT_I8L ? 128 : 0;
        f.dim = ix->dim;
        f.bd = io.bd;
        f.offsets = io.offsets;
        f.labels = ix->labels;
        f.perm = p.fmt == FMT_I8 || p.fmt == FMT_I8L ? ix->perm : nullptr;
        f.n_rows = ix->rows[p.fmt];
        f.n_refs = ix->n_refs;
        f.n_lists = p.n_lists;
        f.kp_stride = p.kpb;
        f.k = io.k;
        f.n_classes = ix->n_classes;
        f.q_cap = io.q_cap;
        f.part_d = io.part_d;
        f.part_i = io.part_i;
        f.status = w->status;
        if (p.pl)
            LN_HIP(launch_refine(p.fmt, t, f, io.q_cap, s));
        else
            LN_HIP(launch_finish(f, io.q_cap, s));
        LN_HIP(launch_argmin(io.bd, io.img_cap, ix->n_classes, s));
    }
    return LNBNN_OK;
}

}  // namespace lnbnn

// ===========================================================================
// index
// ===========================================================================
static int free_index_buffers(lnbnn_index *ix)
{
    for (int f = 0; f < kNumFmt; ++f) {
        if (ix->frag[f]) dfree(ix->frag[f]);
        ix->frag[f] = nullptr;
    }
    // seeds of the two exact 16-bit formats share one buffer
    if (ix->seed[FMT_F16]) dfree(ix->seed[FMT_F16]);
    else if (ix->seed[FMT_BF16]) dfree(ix->seed[FMT_BF16]);
    if (ix->seed[FMT_FP8]) dfree(ix->seed[FMT_FP8]);
    if (ix->seed[FMT_I8]) dfree(ix->seed[FMT_I8]);
    if (ix->seed[FMT_I8L]) dfree(ix->seed[FMT_I8L]);
    if (ix->seed[FMT_I8N]) dfree(ix->seed[FMT_I8N]);
    for (int f = 0; f < kNumFmt; ++f) ix->seed[f] = nullptr;
    if (ix->perm) dfree(ix->perm);
    ix->perm = nullptr;
    if (ix->tile_class) dfree(ix->tile_class);
    ix->tile_class = nullptr;
    if (ix->labels) dfree(ix->labels);
    if (ix->ref_f32) dfree(ix->ref_f32);
    if (ix->row_scale) dfree(ix->row_scale);
    ix->labels = nullptr;
    ix->ref_f32 = nullptr;
    ix->row_scale = nullptr;
    std::lock_guard<std::mutex> lock(ix->retired_mu);
    for (void *p : ix->retired) dfree(p);
    ix->retired.clear();
    return LNBNN_OK;
}

static void free_index_handles(lnbnn_index *ix)
{
    for (auto &e : ix->tev)
        if (e) (void)hipEventDestroy(e);
    if (ix->ws_free) (void)hipEventDestroy(ix->ws_free);
    if (ix->own_stream) stream_release(ix->device, ix->own_stream);
}

// The class-sorted INT8 copy of the index for the original NBNN rule
// (Algorithm 1 needs every class's nearest reference): references sorted by
// class (stable), every class padded to a multiple of 256 rows so that a
// class never shares a 32-row tile or an 8-tile stage with another, and
// the class of every tile.  Every class must own a reference.
struct NbnnHost {
    std::vector<int32_t> perm, tile_class;
};

static int build_nbnn_layout(lnbnn_index *ix, const uint8_t *d_refs, const int32_t *hlab, hipStream_t s,
                             NbnnHost &h, int64_t *bytes)
{
    if (ix->dim != kDim) return set_err(LNBNN_EINVAL, "the original NBNN mode takes %d-byte descriptors", kDim);
    const int32_t nc = ix->n_classes;
    // Rows sorted by (class, parity of ||r - 128||^2), each (class, parity)
    // group padded to whole stages: every stage then holds one class and one
    // parity, so the kernel knows a tile's exact smallest key from its
    // smallest accumulator value (key = 2 D + parity).
    std::vector<uint8_t> par(ix->n_refs);
    {
        uint8_t *d_par = nullptr;
        LN_HIP(dmalloc_async((void **)&d_par, std::max<int64_t>(1, ix->n_refs), s));
        hipError_t e = launch_row_parity(d_refs, ix->n_refs, kDim, d_par, s);
        if (e == hipSuccess) e = hipMemcpyAsync(par.data(), d_par, ix->n_refs, hipMemcpyDeviceToHost, s);
        (void)hipFreeAsync(d_par, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_err(e, "row parity");
    }
    std::vector<int64_t> cnt(2 * (size_t)nc, 0), start(2 * (size_t)nc + 1, 0);
    for (int64_t j = 0; j < ix->n_refs; ++j) cnt[2 * (size_t)hlab[j] + par[j]] += 1;
    for (int32_t c = 0; c < nc; ++c)
        if (cnt[2 * c] + cnt[2 * c + 1] == 0)
            return set_err(LNBNN_EINVAL, "the original NBNN mode needs every class to own a reference (class %d has none)",
                           c);
    for (int32_t g = 0; g < 2 * nc; ++g) start[g + 1] = start[g] + (cnt[g] + kPadRows - 1) / kPadRows * kPadRows;
    const int64_t n_nb = start[2 * nc];
    if (n_nb >= (int64_t)0x7fffffff) return set_err(LNBNN_EINVAL, "class-sorted index too large");
    h.perm.assign(n_nb, -1);
    std::vector<int64_t> next(start.begin(), start.end() - 1);
    for (int64_t j = 0; j < ix->n_refs; ++j) h.perm[next[2 * (size_t)hlab[j] + par[j]]++] = (int32_t)j;
    // per tile: 2 * class + parity
    h.tile_class.resize(n_nb / kTileRows);
    for (int32_t g = 0; g < 2 * nc; ++g)
        for (int64_t t = start[g] / kTileRows; t < start[g + 1] / kTileRows; ++t) h.tile_class[t] = g;
    int rc;
    int32_t *d_perm = nullptr, *iseed = nullptr;
    if ((rc = grow(ix, (void **)&ix->tile_class, n_nb / kTileRows, 4))) return rc;
    if ((rc = grow(ix, (void **)&ix->frag[FMT_I8N], n_nb * kDim, 1))) return rc;
    if ((rc = grow(ix, (void **)&iseed, n_nb, 4))) return rc;
    ix->seed[FMT_I8N] = reinterpret_cast<float *>(iseed);
    *bytes = n_nb * (kDim + 4) + n_nb / kTileRows * 4;
    LN_HIP(dmalloc_async((void **)&d_perm, n_nb * 4, s));
    hipError_t e = hipMemcpyAsync(d_perm, h.perm.data(), n_nb * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ix->tile_class, h.tile_class.data(), h.tile_class.size() * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = launch_pack_i8(d_refs, n_nb, kDim, ix->frag[FMT_I8N], iseed, s, d_perm);
    (void)hipFreeAsync(d_perm, s);
    if (e != hipSuccess) return hip_err(e, "class-sorted pack");
    ix->rows[FMT_I8N] = n_nb;
    return LNBNN_OK;
}

// The INT8 copy of the index: rows by parity of ||r - 128||^2 (the even ones
// first, each part in reference order and padded to 256 rows), their seeds and
// the reference of every packed row.
static int build_i8(lnbnn_index *ix, const uint8_t *d_refs, int fmt, hipStream_t s, int64_t *bytes)
{
    const int64_t n = ix->n_refs, n_blocks = (n + 255) / 256;
    auto up = [](int64_t r) { return (r + kPadRows - 1) / kPadRows * kPadRows; };
    const int64_t most = up(n) + kPadRows;           // rows, however the parities fall
    int32_t *iseed = nullptr;
    int rc = grow(ix, (void **)&ix->frag[fmt], most * ix->dim, 1);
    if (!rc) rc = grow(ix, (void **)&iseed, most, 4);
    if (!rc) ix->seed[fmt] = reinterpret_cast<float *>(iseed);
    if (!rc) rc = grow(ix, (void **)&ix->perm, most, 4);
    if (rc) return rc;
    // the parity of every reference and the blocks' odd counts sit in the seeds'
    // buffer until the rows are packed: n + n / 64 of its 4 n bytes
    uint8_t *d_par = reinterpret_cast<uint8_t *>(iseed);
    int32_t *block_odd = iseed + (n + 3) / 4;
    int32_t n_odd = 0;
    hipError_t e = launch_row_parity(d_refs, n, ix->dim, d_par, s);
    if (e == hipSuccess) e = launch_parity_count(d_par, n, block_odd, s);
    if (e == hipSuccess) e = hipMemcpyAsync(&n_odd, block_odd + n_blocks, 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    const int64_t even_pad = up(n - n_odd), n_pad = even_pad + up(n_odd);
    if (e == hipSuccess) e = launch_parity_perm(d_par, n, block_odd, even_pad, n_pad, ix->perm, s);
    if (e == hipSuccess) e = launch_pack_i8(d_refs, n_pad, ix->dim, ix->frag[fmt], iseed, s, ix->perm);
    if (e != hipSuccess) rc = hip_err(e, "pack i8");
    ix->rows[fmt] = n_pad;
    ix->odd_tile0 = (int32_t)(even_pad / kTileRows);
    *bytes += most * (ix->dim + 8);
    return rc;
}

extern "C" int lnbnn_build_index(const void *refs, int dtype, int64_t n_refs, int32_t dim,
                                 const int32_t *labels, int32_t n_classes, uint32_t mode_mask,
                                 int64_t hbm_budget_bytes, uint32_t flags, void *stream,
                                 lnbnn_index **out)
{
    if (!out || !refs || !labels) return set_err(LNBNN_EINVAL, "NULL argument");
    if (dim != LNBNN_DIM && dim != LNBNN_DIM_LOC)
        return set_err(LNBNN_EINVAL, "dim must be %d or %d (got %d)", LNBNN_DIM, LNBNN_DIM_LOC, dim);
    if (dim == LNBNN_DIM_LOC && (dtype != LNBNN_U8 || mode_mask != LNBNN_MODE_BIT(LNBNN_EXACT_I8)))
        return set_err(LNBNN_EINVAL, "dim %d (location-augmented) needs u8 data and the INT8 mode alone",
                       LNBNN_DIM_LOC);
    if (n_refs < 1 || n_refs >= (int64_t)0x7fffffff - kPadRows)
        return set_err(LNBNN_EINVAL, "n_refs out of range: %lld", (long long)n_refs);
    if (n_classes < 1) return set_err(LNBNN_EINVAL, "n_classes must be >= 1");
    if (dtype != LNBNN_U8 && dtype != LNBNN_F32) return set_err(LNBNN_EINVAL, "bad dtype %d", dtype);
    if (hbm_budget_bytes < 0) return set_err(LNBNN_EINVAL, "negative HBM budget");
    const uint32_t exact = LNBNN_MODE_BIT(LNBNN_EXACT_F16) | LNBNN_MODE_BIT(LNBNN_EXACT_BF16) |
                           LNBNN_MODE_BIT(LNBNN_EXACT_I8) | LNBNN_MODE_BIT(LNBNN_NBNN_I8);
    const uint32_t fp8m = LNBNN_MODE_BIT(LNBNN_FP8_RERANK) | LNBNN_MODE_BIT(LNBNN_FP8_RERANK_2K);
    if (mode_mask == 0) return set_err(LNBNN_EINVAL, "empty mode mask");
    if (dtype == LNBNN_U8 && (mode_mask & ~exact))
        return set_err(LNBNN_EINVAL, "mode mask 0x%x: u8 data builds only the exact modes", mode_mask);
    if (dtype == LNBNN_F32 && (mode_mask & ~fp8m))
        return set_err(LNBNN_EINVAL, "mode mask 0x%x: float data builds only the FP8 re-rank modes", mode_mask);
    if (flags & ~(uint32_t)LNBNN_DEVICE_PTRS) return set_err(LNBNN_EINVAL, "unknown flags 0x%x", flags);
    const bool dev_in = flags & LNBNN_DEVICE_PTRS;
    if (!dev_in) {
        for (int64_t j = 0; j < n_refs; ++j)
            if (labels[j] < 0 || labels[j] >= n_classes)
                return set_err(LNBNN_EINVAL, "label[%lld] = %d outside [0, %d)", (long long)j, labels[j],
                               n_classes);
    }

    int dev = 0;
    LN_HIP(hipGetDevice(&dev));
    std::unique_ptr<lnbnn_index> ix(new lnbnn_index());
    ix->device = dev;
    ix->dtype = dtype;
    ix->dim = dim;
    ix->n_refs = n_refs;
    ix->n_pad = (n_refs + kPadRows - 1) / kPadRows * kPadRows;
    ix->n_classes = n_classes;
    ix->modes = mode_mask;
    ix->ws.device = dev;
    LN_HIP(hipDeviceGetAttribute(&ix->cu_count, hipDeviceAttributeMultiprocessorCount, dev));
    int rc = stream_acquire(dev, &ix->own_stream);
    if (rc) return rc;
    hipStream_t s = stream ? (hipStream_t)stream : ix->own_stream;
    lnbnn_index *ixp = ix.get();
    auto fail = [&](int rc) {
        (void)hipStreamSynchronize(s);
        free_index_buffers(ix.get());
        free_index_handles(ix.get());
        return rc;
    };
    for (auto &e : ix->tev) {
        const hipError_t err = hipEventCreate(&e);
        if (err != hipSuccess) return fail(hip_err(err, "hipEventCreate"));
    }
    {
        const hipError_t err = hipEventCreateWithFlags(&ix->ws_free, hipEventDisableTiming);
        if (err != hipSuccess) return fail(hip_err(err, "hipEventCreate"));
    }

    // labels: device copy, and validation when they came as device memory: on the
    // device (2.3M labels read back and checked here took 2 ms), but a few are
    // read back at once (314 references, 16-bit build 48 us against 59)
    if ((rc = grow(ixp, (void **)&ix->labels, n_refs + 1, 4))) return fail(rc);
    std::vector<int32_t> hl;           // host copy of device labels (few, or the class-sorted layout)
    constexpr int64_t kFewLabels = 8192;
    if (dev_in && n_refs <= kFewLabels) {
        hl.resize(n_refs);
        // the blocking copy also follows the process's blocking streams, on
        // which the inputs may still be written
        hipError_t e = hipMemcpy(hl.data(), labels, n_refs * 4, hipMemcpyDeviceToHost);
        if (e != hipSuccess) return fail(hip_err(e, "hipMemcpy(labels)"));
        for (int64_t j = 0; j < n_refs; ++j)
            if (hl[j] < 0 || hl[j] >= n_classes)
                return fail(set_err(LNBNN_EINVAL, "label[%lld] = %d outside [0, %d)", (long long)j, hl[j], n_classes));
        e = hipMemcpyAsync(ix->labels, labels, n_refs * 4, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return fail(hip_err(e, "hipMemcpyAsync(labels)"));
    } else if (dev_in) {
        // the same wait (with the labels copied on the NULL stream instead, which
        // the index's own follows: 95 us a 16-bit build of 16,385 references, now 60)
        hipError_t e = hipStreamSynchronize(nullptr);
        if (e == hipSuccess) e = hipMemcpyAsync(ix->labels, labels, n_refs * 4, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return fail(hip_err(e, "hipMemcpyAsync(labels)"));
        int32_t bad = 0, value = 0;    // first label out of range (n_refs: none), in the spare last element
        e = launch_check_labels(ix->labels, n_refs, n_classes, ix->labels + n_refs, s);
        if (e == hipSuccess) e = hipMemcpyAsync(&bad, ix->labels + n_refs, 4, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e == hipSuccess && bad < n_refs) e = hipMemcpy(&value, ix->labels + bad, 4, hipMemcpyDeviceToHost);
        if (e == hipSuccess && (mode_mask & LNBNN_MODE_BIT(LNBNN_NBNN_I8)) && bad >= n_refs) {
            hl.resize(n_refs);
            e = hipMemcpy(hl.data(), ix->labels, n_refs * 4, hipMemcpyDeviceToHost);
        }
        if (e != hipSuccess) return fail(hip_err(e, "label check"));
        if (bad < n_refs)
            return fail(set_err(LNBNN_EINVAL, "label[%lld] = %d outside [0, %d)", (long long)bad, value, n_classes));
    } else {
        hipError_t e = hipMemcpyAsync(ix->labels, labels, n_refs * 4, hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return fail(hip_err(e, "hipMemcpyAsync(labels)"));
    }

    // references: stage the rows on the device, then pack per mode
    const int64_t rbytes = n_refs * row_bytes(dtype, dim);
    const void *d_refs = refs;
    void *staged = nullptr;
    if (dtype == LNBNN_F32) {
        // the FP32 rows stay resident for the exact re-rank
        if ((rc = grow(ixp, (void **)&ix->ref_f32, n_refs * kDim, 4))) return fail(rc);
        hipError_t e = hipMemcpyAsync(ix->ref_f32, refs, (size_t)rbytes,
                                      dev_in ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return fail(hip_err(e, "hipMemcpyAsync(refs)"));
        d_refs = ix->ref_f32;
    } else if (!dev_in) {
        // stream-ordered staging: freeing it does not synchronise the device
        hipError_t e = fault_injected("alloc") ? hipErrorOutOfMemory : dmalloc_async(&staged, (size_t)rbytes, s);
        if (e != hipSuccess) return fail(hip_err(e, "hipMallocAsync(staging)"));
        e = hipMemcpyAsync(staged, refs, (size_t)rbytes, hipMemcpyHostToDevice, s);
        if (e != hipSuccess) {
            (void)hipFreeAsync(staged, s);
            return fail(hip_err(e, "hipMemcpyAsync(refs)"));
        }
        d_refs = staged;
    }
    float *seed = nullptr;
    int64_t bytes = n_refs * 4 + (dtype == LNBNN_F32 ? rbytes : 0);
    // seeds of the 16-bit or the FP8 copy (the INT8 copies have their own)
    if (dtype == LNBNN_F32 || (mode_mask & (LNBNN_MODE_BIT(LNBNN_EXACT_F16) | LNBNN_MODE_BIT(LNBNN_EXACT_BF16)))) {
        rc = grow(ixp, (void **)&seed, ix->n_pad, 4);
        if (!rc) bytes += ix->n_pad * 4;
    }
    bool seeded = false;
    if (dtype == LNBNN_F32) {
        if (!rc) rc = grow(ixp, (void **)&ix->row_scale, ix->n_pad, 4);
        if (!rc) rc = grow(ixp, (void **)&ix->frag[FMT_FP8], ix->n_pad * kDim, 1);
        if (!rc) {
            bytes += ix->n_pad * (4 + kDim);
            hipError_t e = launch_fp8_index(static_cast<const float *>(d_refs), n_refs, ix->n_pad,
                                            ix->frag[FMT_FP8], seed, ix->row_scale, s);
            if (e != hipSuccess) rc = hip_err(e, "fp8 pack");
            seeded = true;
            ix->seed[FMT_FP8] = seed;
        }
    }
    for (int mode : {LNBNN_EXACT_F16, LNBNN_EXACT_BF16}) {
        if (rc || dtype != LNBNN_U8 || !(mode_mask & LNBNN_MODE_BIT(mode))) continue;
        const int fmt = mode_fmt(mode);
        if ((rc = grow(ixp, (void **)&ix->frag[fmt], ix->n_pad * kDim * 2, 1))) break;
        bytes += ix->n_pad * kDim * 2;
        hipError_t e = launch_pack_u8(static_cast<const uint8_t *>(d_refs), n_refs, ix->n_pad, fmt, ix->frag[fmt],
                                      seeded ? nullptr : seed, s);
        if (e != hipSuccess) {
            rc = hip_err(e, "pack");
            break;
        }
        seeded = true;
        ix->seed[fmt] = seed;
    }
    for (int f = 0; f < kNumFmt; ++f) ix->rows[f] = ix->n_pad;
    if (!rc && dtype == LNBNN_U8 && (mode_mask & LNBNN_MODE_BIT(LNBNN_EXACT_I8)))
        rc = build_i8(ixp, static_cast<const uint8_t *>(d_refs), index_fmt(ixp, LNBNN_EXACT_I8), s, &bytes);
    NbnnHost nbh;   // host arrays of the class-sorted copy: alive until the sync below
    if (!rc && (mode_mask & LNBNN_MODE_BIT(LNBNN_NBNN_I8))) {
        int64_t nb_bytes = 0;
        rc = build_nbnn_layout(ixp, static_cast<const uint8_t *>(d_refs), dev_in ? hl.data() : labels, s, nbh,
                               &nb_bytes);
        bytes += nb_bytes;
    }
    if (staged) (void)hipFreeAsync(staged, s);
    hipError_t e = hipStreamSynchronize(s);
    if (rc) {
        if (seed && !seeded) dfree(seed);
        return fail(rc);
    }
    if (e != hipSuccess) return fail(hip_err(e, "build_index sync"));
    ix->device_bytes = bytes;
    size_t free_b = 0, total_b = 0;
    LN_HIP(hipMemGetInfo(&free_b, &total_b));
    const int64_t env_b = env_budget();
    free_b += kept_bytes(dev);
    ix->hbm_budget = hbm_budget_bytes ? hbm_budget_bytes : env_b ? env_b : (int64_t)(free_b / 4);
    log_line("index built: %lld references, dim %d, %d classes, modes 0x%x, %lld device bytes, serving budget %lld bytes",
             (long long)ix->n_refs, ix->dim, ix->n_classes, ix->modes, (long long)ix->device_bytes,
             (long long)ix->hbm_budget);
    *out = ix.release();
    return LNBNN_OK;
}

extern "C" int lnbnn_index_free(lnbnn_index *ix)
{
    if (!ix) return LNBNN_OK;
    if (server_pending(ix)) return set_err(LNBNN_EBUSY, "index has pending tickets");
    server_stop(ix);                       // joins the serving threads after their streams drain
    (void)hipSetDevice(ix->device);
    // the index's own work: the last classify call and its stream
    (void)ws_sync(ix);
    if (ix->own_stream) (void)hipStreamSynchronize(ix->own_stream);
    // and calls that leave no mark (lnbnn_classify_noalloc on a caller's
    // stream): the buffers may go to another index at once.  Where the device
    // cannot be waited for (a capture elsewhere), they go back to the driver.
    struct KeepScope {
        ~KeepScope() { t_keep_frees = true; }
    } scope;
    if (hipDeviceSynchronize() != hipSuccess) {
        (void)hipGetLastError();
        t_keep_frees = false;
    }
    drop_graphs(ix);
    free_index_buffers(ix);
    free_index_handles(ix);
    delete ix;
    return LNBNN_OK;
}

extern "C" int lnbnn_trim(void)
{
    std::lock_guard<std::mutex> lock(g_kept_mu);
    drop_kept_locked(0);
    return LNBNN_OK;
}

extern "C" int lnbnn_index_stream(const lnbnn_index *ix, void **stream)
{
    if (!ix || !stream) return set_err(LNBNN_EINVAL, "NULL argument");
    *stream = ix->own_stream;
    return LNBNN_OK;
}

extern "C" int lnbnn_index_info(const lnbnn_index *ix, int64_t *n_refs, int32_t *n_classes,
                                uint32_t *mode_mask, int64_t *device_bytes)
{
    if (!ix) return set_err(LNBNN_EINVAL, "NULL index");
    if (n_refs) *n_refs = ix->n_refs;
    if (n_classes) *n_classes = ix->n_classes;
    if (mode_mask) *mode_mask = ix->modes;
    if (device_bytes) *device_bytes = ix->device_bytes;
    return LNBNN_OK;
}

// ===========================================================================
// classify
// ===========================================================================
int lnbnn::validate_classify(const lnbnn_index *ix, const void *queries, int dtype, const int64_t *off,
                             int32_t n_images, int32_t k, int mode, uint32_t flags, bool has_out_class,
                             const int32_t *nbr_idx, const float *nbr_dist)
{
    if (!ix) return set_err(LNBNN_EINVAL, "NULL index");
    if (!off || !has_out_class) return set_err(LNBNN_EINVAL, "NULL img_offsets or out_class");
    if (n_images < 0) return set_err(LNBNN_EINVAL, "n_images < 0");
    if (flags & ~(uint32_t)(LNBNN_DEVICE_PTRS | LNBNN_PER_IMAGE_LAUNCH | LNBNN_NO_GRAPH | LNBNN_TIMING))
        return set_err(LNBNN_EINVAL, "unknown flags 0x%x", flags);
    if (mode < 0 || mode >= kNumModes || !(ix->modes & LNBNN_MODE_BIT(mode)))
        return set_err(LNBNN_EINVAL, "mode %d is not materialised in this index", mode);
    const int want = is_fp8_mode(mode) ? LNBNN_F32 : LNBNN_U8;
    if (dtype != want) return set_err(LNBNN_EINVAL, "dtype %d does not match mode %d", dtype, mode);
    if (k < 1 || k > LNBNN_MAX_K) return set_err(LNBNN_EINVAL, "k = %d outside [1, %d]", k, LNBNN_MAX_K);
    if ((int64_t)k + 1 > ix->n_refs) return set_err(LNBNN_EINVAL, "k + 1 > n_refs");
    if (mode == LNBNN_NBNN_I8 && (nbr_idx || nbr_dist))
        return set_err(LNBNN_EINVAL, "the original NBNN mode returns no neighbour lists");
    if (is_fp8_mode(mode)) {
        if (k > kMaxFp8K) return set_err(LNBNN_EINVAL, "FP8 re-rank mode needs k <= %d", kMaxFp8K);
        if ((int64_t)fp8_candidates(k) > ix->n_refs) return set_err(LNBNN_EINVAL, "4k > n_refs");
    }
    if ((nbr_idx == nullptr) != (nbr_dist == nullptr))
        return set_err(LNBNN_EINVAL, "out_nbr_idx and out_nbr_dist must both be set or both NULL");
    if (off[0] != 0) return set_err(LNBNN_EINVAL, "img_offsets[0] must be 0");
    for (int32_t m = 0; m < n_images; ++m)
        if (off[m + 1] < off[m]) return set_err(LNBNN_EINVAL, "img_offsets decrease at %d", m);
    if (off[n_images] > 0 && !queries) return set_err(LNBNN_EINVAL, "NULL queries");
    return LNBNN_OK;
}

GraphKey lnbnn::graph_key(const Plan &p, const BatchIO &io)
{
    auto at = [](const void *x) { return (int64_t)(uintptr_t)x; };
    return GraphKey{wait_spin_limit(), p.variant, p.fmt * 1000 + p.kpb, p.n_lists, p.chunk_tiles, p.grid, io.q_cap,
                    io.img_cap, io.k, io.mode, at(io.offsets), at(io.bd), at(io.part_d), at(io.part_i), at(io.q8),
                    at(io.cand)};
}

// Replay (capturing on first use) the launch sequence of a batch.  The
// caller has made sure that no earlier replay of these graphs is still in
// flight when an entry is evicted (the workspace's work is ordered on one
// fence, and eviction waits for it).
int lnbnn::launch_graph(std::map<GraphKey, GraphEntry> &graphs, uint64_t &clock, lnbnn_index *ix, const Plan &p,
                        const BatchIO &io, hipStream_t s)
{
    const GraphKey key = graph_key(p, io);
    auto it = graphs.find(key);
    if (it == graphs.end()) {
        if (graphs.size() >= kMaxGraphs) {
            auto lru = graphs.begin();
            for (auto g = graphs.begin(); g != graphs.end(); ++g)
                if (g->second.last_use < lru->second.last_use) lru = g;
            if (lru->second.exec) LN_HIP(hipGraphExecDestroy(lru->second.exec));
            graphs.erase(lru);
        }
        GraphEntry g;
        LN_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        int rc = enqueue_batch(ix, p, io, s, nullptr);
        hipGraph_t graph = nullptr;
        hipError_t e = hipStreamEndCapture(s, &graph);
        if (rc) {
            if (graph) (void)hipGraphDestroy(graph);
            return rc;
        }
        if (e != hipSuccess) return hip_err(e, "hipStreamEndCapture");
        e = hipGraphInstantiate(&g.exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) return hip_err(e, "hipGraphInstantiate");
        log_line("graph captured: mode %d, k %d, %s, %d slices, chunk %d tiles, grid %d, capacity %lld descriptors / "
                 "%lld images (%zu cached)", io.mode, io.k, variant_name(p.variant), p.n_slices, p.chunk_tiles, p.grid,
                 (long long)io.q_cap, (long long)io.img_cap, graphs.size() + 1);
        it = graphs.emplace(key, g).first;
    }
    it->second.last_use = ++clock;
    LN_HIP(hipGraphLaunch(it->second.exec, s));
    return LNBNN_OK;
}

// The plain per-image form: one launch sequence per image, each planned for
// that image alone (no graph).  With `kev`, the distance-kernel time of every
// launch is summed.
static int classify_per_image(lnbnn_index *ix, const void *dq, const int64_t *off, int32_t n_images,
                              int32_t k, int mode, int32_t *cls, void *totals, int32_t *nbr_idx, float *nbr_dist,
                              hipStream_t s, hipEvent_t *kev)
{
    Workspace &ws = ix->ws;
    const int kp = k + 1;
    std::vector<Plan> plans(n_images);
    for (int32_t m = 0; m < n_images; ++m) {
        const int64_t nm = off[m + 1] - off[m];
        int rc = make_plan(ix, mode, k, std::max<int64_t>(1, nm), nm, kSplitLists, &plans[m]);
        if (rc) return rc;
    }
    const int64_t rb = row_bytes(ix->dtype, ix->dim);
    std::vector<BatchDesc> bds(n_images);
    std::vector<int64_t> offs(2 * (size_t)n_images);
    for (int32_t m = 0; m < n_images; ++m) {
        bds[m].n_q = off[m + 1] - off[m];
        bds[m].n_img = 1;
        bds[m].q = static_cast<const uint8_t *>(dq) + off[m] * rb;
        bds[m].cls = cls + m;
        bds[m].nbr_idx = nbr_idx ? nbr_idx + off[m] * kp : nullptr;
        bds[m].nbr_dist = nbr_dist ? nbr_dist + off[m] * kp : nullptr;
        bds[m].walk = plans[m].walk;
        bds[m].totals = static_cast<uint8_t *>(totals) + (int64_t)m * ix->n_classes * 8;
        offs[2 * m] = 0;
        offs[2 * m + 1] = bds[m].n_q;
    }
    LN_HIP(hipMemcpyAsync(ws.bd, bds.data(), n_images * sizeof(BatchDesc), hipMemcpyHostToDevice, s));
    LN_HIP(hipMemcpyAsync(ws.offsets, offs.data(), offs.size() * 8, hipMemcpyHostToDevice, s));
    if (!is_fp8_mode(mode) && mode != LNBNN_NBNN_I8)
        LN_HIP(launch_fill_u64(static_cast<unsigned long long *>(totals), (int64_t)n_images * ix->n_classes, s));
    double kms = 0;
    for (int32_t m = 0; m < n_images; ++m) {
        BatchIO io;
        io.offsets = ws.offsets + 2 * m;
        io.bd = ws.bd + m;
        io.q_cap = plans[m].q_cap;
        io.img_cap = 1;
        io.k = k;
        io.mode = mode;
        io.ws = &ws;
        io.part_d = ws.part_d;
        io.part_i = ws.part_i;
        io.q8 = ws.q8;
        io.qsc = ws.qsc;
        io.cand = ws.cand;
        io.upd_cls = ws.upd_cls;
        io.upd_delta = ws.upd_delta;
        int rc = enqueue_batch(ix, plans[m], io, s, kev);
        if (rc) return rc;
        if (kev) {
            LN_HIP(hipEventSynchronize(kev[1]));
            float ms = 0;
            LN_HIP(hipEventElapsedTime(&ms, kev[0], kev[1]));
            kms += ms;
        }
    }
    if (kev) {
        ix->last_timing.dist_kernel_ms = kms;
        ix->last_timing.dist_launches = n_images;
    }
    return LNBNN_OK;
}

extern "C" int lnbnn_classify(lnbnn_index *ix, const void *queries, int dtype, const int64_t *img_offsets,
                              int32_t n_images, int32_t k, int mode, uint32_t flags, int32_t *out_class,
                              void *out_totals, int32_t *out_nbr_idx, float *out_nbr_dist, void *stream)
{
    int rc = validate_classify(ix, queries, dtype, img_offsets, n_images, k, mode, flags, out_class != nullptr,
                               out_nbr_idx, out_nbr_dist);
    if (rc) return rc;
    if (n_images == 0) return LNBNN_OK;
    std::lock_guard<std::mutex> lock(ix->mu);
    LN_HIP(hipSetDevice(ix->device));
    hipStream_t s = stream ? (hipStream_t)stream : ix->own_stream;
    const bool dev = flags & LNBNN_DEVICE_PTRS;
    const bool per_image = flags & LNBNN_PER_IMAGE_LAUNCH;
    const bool timed = flags & LNBNN_TIMING;
    const bool direct = (flags & LNBNN_NO_GRAPH) || timed;   // events inside a graph cannot be read back
    const int kp = k + 1;
    const bool fp8 = is_fp8_mode(mode);
    const int64_t n_q = img_offsets[n_images];
    const int64_t rb = row_bytes(dtype, ix->dim);
    const int64_t nc = ix->n_classes;

    // Capacities: a batched call is planned for power-of-two buckets of its
    // descriptor and image counts, so one captured graph serves every batch
    // up to the bucket (the data pointers travel in the batch descriptor).
    Plan plan;
    int64_t part = 0, q_max = 1, q_cap = 1, img_cap = n_images;
    if (per_image) {
        for (int32_t m = 0; m < n_images; ++m) {
            Plan pm;
            const int64_t nm = std::max<int64_t>(1, img_offsets[m + 1] - img_offsets[m]);
            if ((rc = make_plan(ix, mode, k, nm, img_offsets[m + 1] - img_offsets[m], kSplitLists, &pm))) return rc;
            part = std::max(part, batch_elems(ix, pm, pm.q_cap));
            q_max = std::max(q_max, nm);
        }
        q_cap = std::max<int64_t>(1, n_q);
    } else {
        q_cap = cap_bucket(n_q, 1024);
        img_cap = cap_bucket(n_images, 8);
        if ((rc = make_plan(ix, mode, k, q_cap, n_q, kSplitLists, &plan))) return rc;
        part = work_elems(ix, plan, plan.q_cap);
        q_max = plan.q_cap;
    }
    const bool want_nbr = out_nbr_idx != nullptr;
    if ((rc = ensure_ws(ix, ix->ws, q_cap, img_cap, part, (want_nbr && !dev) ? n_q * kp : 0, dev ? 0 : n_q * rb,
                        fp8)))
        return rc;
    if (fp8 && (rc = ensure_fp8_ws(ix, ix->ws, q_max, fp8_candidates(k), k))) return rc;
    Workspace &ws = ix->ws;

    // the shared workspace may still be read by a call on another stream
    if ((rc = ws_order(ix, s))) return rc;
    // from here on, every exit (errors included) marks the end of this
    // call's use of the workspace on `s`
    struct WsFence {
        lnbnn_index *ix;
        hipStream_t s;
        bool armed;
        ~WsFence()
        {
            if (armed) (void)ws_mark(ix, s);
        }
    } fence{ix, s, true};
    const void *dq = queries;
    if (!dev && n_q > 0) {
        LN_HIP(hipMemcpyAsync(ws.q, queries, (size_t)(n_q * rb), hipMemcpyHostToDevice, s));
        dq = ws.q;
    }
    int32_t *d_cls = dev ? out_class : ws.cls;
    int32_t *d_nbr_i = want_nbr ? (dev ? out_nbr_idx : ws.nbr_idx) : nullptr;
    float *d_nbr_d = want_nbr ? (dev ? out_nbr_dist : ws.nbr_dist) : nullptr;
    // totals go straight to an aligned device buffer of the caller's
    void *ws_tot = fp8 ? (void *)ws.totals_f64 : (void *)ws.totals;
    void *d_tot = dev && out_totals && (uintptr_t)out_totals % 8 == 0 ? out_totals : ws_tot;

    hipEvent_t *kev = timed ? ix->tev : nullptr;
    if (timed) LN_HIP(hipEventRecord(ix->tev[2], s));
    if (per_image) {
        rc = classify_per_image(ix, dq, img_offsets, n_images, k, mode, d_cls, d_tot, d_nbr_i, d_nbr_d, s, kev);
        if (rc) return rc;
    } else {
        const BatchDesc hb{n_q, n_images, dq, d_cls, d_nbr_i, d_nbr_d, d_tot, plan.walk};
        if ((rc = begin_batch(ix, mode, hb, img_offsets, ws.bd, ws.offsets, nullptr, s))) return rc;
        BatchIO io;
        io.offsets = ws.offsets;
        io.bd = ws.bd;
        io.q_cap = plan.q_cap;
        io.img_cap = img_cap;
        io.k = k;
        io.mode = mode;
        io.ws = &ws;
        io.part_d = ws.part_d;
        io.part_i = ws.part_i;
        io.q8 = ws.q8;
        io.qsc = ws.qsc;
        io.cand = ws.cand;
        io.upd_cls = ws.upd_cls;
        io.upd_delta = ws.upd_delta;
        if (direct) {
            if ((rc = enqueue_batch(ix, plan, io, s, kev))) return rc;
        } else {
            if (ix->graphs.size() >= kMaxGraphs && !ix->graphs.count(graph_key(plan, io)) && (rc = ws_sync(ix)))
                return rc;                                  // an eviction: no replay in flight
            if ((rc = launch_graph(ix->graphs, ix->graph_clock, ix, plan, io, s))) return rc;
        }
    }
    if (timed) LN_HIP(hipEventRecord(ix->tev[3], s));

    // outputs
    if (out_totals && d_tot != out_totals)
        LN_HIP(hipMemcpyAsync(out_totals, ws_tot, (size_t)(n_images * nc * 8),
                              dev ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, s));
    if (!dev) {
        LN_HIP(hipMemcpyAsync(out_class, ws.cls, (size_t)n_images * 4, hipMemcpyDeviceToHost, s));
        if (want_nbr) {
            LN_HIP(hipMemcpyAsync(out_nbr_idx, ws.nbr_idx, (size_t)(n_q * kp * 4), hipMemcpyDeviceToHost, s));
            LN_HIP(hipMemcpyAsync(out_nbr_dist, ws.nbr_dist, (size_t)(n_q * kp * 4), hipMemcpyDeviceToHost, s));
        }
    }
    fence.armed = false;
    LN_HIP(ws_mark(ix, s));
    if (!dev) LN_HIP(hipStreamSynchronize(s));
    if (timed) {
        LN_HIP(hipEventSynchronize(ix->tev[3]));
        float ms = 0;
        if (!per_image) {
            LN_HIP(hipEventElapsedTime(&ms, ix->tev[0], ix->tev[1]));
            ix->last_timing.dist_kernel_ms = ms;
            ix->last_timing.dist_launches = 1;
        }
        LN_HIP(hipEventElapsedTime(&ms, ix->tev[2], ix->tev[3]));
        ix->last_timing.total_ms = ms;
        ix->last_timing.slices = per_image ? 0 : plan.n_slices;
        ix->last_timing.tile_variant = per_image ? -1 : plan.variant;
        ix->has_timing = true;
    }
    // a completed sequence (host pointers, or a timed call) reports a
    // bounded wait that gave up
    if (!dev || timed) return status_check(ws);
    return LNBNN_OK;
}

extern "C" int lnbnn_sync_status(lnbnn_index *ix)
{
    if (!ix) return set_err(LNBNN_EINVAL, "NULL index");
    std::lock_guard<std::mutex> lock(ix->mu);
    LN_HIP(hipSetDevice(ix->device));
    if (!ix->ws.h_status) return LNBNN_OK;
    const int rc = ws_sync(ix);
    if (rc) return rc;
    return status_check(ix->ws);
}

extern "C" int lnbnn_last_timing(const lnbnn_index *ix, lnbnn_timing *out)
{
    if (!ix || !out) return set_err(LNBNN_EINVAL, "NULL argument");
    if (!ix->has_timing) return set_err(LNBNN_EINVAL, "no timed classify has run on this index");
    *out = ix->last_timing;
    return LNBNN_OK;
}

// ===========================================================================
// variants and autotuner
// ===========================================================================
extern "C" int32_t lnbnn_num_variants(void) { return num_variants(); }
extern "C" const char *lnbnn_variant_name(int32_t v) { return variant_name(v); }

extern "C" int lnbnn_set_tuning(lnbnn_index *ix, int mode, int32_t k, const lnbnn_tuning *t)
{
    if (!ix || !t) return set_err(LNBNN_EINVAL, "NULL argument");
    if (mode < 0 || mode >= kNumModes || !(ix->modes & LNBNN_MODE_BIT(mode))) return set_err(LNBNN_EINVAL, "bad mode");
    if (k < 1 || k > LNBNN_MAX_K) return set_err(LNBNN_EINVAL, "bad k");
    if (t->chunk_tiles < 0 || t->chunk_tiles % 8 != 0) return set_err(LNBNN_EINVAL, "chunk_tiles must be a multiple of 8");
    if (t->max_workgroups < 0) return set_err(LNBNN_EINVAL, "negative max_workgroups");
    const int fmt = index_fmt(ix, mode);
    const int list_len = dist_list_len(mode, k);
    const int kpb = kp_bucket(list_len, fmt);
    if (kpb == 0) return set_err(LNBNN_EINVAL, "k = %d is not supported by mode %d", k, mode);
    if (t->variant >= 0 && !variant_serves(t->variant, mode, fmt, list_len))
        return set_err(LNBNN_EINVAL, "variant %d cannot serve k = %d", t->variant, k);
    std::lock_guard<std::mutex> lock(ix->plan_mu);
    if (t->variant < 0 && t->chunk_tiles == 0 && t->max_workgroups == 0)
        ix->pinned.erase({mode, kpb});
    else
        ix->pinned[{mode, kpb}] = lnbnn_index::Pin{*t, 0};
    return LNBNN_OK;
}

extern "C" int lnbnn_set_variant(lnbnn_index *ix, int mode, int32_t k, int32_t v)
{
    lnbnn_tuning t{v < 0 ? -1 : v, 0, 0};
    return lnbnn_set_tuning(ix, mode, k, &t);
}

// Flat JSON object of string -> integer, the tuning cache format.
static std::map<std::string, int> read_cache(const char *path)
{
    std::map<std::string, int> m;
    std::ifstream f(path);
    if (!f) return m;
    std::stringstream ss;
    ss << f.rdbuf();
    const std::string s = ss.str();
    size_t i = 0;
    while ((i = s.find('"', i)) != std::string::npos) {
        const size_t j = s.find('"', i + 1);
        if (j == std::string::npos) break;
        const std::string key = s.substr(i + 1, j - i - 1);
        const size_t c = s.find(':', j);
        if (c == std::string::npos) break;
        m[key] = atoi(s.c_str() + c + 1);
        i = s.find_first_of(",}", c);
        if (i == std::string::npos) break;
    }
    return m;
}

static void write_cache(const char *path, const std::map<std::string, int> &m)
{
    const std::string tmp = std::string(path) + ".tmp";
    std::ofstream f(tmp);
    f << "{\n";
    size_t n = 0;
    for (auto &kv : m) f << "  \"" << kv.first << "\": " << kv.second << (++n < m.size() ? ",\n" : "\n");
    f << "}\n";
    f.close();
    std::rename(tmp.c_str(), path);
}

extern "C" int lnbnn_autotune(lnbnn_index *ix, const void *queries_dev, int dtype, const int64_t *img_offsets,
                              int32_t n_images, int32_t k, int mode, const char *cache_path,
                              int32_t *best_variant, void *stream)
{
    int rc = validate_classify(ix, queries_dev, dtype, img_offsets, n_images, k, mode, LNBNN_DEVICE_PTRS, true,
                               nullptr, nullptr);
    if (rc) return rc;
    if (!cache_path) {
        const char *e = getenv("LNBNN_TUNE_CACHE");
        if (e && *e) cache_path = e;
    }
    const int fmt = index_fmt(ix, mode);
    const int kpb = kp_bucket(dist_list_len(mode, k), fmt);
    // the setting holds for plans within 8x of this batch's capacity bucket:
    // the fastest shape for a full batch is not the fastest for serving-size
    // batches, which keep the defaults
    const int64_t min_q = cap_bucket(std::max<int64_t>(img_offsets[n_images], 1), 1024) / 8;
    char arch[64] = "gfx";
    {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, ix->device) == hipSuccess) snprintf(arch, sizeof arch, "%s", prop.gcnArchName);
    }
    std::ostringstream key;
    key << "arch=" << arch << ",n_refs=" << ix->n_refs << ",dim=" << ix->dim << ",kp=" << kpb << ",mode=" << mode;
    if (cache_path) {
        auto m = read_cache(cache_path);
        auto it = m.find(key.str());
        // cache value: variant | chunk_tiles << 8 (chunk 0 = whole slice)
        const int cv = it != m.end() ? it->second & 0xff : -1;
        const int cc = it != m.end() ? it->second >> 8 : 0;
        if (it != m.end() && variant_serves(cv, mode, fmt, dist_list_len(mode, k)) && cc >= 0 && cc % 8 == 0) {
            {
                std::lock_guard<std::mutex> lock(ix->plan_mu);
                ix->pinned[{mode, kpb}] = lnbnn_index::Pin{lnbnn_tuning{cv, cc, 0}, min_q};
            }
            if (best_variant) *best_variant = cv;
            log_line("tuner: cache hit %s -> %s, chunk %d", key.str().c_str(), variant_name(cv), cc);
            return LNBNN_OK;
        }
    }
    hipStream_t ts = stream ? (hipStream_t)stream : ix->own_stream;
    int32_t *d_cls = nullptr;
    // stream-ordered: freeing it does not synchronise the device
    LN_HIP(dmalloc_async((void **)&d_cls, std::max<int32_t>(1, n_images) * 4, ts));
    // time of the whole launch sequence with one (variant, chunk) setting: mean of
    // two runs after one warm-up run.  (Not the distance kernel's alone: shared
    // lists leave the rows of the best tiles to the kernel after it.)
    auto time_setting = [&](int v, int chunk, double *ms) {
        lnbnn_tuning t{v, chunk, 0};
        int r = lnbnn_set_tuning(ix, mode, k, &t);
        double tot = 0, dist = 0;
        for (int rep = 0; rep < 3 && !r; ++rep) {
            r = lnbnn_classify(ix, queries_dev, dtype, img_offsets, n_images, k, mode,
                               LNBNN_DEVICE_PTRS | LNBNN_NO_GRAPH | LNBNN_TIMING, d_cls, nullptr, nullptr, nullptr,
                               stream);
            if (!r && rep > 0) {
                tot += ix->last_timing.total_ms;
                dist += ix->last_timing.dist_kernel_ms;
            }
        }
        *ms = tot / 2;
        if (!r)
            log_line("tuner: mode %d, k %d: %s, chunk %d: %.2f ms, distance kernel %.2f ms", mode, k, variant_name(v),
                     chunk, *ms, dist / 2);
        return r;
    };
    // every variant with whole-slice sweeps, then chunk lengths (chunk-major
    // walk: the workgroups of an XCD sweep the same references together) for
    // the two fastest variants
    std::vector<std::pair<double, int>> by_variant;
    const int list_len = dist_list_len(mode, k);
    for (int v = 0; v < num_variants() && !rc; ++v) {
        if (!variant_serves(v, mode, fmt, list_len)) continue;
        double ms = 0;
        if (!(rc = time_setting(v, 0, &ms))) by_variant.push_back({ms, v});
    }
    std::sort(by_variant.begin(), by_variant.end());
    int best = by_variant.empty() ? -1 : by_variant[0].second, best_chunk = 0;
    double best_ms = by_variant.empty() ? 1e30 : by_variant[0].first;
    for (size_t i = 0; i < by_variant.size() && i < 2 && !rc; ++i) {
        for (int chunk : {2048, 4096, 8192}) {
            double ms = 0;
            if ((rc = time_setting(by_variant[i].second, chunk, &ms))) break;
            if (ms < best_ms) {
                best_ms = ms;
                best = by_variant[i].second;
                best_chunk = chunk;
            }
        }
    }
    (void)hipFreeAsync(d_cls, ts);
    if (rc || best < 0) {
        lnbnn_set_variant(ix, mode, k, -1);
        return rc ? rc : set_err(LNBNN_EINVAL, "no variant can serve mode %d with k = %d", mode, k);
    }
    {
        std::lock_guard<std::mutex> lock(ix->plan_mu);
        ix->pinned[{mode, kpb}] = lnbnn_index::Pin{lnbnn_tuning{best, best_chunk, 0}, min_q};
    }
    if (best_variant) *best_variant = best;
    log_line("tuner: %s -> %s, chunk %d (%.2f ms; %zu variants timed)", key.str().c_str(), variant_name(best),
             best_chunk, best_ms, by_variant.size());
    if (cache_path) {
        auto m = read_cache(cache_path);
        m[key.str()] = best | (best_chunk << 8);
        write_cache(cache_path, m);
    }
    return LNBNN_OK;
}

extern "C" const char *lnbnn_last_error(void) { return g_err.c_str(); }
