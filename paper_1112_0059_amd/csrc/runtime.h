// Host runtime shared by the classify path and the serving loop.
#pragma once

#include <array>
#include <atomic>
#include <condition_variable>
#include <cstdarg>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <tuple>
#include <unordered_map>
#include <vector>

#include "../../include/lnbnn.h"
#include "internal.h"

namespace lnbnn {

int set_err(int code, const char *fmt, ...);
int hip_err(hipError_t e, const char *what);
bool fault_injected(const char *site);
bool log_enabled();
void log_line(const char *fmt, ...) __attribute__((format(printf, 1, 2)));

#define LN_HIP(expr)                                   \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return hip_err(e_, #expr); \
    } while (0)

// Device buffers for one batch in flight.  Capacities only grow.
struct Workspace {
    int64_t q_cap = 0;          // query descriptors
    int64_t img_cap = 0;        // images
    int64_t part_cap = 0;       // elements of part_d / part_i
    int64_t nbr_cap = 0;        // elements of nbr_idx / nbr_dist
    int64_t qbytes_cap = 0;     // bytes of staged queries
    void *q = nullptr;
    int64_t *offsets = nullptr;
    BatchDesc *bd = nullptr;
    float *part_d = nullptr;
    int32_t *part_i = nullptr;
    unsigned long long *totals = nullptr;
    double *totals_f64 = nullptr;
    int32_t *cls = nullptr;
    int32_t *nbr_idx = nullptr;
    float *nbr_dist = nullptr;
    // FP8 mode
    int64_t q8_cap = 0;         // queries
    int64_t cand_cap = 0;       // elements of cand
    int64_t upd_cap = 0;        // elements of upd_cls / upd_delta
    uint4 *q8 = nullptr;        // [q8_cap, 8] FP8 codes
    int32_t *qsc = nullptr;     // [q8_cap] E8M0 query scales
    int32_t *cand = nullptr;
    int32_t *upd_cls = nullptr;
    double *upd_delta = nullptr;
    // status word of the launch sequences run on this workspace
    // (kStatusWaitGaveUp: a bounded stage wait gave up): pinned host memory,
    // and its device address
    int32_t *status = nullptr;
    int32_t *h_status = nullptr;
    int device = 0;
    ~Workspace();
    int64_t bytes() const;
};

struct Plan {
    int variant = 0;
    int fmt = 0;
    int kpb = 0;                // compiled list length
    bool pl = false;            // shared lists (of tiles)
    int n_slices = 1;           // most pieces a query block's sweep is cut into
    int n_lists = 2;            // one list per lane group: n_slices * lists per slice
    Walk walk{};                // the split, chosen for the batch's own size
    int block = 0;              // queries per block
    int grid = 1;
    int max_lists = 0;          // shared lists: most partial lists per query
    int64_t lists = 0;          // shared lists: partial lists this batch uses
    int chunk_tiles = 8;        // tiles per chunk of the chunk-major walk
    int64_t q_cap = 0;          // capacity the plan (and part buffers) serve
};

// Partial lists per query a shared-list plan may split into: one per
// workgroup of a full grid where a call's own workspace holds them, and as
// many as the one-list-per-lane-group plans where buffers are sized for
// those (the serving slots' share of the budget).
constexpr int kSplitLists = 256;

// Everything a batch launch sequence needs; pointers are device pointers.
struct BatchIO {
    const Workspace *ws = nullptr;      // owner of the buffers below (capacity checks)
    const int64_t *offsets = nullptr;
    const BatchDesc *bd = nullptr;
    int64_t q_cap = 0;
    int64_t img_cap = 0;
    int32_t k = 0;
    int mode = 0;
    float *part_d = nullptr;
    int32_t *part_i = nullptr;
    // FP8 mode
    uint4 *q8 = nullptr;
    int32_t *qsc = nullptr;
    int32_t *cand = nullptr;
    int32_t *upd_cls = nullptr;
    double *upd_delta = nullptr;
};

// What a captured sequence depends on: the plan, the capacities, the
// workspace buffers and the stage-wait bound (all kernel arguments frozen into
// it).  The caller's queries and outputs, and the batch's own split, travel in
// the batch descriptor.
using GraphKey = std::array<int64_t, 16>;

struct GraphEntry {
    hipGraphExec_t exec = nullptr;
    uint64_t last_use = 0;       // LRU stamp
};

// Captured launch sequences of one workspace, keyed by plan and capacity
// bucket (never by the caller's data pointers, which travel in the batch
// descriptor); at most kMaxGraphs are kept, the least recently used is
// destroyed first.
constexpr size_t kMaxGraphs = 8;

struct Server;

}  // namespace lnbnn

struct lnbnn_index {
    int device = 0;
    int dtype = 0;
    int dim = lnbnn::kDim;          // 128, or 160 (location-augmented, INT8 mode only)
    int64_t n_refs = 0;
    int64_t n_pad = 0;
    int32_t n_classes = 0;
    uint32_t modes = 0;
    int64_t hbm_budget = 0;
    int cu_count = 0;
    hipStream_t own_stream = nullptr;

    uint4 *frag[lnbnn::kNumFmt] = {};
    float *seed[lnbnn::kNumFmt] = {};
    int32_t *labels = nullptr;
    float *ref_f32 = nullptr;       // FP8 mode: FP32 references for the re-rank
    int32_t *row_scale = nullptr;   // FP8 mode: E8M0 exponent of every padded row
    // INT8 mode: rows packed by the parity of ||r - 128||^2, the even ones
    // first; the reference of every packed row (-1: padding), and the first
    // tile of the odd ones
    int32_t *perm = nullptr;
    int32_t odd_tile0 = 0;
    // original NBNN mode: the class-sorted INT8 copy (each class's rows
    // grouped by the parity of ||r - 128||^2, every group padded to 256
    // rows), and 2 x class + parity of each of its tiles
    int32_t *tile_class = nullptr;
    int64_t rows[lnbnn::kNumFmt] = {};   // padded rows of each packed format
    int64_t device_bytes = 0;

    std::mutex mu;                                     // classify path (workspace, graphs)
    std::mutex plan_mu;                                // tuning and occupancy caches
    lnbnn::Workspace ws;
    // (mode, kp bucket) -> launch tuning, for plans of at least min_q queries'
    // capacity (a tuned setting holds for batches of the size it was timed on)
    struct Pin {
        lnbnn_tuning t;
        int64_t min_q;
    };
    std::map<std::pair<int, int>, Pin> pinned;
    std::map<std::tuple<int, int, int>, int> occupancy;  // (variant, fmt, kpb) -> blocks/CU
    std::map<lnbnn::GraphKey, lnbnn::GraphEntry> graphs;
    uint64_t graph_clock = 0;
    // device buffers replaced by a larger one: kept until the index is
    // freed, since work in flight (or a graph being captured elsewhere) may
    // still use them and hipFree would synchronise the whole device
    std::vector<void *> retired;
    std::mutex retired_mu;
    lnbnn_timing last_timing{};
    bool has_timing = false;
    hipEvent_t tev[4] = {nullptr, nullptr, nullptr, nullptr};
    // Last use of `ws`: on the index's own stream (which outlives it and runs
    // its work in order, so calls that stay on it need no event), or on a
    // caller's, marked by the event.
    enum class WsUse { none, own, event };
    WsUse ws_use = WsUse::none;
    hipEvent_t ws_free = nullptr;

    lnbnn::Server *server = nullptr;   // owned; created by the first submit, deleted by server_stop
    std::mutex server_mu;
};

namespace lnbnn {

// Argument checks shared by the classify entry points (no device call).
int validate_classify(const lnbnn_index *ix, const void *queries, int dtype, const int64_t *off, int32_t n_images,
                      int32_t k, int mode, uint32_t flags, bool has_out_class, const int32_t *nbr_idx,
                      const float *nbr_dist);
int mode_fmt(int mode);
bool is_fp8_mode(int mode);
int index_fmt(const lnbnn_index *ix, int mode);   // mode_fmt, with the 160-element INT8 tiles where they apply
// Plan for a batch of n_q queries in buffers of q_cap.  max_lists: most
// partial lists per query of a shared-list plan (1: no block is split, and no
// default shape keeps several lists per query where one would do).
int make_plan(lnbnn_index *ix, int mode, int k, int64_t q_cap, int64_t n_q, int max_lists, Plan *out);
// Elements of part_d / part_i the plan's batch needs (the lists, or the
// original NBNN mode's per-class minima), and the most that any batch of up to
// q_cap queries planned alike needs.
int64_t batch_elems(const lnbnn_index *ix, const Plan &p, int64_t q_cap);
int64_t work_elems(const lnbnn_index *ix, const Plan &p, int64_t q_cap);
// Hand a batch to the device: its descriptor and offsets into `dst` / `dst_off`
// and, for the exact modes, its totals cleared.  Precedes enqueue_batch (or the
// replay of its captured sequence) on the stream.
int begin_batch(const lnbnn_index *ix, int mode, const BatchDesc &bd, const int64_t *off, BatchDesc *dst,
                int64_t *dst_off, int32_t *status, hipStream_t s);
// Enqueue distance kernel + finish + argmin for one batch (the data
// pointers come from the batch descriptor io.bd).  When `kev` is not null,
// events 0/1 bracket the distance kernel.
int enqueue_batch(lnbnn_index *ix, const Plan &p, const BatchIO &io, hipStream_t s, hipEvent_t *kev);
// Bounded-wait spin limit for the distance kernel (LNBNN_WAIT_SPINS).
int32_t wait_spin_limit();
// After the workspace's sequences have completed: LNBNN_EDEVICE (and the
// status word cleared) if a bounded wait gave up.
int status_check(Workspace &ws);
// Capacity bucket: the next power of two >= max(n, lo).
int64_t cap_bucket(int64_t n, int64_t lo);
int ensure_ws(lnbnn_index *ix, Workspace &ws, int64_t q_cap, int64_t img_cap, int64_t part,
              int64_t nbr, int64_t qbytes, bool need_f64);
int ensure_fp8_ws(lnbnn_index *ix, Workspace &ws, int64_t q_cap, int n_cand, int k);
int fp8_candidates(int k);
int dist_list_len(int mode, int k);
int64_t row_bytes(int dtype, int dim);

int launch_graph(std::map<GraphKey, GraphEntry> &graphs, uint64_t &clock, lnbnn_index *ix, const Plan &p,
                 const BatchIO &io, hipStream_t s);
void drop_graphs(std::map<GraphKey, GraphEntry> &graphs);
GraphKey graph_key(const Plan &p, const BatchIO &io);

// Frees a device buffer that dmalloc gave out and no work uses any more: it is
// kept for the next allocation of its size, up to kKeptBytes per process (oldest
// freed first; all of it when an allocation fails, and in lnbnn_trim).  An index that is
// rebuilt again and again would otherwise outrun the driver, which wipes freed
// memory at about 40 GB/s: 2.27M references rebuilt every 1.4 ms came to 8 ms
// and more a build once the wiped memory was used up.
constexpr size_t kKeptBytes = size_t(1) << 30;
void dfree(void *p);

// Streams of the indexes, kept when an index is freed and given to the next one
// on the device: as many as indexes ever lived at once.  They are never
// destroyed, because a caller's allocator may still order a buffer's reuse
// after the stream an index wrote it on.
int stream_acquire(int device, hipStream_t *out);
void stream_release(int device, hipStream_t s);

void server_stop(lnbnn_index *ix);
bool server_pending(lnbnn_index *ix);

}  // namespace lnbnn
