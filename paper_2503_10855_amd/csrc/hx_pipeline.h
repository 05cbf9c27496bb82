// hx_pipeline.h -- host-side state behind the hx_pipeline handle.
// Internal to libhx.so.
#pragma once

#include <hip/hip_runtime.h>

#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/hx.h"
#include "hx_kernels.h"

namespace hx {

// Thread-local error text behind hx_last_error().
void set_error(const char* fmt, ...);
hx_status fail(hx_status st, const char* fmt, ...);
// The scheduling language (hx_sched.cpp): text -> schedule, and back.
hx_status compile_schedule(const char* text, hx_schedule* out);
std::string schedule_text(const hx_schedule& s);
hx_status hip_fail(hipError_t e, const char* what);

// Diagnostics (hx_log.cpp): HX_LOG=<level> prints lines of at most that
// level to stderr; HX_TRACE=1 turns TraceRange into a roctx range.
int log_level();
void logf(int level, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
struct TraceRange {
    bool on;
    explicit TraceRange(const char* name);
    ~TraceRange();
    TraceRange(const TraceRange&) = delete;
    TraceRange& operator=(const TraceRange&) = delete;
};

// Make `dev` current for the lifetime of the guard.
struct DeviceGuard {
    int prev = -1, dev;
    explicit DeviceGuard(int d) : dev(d) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) (void)hipSetDevice(dev);
    }
    ~DeviceGuard() {
        if (prev >= 0 && prev != dev) (void)hipSetDevice(prev);
    }
};

// A device or pinned host buffer of the pipeline.  Every one is allocated
// by hx_pipeline_create (alloc) and released by hx_pipeline_destroy; no
// call path allocates.  Allocations are counted on the owning pipeline's
// MemStats.
struct MemStats {
    size_t device_bytes = 0, pinned_bytes = 0;
    uint64_t allocations = 0;
};
struct DevBuf {
    void* ptr = nullptr;
    size_t bytes = 0;
    hipError_t alloc(size_t n, MemStats& m);
    void release();
};
struct HostBuf {
    void* ptr = nullptr;
    size_t bytes = 0;
    hipError_t alloc(size_t n, MemStats& m);
    void release();
};

// Capacities of one batch context, fixed at creation.
struct BatchCaps {
    int64_t items1 = 0, items2 = 0, items0 = 0;  // work items per pass
    int64_t list_entries = 0;                    // SPECULATE listing
    int64_t ways = 0;        // words of max slots, and of bounds
    int32_t slot_step = 1;   // words between max slots (8 B between bounds)
    size_t table_bytes = 0;
    int64_t code_elems = 0;                      // STORE code plane (0: none)
};

// Resources of one in-flight batched launch.  Batched calls pick one of a
// few of these so launches on different streams never share scratch.
struct BatchContext {
    bool ready = false;
    DevBuf table;               // device descriptor table
    HostBuf h_table;            // pinned staging copy of the table
    DevBuf state;               // the small arrays, SPECULATE's bounds and epoch first
    uint32_t* slots = nullptr;  // in state: two sets of BatchCaps::ways max slots
    uint32_t* cand_n = nullptr; // SPECULATE: entries each tile listed
    int32_t* redo = nullptr;    // SPECULATE: tiles whose lists overflowed
    DevBuf code;                // pass-1 store buffer (STORE batches)
    DevBuf cand_code, cand_row; // SPECULATE: listed pixels
    hipEvent_t ev_done = nullptr;
    hipEvent_t ev_prev = nullptr;   // of an earlier call
    hipEvent_t ev_t[5] = {};    // timing mode
    bool in_flight = false;
    // A call recorded into a graph reads this context's table and scratch at
    // every replay: no other call may ever use them.
    bool recorded = false;
    uint64_t last_use = 0;      // the pipeline's call counter at the last use
    // Leading words of each set of max slots that a call may have left
    // non-zero, and those the table's images use.
    int32_t dirty[2] = {0, 0};
    int32_t n_ways = 0;
    int64_t n_items[3] = {0, 0, 0};  // the table's items of pass 0, 1, 2
    // The call whose table the device copy holds: a repeat of the same
    // batch (same descriptors, outputs and pass mode) reuses it as is.
    std::vector<hx_image> last_imgs;
    float* last_dmax = nullptr;
    int last_pass = -1;
    int last_ty = 0, last_c = 0;
    bool default_ty = false;   // last_ty was the default for these images
};

// A batch's class for the batch autotuner: floor(log2) of its total
// pixels and of its image count.
struct BatchKey {
    int px, n;
    bool operator<(const BatchKey& o) const { return px != o.px ? px < o.px : n < o.n; }
};
BatchKey batch_key(const hx_image* imgs, int32_t n);
// The batched launch's schedule: rows per sweep tile, pass structure, and
// which of SPECULATE's two pass 2 kernels.
struct BatchChoice {
    int ty = 0;
    int pass = 0;
    int claim = 0;
};
// Tile heights the batched form accepts (multiples of 8 in [kBatchTyMin,
// kBatchTyMax]) and the ones the batch autotuner tries.
constexpr int kBatchTyMin = 16, kBatchTyMax = 256;

struct ShapeClass {
    int hb, wb;  // floor(log2(H)), floor(log2(W))
    bool operator<(const ShapeClass& o) const {
        return hb != o.hb ? hb < o.hb : wb < o.wb;
    }
};
ShapeClass shape_class(int64_t H, int64_t W);

}  // namespace hx

struct hx_pipeline {
    int device = 0;
    hx_params prm{};
    hx::Taps taps{};
    int cu_count = 0;
    hx::MemStats mem;

    bool forced = false;
    hx_schedule forced_sched{};
    std::map<hx::ShapeClass, hx_schedule> tuned;
    std::map<hx::BatchKey, hx::BatchChoice> batch_tuned;  // the batch autotuner's

    // Per-image scratch (forms IMAGE, STAGES, SRAD), one set shared by
    // every per-image call; plane_elems is each plane's capacity.
    int64_t plane_elems = 0;
    hx::DevBuf slot1;
    hx::DevBuf planeA;   // STORE code / B / SRAD's second J plane
    hx::DevBuf planeL;   // L / SRAD's c plane
    hx::DevBuf planeG2, planeZ, bufPart;
    hx::DevBuf srad_part;
    // Ordering of per-image calls on the shared scratch: each records the
    // event on its stream; a call on another stream waits for it first.
    // Calls recorded into a graph are ordered among those of one capture.
    struct ImgOrder {
        hipEvent_t ev = nullptr;
        hipStream_t stream = nullptr;
        bool used = false;
        unsigned long long capture = 0;   // the last call's (0: not recorded)
    };
    ImgOrder img_order, rec_order;
    // Scratch of the STORE forms: two max slots (each call uses one and
    // leaves the other at zero for the next call; next_zero says the
    // previous call did) and the code plane, and for blur sizes above 7 the
    // plane of B.
    struct ImgScratch {
        uint32_t* slots = nullptr;
        int parity = 0;
        bool next_zero = false;
        float* code = nullptr;
        float* blur = nullptr;
    };
    ImgScratch img_shared;
    // Of calls recorded into a graph, which run any number of times at any
    // point between the others: the shared planes, and one max slot that no
    // other call uses and each recorded call clears itself.
    ImgScratch img_rec;
    uint32_t* img_last_slot = nullptr;   // of the last call on img_shared or img_rec
    // A set of its own for STORE-form calls on one stream, the first that
    // makes one: no other stream's call ever uses it, so its calls are
    // ordered by their stream alone and record no event (one costs about 3
    // of the 17 us of a 1080p call).
    ImgScratch img_own;
    hx::DevBuf planeOwn, planeOwnB;
    hipStream_t own_stream = nullptr;
    bool own_taken = false;

    // Batched launches.
    static constexpr int kMaxContexts = 8;
    int n_ctx = 0;
    hx::BatchCaps caps;
    hx::BatchContext ctx[kMaxContexts];
    uint64_t use_clock = 0;
    std::mutex batch_mu;  // guards context choice (the server calls from
                          // its own thread)
    bool timing = false;
    int last_timed_ctx = -1;
};

namespace hx {

// The schedule a call on an H x W image uses (forced > tuned > default),
// with the pipeline's fixed knobs applied.
hx_schedule choose_schedule(const hx_pipeline* p, int64_t H, int64_t W);
hx_status validate_schedule(const hx_pipeline* p, const hx_schedule& s);
hx_status validate_image(const hx_pipeline* p, const hx_image* img);

// The per-image form with an explicit schedule (used by hx_edge_detect
// and the autotuner): on the private scratch if the stream owns it (may_own:
// or takes it), else on the shared one after the previous call there.
hx_status run_image_ordered(hx_pipeline* p, const hx_image* img, float* d_max,
                            const hx_schedule& s, hipStream_t stream, bool may_own = true);
// Pass structure of batched calls unless one is fixed: SPECULATE reads
// the input about 1.1 times (once, plus the sampled bands) and measured
// fastest on the 64 x 1920x1080 batch (0.186 ms a call against 0.288 ms
// for RECOMPUTE and 0.387 ms for STORE).
constexpr int kBatchPass = HX_PASS_SPECULATE;

// The batched form.  pass_mode / ty 0: the batch autotuner's choice for
// the batch's class, else SPECULATE / the default tile height.  ctx >= 0
// runs on that batch context (waiting for its previous batch) instead of
// the one the context policy picks; the batch autotuner uses it to keep
// one batch in flight per context.  A call recorded into a graph keeps its
// context for good; when only one is left for the calls that run at once, it
// runs image by image without one.  count: timing mode applies to it.
// claim: BatchChoice's, -1 the tuned one (else 0).
hx_status run_batched(hx_pipeline* p, const hx_image* imgs, int32_t n,
                      float* d_max, int pass_mode, int ty, hipStream_t stream,
                      int ctx = -1, bool count = true, int claim = -1);
// Contexts that no recorded call holds.
int free_contexts(const hx_pipeline* p);
// Wait for a context's last launch.
hx_status ctx_wait(BatchContext& c);

}  // namespace hx
