// dart_runtime.h -- host-side objects shared by the runtime and the server.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <mutex>
#include <utility>
#include <vector>

#include "../../include/dart.h"
#include "dart_internal.h"

namespace dart {
// Process-wide, never repeated: a stack created where a freed one lived, or
// re-laid, never matches a cached plan of another.
uint64_t next_generation();
}  // namespace dart

struct dart_stack {
    dart::StackDev dev{};
    dart_dtype storage = DART_F32;
    std::vector<double> times;
    std::vector<char> filled;
    uint64_t bytes = 0;
    uint64_t generation = dart::next_generation();  // renewed whenever the resident layout
                                                    // or data change
    int device = 0;
    dart_tuning tuning{32, 2, 8, 0, 1, 0, 4};
    bool interval = false;             // a streamed interval (marched in whole rays)
    bool placed = false;               // set by dart_stack_set_placement
    double origin[3] = {0, 0, 0}, centre[3] = {0, 0, 0};
    bool tuned = false;
    std::mutex mu;
    std::vector<std::pair<hipStream_t, hipEvent_t>> uses;  // last render per stream
    std::atomic<int> pinned{0};                            // server requests holding the stack
    // labelled stack: its sub-domains (owned by the caller) and their device
    // descriptors; a stack that is a sub-domain counts the labelled stacks
    // holding it in `refs`
    std::vector<dart_stack *> parts;
    dart::Block *dev_blocks = nullptr;
    std::atomic<int> refs{0};
    std::atomic<bool> rendered{false};       // (labelled) by a call before this one
    std::vector<const void *> block_planes;  // the sub-domains' planes in dev_blocks
    std::atomic<bool> planes_named{false};   // dev_blocks names every sub-domain's
    std::vector<dart_stack *> holders;       // labelled and vector stacks that hold this one
    bool labelled() const { return !parts.empty(); }
    // vector stack: its components (owned by the caller, counted in refs);
    // dev is component 0's
    std::vector<dart_stack *> comps;
    void *packed = nullptr;             // emissivity of components 1.., packed (device)
    std::vector<uint64_t> packed_gen;   // the components' generations when packed
    // emissivity plane (StackDev::jplane) of a plain stack: built
    // at the first render after the records change, when memory allows
    void *jplane = nullptr;
    uint64_t jplane_bytes = 0;
    // the generation it was packed from (0: never); read without the lock by
    // planners on other threads, so published after the pack has completed
    std::atomic<uint64_t> jplane_gen{0};
    std::vector<char> plane_ok;         // epochs whose elements are those of the records
    uint64_t jplane_no_room = 0;        // a generation for which hipMalloc failed
    // the plane's elements in pairs (F_PAIRS), for batches of a large 16-bit stack
    // that is rendered again and again; published like the plane
    void *pairs = nullptr;
    uint64_t pairs_bytes = 0;
    std::atomic<uint64_t> pairs_gen{0};
    uint64_t pairs_no_room = 0;
    uint64_t walked_gen = 0;            // the generation whose batches `walked` counts
    double walked = 0;                  // cells walked by them, as pairs_due estimates
    std::atomic<bool> tuning_now{false};  // (inside dart_autotune)
    bool vector() const { return !comps.empty(); }
    int channels() const { return comps.empty() ? 1 : (int)comps.size(); }
};

namespace dart {

dart_status fail(dart_status st, const char *fmt, ...);
dart_status hip_fail(hipError_t e, const char *what);
int device_cus(int dev);
uint32_t record_bytes(int store);
// dart_stack_create; rendered: the stack is rendered itself (a streamer's ring is not,
// and needs no emissivity plane).
dart_status create_stack(const int32_t dims[3], const double cell[3], int32_t n_epochs,
                         const double *epoch_times, dart_dtype storage, bool rendered,
                         dart_stack **out);
dart_status resolve_view(const dart_stack *s, const dart_view *v, RayView *rv);
// Packs the stack's emissivity plane when it is missing or stale (allocating it
// only if may_alloc); a stack without one is rendered from whole records.
dart_status refresh_jplane(const dart_stack *s, hipStream_t stream, bool may_alloc);
// Counts a batch's rays through the stack; whether its pairs are due, and packing them.
bool pairs_due(const dart_stack *s, double rays);
dart_status pack_pairs(const dart_stack *s, hipStream_t stream);
bool pairs_ready(const dart_stack *s);
// Rays of a view that pairs serve: views of one epoch per cell, of exact time, of
// whole records or of 64-bit plane addresses do not read them.
inline double view_rays(const dart_view &v) {
    const uint32_t other = DART_NEAREST_EPOCH | DART_EXACT_TIME | DART_RECORDS_ONLY |
                           DART_NO_KAHAN | DART_PLANE_ADDR64;
    return (v.flags & other) || v.width < 1 || v.height < 1 ? 0.0 : (double)v.width * v.height;
}
bool jplane_ready(const dart_stack *s);
void note_use(const dart_stack *s, hipStream_t stream);
std::vector<const dart_stack *> each_stack(const dart_stack *const *stacks, int32_t n);  // once
void note_uses(const dart_stack *const *stacks, int32_t n, hipStream_t stream);  // each once
bool stack_busy(const dart_stack *s);
dart_tuning tuning_for(const dart_stack *s);
// Vector stacks: repacks the components' emissivity on `stream` if any
// component was refilled since it was packed (after renders that read the
// packed copy have finished).  No-op for other stacks.
dart_status refresh_vector(const dart_stack *s, hipStream_t stream);

// One launch group of a batch: views of one storage type and ray precision.
struct Group {
    int store = 0;
    bool f64 = false;
    bool labelled = false;  // views of labelled stacks (kernels with the block loop)
    bool vec = false;       // views of vector stacks
    bool exact = false;     // views with exact temporal integration
    bool jp = false;        // views that read their stacks' emissivity planes
    bool jp32 = false;      // ... through 32-bit offsets (planes of at most 4 GiB)
    bool pairs = false;     // ... as pairs
    std::vector<RayView> views;
    // n_tiles tiles: the queued ones [0, q_begin[n_queues]), then n_clear tiles
    // whose rays all miss the grid (k_finish sets their pixels to 0).  As rows
    // (their tiles are written on the device), or one by one where the queue's
    // order does not keep rows or the caller asked for it.
    uint32_t n_tiles = 0;
    std::vector<Run> runs;
    std::vector<Tile> tiles;
    size_t parts = 0;         // values of BatchLaunch::parts (0: no tile is queued by segment)
    uint32_t n_clear = 0;
    size_t view_off = 0, tile_off = 0;  // offsets in the uploaded descriptor arrays
    uint32_t n_queues = 8;
    uint32_t q_begin[MAX_QUEUES + 1] = {};  // chunk bounds
};

// Queue heads and sum slots of a launch of n views in some groups, in 64-bit
// words from the start of one block: first every group's MAX_QUEUES heads, then
// the slots of view 0, 1, ..  Heads and slots have a cache line each (16 words)
// where several wavefronts would otherwise add to one line at a time: 64 slots
// for a single view, fewer for more views (whose wavefronts are spread over the
// views already; the slots of a launch take at most 64 KiB until each view is
// down to one).  compact: heads and slots side by side, one slot per view.
struct SumLayout {
    size_t groups, n;
    uint32_t slots, stride, head_stride;  // slots per view; words; heads: 32-bit words
    SumLayout(size_t n_views, size_t n_groups, bool compact = false);
    size_t head_words() const { return MAX_QUEUES * (size_t)head_stride / 2; }
    // (the start of a block: what is cleared before a launch)
    size_t heads_words() const { return groups * head_words(); }
    size_t sum_words() const { return n * slots * stride; }
    size_t words() const { return heads_words() + sum_words(); }
    uint32_t *head(unsigned long long *block, size_t group) const {
        return (uint32_t *)(block + group * head_words());
    }
    RenderSums sums(unsigned long long *block) const {
        return RenderSums{block + heads_words(), slots - 1u, stride};
    }
    // A view's totals from a host copy of the slots (sum_words() words).
    void total(const unsigned long long *h, size_t view, double *flux, uint64_t *steps) const;
};

// max_parts: the most values of BatchLaunch::parts the caller has room for.
// as_runs: the caller uploads with begin_plan (else every tile is listed).
dart_status plan_batch(const dart_stack *const *stacks, const dart_view *views, int32_t n,
                       void *const *images, const dart_tuning &tun, size_t max_parts,
                       bool as_runs, std::vector<Group> &groups);
// The launches of a plan share one parts array (they run one after the other).
size_t parts_of(const std::vector<Group> &groups);

// Events that say that kernels have read something (a stack's records, staged
// descriptors), so that it may be written again: no kernel's output is passed on by
// them, so they carry no system-scope fence, whose cache write-back delayed the next
// kernel of the stream by several us (ten calls of a light curve 902 -> 856 us, a
// replaced epoch with its render and read-back 377 -> 364 us).
constexpr unsigned READ_EVENT = hipEventDisableTiming | hipEventDisableSystemFence;

// Per-(device, stream) scratch: accumulators, descriptor arrays, image staging,
// pinned upload staging and the last captured batch graph.
struct Workspace {
    hipStream_t stream = nullptr;
    int device = 0;
    std::mutex mu;
    unsigned long long *acc = nullptr;  // queue heads and sum slots (SumLayout)
    size_t acc_cap = 0;
    void *sums_host = nullptr;          // pinned: the views' totals (launch_totals)
    size_t sums_host_cap = 0;
    unsigned long long *flag = nullptr; // device: the first bad element of a load
    bool flag_clear = false;            // it holds ~0
    void *img_host = nullptr;           // pinned: a small host-destined image
    size_t img_host_cap = 0;
    unsigned char *desc = nullptr;      // the plan's view, then tile descriptors
    size_t desc_cap = 0;
    double *parts = nullptr;            // BatchLaunch::parts
    size_t parts_cap = 0;
    unsigned long long *img = nullptr;  // staging for host-destined images
    size_t img_cap = 0;
    void *stage = nullptr;              // pinned host staging for descriptor uploads
    size_t stage_cap = 0;
    hipEvent_t stage_done{};
    bool stage_ready = false;
    hipGraphExec_t graph_exec[2] = {nullptr, nullptr};  // without / with sums
    // the last batch plan (descriptors already on the device), replayed when
    // the next call has the same key
    std::vector<Group> plan_groups;
    std::vector<uint8_t> plan_key;
    bool plan_ready = false;
};

void read_totals(const void *host, int32_t n, double *flux, uint64_t *steps);
Workspace *get_workspace(hipStream_t stream);
hipError_t ws_flag(Workspace *ws);
hipError_t ws_reserve(Workspace *ws, size_t staged, size_t resident, size_t img_u64,
                      size_t acc_words, size_t n_parts = 0);
// The kernels of a plan whose queue heads (and sums) launch_begin has cleared.
// sums: whether they add up flux and cell-steps.
hipError_t enqueue_plan(const std::vector<Group> &groups, const SumLayout &lay,
                        unsigned long long *acc, bool sums, double *parts,
                        const RayView *dviews, const Tile *dtiles, const dart_tuning &tun,
                        int device, hipStream_t stream);
void assign_offsets(std::vector<Group> &groups, size_t *n_views, size_t *n_tiles);
// Bytes of a plan's descriptors on the host (views, then runs or tiles) and on the
// device (views, then tiles).
size_t staged_bytes(const std::vector<Group> &groups);
size_t resident_bytes(const std::vector<Group> &groups);
void pack_descriptors(const std::vector<Group> &groups, void *dst);
// Clears n_clear words and makes the device's descriptors from the packed ones in
// pinned memory.
hipError_t begin_plan(const std::vector<Group> &groups, const void *packed, void *dev,
                      unsigned long long *clear, size_t n_clear, hipStream_t stream);

}  // namespace dart
