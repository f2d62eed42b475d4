// dart_internal.h -- descriptors shared by the HIP kernels and the host runtime.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dart {

enum Store : int { ST_F64 = 0, ST_F32 = 1, ST_F16 = 2, ST_BF16 = 3 };

enum : uint32_t {
    F_NO_LOOKBACK = 0x1u,
    F_NO_BEAMING = 0x2u,
    F_NEAREST = 0x4u,
    F_NO_KAHAN = 0x8u,
    F_F64_DDA = 0x10u,
    F_DEVICE_PTRS = 0x20u,
    F_ACCUMULATE = 0x80u,
    F_EXACT = 0x100u,
    F_PLANE32 = 0x1000u,  // the view's emissivity plane is read through 32-bit offsets
    F_PAIRS = 0x2000u,    // jplane holds pairs: a record's element and the next epoch's
};

// Resident stack as the kernels see it.  Records (j, bx, by, bz) are stored
// epoch-major; inside an epoch the cells are grouped in bricks of
// 2^lb[0] x 2^lb[1] x 2^lb[2] cells (x fastest inside a brick, bricks x-fastest).
struct StackDev {
    const void *data;       // resident records
    // Emissivity plane: the j field of every record packed alone, at the
    // record's own index, in the storage type (FP32, or the 16-bit bits); its
    // sign bit is set when the record must be read whole (velocity bits not
    // all zero, or j itself negative or -0).  Null: read whole records.
    const void *jplane;
    const double *times;    // [M] epoch times (device)
    const double *inv_dt;   // [M] 1 / (t_{m+1} - t_m), 0 for the last epoch (device)
    int64_t epoch_stride;   // records from one epoch to the next (padded to whole bricks;
                            // negative for a streamed interval whose later epoch sits
                            // in an earlier ring slot)
    int32_t n[3];           // cells per axis
    int32_t nb[3];          // bricks per axis
    int32_t lb[3];          // log2 of the brick shape
    int32_t n_epochs;
    int32_t store;          // Store
    double cell[3];
};

// One sub-domain of a labelled stack: its grid and the camera centre in the
// grid's own coordinates (the domain centre minus the grid's origin).
struct Block {
    StackDev st;
    double centre[3];
};

// One view, resolved on the host in FP64.
struct RayView {
    double shat[3], eu[3], ev[3], centre[3];
    double inv_shat[3];     // 1 / s_hat per axis (0 where s_hat has a zero component)
    float shat_hi[3];       // s_hat rounded to FP32, and the rest: s_hat = hi + lo to
    float shat_lo[3];       // ~2^-48, for the FP32 Doppler of 16-bit stacks
    double ps;              // pixel scale
    double t_obs;
    double s_lo, s_hi;      // temporal window expressed in s: [t_obs - t_{M-1}, t_obs - t_0]
                            // (a half-open end is the next representable value inside)
    double p;               // 2 + alpha
    uint32_t flags;
    int32_t width, height;
    int32_t fixed_m;        // NO_LOOKBACK: epoch bracket at t_obs (-1: t_obs outside coverage)
    double fixed_w;         // NO_LOOKBACK: weight of epoch fixed_m + 1
    float fixed_wf;         // the same rounded to FP32 (read as such by FP32 walks)
    // Depth segments: a ray's sum is made of 1 << seg_log2 partial sums over
    // consecutive parts of its chord, added in order; which cells a part holds
    // depends on the view and the ray alone.  seg_items: the parts of a tile are
    // queued on their own (their sums meet in BatchLaunch::parts and k_finish
    // adds them); 0: a lane marches its ray's parts one after the other.  (The plain
    // kernel has its own arrangements, by tile_w_log2.)  The
    // pixels are the same bit for bit.
    int16_t seg_log2, seg_items;
    double sync_gap;        // batched kernel: depth-synchronous horizon (length), 0 = off
    void *image;            // [height][width] float or double (device)
    int32_t out_f64;
    int32_t acc_index;      // slot in the flux / step accumulators
    int32_t tile_w_log2;    // tile width 1 << tile_w_log2, height 64 >> it (plain kernel: 3, 6 or
                            // PLAIN_ROWS)
    StackDev st;            // the stack (a labelled stack: its first sub-domain)
    const Block *blocks;    // labelled stack: its sub-domains (device), else null
    int32_t n_blocks;       // 0 for a plain stack
    // vector stack: n_chan components (2..4) with the same grid and layout;
    // st is component 0 (its velocity sets D for all), chan_data[c - 1] the
    // emissivity of component c packed one value per record index.  Images
    // are [n_chan][height][width].  n_chan = 1 otherwise.
    int32_t n_chan;
    const void *chan_data[3];
};

constexpr int PLAIN_ROWS = 7;  // RayView::tile_w_log2 of k_plain_rows

constexpr int TILE_SEG_SHIFT = 28;  // Tile::view: the view, and above it the depth segment
constexpr int MAX_SEG_LOG2 = 2;

struct Tile {
    uint32_t view;
    uint16_t tx, ty;
};

// A row of tiles as the planner lays it out: `count` tiles from (tx, ty) on, each
// once per depth segment (1 << seg_log2 places side by side), at places `first`
// on of the tile descriptors.  launch_begin writes the descriptors.
struct Run {
    uint32_t first, view, count_seg;  // count | seg_log2 << RUN_SEG_SHIFT
    uint16_t tx, ty;
};
constexpr int RUN_SEG_SHIFT = 24;

constexpr int MAX_QUEUES = 8;

// Where a render adds its flux and cell-steps: view i has slots (flux as double
// bits, then steps), `stride` words apart, and a wavefront adds to slot (its
// number & mask); the host sums a view's slots.  slots null: nobody asked.
// Atomic additions to one cache line take about 12 ns each, one after the
// other, whichever wavefront they come from: with one slot per view, the 4096
// tiles of a 512^2 image spent 98 of their 230 us there.  With a line per slot
// and per queue head (and no sums where none are asked for): one 512^2 image of
// a 128x128x256 FP32 jet 228 -> 171 us, four of the 256x256x512 jet 586 -> 529
// us, nine streamed intervals of two 512^2 views 3.14 -> 1.50 ms.
struct RenderSums {
    unsigned long long *slots;
    uint32_t mask;
    uint32_t stride;
};

// Launch parameters of the persistent batched kernel.
struct BatchLaunch {
    const RayView *views;
    const Tile *tiles;
    uint32_t n_tiles;
    uint32_t *head;         // tile queue heads, one per XCD queue
    uint32_t head_stride;   // words from one head to the next
    uint32_t n_queues;      // at most MAX_QUEUES
    uint32_t q_begin[9];    // queue q holds tiles [q_begin[q], q_begin[q + 1])
    RenderSums sums;
    // partial sums of the tiles queued by depth segment: channel c of lane k of
    // queue position t at (t * C + c) * 64 + k, C = 4 for launches of vector
    // stacks, else 1
    double *parts;
};

// Host-side launchers (dart_kernels.hip).
hipError_t launch_plain(const RayView &v, const RenderSums &sums, hipStream_t s);
// Kernel variant bits: 1 depth-synchronous wavefronts, 2 the launch's views are
// labelled stacks (block loop), 4 exact temporal integration, 8 eight cells per
// batch (else four), 16 vector stacks (with 8, 32 and 64 only), 32 the views'
// stacks have an emissivity plane.
enum : int {
    KV_SYNC = 1, KV_LABELLED = 2, KV_EXACT = 4, KV_K8 = 8, KV_VEC = 16, KV_JP = 32,
    KV_JP32 = 64,  // with KV_JP: the plane through 32-bit byte offsets (F_PLANE32; not with 2)
    KV_PAIRS = 128,  // with KV_JP: the plane as pairs (F_PAIRS; with KV_SYNC and KV_K8 only)
};
hipError_t launch_batch(int store, bool f64_dda, int variant, const BatchLaunch &bl,
                        int grid_blocks, hipStream_t s);
// Marks the samples of positive weight of a render of v (moving_only: only
// those whose record must be read whole, see StackDev::jplane) in a bitmap of
// records (line_log2 < 0) or of lines of 2^line_log2 elements of the record
// index space.
hipError_t launch_mark(const RayView &v, uint32_t *bitmap, int line_log2, bool moving_only,
                       hipStream_t s);
hipError_t launch_popcount(const uint32_t *bitmap, uint64_t words, unsigned long long *out,
                           hipStream_t s);
// plane: the stack's emissivity plane, kept in step with the records (may be null).
hipError_t launch_convert(int src_f64, int store, const void *j, const void *beta, int32_t m0,
                          int32_t count, const StackDev &st, void *data, void *plane,
                          unsigned long long *err, hipStream_t s);
hipError_t launch_rebrick(int store, const StackDev &from, const StackDev &to, void *dst,
                          void *plane, hipStream_t s);
// One epoch of a stack back in the caller's layout, widened to FP64 (FP64
// stacks) or FP32 (the others): j [ncell], beta [ncell][3] (device).
hipError_t launch_read_epoch(const StackDev &st, int32_t m, void *j, void *beta, hipStream_t s);
// Emissivity fields of n resident records into a packed array (vector stacks).
hipError_t launch_pack_j(int store, const void *records, void *out, uint64_t n, hipStream_t s);
// The emissivity plane of n records (StackDev::jplane).
hipError_t launch_pack_jplane(int store, const void *records, void *out, uint64_t n,
                              hipStream_t s);
// Pairs of a plane of m epochs of `stride` elements: element i and element i + stride
// (0 in the last epoch) side by side.  16-bit elements.
hipError_t launch_pack_pairs(const void *plane, void *out, uint64_t stride, int32_t m,
                             hipStream_t s);
hipError_t launch_fill_u64(unsigned long long *p, uint64_t n, unsigned long long value,
                           hipStream_t s);
// What precedes a render's kernels, in one launch: clears n_clear words, copies
// n_copy words (descriptors in pinned host memory, src) and writes the tile
// descriptors of n_runs rows (runs: pinned too).
hipError_t launch_begin(unsigned long long *clear, size_t n_clear, void *dst, const void *src,
                        size_t n_copy, const Run *runs, size_t n_runs, Tile *tiles,
                        hipStream_t s);
// Totals of n views from their slots, written to pinned host memory: flux[n] (as
// double bits), then steps[n].
hipError_t launch_totals(const RenderSums &sums, int32_t n, void *host, hipStream_t s);
hipError_t launch_copy(void *dst, const void *src, uint64_t bytes, hipStream_t s);
// After a batched launch: adds up the parts of the tiles among the n_queued
// queue positions that were queued by segment (parts null: there are none) and
// stores their pixels, and writes 0 to every pixel (and channel) of the n_clear
// tiles that follow them.
hipError_t launch_finish(const RayView *views, const Tile *tiles, uint32_t n_queued,
                         uint32_t n_clear, const double *parts, hipStream_t s);

}  // namespace dart
