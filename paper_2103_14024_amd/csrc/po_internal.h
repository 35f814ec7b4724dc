// Internal declarations shared by the host API (po_api.cpp) and the HIP
// kernels (po_kernels.hip) of libplenoctree.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <hip/hip_vector_types.h>
#include <stdint.h>

#include <algorithm>

#include "plenoctree.h"

#ifdef __HIPCC__
#define PO_HD __host__ __device__
#else
#define PO_HD
#endif

// Kernel-side view of a bound tree (plain data, passed by value).
struct KTree {
    // What the walk reads: the caller's child array [n_top][8], or the
    // library's traversal index (po_tree_build_index), four parts in one
    // buffer:
    //   grid    [8^grid_level] one entry per cell of level grid_level, index
    //           (x << G | y) << G | z; absent when grid_level is 0
    //   nodes   [n_top][8] child entries of the nodes above brick_level,
    //           renumbered; an entry of a level-brick_level cell >= n_top
    //           names brick (entry - n_top).  n_top is 0 where the grid
    //           reaches brick_level
    //   bricks  [n_bricks][8][8][8], the finest cells (x, y, z) below each
    //           internal node of level brick_level
    //   coarse  leaves of level <= grid_level, {leaf, level}, from the end of
    //           the buffer backwards
    // A grid entry is an empty entry (< 0), kIdxCoarse | number of a coarse
    // leaf, or the brick (grid_level == brick_level) or node below the cell.  A
    // brick entry is ((leaf + 1) << 2) | (D - level) of the leaf holding the
    // cell, or an empty entry (po_index_box_entry).
    const int32_t* child;
    const void* sigma;      // [n_leaves] float or half
    const void* sh;         // [n_leaves][stride] float or half
    union {                 // a tree has SG lobes or a codebook, never both
        const float* lobes;     // cb_entries == 0: nullptr (SH basis) or [K][4] spherical-Gaussian lobes
        const void* codebook;   // cb_entries > 0: [K][cb_entries][4] float16 colours; sh holds uint16 indices
    };
    int32_t n_top;          // nodes in `child` (all of the caller's nodes when brick_level == depth)
    int32_t n_leaves;
    int32_t stride;         // elements per SH record
    // depth D, brick_level M (cells below level M are resolved by bricks; M ==
    // D: no bricks), grid_level G (cells of levels <= G are resolved by the
    // grid; 0: no grid) and whether the grid names leaves, a byte each (one
    // word, because scalar loads are of words: as int8_t members a batch's
    // kernel read them through the vector memory in every step)
    uint32_t levels;
    uint32_t index_bytes;   // bytes readable through `child`
    int32_t cb_entries;     // codebook entries per basis function (0: no codebook)
    uint32_t sigma_bytes;   // n_leaves * element size (< 2^32)
    uint32_t sh_bytes;      // n_leaves * stride * element size (< 2^32 - 256)
    double lo[3];           // box minimum corner, world units
    double scale;           // grid units (finest cells) per world unit: 2^D / (2 half)

    PO_HD int depth() const { return (int)(levels & 255u); }
    PO_HD int brick_level() const { return (int)(levels >> 8 & 255u); }
    PO_HD int grid_level() const { return (int)(levels >> 16 & 255u); }
    void set_levels(int D, int M, int G, bool coarse) {
        levels = (uint32_t)D | (uint32_t)M << 8 | (uint32_t)G << 16 | (coarse ? 1u << 24 : 0u);
    }
};

// Traversal index encoding (KTree::child).
constexpr int kIdxCoarse = 1 << 30;
// Finest grid of an index: 8^8 entries, 64 MB.
constexpr int kIdxMaxGrid = 8;
// An empty entry: bit 31, log2 of the edge of its cells (in finest cells) in
// bits 27..30, the levels from such a cell up to the octree's empty cube in
// bits 24..26, and an empty box around cell c: cells to spare below and above
// it on axis k, up to kIdxReach each, in bits 8k..8k+3 and 8k+4..8k+7.  The
// box holds the whole cube as long as that is at most kIdxReach + 1 cells
// wide, so a cube of more is counted in larger cells (up <= 4): with cells of
// the grid's own, the 64 cells of a cube of a sparse tree took five steps
// instead of one (mixed leaves at depth 12, 1920x1080: 0.152 against 0.114 ms).
constexpr int kIdxReach = 15;
PO_HD inline int32_t po_index_box_entry(const int (&c)[3], const int (&lo)[3], const int (&hi)[3], int up, int unit) {
    uint32_t e = 0x80000000u | (uint32_t)unit << 27 | (uint32_t)up << 24;
    for (int k = 0; k < 3; ++k) {
        const int below = c[k] - lo[k], above = hi[k] - c[k];
        e |= (uint32_t)(below < kIdxReach ? below : kIdxReach) << (8 * k) |
             (uint32_t)(above < kIdxReach ? above : kIdxReach) << (8 * k + 4);
    }
    return (int32_t)e;
}
// The entry of cell c (edge 2^unit) from a box [lo, hi] that holds its octree
// cube, `up` levels higher, in cells that are large enough for the cube to fit
// the fields (the box shrinks to whole ones).
PO_HD inline int32_t po_index_cube_entry(const int (&c)[3], const int (&lo)[3], const int (&hi)[3], int up, int unit) {
    const int j = up > 4 ? up - 4 : 0;
    int cj[3], l[3], h[3];
    for (int k = 0; k < 3; ++k) {
        cj[k] = c[k] >> j;
        l[k] = (lo[k] + (1 << j) - 1) >> j;
        h[k] = ((hi[k] + 1) >> j) - 1;
    }
    return po_index_box_entry(cj, l, h, up - j, unit + j);
}
// log2 of the edge of an empty entry's cells, and of its octree cube.
PO_HD inline int po_index_unit(int32_t e) { return (int)((uint32_t)e >> 27 & 15u); }
PO_HD inline int po_index_cube(int32_t e) { return po_index_unit(e) + (int)((uint32_t)e >> 24 & 7u); }

// KOpts::flags bit (internal, beside the caller's): walk the octree's own
// cells, not boxes of several empty ones.  Set where their number matters:
// the steps column of the aux outputs, and a caller's max_steps.
constexpr uint32_t kOptExact = 1u << 31;

struct KOpts {
    float bg[3];
    float stop_T;
    int32_t max_steps;
    uint32_t flags;
    uint32_t sh_off;        // viewer: SH basis functions left out
    float clip[4];          // viewer: slicing half-space n.x + w >= 0 (all zero: none)
};

// True when a render needs the viewer kernels (aux outputs with depth, SH
// subsets or a slicing plane); the plain kernels serve every other call.
inline bool po_view_opts(const KOpts& k, const float* aux) {
    return aux != nullptr || k.sh_off != 0u || k.clip[0] != 0.0f || k.clip[1] != 0.0f || k.clip[2] != 0.0f ||
           k.clip[3] != 0.0f;
}

// Compiled variants of the forward render: plain with the SH basis, plain
// with spherical Gaussians, and the viewer kernel (either basis, chosen per
// tree at run time).  The plain kernels carry no code for the other basis.
// Codebook trees render with PO_FWD_CB and take no viewer options.
enum { PO_FWD_SH = 0, PO_FWD_SG = 1, PO_FWD_VIEW = 2, PO_FWD_CB = 3 };
inline int po_fwd_variant(const KOpts& k, const float* aux, const KTree& t) {
    if (t.cb_entries > 0) return PO_FWD_CB;
    return po_view_opts(k, aux) ? PO_FWD_VIEW : (t.lobes ? PO_FWD_SG : PO_FWD_SH);
}

struct KCam {
    float c2w[12];
    int32_t W, H;
    float fx, fy, cx, cy;
};

// One camera job of a batched launch.
struct KJob {
    KTree tr;
    KCam cam;
    KOpts op;
    float* rgb;
    float* aux;
    int32_t tile_begin;     // first 16x16 tile of the image rendered by this job
    int32_t block_begin;    // first workgroup (before the XCD swizzle) of this job: 4 per 16x16 tile
    int32_t tiles_x;        // ceil(W / 16)
    int32_t pad_;
};

// Work queues of the split camera render: rays whose walk outlasts
// split_cap samples are handed on as 1-16 chunks, and chunks that outlast
// chunk_cap samples hand their remainder on as 1-16 sub-chunks.  Each queue has
// kSplitRegions regions of region_slots slots (a multiple of 64), one counter
// each: kSplitRegionSlots for the queues the library allocates,
// kNoAllocRegionSlots for the fixed queue of the entry point that allocates
// nothing.  A walk whose region is full finishes in its own lane, so the size
// changes the speed, never the result.
#ifndef PO_SPLIT_REGION_SLOTS
#define PO_SPLIT_REGION_SLOTS 16384
#endif
constexpr int kSplitRegions = 64;
constexpr int kSplitRegionSlots = PO_SPLIT_REGION_SLOTS;
constexpr int kNoAllocRegionSlots = 8192;
constexpr int kSplitMaxChunks = 16;
// Step caps up to this many cells are rendered in one pass.
constexpr int kSplitMinMaxSteps = 28;
struct KSplit {
    int32_t* count;        // [kSplitRegions] chunk slots claimed (may exceed the region); count2 follows
    int32_t* count2;       // [kSplitRegions] sub-chunk slots claimed
    int4* info;            // [slots] {first chunk slot of the ray (-1: unused), chunk | count << 8, next chunk slot, 0}
    void* head;            // [slots] 32-byte ray states, at the first slot of each ray
    void* part;            // [slots] 32-byte chunk results
    int4* info2;           // [slots] the same for the sub-chunks of remainders
    void* head2;           // [slots] 32-byte remainders, at their first slot
    void* part2;           // [slots] 32-byte sub-chunk results
    int4* view_part;       // [slots] viewer variant: chunk samples, cells and cut flags
    int4* view_part2;      // [slots] the same for the sub-chunks
    int32_t region_slots;  // slots per region; slots = kSplitRegions * region_slots
    // piece sizes, in data samples (exact: in cells)
    int32_t split_cap;     // walked before a ray is handed on
    int32_t chunk_target;  // wanted per chunk
    int32_t sub_target;    // wanted per sub-chunk
    int32_t chunk_cap;     // a chunk walks before its remainder is handed on
    float ub_frac;         // pieces cover at least this fraction of the finest-cell faces ahead
    bool exact;            // the walks step the octree's own cells
    const float* ray_o;    // ray-list renders: origins [n_rays][3] (camera renders: unused)
    const float* ray_d;    // ray-list renders: directions [n_rays][3]
    int64_t n_rays;
    int32_t* ray_slot;     // kept ray-list render: [n_rays] first chunk slot of each ray, -1 if not handed on
};
// Piece sizes of a split camera render of `waves` waves (four per 16x16
// tile).  About kResidentWaves waves fit on the chip at once (256 CUs x 4
// SIMDs x 4 waves at 128 VGPRs); a launch of several such rounds keeps the
// chip busy through its first walk, so its rays walk further before the
// hand-off and fewer of them wait in the chunk queues.
constexpr int64_t kResidentWaves = 4096;
// In octree cells.
inline void po_cell_piece_sizes(int64_t waves, KSplit* S) {
    const int64_t s = 20 + 18 * waves / kResidentWaves;
    S->exact = true;
    S->split_cap = (int)(s < 28 ? 28 : s > 192 ? 192 : s);
    S->chunk_target = 24;
    S->sub_target = 10;
    S->chunk_cap = 24;
    S->ub_frac = 0.3f;
}
// The sizes in samples, measured (us; float32 800x800, 1280x720 and 512x512 of
// the depth-9 scene, float16 1920x1080, codebook 640x480 and SG-25 400x400 of
// depth 8; in cells, over the octree's own cells: 517 / 811 / 356 / 1006 / 392 /
// 264): 451 / 609 / 327 / 720 / 376 / 260; ub_frac 0.24 458 / 617 / 338 / 734 /
// 391 / 266; chunks and cap of 12 456 / 618 / 330 / 725 / 374 / 262; a first
// walk of 6 + 6 samples a round loses 8 % at 1920x1080.  Smaller sub-chunks or
// a cap below the target overflow the queue where a dense volume fills every
// chunk past its cap.
//
// In octree cells instead for renders that report or cap them (exact), for
// frames of less than half a round of waves (2^17 pixels), where the first
// walk's way to its first sample is the longest part (in samples / in cells,
// us, 256x256 and 320x280, float32: depth 8, K = 9 142 / 122 and 145 / 130; depth
// 9, K = 16 183 / 150 and 207 / 179; depth 10 206 / 167 and 251 / 211; from
// 400x400 as often slower: 154 / 144 at depth 8, 205 / 217 there with K = 25, 417
// / 580 at depth 10 and 640x480), and for trees without a grid, whose walks step
// them anyway (depth 8 256x256 251 / 185, depth 9 512x512 472 / 340).
inline void po_frame_piece_sizes(const KTree& t, int64_t waves, bool exact, KSplit* S) {
    if (exact || waves < kResidentWaves / 2 || t.grid_level() == 0) {
        po_cell_piece_sizes(waves, S);
    } else {
        S->exact = false;
        const int64_t s = 10 + 10 * waves / kResidentWaves;
        S->split_cap = (int)(s < 12 ? 12 : s > 96 ? 96 : s);
        S->chunk_target = 16;
        S->sub_target = 8;
        S->chunk_cap = 16;
        S->ub_frac = 0.4f;
    }
}
// Piece sizes of a split pass over a list of n rays.  The render and the
// backward of the same rays cut them alike: the transmittance in front of
// every piece is then the same float product in both, so the backward stops
// on the sample where the render that produced its colour stopped.  So the
// sizes depend on n and the depth alone, never on the options: a render with
// aux outputs or a step cap cuts as its backward, which has neither, does.
// They count octree cells, which the walks then step (exact); the counts of
// aux outputs so do not depend on how empty space is crossed either.
// From 2^18 rays a frame's (its sizes in samples, over boxes, against these in
// cells: 300,000 rays at depth 8 0.326 against 0.307 ms, at depth 9 with K = 16
// 0.763 against 0.529; 10^6 rays 0.927 against 0.959 and 1.58 against 1.71).
// A batch below 2^18 rays fills the chip for less time than a frame: a first
// walk of a few cells and small pieces (training step of 65,536 rays, depth 8:
// 0.558 ms with the frame's sizes, 0.460 with these).  Its first walk counted
// in samples would cross the empty space in front of the first leaf at one
// wave's speed (52 against 18 us).  Chunks of 8 cells, handed on past 16: 0.304
// ms for the training step (6 and 12: 0.311), 0.455 and 0.483 with 131,072
// rays, and the render of 200,001 0.265 and 0.287.  As many pieces
// as the queue's 2^20 slots hold: past that the walks that find their region
// full finish in their lanes (200,001 rays, depth 8, chunks of 6: 0.535 ms at
// ub_frac 0.2, 0.333 at 0.1; 65,536 rays 0.358 at 0.2, 0.383 at 0.1).
inline void po_rays_piece_sizes(int64_t n, int depth, KSplit* S) {
    if (n >= (1 << 18)) {
        po_cell_piece_sizes(0, S);
    } else {
        S->exact = true;
        S->split_cap = 4;
        S->chunk_target = 8;
        S->sub_target = 8;
        S->chunk_cap = 16;
        S->ub_frac = (float)std::min(0.2, 5.6e6 / (double)(n << depth));
    }
}
// Device bytes of the queues with region_slots slots per region (counters,
// then info, head, part and viewer record of each queue).
constexpr size_t po_split_bytes(int region_slots) {
    return 512 + 2 * (size_t)kSplitRegions * (size_t)region_slots * (16 + 32 + 32 + 16);
}
// Points S at queues laid out in `base` (po_split_bytes(region_slots) bytes).
void po_split_layout(void* base, int region_slots, KSplit* S);
// Bytes of the fixed queue of po_render_camera_noalloc (one copy per device,
// a static device array of the library: about 100 MB).
constexpr size_t kNoAllocBytes = po_split_bytes(kNoAllocRegionSlots);
// Images the fixed queue is sized for: larger ones are rejected.
constexpr int64_t kNoAllocMaxPixels = int64_t(1) << 22;
// Points S at the fixed queue of the current device (its device address is
// looked up once per device, under a lock); allocates nothing.
hipError_t po_noalloc_queue(KSplit* S);

struct po_tree {
    po_tree_desc desc;
    int64_t n_nodes, n_leaves;
    const int32_t* child;
    const void* sigma;
    const void* sh;
    int32_t K;              // coefficients per channel
    int32_t stride;         // elements per SH record
    int32_t vec_bytes;      // widest aligned load of a record: 16, 8 or 4
    bool codebook;          // records are codebook indices (float16 densities)
    void* d_index;          // traversal index owned by the handle (nullptr: none built)
    int index_device;       // device holding d_index
    int64_t n_bricks;
    KTree kt;
};

// Sets the thread's po_last_error message (cleared for PO_OK) and returns s.
po_status po_report(po_status s, const char* msg);

// Launchers (po_kernels.hip).  Arguments are validated by the caller.
hipError_t po_launch_rays(const po_tree* t, int64_t n, const float* o, const float* d,
                          const KOpts& op, float* rgb, float* aux, hipStream_t s);
hipError_t po_launch_backward(const po_tree* t, int64_t n, const float* o, const float* d,
                              const KOpts& op, const float* rgb_fwd, const float* grad_rgb,
                              float* grad_sigma, float* grad_sh, hipStream_t s);
// Renders camera jobs that all share dtype, K and vec_bytes (at most
// PO_BATCH_MAX_JOBS) and the same po_fwd_variant; n_blocks counts
// workgroups, four per 16x16 tile.
hipError_t po_launch_camera_jobs(const po_tree* first, int n_jobs, KJob* jobs, int n_blocks, int variant,
                                 hipStream_t s);
// One camera job as the split render (any forward variant): clears the queue
// counters and launches the four render kernels.
// The queue must not be in use by work on another stream.
hipError_t po_launch_camera_split(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                                  hipStream_t s);
// n rays (n < 2^31) as the split render (any forward variant; aux for the
// viewer variant); the queue must not be in use by work on another stream.
hipError_t po_launch_rays_split(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                                float* rgb, float* aux, const KSplit& S, hipStream_t s);
// Backward of n rays (n < 2^31, float32 tree) in pieces: the first walk,
// the forward of the pieces, their prefixes, then the backward of the pieces.
hipError_t po_launch_backward_split(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                                    const float* rgb_fwd, const float* grad, float* gsig, float* gsh,
                                    const KSplit& S, hipStream_t s);
// Backward of the n rays of a kept split render (po_launch_rays_split with
// S.ray_slot set, same rays, options and queue, nothing else on the queue in
// between): the first walk, the prefixes of the render's own pieces, then
// the backward of the pieces.  Consumes the kept pieces.
hipError_t po_launch_backward_kept(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                                   const float* rgb_fwd, const float* grad, float* gsig, float* gsh,
                                   const KSplit& S, hipStream_t s);
// Adds to an index the boxes of its n_bricks bricks (bricks of the host's
// layout, changed in place) and, for G > 0, the grid with its boxes, from the
// host's nodes (device copy); sat: 8^G words of scratch.
hipError_t po_launch_index(const int32_t* nodes, int n_top, int G, int unit, int64_t n_bricks, int32_t* grid,
                           int32_t* bricks, int32_t* sat, hipStream_t s);
hipError_t po_launch_camera_rays(const KCam& cam, float* o, float* d, hipStream_t s);
// Visibility filter: mode 0 alpha, 1 contribution; weight[n_leaves] raised in place, alpha[H*W] or nullptr.
hipError_t po_launch_leaf_weights(const po_tree* t, const KCam& cam, const KOpts& op, int mode, float* weight,
                                  float* alpha, hipStream_t s);
// Traversal statistics: writes h_sums[4] = {rays, samples, cells,
// child-entry loads} of the one-pass walk of every pixel ray of *cam, or
// (cam NULL) of the n rays (o, d), waiting for the stream.  Calls must not
// overlap (one device buffer).
hipError_t po_traversal_stats_sync(const po_tree* t, const KCam* cam, int64_t n, const float* o, const float* d,
                                   const KOpts& op, unsigned long long* h_sums, hipStream_t s);
hipError_t po_launch_mse_grad(int64_t n, const float* rgb, const float* target, float scale, float* grad,
                              float* sq_sum, hipStream_t s);
hipError_t po_launch_sgd(int64_t n, float* param, float* grad, float lr, bool zero_grad, hipStream_t s);
hipError_t po_launch_gather_rays(int64_t n, const int64_t* idx, int64_t n_src, const float* o, const float* d,
                                 const float* t, float* bo, float* bd, float* bt, hipStream_t s);
hipError_t po_launch_draw_batch(int64_t n, uint64_t seed, uint64_t first, int64_t n_src, const float* o,
                               const float* d, const float* t, float* bo, float* bd, float* bt, float* sq_sum,
                               hipStream_t s);
hipError_t po_read_device_errors(unsigned long long* out);
// Kernel variant a tree renders with (dtype, K, record-load plan); jobs of one
// batched launch must share it.
int po_plan_id(const po_tree* t);
hipError_t po_reset_device_errors();
