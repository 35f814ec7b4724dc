// HIP kernels of libplenoctree for gfx950 (MI355X).
//
// One ray per lane.  A ray is cut into the exact segments between voxel
// boundaries of the sparse octree (Sec. 4.2, "Rendering"): the current
// position is kept as integer coordinates of a finest-level cell; each step
// reads what holds the cell (a leaf, or a box of empty space) from a traversal
// index, or by a descent of the child array from the deepest ancestor shared
// with the cell before, computes the parameter at which the ray leaves it (the
// nearest exit plane), composites the segment if the leaf holds data, and moves
// the coordinates across the exit face.  Each data
// segment is shaded with the sigmoid of the real-SH expansion in the ray
// direction (Sec. 4.1; SH of App. B.1) and composited front to back with
// alpha = 1 - exp(-sigma delta) (Sec. 3, eqn:quad); marching stops once the
// transmittance falls below the threshold (Sec. 4.2) and the background
// takes the remaining transmittance (App. B.3).
//
// The backward kernel replays the identical segment sequence and applies the
// analytic derivatives of App. B.3 with the prefix scheme of its Remark.
//
// Ray geometry (crossing parameters, positions) is evaluated in FP64, leaf
// values, SH and compositing in FP32.  The library is compiled with
// -ffp-contract=off: every fused multiply-add is written out, so the forward
// and backward kernels take bit-identical steps.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "po_internal.h"

// The library is built from this file compiled once per part (PO_PART = 0 ..
// PO_PARTS - 1), in parallel: each part instantiates the kernels of some of
// the launchers below.  Device variables are per part, so each part keeps its
// own error counter and part 0 sums them.
#ifndef PO_PART
#error "compile with -DPO_PART=<n>, 0 <= n < PO_PARTS"
#endif
#define PO_PARTS 8

namespace {
// malformed child entries and step-cap hits met by this part's kernels
__device__ unsigned long long g_po_errors = 0;
#if PO_PART == 0
// sums of po_traversal_stats: rays, samples, cells, child-entry loads
__device__ unsigned long long g_po_stats[4];
// Work queue of po_render_camera_noalloc: a file-scope device array (one
// copy per GPU the library runs on, held until the process ends).  Host code
// never passes this name to a kernel: it is a host-side stand-in there, and
// po_noalloc_queue looks up each device's own address of the array.
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];
#endif

// One wave64 per workgroup: rays finish unevenly, and single-wave workgroups
// let the dispatcher refill a SIMD as soon as any wave retires, which
// shortens the tail of a launch.
constexpr int kBlock = 64;

// ---------------------------------------------------------------------------
// Real SH basis up to degree 4 at a unit direction (App. B.1), written as
// polynomials in x, y, z.  Index l*l + l + m.  Sign convention: P_l^m carries
// the Condon-Shortley phase, which cancels the (-1)^m of the real
// combination, so every coefficient below is positive.
// ---------------------------------------------------------------------------
template <int K>
__device__ __forceinline__ void sh_basis(float x, float y, float z, float (&Y)[K]) {
    Y[0] = 0.28209479177387814f;  // 1/(2 sqrt(pi))
    if constexpr (K > 1) {
        Y[1] = 0.4886025119029199f * y;  // sqrt(3/(4 pi))
        Y[2] = 0.4886025119029199f * z;
        Y[3] = 0.4886025119029199f * x;
    }
    if constexpr (K > 4) {
        const float xx = x * x, yy = y * y, zz = z * z;
        Y[4] = 1.0925484305920792f * (x * y);              // sqrt(15/pi)/2
        Y[5] = 1.0925484305920792f * (y * z);
        Y[6] = 0.31539156525252005f * (3.0f * zz - 1.0f);  // sqrt(5/pi)/4
        Y[7] = 1.0925484305920792f * (x * z);
        Y[8] = 0.5462742152960396f * (xx - yy);            // sqrt(15/pi)/4
        if constexpr (K > 9) {
            Y[9] = 0.5900435899266435f * (y * (3.0f * xx - yy));   // sqrt(35/(2 pi))/4
            Y[10] = 2.890611442640554f * (x * y * z);              // sqrt(105/pi)/2
            Y[11] = 0.4570457994644658f * (y * (5.0f * zz - 1.0f)); // sqrt(21/(2 pi))/4
            Y[12] = 0.3731763325901154f * (z * (5.0f * zz - 3.0f)); // sqrt(7/pi)/4
            Y[13] = 0.4570457994644658f * (x * (5.0f * zz - 1.0f));
            Y[14] = 1.445305721320277f * (z * (xx - yy));           // sqrt(105/pi)/4
            Y[15] = 0.5900435899266435f * (x * (xx - 3.0f * yy));
            if constexpr (K > 16) {
                const float z7a = 7.0f * zz - 1.0f, z7b = 7.0f * zz - 3.0f;
                Y[16] = 2.5033429417967046f * (x * y * (xx - yy));          // 3 sqrt(35/pi)/4
                Y[17] = 1.7701307697799304f * (y * z * (3.0f * xx - yy));   // 3 sqrt(35/(2 pi))/4
                Y[18] = 0.9461746957575601f * (x * y * z7a);                // 3 sqrt(5/pi)/4
                Y[19] = 0.6690465435572892f * (y * z * z7b);                // 3 sqrt(5/(2 pi))/4
                Y[20] = 0.10578554691520431f * ((35.0f * zz - 30.0f) * zz + 3.0f);  // 3/(16 sqrt(pi))
                Y[21] = 0.6690465435572892f * (x * z * z7b);
                Y[22] = 0.47308734787878004f * ((xx - yy) * z7a);           // 3 sqrt(5/pi)/8
                Y[23] = 1.7701307697799304f * (x * z * (xx - 3.0f * yy));
                Y[24] = 0.6258357354491761f * (xx * (xx - 3.0f * yy) - yy * (3.0f * xx - yy));  // 3 sqrt(35/pi)/16
            }
        }
    }
}

// Spherical-Gaussian basis (App. B.1): G_j(d) = exp(lambda_j (d . p_j - 1))
// for the tree's K lobes (axis p_j, normalised here, and bandwidth lambda_j),
// in place of the SH of the same index.  The lobes are uniform across the
// wave and read once per ray.
template <int K>
__device__ __forceinline__ void sg_basis(const float* __restrict__ lobes, float x, float y, float z,
                                         float (&Y)[K]) {
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const float px = lobes[4 * j], py = lobes[4 * j + 1], pz = lobes[4 * j + 2], lam = lobes[4 * j + 3];
        const float c = (x * px + y * py + z * pz) * rsqrtf(px * px + py * py + pz * pz);
        Y[j] = __expf(lam * (c - 1.0f));
    }
}

// Colour basis of a tree at the unit direction (x, y, z).
template <int K>
__device__ __forceinline__ void colour_basis(const KTree& tr, float x, float y, float z, float (&Y)[K]) {
    if (tr.lobes)
        sg_basis<K>(tr.lobes, x, y, z, Y);
    else
        sh_basis<K>(x, y, z, Y);
}

// Buffer resource for raw (byte-addressed) loads from one array: loads at
// offsets outside [0, bytes) return 0 instead of faulting (gfx9 descriptor
// word 3 = 0x00020000: raw buffer, 32-bit data format).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// ---------------------------------------------------------------------------
// Leaf record access.  T is float or __half; values are widened to float.
// ---------------------------------------------------------------------------
// Number of 32-bit words holding NL elements of type T.
template <typename T, int NL>
struct Words {
    static constexpr int NB = NL * (int)sizeof(T);
    static constexpr int N = (NB + 3) / 4;
};

// A density as it lies in memory; sigma_of widens it.  (Two steps, so that a
// float16 density is not waited for where its load is issued.)
__device__ __forceinline__ uint32_t sigma_buf(__amdgpu_buffer_rsrc_t rs, uint32_t off, float*) {
    return __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
}
__device__ __forceinline__ uint32_t sigma_buf(__amdgpu_buffer_rsrc_t rs, uint32_t off, __half*) {
    return __builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
}
template <typename T>
__device__ __forceinline__ float sigma_of(uint32_t raw) {
    if constexpr (sizeof(T) == 4) return __uint_as_float(raw);
    asm volatile("" : "+v"(raw));  // (the conversion stays here)
    return __half2float(__ushort_as_half((unsigned short)raw));
}

// Element i of a record held as raw words, widened to float.
template <typename T, int NW>
__device__ __forceinline__ float word_elem(const uint32_t (&w)[NW], int i) {
    if constexpr (sizeof(T) == 4) {
        return __uint_as_float(w[i]);
    } else {
        const uint32_t h = (i & 1) ? (w[i >> 1] >> 16) : (w[i >> 1] & 0xffffu);
        return __half2float(__ushort_as_half((unsigned short)h));
    }
}

// Logistic sigmoid (Sec. 4.1) with the hardware reciprocal (1 ulp): the
// correctly rounded division costs ~10 instructions per colour channel.
__device__ __forceinline__ float sigmoid(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// ---------------------------------------------------------------------------
// Ray geometry in grid units: the box spans [0, 2^D]^3 and finest cells have
// unit edge.  The ray is og + s * dg with dg the caller's (unnormalised)
// direction scaled to grid units, so no rounding enters the direction; the
// origin transform, the plane-crossing parameters s and the positions are
// evaluated in FP64.  In FP32 the crossing parameter of a far plane carries
// an error of about 2^-24 of the distance travelled, which becomes an error of
// every segment length; with densities of several hundred per unit length
// that exceeds 1e-4 in colour.  Leaf values, SH and compositing stay FP32.
// A segment's length in world units is (s_exit - s_entry) * |d|.
// ---------------------------------------------------------------------------
//
// Cell coordinates are kept mirrored (x -> 2^D - 1 - x) on the axes along which
// the ray runs downwards, so that every step goes up and needs no case for its
// sign; positions and parameters are the tree's own.
struct Ray {
    double og[3];  // origin, grid units
    double dg[3];  // direction (caller's length), grid units per unit of s
    double inv[3]; // 1 / dg
    double len;    // |d| in world units
    float dn[3];   // unit direction, world (SH argument)
    int c[3];      // finest-level coordinates of the current cell, mirrored
    double s;      // current parameter
    double s_end;  // end of the rendered part (slicing plane), else 1e300
    double s_exit; // end of the walk: min(s_end, box exit)
    bool more;     // split walks: the walk stopped at its sample limit with cells left
    int nt;        // split walks: samples taken (exact: cells walked)

    // c ^ flip is the tree's coordinate (recomputed where it is needed: kept,
    // the three would cost a wave per SIMD)
    __device__ __forceinline__ int flip(int k, int N) const { return dg[k] > 0.0 ? 0 : N - 1; }
    // Mirrored coordinate of the cell holding the point at parameter s.
    __device__ __forceinline__ int cell_at(double s, int k, int N) const {
        return (int)fmin(fmax(floor(fma(s, dg[k], og[k])), 0.0), (double)(N - 1)) ^ flip(k, N);
    }
};

// The walk covers the parameters s in [max(s_lo, 0), s_hi] inside the box.
__device__ __forceinline__ bool ray_setup(const KTree& tr, const double (&o)[3], const double (&d)[3], Ray& r,
                                          double s_lo = 0.0, double s_hi = 1e300) {
    const double len2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
    if (!(len2 > 0.0) || !(len2 < 1e300)) return false;
    r.len = sqrt(len2);
    const double il = 1.0 / r.len;
#pragma unroll
    for (int k = 0; k < 3; ++k) r.dn[k] = (float)(d[k] * il);
    const int N = 1 << tr.depth();
    double s0 = fmax(s_lo, 0.0), s1 = s_hi;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r.og[k] = (o[k] - tr.lo[k]) * tr.scale;
        if (!(fabs(r.og[k]) < 1e300)) return false;
        // A ray lying in a grid plane (zero component) belongs to the cell
        // above it (half-open cells): a positive direction component of
        // 1e-300 grid units gives exactly that, with exit parameters of
        // ~1e300 that never win, and needs no special case in the walk.
        const double g = d[k] * tr.scale;
        r.dg[k] = (g == 0.0) ? 1e-300 : g;
        r.inv[k] = 1.0 / r.dg[k];
        const double ta = (0.0 - r.og[k]) * r.inv[k];
        const double tb = ((double)N - r.og[k]) * r.inv[k];
        s0 = fmax(s0, fmin(ta, tb));
        s1 = fmin(s1, fmax(ta, tb));
    }
    if (!(s1 > s0)) return false;
#pragma unroll
    for (int k = 0; k < 3; ++k) r.c[k] = r.cell_at(s0, k, N);
    r.s = s0;
    r.s_end = s_hi;
    r.s_exit = s1;
    return true;
}

// Parameter range [s_lo, s_hi] of the ray o + s d inside the slicing
// half-space n.x + w >= 0 of the viewer (Sec. 5.5); a ray parallel to the
// plane and outside it gets an empty range.  An all-zero plane keeps the
// whole ray.
__device__ __forceinline__ void clip_range(const KOpts& op, const double (&o)[3], const double (&d)[3],
                                           double& s_lo, double& s_hi) {
    const double nx = op.clip[0], ny = op.clip[1], nz = op.clip[2], w = op.clip[3];
    const double p0 = nx * o[0] + ny * o[1] + nz * o[2] + w;
    const double pd = nx * d[0] + ny * d[1] + nz * d[2];
    const double t = -p0 / pd;  // crossing (unused when pd == 0)
    s_lo = pd > 0.0 ? t : (((pd == 0.0) & (p0 < 0.0)) ? 1e300 : 0.0);
    s_hi = pd < 0.0 ? t : 1e300;
}

// Child slot of cell c (the tree's coordinates) below a node of level L (bits
// D-1-L of the coordinates).
__device__ __forceinline__ uint32_t child_slot(const int (&c)[3], int D, int L) {
    const int sft = D - 1 - L;
    return (uint32_t)((((c[0] >> sft) & 1) << 2) | (((c[1] >> sft) & 1) << 1) | ((c[2] >> sft) & 1));
}

// No limit (march's cap).
constexpr int kNoCap = 0x7fffffff;
// True for renders that walk the octree's own cells one by one: those that
// report or cap their number (see kOptExact).
__device__ __forceinline__ bool exact_cells(const KOpts& op) { return (op.flags & kOptExact) != 0u; }

// The walk of one ray through the cells of the tree.
//
// A step resolves the entry of cell c (a leaf, or empty space), computes the
// parameter at which the ray leaves the cell, moves the coordinates across the
// exit face and starts the read of the next cell's entry.
//
// Entries.  With a grid (tr.grid_level() G > 0) the level-G cell holding c is
// one read, and the 8x8x8 brick below it another, whatever the cell crossed
// before: no node path is kept.  An empty entry names the box of empty space
// around its cell, so that one step crosses it whole (po_index_cube_entry);
// exact keeps to the octree's own empty cubes, whose number is what the aux
// output and po_traversal_stats count and max_steps caps.  The segments of
// the data leaves are the same either way: a leaf is entered through one of
// its faces, and the parameter of that plane does not depend on the box that
// ends there.  Per 800x800 frame of the depth-9 scene: 28.8 -> 18.1 cells and
// 46 -> 22 entry reads per ray.
//
// Without a grid (a caller's child array, or the levels between G and the
// bricks of a tree deeper than the grid) the walk descends through child
// entries; stk, this lane's column of a [level][kBlock] node stack in LDS,
// holds the node of every level on the path to c, and the next descent
// restarts from the deepest ancestor shared by the old and the new cell (the
// level of the highest differing coordinate bit).  The index is read through
// a buffer descriptor: an entry beyond it reads as 0 (empty), and an internal
// entry below depth D or past the node count is counted as malformed and
// taken as empty.

// What one step crossed.
struct Cell {
    int leaf;     // data leaf, or -1: empty space
    float delta;  // length of the segment, world units
    float t_in;   // distance of its start from the ray origin
    bool cpl;     // the cell ends inside the walked range (kClip)
    bool last;    // the walk ends with this cell
    int u;        // log2 of the edge of the cell's cube (without its empty box)
};

// What the walk needs of a tree, held in scalar registers while it runs (read
// through the kernel arguments, the compiler fetched them anew in every step).
__device__ __forceinline__ uint32_t held(uint32_t v) {
    asm volatile("" : "+v"(v));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ int held(int v) { return (int)held((uint32_t)v); }
__device__ __forceinline__ const void* held(const void* p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<const void*>((uint64_t)held((uint32_t)(a >> 32)) << 32 | held((uint32_t)a));
}
struct Index {
    __amdgpu_buffer_rsrc_t rs;
    uint32_t bytes, node0, brick0;  // end of the index; byte offsets of node 0 and brick 0
    int D, M, G, q;                 // q = D - G
    int top;                        // 2^D - 1
    int n_top, n_leaves;
    int coarse;                     // the grid names leaves

    __device__ __forceinline__ explicit Index(const KTree& tr) {
        bytes = held(tr.index_bytes);
        rs = raw_rsrc(held(static_cast<const void*>(tr.child)), bytes);
        const uint32_t levels = held(tr.levels);
        D = (int)(levels & 255u);
        M = (int)(levels >> 8 & 255u);
        G = held((int)(levels >> 16 & 255u));
        q = held(D - G);
        top = held((1 << D) - 1);
        coarse = held((int)(levels >> 24));
        n_top = tr.n_top;
        n_leaves = tr.n_leaves;
        node0 = G > 0 ? 4u << (3 * G) : 0u;
        brick0 = held(node0 + (uint32_t)n_top * 32u);
    }
    __device__ __forceinline__ int entry(uint32_t at) const {
        return __builtin_amdgcn_raw_buffer_load_b32(rs, at, 0, 0);
    }
    // The same, waited for at once: a load that only some lanes make is waited
    // for where they make it.  (Left to its first use, the wait would stand in
    // every lane's path and, loads returning in order, wait for the gather.)
    __device__ __forceinline__ int entry_now(uint32_t at) const {
        int e = entry(at);
        asm volatile("" : "+v"(e));
        return e;
    }
    // Byte offsets of the entries of cell c (the tree's coordinates): the grid's,
    // a brick's ([x][y][z] of the low three bits), a node's.
    __device__ __forceinline__ uint32_t grid_at(const int (&c)[3]) const {
        return (uint32_t)((((c[0] >> q) << G | (c[1] >> q)) << G) | (c[2] >> q)) << 2;
    }
    static __device__ __forceinline__ uint32_t brick_at(uint32_t brick, const int (&c)[3]) {
        return brick + ((uint32_t)(((c[0] & 7) << 6) | ((c[1] & 7) << 3) | (c[2] & 7)) << 2);
    }
    __device__ __forceinline__ uint32_t slot_at(const int (&c)[3], int node, int L) const {
        return node0 + (((uint32_t)node << 5) | (child_slot(c, D, L) << 2));
    }
};

// The three walks.  Kernels are compiled for each, and the batched ones also for
// launches that mix them (those choose by a branch of the wave in front of the
// loop).  One loop that tested the way in every step took 2 to 14 % longer on
// direct trees (64x64 23.3 against 20.4 us, 800x800 410 against 391), and 20 to
// 30 % on trees without an index, whose steps ran through the branches of the
// nodes'.  Loops side by side in one kernel cost it registers: all three, and
// float32 K = 16 at 800x800 lost 7 % to spills around them; the last two, and
// 300,000 rays without an index took 397 us for 358 (K = 9), 468 for 431.
enum Way {
    kDirect,  // the grid reaches the bricks (indexed trees of depth 4 to 11)
    kPlain,   // the caller's child array
    kNodes,   // an index with nodes between the grid and the bricks
    kAny      // kernels: any of the three
};
__host__ __device__ inline Way way_of(int D, int M, int G) {
    return G > 0 && G == M ? kDirect : G == 0 && M == D ? kPlain : kNodes;
}

// CLIP: the walk also ends at r.s_end.  CHUNK: r.s_end is a piece's end, and
// cpl says whether the next piece starts outside this cell.
//
// A wave's time is the chain of its longest ray: about 350 instructions a step
// (223 vector, 127 scalar) and one or two index reads kept the SIMDs' waves
// issuing 25 % and waiting 75 % of their cycles, with 1.8 waves of 4 resident
// on average.  So the step is kept short: mirrored axes, entries that carry
// their own box, and a branch-free path for trees whose grid reaches the
// bricks, in kernels of its own (now about 210 instructions a step without the
// shading, 153 vector and 55 scalar).
template <bool CLIP, bool CHUNK, Way WAY>
struct Walker {
    int e;
    int bad;        // met a malformed entry
    bool inb;       // e is the brick entry of c
    // inb: byte offset of the brick; else (as int) the level of the node whose
    // entry e is, e describing a cell one level below, or -1: e is a grid entry
    uint32_t bofs;

    __device__ __forceinline__ void start(const Index& ix, const Ray& r, int* __restrict__ stk) {
        inb = false;
        bad = 0;
        const int N = ix.top + 1;
        const int c[3] = {r.c[0] ^ r.flip(0, N), r.c[1] ^ r.flip(1, N), r.c[2] ^ r.flip(2, N)};
        if (WAY == kDirect || (WAY == kNodes && ix.G > 0)) {
            bofs = 0xffffffffu;
            e = ix.entry(ix.grid_at(c));
        } else {
            bofs = 0;
            stk[0] = 0;
            e = ix.entry(ix.slot_at(c, 0, 0));
        }
    }

    // The descent of a tree without an index: e is the entry of a cell below a
    // level-bofs node.
    __device__ __forceinline__ void descend(const Index& ix, const int (&c)[3], int* __restrict__ stk, int& leaf,
                                            int& u) {
        int L = (int)bofs + 1;
        while ((e > 0) & (e < ix.n_top) & (L < ix.D)) {
            const int node = e;
            stk[L * kBlock] = node;
            e = ix.entry_now(ix.slot_at(c, node, L));
            ++L;
        }
        leaf = e < 0 ? -1 - e : -1;
        u = ix.D - L;
        if ((e > 0) | (leaf >= ix.n_leaves)) {  // past the nodes or leaves, or internal at the deepest level
            bad = 1;
            leaf = -1;
        }
    }

    // The descent of an index that keeps nodes: from the grid, or from the
    // deepest ancestor shared with the cell before, to a leaf, empty space or
    // a brick.  (An index is made from a checked array: no entry is malformed.)
    __device__ __forceinline__ void resolve(const Index& ix, const int (&c)[3], int* __restrict__ stk, bool exact,
                                            int& leaf, int& u, uint32_t& ext) {
        bool node = !inb & ((int)bofs >= 0);  // e is a node's entry
        if (!inb & !node & ((uint32_t)e < (uint32_t)kIdxCoarse)) {  // the grid names a node
            node = true;
            bofs = (uint32_t)ix.G;
            stk[ix.G * kBlock] = e;
            e = ix.entry_now(ix.slot_at(c, e, ix.G));
        }
        int L = (int)bofs + 1;  // e is the entry of the level-L cell holding c
        if (node) {
            while ((e > 0) & (e < ix.n_top)) {
                const int at = e;
                stk[L * kBlock] = at;
                e = ix.entry_now(ix.slot_at(c, at, L));
                ++L;
            }
            if (e > 0) {  // the level-M cube holding c is a brick: one load gives the leaf
                bofs = ix.brick0 + (uint32_t)(e - ix.n_top) * 2048u;
                e = ix.entry_now(ix.brick_at(bofs, c));
                inb = true;
                node = false;
            }
        }
        decode(ix, exact, node, leaf, u, ext);
        leaf = node ? -1 - e : leaf;
        u = node ? ix.D - L : u;
        ext = node ? 0u : ext;
    }
    // The leaf of a brick or grid entry (node: neither), -1 for empty space, log2 of the
    // edge of its cell, and for empty space how far the box reaches beyond.
    __device__ __forceinline__ void decode(const Index& ix, bool exact, bool node, int& leaf, int& u,
                                           uint32_t& ext) const {
        leaf = e < 0 ? -1 : (e >> 2) - 1;
        u = e < 0 ? po_index_unit(e) : e & 3;
        ext = e < 0 ? (uint32_t)e : 0u;
        if (exact) {
            u = e < 0 ? po_index_cube(e) : u;
            ext = 0;
        }
        if (ix.coarse) {
            if (!inb & !node & (e >= 0)) {
                // a leaf of level <= G: its number and level in a side table
                const uint32_t at = ix.bytes - 8u - ((uint32_t)(e & (kIdxCoarse - 1)) << 3);
                const auto q = __builtin_amdgcn_raw_buffer_load_b64(ix.rs, at, 0, 0);
                int l = (int)q[0], level = (int)q[1];
                asm volatile("" : "+v"(l), "+v"(level));
                leaf = l;
                u = ix.D - level;
            }
        }
    }

    // One cell.  cell_cap: the walk ends with it whatever it is; smp_cap: it
    // ends with it if it holds a sample.  At the end of the walk r.s and r.c
    // are at the start of the next cell.  A lane whose walk has ended (live
    // unset; cell_cap and inb set) keeps them.
    __device__ __forceinline__ Cell step(const Index& ix, Ray& r, bool exact, bool cell_cap, bool smp_cap,
                                         int* __restrict__ stk, bool live = true) {
        const int N = ix.top + 1;
        Cell o;
        // sign of the direction (0, or -1 on mirrored axes) and what follows
        // from it are made anew in every step: kept, they would take registers
        // that the records in flight need
        int sg[3], flip[3], c[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            int hi = __double2hiint(r.dg[k]);
            asm volatile("" : "+v"(hi));
            sg[k] = hi >> 31;
            flip[k] = sg[k] & ix.top;
            c[k] = r.c[k] ^ flip[k];
        }
        int leaf, u;
        uint32_t ext;
        if constexpr (WAY == kDirect) {
            if (!inb & ((uint32_t)e < (uint32_t)kIdxCoarse)) {
                bofs = ix.brick0 + (uint32_t)e * 2048u;
                e = ix.entry_now(ix.brick_at(bofs, c));
                inb = true;
            }
            decode(ix, exact, false, leaf, u, ext);
        } else if constexpr (WAY == kPlain) {
            descend(ix, c, stk, leaf, u);
            ext = 0;
        } else {
            resolve(ix, c, stk, exact, leaf, u, ext);
        }
        // exit parameter: the nearest far face
        int end[3];  // last cell of the box ahead
        double sk[3];
        const int w = (1 << u) - 1;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            end[k] = (((r.c[k] >> u) + (int)((ext >> (8 * k + 4 + (sg[k] & -4))) & 15u)) << u) | w;
            // the face behind it: end + 1, or in the tree's coordinates on a
            // mirrored axis 2^D - 1 - end
            sk[k] = ((double)((end[k] ^ flip[k]) + 1 + sg[k]) - r.og[k]) * r.inv[k];
        }
        double se = fmax(fmin(fmin(sk[0], sk[1]), sk[2]), r.s);
        o.cpl = true;
        if constexpr (CLIP) {
            if constexpr (CHUNK) {
                // a piece's cell is cut when the next piece starts inside it;
                // that piece finds its first cell from the point at s_end as
                // ray_setup does, so the two agree on every cell (a cell
                // ending at s_end up to rounding is complete here exactly
                // when the next piece starts in a later cell)
                if (se > r.s_end) {
                    bool inside = true;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const int d = ((r.cell_at(r.s_end, k, N) ^ flip[k]) >> u) - (c[k] >> u);
                        inside &= (d <= (int)((ext >> (8 * k + 4)) & 15u)) & (-d <= (int)((ext >> (8 * k)) & 15u));
                    }
                    o.cpl = !inside;
                }
            } else {
                o.cpl = se <= r.s_end;
            }
            se = fmin(se, r.s_end);
        }
        o.leaf = leaf;
        o.u = u;
        o.delta = (float)((se - r.s) * r.len);
        o.t_in = (float)(r.s * r.len);
        // next cell: axes whose face is reached step to the neighbouring cell;
        // the others take the finest cell of the exit point, kept inside the
        // current box and never moving against the ray (truncation equals
        // floor here: the result is clamped).  Clamped to the grid on both
        // sides before it is mirrored: a ray that has just entered through the
        // upper face of an axis it runs down is at 2^D up to rounding, which
        // mirrored would lie past the far end of any box
        int nc[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            int q = min(max((int)fma(se, r.dg[k], r.og[k]), 0), ix.top) ^ flip[k];
            asm volatile("" : "+v"(q));  // (or the compiler branches around it)
            nc[k] = sk[k] <= se ? end[k] + 1 : max(min(q, end[k]), r.c[k]);
        }
        bool out = ((nc[0] | nc[1] | nc[2]) & N) != 0;  // a coordinate of N: past the box
        if constexpr (CLIP) out |= se >= r.s_end;
        r.s = live ? se : r.s;
        const bool capped = !out & (cell_cap | (smp_cap & (leaf >= 0) & (o.delta > 0.0f)));
        r.more = live ? capped : r.more;
        o.last = out | capped;
        const uint32_t diff = (uint32_t)((r.c[0] ^ nc[0]) | (r.c[1] ^ nc[1]) | (r.c[2] ^ nc[2]));
        if (!out & live) {
#pragma unroll
            for (int k = 0; k < 3; ++k) r.c[k] = nc[k];
        }
        // read the next cell's entry (nothing after the last step: an offset
        // past the index): inside the same brick the brick's, else the grid's
        uint32_t at;
#pragma unroll
        for (int k = 0; k < 3; ++k) c[k] = nc[k] ^ flip[k];
        if constexpr (WAY == kDirect) {
            inb = inb & (diff < 8u);
            at = inb ? ix.brick_at(bofs, c) : ix.grid_at(c);
        } else if constexpr (WAY == kPlain) {
            at = 0;
            if (!o.last) {
                bofs = (uint32_t)(ix.D - 32 + __clz((int)diff));
                at = ix.slot_at(c, stk[(int)bofs * kBlock], (int)bofs);
            }
        } else {
            // the cells agree on the coordinate bits above the highest
            // differing one: without a grid the walk restarts below the deepest
            // common ancestor above the brick level (from the stack)
            const int D = ix.D, M = ix.M, G = ix.G;
            const int la = D - 32 + __clz((int)diff);
            at = 0;
            if (!o.last) {
                if (inb & (la >= M)) {
                    at = ix.brick_at(bofs, c);
                } else {
                    inb = false;
                    if ((G > 0) & (la < G)) {
                        bofs = 0xffffffffu;
                        at = ix.grid_at(c);
                    } else {
                        bofs = (uint32_t)la;
                        at = ix.slot_at(c, stk[la * kBlock], la);
                    }
                }
            }
        }
        e = ix.entry(o.last ? ix.bytes : at);
        return o;
    }
};

// ---------------------------------------------------------------------------
// Samples of a wave.  The data segments that its rays cross are collected in a
// queue in LDS, in the order of the steps, and shaded 64 at a time, one per
// lane whatever ray it belongs to; then every ray composites its own, front to
// back.
//
// Why a queue.  What a sample's colour and opacity need (leaf, segment length,
// the ray's basis values) does not depend on the samples in front of it.  Shaded
// by its own ray's lane, at the step that met it, a gather ran with the 20-30
// lanes of 64 that had a sample at that step, held the registers of all 64, and
// delayed the walk: loads return in order, so the read of a cell's entry waited
// for the gather before it.  Through the queue every gather and contraction
// runs with all lanes, and the steps between two of them wait for nothing but
// the index.
// ---------------------------------------------------------------------------
constexpr int kQueue = 2 * kBlock;  // up to 63 samples left over and 64 new ones
struct Sample {
    uint32_t leaf;
    float delta;     // segment length, world units
    uint32_t info;   // ray's lane | its cell is cut by the end of the walk << 6 | number of the step << 7
    uint32_t next;   // slot of the same ray's next sample
};
__device__ __forceinline__ Sample* sample_queue() {
    __shared__ __align__(16) Sample s_queue[kQueue];
    return s_queue;
}
// Start distances of the queue's segments (viewer).
__device__ __forceinline__ float* sample_starts() {
    __shared__ float s_t[kQueue];
    return s_t;
}
// Results of the 64 samples being shaded: {e^-(sigma delta), colour}, -1 for a
// leaf without density; the viewer's depth terms.
__device__ __forceinline__ float4* shaded() {
    __shared__ __align__(16) float4 s_shaded[kBlock];
    return s_shaded;
}
__device__ __forceinline__ float* shaded_depth() {
    __shared__ float s_depth[kBlock];
    return s_depth;
}
// Basis values of the wave's rays, [k / 4][lane][k % 4]: a lane reads its own in
// (K + 3) / 4 wide loads without bank conflicts.  In LDS they cost no registers
// while a walk steps (float32 K = 16: kept in registers, the walk's loop would
// spill at 4 waves per SIMD).
template <int K>
__device__ __forceinline__ float4* basis_values() {
    __shared__ __align__(16) float4 s_Y[(K + 3) / 4 * kBlock];
    return s_Y;
}
template <int K>
__device__ __forceinline__ void read_basis(uint32_t lane, float (&Y)[K]) {
    const float4* p = basis_values<K>() + lane;
#pragma unroll
    for (int q = 0; q < (K + 3) / 4; ++q) {
        const float4 v = p[q * kBlock];
        Y[4 * q] = v.x;
        if (4 * q + 1 < K) Y[4 * q + 1] = v.y;
        if (4 * q + 2 < K) Y[4 * q + 2] = v.z;
        if (4 * q + 3 < K) Y[4 * q + 3] = v.w;
    }
}
__device__ __forceinline__ int rank_in(uint64_t m) {  // lanes of m below this one
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

template <class S, class = void>
struct is_chunk : std::false_type {};
template <class S>
struct is_chunk<S, std::void_t<decltype(S::kChunk)>> : std::bool_constant<S::kChunk> {};

// Walks the segments of the wave's rays; every lane of the wave calls it, and
// those with `walk` set have a ray.  smp.shade(head, n) shades the n samples
// from slot `head` of the queue on, smp.composite(...) adds one of them to its
// ray and returns true to stop it, and smp.finish(head, n) then runs with every
// lane.
// Returns the number of cells visited, up to the one after the stop.
//
// A ray that has stopped early has walked up to a queue's length past the
// stop, which changes nothing but the time (malformed entries there are not
// counted).
//
// SPLIT: reaching `cap` data samples (exact: cells) with cells left stops the
// walk; it leaves r.s and r.c at the start of the next cell and sets r.more
// (unless the last sample ended it by early stopping), so that it can be
// resumed or handed on.  (Samples, so that the hand-off does not depend on how
// empty space is crossed.)  So does reaching max_steps, which without SPLIT is
// an error.
template <class Sampler, bool SPLIT, Way WAY>
__device__ __forceinline__ int march_queued(const Index& ix, Ray& r, bool walk, int max_steps, int cap, bool exact,
                                            int* __restrict__ stk, Sampler& smp) {
    constexpr bool CHUNK = is_chunk<Sampler>::value;
    constexpr bool VIEW = Sampler::kView;
    Walker<Sampler::kClip, CHUNK, WAY> w;
    Sample* Q = sample_queue();
    int steps = 0, nt = 0, bad_step = kNoCap;
    // this ray's samples in the queue: how many, the first and the last
    int mine = 0;
    uint32_t first = 0, last = 0;
    // the wave's queue: first slot and length
    uint32_t head = 0, count = 0;
    r.more = false;
    if (walk) w.start(ix, r, stk);
    while (true) {
        bool take = false;
        Cell c;
        if (walk) {
            ++steps;
            const bool cell_cap = (steps >= max_steps) | (SPLIT && exact && steps >= cap);
            c = w.step(ix, r, exact, cell_cap, SPLIT && !exact && nt + 1 >= cap, stk);
            if (w.bad & (bad_step == kNoCap)) bad_step = steps;
            walk = !c.last;
            take = (c.leaf >= 0) & (c.delta > 0.0f);
            if constexpr (CHUNK) {
                smp.cpl = c.cpl;
                if (steps == 1) {
                    if (smp.skip0 < 0) smp.skip0 = c.delta > 0.0f ? 0 : 1;
                    // a piece's first cell without a sample (the zero-length
                    // rest of a cell the previous piece cut, or a start on a
                    // face) still carries the stop test at its end
                    if (!take && smp.test_first(c.cpl)) {
                        walk = false;
                        r.more = false;
                    }
                }
            }
        }
        const uint64_t m = __ballot(take);
        if (m != 0ull) {
            if (take) {
                const uint32_t slot = (head + count + (uint32_t)rank_in(m)) % kQueue;
                Sample q;
                q.leaf = (uint32_t)c.leaf;
                q.delta = c.delta;
                q.info = threadIdx.x | (c.cpl ? 0u : 64u) | (uint32_t)steps << 7;
                q.next = 0;
                Q[slot] = q;
                if constexpr (VIEW) sample_starts()[slot] = c.t_in;
                if (mine == 0)
                    first = slot;
                else
                    Q[last].next = slot;
                last = slot;
                ++mine;
                ++nt;
            }
            count += (uint32_t)__popcll(m);
        }
        const bool walking = __ballot(walk) != 0ull;
        if (count >= (uint32_t)kBlock || (!walking && count > 0)) {
            const uint32_t n = min(count, (uint32_t)kBlock);
            __builtin_amdgcn_wave_barrier();
            smp.shade(head, n);
            __builtin_amdgcn_wave_barrier();
            while (mine > 0) {
                const uint32_t at = (first - head) % kQueue;
                if (at >= n) break;
                const Sample q = Q[first];
                --mine;
                const bool stop = smp.composite(q, first, at);
                first = q.next;
                if (stop) {
                    // the stop counts the cell behind it, where there is one
                    const int seen = (int)(q.info >> 7) + 1;
                    steps = walk ? seen : min(steps, seen);
                    walk = false;
                    r.more = false;
                    mine = 0;
                }
            }
            __builtin_amdgcn_wave_barrier();
            smp.finish(head, n);
            head = (head + n) % kQueue;
            count -= n;
        } else if (!walking) {
            break;
        }
    }
    r.nt = exact ? steps : nt;
    // a lane that met a malformed entry or the step cap is counted once
    if ((bad_step <= steps) | (!SPLIT & r.more)) atomicAdd(&g_po_errors, 1ull);
    return steps;
}

// The same walk with every sample shaded by its own ray's lane, one step after
// the step that met it: smp.issue(leaf, delta, t, cut) starts the loads of the
// leaf (leaf -1: a lane without a sample, which loads nothing), and
// smp.consume() shades and composites them and returns true to stop the walk.
// The read of the next cell's entry is started before, so that compositing
// runs while it is in flight.
template <class Sampler, bool SPLIT, Way WAY>
__device__ __forceinline__ int march_inline(const Index& ix, Ray& r, int max_steps, int cap, bool exact,
                                            int* __restrict__ stk, Sampler& smp) {
    constexpr bool CHUNK = is_chunk<Sampler>::value;
    Walker<Sampler::kClip, CHUNK, WAY> w;
    int steps = 0, nt = 0;
    bool pending = false, stop = false;
    w.start(ix, r, stk);
    __builtin_amdgcn_sched_barrier(0);  // (the entry's load first)
    // an empty gather, so that every path into the loop has the same loads in
    // flight behind the entry (the compiler then waits for the entry alone)
    smp.issue(-1, 0.0f, 0.0f, false);
    while (true) {
        ++steps;
        const bool cell_cap = (steps >= max_steps) | (SPLIT && exact && steps >= cap);
        const Cell c = w.step(ix, r, exact, cell_cap, SPLIT && !exact && nt + 1 >= cap, stk);
        __builtin_amdgcn_sched_barrier(0);
        if (pending) stop = smp.consume();
        pending = !stop & (c.leaf >= 0) & (c.delta > 0.0f);
        if constexpr (CHUNK) {
            smp.cpl = c.cpl;
            if (steps == 1) {
                if (smp.skip0 < 0) smp.skip0 = c.delta > 0.0f ? 0 : 1;
                // a piece's first cell without a sample (the zero-length rest of
                // a cell the previous piece cut, or a start on a face) still
                // carries the stop test at its end
                if (!pending) stop = smp.test_first(c.cpl);
            }
        }
        smp.issue(pending ? c.leaf : -1, c.delta, c.t_in, !c.cpl);
        nt += pending ? 1 : 0;
        if (c.last | stop) break;
    }
    const bool capped = r.more;
    if (pending) stop = smp.consume();
    r.more &= !stop;
    r.nt = exact ? steps : nt;
    // a lane that met a malformed entry or the step cap is counted once
    if (w.bad | (!SPLIT & capped)) atomicAdd(&g_po_errors, 1ull);
    return steps;
}

// march_inline for records that the four lanes of a quad load together: every
// lane of the wave takes every step, a ray that has ended standing still, and
// smp.consume(pending) runs in all of them.
//
// Why.  A float32 record of 16 coefficients is 192 bytes, 12 loads a lane, and
// every load that sends 64 lanes to 64 lines holds the address unit four times
// as long as one that sends each quad to one line (12 loads of the record's
// first 64 bytes took nearly as long as the whole record, 4 of them 28 % less
// of an 800x800 frame and 38 % less of 1920x1080).  By quads one load reads a
// channel of one of the quad's four records, 64 bytes side by side; each lane
// contracts its quarter with the basis of the ray it belongs to, and the four
// parts meet in three exchanges inside the quad.  800x800 float32 K = 16: 427
// to 403 us, 1920x1080 881 to 771.  Not for float16 (8 bytes a lane and so
// twice the loads: 605 to 723 us at 1920x1080), nor for K = 9, whose channels
// are no whole lines.
template <class Sampler, bool SPLIT, Way WAY>
__device__ __forceinline__ int march_quads(const Index& ix, Ray& r, bool walk, int max_steps, int cap, bool exact,
                                           int* __restrict__ stk, Sampler& smp) {
    constexpr bool CHUNK = is_chunk<Sampler>::value;
    Walker<Sampler::kClip, CHUNK, WAY> w;
    int steps = 0, nt = 0;
    bool live = walk, pending = false, stop = false;
    r.more = false;
    if (!walk) {  // any ray inside the box
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            r.og[k] = 0.0;
            r.dg[k] = r.inv[k] = 1.0;
            r.c[k] = 0;
        }
        r.s = r.s_end = 0.0;
        r.len = 1.0;
    }
    w.start(ix, r, stk);
    __builtin_amdgcn_sched_barrier(0);
    smp.issue(-1, 0.0f, 0.0f, false);
    do {
        steps += live ? 1 : 0;
        w.e = live ? w.e : 0;  // (past the end: no leaf)
        w.inb |= !live;
        const bool cell_cap = !live | (steps >= max_steps) | (SPLIT && exact && steps >= cap);
        const Cell c = w.step(ix, r, exact, cell_cap, SPLIT && !exact && nt + 1 >= cap, stk, live);
        __builtin_amdgcn_sched_barrier(0);
        if (__ballot(pending) != 0ull) stop |= smp.consume(pending);
        pending = live & !stop & (c.leaf >= 0) & (c.delta > 0.0f);
        if constexpr (CHUNK) {
            if (live) {
                smp.cpl = c.cpl;
                if (steps == 1) {
                    if (smp.skip0 < 0) smp.skip0 = c.delta > 0.0f ? 0 : 1;
                    if (!pending) stop = smp.test_first(c.cpl);
                }
            }
        }
        smp.issue(pending ? c.leaf : -1, c.delta, c.t_in, !c.cpl);
        nt += pending ? 1 : 0;
        live &= !(c.last | stop);
    } while (__ballot(live) != 0ull);
    const bool capped = r.more;
    if (__ballot(pending) != 0ull) stop |= smp.consume(pending);
    r.more &= !stop;
    r.nt = exact ? steps : nt;
    // a lane that met a malformed entry or the step cap is counted once
    if (w.bad | (!SPLIT & capped)) atomicAdd(&g_po_errors, 1ull);
    return steps;
}

// Which of the three a sampler takes: quads where its records are whole lines by
// channel (kQuads); else the queue (kQueued) or its own lane.  The queue costs
// about 45 instructions a step, and saves the waits on gathers and the lanes
// without a sample.  It pays where a sample is expensive: records over 192 bytes (SG-25
// 400x400, float32: 0.219 against 0.259 ms), codebooks (640x480: 0.306 against
// 0.377) and gradients (8191 rays forward and backward: 0.291 against 0.486),
// not for smaller records (800x800 float32 K = 16: 0.497 against 0.451) or the
// densities alone (filter 800x800: 0.379 against 0.330).
template <class Sampler, bool SPLIT, Way WAY>
__device__ __forceinline__ int march_way(const Index& ix, Ray& r, bool walk, int max_steps, int cap, bool exact,
                                         int* __restrict__ stk, Sampler& smp) {
    if constexpr (Sampler::kQueued) {
        return march_queued<Sampler, SPLIT, WAY>(ix, r, walk, max_steps, cap, exact, stk, smp);
    } else if constexpr (Sampler::kQuads) {
        return march_quads<Sampler, SPLIT, WAY>(ix, r, walk, max_steps, cap, exact, stk, smp);
    } else {
        r.more = false;
        r.nt = 0;
        return walk ? march_inline<Sampler, SPLIT, WAY>(ix, r, max_steps, cap, exact, stk, smp) : 0;
    }
}
template <bool SPLIT, Way WAY, class Sampler>
__device__ __forceinline__ int march(const KTree& tr, Ray& r, bool walk, int max_steps, int cap, bool exact,
                                     int* __restrict__ stk, Sampler& smp) {
    const Index ix(tr);
    if constexpr (WAY != kAny) {
        return march_way<Sampler, SPLIT, WAY>(ix, r, walk, max_steps, cap, exact, stk, smp);
    } else {
        switch (way_of(ix.D, ix.M, ix.G)) {
        case kDirect: return march_way<Sampler, SPLIT, kDirect>(ix, r, walk, max_steps, cap, exact, stk, smp);
        case kPlain: return march_way<Sampler, SPLIT, kPlain>(ix, r, walk, max_steps, cap, exact, stk, smp);
        default: return march_way<Sampler, SPLIT, kNodes>(ix, r, walk, max_steps, cap, exact, stk, smp);
        }
    }
}

template <typename T, int K, int NW>
__device__ __forceinline__ float dot_channel(const uint32_t (&w)[NW], int base, const float (&Y)[K]) {
    if constexpr (std::is_same_v<T, float> && K == 16) {
        // in four parts, as quad_dots adds them (the backward's colours and the
        // render's have the same bits)
        float z[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            z[q] = word_elem<T>(w, base + 4 * q) * Y[4 * q];
#pragma unroll
            for (int k = 1; k < 4; ++k) z[q] = fmaf(word_elem<T>(w, base + 4 * q + k), Y[4 * q + k], z[q]);
        }
        return (z[0] + z[1]) + (z[2] + z[3]);
    } else {
        float z = word_elem<T>(w, base) * Y[0];
#pragma unroll
        for (int k = 1; k < K; ++k) z = fmaf(word_elem<T>(w, base + k), Y[k], z);
        return z;
    }
}

// Loads one record (NL elements, a whole number of VEC-byte vectors) at byte
// offset `off` of a raw buffer.  An offset at or beyond the end of the buffer
// returns zeros and touches no memory, which lets lanes without a sample run
// the same straight-line code.
template <typename T, int NL, int VEC>
__device__ __forceinline__ void load_record(__amdgpu_buffer_rsrc_t rs, uint32_t off, uint32_t (&w)[Words<T, NL>::N]) {
    static_assert(Words<T, NL>::NB % VEC == 0, "a record is loaded in whole vectors");
#pragma unroll
    for (int v = 0; v < Words<T, NL>::NB / VEC; ++v) {
        if constexpr (VEC == 16) {
            const auto q = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * v, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) w[4 * v + i] = q[i];
        } else if constexpr (VEC == 8) {
            const auto q = __builtin_amdgcn_raw_buffer_load_b64(rs, off + 8 * v, 0, 0);
            w[2 * v] = q[0];
            w[2 * v + 1] = q[1];
        } else {
            w[v] = __builtin_amdgcn_raw_buffer_load_b32(rs, off + 4 * v, 0, 0);
        }
    }
}

// Value of x in lane I of this lane's quad, and in the lane whose number
// differs from this one's in bit BIT.
template <int I>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x55 * I, 0xf, 0xf, true);
}
template <int BIT>
__device__ __forceinline__ float quad_swap(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), BIT == 0 ? 0xB1 : 0x4E, 0xf, 0xf, true));
}
// Basis values of the wave's rays as quads read them: [lane][k], the 16
// float4 of four lanes padded to 20, so that the quads of 16 lanes read
// different banks.
constexpr int kQuadBasis = 20;
__device__ __forceinline__ float4* quad_basis() {
    __shared__ __align__(16) float4 s_Yq[kQuadBasis * kBlock / 4];
    return s_Yq;
}

// Leaf arrays of a tree with float32 or float16 records, bound to buffers.
template <typename T, int K, int VEC, int NL>
struct Records {
    __amdgpu_buffer_rsrc_t sig, shb;
    uint32_t sig_end, sh_end, rec_bytes;

    __device__ __forceinline__ void bind(const KTree& tr) {
        sig_end = held(tr.sigma_bytes);
        sh_end = held(tr.sh_bytes);
        sig = raw_rsrc(held(tr.sigma), sig_end);
        shb = raw_rsrc(held(tr.sh), sh_end);
        rec_bytes = held((uint32_t)tr.stride * (uint32_t)sizeof(T));
    }
    // Density (clamped) and colour of the leaf of this lane's sample, for the
    // ray of lane src; on false: no sample.
    __device__ __forceinline__ float eval(bool on, uint32_t leaf, uint32_t src, float (&col)[3]) const {
        uint32_t w[Words<T, NL>::N];
        const uint32_t raw = sigma_buf(sig, on ? leaf * (uint32_t)sizeof(T) : sig_end, (T*)nullptr);
        load_record<T, NL, VEC>(shb, on ? leaf * rec_bytes : sh_end, w);
        float Y[K];
        read_basis<K>(src, Y);
#pragma unroll
        for (int c = 0; c < 3; ++c) col[c] = sigmoid(dot_channel<T, K>(w, c * K, Y));
        return fmaxf(sigma_of<T>(raw), 0.0f);
    }
};

// Codebook leaves (App. B.2): the record holds one 16-bit codebook position
// per basis function; a sample gathers the K float16 colours (8 bytes each,
// from the per-basis codebooks) and shades as an SH leaf.
template <int K, int VEC, int NL>
struct CbRecords {
    __amdgpu_buffer_rsrc_t sig, shb, cb;
    uint32_t sig_end, sh_end, rec_bytes, cb_basis_bytes;

    __device__ __forceinline__ void bind(const KTree& tr) {
        sig = raw_rsrc(tr.sigma, tr.sigma_bytes);
        shb = raw_rsrc(tr.sh, tr.sh_bytes);
        sig_end = tr.sigma_bytes;
        sh_end = tr.sh_bytes;
        rec_bytes = (uint32_t)tr.stride * 2u;
        cb_basis_bytes = (uint32_t)tr.cb_entries * 8u;
        cb = raw_rsrc(tr.codebook, (uint32_t)K * cb_basis_bytes);
    }
    __device__ __forceinline__ float eval(bool on, uint32_t leaf, uint32_t src, float (&col)[3]) const {
        uint32_t w[Words<__half, NL>::N];
        const uint32_t raw = sigma_buf(sig, on ? leaf * 2u : sig_end, (__half*)nullptr);
        load_record<__half, NL, VEC>(shb, on ? leaf * rec_bytes : sh_end, w);
        const float s = fmaxf(sigma_of<__half>(raw), 0.0f);
        float Y[K];
        read_basis<K>(src, Y);
        uint32_t e0[K], e1[K];
        const uint32_t none = (uint32_t)K * cb_basis_bytes;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t pos = (w[k >> 1] >> (16 * (k & 1))) & 0xffffu;
            const auto q = __builtin_amdgcn_raw_buffer_load_b64(
                cb, s > 0.0f ? (uint32_t)k * cb_basis_bytes + pos * 8u : none, 0, 0);
            e0[k] = q[0];
            e1[k] = q[1];
        }
        float z0 = 0.0f, z1 = 0.0f, z2 = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            z0 = fmaf(__half2float(__ushort_as_half((unsigned short)(e0[k] & 0xffffu))), Y[k], z0);
            z1 = fmaf(__half2float(__ushort_as_half((unsigned short)(e0[k] >> 16))), Y[k], z1);
            z2 = fmaf(__half2float(__ushort_as_half((unsigned short)(e1[k] & 0xffffu))), Y[k], z2);
        }
        col[0] = sigmoid(z0);
        col[1] = sigmoid(z1);
        col[2] = sigmoid(z2);
        return s;
    }
};

// The integral of t sigma T(t) over a segment [ta, ta + delta] of optical
// depth tau, from T = 1 (ex = e^-tau): ta alpha + delta f, f = alpha / tau -
// e^-tau, from its series below tau = 0.05 (alpha / tau cancels there).
__device__ __forceinline__ float depth_term(float tau, float ex, float delta, float ta) {
    const float al = 1.0f - ex;
    const float f = tau < 0.05f
                        ? tau * (0.5f - tau * (1.0f / 3.0f - tau * (0.125f - tau * (1.0f / 30.0f - tau * (1.0f / 144.0f)))))
                        : al / tau - ex;
    return fmaf(ta, al, delta * f);
}

// Forward shading and compositing of the samples of a wave's rays (Sec. 3
// eqn:quad, Sec. 4.1 colour, App. B.3 clamp of the raw density).  VIEW adds
// the viewer outputs of Sec. 5.5: the expected termination distance and the
// end of the walk at a slicing plane.
template <class Rec, bool VIEW>
struct FwdQueued : Rec {
    static constexpr bool kClip = VIEW;
    static constexpr bool kView = VIEW;
    static constexpr bool kQueued = true;
    static constexpr bool kQuads = false;
    float stopT;
    float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, Tl = 1.0f;
    float dep = 0.0f;
    int ns = 0;

    __device__ __forceinline__ void shade(uint32_t head, uint32_t n) {
        const uint32_t slot = (head + threadIdx.x) % kQueue;
        const Sample q = sample_queue()[slot];
        const bool on = threadIdx.x < n;
        float col[3];
        const float s = Rec::eval(on, q.leaf, q.info & 63u, col);
        const float tau = s * q.delta;
        const float ex = __expf(-tau);
        shaded()[threadIdx.x] = make_float4(s > 0.0f ? ex : -1.0f, col[0], col[1], col[2]);
        if constexpr (VIEW) shaded_depth()[threadIdx.x] = depth_term(tau, ex, q.delta, sample_starts()[slot]);
    }
    // Composites one sample of this lane's ray (slot of the queue, number `at`
    // of the shaded ones); true when early stopping ends the ray.
    __device__ __forceinline__ bool composite(const Sample&, uint32_t, uint32_t at) {
        ++ns;
        const float4 v = shaded()[at];
        if (v.x < 0.0f) return false;
        const float wgt = Tl * (1.0f - v.x);
        c0 = fmaf(wgt, v.y, c0);
        c1 = fmaf(wgt, v.z, c1);
        c2 = fmaf(wgt, v.w, c2);
        if constexpr (VIEW) dep = fmaf(Tl, shaded_depth()[at], dep);
        Tl = Tl * v.x;
        return Tl < stopT;
    }
    __device__ __forceinline__ void finish(uint32_t, uint32_t) {}
};

// The same for samples shaded by their own ray's lane (march_inline, march_quads).
template <typename T, int K, int VEC, int NL, bool VIEW>
struct FwdInline : Records<T, K, VEC, NL> {
    static constexpr bool kClip = VIEW;
    static constexpr bool kView = VIEW;
    static constexpr bool kQueued = false;
    float stopT;
    float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, Tl = 1.0f;
    float dep = 0.0f;
    int ns = 0;
    // a record of 16 float32 per channel is loaded by the quad of lanes
    static constexpr bool kQuads = std::is_same_v<T, float> && K == 16 && VEC == 16;
    // in flight
    uint32_t raw;
    float delta, ta;
    bool cut;
    uint32_t w[Words<T, NL>::N];  // kQuads: [channel][lane of the quad][4], this lane's quarter of its records

    __device__ __forceinline__ void issue(int leaf, float d, float t_in, bool is_cut) {
        raw = sigma_buf(this->sig, leaf < 0 ? this->sig_end : (uint32_t)leaf * (uint32_t)sizeof(T), (T*)nullptr);
        const uint32_t off = leaf < 0 ? this->sh_end : (uint32_t)leaf * this->rec_bytes;
        if constexpr (kQuads) {
            const uint32_t l = 16u * (threadIdx.x & 3u);
            const uint32_t rec[4] = {quad_bcast<0>(off) + l, quad_bcast<1>(off) + l, quad_bcast<2>(off) + l,
                                     quad_bcast<3>(off) + l};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const auto q = __builtin_amdgcn_raw_buffer_load_b128(this->shb, rec[i] + 64 * c, 0, 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j) w[16 * c + 4 * i + j] = q[j];
                }
        } else {
            load_record<T, NL, VEC>(this->shb, off, w);
        }
        delta = d;
        cut = is_cut;
        if constexpr (VIEW) ta = t_in;
    }
    // The contraction of every lane's record, by the quads.
    __device__ __forceinline__ void quad_dots(float (&z)[3]) const {
        const uint32_t lane = threadIdx.x;
        const bool b0 = (lane & 1u) != 0u, b1 = (lane & 2u) != 0u;
        const float4* Yq = quad_basis() + (lane >> 2) * kQuadBasis + (lane & 3u);
        float p[3][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 y = Yq[4 * i];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const uint32_t* x = w + 16 * c + 4 * i;
                p[c][i] = fmaf(__uint_as_float(x[3]), y.w,
                               fmaf(__uint_as_float(x[2]), y.z,
                                    fmaf(__uint_as_float(x[1]), y.y, __uint_as_float(x[0]) * y.x)));
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            float t[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float keep = b0 ? p[c][2 * h + 1] : p[c][2 * h], give = b0 ? p[c][2 * h] : p[c][2 * h + 1];
                t[h] = keep + quad_swap<0>(give);
            }
            const float keep = b1 ? t[1] : t[0], give = b1 ? t[0] : t[1];
            z[c] = keep + quad_swap<1>(give);
        }
    }
    __device__ __forceinline__ bool consume(bool pending = true) {
        float z[3];
        if constexpr (kQuads) quad_dots(z);
        if (kQuads & !pending) return false;
        ++ns;
        const float s = fmaxf(sigma_of<T>(raw), 0.0f);
        if (!(s > 0.0f)) return false;
        const float tau = s * delta;
        const float ex = __expf(-tau);
        const float wgt = Tl * (1.0f - ex);
        if constexpr (!kQuads) {
            float Y[K];
            read_basis<K>(threadIdx.x, Y);
#pragma unroll
            for (int c = 0; c < 3; ++c) z[c] = dot_channel<T, K>(w, c * K, Y);
        }
        c0 = fmaf(wgt, sigmoid(z[0]), c0);
        c1 = fmaf(wgt, sigmoid(z[1]), c1);
        c2 = fmaf(wgt, sigmoid(z[2]), c2);
        if constexpr (VIEW) dep = fmaf(Tl, depth_term(tau, ex, delta, ta), dep);
        Tl = Tl * ex;
        return Tl < stopT;
    }
};

// The SH or SG basis of a variant at this lane's ray direction, into the
// wave's LDS array.
template <int K, int V, bool QUADS = false>
__device__ __forceinline__ void init_basis(const KTree& tr, const KOpts& op, const Ray& r) {
    float Y[K];
    if constexpr (V == PO_FWD_SG)
        sg_basis<K>(tr.lobes, r.dn[0], r.dn[1], r.dn[2], Y);
    else if constexpr (V == PO_FWD_VIEW)
        colour_basis<K>(tr, r.dn[0], r.dn[1], r.dn[2], Y);
    else
        sh_basis<K>(r.dn[0], r.dn[1], r.dn[2], Y);
    if constexpr (V == PO_FWD_VIEW) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if ((op.sh_off >> k) & 1u) Y[k] = 0.0f;
    }
    float4* p = QUADS ? quad_basis() + (threadIdx.x >> 2) * kQuadBasis + (threadIdx.x & 3u) * 4u
                      : basis_values<K>() + threadIdx.x;
#pragma unroll
    for (int q = 0; q < (K + 3) / 4; ++q)
        p[QUADS ? q : q * kBlock] = make_float4(Y[4 * q], 4 * q + 1 < K ? Y[4 * q + 1] : 0.0f, 4 * q + 2 < K ? Y[4 * q + 2] : 0.0f,
                                    4 * q + 3 < K ? Y[4 * q + 3] : 0.0f);
}

// One chunk [s_lo, s_hi] of a split ray.  The chunk composites from T = 1
// (or from a known transmittance when it is walked again); because
// compositing is associative, chunk results combine front to back with the
// over operator.  Early stopping is tested where the sequential walk tests it,
// at the end of a cell: a sample whose cell continues past s_hi (cut by the
// chunk boundary: the next chunk starts inside it) is composited without a
// test, and its remainder, the first cell of the next chunk, carries the
// test, also when it has zero length and takes no sample.  Tlast is T after the last
// tested sample (-1: none); the chunk stops itself once T < stopT there,
// since its walk cannot matter past that point for any transmittance in
// front of it.
template <class Base>
struct ChunkOf : Base {
    static constexpr bool kClip = true;
    static constexpr bool kChunk = true;
    bool cpl = true;        // the last cell walked ends inside the piece
    bool hit = false;       // stopped by stopT
    bool smp_cut = false;   // the last composited sample was cut by the walk's end
    int skip0 = -1;         // 1: the first cell had zero length (the walk began on its far face)
    float Tlast = -1.0f;

    __device__ __forceinline__ bool composite(const Sample& q, uint32_t slot, uint32_t at) {
        return tested(Base::composite(q, slot, at), (q.info & 64u) != 0u);
    }
    __device__ __forceinline__ bool consume(bool pending = true) {
        const bool st = Base::consume(pending);
        return pending && tested(st, this->cut);
    }
    __device__ __forceinline__ bool tested(bool st, bool is_cut) {
        smp_cut = is_cut;
        if (is_cut) return false;
        Tlast = this->Tl;
        hit |= st;
        return st;
    }
    // the stop test at the end of a first cell that took no sample (c: the
    // cell ends inside the piece)
    __device__ __forceinline__ bool test_first(bool c) {
        if (!c) return false;
        Tlast = this->Tl;
        const bool st = this->Tl < this->stopT;
        hit |= st;
        return st;
    }
};

// Samplers: a whole ray's, and of the split render the first walk's and a
// piece's.  Pieces of plain walks shade records over 192 bytes in their own
// lane: the queue costs by the step, of which they take half as many again
// (300,000 rays, float32 K = 25, depth 8: 693 us through it, 555 without), while
// whole rays, whose lanes drift apart, still gain by it (1920x1080: 995, 1210).
template <typename T, int K, int VEC, int NL, int V, bool QUEUE = (sizeof(T) * 3 * K > 192)>
using RaySampler = std::conditional_t<
    V == PO_FWD_CB, FwdQueued<CbRecords<K, VEC, NL>, false>,
    std::conditional_t<QUEUE, FwdQueued<Records<T, K, VEC, NL>, V == PO_FWD_VIEW>,
                       FwdInline<T, K, VEC, NL, V == PO_FWD_VIEW>>>;
template <typename T, int K, int VEC, int NL, int V, Way WAY>
using FirstSampler = RaySampler<T, K, VEC, NL, V, (sizeof(T) * 3 * K > 192 && WAY != kPlain)>;
template <typename T, int K, int VEC, int NL, int V, Way WAY>
using ChunkSampler = ChunkOf<FirstSampler<T, K, VEC, NL, V, WAY>>;

// Binds a forward sampler to a tree (every lane), and a ray's basis.
template <int K, int V, class Smp>
__device__ __forceinline__ void fwd_init(Smp& smp, const KTree& tr, const KOpts& op, bool ray, const Ray& r) {
    smp.bind(tr);
    smp.stopT = op.stop_T;
    if (ray) init_basis<K, V, Smp::kQuads>(tr, op, r);
}

// Renders the wave's rays (valid: this lane has one): colour (background
// included), final T, samples, steps and, in the viewer variant, the expected
// termination distance, SH subsets and the slicing plane.  V is a PO_FWD_*
// variant.
template <typename T, int K, int VEC, int NL, int V, Way WAY>
__device__ __forceinline__ void render_one(const KTree& tr, const KOpts& op, bool valid, const double (&o)[3],
                                           const double (&d)[3], int* __restrict__ stk, float (&C)[3], float& Tr,
                                           int& ns, int& steps, float& dep) {
    Ray r;
    double s_lo = 0.0, s_hi = 1e300;
    if constexpr (V == PO_FWD_VIEW) clip_range(op, o, d, s_lo, s_hi);
    const bool walk = valid && ray_setup(tr, o, d, r, s_lo, s_hi);
    RaySampler<T, K, VEC, NL, V> smp;
    fwd_init<K, V>(smp, tr, op, walk, r);
    steps = march<false, WAY>(tr, r, walk, op.max_steps, kNoCap, exact_cells(op), stk, smp);
    Tr = smp.Tl;
    ns = smp.ns;
    dep = smp.dep;
    C[0] = fmaf(Tr, op.bg[0], smp.c0);
    C[1] = fmaf(Tr, op.bg[1], smp.c1);
    C[2] = fmaf(Tr, op.bg[2], smp.c2);
}

// Workgroups are dispatched round-robin over the 8 XCDs (workgroup b runs on
// XCD b % 8).  Remap so that each XCD receives one contiguous range of the
// logical workgroup order (neighbouring tiles share its L2).  The grid has
// 8 * ceil(n / 8) workgroups; returns -1 for the padding ones.
__device__ __forceinline__ int64_t xcd_swizzle(int64_t b, int64_t n_logical) {
    const int64_t per = (n_logical + 7) / 8;
    const int64_t l = (b % 8) * per + b / 8;
    return l < n_logical ? l : -1;
}

// Logical workgroup of hardware workgroup b when runs of `chunk` logical
// workgroups (a tile row) are dealt round-robin over the 8 XCDs: XCD x gets
// runs x, x + 8, ...  The grid has 8 * chunk * ceil(ceil(n_logical / chunk) / 8)
// workgroups (rows_grid); returns -1 for the padding ones.  Camera walks deal
// tile rows this way: every XCD then holds a share of the frame's longest
// walks, which crowd into the middle rows (one-pass depth-9 800x800 FP32
// frame: 0.706 against 0.854 ms with a contiguous band of rows per XCD).
__device__ __forceinline__ int64_t xcd_interleave(int64_t b, int64_t n_logical, int64_t chunk) {
    const int64_t x = b & 7, j = b >> 3;
    const int64_t l = ((j / chunk) * 8 + x) * chunk + (j % chunk);
    return l < n_logical ? l : -1;
}
template <typename T, int K, int VEC, int NL, int V, Way WAY>
__global__ __launch_bounds__(kBlock) void k_render_rays(KTree tr, int64_t n, int64_t n_blocks,
                                                        const float* __restrict__ o,
                                                        const float* __restrict__ d, KOpts op,
                                                        float* __restrict__ rgb, float* __restrict__ aux) {
    const int64_t blk = xcd_swizzle(blockIdx.x, n_blocks);
    if (blk < 0) return;
    const int64_t i = blk * kBlock + threadIdx.x;
    const bool valid = i < n;
    double ro[3] = {0.0, 0.0, 0.0}, rd[3] = {0.0, 0.0, 0.0};
    if (valid) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            ro[k] = (double)o[3 * i + k];
            rd[k] = (double)d[3 * i + k];
        }
    }
    float C[3], Tr, dep;
    int ns, steps;
    extern __shared__ int po_stack[];
    render_one<T, K, VEC, NL, V, WAY>(tr, op, valid, ro, rd, po_stack + threadIdx.x, C, Tr, ns, steps, dep);
    if (!valid) return;
    rgb[3 * i + 0] = C[0];
    rgb[3 * i + 1] = C[1];
    rgb[3 * i + 2] = C[2];
    if constexpr (V == PO_FWD_VIEW) {
        if (aux) {
            aux[4 * i + 0] = Tr;
            aux[4 * i + 1] = (float)ns;
            aux[4 * i + 2] = (float)steps;
            aux[4 * i + 3] = dep;
        }
    }
}

// Pinhole ray through the centre of pixel (px, py), in FP64 like the rest of
// the ray geometry (direction not normalised).
__device__ __forceinline__ void pixel_ray(const KCam& cam, int px, int py, double (&ro)[3], double (&rd)[3]) {
    const double x = ((double)px + 0.5 - (double)cam.cx) / (double)cam.fx;
    const double y = -(((double)py + 0.5 - (double)cam.cy) / (double)cam.fy);
    const float* M = cam.c2w;
    rd[0] = (double)M[0] * x + (double)M[1] * y - (double)M[2];
    rd[1] = (double)M[4] * x + (double)M[5] * y - (double)M[6];
    rd[2] = (double)M[8] * x + (double)M[9] * y - (double)M[10];
    ro[0] = (double)M[3];
    ro[1] = (double)M[7];
    ro[2] = (double)M[11];
}

__global__ __launch_bounds__(256) void k_camera_rays(KCam cam, float* __restrict__ o, float* __restrict__ d) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= (int64_t)cam.W * cam.H) return;
    double ro[3], rd[3];
    pixel_ray(cam, (int)(p % cam.W), (int)(p / cam.W), ro, rd);
    const double il = 1.0 / sqrt(rd[0] * rd[0] + rd[1] * rd[1] + rd[2] * rd[2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        o[3 * p + k] = (float)ro[k];
        d[3 * p + k] = (float)(rd[k] * il);
    }
}

template <int MAXJ>
struct KBatch {
    KJob job[MAXJ];
    int32_t n_jobs;
    int32_t n_blocks;
};
// passed by value as the kernel argument block, limited to 4 KiB
static_assert(sizeof(KBatch<PO_BATCH_MAX_JOBS>) <= 4096, "batched kernel arguments exceed 4 KiB");

// Camera jobs: a 16x16 tile is rendered by four single-wave workgroups, one
// per 8x8 quadrant; lane l takes the pixel (l & 7, l >> 3) of its quadrant.
template <typename T, int K, int VEC, int NL, int MAXJ, int V, Way WAY>
__global__ __launch_bounds__(kBlock) void k_render_camera(KBatch<MAXJ> B) {
    // one camera: tile rows dealt over the XCDs; batches: one contiguous range per XCD
    const int64_t b = MAXJ == 1 ? xcd_interleave(blockIdx.x, B.n_blocks, 4 * (int64_t)B.job[0].tiles_x)
                                : xcd_swizzle(blockIdx.x, B.n_blocks);
    if (b < 0) return;
    int j = 0;
    if constexpr (MAXJ > 1) {
        for (int q = 1; q < B.n_jobs; ++q)
            if (b >= B.job[q].block_begin) j = q;
    }
    const KJob& J = B.job[j];
    const int q = (int)(b - J.block_begin);
    const int tile = J.tile_begin + (q >> 2), quad = q & 3;
    const int tx = tile % J.tiles_x, ty = tile / J.tiles_x;
    const int lane = threadIdx.x;
    const int px = tx * 16 + (quad & 1) * 8 + (lane & 7);
    const int py = ty * 16 + (quad >> 1) * 8 + (lane >> 3);
    const bool valid = (px < J.cam.W) & (py < J.cam.H);
    double ro[3], rd[3];
    pixel_ray(J.cam, px, py, ro, rd);
    float C[3], Tr, dep;
    int ns, steps;
    extern __shared__ int po_stack[];
    render_one<T, K, VEC, NL, V, WAY>(J.tr, J.op, valid, ro, rd, po_stack + threadIdx.x, C, Tr, ns, steps, dep);
    if (!valid) return;
    const size_t p = (size_t)py * J.cam.W + px;
    J.rgb[3 * p + 0] = C[0];
    J.rgb[3 * p + 1] = C[1];
    J.rgb[3 * p + 2] = C[2];
    if constexpr (V == PO_FWD_VIEW) {
        if (J.aux) {
            J.aux[4 * p + 0] = Tr;
            J.aux[4 * p + 1] = (float)ns;
            J.aux[4 * p + 2] = (float)steps;
            J.aux[4 * p + 3] = dep;
        }
    }
}

// ---------------------------------------------------------------------------
// Split camera render.  The frame time of a one-pass render is set by its
// longest walks (a few hundred cells, against a median of a few), which run
// one cell at a time while most of the chip idles.  Compositing is
// associative (Sec. 3, eqn:quad: a range of segments acts on what lies behind
// it as (C, T) -> C_range + T_range C), so a long walk can be cut into
// pieces walked in parallel and joined front to back:
//   k_render_camera_split  walks every ray for at most split_cap samples;
//                          a ray with cells left is handed on: its state
//                          (s, T, C) and 1-16 chunks, equal parameter
//                          intervals of the rest of the ray;
//   k_render_chunks        walks one chunk per lane for at most chunk_cap
//                          samples; a chunk with cells left hands its
//                          remainder on as 1-16 sub-chunks (cells are
//                          bunched along a ray, so equal intervals are not
//                          equal work; the walked part of the chunk tells
//                          how dense the rest is);
//   k_render_subchunks     walks one sub-chunk per lane to its end;
//   k_render_join          combines each ray's pieces in order and writes
//                          the pixel.  Where early stopping ends the ray
//                          inside a piece (T below stop_T after a cell), the
//                          piece is walked again from its start with the
//                          known transmittance and stops where the one-pass
//                          walk stops.
// The result equals the one-pass render up to float rounding.  The queues
// are split into regions (one counter each) to spread the slot claims; a
// walk that finds its region full finishes in the lane that holds it.
// ---------------------------------------------------------------------------

// Queues are XCD-local: workgroup b runs on XCD b % 8 (the dispatcher deals
// workgroups round-robin over the XCDs), claims its pieces in one of that
// XCD's eight regions (8 x + (b / 8) mod 8), and the piece kernels take the
// slots of XCD x's regions with workgroups that run on XCD x (split_slot).
// A piece's head, its result and the join's reads of it then stay in the L2
// of the XCD that wrote them (each XCD has its own L2).  The first walk
// deals tile rows over the XCDs (xcd_interleave), so that every XCD gets a
// share of the frame's long walks and its regions fill evenly.  Depth-9
// 800x800 FP32: 0.586 against 0.631 ms with regions shared by all XCDs;
// with XCD-local regions but contiguous screen bands per XCD, 1.01 ms (the
// middle bands hold most long walks).
__device__ __forceinline__ int claim_region() { return (int)((blockIdx.x & 7) * 8 + ((blockIdx.x >> 3) & 7)); }
struct ContHead {
    double s;             // parameter where the first walk stopped (start of the next cell)
    float T, c0, c1, c2;  // transmittance and colour so far
    int32_t pix;          // pixel index py * W + px
    int32_t pad;
};
static_assert(sizeof(ContHead) == 32, "queue record layout");

struct SubHead {
    double lo, hi;        // remainder of a chunk: [lo, hi] (hi 1e300: to the box exit)
    int32_t pix;
    int32_t pad[3];
};
static_assert(sizeof(SubHead) == 32, "queue record layout");

// Result of a walked piece: colour and transmittance composited from T = 1,
// T after its last tested sample (-1: none), and for a chunk its remainder's
// sub-chunks (first slot, count; -1 none).
// dep: the viewer variant's depth integral of the piece (from T = 1); its
// samples and cells, and whether its last sample / cell was cut by the
// piece's end (the next piece counts that cell again), go to a side record
// {ns, steps, cut_smp, cut} that only the viewer variant touches.
struct PieceOut {
    float c0, c1, c2, T;
    float Tlast;
    int32_t sub, n_sub;
    float dep;
};
static_assert(sizeof(PieceOut) == 32, "queue record layout");

// Ray idx of a split render: pixel idx = py * W + px of the job's camera
// (SRC 0) or entry idx of the caller's ray arrays (SRC 1).
template <int SRC>
__device__ __forceinline__ void ray_of(const KJob& J, const KSplit& S, int idx, double (&ro)[3], double (&rd)[3]) {
    if constexpr (SRC == 0) {
        pixel_ray(J.cam, idx % J.cam.W, idx / J.cam.W, ro, rd);
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            ro[k] = (double)S.ray_o[3 * (size_t)idx + k];
            rd[k] = (double)S.ray_d[3 * (size_t)idx + k];
        }
    }
}

// End parameter of a split ray's walk: the slicing plane of the viewer
// variant, else 1e300 (the box exit).
template <int V, int SRC>
__device__ __forceinline__ double walk_end(const KJob& J, const KSplit& S, int idx) {
    if constexpr (V == PO_FWD_VIEW) {
        double ro[3], rd[3];
        ray_of<SRC>(J, S, idx, ro, rd);
        double lo, hi;
        clip_range(J.op, ro, rd, lo, hi);
        return hi;
    } else {
        return 1e300;
    }
}

// Piece k of n of the parameter range [a, hi] of ray idx: equal intervals of
// [a, min(hi, box exit)], the last one running to hi itself.  Sets up r for
// the walk of the piece; false when the piece is empty.
template <int SRC>
__device__ __forceinline__ bool piece_setup(const KJob& J, const KSplit& S, int idx, double a, double hi, int k,
                                            int n, Ray& r) {
    double ro[3], rd[3];
    ray_of<SRC>(J, S, idx, ro, rd);
    if (!ray_setup(J.tr, ro, rd, r, a, hi)) return false;
    const double len = r.s_exit - a;
    const double lo = k == 0 ? a : a + len * (double)k / (double)n;
    const double up = k + 1 < n ? a + len * (double)(k + 1) / (double)n : hi;
    return ray_setup(J.tr, ro, rd, r, lo, up);
}

// Bounds of piece k of n of [a, hi] (as piece_setup cuts it).
template <int SRC>
__device__ __forceinline__ void piece_bounds(const KJob& J, const KSplit& S, int idx, double a, double hi, int k,
                                             int n, double& lo, double& up) {
    double ro[3], rd[3];
    ray_of<SRC>(J, S, idx, ro, rd);
    Ray r;
    const double e = ray_setup(J.tr, ro, rd, r, a, hi) ? r.s_exit : a;
    lo = k == 0 ? a : a + (e - a) * (double)k / (double)n;
    up = k + 1 < n ? a + (e - a) * (double)(k + 1) / (double)n : hi;
}

// Start of this lane's walk and end of its ray, kept in LDS (not in registers)
// while the walk runs.
__device__ __forceinline__ double2* walk_range() {
    __shared__ double2 s_range[kBlock];
    return s_range + threadIdx.x;
}

// Pieces wanted for the rest of a walk from r.s on that took r.nt samples
// (exact renders: cells) over its walk_range: about `target` each, from the
// number per unit parameter so far, and at least ub_frac of the finest-cell
// faces ahead.
__device__ __forceinline__ int pieces_wanted(const Ray& r, const KSplit& S, int target) {
    const double2 range = *walk_range();
    const double rest = range.y - r.s;
    double est = (double)r.nt * rest / fmax(r.s - range.x, 1e-300);
    est = fmax(est, (double)S.ub_frac * rest * (fabs(r.dg[0]) + fabs(r.dg[1]) + fabs(r.dg[2])));
    return (int)fmin(fmax(ceil(est / (double)target), 1.0), (double)kSplitMaxChunks);
}

// Claims the wave's pieces in one atomic: sum(want) slots of a region, laid
// out level-major (piece 0 of every lane that wants pieces, in lane order,
// then piece 1, ...), so that a wave of consecutive slots walks neighbouring
// rays at similar depths.  Writes every claimed slot's info {first slot of
// its piece list, piece | count << 8, next slot or -1, 0} and returns this
// lane's first slot, or -1 (want == 0, or the region cannot hold the claim:
// its claimed slots are then marked unused).  Every lane of the wave must
// call it.
__device__ __forceinline__ int claim_pieces(int32_t* count, int4* __restrict__ info, int region, int want,
                                            int region_slots) {
    const int lane = (int)threadIdx.x;
    int tot = want;
#pragma unroll
    for (int o = kBlock / 2; o >= 1; o >>= 1) tot += __shfl_xor(tot, o);
    if (tot == 0) return -1;
    int base = 0;
    if (lane == 0) base = atomicAdd(count + region, tot);
    base = __shfl(base, 0);
    const int rbase = region * region_slots;
    if (base + tot > region_slots) {
        for (int i = base + lane; i < min(base + tot, region_slots); i += kBlock) info[rbase + i].x = -1;
        return -1;
    }
    const uint64_t below = (1ull << lane) - 1ull;
    uint64_t mk = __ballot(want > 0);
    int at = rbase + base, first = -1;
    for (int j = 0; j < kSplitMaxChunks && mk != 0ull; ++j) {
        const uint64_t mk1 = __ballot(want > j + 1);
        const int at1 = at + __popcll(mk);
        if (want > j) {
            const int slot = at + __popcll(mk & below);
            if (j == 0) first = slot;
            const int next = want > j + 1 ? at1 + __popcll(mk1 & below) : -1;
            info[slot] = make_int4(first, j | (want << 8), next, 0);
        }
        at = at1;
        mk = mk1;
    }
    return first;
}

// The first walk of a split render for ray idx (valid: idx names a ray):
// at most split_cap samples, then the ray is handed on or, if its region of
// the queue is full, walked to its end here.  Every lane of the wave must
// call it.
template <typename T, int K, int VEC, int NL, int V, int SRC, Way WAY>
__device__ __forceinline__ void first_walk(const KJob& J, const KSplit& S, int idx, bool valid) {
    const KTree& tr = J.tr;
    const KOpts& op = J.op;
    extern __shared__ int po_stack[];
    int* stk = po_stack + threadIdx.x;
    using Smp = FirstSampler<T, K, VEC, NL, V, WAY>;
    Smp smp;
    Ray r;
    int want = 0, steps = 0, h = -1;
    bool walk = false, handed = false;
    if (valid) {
        double ro[3], rd[3];
        ray_of<SRC>(J, S, idx, ro, rd);
        double s_lo = 0.0, s_hi = 1e300;
        if constexpr (V == PO_FWD_VIEW) clip_range(op, ro, rd, s_lo, s_hi);
        walk = ray_setup(tr, ro, rd, r, s_lo, s_hi);
        if (walk) *walk_range() = make_double2(r.s, r.s_exit);
    }
    fwd_init<K, V>(smp, tr, op, walk, r);
    // the second pass finishes the walks whose region is full
    for (int pass = 0; pass < 2; ++pass) {
        steps += march<true, WAY>(tr, r, walk, op.max_steps - steps, pass ? kNoCap : S.split_cap, S.exact, stk, smp);
        if (walk & r.more) {
            if (steps >= op.max_steps)
                atomicAdd(&g_po_errors, 1ull);  // the step cap proper
            else
                want = pieces_wanted(r, S, S.chunk_target);
        }
        if (pass) break;
        h = claim_pieces(S.count, S.info, claim_region(), want, S.region_slots);
        handed = (want > 0) & (h >= 0);
        walk = (want > 0) & (h < 0);
        if (__ballot(walk) == 0ull) break;
    }
    if (handed) {
        ContHead hd;
        hd.s = r.s;
        hd.T = smp.Tl;
        hd.c0 = smp.c0;
        hd.c1 = smp.c1;
        hd.c2 = smp.c2;
        hd.pix = idx;
        hd.pad = 0;
        reinterpret_cast<ContHead*>(S.head)[h] = hd;
    }
    const size_t p = (size_t)idx;
    if constexpr (SRC == 1) {
        // a kept render records which rays it handed on, for its backward
        if (valid && S.ray_slot) S.ray_slot[p] = handed ? h : -1;
    }
    if (valid && !handed) {
        J.rgb[3 * p + 0] = fmaf(smp.Tl, op.bg[0], smp.c0);
        J.rgb[3 * p + 1] = fmaf(smp.Tl, op.bg[1], smp.c1);
        J.rgb[3 * p + 2] = fmaf(smp.Tl, op.bg[2], smp.c2);
    }
    if constexpr (V == PO_FWD_VIEW) {
        // aux of a handed-on ray: the first walk's counts and depth, which
        // the join completes
        if (valid && J.aux) {
            J.aux[4 * p + 0] = smp.Tl;
            J.aux[4 * p + 1] = (float)smp.ns;
            J.aux[4 * p + 2] = (float)steps;
            J.aux[4 * p + 3] = smp.dep;
        }
    }
}

// The plain (SH, SG) walks of records up to 192 bytes are held to 128 VGPRs
// (4 waves per SIMD; float32 K = 16 in dword loads or with nodes, and float16
// K = 25, then keep up to 112 bytes of scratch, used before and after the walk's
// loop).  Larger records and the viewer and
// codebook variants would spill inside it (K=25 float32: 180 bytes of scratch,
// half the frame rate), so they keep their natural count.
template <typename T, int K, int V>
constexpr int kPieceWaves = (V == PO_FWD_SH || V == PO_FWD_SG) && sizeof(T) * 3 * K <= 192
                                ? 4
                                : 1;

template <typename T, int K, int VEC, int NL, int V, Way WAY>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kPieceWaves<T, K, V>, 8))) void k_render_camera_split(KBatch<1> B, KSplit S) {
    const int64_t b = xcd_interleave(blockIdx.x, B.n_blocks, 4 * B.job[0].tiles_x);
    if (b < 0) return;
    const KJob& J = B.job[0];
    const int q = (int)b;
    const int tile = J.tile_begin + (q >> 2), quad = q & 3;
    const int tx = tile % J.tiles_x, ty = tile / J.tiles_x;
    const int lane = threadIdx.x;
    const int px = tx * 16 + (quad & 1) * 8 + (lane & 7);
    const int py = ty * 16 + (quad >> 1) * 8 + (lane >> 3);
    const bool valid = (px < J.cam.W) & (py < J.cam.H);
    first_walk<T, K, VEC, NL, V, 0, WAY>(J, S, valid ? py * J.cam.W + px : 0, valid);
}

template <typename T, int K, int VEC, int NL, int V, Way WAY>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kPieceWaves<T, K, V>, 8))) void k_render_rays_split(KBatch<1> B, KSplit S) {
    const int64_t b = xcd_swizzle(blockIdx.x, B.n_blocks);
    if (b < 0) return;
    const int64_t i = b * kBlock + threadIdx.x;
    const bool valid = i < S.n_rays;
    first_walk<T, K, VEC, NL, V, 1, WAY>(B.job[0], S, valid ? (int)i : 0, valid);
}

__global__ void k_zero_i32(int32_t* __restrict__ p, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) p[i] = 0;
}

// Queue slot of this thread (workgroup blockIdx.x - first, first a multiple
// of 8), or -1 past the claimed slots.  Workgroup b serves the regions of
// its own XCD x = b % 8, and within them consecutive workgroups take
// consecutive 64-slot blocks of the claimed slots, region after region
// (faster than interleaving the regions: 735 against 1035 us per depth-9
// frame).  The grid covers the queue's capacity, which the claims fill only
// in part: with the blocks of each region counted from its claims, the
// workgroups past the claimed blocks of all eight regions are the last ones
// dispatched and find nothing, instead of each region's empty blocks
// standing in the dispatch order in front of the next region's work.
__device__ __forceinline__ int split_slot(const int32_t* count, int region_slots, int first = 0) {
    const int b = (int)blockIdx.x - first;
    const int x = b & 7;
    int t = b >> 3;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int n = min(count[8 * x + i], region_slots);
        const int nb = (n + kBlock - 1) / kBlock;
        if (t < nb) {
            const int local = t * kBlock + (int)threadIdx.x;
            return local < n ? (8 * x + i) * region_slots + local : -1;
        }
        t -= nb;
    }
    return -1;
}

template <typename T, int K, int VEC, int NL, int V, int SRC, Way WAY>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kPieceWaves<T, K, V>, 8))) void k_render_chunks(
    KBatch<1> B, KSplit S) {
    const int q = split_slot(S.count, S.region_slots);
    const int4 in = q < 0 ? make_int4(-1, 0, -1, 0) : S.info[q];
    const int h = in.x;
    const KJob& J = B.job[0];
    using Smp = ChunkSampler<T, K, VEC, NL, V, WAY>;
    Smp smp;
    Ray r;
    int want = 0, steps = 0, pix = 0, sub = -1;
    extern __shared__ int po_stack[];
    int* stk = po_stack + threadIdx.x;
    bool walk = false;
    if (h >= 0) {
        const int mj = in.y;
        const ContHead hd = reinterpret_cast<const ContHead*>(S.head)[h];
        pix = hd.pix;
        walk = piece_setup<SRC>(J, S, pix, hd.s, walk_end<V, SRC>(J, S, pix), mj & 255, mj >> 8, r);
        if (walk) *walk_range() = make_double2(r.s, r.s_exit);
    }
    if (__ballot(h >= 0) == 0ull) return;
    fwd_init<K, V>(smp, J.tr, J.op, walk, r);
    // the second pass finishes the walks whose region is full
    for (int pass = 0; pass < 2; ++pass) {
        steps += march<true, WAY>(J.tr, r, walk, J.op.max_steps - steps, pass ? kNoCap : S.chunk_cap, S.exact, stk, smp);
        if (walk & r.more) {
            if (steps >= J.op.max_steps)
                atomicAdd(&g_po_errors, 1ull);
            else
                want = pieces_wanted(r, S, S.sub_target);
        }
        if (pass) break;
        sub = claim_pieces(S.count2, S.info2, claim_region(), want, S.region_slots);
        walk = (want > 0) & (sub < 0);
        if (want > 0) {
            if (sub >= 0) {
                SubHead sh;
                sh.lo = r.s;
                sh.hi = r.s_end;
                sh.pix = pix;
                sh.pad[0] = sh.pad[1] = sh.pad[2] = 0;
                reinterpret_cast<SubHead*>(S.head2)[sub] = sh;
            } else {
                want = 0;
            }
        }
        if (__ballot(walk) == 0ull) break;
    }
    if (h >= 0) {
        PieceOut o;
        o.c0 = smp.c0;
        o.c1 = smp.c1;
        o.c2 = smp.c2;
        o.T = smp.Tl;
        o.Tlast = smp.Tlast;
        o.sub = sub;
        o.n_sub = want;
        o.dep = smp.dep;
        reinterpret_cast<PieceOut*>(S.part)[q] = o;
        if constexpr (V == PO_FWD_VIEW)
            S.view_part[q] = make_int4(smp.ns, steps - max(smp.skip0, 0), smp.smp_cut ? 1 : 0,
                                       (want == 0 && !smp.cpl) ? 1 : 0);
    }
}

template <typename T, int K, int VEC, int NL, int V, int SRC, Way WAY>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kPieceWaves<T, K, V>, 8))) void k_render_subchunks(
    KBatch<1> B, KSplit S) {
    const int q = split_slot(S.count2, S.region_slots);
    const int4 in = q < 0 ? make_int4(-1, 0, -1, 0) : S.info2[q];
    const int h = in.x;
    if (__ballot(h >= 0) == 0ull) return;
    const KJob& J = B.job[0];
    using Smp = ChunkSampler<T, K, VEC, NL, V, WAY>;
    Smp smp;
    Ray r;
    bool walk = false;
    if (h >= 0) {
        const int mj = in.y;
        const SubHead sh = reinterpret_cast<const SubHead*>(S.head2)[h];
        walk = piece_setup<SRC>(J, S, sh.pix, sh.lo, sh.hi, mj & 255, mj >> 8, r);
    }
    fwd_init<K, V>(smp, J.tr, J.op, walk, r);
    extern __shared__ int po_stack[];
    const int steps = march<false, WAY>(J.tr, r, walk, J.op.max_steps, kNoCap, S.exact, po_stack + threadIdx.x, smp);
    if (h < 0) return;
    PieceOut o;
    o.c0 = smp.c0;
    o.c1 = smp.c1;
    o.c2 = smp.c2;
    o.T = smp.Tl;
    o.Tlast = smp.Tlast;
    o.sub = -1;
    o.n_sub = 0;
    o.dep = smp.dep;
    reinterpret_cast<PieceOut*>(S.part2)[q] = o;
    if constexpr (V == PO_FWD_VIEW)
        S.view_part2[q] = make_int4(smp.ns, steps - max(smp.skip0, 0), smp.smp_cut ? 1 : 0, smp.cpl ? 0 : 1);
}

// Front-to-back join of the pieces of the ray whose first slot is q (ray: this
// lane has one; every lane of the wave calls it).  Running state: transmittance
// and colour in front, and for the viewer variant the depth integral, sample
// and cell counts, and whether the last piece joined ended in a cut cell
// (counted again by the next piece).
struct JoinAcc {
    float Tp;
    float c[3];
    float dep;
    int ns, steps, cut_smp, cut;
};

// Where early stopping ends a ray inside a piece (T below stop_T after a
// tested sample), the piece is walked again from the known transmittance; the
// rays of the wave that have reached such a piece are walked together.
// keep: over each piece's result the transmittance and colour prefix in front
// of it is written, and whether it lies before the early stop (Tlast 1) or not
// (-1): the prefixes a backward over these pieces differentiates from.
template <typename T, int K, int VEC, int NL, int V, int SRC, Way WAY>
__device__ __forceinline__ void join_ray(const KJob& J, const KSplit& S, int q, bool ray, int m, const ContHead& hd,
                                         bool keep, JoinAcc& A) {
    PieceOut* part = reinterpret_cast<PieceOut*>(S.part);
    PieceOut* part2 = reinterpret_cast<PieceOut*>(S.part2);
    const SubHead* head2 = reinterpret_cast<const SubHead*>(S.head2);
    using Smp = ChunkSampler<T, K, VEC, NL, V, WAY>;
    // next chunk j in slot qj; sub-chunk k of n_sub of the chunk before it, in slot qk
    int j = 0, qj = q, k = 0, n_sub = 0, sub = -1, qk = -1;
    bool more = ray, done = false;
    while (true) {
        bool again = false, is_sub = false;
        PieceOut o;
        while (more & !again) {
            PieceOut* rec;
            const int4* vp;
            is_sub = k < n_sub;
            if (is_sub) {
                rec = part2 + qk;
                vp = S.view_part2 + qk;
                qk = S.info2[qk].z;
                ++k;
            } else if (j < m) {
                rec = part + qj;
                vp = S.view_part + qj;
                qj = S.info[qj].z;
                ++j;
            } else {
                more = false;
                break;
            }
            o = *rec;
            if (!is_sub) {
                n_sub = o.n_sub;
                sub = qk = o.sub;
                k = 0;
            }
            if (keep) {
                PieceOut p = o;
                p.c0 = A.c[0];
                p.c1 = A.c[1];
                p.c2 = A.c[2];
                p.T = A.Tp;
                p.Tlast = done ? -1.0f : 1.0f;
                *rec = p;
            }
            if (done) continue;
            again = (o.Tlast >= 0.0f) & (A.Tp * o.Tlast < J.op.stop_T);
            if (again) break;
            A.c[0] = fmaf(A.Tp, o.c0, A.c[0]);
            A.c[1] = fmaf(A.Tp, o.c1, A.c[1]);
            A.c[2] = fmaf(A.Tp, o.c2, A.c[2]);
            if constexpr (V == PO_FWD_VIEW) {
                const int4 c = *vp;  // ns, steps, cut_smp, cut
                A.dep = fmaf(A.Tp, o.dep, A.dep);
                A.ns += c.x - c.z;
                A.steps += c.y - c.w;
                A.cut_smp = c.z;
                A.cut = c.w;
            }
            A.Tp = A.Tp * o.T;
        }
        if (__ballot(again) == 0ull) break;
        // the walk stops inside this piece: walk it again from Tp (a chunk
        // whose remainder was handed on ends where its remainder begins)
        Smp smp;
        Ray r;
        bool walk = false;
        if (again) {
            smp.Tl = A.Tp;
            double lo, up;
            if (is_sub) {
                const SubHead sh = head2[sub];
                piece_bounds<SRC>(J, S, hd.pix, sh.lo, sh.hi, k - 1, n_sub, lo, up);
            } else {
                piece_bounds<SRC>(J, S, hd.pix, hd.s, walk_end<V, SRC>(J, S, hd.pix), j - 1, m, lo, up);
                if (n_sub > 0) up = head2[sub].lo;
            }
            walk = piece_setup<SRC>(J, S, hd.pix, lo, up, 0, 1, r);
        }
        fwd_init<K, V>(smp, J.tr, J.op, walk, r);
        extern __shared__ int po_stack[];
        const int steps = march<false, WAY>(J.tr, r, walk, J.op.max_steps, kNoCap, S.exact, po_stack + threadIdx.x, smp);
        if (again) {
            A.c[0] += smp.c0;
            A.c[1] += smp.c1;
            A.c[2] += smp.c2;
            A.Tp = smp.Tl;
            if constexpr (V == PO_FWD_VIEW) {
                A.dep += smp.dep;
                A.cut_smp = smp.hit ? 0 : (smp.smp_cut ? 1 : 0);
                A.cut = (smp.hit || (!is_sub && n_sub > 0) || smp.cpl) ? 0 : 1;
                A.ns += smp.ns - A.cut_smp;
                A.steps += steps - max(smp.skip0, 0) - A.cut;
            }
            // (rounding can leave T just above stop_T; then the later pieces still count)
            done = smp.hit;
            if (done & !keep) more = false;
        }
    }
}

template <typename T, int K, int VEC, int NL, int V, int SRC, Way WAY>
__global__ __launch_bounds__(kBlock) void k_render_join(KBatch<1> B, KSplit S) {
    const int q = split_slot(S.count, S.region_slots);
    const int4 in = q < 0 ? make_int4(-1, 0, -1, 0) : S.info[q];
    const bool ray = (q >= 0) & (in.x == q);  // the first slot of a ray
    if (__ballot(ray) == 0ull) return;
    const KJob& J = B.job[0];
    ContHead hd;
    if (ray) hd = reinterpret_cast<const ContHead*>(S.head)[q];
    const size_t p = ray ? (size_t)hd.pix : 0;
    bool keep = false;  // a kept ray-list render
    if constexpr (SRC == 1 && V != PO_FWD_VIEW) keep = S.ray_slot != nullptr;
    JoinAcc A;
    A.Tp = hd.T;
    A.c[0] = hd.c0;
    A.c[1] = hd.c1;
    A.c[2] = hd.c2;
    A.dep = 0.0f;
    A.ns = A.steps = A.cut_smp = A.cut = 0;
    if constexpr (V == PO_FWD_VIEW) {
        if (ray && J.aux) {
            A.ns = (int)J.aux[4 * p + 1];
            A.steps = (int)J.aux[4 * p + 2];
            A.dep = J.aux[4 * p + 3];
        }
    }
    join_ray<T, K, VEC, NL, V, SRC, WAY>(J, S, q, ray, in.y >> 8, hd, keep, A);
    if (!ray) return;
    J.rgb[3 * p + 0] = fmaf(A.Tp, J.op.bg[0], A.c[0]);
    J.rgb[3 * p + 1] = fmaf(A.Tp, J.op.bg[1], A.c[1]);
    J.rgb[3 * p + 2] = fmaf(A.Tp, J.op.bg[2], A.c[2]);
    if constexpr (V == PO_FWD_VIEW) {
        if (J.aux) {
            // the last piece's cut cell (at the slicing plane) has no next piece
            J.aux[4 * p + 0] = A.Tp;
            J.aux[4 * p + 1] = (float)(A.ns + A.cut_smp);
            J.aux[4 * p + 2] = (float)(A.steps + A.cut);
            J.aux[4 * p + 3] = A.dep;
        }
    }
}

// Gradient of one ray's samples (App. B.3): the forward colour C is the
// first pass; this second pass keeps the prefix P_i of w_k c_k, so that
// dC/dsigma_i = delta_i (c_i T_{i+1} - (C - P_i)) (zero where the raw density
// is <= 0) and dC/dk = w_i c_i (1 - c_i) Y, contracted with dL/dC and added
// to the leaf gradients with float atomics, once for every 64 samples of the
// wave: the density gradients by the samples' lanes, the 3K coefficient
// gradients z_c Y_k by all lanes together, consecutive lanes taking consecutive
// coefficients, so that one atomic instruction covers whole records.  Atomics
// complete in order with the loads behind them, so adding each step's samples
// at once held up the next step by an L2 round trip.
template <int K, int VEC, int NL>
struct BwdSampler : Records<float, K, VEC, NL> {
    static constexpr bool kClip = false;
    static constexpr bool kView = false;
    static constexpr bool kQueued = true;
    static constexpr bool kQuads = false;
    static constexpr int NE = 3 * K;
    static constexpr uint32_t kNone = 0xffffffffu;  // Sample::info: no gradient
    int stride;
    float stopT;
    float g0, g1, g2, C0, C1, C2;
    float* gsig;
    float* gsh;
    float Tl = 1.0f, P0 = 0.0f, P1 = 0.0f, P2 = 0.0f;

    __device__ __forceinline__ void shade(uint32_t head, uint32_t n) {
        Sample* q = sample_queue() + (head + threadIdx.x) % kQueue;
        const bool on = threadIdx.x < n;
        float col[3];
        const float s = this->eval(on, q->leaf, q->info & 63u, col);
        shaded()[threadIdx.x] = make_float4(s > 0.0f ? __expf(-(s * q->delta)) : -1.0f, col[0], col[1], col[2]);
    }
    // Leaves {density gradient, z_0, z_1, z_2} in the place of the sample's
    // result (opacity -1: no density, zero weight, and dC/dsigma is masked).
    __device__ __forceinline__ bool composite(const Sample& q, uint32_t, uint32_t at) {
        const float4 v = shaded()[at];
        if (v.x < 0.0f) return false;
        const float ex = v.x, c0 = v.y, c1 = v.z, c2 = v.w;
        const float wgt = Tl * (1.0f - ex);
        const float Tn = Tl * ex;
        P0 = fmaf(wgt, c0, P0);
        P1 = fmaf(wgt, c1, P1);
        P2 = fmaf(wgt, c2, P2);
        float gs = g0 * (c0 * Tn - (C0 - P0));
        gs = fmaf(g1, c1 * Tn - (C1 - P1), gs);
        gs = fmaf(g2, c2 * Tn - (C2 - P2), gs);
        shaded()[at] = make_float4(gs * q.delta, g0 * wgt * c0 * (1.0f - c0), g1 * wgt * c1 * (1.0f - c1),
                                   g2 * wgt * c2 * (1.0f - c2));
        staged()[at] = q.info & 63u;
        Tl = Tn;
        return Tl < stopT;
    }
    // The ray's lane of every shaded sample with a gradient, else kNone.
    static __device__ __forceinline__ uint32_t* staged() {
        __shared__ uint32_t s_staged[kBlock];
        return s_staged;
    }
    __device__ __forceinline__ void finish(uint32_t head, uint32_t n) {
        const uint32_t lane = threadIdx.x;
        const uint32_t src = lane < n ? staged()[lane] : kNone;
        const uint32_t leaf = sample_queue()[(head + lane) % kQueue].leaf;
        const uint64_t m = __ballot(src != kNone);
        // compacted: {leaf, lane of the ray, number of the sample} of the samples with a gradient
        __shared__ uint32_t s_leaf[kBlock], s_at[kBlock];
        if (src != kNone) {
            atomicAdd(gsig + leaf, shaded()[lane].x);
            const int i = rank_in(m);
            s_leaf[i] = leaf;
            s_at[i] = src | lane << 8;
        }
        __builtin_amdgcn_wave_barrier();
        const float* Z = reinterpret_cast<const float*>(shaded());
        const float* Y = reinterpret_cast<const float*>(basis_values<K>());
        const uint32_t total = (uint32_t)__popcll(m) * NE;
        for (uint32_t it = lane; it < total; it += kBlock) {
            const uint32_t i = it / NE, e = it - i * NE, c = e / K, k = e - c * K;
            const uint32_t a = s_at[i];
            atomicAdd(gsh + (size_t)s_leaf[i] * stride + e, Z[4 * (a >> 8) + 1 + c] * Y[4 * ((k >> 2) * kBlock + (a & 255u)) + (k & 3)]);
        }
        __builtin_amdgcn_wave_barrier();
        staged()[lane] = kNone;
    }
};

// Binds a backward sampler to a tree (every lane), and to ray i: its incoming
// gradient and colour, and the basis of its direction.  Returns whether the
// ray has a gradient.
template <int K, class Smp>
__device__ __forceinline__ bool bwd_init(Smp& smp, const KTree& tr, const KOpts& op, bool ray, const Ray& r, size_t i,
                                         const float* __restrict__ rgb_fwd, const float* __restrict__ grad,
                                         float* gsig, float* gsh) {
    smp.bind(tr);
    smp.stride = tr.stride;
    smp.stopT = op.stop_T;
    smp.gsig = gsig;
    smp.gsh = gsh;
    Smp::staged()[threadIdx.x] = Smp::kNone;
    if (!ray) return false;
    smp.g0 = grad[3 * i];
    smp.g1 = grad[3 * i + 1];
    smp.g2 = grad[3 * i + 2];
    if (smp.g0 == 0.0f && smp.g1 == 0.0f && smp.g2 == 0.0f) return false;
    smp.C0 = rgb_fwd[3 * i];
    smp.C1 = rgb_fwd[3 * i + 1];
    smp.C2 = rgb_fwd[3 * i + 2];
    init_basis<K, PO_FWD_VIEW>(tr, op, r);
    return true;
}

// Backward kernel: replays the forward walk of each ray.
template <int K, int VEC, int NL, Way WAY>
__global__ __launch_bounds__(kBlock) void k_backward(KTree tr, int64_t n, int64_t n_blocks,
                                                     const float* __restrict__ o,
                                                     const float* __restrict__ d, KOpts op,
                                                     const float* __restrict__ rgb_fwd,
                                                     const float* __restrict__ grad,
                                                     float* __restrict__ gsig, float* __restrict__ gsh) {
    const int64_t blk = xcd_swizzle(blockIdx.x, n_blocks);
    if (blk < 0) return;
    const int64_t i = blk * kBlock + threadIdx.x;
    Ray r;
    bool ray = i < n;
    if (ray) {
        const double ro[3] = {(double)o[3 * i], (double)o[3 * i + 1], (double)o[3 * i + 2]};
        const double rd[3] = {(double)d[3 * i], (double)d[3 * i + 1], (double)d[3 * i + 2]};
        ray = ray_setup(tr, ro, rd, r);
    }
    BwdSampler<K, VEC, NL> smp;
    ray = bwd_init<K>(smp, tr, op, ray, r, (size_t)i, rgb_fwd, grad, gsig, gsh);
    extern __shared__ int po_stack[];
    march<false, WAY>(tr, r, ray, op.max_steps, kNoCap, exact_cells(op), po_stack + threadIdx.x, smp);
}

// ---------------------------------------------------------------------------
// Split backward.  The gradient of a ray's pieces needs, at the start of each
// piece, the transmittance T and the colour prefix P = sum of w_k c_k of
// everything in front of it (App. B.3: dC/dsigma_i = delta_i (c_i T_{i+1} -
// (C - P_i)), dC/dk = w_i c_i (1 - c_i) Y).  A piece that cuts a cell is a
// segment of its own: the two parts' gradients add up to the whole cell's.
//   k_backward_split      the backward of the first split_cap samples of
//                         every ray, which then hands the rest on as chunks
//                         (head state: s, T, P);
//   k_render_chunks,
//   k_render_subchunks    the forward of the pieces (colour and transmittance
//                         from T = 1), as in the split render;
//   k_piece_prefix        per ray, front to back: T and P at the start of
//                         every piece and which pieces lie before the early
//                         stop (the piece holding it walked again, as in the
//                         join), written over the piece's forward result;
//   k_backward_pieces     the backward of every piece before the stop, from
//                         its T and P (chunks, then sub-chunks).
// ---------------------------------------------------------------------------
template <int K, int VEC, int NL, Way WAY>
__global__ __launch_bounds__(kBlock) void k_backward_split(KBatch<1> B, KSplit S, const float* __restrict__ rgb_fwd,
                                                           const float* __restrict__ grad, float* __restrict__ gsig,
                                                           float* __restrict__ gsh) {
    const int64_t b = xcd_swizzle(blockIdx.x, B.n_blocks);
    if (b < 0) return;
    const int64_t i = b * kBlock + threadIdx.x;
    const KJob& J = B.job[0];
    const KTree& tr = J.tr;
    using Smp = BwdSampler<K, VEC, NL>;
    Smp smp;
    extern __shared__ int po_stack[];
    int* stk = po_stack + threadIdx.x;
    Ray r;
    int want = 0, steps = 0;
    bool live = i < S.n_rays;
    if (live) {
        double ro[3], rd[3];
        ray_of<1>(J, S, (int)i, ro, rd);
        live = ray_setup(tr, ro, rd, r);
    }
    live = bwd_init<K>(smp, tr, J.op, live, r, (size_t)i, rgb_fwd, grad, gsig, gsh);
    if (live) *walk_range() = make_double2(r.s, r.s_exit);
    // the second pass finishes the walks whose region is full
    for (int pass = 0; pass < 2; ++pass) {
        steps += march<true, WAY>(tr, r, live, J.op.max_steps - steps, pass ? kNoCap : S.split_cap, S.exact, stk, smp);
        if (live & r.more) {
            if (steps >= J.op.max_steps)
                atomicAdd(&g_po_errors, 1ull);
            else
                want = pieces_wanted(r, S, S.chunk_target);
        }
        if (pass) break;
        const int h = claim_pieces(S.count, S.info, claim_region(), want, S.region_slots);
        if ((want > 0) & (h >= 0)) {
            ContHead hd;
            hd.s = r.s;
            hd.T = smp.Tl;
            hd.c0 = smp.P0;
            hd.c1 = smp.P1;
            hd.c2 = smp.P2;
            hd.pix = (int)i;
            hd.pad = 0;
            reinterpret_cast<ContHead*>(S.head)[h] = hd;
        }
        live = (want > 0) & (h < 0);
        if (__ballot(live) == 0ull) break;
    }
}

// The backward's first walk over the rays of a kept render
// (po_render_rays_keep): the render's pieces, their heads (s, T and the
// colour prefix P after its first walk) and ray_slot stay in the queue, so
// a ray the render handed on is differentiated over the same first
// split_cap samples and its pieces are not walked forward again; a ray it
// did not hand on (ended within the first walk, or its region was full) is
// differentiated to its end here.
template <int K, int VEC, int NL, Way WAY>
__global__ __launch_bounds__(kBlock) void k_backward_first_kept(KBatch<1> B, KSplit S,
                                                                const float* __restrict__ rgb_fwd,
                                                                const float* __restrict__ grad,
                                                                float* __restrict__ gsig, float* __restrict__ gsh) {
    const int64_t b = xcd_swizzle(blockIdx.x, B.n_blocks);
    if (b < 0) return;
    const int64_t i = b * kBlock + threadIdx.x;
    const KJob& J = B.job[0];
    const KTree& tr = J.tr;
    using Smp = BwdSampler<K, VEC, NL>;
    Smp smp;
    extern __shared__ int po_stack[];
    Ray r;
    bool live = i < S.n_rays, handed = false;
    if (live) {
        double ro[3], rd[3];
        ray_of<1>(J, S, (int)i, ro, rd);
        handed = S.ray_slot[i] >= 0;
        live = ray_setup(tr, ro, rd, r);
    }
    live = bwd_init<K>(smp, tr, J.op, live, r, (size_t)i, rgb_fwd, grad, gsig, gsh);
    const int steps = march<true, WAY>(tr, r, live, J.op.max_steps, handed ? S.split_cap : kNoCap, S.exact,
                                       po_stack + threadIdx.x, smp);
    if (live & r.more & (steps >= J.op.max_steps)) atomicAdd(&g_po_errors, 1ull);  // the step cap proper
}

// The prefixes of a ray's pieces, as the join of a kept render writes them.
template <int K, int VEC, int NL, int V, Way WAY>
__global__ __launch_bounds__(kBlock) void k_piece_prefix(KBatch<1> B, KSplit S) {
    const int q = split_slot(S.count, S.region_slots);
    const int4 in = q < 0 ? make_int4(-1, 0, -1, 0) : S.info[q];
    const bool ray = (q >= 0) & (in.x == q);
    if (__ballot(ray) == 0ull) return;
    ContHead hd;
    if (ray) hd = reinterpret_cast<const ContHead*>(S.head)[q];
    JoinAcc A;
    A.Tp = hd.T;
    A.c[0] = hd.c0;
    A.c[1] = hd.c1;
    A.c[2] = hd.c2;
    A.dep = 0.0f;
    A.ns = A.steps = A.cut_smp = A.cut = 0;
    join_ray<float, K, VEC, NL, V, 1, WAY>(B.job[0], S, q, ray, in.y >> 8, hd, true, A);
}

// The first kSplitRegions * region_slots / kBlock workgroups take the walked parts of the
// chunks, the others the sub-chunks: the two sets are independent once their
// prefixes are known, so one launch overlaps their tails.
template <int K, int VEC, int NL, Way WAY>
__global__ __launch_bounds__(kBlock) void k_backward_pieces(KBatch<1> B, KSplit S, const float* __restrict__ rgb_fwd,
                                                            const float* __restrict__ grad, float* __restrict__ gsig,
                                                            float* __restrict__ gsh) {
    const int half = kSplitRegions * (S.region_slots / kBlock);
    const bool sub = blockIdx.x >= (unsigned)half;
    const int q = split_slot(sub ? S.count2 : S.count, S.region_slots, sub ? half : 0);
    const int4 in = q < 0 ? make_int4(-1, 0, -1, 0) : (sub ? S.info2 : S.info)[q];
    PieceOut o;
    bool live = in.x >= 0;
    if (live) {
        o = reinterpret_cast<const PieceOut*>(sub ? S.part2 : S.part)[q];
        live = !(o.Tlast < 0.0f);  // not behind the early stop
    }
    if (__ballot(live) == 0ull) return;
    const KJob& J = B.job[0];
    int idx = 0;
    Ray r;
    if (live) {
        const int k = in.y & 255, n = in.y >> 8;
        if (sub) {
            const SubHead sh = reinterpret_cast<const SubHead*>(S.head2)[in.x];
            idx = sh.pix;
            live = piece_setup<1>(J, S, idx, sh.lo, sh.hi, k, n, r);
        } else {
            const ContHead hd = reinterpret_cast<const ContHead*>(S.head)[in.x];
            idx = hd.pix;
            double lo, up;
            piece_bounds<1>(J, S, idx, hd.s, 1e300, k, n, lo, up);
            if (o.n_sub > 0) up = reinterpret_cast<const SubHead*>(S.head2)[o.sub].lo;
            live = piece_setup<1>(J, S, idx, lo, up, 0, 1, r);
        }
    }
    using Smp = ChunkOf<BwdSampler<K, VEC, NL>>;
    Smp smp;
    live = bwd_init<K>(smp, J.tr, J.op, live, r, (size_t)idx, rgb_fwd, grad, gsig, gsh);
    smp.Tl = o.T;
    smp.P0 = o.c0;
    smp.P1 = o.c1;
    smp.P2 = o.c2;
    extern __shared__ int po_stack[];
    march<false, WAY>(J.tr, r, live, J.op.max_steps, kNoCap, S.exact, po_stack + threadIdx.x, smp);
}

// Visibility filter of the conversion (Sec. 4.2, "Filtering"): alpha
// renders of a camera that raise every leaf's weight to the largest weight
// of a segment in it, MODE 0 the segment's alpha 1 - exp(-sigma delta),
// MODE 1 its contribution T alpha.  Only the densities are gathered.  The
// weights are non-negative floats, whose bit patterns order like unsigned
// integers, so the maximum is an integer atomic.
template <typename T, int MODE>
struct WeightSampler {
    static constexpr bool kClip = false;
    static constexpr bool kView = false;
    static constexpr bool kQueued = false;
    static constexpr bool kQuads = false;
    __amdgpu_buffer_rsrc_t sig;
    uint32_t sig_end;
    float stopT;
    unsigned* wt;
    float Tl = 1.0f;
    // in flight
    int leaf;
    uint32_t raw;
    float delta;

    __device__ __forceinline__ void issue(int l, float d, float, bool) {
        leaf = l;
        raw = sigma_buf(sig, l < 0 ? sig_end : (uint32_t)l * (uint32_t)sizeof(T), (T*)nullptr);
        delta = d;
    }
    __device__ __forceinline__ bool consume() {
        const float s = fmaxf(sigma_of<T>(raw), 0.0f);
        if (!(s > 0.0f)) return false;
        const float ex = __expf(-(s * delta));
        const float al = 1.0f - ex;
        const float w = MODE ? Tl * al : al;
        if (w > 0.0f) atomicMax(wt + leaf, __float_as_uint(w));
        Tl = Tl * ex;
        return Tl < stopT;
    }
};

// One camera, 16x16 tiles of four 8x8 single-wave workgroups as in
// k_render_camera; alpha (or nullptr) receives 1 - T per pixel.
template <typename T, int MODE, Way WAY>
__global__ __launch_bounds__(kBlock) void k_leaf_weights(KTree tr, KCam cam, KOpts op, int n_blocks,
                                                         unsigned* __restrict__ wt, float* __restrict__ alpha) {
    const int tiles_x = (cam.W + 15) / 16;
    const int64_t b = xcd_interleave(blockIdx.x, n_blocks, 4 * (int64_t)tiles_x);
    if (b < 0) return;
    const int tile = (int)(b >> 2), quad = (int)(b & 3);
    const int lane = threadIdx.x;
    const int px = (tile % tiles_x) * 16 + (quad & 1) * 8 + (lane & 7);
    const int py = (tile / tiles_x) * 16 + (quad >> 1) * 8 + (lane >> 3);
    const bool valid = (px < cam.W) & (py < cam.H);
    double ro[3], rd[3];
    pixel_ray(cam, px, py, ro, rd);
    Ray r;
    const bool walk = valid && ray_setup(tr, ro, rd, r);
    WeightSampler<T, MODE> smp;
    smp.sig_end = held(tr.sigma_bytes);
    smp.sig = raw_rsrc(held(tr.sigma), smp.sig_end);
    smp.stopT = op.stop_T;
    smp.wt = wt;
    extern __shared__ int po_stack[];
    march<false, WAY>(tr, r, walk, op.max_steps, kNoCap, exact_cells(op), po_stack + threadIdx.x, smp);
    if (valid && alpha) alpha[(size_t)py * cam.W + px] = 1.0f - smp.Tl;
}

// One ray of k_traversal_stats: adds its samples, cells and loads.
template <typename T, Way WAY>
__device__ __forceinline__ void stats_walk(const KTree& tr, const Index& ix, const KOpts& op, Ray& r, int* stk,
                                           unsigned long long (&v)[4]) {
    const __amdgpu_buffer_rsrc_t sig = raw_rsrc(tr.sigma, tr.sigma_bytes);
    Walker<false, false, WAY> w;
    w.start(ix, r, stk);
    const int D = tr.depth(), M = tr.brick_level();
    // la: level the descent to the cell starts from; was_in: the cell
    // before lay in a brick
    int steps = 0, ns = 0, loads = 0, la = 0;
    bool was_in = false, pending = false, bad = false;
    uint32_t raw = 0;
    float Tl = 1.0f, delta = 0.0f;
    while (true) {
        ++steps;
        const int from[3] = {r.c[0], r.c[1], r.c[2]};
        const Cell c = w.step(ix, r, true, steps >= op.max_steps, false, stk);
        const int lvl = D - c.u;
        loads += (was_in & (la >= M)) ? 1 : (lvl <= M ? lvl - la : M - la + 1);
        was_in = lvl > M;
        la = D - 32 + __clz((from[0] ^ r.c[0]) | (from[1] ^ r.c[1]) | (from[2] ^ r.c[2]));
        bad |= r.more;
        // the previous sample is composited one cell later, as the
        // render counts it
        bool stop = false;
        if (pending) {
            ++ns;
            const float s = fmaxf(sigma_of<T>(raw), 0.0f);
            if (s > 0.0f) {
                Tl = Tl * __expf(-(s * delta));
                stop = Tl < op.stop_T;
            }
        }
        pending = !stop & (c.leaf >= 0) & (c.delta > 0.0f);
        if (pending) {
            raw = sigma_buf(sig, (uint32_t)c.leaf * (uint32_t)sizeof(T), (T*)nullptr);
            delta = c.delta;
        }
        if (c.last | stop) break;
    }
    if (pending) ++ns;
    if (bad | (w.bad != 0)) atomicAdd(&g_po_errors, 1ull);
    v[2] = (unsigned long long)steps;
    v[1] = (unsigned long long)ns;
    v[3] = (unsigned long long)loads;
}

// Traversal statistics of a camera render: the walk of the octree's own cells
// that gathers only the densities (the early stop depends on nothing else;
// its transmittance arithmetic is the render's, so it stops at the same
// sample) and counts, per ray, the data samples (segments of positive length
// in data leaves, as the aux output counts them), the cells visited and the
// child entries that a descent from the deepest ancestor shared with the cell
// before reads.  Sums over the image go to sums[4] =
// {rays, samples, cells, child-entry loads}, one atomic per wave and counter.
// SRC 0: the pixel rays of cam (16x16 tiles of four 8x8 waves); SRC 1: the
// n rays (o, d), 64 per wave.
template <typename T, int SRC>
__global__ __launch_bounds__(kBlock) void k_traversal_stats(KTree tr, KCam cam, const float* __restrict__ o,
                                                            const float* __restrict__ d, int64_t n, KOpts op,
                                                            int n_blocks, unsigned long long* __restrict__ sums) {
    const int64_t b = xcd_swizzle(blockIdx.x, n_blocks);
    if (b < 0) return;
    const int lane = threadIdx.x;
    bool valid;
    double ro[3], rd[3];
    if constexpr (SRC == 0) {
        const int tiles_x = (cam.W + 15) / 16;
        const int tile = (int)(b >> 2), quad = (int)(b & 3);
        const int px = (tile % tiles_x) * 16 + (quad & 1) * 8 + (lane & 7);
        const int py = (tile / tiles_x) * 16 + (quad >> 1) * 8 + (lane >> 3);
        valid = (px < cam.W) & (py < cam.H);
        if (valid) pixel_ray(cam, px, py, ro, rd);
    } else {
        const int64_t i = b * kBlock + lane;
        valid = i < n;
        if (valid) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                ro[k] = (double)o[3 * i + k];
                rd[k] = (double)d[3 * i + k];
            }
        }
    }
    unsigned long long v[4] = {valid ? 1ull : 0ull, 0ull, 0ull, 0ull};
    if (valid) {
        Ray r;
        if (ray_setup(tr, ro, rd, r)) {
            extern __shared__ int po_stack[];
            int* stk = po_stack + threadIdx.x;
            const Index ix(tr);
            switch (way_of(ix.D, ix.M, ix.G)) {
            case kDirect: stats_walk<T, kDirect>(tr, ix, op, r, stk, v); break;
            case kPlain: stats_walk<T, kPlain>(tr, ix, op, r, stk, v); break;
            default: stats_walk<T, kNodes>(tr, ix, op, r, stk, v);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        unsigned long long x = v[k];
        for (int o = kBlock / 2; o >= 1; o >>= 1) x += __shfl_xor(x, o);
        if (lane == 0 && x != 0ull) atomicAdd(sums + k, x);
    }
}

// Loss gradient of the NeRF loss (Sec. 3, eqn:nerfloss) for one batch: one
// thread per ray; squared errors are summed within the wave and added once
// per wave.
// Grid-stride over the rays; the squared errors are summed per workgroup
// (waves, then LDS) and added with one float atomic per workgroup: one
// atomic per wave on the single sum address serialised in L2 (15 us for
// 65536 rays).
__global__ __launch_bounds__(256) void k_mse_grad(int64_t n, const float* __restrict__ rgb,
                                                  const float* __restrict__ target, float scale,
                                                  float* __restrict__ grad, float* __restrict__ sq_sum) {
    float e2 = 0.0f;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float e = rgb[3 * i + c] - target[3 * i + c];
            grad[3 * i + c] = scale * (2.0f * e);
            e2 = fmaf(e, e, e2);
        }
    }
    for (int off = 32; off > 0; off >>= 1) e2 += __shfl_xor(e2, off, 64);
    __shared__ float part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = e2;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float t = (part[0] + part[1]) + (part[2] + part[3]);
        if (t != 0.0f) atomicAdd(sq_sum, t);
    }
}

// Batch rows of a training step: three rows of 3 floats per ray.
__global__ __launch_bounds__(256) void k_gather_rays(int64_t n, const int64_t* __restrict__ idx, int64_t n_src,
                                                     const float* __restrict__ o, const float* __restrict__ d,
                                                     const float* __restrict__ t, float* __restrict__ bo,
                                                     float* __restrict__ bd, float* __restrict__ bt) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t j = idx[i];
    const bool ok = (j >= 0) & (j < n_src);
    if (!ok) atomicAdd(&g_po_errors, 1ull);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        bo[3 * i + c] = ok ? o[3 * j + c] : 0.0f;
        bd[3 * i + c] = ok ? d[3 * j + c] : 0.0f;
        bt[3 * i + c] = ok ? t[3 * j + c] : 0.0f;
    }
}

// A training batch drawn on the device: element `first + i` of the SplitMix64
// sequence of `seed` (Steele, Lea and Flood, "Fast splittable pseudorandom
// number generators", OOPSLA 2014: the state advances by the golden-ratio
// increment and each output is the state passed through the variant-13
// finaliser) picks row floor(z * n_src / 2^64), and the three rows are
// gathered.  Thread 0 also clears the loss accumulator of the batch.
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t k) {
    uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__global__ __launch_bounds__(256) void k_draw_batch(int64_t n, uint64_t seed, uint64_t first, int64_t n_src,
                                                    const float* __restrict__ o, const float* __restrict__ d,
                                                    const float* __restrict__ t, float* __restrict__ bo,
                                                    float* __restrict__ bd, float* __restrict__ bt,
                                                    float* __restrict__ sq_sum) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    if (i == 0 && sq_sum) sq_sum[0] = 0.0f;
    const int64_t j = (int64_t)__umul64hi(splitmix64(seed, first + (uint64_t)i), (uint64_t)n_src);
    for (int c = 0; c < 3; ++c) {
        bo[3 * i + c] = o[3 * j + c];
        bd[3 * i + c] = d[3 * j + c];
        bt[3 * i + c] = t[3 * j + c];
    }
}

#if PO_PART == 0
// ---------------------------------------------------------------------------
// The device half of po_tree_build_index.  The host lays out nodes and bricks
// (index_of); these kernels add what the walk crosses empty space with: the
// grid, and the empty box of every empty entry.
// ---------------------------------------------------------------------------

// Grows an empty box [lo, hi] (inclusive) by one layer at a time, the six
// sides in turn, until every side meets an occupied cell (empty(lo, hi) false
// for the layer), the limit [0, n) or `most` layers.  Growing the sides in
// turn keeps the box near a cube, which no direction of travel is hurt by.
template <class Empty>
__device__ __forceinline__ void grow_box(int (&lo)[3], int (&hi)[3], int n, int most, Empty empty) {
    unsigned live = 63u;
    for (int it = 0; it < most && live; ++it) {
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            if (!((live >> f) & 1u)) continue;
            const int a = f >> 1;
            int l[3] = {lo[0], lo[1], lo[2]}, h[3] = {hi[0], hi[1], hi[2]};
            const int at = (f & 1) ? hi[a] + 1 : lo[a] - 1;
            l[a] = h[a] = at;
            if (at < 0 || at >= n || !empty(l, h)) {
                live &= ~(1u << f);
                continue;
            }
            if (f & 1)
                hi[a] = at;
            else
                lo[a] = at;
        }
    }
}

// One wave per brick: the boxes of its empty cells, inside the brick, and its
// entries from the order of the host's child slots to x, y, z.  The
// brick's occupancy is held as eight 64-bit masks (one per x, bit 8 y + z), so
// a layer is tested in one to eight ANDs.
__global__ __launch_bounds__(kBlock) void k_index_bricks(int32_t* __restrict__ bricks) {
    __shared__ unsigned occ[16];
    int32_t* B = bricks + (size_t)blockIdx.x * 512;
    const int lane = (int)threadIdx.x;
    if (lane < 16) occ[lane] = 0u;
    __syncthreads();
    int32_t v[8];
    int cx[8][3];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int q = i * 64 + lane;  // slot1 << 6 | slot2 << 3 | slot3
        v[i] = B[q];
        cx[i][0] = ((q >> 8 & 1) << 2) | ((q >> 5 & 1) << 1) | (q >> 2 & 1);
        cx[i][1] = ((q >> 7 & 1) << 2) | ((q >> 4 & 1) << 1) | (q >> 1 & 1);
        cx[i][2] = ((q >> 6 & 1) << 2) | ((q >> 3 & 1) << 1) | (q & 1);
        const int bit = cx[i][1] * 8 + cx[i][2];
        if ((v[i] >> 2) != 0) atomicOr(&occ[cx[i][0] * 2 + (bit >> 5)], 1u << (bit & 31));
    }
    __syncthreads();
    auto empty = [&](const int (&l)[3], const int (&h)[3]) {
        const uint64_t z = ((2ull << h[2]) - 1ull) & ~((1ull << l[2]) - 1ull);  // bits l..h of a byte
        const uint64_t y = (h[1] == 7 ? ~0ull : (1ull << (8 * (h[1] + 1))) - 1ull) & ~((1ull << (8 * l[1])) - 1ull);
        const uint64_t m = (z * 0x0101010101010101ull) & y;
        uint64_t any = 0ull;
        for (int x = l[0]; x <= h[0]; ++x) any |= ((uint64_t)occ[2 * x + 1] << 32 | occ[2 * x]) & m;
        return any == 0ull;
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        int32_t* out = B + (cx[i][0] << 6 | cx[i][1] << 3 | cx[i][2]);
        if ((v[i] >> 2) != 0) {
            *out = v[i];
            continue;
        }
        const int up = v[i] & 3, w = (1 << up) - 1;
        int lo[3], hi[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            lo[k] = cx[i][k] & ~w;
            hi[k] = cx[i][k] | w;
        }
        grow_box(lo, hi, 8, 8, empty);
        *out = po_index_box_entry(cx[i], lo, hi, up, 0);
    }
}

// One thread per grid cell: descends the host's nodes to the cell's leaf,
// empty cube, brick or level-G node.  A leaf entry of the nodes there is
// -(number in the coarse table) - 1.  Empty cells get their octree cube only.
__global__ __launch_bounds__(256) void k_index_grid(const int32_t* __restrict__ nodes, int n_top, int G, int unit,
                                                    int32_t* __restrict__ grid) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= (1u << (3 * G))) return;
    const int c[3] = {(int)(i >> (2 * G)), (int)(i >> G) & ((1 << G) - 1), (int)i & ((1 << G) - 1)};
    int32_t e = 0;
    int L = 0;  // e: node of level L holding the cell
    do {
        e = nodes[(size_t)e * 8 + child_slot(c, G, L)];
        ++L;
    } while (L < G && e > 0 && e < n_top);
    if (e < 0)
        e = kIdxCoarse | (-e - 1);
    else if (e == 0)
        e = po_index_box_entry(c, c, c, G - L, unit);
    else if (e >= n_top)
        e -= n_top;  // a brick: G == M
    grid[i] = e;
}

// Summed-area table of the grid's occupancy, one axis per launch (axis 2
// reads the grid): one thread per line of n = 2^G cells.
__global__ __launch_bounds__(256) void k_index_sums(const int32_t* __restrict__ grid, int32_t* __restrict__ sat, int G,
                                                    int axis) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    const uint32_t n = 1u << G;
    if (i >= n * n) return;
    const uint32_t a = i >> G, b = i & (n - 1);
    const uint32_t base = axis == 2 ? (a << G | b) << G : axis == 1 ? (a << (2 * G) | b) : i;
    const uint32_t step = axis == 2 ? 1u : axis == 1 ? n : n * n;
    int32_t sum = 0;
    for (uint32_t q = 0; q < n; ++q) {
        const uint32_t at = base + q * step;
        sum += axis == 2 ? (grid[at] < 0 ? 0 : 1) : sat[at];
        sat[at] = sum;
    }
}

// One thread per grid cell: the empty box of an empty cell, in grid cells.
__global__ __launch_bounds__(256) void k_index_grid_boxes(const int32_t* __restrict__ sat, int G, int unit,
                                                          int32_t* __restrict__ grid) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= (1u << (3 * G))) return;
    const int32_t e = grid[i];
    if (e >= 0) return;
    const int n = 1 << G;
    const int c[3] = {(int)(i >> (2 * G)), (int)(i >> G) & (n - 1), (int)i & (n - 1)};
    // (as k_index_grid wrote it: a box of one cell, in cells of the grid)
    const int up = po_index_cube(e) - unit, w = (1 << up) - 1;
    auto S = [&](int x, int y, int z) {  // cells occupied in [0, x] x [0, y] x [0, z]
        return (x < 0 || y < 0 || z < 0) ? 0 : sat[((((uint32_t)x << G) | (uint32_t)y) << G) | (uint32_t)z];
    };
    auto empty = [&](const int (&l)[3], const int (&h)[3]) {
        const int a = l[0] - 1, b = l[1] - 1, d = l[2] - 1;
        return S(h[0], h[1], h[2]) - S(a, h[1], h[2]) - S(h[0], b, h[2]) - S(h[0], h[1], d) + S(a, b, h[2]) +
                   S(a, h[1], d) + S(h[0], b, d) - S(a, b, d) ==
               0;
    };
    int lo[3], hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lo[k] = c[k] & ~w;
        hi[k] = c[k] | w;
    }
    grow_box(lo, hi, n, kIdxReach, empty);
    grid[i] = po_index_cube_entry(c, lo, hi, up, unit);
}
#endif

// Plain SGD on the leaf values (Sec. 4.3): p -= lr g, optionally clearing g.
__global__ __launch_bounds__(256) void k_sgd(int64_t n, float* __restrict__ p, float* __restrict__ g, float lr,
                                             int zero_grad) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    p[i] = fmaf(-lr, gi, p[i]);
    if (zero_grad) g[i] = 0.0f;
}

inline int64_t grid_for(int64_t n_blocks) { return 8 * ((n_blocks + 7) / 8); }
// Grid of xcd_interleave over n_blocks logical workgroups in runs of chunk.
inline int64_t rows_grid(int64_t n_blocks, int64_t chunk) { return 8 * chunk * (((n_blocks + chunk - 1) / chunk + 7) / 8); }

inline Way way_of(const KTree& t) { return way_of(t.depth(), t.brick_level(), t.grid_level()); }
// The kernels of a batch: direct ones, else those for any tree.
inline Way way_of(int n_jobs, const KJob* jobs) {
    for (int j = 0; j < n_jobs; ++j)
        if (way_of(jobs[j].tr) != kDirect) return kAny;
    return kDirect;
}

// Dynamic LDS of the node stack: one int per lane and tree level.  Trees whose
// grid reaches the brick level keep no node path.
inline size_t stack_bytes(const KTree& t) {
    return way_of(t) == kDirect ? 0 : sizeof(int) * kBlock * (size_t)t.depth();
}

// Record-load plan: "fast" loads the padded record with the widest vectors,
// "generic" uses dword loads of exactly the record (rounded to whole dwords).
template <typename T, int K>
struct Plan {
    static constexpr int NE = 3 * K;
    static constexpr int FAST_VEC = (sizeof(T) == 4) ? 16 : ((NE * 2) % 16 == 0 ? 16 : 8);
    static constexpr int FAST_NL = ((NE * (int)sizeof(T) + FAST_VEC - 1) / FAST_VEC) * FAST_VEC / (int)sizeof(T);
    static constexpr int GEN_NL = (sizeof(T) == 2) ? ((NE + 1) / 2) * 2 : NE;
};

template <typename T, int K>
bool use_fast(const po_tree* t) {
    using P = Plan<T, K>;
    return t->vec_bytes >= P::FAST_VEC && t->stride >= P::FAST_NL &&
           ((size_t)t->stride * sizeof(T)) % P::FAST_VEC == 0;
}

// Load plan of codebook records: K 16-bit positions.
template <int K>
struct CbPlan {
    static constexpr int FAST_VEC = (2 * K) % 16 == 0 ? 16 : 8;
    static constexpr int FAST_NL = ((2 * K + FAST_VEC - 1) / FAST_VEC) * FAST_VEC / 2;
    static constexpr int GEN_NL = (K + 1) / 2 * 2;
};

template <int K>
bool use_fast_cb(const po_tree* t) {
    using P = CbPlan<K>;
    return t->vec_bytes >= P::FAST_VEC && t->stride >= P::FAST_NL && ((size_t)t->stride * 2) % P::FAST_VEC == 0;
}

template <typename T, int K, Way W>
hipError_t rays_t(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op, float* rgb,
                  float* aux, hipStream_t s) {
    using P = Plan<T, K>;
    const int64_t nb = (n + kBlock - 1) / kBlock;
    dim3 grid((unsigned)grid_for(nb)), block(kBlock);
    const size_t lds = stack_bytes(t->kt);
    const bool fast = use_fast<T, K>(t);
    const int v = po_fwd_variant(op, aux, t->kt);
    if (v != PO_FWD_VIEW) aux = nullptr;
    if constexpr (std::is_same_v<T, __half>) {
        if (v == PO_FWD_CB) {
            using Q = CbPlan<K>;
            if (use_fast_cb<K>(t))
                hipLaunchKernelGGL((k_render_rays<T, K, Q::FAST_VEC, Q::FAST_NL, PO_FWD_CB, W>), grid, block, lds, s,
                                   t->kt, n, nb, o, d, op, rgb, nullptr);
            else
                hipLaunchKernelGGL((k_render_rays<T, K, 4, Q::GEN_NL, PO_FWD_CB, W>), grid, block, lds, s, t->kt, n, nb,
                                   o, d, op, rgb, nullptr);
            return hipGetLastError();
        }
    }
#define PO_RAYS(V_)                                                                                              \
    do {                                                                                                        \
        if (fast)                                                                                               \
            hipLaunchKernelGGL((k_render_rays<T, K, P::FAST_VEC, P::FAST_NL, V_, W>), grid, block, lds, s, t->kt, n, \
                               nb, o, d, op, rgb, aux);                                                         \
        else                                                                                                    \
            hipLaunchKernelGGL((k_render_rays<T, K, 4, P::GEN_NL, V_, W>), grid, block, lds, s, t->kt, n, nb, o, d, \
                               op, rgb, aux);                                                                   \
    } while (0)
    if (v == PO_FWD_VIEW)
        PO_RAYS(PO_FWD_VIEW);
    else if (v == PO_FWD_SG)
        PO_RAYS(PO_FWD_SG);
    else
        PO_RAYS(PO_FWD_SH);
#undef PO_RAYS
    return hipGetLastError();
}

template <typename T, int K, int MAXJ, Way W>
hipError_t camera_t(const po_tree* t, int n_jobs, KJob* jobs, int n_blocks, int variant, hipStream_t s) {
    using P = Plan<T, K>;
    KBatch<MAXJ> B;
    for (int j = 0; j < n_jobs; ++j) B.job[j] = jobs[j];
    for (int j = n_jobs; j < MAXJ; ++j) B.job[j] = jobs[0];
    B.n_jobs = n_jobs;
    B.n_blocks = n_blocks;
    size_t lds = 0;
    for (int j = 0; j < n_jobs; ++j) lds = std::max(lds, stack_bytes(jobs[j].tr));
    dim3 grid((unsigned)(MAXJ == 1 ? rows_grid(n_blocks, 4 * (int64_t)jobs[0].tiles_x) : grid_for(n_blocks))),
        block(kBlock);
    if constexpr (std::is_same_v<T, __half>) {
        if (variant == PO_FWD_CB) {
            using Q = CbPlan<K>;
            if (use_fast_cb<K>(t))
                hipLaunchKernelGGL((k_render_camera<T, K, Q::FAST_VEC, Q::FAST_NL, MAXJ, PO_FWD_CB, W>), grid, block, lds,
                                   s, B);
            else
                hipLaunchKernelGGL((k_render_camera<T, K, 4, Q::GEN_NL, MAXJ, PO_FWD_CB, W>), grid, block, lds, s, B);
            return hipGetLastError();
        }
    }
    const bool fast = use_fast<T, K>(t);
#define PO_CAM(V_)                                                                                               \
    do {                                                                                                        \
        if (fast)                                                                                               \
            hipLaunchKernelGGL((k_render_camera<T, K, P::FAST_VEC, P::FAST_NL, MAXJ, V_, W>), grid, block, lds, s, B); \
        else                                                                                                    \
            hipLaunchKernelGGL((k_render_camera<T, K, 4, P::GEN_NL, MAXJ, V_, W>), grid, block, lds, s, B);        \
    } while (0)
    if (variant == PO_FWD_VIEW)
        PO_CAM(PO_FWD_VIEW);
    else if (variant == PO_FWD_SG)
        PO_CAM(PO_FWD_SG);
    else
        PO_CAM(PO_FWD_SH);
#undef PO_CAM
    return hipGetLastError();
}

template <typename T, int K, int SRC, Way W>
hipError_t split_t(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S, hipStream_t s) {
    using P = Plan<T, K>;
    KBatch<1> B;
    B.job[0] = job;
    B.n_jobs = 1;
    B.n_blocks = n_blocks;
    // counters cleared by a kernel rather than a memset node, so that the
    // launches can also be captured in a graph
    hipLaunchKernelGGL(k_zero_i32, dim3(2), dim3(kSplitRegions), 0, s, S.count, 2 * kSplitRegions);
    // camera: tile rows dealt over the XCDs (xcd_interleave)
    const int64_t g1n = SRC == 0 ? rows_grid(n_blocks, 4 * (int64_t)job.tiles_x) : grid_for(n_blocks);
    dim3 g1((unsigned)g1n), g2((unsigned)(kSplitRegions * (S.region_slots / kBlock))), blk(kBlock);
    const size_t lds = stack_bytes(job.tr);
    const bool fast = use_fast<T, K>(t);
#define PO_SPLIT(VEC_, NL_, V_)                                                                        \
    do {                                                                                              \
        if constexpr (SRC == 0)                                                                       \
            hipLaunchKernelGGL((k_render_camera_split<T, K, VEC_, NL_, V_, W>), g1, blk, lds, s, B, S);  \
        else                                                                                          \
            hipLaunchKernelGGL((k_render_rays_split<T, K, VEC_, NL_, V_, W>), g1, blk, lds, s, B, S);    \
        hipLaunchKernelGGL((k_render_chunks<T, K, VEC_, NL_, V_, SRC, W>), g2, blk, lds, s, B, S);      \
        hipLaunchKernelGGL((k_render_subchunks<T, K, VEC_, NL_, V_, SRC, W>), g2, blk, lds, s, B, S);   \
        hipLaunchKernelGGL((k_render_join<T, K, VEC_, NL_, V_, SRC, W>), g2, blk, lds, s, B, S);        \
    } while (0)
    if constexpr (std::is_same_v<T, __half>) {
        if (variant == PO_FWD_CB) {
            using Q = CbPlan<K>;
            if (use_fast_cb<K>(t))
                PO_SPLIT(Q::FAST_VEC, Q::FAST_NL, PO_FWD_CB);
            else
                PO_SPLIT(4, Q::GEN_NL, PO_FWD_CB);
            return hipGetLastError();
        }
    }
    if (variant == PO_FWD_SG) {
        if (fast)
            PO_SPLIT(P::FAST_VEC, P::FAST_NL, PO_FWD_SG);
        else
            PO_SPLIT(4, P::GEN_NL, PO_FWD_SG);
    } else if (variant == PO_FWD_VIEW) {
        if (fast)
            PO_SPLIT(P::FAST_VEC, P::FAST_NL, PO_FWD_VIEW);
        else
            PO_SPLIT(4, P::GEN_NL, PO_FWD_VIEW);
    } else {
        if (fast)
            PO_SPLIT(P::FAST_VEC, P::FAST_NL, PO_FWD_SH);
        else
            PO_SPLIT(4, P::GEN_NL, PO_FWD_SH);
    }
#undef PO_SPLIT
    return hipGetLastError();
}

template <int K, Way W>
hipError_t backward_split_t(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                            const float* rgb_fwd, const float* grad, float* gsig, float* gsh, const KSplit& S0,
                            hipStream_t s) {
    using P = Plan<float, K>;
    KBatch<1> B;
    std::memset(&B, 0, sizeof B);
    B.job[0].tr = t->kt;
    B.job[0].op = op;
    B.n_jobs = 1;
    B.n_blocks = (int)((n + kBlock - 1) / kBlock);
    KSplit S = S0;
    S.ray_o = o;
    S.ray_d = d;
    S.n_rays = n;
    // the pieces of the render of the same rays (before the grids: they
    // cover the queue regions as this pass lays them out)
    po_rays_piece_sizes(n, t->kt.depth(), &S);
    hipLaunchKernelGGL(k_zero_i32, dim3(2), dim3(kSplitRegions), 0, s, S.count, 2 * kSplitRegions);
    dim3 g1((unsigned)grid_for(B.n_blocks)), g2((unsigned)(kSplitRegions * (S.region_slots / kBlock))),
        g3(2u * g2.x), blk(kBlock);
    const size_t lds = stack_bytes(t->kt);
    const bool sg = t->kt.lobes != nullptr;
#define PO_BSPLIT(VEC_, NL_)                                                                                    \
    do {                                                                                                       \
        hipLaunchKernelGGL((k_backward_split<K, VEC_, NL_, W>), g1, blk, lds, s, B, S, rgb_fwd, grad, gsig, gsh); \
        if (sg) {                                                                                              \
            hipLaunchKernelGGL((k_render_chunks<float, K, VEC_, NL_, PO_FWD_SG, 1, W>), g2, blk, lds, s, B, S);   \
            hipLaunchKernelGGL((k_render_subchunks<float, K, VEC_, NL_, PO_FWD_SG, 1, W>), g2, blk, lds, s, B, S); \
            hipLaunchKernelGGL((k_piece_prefix<K, VEC_, NL_, PO_FWD_SG, W>), g2, blk, lds, s, B, S);              \
        } else {                                                                                               \
            hipLaunchKernelGGL((k_render_chunks<float, K, VEC_, NL_, PO_FWD_SH, 1, W>), g2, blk, lds, s, B, S);   \
            hipLaunchKernelGGL((k_render_subchunks<float, K, VEC_, NL_, PO_FWD_SH, 1, W>), g2, blk, lds, s, B, S); \
            hipLaunchKernelGGL((k_piece_prefix<K, VEC_, NL_, PO_FWD_SH, W>), g2, blk, lds, s, B, S);              \
        }                                                                                                      \
        hipLaunchKernelGGL((k_backward_pieces<K, VEC_, NL_, W>), g3, blk, lds, s, B, S, rgb_fwd, grad, gsig, gsh);    \
    } while (0)
    if (use_fast<float, K>(t))
        PO_BSPLIT(P::FAST_VEC, P::FAST_NL);
    else
        PO_BSPLIT(4, P::GEN_NL);
#undef PO_BSPLIT
    return hipGetLastError();
}

// The backward of a kept render: its pieces are in the queue already, and
// its join wrote each piece's prefix over the piece's result, so neither
// the chunk and sub-chunk kernels nor k_piece_prefix run again, and the
// counters are not cleared.
template <int K, Way W>
hipError_t backward_kept_t(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                           const float* rgb_fwd, const float* grad, float* gsig, float* gsh, const KSplit& S0,
                           hipStream_t s) {
    using P = Plan<float, K>;
    KBatch<1> B;
    std::memset(&B, 0, sizeof B);
    B.job[0].tr = t->kt;
    B.job[0].op = op;
    B.n_jobs = 1;
    B.n_blocks = (int)((n + kBlock - 1) / kBlock);
    KSplit S = S0;
    S.ray_o = o;
    S.ray_d = d;
    S.n_rays = n;
    po_rays_piece_sizes(n, t->kt.depth(), &S);
    dim3 g1((unsigned)grid_for(B.n_blocks)), g3(2u * (unsigned)(kSplitRegions * (S.region_slots / kBlock))),
        blk(kBlock);
    const size_t lds = stack_bytes(t->kt);
#define PO_BKEPT(VEC_, NL_)                                                                                       \
    do {                                                                                                         \
        hipLaunchKernelGGL((k_backward_first_kept<K, VEC_, NL_, W>), g1, blk, lds, s, B, S, rgb_fwd, grad, gsig,    \
                           gsh);                                                                                 \
        hipLaunchKernelGGL((k_backward_pieces<K, VEC_, NL_, W>), g3, blk, lds, s, B, S, rgb_fwd, grad, gsig, gsh);  \
    } while (0)
    if (use_fast<float, K>(t))
        PO_BKEPT(P::FAST_VEC, P::FAST_NL);
    else
        PO_BKEPT(4, P::GEN_NL);
#undef PO_BKEPT
    return hipGetLastError();
}

template <int K, Way W>
hipError_t backward_t(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                      const float* rgb_fwd, const float* grad, float* gsig, float* gsh, hipStream_t s) {
    using P = Plan<float, K>;
    const int64_t nb = (n + kBlock - 1) / kBlock;
    dim3 grid((unsigned)grid_for(nb)), block(kBlock);
    if (use_fast<float, K>(t))
        hipLaunchKernelGGL((k_backward<K, P::FAST_VEC, P::FAST_NL, W>), grid, block, stack_bytes(t->kt), s,
                           t->kt, n, nb, o, d, op, rgb_fwd, grad, gsig, gsh);
    else
        hipLaunchKernelGGL((k_backward<K, 4, P::GEN_NL, W>), grid, block, stack_bytes(t->kt), s, t->kt, n, nb,
                           o, d, op, rgb_fwd, grad, gsig, gsh);
    return hipGetLastError();
}

}  // namespace

// EXPR with the coefficient count KK of a tree and, PO_DISPATCH, the walk W of
// its kernels.
#define PO_DISPATCH_K(K_, EXPR)                      \
    switch (K_) {                                    \
        case 1: { constexpr int KK = 1; return EXPR; }   \
        case 4: { constexpr int KK = 4; return EXPR; }   \
        case 9: { constexpr int KK = 9; return EXPR; }   \
        case 16: { constexpr int KK = 16; return EXPR; } \
        case 25: { constexpr int KK = 25; return EXPR; } \
        default: return hipErrorInvalidValue;        \
    }
#define PO_DISPATCH(K_, WAY_, EXPR)                                              \
    switch (WAY_) {                                                              \
        case kDirect: { constexpr Way W = kDirect; PO_DISPATCH_K(K_, EXPR) }     \
        case kPlain: { constexpr Way W = kPlain; PO_DISPATCH_K(K_, EXPR) }       \
        default: { constexpr Way W = kNodes; PO_DISPATCH_K(K_, EXPR) }           \
    }
#define PO_DISPATCH_BATCH(K_, WAY_, EXPR)                                        \
    switch (WAY_) {                                                              \
        case kDirect: { constexpr Way W = kDirect; PO_DISPATCH_K(K_, EXPR) }     \
        default: { constexpr Way W = kAny; PO_DISPATCH_K(K_, EXPR) }             \
    }

// Launchers of the parts, by leaf type (defined in the part named).
hipError_t po_camera_jobs_f32(const po_tree* first, int n_jobs, KJob* jobs, int n_blocks, int variant,
                              hipStream_t s);                                                   // part 1
hipError_t po_camera_jobs_f16(const po_tree* first, int n_jobs, KJob* jobs, int n_blocks, int variant,
                              hipStream_t s);                                                   // part 2
hipError_t po_camera_split_f32(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                               hipStream_t s);                                                  // part 3
hipError_t po_camera_split_f16(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                               hipStream_t s);                                                  // part 4
hipError_t po_rays_split_f32(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                             hipStream_t s);                                                    // part 5
hipError_t po_rays_split_f16(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                             hipStream_t s);                                                    // part 6
// Reads (and with reset, clears) part n's error counter; the device is synchronised by the caller.
#define PO_PART_ERRORS_DECL(n) hipError_t po_part_errors_##n(unsigned long long* out, bool reset);
PO_PART_ERRORS_DECL(0)
PO_PART_ERRORS_DECL(1)
PO_PART_ERRORS_DECL(2)
PO_PART_ERRORS_DECL(3)
PO_PART_ERRORS_DECL(4)
PO_PART_ERRORS_DECL(5)
PO_PART_ERRORS_DECL(6)
PO_PART_ERRORS_DECL(7)
#undef PO_PART_ERRORS_DECL

#define PO_PART_ERRORS_DEF(n)                                                                              \
    hipError_t po_part_errors_##n(unsigned long long* out, bool reset) {                                  \
        if (reset) {                                                                                       \
            const unsigned long long zero = 0ull;                                                          \
            return hipMemcpyToSymbol(HIP_SYMBOL(g_po_errors), &zero, sizeof(zero), 0, hipMemcpyHostToDevice); \
        }                                                                                                  \
        return hipMemcpyFromSymbol(out, HIP_SYMBOL(g_po_errors), sizeof(unsigned long long), 0,            \
                                   hipMemcpyDeviceToHost);                                                 \
    }

#if PO_PART == 1
PO_PART_ERRORS_DEF(1)
hipError_t po_camera_jobs_f32(const po_tree* first, int n_jobs, KJob* jobs, int n_blocks, int variant,
                              hipStream_t s) {
    if (n_jobs == 1) {
        PO_DISPATCH(first->K, way_of(first->kt),
                    (camera_t<float, KK, 1, W>(first, n_jobs, jobs, n_blocks, variant, s)));
    }
    PO_DISPATCH_BATCH(first->K, way_of(n_jobs, jobs),
                      (camera_t<float, KK, PO_BATCH_MAX_JOBS, W>(first, n_jobs, jobs, n_blocks, variant, s)));
}
#endif

#if PO_PART == 2
PO_PART_ERRORS_DEF(2)
hipError_t po_camera_jobs_f16(const po_tree* first, int n_jobs, KJob* jobs, int n_blocks, int variant,
                              hipStream_t s) {
    if (n_jobs == 1) {
        PO_DISPATCH(first->K, way_of(first->kt),
                    (camera_t<__half, KK, 1, W>(first, n_jobs, jobs, n_blocks, variant, s)));
    }
    PO_DISPATCH_BATCH(first->K, way_of(n_jobs, jobs),
                      (camera_t<__half, KK, PO_BATCH_MAX_JOBS, W>(first, n_jobs, jobs, n_blocks, variant, s)));
}
#endif

#if PO_PART == 3
PO_PART_ERRORS_DEF(3)
hipError_t po_camera_split_f32(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                               hipStream_t s) {
    PO_DISPATCH(t->K, way_of(t->kt), (split_t<float, KK, 0, W>(t, job, n_blocks, variant, S, s)));
}
#endif

#if PO_PART == 4
PO_PART_ERRORS_DEF(4)
hipError_t po_camera_split_f16(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                               hipStream_t s) {
    PO_DISPATCH(t->K, way_of(t->kt), (split_t<__half, KK, 0, W>(t, job, n_blocks, variant, S, s)));
}
#endif

#if PO_PART == 5
PO_PART_ERRORS_DEF(5)
hipError_t po_rays_split_f32(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                             hipStream_t s) {
    PO_DISPATCH(t->K, way_of(t->kt), (split_t<float, KK, 1, W>(t, job, n_blocks, variant, S, s)));
}
#endif

#if PO_PART == 6
PO_PART_ERRORS_DEF(6)
hipError_t po_rays_split_f16(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                             hipStream_t s) {
    PO_DISPATCH(t->K, way_of(t->kt), (split_t<__half, KK, 1, W>(t, job, n_blocks, variant, S, s)));
}
#endif

#if PO_PART == 7
PO_PART_ERRORS_DEF(7)
hipError_t po_launch_backward_split(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                                    const float* rgb_fwd, const float* grad, float* gsig, float* gsh,
                                    const KSplit& S, hipStream_t s) {
    PO_DISPATCH(t->K, way_of(t->kt), (backward_split_t<KK, W>(t, n, o, d, op, rgb_fwd, grad, gsig, gsh, S, s)));
}

hipError_t po_launch_backward_kept(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                                   const float* rgb_fwd, const float* grad, float* gsig, float* gsh,
                                   const KSplit& S, hipStream_t s) {
    PO_DISPATCH(t->K, way_of(t->kt), (backward_kept_t<KK, W>(t, n, o, d, op, rgb_fwd, grad, gsig, gsh, S, s)));
}
#endif

#if PO_PART == 0
PO_PART_ERRORS_DEF(0)
hipError_t po_launch_rays(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                          float* rgb, float* aux, hipStream_t s) {
    if (t->desc.dtype == PO_F32) {
        PO_DISPATCH(t->K, way_of(t->kt), (rays_t<float, KK, W>(t, n, o, d, op, rgb, aux, s)));
    } else {
        PO_DISPATCH(t->K, way_of(t->kt), (rays_t<__half, KK, W>(t, n, o, d, op, rgb, aux, s)));
    }
}

hipError_t po_launch_camera_jobs(const po_tree* first, int n_jobs, KJob* jobs, int n_blocks, int variant,
                                 hipStream_t s) {
    return first->desc.dtype == PO_F32 ? po_camera_jobs_f32(first, n_jobs, jobs, n_blocks, variant, s)
                                       : po_camera_jobs_f16(first, n_jobs, jobs, n_blocks, variant, s);
}

hipError_t po_launch_camera_split(const po_tree* t, const KJob& job, int n_blocks, int variant, const KSplit& S,
                                  hipStream_t s) {
    return t->desc.dtype == PO_F32 ? po_camera_split_f32(t, job, n_blocks, variant, S, s)
                                   : po_camera_split_f16(t, job, n_blocks, variant, S, s);
}

hipError_t po_launch_rays_split(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                                float* rgb, float* aux, const KSplit& S0, hipStream_t s) {
    KJob job;
    std::memset(&job, 0, sizeof job);
    job.tr = t->kt;
    job.op = op;
    job.rgb = rgb;
    job.aux = aux;
    KSplit S = S0;
    S.ray_o = o;
    S.ray_d = d;
    S.n_rays = n;
    po_rays_piece_sizes(n, t->kt.depth(), &S);
    const int n_blocks = (int)((n + kBlock - 1) / kBlock);
    const int variant = po_fwd_variant(op, aux, t->kt);
    return t->desc.dtype == PO_F32 ? po_rays_split_f32(t, job, n_blocks, variant, S, s)
                                   : po_rays_split_f16(t, job, n_blocks, variant, S, s);
}

hipError_t po_launch_backward(const po_tree* t, int64_t n, const float* o, const float* d, const KOpts& op,
                              const float* rgb_fwd, const float* grad, float* gsig, float* gsh, hipStream_t s) {
    PO_DISPATCH(t->K, way_of(t->kt), (backward_t<KK, W>(t, n, o, d, op, rgb_fwd, grad, gsig, gsh, s)));
}

hipError_t po_launch_index(const int32_t* nodes, int n_top, int G, int unit, int64_t n_bricks, int32_t* grid,
                           int32_t* bricks, int32_t* sat, hipStream_t s) {
    if (n_bricks > 0) hipLaunchKernelGGL(k_index_bricks, dim3((unsigned)n_bricks), dim3(kBlock), 0, s, bricks);
    if (G > 0) {
        const unsigned cells = ((1u << (3 * G)) + 255u) / 256u, lines = ((1u << (2 * G)) + 255u) / 256u;
        hipLaunchKernelGGL(k_index_grid, dim3(cells), dim3(256), 0, s, nodes, n_top, G, unit, grid);
        for (int axis = 2; axis >= 0; --axis)
            hipLaunchKernelGGL(k_index_sums, dim3(lines), dim3(256), 0, s, grid, sat, G, axis);
        hipLaunchKernelGGL(k_index_grid_boxes, dim3(cells), dim3(256), 0, s, sat, G, unit, grid);
    }
    return hipGetLastError();
}

hipError_t po_launch_leaf_weights(const po_tree* t, const KCam& cam, const KOpts& op, int mode, float* weight,
                                  float* alpha, hipStream_t s) {
    const int n_blocks = 4 * ((cam.W + 15) / 16) * ((cam.H + 15) / 16);
    dim3 grid((unsigned)rows_grid(n_blocks, 4 * (int64_t)((cam.W + 15) / 16))), block(kBlock);
    const size_t lds = stack_bytes(t->kt);
    unsigned* wt = reinterpret_cast<unsigned*>(weight);
    const Way way = way_of(t->kt);
#define PO_WEIGHTS_WAY(T_, MODE_, W_)                                                                            \
    hipLaunchKernelGGL((k_leaf_weights<T_, MODE_, W_>), grid, block, lds, s, t->kt, cam, op, n_blocks, wt, alpha)
#define PO_WEIGHTS(T_, MODE_)                     \
    do {                                          \
        if (way == kDirect)                       \
            PO_WEIGHTS_WAY(T_, MODE_, kDirect);   \
        else if (way == kPlain)                   \
            PO_WEIGHTS_WAY(T_, MODE_, kPlain);    \
        else                                      \
            PO_WEIGHTS_WAY(T_, MODE_, kNodes);    \
    } while (0)
    if (t->desc.dtype == PO_F32) {
        if (mode == 0)
            PO_WEIGHTS(float, 0);
        else
            PO_WEIGHTS(float, 1);
    } else {
        if (mode == 0)
            PO_WEIGHTS(__half, 0);
        else
            PO_WEIGHTS(__half, 1);
    }
#undef PO_WEIGHTS
#undef PO_WEIGHTS_WAY
    return hipGetLastError();
}

hipError_t po_traversal_stats_sync(const po_tree* t, const KCam* cam, int64_t n, const float* o, const float* d,
                                   const KOpts& op, unsigned long long* h_sums, hipStream_t s) {
    // the sums live in this part's g_po_stats; the caller serialises calls
    unsigned long long* d_sums = nullptr;
    hipError_t e = hipGetSymbolAddress((void**)&d_sums, HIP_SYMBOL(g_po_stats));
    if (e != hipSuccess) return e;
    if ((e = hipMemsetAsync(d_sums, 0, 4 * sizeof(unsigned long long), s)) != hipSuccess) return e;
    KCam c;
    std::memset(&c, 0, sizeof c);
    if (cam) c = *cam;
    const int n_blocks = cam ? 4 * ((c.W + 15) / 16) * ((c.H + 15) / 16) : (int)((n + kBlock - 1) / kBlock);
    dim3 grid((unsigned)grid_for(n_blocks)), block(kBlock);
    const size_t lds = stack_bytes(t->kt);
    const bool f32 = t->desc.dtype == PO_F32;
    if (cam && f32)
        hipLaunchKernelGGL((k_traversal_stats<float, 0>), grid, block, lds, s, t->kt, c, o, d, n, op, n_blocks, d_sums);
    else if (cam)
        hipLaunchKernelGGL((k_traversal_stats<__half, 0>), grid, block, lds, s, t->kt, c, o, d, n, op, n_blocks, d_sums);
    else if (f32)
        hipLaunchKernelGGL((k_traversal_stats<float, 1>), grid, block, lds, s, t->kt, c, o, d, n, op, n_blocks, d_sums);
    else
        hipLaunchKernelGGL((k_traversal_stats<__half, 1>), grid, block, lds, s, t->kt, c, o, d, n, op, n_blocks, d_sums);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipMemcpyAsync(h_sums, d_sums, 4 * sizeof(unsigned long long), hipMemcpyDeviceToHost, s)) !=
        hipSuccess)
        return e;
    return hipStreamSynchronize(s);
}

hipError_t po_launch_camera_rays(const KCam& cam, float* o, float* d, hipStream_t s) {
    const int64_t n = (int64_t)cam.W * cam.H;
    hipLaunchKernelGGL(k_camera_rays, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cam, o, d);
    return hipGetLastError();
}

hipError_t po_launch_mse_grad(int64_t n, const float* rgb, const float* target, float scale, float* grad,
                              float* sq_sum, hipStream_t s) {
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_mse_grad, dim3((unsigned)(blocks < 512 ? blocks : 512)), dim3(256), 0, s, n, rgb, target,
                       scale, grad, sq_sum);
    return hipGetLastError();
}

hipError_t po_launch_gather_rays(int64_t n, const int64_t* idx, int64_t n_src, const float* o, const float* d,
                                 const float* t, float* bo, float* bd, float* bt, hipStream_t s) {
    hipLaunchKernelGGL(k_gather_rays, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, idx, n_src, o, d, t,
                       bo, bd, bt);
    return hipGetLastError();
}

hipError_t po_launch_draw_batch(int64_t n, uint64_t seed, uint64_t first, int64_t n_src, const float* o,
                               const float* d, const float* t, float* bo, float* bd, float* bt, float* sq_sum,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_draw_batch, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, seed, first, n_src, o, d,
                       t, bo, bd, bt, sq_sum);
    return hipGetLastError();
}

hipError_t po_launch_sgd(int64_t n, float* param, float* grad, float lr, bool zero_grad, hipStream_t s) {
    hipLaunchKernelGGL(k_sgd, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, param, grad, lr,
                       zero_grad ? 1 : 0);
    return hipGetLastError();
}

hipError_t po_read_device_errors(unsigned long long* out) {
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return e;
    hipError_t (*const part[PO_PARTS])(unsigned long long*, bool) = {
        po_part_errors_0, po_part_errors_1, po_part_errors_2, po_part_errors_3,
        po_part_errors_4, po_part_errors_5, po_part_errors_6, po_part_errors_7};
    unsigned long long sum = 0;
    for (int i = 0; i < PO_PARTS; ++i) {
        unsigned long long v = 0;
        if ((e = part[i](&v, false)) != hipSuccess) return e;
        sum += v;
    }
    *out = sum;
    return hipSuccess;
}

hipError_t po_reset_device_errors() {
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return e;
    hipError_t (*const part[PO_PARTS])(unsigned long long*, bool) = {
        po_part_errors_0, po_part_errors_1, po_part_errors_2, po_part_errors_3,
        po_part_errors_4, po_part_errors_5, po_part_errors_6, po_part_errors_7};
    for (int i = 0; i < PO_PARTS; ++i)
        if ((e = part[i](nullptr, true)) != hipSuccess) return e;
    return hipSuccess;
}

namespace {
constexpr int kNoAllocDevices = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kNoAllocDevices];  // device address of `scratch`, per device (nullptr: not looked up yet)
}  // namespace

hipError_t po_noalloc_queue(KSplit* S) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kNoAllocDevices) return hipErrorInvalidDevice;
    void* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_noalloc_mu);
        if (!g_noalloc_ptr[dev]) {
            // first call on this device, which is current: its copy of the array
            e = hipGetSymbolAddress(&g_noalloc_ptr[dev], HIP_SYMBOL(scratch));
            if (e != hipSuccess) {
                g_noalloc_ptr[dev] = nullptr;
                return e;
            }
        }
        ptr = g_noalloc_ptr[dev];
    }
    po_split_layout(ptr, kNoAllocRegionSlots, S);
    return hipSuccess;
}

int po_plan_id(const po_tree* t) {
    // record kind (float32, float16, codebook), K and the load plan
    const int kind = t->codebook ? 2 : (t->desc.dtype == PO_F32 ? 0 : 1);
    bool fast = false;
    switch (t->K) {
#define PO_PLAN_CASE(KK)                                                                                    \
    case KK:                                                                                                \
        fast = kind == 2 ? use_fast_cb<KK>(t) : (kind == 0 ? use_fast<float, KK>(t) : use_fast<__half, KK>(t)); \
        break;
        PO_PLAN_CASE(1)
        PO_PLAN_CASE(4)
        PO_PLAN_CASE(9)
        PO_PLAN_CASE(16)
        PO_PLAN_CASE(25)
#undef PO_PLAN_CASE
    }
    return (kind * 64 + t->K) * 2 + (fast ? 1 : 0);
}
#endif  // PO_PART == 0
