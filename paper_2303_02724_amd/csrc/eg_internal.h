// eg_internal.h -- shared definitions of the HIP extremum-graph library.
//
// Vertex order.  The simulated-perturbation order of Sec. 3.3 (u below v iff
// f[u] < f[v], or f[u] == f[v] and u < v) is evaluated with a 32-bit
// order-preserving integer image of the float (order_key): after -0 is mapped
// to +0, x < y as floats iff key(x) < key(y) as unsigned integers.  Ties
// between equal keys are decided by linear index.  For the minimum graph the
// order is reversed, which equals using ~key with the tie-break reversed.
//
// Neighbour rows.  The 2(2^n - 1) Freudenthal neighbours (Alg. 1) are stored
// as rows sorted lexicographically by coordinate offset: the {0,-1}^n rows
// first, then the {0,1}^n rows.  For any in-bounds neighbours this row order is
// the order of their linear indices, and the vertex itself sits between the
// two halves.  So a scan of the closed neighbourhood in row order visits
// vertices in increasing index order, and "later wins ties" is a single >=.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "eg.h"

namespace eg {

constexpr int kMaxNb = 126;         // 2(2^6 - 1)
constexpr int kJumpHops = 64;       // default links per pointer-jumping pass
constexpr int kCappedSweeps = 4;    // most sweeps over a capped exit list
constexpr int kSumRow = 8192;  // entries per row of the stage (d) block sums
constexpr int kArcBlocks = 4096;    // most blocks per field of the stage (d) kernels
// The exit list of a grid of many tiles is split into regions, one for each of
// the eight XCDs (workgroups are dispatched to them round-robin).  A tile
// claims its block with an atomic on its region's counter (in turn, over all
// launches of a grid, so that the regions fill evenly): one counter for all
// serialised the tiles' claims at 12.5 ns each, 410 us at 512^3, which hid
// everything else the classification gained.  And the kernels that resolve a
// region run on its XCD, whose tiles are neighbours, so their gathers meet in
// one L2.  Below kRegionTiles tiles an uneven split could fill one region, so
// there is only one.  The tiles counted are those of the default shape: the
// list's layout follows from the grid alone, so that stages which run with
// other tiles (a tuning word changed between them, the fixed tile of the typed
// classification) agree on it.
constexpr int kRegions = 8;
constexpr int kRegionTiles = 512;
constexpr int kRegionStride = 32;  // counters lie 128 bytes apart
static_assert(kArcBlocks + kRegions * kRegionStride <= kSumRow, "the counters sit behind row 0's block sums");
constexpr int kArcVertsPerBlock = 8192;  // stage (d) blocks: one per this many vertices
constexpr int kTile3Y = 8, kTile3Z = 8;  // default 3D tile: 64 x 8 x 8 vertices
constexpr int kTile2Y = 32;             // default 2D tile: 64 x 32 vertices

// Decoded eg_out.tuning.
struct Tuning {
    int tile3;  // 0: 64x8x8, 1: 64x4x16, 2: 64x8x4
    int tile2;  // 0: 64x32, 1: 64x16
    int hops;   // links per label sweep
    int64_t exit_cap;  // most exit-list entries (0: the default capacity)
};
bool decode_tuning(uint32_t t, Tuning* out);
// Most sweeps of a label kernel over its entries on a grid of n vertices: a
// steepest-ascent path has fewer than n links and every sweep leaves an entry
// at least `hops` links further on or final.
__host__ __device__ inline int sweeps_for(const Tuning& t, int64_t n) { return (int)(n / t.hops) + 2; }
inline void tile_shape(const Tuning& t, int ndim, int* ty, int* tz)
{
    if (ndim == 3) {
        static const int ys[3] = {8, 4, 8}, zs[3] = {8, 16, 4};
        *ty = ys[t.tile3];
        *tz = zs[t.tile3];
    } else {
        static const int ys[2] = {32, 16};
        *ty = ys[t.tile2];
        *tz = 1;
    }
}

// counter slots in the workspace (uint32 each)
enum : int {
    C_NAN = 0,
    C_NMAX = 1,
    C_NSAD = 2,
    C_PASSES = 6,  // sweeps over the labels of untiled grids and of capped exit lists
    C_CODES = 16,  // capped exit lists: the tile-ordered pass left labels open
    C_OPEN = 17,   // labels left over by the last label kernel (an internal error)
    C_SLOTS = 64,
};

struct Grid {
    int32_t ndim;
    int32_t N;
    int32_t dims[EG_MAX_NDIM];
};

// Critical vertices between classification and stage (d) are kept as two
// bitmasks (maxima, saddles) in a row-padded layout: the grid is cut into
// rows along its fastest axis (X vertices each), every row takes XW =
// ceil(X / 64) 64-bit words, and vertex (row, x) is bit x % 64 of word
// row * XW + x / 64.  A wave of a 64-wide tile writes exactly one word per
// row, and a scan over the words lists the vertices in ascending order.
inline int64_t mask_words(int64_t N, int64_t X) { return (N / X) * ((X + 63) / 64); }

// Carved workspace.
struct Work {
    uint32_t* ctr;    // [C_SLOTS]
    uint64_t* mmask;  // [words] maxima
    uint64_t* smask;  // [words] saddles
    uint32_t* bsum;   // [4 * kSumRow] per-block counts of stage (d)
    uint4* atmp;      // [cap_sad] the first four arcs of every saddle ([2 cap_sad], eight, from 4D on)
    uint32_t* claims; // exit-list counters, region r at [kRegionStride r] (behind row 0 of bsum)
    uint32_t* exits;  // [cap_exit] exit vertices published by the tiles
    int32_t* exres;   // [cap_exit] their labels while being resolved
    uint32_t* keys;   // [N] order keys of the untiled grids (1D, 4D, 5D); else null
    int64_t words;
    int64_t cap_exit;
    size_t bytes;
};

// Pointers to device memory in the structs below are typed as global-memory
// pointers in device code (same 64-bit layout as the host's plain pointers).
// Structs read from a batch plan would otherwise give the compiler generic
// pointers, whose flat instructions also wait on the LDS counter.
#if defined(__HIP_DEVICE_COMPILE__)
#define EG_GPTR(T) __attribute__((address_space(1))) T*
#else
#define EG_GPTR(T) T*
#endif
template <class T>
__host__ __device__ inline EG_GPTR(T) gptr(T* p)
{
    return (EG_GPTR(T))p;
}

// Everything a classification tile needs to know about its field.
struct TileArgs {
    EG_GPTR(const float) f;
    EG_GPTR(int32_t) lab;
    EG_GPTR(int32_t) ptr;
    EG_GPTR(uint32_t) ctr;
    EG_GPTR(uint64_t) mmask;
    EG_GPTR(uint64_t) smask;
    EG_GPTR(uint32_t) exits;
    EG_GPTR(uint32_t) claims;  // entries requested, region r at [kRegionStride r]
    int32_t X, Y, Z, tiles_x, tiles_y, ntiles;
    uint32_t cap_region;       // entries per region
    uint32_t regions;          // 1 or kRegions
    uint32_t dtype;            // the samples behind f (eg_dtype)
    uint32_t first;            // workgroups of the grid before this launch's (the slabs of a streamed build)
};

// Everything stage (d) needs to know about its field.
struct ArcArgs {
    EG_GPTR(const float) f;
    EG_GPTR(const uint32_t) keys;  // order keys when classification stored them, else null
    EG_GPTR(const int32_t) lab;
    EG_GPTR(const uint64_t) mmask;
    EG_GPTR(const uint64_t) smask;
    EG_GPTR(uint32_t) bsum;
    EG_GPTR(uint4) atmp;
    EG_GPTR(uint32_t) ctr;
    EG_GPTR(int32_t) header;
    EG_GPTR(int32_t) maxima;
    EG_GPTR(int32_t) saddles;
    EG_GPTR(int32_t) beta;  // may be null
    EG_GPTR(int32_t) offsets;
    EG_GPTR(int32_t) arcs;
    int32_t ndim, minima, N, X, XW, words;
    int32_t dims[EG_MAX_NDIM];
    uint32_t cap_max, cap_sad, cap_arc;
    int32_t arc_blocks;  // blocks of this field in the stage (d) kernels (<= kArcBlocks)
    int32_t dtype;       // the samples behind f (eg_dtype)
    // flag of the last label kernel (set: some label is still a code, the
    // header reports EG_ERR_UNRESOLVED); null: not checked
    EG_GPTR(const uint32_t) last_flag;
};

// The outputs of eg_paths for one field.
struct PathArgs {
    EG_GPTR(const int32_t) ptr;
    EG_GPTR(int32_t) pair_offsets;
    EG_GPTR(int32_t) path_offsets;
    EG_GPTR(int32_t) vertices;
    EG_GPTR(int32_t) header;
    EG_GPTR(int32_t) rec;  // scratch for the vertices the count pass meets (the exit list and its labels)
    int64_t cap_rec;
    uint32_t cap_paths, cap_vertices;
};

// One field of a batch (device-resident plan, built on the host).
struct BatchField {
    TileArgs ta;
    ArcArgs arc;
    int32_t ndim, minima, N, pad0;
    int64_t tile_base;   // exclusive prefix over fields of tiles
    int64_t arc_base;    // ... of stage (d) blocks
    EG_GPTR(int32_t) exres;
};

struct BatchPlan {
    int32_t count, pad0;
    Tuning tuning;
    int64_t total_tiles, total_arc_blocks;
    // fields are ordered by class (2D max, 2D min, 3D max, 3D min); class c
    // owns fields [class_field[c], class_field[c + 1]) and tiles
    // [class_tile[c], class_tile[c + 1])
    int32_t class_field[5];
    int32_t capped;              // some field's exit list is capped (exits_capped)
    int64_t class_tile[5];
    EG_GPTR(uint32_t) bctr;      // [C_SLOTS] batch counters (label flags)
    EG_GPTR(BatchField) fields;  // device address of fields[] (right after this header)
    const BatchPlan* dev; // device address of this plan (start of the batch workspace)
    int64_t plan_bytes;
};

// Host: table rows for ndim (Alg. 1), independent of dims.  Returns k.  The
// adjacency of row j is adj[j * W .. j * W + W), W = (k + 63) / 64 words.
int make_rows(int ndim, int8_t (*off)[EG_MAX_NDIM], uint64_t* adj);
// Host: carve (or size, when base == nullptr) the workspace of a grid with N
// vertices.
Work carve(void* base, int ndim, int64_t N, int64_t X, int64_t cap_sad, int64_t exit_cap = 0);
// Exit-list capacity for a grid of N vertices (label codes need N + cap < 2^31).
int64_t exit_capacity(int64_t N);
// Whether the list of a grid of N vertices holds less than the entries that its
// tiles may want: capped by the tuning word, or by the codes' room on a grid
// near 2^31 vertices.
inline bool exits_capped(const Work& w, int64_t N) { return w.cap_exit < (N / 2 > 4096 ? N / 2 : 4096); }
// ------------------------------------------------------------------ device

// Keys lie in [1, 0xFFFFFFFE] in both modes (non-NaN values map into
// [0x007FFFFF, 0xFF800000]; NaN patterns, reported as an error, are clamped),
// so 0 is a sentinel below every vertex, used for positions outside the grid:
// no pointer can ever leave the grid.
// Adding +0.0 turns -0 into +0 (round to nearest) and leaves every other
// value unchanged; the sign-dependent flip makes unsigned order equal float
// order; the clamp keeps NaN patterns off the sentinel.
__device__ __forceinline__ uint32_t order_key(float x)
{
    const uint32_t b = __float_as_uint(x + 0.0f);
    const uint32_t k = b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
    return min(max(k, 1u), 0xFFFFFFFEu);
}

template <bool MINMODE>
__device__ __forceinline__ uint32_t mode_key(float x)
{
    const uint32_t k = order_key(x);
    return MINMODE ? ~k : k;
}

// f(std::integral_constant<int, i>) for i in [I, N): compile-time row indices.
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// Upper-link masks, one 32-bit word per 32 rows, built from the highest row
// down: up = 2 up + (u above c), where the comparison's lane mask is the carry
// of an add that doubles the word (two instructions per row); a row that wins
// ties is above at equal keys.
template <bool WINS_TIE>
__device__ __forceinline__ uint32_t push_above(uint32_t up, uint32_t u, uint32_t c)
{
    uint32_t r;
    if constexpr (WINS_TIE)
        asm("v_cmp_ge_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %3, %3, vcc" : "=v"(r) : "v"(u), "v"(c), "v"(up) : "vcc");
    else
        asm("v_cmp_gt_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %3, %3, vcc" : "=v"(r) : "v"(u), "v"(c), "v"(up) : "vcc");
    return r;
}
// The first row's comparison as the mask's lowest bit (no zero to double).
template <bool WINS_TIE>
__device__ __forceinline__ uint32_t first_above(uint32_t u, uint32_t c)
{
    uint32_t r;
    if constexpr (WINS_TIE)
        asm("v_cmp_ge_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, 0, 0, vcc" : "=v"(r) : "v"(u), "v"(c) : "vcc");
    else
        asm("v_cmp_gt_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, 0, 0, vcc" : "=v"(r) : "v"(u), "v"(c) : "vcc");
    return r;
}

// Workgroups are dispatched to the eight XCDs round-robin: workgroup b of n
// takes item xcd_run(b, n), so that each XCD works on a run of consecutive
// items (the first n % 8 runs are one item longer).
__device__ __forceinline__ int xcd_run(int b, int n)
{
    const int x = b & 7;
    return x * (n >> 3) + min(x, n & 7) + (b >> 3);
}

// Links between label entries (see the codes below and eg_classify.hip): at
// device scope when `fresh`.
__device__ __forceinline__ int link_at(const int32_t* p, bool fresh)
{
    return fresh ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
__device__ __forceinline__ int next_link(const int32_t* lab, const int32_t* res, int N, int x, bool fresh)
{
    return link_at(x >= -N ? lab + (-x - 1) : res + (-x - 1 - N), fresh);
}

// One sweep over a[0, n) by quads t, t + stride, ..., the last n % 4 entries by
// threads t < n % 4: four consecutive entries per thread (one 16-byte access,
// four independent chains in flight).  Returns whether an entry of this thread
// is not final.
__device__ __forceinline__ bool sweep(int32_t* a, uint32_t n, const int32_t* lab, const int32_t* res, int N, int hops,
                                      uint32_t t, uint32_t stride, bool fresh)
{
    int4* a4 = reinterpret_cast<int4*>(a);
    const uint32_t nq = n >> 2;
    bool open = false;
    for (uint32_t q = t; q < nq; q += stride) {
        const int4 x = a4[q];
        if ((x.x | x.y | x.z | x.w) >= 0) continue;  // all four final
        int y0 = x.x, y1 = x.y, y2 = x.z, y3 = x.w;
        for (int h = 0; (y0 < 0 || y1 < 0 || y2 < 0 || y3 < 0) && h < hops; ++h) {
            if (y0 < 0) y0 = next_link(lab, res, N, y0, fresh);
            if (y1 < 0) y1 = next_link(lab, res, N, y1, fresh);
            if (y2 < 0) y2 = next_link(lab, res, N, y2, fresh);
            if (y3 < 0) y3 = next_link(lab, res, N, y3, fresh);
        }
        a4[q] = make_int4(y0, y1, y2, y3);
        open |= (y0 | y1 | y2 | y3) < 0;
    }
    if (t < (n & 3u)) {
        const uint32_t i = (nq << 2) + t;
        int y = a[i];
        for (int h = 0; y < 0 && h < hops; ++h) y = next_link(lab, res, N, y, fresh);
        a[i] = y;
        open |= y < 0;
    }
    return open;
}

// Number i of n (a power of two) with its bits reversed (why the sweeps are
// dealt out in that order: eg_classify.hip).
__device__ __forceinline__ uint32_t spread(uint32_t i, uint32_t n) { return (__brev(i) >> 1) >> __clz(n); }

// The region of the exit list that a workgroup works on, the workgroup's
// first quad in it and the quads between its rounds (nb workgroups, a multiple
// of the regions, blk one of them).
struct ExitPart {
    uint32_t n, at, t, stride;  // entries, index of the first in the list
};
__device__ __forceinline__ ExitPart exit_part(const uint32_t* claims, uint32_t cap_region, uint32_t regions,
                                              uint32_t blk, uint32_t nb)
{
    const uint32_t r = blk & (regions - 1u);
    const uint32_t req = __hip_atomic_load(&claims[kRegionStride * r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t step = regions == 1 ? 0 : 3;
    return ExitPart{req < cap_region ? req : cap_region, r * cap_region, (blk >> step) * 256 + threadIdx.x,
                    (nb >> step) * 256};
}

// Sweeps over all n labels until none is open, by workgroup blk of nb (a power
// of two); counts them in ctr[C_PASSES] and raises *left if some stay open.
__device__ __forceinline__ void codes_rest(int32_t* lab, const int32_t* res, int32_t n, int hops, int sweeps,
                                           uint32_t blk, uint32_t nb, uint32_t* ctr, uint32_t* left)
{
    const uint32_t waves = 4u * nb;
    const uint32_t t = spread(4u * blk + (threadIdx.x >> 6), waves) * 64u + (threadIdx.x & 63u);
    bool open = true;
    int k = 0;
    for (; __ballot(open) != 0 && k < sweeps; ++k)
        open = sweep(lab, (uint32_t)n, lab, res, n, hops, t, 64u * waves, k > 0);
    const bool rest = __ballot(open) != 0;
    if (__lane_id() != 0) return;
    if (rest) atomicOr(left, 1u);
    if (k > 1 || (blk == 0 && threadIdx.x == 0)) atomicMax(&ctr[C_PASSES], (uint32_t)k);
}

// First values of a part of the exit list: its vertices' label codes.
__device__ __forceinline__ void exit_first(const ExitPart& p, const uint32_t* exits, int32_t* res, const int32_t* lab)
{
    const uint32_t nq = p.n >> 2;
    const uint4* e4 = reinterpret_cast<const uint4*>(exits + p.at);
    int4* r4 = reinterpret_cast<int4*>(res + p.at);
    for (uint32_t q = p.t; q < nq; q += p.stride) {
        const uint4 e = e4[q];
        r4[q] = make_int4(lab[e.x], lab[e.y], lab[e.z], lab[e.w]);
    }
    if (p.t < (p.n & 3u)) {
        const uint32_t i = p.at + (nq << 2) + p.t;
        res[i] = lab[exits[i]];
    }
}

// ------------------------------------------------------------------ launchers

// Counters and header to zero.
hipError_t launch_init(const Work& w, int32_t* header, hipStream_t s);
hipError_t launch_classify(const float* f, const Grid& g, bool minima, int32_t* lab, int32_t* ptr, const Work& w,
                           const Tuning& tu, hipStream_t s);
// Classification of the 2D/3D tiles [first, first + count) (tiles in C order:
// tile rows along axis 0 are contiguous ranges); count < 0: every tile.
hipError_t launch_classify_tiled(const float* f, const Grid& g, bool minima, int32_t* lab, int32_t* ptr,
                                 const Work& w, const Tuning& tu, hipStream_t s, int64_t first = 0,
                                 int64_t count = -1);
// The same for a 3D field of another sample type (the default tile).
hipError_t launch_classify_typed(int dtype, const void* f, const Grid& g, bool minima, int32_t* lab, int32_t* ptr,
                                 const Work& w, hipStream_t s);
// Regions of the exit list of a 2D or 3D grid, and entries per region.
inline uint32_t exit_regions(const Grid& g)
{
    const int64_t tx = (g.dims[g.ndim - 1] + int64_t(63)) / 64;
    const int64_t rows = g.ndim == 3 ? (g.dims[1] + int64_t(kTile3Y - 1)) / kTile3Y *
                                           ((g.dims[0] + int64_t(kTile3Z - 1)) / kTile3Z)
                                     : (g.dims[0] + int64_t(kTile2Y - 1)) / kTile2Y;
    return tx * rows >= kRegionTiles ? kRegions : 1;
}
inline uint32_t region_capacity(int64_t cap, uint32_t regions)
{
    return regions == 1 ? (uint32_t)cap : (uint32_t)(cap / regions) & ~3u;
}
TileArgs tile_args(const float* f, const Grid& g, int32_t* lab, int32_t* ptr, const Work& w, int ty, int tz);
ArcArgs arc_args(const float* f, const Grid& g, const eg_out& o, const Work& w);
uint32_t arc_blocks(int64_t N);
hipError_t launch_classify_batched(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s);
hipError_t launch_batched_init(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s);
hipError_t launch_batched_rest(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s);

// Label codes between classification and the label pass (int32):
//   x >= 0            final: the maximum x
//   -N <= x <= -1     "same label as vertex -x-1" (a later vertex of the path)
//   x < -N            "same label as exit-list entry -x-1-N"
__device__ __forceinline__ int exit_list_code(int N, uint32_t idx) { return -(N + 1 + (int)idx); }
hipError_t launch_labels(const Grid& g, int32_t* lab, const Work& w, const Tuning& tu, hipStream_t s);
// Tile-ordered per-vertex label pass (2D/3D grids); raises ctr[flag_slot] if some
// vertex is not final after `hops` links.
hipError_t launch_final_tiled(const Grid& g, int32_t* lab, const Work& w, const Tuning& tu, int hops, int flag_slot,
                              hipStream_t s);
// The tile-ordered pass over every field of a batch; raises bctr[C_OPEN]
// (bctr[C_CODES] where lists are capped).
hipError_t launch_final_tiled_batched(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s);
// Stage (d) of one field: ascending maxima and saddles from the bitmasks,
// the arcs of every saddle, the CSR and the header.
hipError_t launch_arcs(const ArcArgs& a, hipStream_t s);
// Gradient-path geometry of one field (after stage (d)).
hipError_t launch_paths(const ArcArgs& a, const PathArgs& p, hipStream_t s);
// Stage (d) of every field of a batch (fields are blockIdx.y).
hipError_t launch_arcs_batched(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s);

}  // namespace eg
