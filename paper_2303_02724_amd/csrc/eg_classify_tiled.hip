// eg_classify_tiled.hip -- LDS-tiled classification for 2D and 3D grids.
//
// One workgroup (4 waves) owns a tile of 64 (x, the fastest axis) x TY (x TZ)
// vertices.  It stages the tile plus a one-vertex halo of order keys in LDS
// (coalesced rows; positions outside the grid get the sentinel key 0, which
// is below every vertex, so boundary vertices need no special case: a missing
// neighbour is never upper and never the steepest one).  Then, per vertex:
//
//   (a) steepest-ascent pointer: highest vertex of the closed neighbourhood
//       (Sec. 3.3; the vertex itself iff its upper link is empty);
//   (c) the upper-link mask over the 2(2^n - 1) Freudenthal rows (Alg. 1) and
//       its connectivity from a compile-time table: empty = maximum,
//       disconnected = saddle (beta+ >= 2, Table 1);
//   (b, first part) tile-local pointer jumping in LDS: every pointer is
//       followed while it stays inside the tile, so the kernel writes, for
//       each vertex, either its maximum or the first vertex of its
//       steepest-ascent path outside the tile.  The global pass then needs
//       only a few hops per vertex.
//
// Workgroups are mapped to tiles so that the tiles of one XCD are
// consecutive in memory (their halos then meet in the same L2).
#include "eg_tile.h"

namespace eg {

// Label pass over a tiled grid, one workgroup per tile: the exit codes of a
// tile's vertices point into that tile's own block of the exit list, which
// stays in cache while the tile's rows stream through.  Every list entry is
// final by now.  Vertex codes (a tile whose exits did not fit its region of the
// list) follow their path, one link per tile on it: to its end where the list
// as a whole has room (few tiles overflow their region then; a path has fewer
// than N links, which bounds the walk whatever the label array holds), `hops`
// links where it is capped, and the sweeps of k_codes_rest do what is left.
template <int TY, int TZ, bool WHOLE>
__device__ __forceinline__ void final_rows(const TileArgs& a, int b, const int32_t* __restrict__ res, int hops, uint32_t* flag)
{
    constexpr int YPT = TY / 4;
    const int X = a.X, Y = a.Y, Z = a.Z;
    const int N = X * Y * Z;
    const int SY = X, SZ = X * Y;
    int32_t* lab = a.lab;
    // the wave index is uniform: keep it (and every row quantity) scalar
    const int tid = threadIdx.x, lx = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tx = b % a.tiles_x;
    const int rr = b / a.tiles_x;
    const int ty = rr % a.tiles_y;
    const int tz = rr / a.tiles_y;
    const int gx = tx * 64 + lx;
    constexpr int VPT = YPT * TZ;
    bool notdone = false;
    int vid[VPT], x[VPT];
    // every load of the thread first, then the exit-list look-ups, then the
    // stores: loads and stores of the same array would otherwise serialise
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
        const int gy = ty * TY + wv + 4 * (k / TZ), gz = tz * TZ + (k % TZ);
        const bool in = gx < X && gy < Y && gz < Z;
        vid[k] = in ? gz * SZ + gy * SY + gx : -1;
        x[k] = in ? (WHOLE ? __builtin_nontemporal_load(&lab[vid[k]]) : lab[vid[k]]) : 0;
    }
#pragma unroll
    for (int k = 0; k < VPT; ++k)
        if (x[k] < -N) x[k] = res[-x[k] - 1 - N];
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
        if (x[k] < 0) {
            int y = x[k];
            for (int h = 0; y < 0 && h < hops; ++h) y = y >= -N ? lab[-y - 1] : res[-y - 1 - N];
            x[k] = y;
            notdone |= y < 0;
        }
    }
#pragma unroll
    for (int k = 0; k < VPT; ++k)
        if (vid[k] >= 0) {
            if (WHOLE)
                __builtin_nontemporal_store(x[k], &lab[vid[k]]);
            else
                lab[vid[k]] = x[k];
        }
    if (__ballot(notdone) != 0 && __lane_id() == 0) atomicOr(flag, 1u);
}

// Rows of whole 128-byte lines stream past the caches' normal retention (codes
// and labels are used once; 512^3 210 -> 206 us).  Other rows share their first
// and last lines, and their waves' accesses straddle lines, whose halves should
// meet in the cache rather than go to memory by themselves: 256 fields of any
// sizes in a batch 536 -> 345 us (3D) and 339 -> 219 (2D); whole builds of
// 301 x 384 x 449 float64 samples 607 -> 575 us, of 201 x 190 x 333 258 -> 245.
template <int TY, int TZ>
__device__ __forceinline__ void final_tile(const TileArgs& a, int b, const int32_t* __restrict__ res, int hops, uint32_t* flag)
{
    if ((a.X & 31) == 0)
        final_rows<TY, TZ, true>(a, b, res, hops, flag);
    else
        final_rows<TY, TZ, false>(a, b, res, hops, flag);
}

template <int TY, int TZ>
__global__ __launch_bounds__(256) void k_final_tiled(TileArgs a, const int32_t* __restrict__ res, int hops,
                                                         int flag_slot)
{
    final_tile<TY, TZ>(a, xcd_run(blockIdx.x, a.ntiles), res, hops, &a.ctr[flag_slot]);
}

// The same pass over the tiles of every 2D (or every 3D) field of a batch:
// classes 2 * (NDIM - 2) and the one after it (maximum and minimum graphs)
// own consecutive tiles.
template <int NDIM, int TY, int TZ>
__global__ __launch_bounds__(256) void k_final_tiled_batched(const BatchPlan* __restrict__ plan)
{
    constexpr int c0 = 2 * (NDIM - 2);
    const EG_GPTR(BatchField) fs = plan->fields;
    const int64_t item = plan->class_tile[c0] + blockIdx.x;
    int lo = plan->class_field[c0], hi = plan->class_field[c0 + 2] - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (fs[mid].tile_base <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    const int f = __builtin_amdgcn_readfirstlane(lo);
    const TileArgs a = fs[f].ta;
    const bool capped = plan->capped != 0;
    final_tile<TY, TZ>(a, (int)(item - fs[f].tile_base), fs[f].exres, capped ? plan->tuning.hops : fs[f].N,
                       &plan->bctr[capped ? C_CODES : C_OPEN]);
}

hipError_t launch_final_tiled_batched(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s)
{
    const Tuning& tu = hplan.tuning;
    const int64_t t2 = hplan.class_tile[2] - hplan.class_tile[0];
    const int64_t t3 = hplan.class_tile[4] - hplan.class_tile[2];
    if (t2 > 0) {
        if (tu.tile2 == 1)
            hipLaunchKernelGGL((k_final_tiled_batched<2, 16, 1>), dim3((unsigned)t2), dim3(256), 0, s, dplan);
        else
            hipLaunchKernelGGL((k_final_tiled_batched<2, 32, 1>), dim3((unsigned)t2), dim3(256), 0, s, dplan);
    }
    if (t3 > 0) {
        if (tu.tile3 == 1)
            hipLaunchKernelGGL((k_final_tiled_batched<3, 4, 16>), dim3((unsigned)t3), dim3(256), 0, s, dplan);
        else if (tu.tile3 == 2)
            hipLaunchKernelGGL((k_final_tiled_batched<3, 8, 4>), dim3((unsigned)t3), dim3(256), 0, s, dplan);
        else
            hipLaunchKernelGGL((k_final_tiled_batched<3, 8, 8>), dim3((unsigned)t3), dim3(256), 0, s, dplan);
    }
    return hipGetLastError();
}

// The tiles [first, first + count): every tile of the grid, or the tile rows
// of one slab of a streamed build.  Five waves per SIMD, as many as the LDS of
// the default tile allows, leave 96 registers; its variants spill up to nine
// (full tiles about two, by the bytes that they write beyond their outputs),
// which costs less than the wave does (512^3: 6 % slower with 105 registers
// and four waves).
template <bool MINMODE, int TY, int TZ, bool PTR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_classify3d(TileArgs a, int count)
{
    __shared__ __align__(8) Tile3Lds<TY, TZ> s;
    tile3d<MINMODE, TY, TZ, PTR, SRC_F32>(a, (int)a.first + xcd_run(blockIdx.x, count), s);
}

template <bool MINMODE, int TY>
__global__ __launch_bounds__(256) void k_classify2d(TileArgs a, int count)
{
    __shared__ uint32_t s_u[66 * (TY + 2)];
    __shared__ int32_t s_nxt[64 * TY];
    __shared__ uint32_t s_tmp[8];
    tile2d<MINMODE, TY>(a, (int)a.first + xcd_run(blockIdx.x, count), s_u, s_nxt, s_tmp);
}

TileArgs tile_args(const float* f, const Grid& g, int32_t* lab, int32_t* ptr, const Work& w, int ty, int tz)
{
    TileArgs a{};
    a.f = gptr(f);
    a.lab = gptr(lab);
    a.ptr = gptr(ptr);
    a.ctr = gptr(w.ctr);
    a.mmask = gptr(w.mmask);
    a.smask = gptr(w.smask);
    a.exits = gptr(w.exits);
    a.claims = gptr(w.claims);
    a.X = g.dims[g.ndim - 1];
    a.Y = g.dims[g.ndim - 2];
    a.Z = g.ndim == 3 ? g.dims[0] : 1;
    a.tiles_x = (a.X + 63) / 64;
    a.tiles_y = (a.Y + ty - 1) / ty;
    const int tiles_z = (a.Z + tz - 1) / tz;
    a.ntiles = a.tiles_x * a.tiles_y * tiles_z;
    a.regions = exit_regions(g);
    a.cap_region = region_capacity(w.cap_exit, a.regions);
    return a;
}

// Classification of a batch: for each class of fields (2D/3D x maximum/
// minimum graph) one launch covers the work list of (field, tile) items of
// that class, one workgroup per item, which runs the tile code of its field.
template <int NDIM, bool MINMODE, int TY, int TZ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_classify_batched(const BatchPlan* __restrict__ plan, int cls)
{
    constexpr int HALO2 = 66 * (TY + 2);
    using Lds3 = Tile3Lds<TY, TZ>;
    constexpr int WORDS = NDIM == 3 ? (int)(sizeof(Lds3) / 4) : 8 + HALO2 + 64 * TY;
    __shared__ __align__(8) uint32_t s_mem[WORDS];
    const EG_GPTR(BatchField) fs = plan->fields;
    const int f0 = plan->class_field[cls], f1 = plan->class_field[cls + 1];
    const int64_t item = plan->class_tile[cls] + blockIdx.x;
    // the field of this item: binary search over the class's tile bases
    int lo = f0, hi = f1 - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (fs[mid].tile_base <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    const int f = __builtin_amdgcn_readfirstlane(lo);
    const int tile = (int)(item - fs[f].tile_base);
    const TileArgs a = fs[f].ta;
    if constexpr (NDIM == 3) {
        Lds3& s = *reinterpret_cast<Lds3*>(s_mem);
        if (a.ptr)
            tile3d<MINMODE, TY, TZ, true, SRC_F32>(a, tile, s);
        else
            tile3d<MINMODE, TY, TZ, false, SRC_F32>(a, tile, s);
    } else {
        tile2d<MINMODE, TY>(a, tile, s_mem + 8, reinterpret_cast<int32_t*>(s_mem + 8 + HALO2), s_mem);
    }
}

template <int NDIM, int TY, int TZ>
static void launch_class(int c, unsigned grid, const BatchPlan* dplan, hipStream_t s)
{
    if (c & 1)
        hipLaunchKernelGGL((k_classify_batched<NDIM, true, TY, TZ>), dim3(grid), dim3(256), 0, s, dplan, c);
    else
        hipLaunchKernelGGL((k_classify_batched<NDIM, false, TY, TZ>), dim3(grid), dim3(256), 0, s, dplan, c);
}

hipError_t launch_classify_batched(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s)
{
    for (int c = 0; c < 4; ++c) {
        const int64_t tiles = hplan.class_tile[c + 1] - hplan.class_tile[c];
        if (tiles <= 0) continue;
        const unsigned grid = (unsigned)tiles;
        const Tuning& tu = hplan.tuning;
        if (c < 2) {
            if (tu.tile2 == 1)
                launch_class<2, 16, 1>(c, grid, dplan, s);
            else
                launch_class<2, 32, 1>(c, grid, dplan, s);
        } else {
            if (tu.tile3 == 1)
                launch_class<3, 4, 16>(c, grid, dplan, s);
            else if (tu.tile3 == 2)
                launch_class<3, 8, 4>(c, grid, dplan, s);
            else
                launch_class<3, 8, 8>(c, grid, dplan, s);
        }
    }
    return hipGetLastError();
}

template <int TY, int TZ>
static void launch_3d(const TileArgs& a, bool minima, int count, hipStream_t s)
{
    const dim3 g(count), b(256);
    if (minima) {
        if (a.ptr)
            hipLaunchKernelGGL((k_classify3d<true, TY, TZ, true>), g, b, 0, s, a, count);
        else
            hipLaunchKernelGGL((k_classify3d<true, TY, TZ, false>), g, b, 0, s, a, count);
    } else {
        if (a.ptr)
            hipLaunchKernelGGL((k_classify3d<false, TY, TZ, true>), g, b, 0, s, a, count);
        else
            hipLaunchKernelGGL((k_classify3d<false, TY, TZ, false>), g, b, 0, s, a, count);
    }
}

template <int TY>
static void launch_2d(const TileArgs& a, bool minima, int count, hipStream_t s)
{
    if (minima)
        hipLaunchKernelGGL((k_classify2d<true, TY>), dim3(count), dim3(256), 0, s, a, count);
    else
        hipLaunchKernelGGL((k_classify2d<false, TY>), dim3(count), dim3(256), 0, s, a, count);
}

hipError_t launch_final_tiled(const Grid& g, int32_t* lab, const Work& w, const Tuning& tu, int hops, int flag_slot,
                              hipStream_t s)
{
    int ty, tz;
    tile_shape(tu, g.ndim, &ty, &tz);
    const TileArgs a = tile_args(nullptr, g, lab, nullptr, w, ty, tz);
    if (g.ndim == 3) {
        if (tu.tile3 == 1)
            hipLaunchKernelGGL((k_final_tiled<4, 16>), dim3(a.ntiles), dim3(256), 0, s, a, w.exres, hops, flag_slot);
        else if (tu.tile3 == 2)
            hipLaunchKernelGGL((k_final_tiled<8, 4>), dim3(a.ntiles), dim3(256), 0, s, a, w.exres, hops, flag_slot);
        else
            hipLaunchKernelGGL((k_final_tiled<8, 8>), dim3(a.ntiles), dim3(256), 0, s, a, w.exres, hops, flag_slot);
    } else if (g.ndim == 2) {
        if (tu.tile2 == 1)
            hipLaunchKernelGGL((k_final_tiled<16, 1>), dim3(a.ntiles), dim3(256), 0, s, a, w.exres, hops, flag_slot);
        else
            hipLaunchKernelGGL((k_final_tiled<32, 1>), dim3(a.ntiles), dim3(256), 0, s, a, w.exres, hops, flag_slot);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_classify_tiled(const float* f, const Grid& g, bool minima, int32_t* lab, int32_t* ptr,
                                 const Work& w, const Tuning& tu, hipStream_t s, int64_t first, int64_t count)
{
    int ty, tz;
    tile_shape(tu, g.ndim, &ty, &tz);
    TileArgs a = tile_args(f, g, lab, ptr, w, ty, tz);
    if (count < 0) {
        first = 0;
        count = a.ntiles;
    }
    if (first < 0 || first + count > a.ntiles) return hipErrorInvalidValue;
    if (count == 0) return hipSuccess;
    a.first = (uint32_t)first;
    const int n = (int)count;
    if (g.ndim == 3) {
        if (tu.tile3 == 1)
            launch_3d<4, 16>(a, minima, n, s);
        else if (tu.tile3 == 2)
            launch_3d<8, 4>(a, minima, n, s);
        else
            launch_3d<8, 8>(a, minima, n, s);
    } else if (g.ndim == 2) {
        if (tu.tile2 == 1)
            launch_2d<16>(a, minima, n, s);
        else
            launch_2d<32>(a, minima, n, s);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace eg
