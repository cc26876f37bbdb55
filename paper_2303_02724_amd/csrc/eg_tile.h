// eg_tile.h -- device code of one 2D or 3D classification tile (see
// eg_classify_tiled.hip for the method), shared by the kernels of float32
// fields and of the other sample types.
#pragma once
#include <utility>

#include "eg_internal.h"
#include "eg_rows.h"
#include "eg_sample.h"

namespace eg {

namespace {
__constant__ Conn3 c_conn3 = make_conn3();
}

constexpr uint64_t make_conn2()
{
    constexpr Rows<2> r = make_rows_ce<2>();
    uint64_t c = 0;
    for (uint32_t m = 1; m < 64u; ++m)
        if (closure_ce<2>(r, m & (~m + 1u), m) == m) c |= uint64_t(1) << m;
    return c;
}

template <int NDIM, int J>
struct Row {
    static constexpr Rows<NDIM> R = make_rows_ce<NDIM>();
    static constexpr int dz = NDIM == 3 ? R.d[J][0] : 0;
    static constexpr int dy = R.d[J][NDIM - 2];
    static constexpr int dx = R.d[J][NDIM - 1];
};

template <int NDIM>
struct Pack {
    static_assert(NDIM <= 3, "two bits per row must fit 32 bits");
    static constexpr Rows<NDIM> R = make_rows_ce<NDIM>();
    static constexpr uint32_t z = NDIM == 3 ? (uint32_t)pack_axis<NDIM>(R, 0) : 0x55555555u;
    static constexpr uint32_t y = (uint32_t)pack_axis<NDIM>(R, NDIM - 2);
    static constexpr uint32_t x = (uint32_t)pack_axis<NDIM>(R, NDIM - 1);
};

// Label encoding written by the classification kernels: a value m >= 0 is
// final (the maximum m); a value -(e + 1) < 0 says "same label as vertex e",
// a later vertex of the steepest-ascent path.  The jump kernel resolves the
// negative entries.

// Resolve the tile's successor array by pointer jumping.  cur[k] holds the
// successor of this thread's k-th vertex (s_idx(k) is its tile index), scaled
// by UNIT (1: tile indices; 4: byte offsets into s_nxt, which spares the
// address shift in every round): below UNIT TILE a vertex of the tile, at or
// above it a tile-local maximum (UNIT (TILE + its own index)), < 0 the
// tile-local code of the exit by which the path leaves the tile; the last two
// end a chain.  Each round replaces every successor inside the tile by that
// vertex's successor, in place.  Only the owning wave writes an entry, and
// every value written is a vertex further along the same path (or its end),
// so any value a wave reads, old or new, is a valid successor that moves its
// chain forward.  Hence every wave runs its own rounds until its own chains
// have ended, with no barrier (a wave that finishes early leaves final
// entries behind); log2 of the longest in-tile path bounds the rounds.  Call
// after a barrier that follows the last store to s_nxt.
template <int VPT, int TILE, int UNIT, class Idx>
__device__ __forceinline__ void double_tile_chains(int (&cur)[VPT], int32_t* s_nxt, Idx s_idx)
{
    static_assert(UNIT == 1 || UNIT == 4, "tile indices or byte offsets");
    constexpr unsigned END = (unsigned)TILE * UNIT;
    bool pending = false;
#pragma unroll
    for (int k = 0; k < VPT; ++k) pending |= (unsigned)cur[k] < END;
    if (__ballot(pending) == 0) return;
    if constexpr (UNIT == 4) {
        // every round issues all its reads before it writes, with no branch:
        // an entry that has ended reads its own slot, which holds its current
        // value
        do {
            int m[VPT];
#pragma unroll
            for (int k = 0; k < VPT; ++k) {
                const int n = cur[k];
                const int at = (unsigned)n < END ? n : 4 * s_idx(k);
                m[k] = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(s_nxt) + at);
            }
            uint32_t lo = ~0u;
#pragma unroll
            for (int k = 0; k < VPT; ++k) {
                cur[k] = m[k];
                s_nxt[s_idx(k)] = m[k];
                lo = min(lo, (uint32_t)m[k]);
            }
            pending = lo < END;
        } while (__ballot(pending) != 0);
        return;
    }
    // the test at the bottom keeps every cur[k] in one register across rounds
    do {
        pending = false;
#pragma unroll
        for (int k = 0; k < VPT; ++k) {
            const int n = cur[k];
            if ((unsigned)n < END) {
                const int m = s_nxt[n];
                cur[k] = m;
                s_nxt[s_idx(k)] = m;
                pending |= (unsigned)m < END;
            }
        }
    } while (__ballot(pending) != 0);
}

// Every vertex whose steepest step leaves the tile gets its own entry of the
// exit list, which records the step's target; before the tile's chains are
// resolved, cur[k] < 0 holds -(target + 1) for such a vertex.  rank_exits
// numbers the tile's exits without a scan: per k, a wave ballot of its
// exiting lanes, the lane's rank among them (mbcnt) and the running count of
// the wave (scalar).  The targets go to s_exv in rank order and cur[k] becomes
// the tile-local code -(rank + 1), which the pointer doubling hands to every
// vertex whose path leaves the tile there.  One atomic per tile claims the
// tile's block of its region of the list: thread 0 issues it here and first needs its value
// in place_exits, after the doubling, so the round trip of a device-wide
// atomic overlaps the doubling instead of stalling the workgroup.  Writes
// s_exv after a barrier, so the caller may alias it with the halo.
template <int VPT>
__device__ __forceinline__ uint32_t rank_exits(int (&cur)[VPT], uint32_t* s_tmp, uint32_t* s_exv,
                                               uint32_t* __restrict__ counter, uint32_t& claim)
{
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t wave_total = 0;
#pragma unroll
    for (int k = 0; k < VPT; ++k) wave_total += (uint32_t)__popcll(__ballot(cur[k] < 0));
    if ((tid & 63) == 0) s_tmp[w] = wave_total;
    __syncthreads();
    uint32_t r0 = 0;  // first rank of this wave's k-th group (uniform)
    for (int k = 0; k < w; ++k) r0 += s_tmp[k];
    const uint32_t total = s_tmp[0] + s_tmp[1] + s_tmp[2] + s_tmp[3];
    claim = 0;
    if (tid == 0 && total) claim = atomicAdd(counter, total);
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
        const uint64_t bal = __ballot(cur[k] < 0);
        if (cur[k] < 0) {
            const uint32_t r =
                r0 + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            s_exv[r] = (uint32_t)(-cur[k] - 1);
            cur[k] = -(int)r - 1;
        }
        r0 += (uint32_t)__popcll(bal);
    }
    return total;
}

// After the doubling: the tile's block of the exit list starts at the claimed
// base; the block is written with coalesced stores.  Entries below the
// capacity are always written, so the list never holds garbage even when the
// tile's block does not fit; such a tile gives its vertices the vertex codes
// of their exits' targets instead of list codes.  Returns whether it fit.
__device__ __forceinline__ bool place_exits(uint32_t total, uint32_t claim, const uint32_t* s_exv, uint32_t* s_tmp,
                                            const TileArgs& a, uint32_t region, uint32_t& base)
{
    const int tid = threadIdx.x;
    if (tid == 0) s_tmp[4] = claim;
    __syncthreads();
    const uint32_t first = s_tmp[4], cap = a.cap_region;
    base = region * cap + first;
    for (uint32_t i = tid; i < total; i += 256)
        if (first + i < cap) a.exits[base + i] = s_exv[i];
    return (uint64_t)first + total <= cap;
}

// The offset that turns a tile-local exit code n < 0 into the label code of
// its list entry: exit_list_code(N, base - n - 1) = n - (N + base).  A tile
// whose block did not fit turns its codes into the vertex codes of the exits'
// targets here instead (offset 0).
template <int VPT>
__device__ __forceinline__ int exit_offset(int (&cur)[VPT], bool fit, uint32_t base, const uint32_t* s_exv, int N)
{
    if (fit) return N + (int)base;
#pragma unroll
    for (int k = 0; k < VPT; ++k)
        if (cur[k] < 0) cur[k] = -(int)s_exv[-cur[k] - 1] - 1;
    return 0;
}

// Critical-vertex bitmasks: each wave handles one 64-vertex row segment of
// the tile per step, which is exactly one mask word (tiles start at
// multiples of 64 along x).  Step k parks its maxima word in lane k and its
// saddle word in lane 32 + k; at the end every lane stores at most one word,
// so the masks cost one store instruction per wave and no atomics.
// v_writelane_b32 (lane `lane` of a vector register takes a scalar value) and
// v_bfe_u32 (which reads only the low five bits of the offset), as the
// compiler's own intrinsics
extern "C" __device__ int eg_writelane(int src, int lane, int old) __asm("llvm.amdgcn.writelane.i32");
extern "C" __device__ uint32_t eg_ubfe(uint32_t src, uint32_t offset, uint32_t width) __asm("llvm.amdgcn.ubfe.i32");

__device__ __forceinline__ void park_word(uint64_t& mine, bool pred, int lane)
{
    const uint64_t b = __ballot(pred);
    uint32_t lo = (uint32_t)eg_writelane((int)(uint32_t)b, lane, (int)(uint32_t)mine);
    uint32_t hi = (uint32_t)eg_writelane((int)(uint32_t)(b >> 32), lane, (int)(uint32_t)(mine >> 32));
    // pin the word here: otherwise the selects sink to the final store and
    // every step's two ballots stay alive in scalar registers until then
    asm volatile("" : "+v"(lo), "+v"(hi));
    mine = ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ void store_words(const TileArgs& a, uint64_t word, int vpt, int row, bool row_in, int tx)
{
    // row: the grid row (gz * Y + gy) of this lane's step; row_in: it exists
    const int lane = __lane_id();
    if ((lane & 31) < vpt && row_in) {
        const int64_t at = (int64_t)row * a.tiles_x + tx;
        (lane < 32 ? a.mmask : a.smask)[at] = word;
    }
}

// A tile of a 2D grid.
template <bool MINMODE, int TY>
__device__ __forceinline__ void tile2d(const TileArgs& a, int b, uint32_t* s_u, int32_t* s_nxt, uint32_t* s_tmp)
{
    static_assert(TY % 4 == 0, "four waves split the rows");
    constexpr int K = 6;
    constexpr int TX = 64;
    constexpr int HX = TX + 2, HY = TY + 2;
    constexpr int TILE = TX * TY;
    constexpr int VPT = TY / 4;
    const float* __restrict__ f = a.f;
    const int X = a.X, Y = a.Y;
    int32_t* __restrict__ lab = a.lab;
    int32_t* __restrict__ ptr = a.ptr;
    uint32_t* __restrict__ ctr = a.ctr;

    // the wave index is uniform: keep it (and every row quantity) scalar
    const int tid = threadIdx.x, lx = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tx = b % a.tiles_x;
    const int ty = b / a.tiles_x;
    const int x0 = tx * TX, y0 = ty * TY;

    bool nan = false;
    {
        // rows of 64 aligned values, one per lane, from a uniform row address
        // (rows outside the grid read a clamped row and are replaced), then
        // the two edge columns of every row (one value per thread); all loads
        // are issued before the first is used
        constexpr int RPW = (HY + 3) / 4;
        constexpr int EDGES = 2 * HY;
        static_assert(EDGES <= 256, "one edge value per thread");
        const int gx = x0 + lx;
        const bool xin = gx < X;
        const int gxc = xin ? gx : X - 1;
        float vals[RPW];
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int gy = y0 + wv + 4 * i - 1;
            const int gyc = min(max(gy, 0), Y - 1);
            vals[i] = f[(int64_t)gyc * X + gxc];
        }
        const int erow = tid >> 1;
        const int egx = (tid & 1) ? x0 + TX : x0 - 1;
        const int egy = y0 + erow - 1;
        const bool ein = tid < EDGES && (unsigned)egx < (unsigned)X && (unsigned)egy < (unsigned)Y;
        const float eval = f[ein ? (int64_t)egy * X + egx : 0];
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int hy = wv + 4 * i;  // uniform
            if (hy < HY) {
                const int gy = y0 + hy - 1;
                const bool ok = xin && (unsigned)gy < (unsigned)Y;
                nan |= ok && hy >= 1 && hy <= TY && vals[i] != vals[i];
                s_u[hy * HX + lx + 1] = ok ? mode_key<MINMODE>(vals[i]) : 0u;
            }
        }
        if (tid < EDGES) s_u[erow * HX + ((tid & 1) ? HX - 1 : 0)] = ein ? mode_key<MINMODE>(eval) : 0u;
    }
    __syncthreads();

    constexpr uint64_t CONN2 = make_conn2();
    static_assert(VPT <= 32, "one mask word per lane");
    int nxt[VPT];
    uint64_t word = 0;  // this lane's parked mask word
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
        const int ly = wv + 4 * k;
        const int gx = x0 + lx, gy = y0 + ly;
        const bool in = gx < X && gy < Y;
        const int li = ly * TX + lx;
        int n = TILE + li;  // vertices outside the grid end their own chain and are never written
        bool is_max = false, is_sad = false;
        int v = 0;
        if (in) {
            const int c = (ly + 1) * HX + (lx + 1);
            const uint32_t uv = s_u[c];
            uint32_t up = 0, best_u = 0;
            int best_j = K;  // K stands for the vertex itself
            // closed neighbourhood in index order (reversed for the minimum
            // graph), so that the later of two equal keys wins with >=
            static_for<0, K + 1>([&](auto step) {
                constexpr int s = decltype(step)::value;
                constexpr int pos = MINMODE ? K - s : s;
                if constexpr (pos == K / 2) {
                    if (uv >= best_u) {
                        best_u = uv;
                        best_j = K;
                    }
                } else {
                    constexpr int j = pos < K / 2 ? pos : pos - 1;
                    using RJ = Row<2, j>;
                    constexpr int off = RJ::dy * HX + RJ::dx;
                    constexpr bool wins_tie = (j >= K / 2) != MINMODE;
                    const uint32_t u = s_u[c + off];
                    const bool above = wins_tie ? (u >= uv) : (u > uv);
                    up |= uint32_t(above) << j;
                    if (u >= best_u) {
                        best_u = u;
                        best_j = j;
                    }
                }
            });
            is_max = up == 0;
            is_sad = !is_max && !((CONN2 >> up) & 1ull);
            v = gy * X + gx;
            int pv = v;
            if (best_j == K) {
                n = TILE + li;  // a maximum ends its chain
            } else {
                const int dy = (int)((Pack<2>::y >> (2 * best_j)) & 3u) - 1;
                const int dx = (int)((Pack<2>::x >> (2 * best_j)) & 3u) - 1;
                pv = v + dy * X + dx;
                const int ly2 = ly + dy, lx2 = lx + dx;
                const bool inside = (unsigned)ly2 < (unsigned)TY && (unsigned)lx2 < (unsigned)TX;
                n = inside ? ly2 * TX + lx2 : -(pv + 1);
            }
            if (ptr) ptr[v] = pv;
        }
        nxt[k] = n;
        park_word(word, is_max, k);
        park_word(word, is_sad, 32 + k);
    }
    {
        const int ly = wv + 4 * (__lane_id() & 31);
        store_words(a, word, VPT, y0 + ly, y0 + ly < Y, tx);
    }
    if (__ballot(nan) != 0 && __lane_id() == 0) atomicOr(&ctr[C_NAN], 1u);
    const int N = X * Y;
    uint32_t claim;
    const uint32_t region = (a.first + blockIdx.x) & (a.regions - 1u);
    uint32_t* counter = a.claims + kRegionStride * region;
    const uint32_t nexit = rank_exits<VPT>(nxt, s_tmp, s_u, counter, claim);  // the halo is no longer read
    auto s_idx = [&](int k) { return (wv + 4 * k) * TX + lx; };
#pragma unroll
    for (int k = 0; k < VPT; ++k) s_nxt[s_idx(k)] = nxt[k];
    __syncthreads();
    // global offset of every tile row from the tile's first vertex (one LDS
    // read per vertex instead of quarter-rate multiplies)
    __shared__ int s_rowoff[TY];
    if (tid < TY) s_rowoff[tid] = tid * X;
    double_tile_chains<VPT, TILE, 1>(nxt, s_nxt, s_idx);
    uint32_t base;
    const bool fit = place_exits(nexit, claim, s_u, s_tmp, a, region, base);
    const int xoff = exit_offset<VPT>(nxt, fit, base, s_u, N);
    const int tile0 = y0 * X + x0;
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
        const int ly = wv + 4 * k;
        const int n = nxt[k];
        if (x0 + lx < X && y0 + ly < Y)
            lab[tile0 + s_rowoff[ly] + lx] = n >= 0 ? tile0 + s_rowoff[(n - TILE) >> 6] + (n & 63) : n - xoff;
    }
}

// 3D variant tuned for large grids.  Rows of the halo are loaded aligned
// (one 256-byte wave load per row plus the two edge columns); each thread
// walks YPT neighbouring rows of the tile along z together, with a sliding
// window of three planes of the positions their neighbourhoods touch (ten for
// two rows, so a vertex costs 5 LDS reads instead of 15); pointer targets stay
// in registers until the halo is no longer needed, then reuse its LDS for the
// tile-local chains, which are resolved by pointer doubling.
//
// Steepest candidate.  A key and the code of its position, six bits that grow
// in visiting order, make one 64-bit number, key << 31 | code << 2; as the
// bits of a double it is positive and finite (keys stay below kKeyTop), so
// v_max_f64, which issues as fast as a 32-bit maximum, takes the larger key
// and among equal keys the later position: the exact steepest candidate, its
// code included, with no second look.  The closed neighbourhood is the four
// upper positions (self included) of the vertex's plane and of the one above,
// and the four lower ones of its plane and of the one below.  Each plane's
// upper and lower maxima are formed once, from pairs shared by the rows, and
// serve two vertices each: 20 vector instructions a vertex, where the maximum
// of 15 bucketed keys, the exact maximum and the test that both agree took 39.
// 512^3, classification: 462 -> 421 us, and 410 once the tiles no longer claimed
// their exits from one counter.
//
// Successor of a vertex as one 32-bit word per code, read from LDS with the
// global offset in one paired read:
//   bits 0..5   faces of the tile the step crosses if the vertex lies on them
//               (x-, x+, y-, y+, z-, z+)
//   bits 6..31  tile-local offset in bytes of the chain array (signed)
// The vertex itself (a maximum) has no faces and the offset 4 TILE, which
// turns its own byte offset into the chain end 4 (TILE + index).  The 3D
// chains hold byte offsets, so a doubling round reads its successor's entry
// without an address shift.

// Store to lane lx of a row whose first element sits at the uniform address
// `row`: the address stays scalar and only the lane's byte offset lives in a
// vector register.
__device__ __forceinline__ void store_row(int32_t* row, uint32_t lane_b, int32_t v)
{
    *reinterpret_cast<int32_t*>(reinterpret_cast<char*>(row) + lane_b) = v;
}

// A key with the code of its position (an inline constant, at most 64: two
// instructions, where the compiler's own 64-bit shift takes two moves more),
// and the larger of two of them.
template <uint32_t CODE>
__device__ __forceinline__ uint64_t coded(uint32_t key)
{
    static_assert(CODE <= 64, "an inline constant");
    uint32_t lo;
    asm("v_lshl_or_b32 %0, %1, 31, %2" : "=v"(lo) : "v"(key), "n"(CODE));
    return (uint64_t)(key >> 1) << 32 | lo;
}
__device__ __forceinline__ uint64_t later_max(uint64_t a, uint64_t b)
{
    uint64_t r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Keys of numbers lie in [0x00800000, 0xFF800000] (the infinities at the ends);
// keys outside come from NaN patterns.
__device__ __forceinline__ bool nan_key(uint32_t k) { return k < 0x00800000u || k > 0xFF800000u; }

template <int TY, int HY, int HX>
__device__ __forceinline__ constexpr uint32_t succ_pack(int dz, int dy, int dx)
{
    const int loff = (dz * TY + dy) * 64 + dx;
    const uint32_t em = (dx < 0 ? 1u : 0u) | (dx > 0 ? 2u : 0u) | (dy < 0 ? 4u : 0u) | (dy > 0 ? 8u : 0u) |
                        (dz < 0 ? 16u : 0u) | (dz > 0 ? 32u : 0u);
    return em | (uint32_t(4 * loff) << 6);
}

// Halo of a 3D tile of a field of samples T: rows of 64 aligned values, one
// per lane, from a uniform row address (rows outside the grid read a clamped
// row), then the two edge columns of every row; all loads first.  Positions
// outside the grid get the key 0.  `nan`: a sample is a NaN; returns whether
// equal keys of this tile mean equal samples.  For the wide types that holds
// where the exact keys lie within about 2^31 of the tile's first vertex's
// (then their distances from near_base are the keys), or where every sample is
// a float32 (or short of the clamped ends, for 32-bit integers); uses
// s_flag[0..3].
template <class T, bool MINMODE, int TY, int TZ, bool FULL>
__device__ __forceinline__ bool stage_samples(const TileArgs& a, int x0, int y0, int z0, uint32_t* s_u,
                                              uint32_t* s_flag, bool& nan)
{
    constexpr int HX = 66, HY = TY + 2, HZ = TZ + 2;
    constexpr int ROWS = HY * HZ;
    constexpr int RPW = (ROWS + 3) / 4;
    constexpr int EDGES = 2 * ROWS;
    static_assert(ROWS % 4 == 0 && EDGES <= 256, "four waves split the rows, one edge value per thread");
    EG_GPTR(const T) f = (EG_GPTR(const T))a.f;
    const int X = a.X, Y = a.Y, Z = a.Z;
    const int tid = threadIdx.x, lx = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gx = x0 + lx;
    const bool xin = FULL || gx < X;
    const int gxc = xin ? gx : X - 1;
    T vals[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int row = wv + 4 * i;
        const int gy = min(max(y0 + row % HY - 1, 0), Y - 1), gz = min(max(z0 + row / HY - 1, 0), Z - 1);
        vals[i] = (f + (int64_t)(gz * Y + gy) * X)[gxc];
    }
    const int erow = tid >> 1;
    const int egx = (tid & 1) ? x0 + 64 : x0 - 1, egy = y0 + erow % HY - 1, egz = z0 + erow / HY - 1;
    const bool ein = tid < EDGES && (unsigned)egx < (unsigned)X && (unsigned)egy < (unsigned)Y &&
                     (unsigned)egz < (unsigned)Z;
    const T eval = f[ein ? (int64_t)(egz * Y + egy) * X + egx : 0];
    nan = ein && eval != eval;
    auto row_in = [&](int i) {
        const int row = wv + 4 * i;
        return xin && (unsigned)(y0 + row % HY - 1) < (unsigned)Y && (unsigned)(z0 + row / HY - 1) < (unsigned)Z;
    };
    uint32_t* own = s_u + wv * HX + lx + 1;  // the rows at immediate offsets
    uint32_t* edge = s_u + erow * HX + ((tid & 1) ? HX - 1 : 0);
    if constexpr (sizeof(T) < 4) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) own[4 * i * HX] = row_in(i) ? tile_key<MINMODE>(vals[i]) : 0u;
        if (tid < EDGES) *edge = ein ? tile_key<MINMODE>(eval) : 0u;
        return true;
    } else {
        const uint64_t base = near_base(exact_of(f[(int64_t)(z0 * Y + y0) * X + x0]));
        uint32_t near[RPW];
        bool far = false, round = false;
        auto look = [&](T x, bool in) {
            const uint64_t r = exact_of(x) - base;
            far |= in && r - 1u >= (uint64_t)kKeyTop - 1u;
            round |= in && !key_is_exact(x);
            nan |= in && x != x;
            return (uint32_t)r;
        };
#pragma unroll
        for (int i = 0; i < RPW; ++i) near[i] = look(vals[i], row_in(i));
        const uint32_t near_edge = look(eval, ein);
        const uint32_t flags = (__ballot(far) != 0 ? 1u : 0u) | (__ballot(round) != 0 ? 2u : 0u);
        if (lx == 0) s_flag[wv] = flags;
        __syncthreads();
        const uint32_t all = s_flag[0] | s_flag[1] | s_flag[2] | s_flag[3];
        if (all & 1u) {
#pragma unroll
            for (int i = 0; i < RPW; ++i) own[4 * i * HX] = row_in(i) ? tile_key<MINMODE>(vals[i]) : 0u;
            if (tid < EDGES) *edge = ein ? tile_key<MINMODE>(eval) : 0u;
        } else {
#pragma unroll
            for (int i = 0; i < RPW; ++i) own[4 * i * HX] = row_in(i) ? (MINMODE ? kKeyTop - near[i] : near[i]) : 0u;
            if (tid < EDGES) *edge = ein ? (MINMODE ? kKeyTop - near_edge : near_edge) : 0u;
        }
        return all != 3u;
    }
}

template <bool MINMODE, int TY, int TZ, bool FULL, int SRC>
__device__ __forceinline__ bool stage_typed(const TileArgs& a, int x0, int y0, int z0, uint32_t* s_u,
                                            uint32_t* s_flag, bool& nan)
{
#define EG_STAGE(CODE, T) \
    case CODE: return stage_samples<T, MINMODE, TY, TZ, FULL>(a, x0, y0, z0, s_u, s_flag, nan);
    if constexpr (SRC == SRC_INT) {
        switch (a.dtype) {
            EG_STAGE(EG_I8, int8_t)
            EG_STAGE(EG_U8, uint8_t)
            EG_STAGE(EG_I16, int16_t)
            EG_STAGE(EG_U16, uint16_t)
        }
    } else {
        switch (a.dtype) {
            EG_STAGE(EG_F64, double)
            EG_STAGE(EG_I32, int32_t)
            EG_STAGE(EG_U32, uint32_t)
            EG_STAGE(EG_I64, int64_t)
            EG_STAGE(EG_U64, uint64_t)
        }
    }
#undef EG_STAGE
    return false;
}

// v_readlane_b32 with a uniform lane
extern "C" __device__ int eg_readlane(int src, int lane) __asm("llvm.amdgcn.readlane.i32");

// Words of a 3D tile's small LDS tables (s_tmp).
constexpr int kTile3Words = 8 + 2 * (48 + 8) + 48;

template <bool MINMODE, int TY, int TZ, bool FULL, bool PTR, int SRC>
__device__ __forceinline__ void tile3d_body(const TileArgs& a, int b, uint32_t* s_u, uint32_t* s_conn, uint32_t* s_tmp)
{
    constexpr int K = 14;
    constexpr int TX = 64;
    constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2;
    constexpr int HALO = HX * HY * HZ;
    constexpr int TILE = TX * TY * TZ;
    constexpr int YPT = TY / 4;
    constexpr int VPT = YPT * TZ;
    // only vertices on the tile's faces can step out of it
    constexpr int SURF = TILE - (TX - 2) * (TY - 2) * (TZ - 2);
    static_assert(TILE + SURF <= HALO, "the chains and the exit targets reuse the halo's LDS");
    static_assert(TY % 4 == 0, "four waves split the y rows");
    static_assert(((TY * TZ) & (TY * TZ - 1)) == 0, "row count is a power of two");
    const float* __restrict__ f = a.f;
    const int X = a.X, Y = a.Y, Z = a.Z;
    int32_t* __restrict__ lab = a.lab;
    int32_t* __restrict__ ptr = a.ptr;
    uint32_t* __restrict__ ctr = a.ctr;
    int32_t* s_nxt = reinterpret_cast<int32_t*>(s_u);
    // by code: packed successor and global offset (row c of the thread reads
    // kCodeRow entries before or after, see `code_of`)
    constexpr int kCodeRow = 4;
    uint32_t* s_succ = s_tmp + 8 + kCodeRow;  // [48] successors, then [48] offsets behind kCodes entries
    constexpr int kCodes = 48 + 2 * kCodeRow;
    // by visiting step (wide samples): the same and the halo index offset
    uint32_t* s_pack = s_tmp + 8 + 2 * kCodes;
    int32_t* s_gdel = reinterpret_cast<int32_t*>(s_pack + 16);
    int32_t* s_hoff = reinterpret_cast<int32_t*>(s_pack + 32);

    // the wave index is uniform: keep it (and every row quantity) scalar
    const int tid = threadIdx.x, lx = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tx = b % a.tiles_x;
    const int rr = b / a.tiles_x;
    const int ty = rr % a.tiles_y;
    const int tz = rr / a.tiles_y;
    const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
    const int SY = X;
    const int SZ = X * Y;
    // Code of a position: plane (below, own, above), row and column, each from
    // the lowest index up; reversed in the minimum graph, where the earlier of
    // two equal vertices is the higher one.
    if (tid < 48) {
        const int pos = MINMODE ? 47 - tid : tid;
        const int dz = (pos >> 4) - 1, dy = ((pos >> 2) & 3) - 1, dx = (pos & 3) - 1;
        const bool self = dz == 0 && dy == 0 && dx == 0;
        s_succ[tid] = self ? (uint32_t)(4 * TILE) << 6 : succ_pack<TY, HY, HX>(dz, dy, dx);
        s_succ[kCodes + tid] = (uint32_t)(dz * SZ + dy * SY + dx);
    }
    if constexpr (SRC == SRC_WIDE) {
        if (tid <= K) {
            // entry st: the candidate visited at step st (the vertex itself at K / 2)
            const int pos = MINMODE ? K - tid : tid;
            uint32_t pk = (uint32_t)(4 * TILE) << 6;
            int gd = 0, ho = 0;
            if (pos != K / 2) {
                const int j = pos < K / 2 ? pos : pos - 1;
                const int dz = (int)((Pack<3>::z >> (2 * j)) & 3u) - 1;
                const int dy = (int)((Pack<3>::y >> (2 * j)) & 3u) - 1;
                const int dx = (int)((Pack<3>::x >> (2 * j)) & 3u) - 1;
                pk = succ_pack<TY, HY, HX>(dz, dy, dx);
                gd = dz * SZ + dy * SY + dx;
                ho = (dz * HY + dy) * HX + dx;
            }
            s_pack[tid] = pk;
            s_gdel[tid] = gd;
            s_hoff[tid] = ho;
        }
    }

    bool nan = false;
    [[maybe_unused]] bool exact = true;  // equal keys are equal samples
    if constexpr (SRC != SRC_F32) {
        s_conn[tid] = c_conn3.w[tid];
        s_conn[tid + 256] = c_conn3.w[tid + 256];
        exact = stage_typed<MINMODE, TY, TZ, FULL, SRC>(a, x0, y0, z0, s_u, s_tmp, nan);
    } else {
        // every load of this thread is issued before the first one is used:
        // rows of 64 aligned values (one per lane) from a uniform row address,
        // then the two edge columns of every row (one value per thread);
        // positions outside the grid get the sentinel key 0
        constexpr int ROWS = HY * HZ;
        constexpr int RPW = (ROWS + 3) / 4;
        // every row index a wave takes exists when the rows split evenly
        // (all the tile shapes here): the test then folds away instead of
        // leaving a lane mask per row alive until the stores
        constexpr bool EVEN = ROWS % 4 == 0;
        constexpr int EDGES = 2 * ROWS;
        static_assert(EDGES <= 256, "one edge value per thread");
        static_assert(RPW <= 32, "row flags fit a word");
        const uint32_t* __restrict__ fb = reinterpret_cast<const uint32_t*>(f);
        const int gx = x0 + lx;
        const bool xin = gx < X;
        const int gxc = FULL ? gx : (xin ? gx : X - 1);  // lanes past the grid read a safe address
        const uint32_t lane_boff = 4u * (uint32_t)gxc;
        uint32_t vals[RPW];
        uint32_t rin_bits = 0;  // rows of this wave inside the grid (bit i)
        // a tile whose halo rows all lie in the grid (most of them) steps
        // through its rows by byte offsets from the halo's first row, four
        // rows at a time, on the scalar unit: no per-row division, clamp,
        // test or 64-bit address
        const bool interior = EVEN && y0 >= 1 && z0 >= 1 && y0 + TY < Y && z0 + TZ < Z &&
                              (int64_t)(TZ + 1) * SZ + (int64_t)(TY + 1) * SY + X < (int64_t(1) << 29);
        if (interior) {
            // a raw buffer at the halo's first row: the lane's byte offset in
            // a vector register, the row's in a scalar one (offsets stay
            // below 2^31 bytes, checked above, so the record limit 2^31 - 1
            // never clips a load); the last descriptor word selects 32-bit
            // data, as for any raw dword access on this architecture
            const uint32_t* org = fb + ((int64_t)(z0 - 1) * SZ + (int64_t)(y0 - 1) * SY);
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(org), (short)0, 0x7fffffff, 0x00020000);
            int hy = wv;
            uint32_t off = 4u * (uint32_t)(wv * SY);
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                vals[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, lane_boff, off, 0);
                const bool wrap = hy + 4 >= HY;
                off += wrap ? 4u * (uint32_t)(SZ + (4 - HY) * SY) : 4u * (uint32_t)(4 * SY);
                hy += wrap ? 4 - HY : 4;
            }
            rin_bits = RPW == 32 ? ~0u : (1u << RPW) - 1u;
        } else {
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                const int row = wv + 4 * i;
                const int hy = row % HY, hz = row / HY;
                const int gy = y0 + hy - 1, gz = z0 + hz - 1;
                rin_bits |= ((EVEN || row < ROWS) && (unsigned)gy < (unsigned)Y && (unsigned)gz < (unsigned)Z ? 1u : 0u)
                            << i;
                // rows outside the grid read a clamped row (their keys are
                // replaced below): the address needs no per-row condition
                const int gyc = min(max(gy, 0), Y - 1), gzc = min(max(gz, 0), Z - 1);
                const char* rowp = reinterpret_cast<const char*>(fb + ((int64_t)gzc * SZ + (int64_t)gyc * SY));
                vals[i] = *reinterpret_cast<const uint32_t*>(rowp + lane_boff);
            }
        }
        rin_bits = __builtin_amdgcn_readfirstlane(rin_bits);
        // edge value of this thread: row tid >> 1, left (x0 - 1) or right (x0 + 64)
        const int erow = tid >> 1;
        const int ehy = erow % HY, ehz = erow / HY;
        const int egx = (tid & 1) ? x0 + TX : x0 - 1;
        const int egy = y0 + ehy - 1, egz = z0 + ehz - 1;
        const bool ein = tid < EDGES && (unsigned)egx < (unsigned)X && (unsigned)egy < (unsigned)Y &&
                         (unsigned)egz < (unsigned)Z;
        const uint32_t eval = fb[ein ? egz * SZ + egy * SY + egx : 0];
        const uint32_t conn_a = c_conn3.w[tid], conn_b = c_conn3.w[tid + 256];
        s_conn[tid] = conn_a;
        s_conn[tid + 256] = conn_b;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int row = wv + 4 * i;
            const bool ok = ((rin_bits >> i) & 1u) && (FULL || xin);
            // one base address, the rows at immediate offsets from it
            if (EVEN || row < ROWS) (s_u + wv * HX + lx + 1)[4 * i * HX] = ok ? bits_key<MINMODE>(vals[i]) : 0u;
        }
        if (tid < EDGES) s_u[erow * HX + ((tid & 1) ? HX - 1 : 0)] = ein ? bits_key<MINMODE>(eval) : 0u;
    }
    __syncthreads();

    static_assert(VPT <= 32, "one mask word per lane");
    int nxt[VPT];
    uint64_t word = 0;  // this lane's parked mask word
    // x faces of the tile this lane's columns lie on (bit 0: lx = 0, bit 1:
    // lx = 63), by shifts rather than compares, so that no lane mask has to
    // stay alive across the unrolled loop
    const uint32_t bx = ((uint32_t)(lx - 1) >> 31) | (((uint32_t)(lx + 1) >> 6) << 1);
    const uint32_t lane_b = 4u * (uint32_t)lx;
    // wide samples: the vertices whose 32-bit keys leave the order open (bit k)
    [[maybe_unused]] uint32_t open = 0;
    [[maybe_unused]] const bool is32 = SRC == SRC_WIDE && sample_size((int)a.dtype) == 4;
    const int gx = x0 + lx;
    const int ly0 = wv * YPT;  // this thread's rows: ly0 .. ly0 + YPT - 1
    // window positions of a plane: row r = -1 .. YPT, column dx
    constexpr int NP = 3 * YPT + 4;
    constexpr auto at = [](int r, int dx) { return r < 0 ? dx + 1 : r < YPT ? 3 * r + 3 + dx : 3 * YPT + 2 + dx; };
    constexpr auto code_of = [](int r, int dx) -> uint32_t {
        const int c = 4 * (r + 1) + dx + 1;
        return 4u * (uint32_t)(MINMODE ? 15 - c : c);
    };
    constexpr uint32_t BELOW = MINMODE ? 128u : 0u, OWN = 64u, ABOVE = MINMODE ? 0u : 128u;  // 4 * 16 * plane
    uint32_t win[3][NP];
    auto load_plane = [&](uint32_t* w, int hz) {
        // one opaque address per plane, at position (-1, -1): the reads lie
        // within (YPT + 1) HX + 2 words of it and pair into ds_read2 without an
        // address of their own
        uint32_t boff = 4u * (uint32_t)((hz * HY + ly0) * HX) + lane_b;
        asm("" : "+v"(boff));
        const uint32_t* p = reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(s_u) + boff);
#pragma unroll
        for (int r = -1; r <= YPT; ++r)
#pragma unroll
            for (int dx = r == YPT ? 0 : -1; dx <= (r < 0 ? 0 : 1); ++dx) w[at(r, dx)] = p[(r + 1) * HX + dx + 1];
    };
    // a plane's lower and upper maxima of every row of the thread (rows r - 1
    // and r, columns -1 and 0; rows r and r + 1, columns 0 and 1), and both
    // together as candidates of the plane's own vertices
    auto maxima = [&](const uint32_t* w, uint64_t* lower, uint64_t* upper, uint64_t* own) {
        uint64_t lp[YPT + 1], up[YPT + 1];
        static_for<0, YPT + 2>([&](auto step) {
            constexpr int r = decltype(step)::value - 1;
            const uint64_t mid = coded<code_of(r, 0)>(w[at(r, 0)]);
            if constexpr (r < YPT) lp[r + 1] = later_max(coded<code_of(r, -1)>(w[at(r, -1)]), mid);
            if constexpr (r >= 0) up[r] = later_max(mid, coded<code_of(r, 1)>(w[at(r, 1)]));
        });
#pragma unroll
        for (int c = 0; c < YPT; ++c) {
            lower[c] = later_max(lp[c], lp[c + 1]);
            upper[c] = later_max(up[c], up[c + 1]);
            own[c] = later_max(lower[c], upper[c]) | OWN;
            upper[c] |= ABOVE;
        }
    };
    // low[c]: the lower maximum of the plane below; mid[c]: the maximum over
    // the planes below and own
    uint64_t low[YPT], mid[YPT];
    auto advance = [&](const uint64_t* lower, const uint64_t* own) {
#pragma unroll
        for (int c = 0; c < YPT; ++c) {
            mid[c] = later_max(low[c], own[c]);
            low[c] = lower[c] | BELOW;
        }
    };
    load_plane(win[0], 0);
    load_plane(win[1], 1);
    {
        uint64_t lower[YPT], upper[YPT], own[YPT];
        maxima(win[0], low, upper, own);
#pragma unroll
        for (int c = 0; c < YPT; ++c) low[c] |= BELOW;
        maxima(win[1], lower, upper, own);
        advance(lower, own);
    }
#pragma unroll
    for (int lz = 0; lz < TZ; ++lz) {
        load_plane(win[(lz + 2) % 3], lz + 2);
        uint64_t lower[YPT], upper[YPT], own[YPT];
        maxima(win[(lz + 2) % 3], lower, upper, own);
        // the steepest candidates first, so that only their codes live on (and
        // their keys, for wide samples)
        uint32_t code[YPT];
        [[maybe_unused]] uint32_t kbest[YPT];
#pragma unroll
        for (int c = 0; c < YPT; ++c) {
            const uint64_t best = later_max(mid[c], upper[c]);
            code[c] = (uint32_t)best;
            asm("" : "+v"(code[c]));
            if constexpr (SRC == SRC_WIDE) kbest[c] = (uint32_t)(best >> 31);
        }
        advance(lower, own);
        const int gz = z0 + lz;
#pragma unroll
        for (int c = 0; c < YPT; ++c) {
            const int ly = ly0 + c;
            const int gy = y0 + ly;
            const bool in = FULL || (gx < X && gy < Y && gz < Z);
            const uint32_t uv = win[(lz + 1) % 3][at(c, 0)];
            if constexpr (SRC == SRC_F32) nan |= in && nan_key(uv);
            // upper-link mask: row 13 first, so that row j ends in bit j; each
            // row's comparison is the carry of an add that doubles the mask
            uint32_t up = 0;
            static_for<0, K>([&](auto step) {
                constexpr int j = K - 1 - decltype(step)::value;
                using RJ = Row<3, j>;
                constexpr bool wins_tie = (j >= K / 2) != MINMODE;
                const uint32_t u = win[(lz + 1 + RJ::dz) % 3][at(c + RJ::dy, RJ::dx)];
                if constexpr (j == K - 1)
                    up = first_above<wins_tie>(u, uv);
                else
                    up = push_above<wins_tie>(up, u, uv);
            });
            const uint32_t slot = code[c] & 0xFCu;  // 4 * code
            if (SRC == SRC_WIDE && !exact) {
                // open: a neighbour meets the vertex, or two candidates lead;
                // 32-bit keys are exact but for the two clamped ends
                uint32_t meet = ~0u;
                int lead = uv == kbest[c];
                static_for<0, K>([&](auto step) {
                    using RJ = Row<3, decltype(step)::value>;
                    const uint32_t u = win[(lz + 1 + RJ::dz) % 3][at(c + RJ::dy, RJ::dx)];
                    meet = min(meet, u ^ uv);
                    lead += u == kbest[c];
                });
                auto clamped = [](uint32_t k) { return k - 2u > kKeyTop - 4u; };
                const bool tie = is32 ? clamped(uv) || clamped(kbest[c]) : meet == 0u || lead > 1;
                open |= (in && tie ? 1u : 0u) << (c * TZ + lz);
            }
            // every quantity below without a branch (the connectivity table
            // marks the empty link as no saddle, so a maximum needs no test of
            // its own)
            const bool is_max = in && up == 0;
            const bool is_sad = in && eg_ubfe(s_conn[up >> 5], up, 1u) == 0u;
            const uint32_t* entry = reinterpret_cast<const uint32_t*>(
                reinterpret_cast<const char*>(s_succ + (MINMODE ? kCodeRow * c : -kCodeRow * c)) + slot);
            uint32_t succ = entry[0], delta = entry[kCodes];
            // both words are wanted on every lane: without this the second is
            // read, and used, under a branch
            asm("" : "+v"(succ), "+v"(delta));
            const int row0 = gz * SZ + gy * SY + x0;  // uniform
            const int pv = row0 + lx + (int)delta;
            const int li4 = 4 * ((lz * TY + ly) * TX) + (int)lane_b;  // byte offset in the chain array
            // leaves the tile iff it steps across a face the vertex lies on
            const uint32_t faces = bx | (ly == 0 ? 4u : 0u) | (ly == TY - 1 ? 8u : 0u) | (lz == 0 ? 16u : 0u) |
                                   (lz == TZ - 1 ? 32u : 0u);
            int leave = -(pv + 1), stay = li4 + ((int)succ >> 6);
            int n = (faces & succ & 63u) ? leave : stay;
            if constexpr (!FULL) n = in ? n : 4 * TILE + li4;  // a vertex outside the grid ends its own chain
            if constexpr (PTR)
                if (in) store_row(ptr + row0, lane_b, pv);
            nxt[c * TZ + lz] = n;
            park_word(word, is_max, c * TZ + lz);
            park_word(word, is_sad, 32 + c * TZ + lz);
        }
    }
    if (SRC == SRC_WIDE && !exact) {
        // the open vertices again, on the samples themselves (the halo's keys
        // still say which neighbours exist): rare on measured data, every
        // vertex on plateaus
        for (int k = 0; k < VPT; ++k) {
            const uint64_t lanes = __ballot((open >> k) & 1u);
            if (lanes == 0) continue;
            const int lz = k % TZ, ly = ly0 + k / TZ;
            const int row0 = (z0 + lz) * SZ + (y0 + ly) * SY + x0;  // uniform
            bool is_max = false, is_sad = false;
            int n = 0;
            if ((open >> k) & 1u) {
                const int v = row0 + lx;
                const int cidx = ((lz + 1) * HY + ly + 1) * HX + lx + 1;
                const uint64_t ev = exact_key<MINMODE>(a.f, (int)a.dtype, v);
                uint32_t up = 0;
                uint64_t best = 0;
                int best_st = K / 2;
#pragma unroll 3
                for (int st = 0; st <= K; ++st) {
                    const bool exists = s_u[cidx + s_hoff[st]] != 0u;
                    const uint64_t e = exact_key<MINMODE>(a.f, (int)a.dtype, exists ? v + s_gdel[st] : v);
                    const bool lead = exists && e >= best;  // the later of two equal ones
                    best = lead ? e : best;
                    best_st = lead ? st : best_st;
                    if (st != K / 2) {
                        const int pos = MINMODE ? K - st : st;
                        const int j = pos < K / 2 ? pos : pos - 1;
                        const bool above = st > K / 2 ? e >= ev : e > ev;
                        up |= (exists && above ? 1u : 0u) << j;
                    }
                }
                is_max = up == 0;
                is_sad = eg_ubfe(s_conn[up >> 5], up, 1u) == 0u;
                const uint32_t p = s_pack[best_st];
                const int pv = v + s_gdel[best_st];
                const uint32_t faces = bx | (ly == 0 ? 4u : 0u) | (ly == TY - 1 ? 8u : 0u) | (lz == 0 ? 16u : 0u) |
                                       (lz == TZ - 1 ? 32u : 0u);
                n = (faces & p & 63u) ? -(pv + 1) : 4 * ((lz * TY + ly) * TX) + (int)lane_b + ((int)p >> 6);
                if constexpr (PTR) store_row(ptr + row0, lane_b, pv);
            }
#pragma unroll
            for (int i = 0; i < VPT; ++i) nxt[i] = i == k && ((lanes >> lx) & 1u) ? n : nxt[i];
            const uint64_t bm = __ballot(is_max), bs = __ballot(is_sad);
            auto patch = [&](uint64_t bits, int lane) {
                const uint64_t old = (uint64_t)(uint32_t)eg_readlane((int)(uint32_t)word, lane) |
                                     (uint64_t)(uint32_t)eg_readlane((int)(uint32_t)(word >> 32), lane) << 32;
                const uint64_t b = (old & ~lanes) | bits;
                const uint32_t lo = (uint32_t)eg_writelane((int)(uint32_t)b, lane, (int)(uint32_t)word);
                const uint32_t hi = (uint32_t)eg_writelane((int)(uint32_t)(b >> 32), lane, (int)(uint32_t)(word >> 32));
                word = ((uint64_t)hi << 32) | lo;
            };
            patch(bm, k);
            patch(bs, 32 + k);
        }
    }
    {
        const int k = __lane_id() & 31;
        const int ly = ly0 + k / TZ, lz = k % TZ;
        store_words(a, word, VPT, (z0 + lz) * Y + y0 + ly, y0 + ly < Y && z0 + lz < Z, tx);
    }
    if (__ballot(nan) != 0 && __lane_id() == 0) atomicOr(&ctr[C_NAN], 1u);
    // exit targets go behind the chains, in LDS the halo no longer needs
    uint32_t claim;
    const uint32_t region = (a.first + blockIdx.x) & (a.regions - 1u);
    uint32_t* counter = a.claims + kRegionStride * region;
    const uint32_t nexit = rank_exits<VPT>(nxt, s_tmp, s_u + TILE, counter, claim);
#pragma unroll
    for (int c = 0; c < YPT; ++c)
#pragma unroll
        for (int lz = 0; lz < TZ; ++lz) s_nxt[(lz * TY + ly0 + c) * TX + lx] = nxt[c * TZ + lz];
    __syncthreads();
    // global offset of every tile row (lz, ly) from the tile's first vertex,
    // so that a tile index becomes a vertex id with one LDS read instead of
    // two quarter-rate multiplies; then every chain inside the tile is
    // followed to its end (double_tile_chains names the three kinds of entry)
    __shared__ int s_rowoff[TY * TZ];
    if (tid < TY * TZ) s_rowoff[tid] = (tid / TY) * SZ + (tid % TY) * SY;
    double_tile_chains<VPT, TILE, 4>(nxt, s_nxt,
                                     [&](int k) { return ((k % TZ) * TY + ly0 + k / TZ) * TX + lx; });
    uint32_t base;
    const bool fit = place_exits(nexit, claim, s_u + TILE, s_tmp, a, region, base);
    const int xoff = exit_offset<VPT>(nxt, fit, base, s_u + TILE, X * Y * Z);
    const int tile0 = z0 * SZ + y0 * SY + x0;
#pragma unroll
    for (int c = 0; c < YPT; ++c) {
        const int ly = ly0 + c;
        const int gy = y0 + ly;
#pragma unroll
        for (int lz = 0; lz < TZ; ++lz) {
            const int gz = z0 + lz;
            const int n = nxt[c * TZ + lz];
            // the row offset is read for every vertex (masked into range), so
            // that the label is a select rather than a branch
            const int ro = s_rowoff[((uint32_t)(n - 4 * TILE) >> 8) & (TY * TZ - 1)];
            if (FULL || (gx < X && gy < Y && gz < Z))
                store_row(lab + (gz * SZ + gy * SY + x0), lane_b, n >= 0 ? tile0 + ro + ((n >> 2) & 63) : n - xoff);
        }
    }
}

// LDS of a 3D tile's workgroup: the small tables first, where the reads' 8-bit
// offsets reach them from address 0.
template <int TY, int TZ>
struct Tile3Lds {
    uint32_t tmp[kTile3Words];
    uint32_t conn[512];
    uint32_t u[66 * (TY + 2) * (TZ + 2)];
};

// Full tiles (every vertex in the grid, the common case) run a variant without
// per-vertex bounds tests; whether pointers are written is a compile-time
// choice too, which keeps the output address out of the unrolled loop.
template <bool MINMODE, int TY, int TZ, bool PTR, int SRC>
__device__ __forceinline__ void tile3d(const TileArgs& a, int b, Tile3Lds<TY, TZ>& s)
{
    const int tx = b % a.tiles_x;
    const int rr = b / a.tiles_x;
    const int ty = rr % a.tiles_y;
    const int tz = rr / a.tiles_y;
    const bool full = (tx + 1) * 64 <= a.X && (ty + 1) * TY <= a.Y && (tz + 1) * TZ <= a.Z;
    if (full)
        tile3d_body<MINMODE, TY, TZ, true, PTR, SRC>(a, b, s.u, s.conn, s.tmp);
    else
        tile3d_body<MINMODE, TY, TZ, false, PTR, SRC>(a, b, s.u, s.conn, s.tmp);
}

}  // namespace eg
