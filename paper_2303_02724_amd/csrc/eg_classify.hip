// eg_classify.hip -- per-vertex classification, labels and saddle reps.
//
// k_classify_slab  stages (a) and (c) of the method for n = 4, 5 and 6: one
//   thread per vertex reads its closed neighbourhood from planes of keys staged
//   in LDS, forms the upper-link mask (Sec. 3.3), the steepest-ascent pointer
//   (highest upper-link vertex, Sec. 3.3) and decides maximum (empty upper link)
//   / saddle (>= 2 components, Table 1) by set algebra on the link's rows
//   (eg_link.h).
// k_classify1d  the same for n = 1, whose link is two vertices.
// k_exit_*, k_final*  stage (b): pointer jumping until every vertex names its
//   maximum (the end of the walk of Alg. 2).
#include "eg_internal.h"
#include "eg_rows.h"
#include "eg_link.h"

namespace eg {

// Counters and header.
__global__ __launch_bounds__(256) void k_init(uint32_t* __restrict__ ctr, uint32_t* __restrict__ claims,
                                              int32_t* __restrict__ header)
{
    const int i = threadIdx.x;
    if (i < C_SLOTS) ctr[i] = 0;
    if (i < kRegions) claims[kRegionStride * i] = 0;
    if (header && i < EG_H_SLOTS) header[i] = 0;
}

hipError_t launch_init(const Work& w, int32_t* header, hipStream_t s)
{
    hipLaunchKernelGGL(k_init, dim3(1), dim3(256), 0, s, w.ctr, w.claims, header);
    return hipGetLastError();
}

// Order keys of every vertex (reversed for the minimum graph), once, for the
// grids whose classification reads neighbours from memory; NaN is flagged.
template <bool MINMODE>
__global__ __launch_bounds__(256) void k_keys(const float* __restrict__ f, int N, uint32_t* __restrict__ keys,
                                              uint32_t* __restrict__ ctr)
{
    bool nan = false;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
        const float x = f[i];
        nan |= x != x;
        keys[i] = mode_key<MINMODE>(x);
    }
    if (__ballot(nan) != 0 && __lane_id() == 0) atomicOr(&ctr[C_NAN], 1u);
}

// 1D: the neighbours are the vertices before and after (key 0, below every
// vertex, past the ends).  Of two equal vertices the later is the higher one, the
// earlier in the minimum graph; a vertex below both neighbours is a saddle.  The
// vertices of a wave are one word of the masks.
template <bool MINMODE>
__global__ __launch_bounds__(256) void k_classify1d(const uint32_t* __restrict__ keys, int32_t N,
                                                    int32_t* __restrict__ lab, int32_t* __restrict__ ptr,
                                                    uint64_t* __restrict__ mmask, uint64_t* __restrict__ smask)
{
    const uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = v < (uint32_t)N;
    bool before = false, after = false;  // above v
    if (in) {
        const uint32_t u = keys[v];
        const uint32_t b = v > 0 ? keys[v - 1] : 0u, a = v + 1 < (uint32_t)N ? keys[v + 1] : 0u;
        before = MINMODE ? b >= u : b > u;
        after = MINMODE ? a > u : a >= u;
        const bool to_after = after && (!before || (MINMODE ? a > b : a >= b));
        const int best = (int)v + (to_after ? 1 : before ? -1 : 0);
        lab[v] = before || after ? -(best + 1) : best;  // "same as best", or final
        if (ptr) ptr[v] = best;
    }
    const uint64_t maxima = __ballot(in && !before && !after), saddles = __ballot(before && after);
    if (in && __lane_id() == 0) {
        mmask[v >> 6] = maxima;
        smask[v >> 6] = saddles;
    }
}

// -------------------------------------------------------- 4D-6D slab tiles
//
// k_classify_slab  pointers, maxima and saddles for n = 4, 5 and 6, with the
//   neighbourhood read from LDS instead of through the caches (62
//   gathers per vertex in 5D, 126 in 6D, leave a kernel that reads them from
//   memory bound by the memory pipeline, not by arithmetic).  A block owns a
//   tile of the hyperplanes orthogonal to axis 0 (4x8x8 vertices in 4D,
//   2x4x4x8 in 5D, 2x2x2x4x8 in 6D, one per thread: short rows lose less on
//   ragged axes, have less halo and fill a byte of the masks, stored without
//   atomics) and a run of zc consecutive planes along axis 0.  Rows of 32 (and
//   atomics on the masks) against rows of 8: 41 x 64 x 60 x 65 186 and 125 us,
//   30 x 31 x 29 x 30 x 33 1380 and 616; in 6D rows of 16 left two waves per
//   SIMD to the LDS instead of three: 16^6 598 and 497.  Blocks of 512 threads
//   were slower everywhere (more waves to a barrier).  Where the axes between
//   the first and the last are so short that most of such a tile lies outside
//   the grid, the tile is wide: 2x4x32, 2x2x2x32 or 2x2x2x2x16 (classification
//   of noise, rows of 8 and wide: 2 x 2 x 2 x 10^6 464 and 145 us, 200 x 200 x 1
//   x 200 495 and 219, 2 x 2 x 2 x 2 x 300 000 224 and 97, 2 x 2 x 2 x 2 x 2 x
//   100 000 227 and 168).  A block keeps three consecutive planes of the tile plus
//   a one-vertex halo in a ring in LDS (positions outside the grid hold key 0,
//   below every vertex, so every row of the table may be read), and slides it
//   along axis 0: while one plane is classified, the loads of the plane after
//   next are in flight.
template <int NDIM, bool WIDE>
__host__ __device__ constexpr int slab_e(int i)  // interior extent along axis i (1..n-1)
{
    if (WIDE) return i == NDIM - 1 ? (NDIM == 6 ? 16 : 32) : NDIM == 4 && i == 2 ? 4 : 2;
    if (i == NDIM - 1) return 8;
    if (NDIM == 4) return i == 2 ? 8 : 4;
    if (NDIM == 5) return i == 1 ? 2 : 4;
    return i == 4 ? 4 : 2;
}
template <int NDIM, bool WIDE>
__host__ __device__ constexpr int slab_hs(int i)  // LDS stride of axis i in a halo plane
{
    int s = 1;
    for (int k = NDIM - 1; k > i; --k) s *= slab_e<NDIM, WIDE>(k) + 2;
    return s;
}
template <int NDIM, bool WIDE>
__host__ __device__ constexpr int slab_size()  // keys per halo plane
{
    return slab_hs<NDIM, WIDE>(0);
}
template <int NDIM, bool WIDE>
__host__ __device__ constexpr int slab_inner()  // vertices per tile plane
{
    int s = 1;
    for (int k = 1; k < NDIM; ++k) s *= slab_e<NDIM, WIDE>(k);
    return s;
}
template <int NDIM, bool WIDE>
int64_t slab_tiles(const Grid& g, int32_t* nt)
{
    int64_t n = 1;
    for (int i = 1; i < NDIM; ++i) {
        nt[i] = (int32_t)((int64_t(g.dims[i]) + slab_e<NDIM, WIDE>(i) - 1) / slab_e<NDIM, WIDE>(i));
        n *= nt[i];
    }
    return n;
}

// A row of the tile is one piece of its mask word.
template <int EX>
struct MaskPiece {
    using type = uint8_t;
};
template <>
struct MaskPiece<16> {
    using type = uint16_t;
};
template <>
struct MaskPiece<32> {
    using type = uint32_t;
};

// The steepest row is found by groups: the rows (and the vertex itself) that
// share their offsets along the first axes differ by {0,1}^Q along the last Q,
// so a group is a corner and 2^Q fixed offsets from it.  Each group's maximum
// is formed as its keys are compared for the mask; the last group that holds
// the highest key is picked, and only its keys are looked at again, from LDS
// (5D: 87 instructions where comparing all 62 rows with the maximum took 159).
// Groups and positions are numbered in linear-index order.
template <int NDIM, bool WIDE>
struct Groups {
    static constexpr int Q = NDIM == 6 ? 3 : 2;
    static constexpr int IN = 1 << Q;            // rows per group
    static constexpr int G = 1 << (NDIM - Q);    // groups per half
    static constexpr int H = (1 << NDIM) - 1;    // rows per half
    static constexpr int of_row(int j)
    {
        return j >= H ? G + ((j - H + 1) >> Q) : G - 1 - ((H - j) >> Q);
    }
    // offset (-1, 0, 1) along axis i of position k of group g
    static __host__ __device__ constexpr int offset(int g, int k, int i)
    {
        const int high = g >= G ? g - G : G - 1 - g;
        const int bit = i < NDIM - Q ? (high >> (NDIM - Q - 1 - i)) & 1 : (k >> (NDIM - 1 - i)) & 1;
        return g >= G ? bit : i < NDIM - Q ? -bit : bit - 1;
    }
    // LDS offset of position k from the group's corner (position 0)
    static constexpr int inner(int k)
    {
        int d = 0;
        for (int i = NDIM - Q; i < NDIM; ++i) d += ((k >> (NDIM - 1 - i)) & 1) * slab_hs<NDIM, WIDE>(i);
        return d;
    }
};

struct SlabArgs {
    int32_t first;               // number of the launch's first block
    int32_t zc;                  // planes along axis 0 per block
    int32_t zblocks;             // blocks along axis 0: ceil(dims[0] / zc)
    int32_t nt[EG_MAX_NDIM];     // tiles along axes 1..n-1
    int32_t st[EG_MAX_NDIM];     // grid strides (st[n-1] = 1)
    int32_t rows_per_plane;      // rows of X vertices in one plane (st[0] / X)
};

template <int NDIM, bool MINMODE, bool WIDE>
__global__ __launch_bounds__(256) void k_classify_slab(const uint32_t* __restrict__ keys, Grid g,
                                                       SlabArgs a, int32_t* __restrict__ lab,
                                                       int32_t* __restrict__ ptr, uint64_t* __restrict__ mmask,
                                                       uint64_t* __restrict__ smask)
{
    constexpr int K = Rows<NDIM>::K;
    constexpr Rows<NDIM> R = make_rows_ce<NDIM>();
    constexpr int S = slab_size<NDIM, WIDE>();
    constexpr int PER = (S + 255) / 256;
    constexpr int EX = slab_e<NDIM, WIDE>(NDIM - 1);
    static_assert(slab_inner<NDIM, WIDE>() == 256, "one interior vertex per thread");
    static_assert(EX == 8 || EX == 16 || EX == 32, "a row of the tile is a piece of its mask word");
    using Piece = typename MaskPiece<EX>::type;
    // halo index of interior position (0,..,0), the smallest a row may reach
    constexpr int B = [] {
        int b = 0;
        for (int i = 1; i < NDIM; ++i) b += slab_hs<NDIM, WIDE>(i);
        return b;
    }();
    __shared__ uint32_t s_ring[3 * S];
    using GR = Groups<NDIM, WIDE>;
    static_assert(2 * GR::G * GR::IN <= 256 && 6 * GR::G <= 256, "the tables are filled in one step");
    __shared__ int32_t s_lin[2 * GR::G * GR::IN];  // linear offset of every position
    __shared__ int32_t s_corner[3][2 * GR::G];     // a group's corner in the ring, by the slot of plane z-1
    const int tid = threadIdx.x;
    if (tid < 2 * GR::G * GR::IN) {
        int lin = 0;
#pragma unroll
        for (int i = 0; i < NDIM; ++i) lin += GR::offset(tid / GR::IN, tid % GR::IN, i) * a.st[i];
        s_lin[tid] = lin;
    }
    if (tid < 6 * GR::G) {
        const int below = tid / (2 * GR::G), grp = tid % (2 * GR::G);
        int d = B;
#pragma unroll
        for (int i = 1; i < NDIM; ++i) d += GR::offset(grp, 0, i) * slab_hs<NDIM, WIDE>(i);
        s_corner[below][grp] = (below + 1 + GR::offset(grp, 0, 0)) % 3 * S + d;
    }

    int rest = a.first + (int)blockIdx.x;
    const int zb = rest % a.zblocks;
    rest /= a.zblocks;
    int t0[NDIM];  // first coordinate of the tile along axes 1..n-1
#pragma unroll
    for (int i = NDIM - 1; i >= 1; --i) {
        const int q = rest % a.nt[i];
        rest /= a.nt[i];
        t0[i] = q * slab_e<NDIM, WIDE>(i);
    }
    const int z0 = zb * a.zc;
    const int z1 = min(z0 + a.zc, g.dims[0]);

    // the halo positions this thread loads: offset inside a plane of the
    // grid, or -1 outside the grid.  Planes below 2^29 vertices are read
    // through a raw buffer of exactly one plane, whose loads return 0 (the key
    // of positions outside the grid) past its end: a position outside has an
    // offset there, a plane outside the grid a buffer of no bytes.  So a load
    // takes no instruction beside itself, and nothing waits for it before the
    // plane is stored.
    const bool small = a.st[0] < (1 << 29);
    int goff[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        int h = tid + 256 * k;
        bool in = h < S;
        int off = 0;
#pragma unroll
        for (int i = NDIM - 1; i >= 1; --i) {
            const int he = slab_e<NDIM, WIDE>(i) + 2;
            const int c = t0[i] + h % he - 1;
            h /= he;
            in &= (c >= 0) & (c < g.dims[i]);
            off += c * a.st[i];
        }
        goff[k] = !in ? (small ? 0x7fffffff : -1) : small ? 4 * off : off;
    }
    // this thread's interior vertex: its halo index minus B, and its offset
    // inside a plane of the grid
    int center = 0, vin = 0;
    bool mine = true;
    {
        int r = tid;
#pragma unroll
        for (int i = NDIM - 1; i >= 1; --i) {
            const int e = r % slab_e<NDIM, WIDE>(i);
            r /= slab_e<NDIM, WIDE>(i);
            const int c = t0[i] + e;
            mine &= c < g.dims[i];
            center += e * slab_hs<NDIM, WIDE>(i);
            vin += c * a.st[i];
        }
    }
    const int X = g.dims[NDIM - 1];
    const int x = t0[NDIM - 1] + tid % EX;
    const int rin = mine ? (vin - x) / X : 0;  // row of the vertex inside its plane
    const int XW = (X + 63) >> 6;

    uint32_t r[PER];
    auto fetch = [&](int z) {
        const bool zok = z >= 0 && z < g.dims[0];
        const int zoff = zok ? z * a.st[0] : 0;
        if (small) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint32_t*>(keys + zoff), (short)0, zok ? 4 * a.st[0] : 0, 0x00020000);
#pragma unroll
            for (int k = 0; k < PER; ++k) r[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, goff[k], 0, 0);
            return;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const bool ok = zok && goff[k] >= 0;
            const uint32_t u = keys[ok ? zoff + goff[k] : 0];
            r[k] = ok ? u : 0u;
        }
    };
    auto put = [&](int slot) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (tid + 256 * k < S) s_ring[slot * S + tid + 256 * k] = r[k];
    };
    fetch(z0 - 1);
    put(0);
    fetch(z0);
    put(1);
    fetch(z0 + 1);
    int sp = 0;  // slot of plane z-1; plane z is in the next slot, z+1 in the one after
    for (int z = z0; z < z1; ++z) {
        const int s1 = sp == 2 ? 0 : sp + 1;
        const int s2 = s1 == 2 ? 0 : s1 + 1;
        __syncthreads();  // slot s2 (plane z-2) is no longer read
        put(s2);
        __syncthreads();
        if (z + 1 < z1) fetch(z + 2);  // in flight during this plane

        const int v = z * a.st[0] + vin;
        bool is_max = false, is_sad = false;
        if (mine) {
            const uint32_t* p0 = s_ring + sp * S + center;
            const uint32_t* p1 = s_ring + s1 * S + center;
            const uint32_t* p2 = s_ring + s2 * S + center;
            const uint32_t uv = p1[B];
            auto key = [&](int j) {
                int d = B;
#pragma unroll
                for (int i = 1; i < NDIM; ++i) d += R.d[j][i] * slab_hs<NDIM, WIDE>(i);
                const uint32_t* p = R.d[j][0] < 0 ? p0 : R.d[j][0] > 0 ? p2 : p1;
                return p[d];
            };
            // the upper-link mask, and the highest key of every group (rows
            // outside the grid hold key 0 < uv)
            // 32 rows per word, pushed from the highest row down so that row
            // j ends in bit j % 32 of word j / 32 (two instructions a row)
            constexpr int NW = (K + 31) / 32;
            uint32_t wd[NW];
            uint32_t gm[2 * GR::G];
#pragma unroll
            for (int i = 0; i < 2 * GR::G; ++i) gm[i] = i == GR::G || i == GR::G - 1 ? uv : 0u;
            static_for<0, K>([&](auto step) {
                constexpr int j = K - 1 - decltype(step)::value;
                constexpr bool wins = (j >= K / 2) != MINMODE;
                const uint32_t u = key(j);
                if constexpr (j == K - 1 || j % 32 == 31)
                    wd[j / 32] = first_above<wins>(u, uv);
                else
                    wd[j / 32] = push_above<wins>(wd[j / 32], u, uv);
                gm[GR::of_row(j)] = max(gm[GR::of_row(j)], u);
            });
            Mask<NDIM> up = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) up |= Mask<NDIM>(wd[w]) << (32 * w);
            // the steepest target: the last position holding the highest key,
            // the first in the minimum graph
            uint32_t top = gm[0];
#pragma unroll
            for (int i = 1; i < 2 * GR::G; ++i) top = max(top, gm[i]);
            int grp = 0, pos = 0;
#pragma unroll
            for (int i = 0; i < 2 * GR::G; ++i) {
                const int k = MINMODE ? 2 * GR::G - 1 - i : i;
                grp = gm[k] == top ? k : grp;
            }
            const uint32_t* corner = s_ring + s_corner[sp][grp] + center;
#pragma unroll
            for (int i = 0; i < GR::IN; ++i) {
                const int k = MINMODE ? GR::IN - 1 - i : i;
                pos = corner[GR::inner(k)] == top ? k : pos;
            }
            is_max = up == 0;
            if (!is_max) is_sad = !link_connected<NDIM>(up);
            const int best = v + s_lin[grp * GR::IN + pos];
            lab[v] = is_max ? v : -(best + 1);
            if (ptr) ptr[v] = best;
        }
        // every row of the tile is one piece of each mask's word, stored by its
        // first lane; the last tile of a row also clears what is left of the
        // row's last word (in one store when it opens the word)
        const uint64_t bm = __ballot(is_max), bs = __ballot(is_sad);
        if (mine && tid % EX == 0) {
            const int64_t row = (int64_t)(z * a.rows_per_plane + rin) * XW;
            const Piece m = (Piece)(bm >> __lane_id()), sd = (Piece)(bs >> __lane_id());
            constexpr int PW = 64 / EX;  // pieces of a word
            const int h = x / EX;
            const bool last = x + EX >= X;
            if (last && h % PW == 0) {
                mmask[row + h / PW] = m;
                smask[row + h / PW] = sd;
            } else {
                Piece* mp = reinterpret_cast<Piece*>(mmask + row);
                Piece* sdp = reinterpret_cast<Piece*>(smask + row);
                mp[h] = m;
                sdp[h] = sd;
                if (last)
                    for (int k = h + 1; k < PW * XW; ++k) mp[k] = sdp[k] = 0;
            }
        }
        sp = s1;
    }
}

constexpr int64_t kSlabBlocks = int64_t(1) << 23;  // most blocks of one launch

template <int NDIM, bool MINMODE, bool WIDE>
static void launch_slab(const Grid& g, int32_t* lab, int32_t* ptr, const Work& w, hipStream_t s)
{
    SlabArgs a{};
    a.st[NDIM - 1] = 1;
    for (int i = NDIM - 2; i >= 0; --i) a.st[i] = a.st[i + 1] * g.dims[i + 1];
    const int64_t tiles = slab_tiles<NDIM, WIDE>(g, a.nt);
    // about 8192 blocks, each over as many planes as that allows
    const int64_t D0 = g.dims[0];
    const int64_t zc = std::min<int64_t>(D0, std::max<int64_t>(1, (D0 * tiles + 8191) / 8192));
    a.zc = (int)zc;
    a.zblocks = (int)((D0 + zc - 1) / zc);
    a.rows_per_plane = a.st[0] / g.dims[NDIM - 1];
    const int64_t blocks = tiles * a.zblocks;  // fewer than 2^31: every tile holds a vertex
    // a launch holds fewer than 2^32 threads; where the axes between the first
    // and the last are short, most of a tile's threads have no vertex (8 X
    // threads for X vertices in a row along the last axis of a 4D grid)
    for (int64_t done = 0; done < blocks; done += kSlabBlocks) {
        a.first = (int)done;
        const int64_t n = std::min<int64_t>(blocks - done, kSlabBlocks);
        hipLaunchKernelGGL((k_classify_slab<NDIM, MINMODE, WIDE>), dim3((unsigned)n), dim3(256), 0, s, w.keys, g, a,
                           lab, ptr, w.mmask, w.smask);
    }
}

template <int NDIM, bool MINMODE>
static void launch_classify_t(const float* f, const Grid& g, int32_t* lab, int32_t* ptr, const Work& w,
                              hipStream_t s)
{
    const int64_t kwant = ((int64_t)g.N + 255) / 256;
    const int kblocks = (int)(kwant < 8192 ? kwant : 8192);
    hipLaunchKernelGGL(k_keys<MINMODE>, dim3(kblocks), dim3(256), 0, s, f, g.N, w.keys, w.ctr);
    if constexpr (NDIM >= 4) {
        // a wide tile takes about one and a half times as long as one with rows
        // of 8 (6D; between 0.8 and 1.7 times in 4D and 5D), so it is taken for
        // two thirds of the tiles or fewer
        int32_t nt[EG_MAX_NDIM];
        const int64_t narrow = slab_tiles<NDIM, false>(g, nt), wide = slab_tiles<NDIM, true>(g, nt);
        if (3 * wide <= 2 * narrow)
            launch_slab<NDIM, MINMODE, true>(g, lab, ptr, w, s);
        else
            launch_slab<NDIM, MINMODE, false>(g, lab, ptr, w, s);
    } else {
        const int blocks = (int)(((int64_t)g.N + 255) / 256);
        hipLaunchKernelGGL(k_classify1d<MINMODE>, dim3(blocks), dim3(256), 0, s, w.keys, g.N, lab, ptr, w.mmask,
                           w.smask);
    }
}

hipError_t launch_classify(const float* f, const Grid& g, bool minima, int32_t* lab, int32_t* ptr, const Work& w,
                           const Tuning& tu, hipStream_t s)
{
    if (g.ndim == 2 || g.ndim == 3) return launch_classify_tiled(f, g, minima, lab, ptr, w, tu, s);
#define EG_CASE(N)                                             \
    case N:                                                    \
        if (minima)                                            \
            launch_classify_t<N, true>(f, g, lab, ptr, w, s);  \
        else                                                   \
            launch_classify_t<N, false>(f, g, lab, ptr, w, s); \
        break;
    switch (g.ndim) {
        EG_CASE(1)
        EG_CASE(4)
        EG_CASE(5)
        EG_CASE(6)
        default:
            return hipErrorInvalidValue;
    }
#undef EG_CASE
    return hipGetLastError();
}

// ------------------------------------------------------------------ labels

// Stage (b): labels.  After classification every vertex holds a final label
// (its maximum) or a code for a later vertex of its steepest-ascent path: a
// vertex id, or an entry of the exit list (the distinct vertices where paths
// leave a tile, published once per tile).  The pass resolves the short exit
// list first, by pointer jumping, and then every vertex with one look-up;
// vertex-id codes (grids without tiling, or a full exit list) are resolved by
// pointer jumping over the label array itself.
//
// Entries are updated in place while other threads read them.  Every value
// ever stored says something true about the same path, so any value read is
// usable.  A sweep follows at most `hops` links per entry and stores how far
// it came; a wave with an entry left over sweeps again, now through links that
// the other waves have advanced too (each sweep multiplies the reach as long as
// all waves keep pace), so no launch has to follow for paths longer than one
// sweep.  No wave waits for another: one that ran alone would still walk its
// paths to their ends, at least `hops` links a sweep, which bounds its sweeps
// (sweeps_for).  Later sweeps read the links at device scope: a plain load
// could return the same old line of a cache every time.
//
// A path through the entries of waves that do not keep pace is walked there
// link by link.  With eight waves a SIMD the hardware serves the oldest first,
// and the youngest, whose entries lay side by side, made two sweeps while the
// others made 150: 57.6 ms for the labels of a 1D slope of 2^24 vertices, 24.7 in
// 4D (2 x 2 x 2 x 2^20), 13.9 for 2 x 2 x 2^25.  So where paths can be that long
// there are four waves a SIMD, which advance together, and their quads are dealt
// out in the bit-reversed order of the waves' numbers (spread), so that the
// entries of older waves lie next to those of any that lag.  They now take 3.0,
// 1.3 and 1.5 ms, in five sweeps (3.2, 1.3 and 1.9 with a launch for every sweep;
// at 2^23 vertices in 1D 1.8 against 1.6); the waves' number alone 4.0 ms in 1D,
// the order alone 3.6.  Storing at device scope too made no difference.

constexpr int kEvenBlocks = 1024;  // four waves a SIMD

// Blocks over n entries, four a thread: a multiple of the XCDs (and of the exit
// list's regions); a power of two where the waves' quads are spread.
static int all_blocks(int64_t n)
{
    const int64_t want = (n / 4 + 255) / 256;
    return (int)(want < 2048 ? (want / 8 + 1) * 8 : 2048);
}
static int even_blocks(int64_t n)
{
    int blocks = 8;
    while (blocks < kEvenBlocks && blocks * int64_t(1024) < n) blocks *= 2;
    return blocks;
}

// The exit list's base and its regions are 16-byte aligned (the workspace is
// carved in 256-byte steps, regions hold a multiple of four entries).
__global__ __launch_bounds__(256) void k_exit_init(TileArgs a, int32_t* __restrict__ res)
{
    exit_first(exit_part(a.claims, a.cap_region, a.regions, blockIdx.x, gridDim.x), a.exits, res, a.lab);
}

// Entries left over after `sweeps` sweeps raise ctr[flag_slot].
__global__ __launch_bounds__(256) void k_exit_jump(TileArgs a, int32_t* res, int N, int hops, int sweeps, bool even,
                                                   int flag_slot)
{
    ExitPart p = exit_part(a.claims, a.cap_region, a.regions, blockIdx.x, gridDim.x);
    if (even) p.t = spread(p.t >> 6, p.stride >> 6) * 64u + (threadIdx.x & 63u);
    const int32_t* lab = a.lab;
    int32_t* part = res + p.at;
    bool open = sweep(part, p.n, lab, res, N, hops, p.t, p.stride, false);
    for (int k = 1; __ballot(open) != 0 && k < sweeps; ++k)
        open = sweep(part, p.n, lab, res, N, hops, p.t, p.stride, true);
    if (__ballot(open) != 0 && __lane_id() == 0) atomicOr(&a.ctr[flag_slot], 1u);
}

// Capped exit lists: labels that the tile-ordered pass left open, by sweeps over
// all of them (labels of a 2 x 2^20 slope with a list of two entries 0.47 ms; 1.95
// when every vertex walked to the end of its path).  A short list may itself
// lead through tiles whose codes only these sweeps advance, so its own stop
// early (kCappedSweeps) and leave such entries as they are.
__global__ __launch_bounds__(256) void k_codes_rest(int32_t* lab, const int32_t* res, int32_t N,
                                                    uint32_t* __restrict__ ctr, int hops, int sweeps)
{
    if (ctr[C_CODES] == 0) return;
    codes_rest(lab, res, N, hops, sweeps, blockIdx.x, gridDim.x, ctr, &ctr[C_OPEN]);
}

// Per-vertex labels of the grids without tiles: every code names a vertex.
// Each XCD resolves a run of consecutive vertices, so that the links of
// neighbouring vertices, which stay close, meet in its L2.
struct LabelRun {
    int32_t* lab;
    uint32_t n, t, stride;
};
__device__ __forceinline__ LabelRun label_run(int32_t* lab, int32_t N, bool even)
{
    // runs of whole quads; the last run ends with the vertices left over
    const uint32_t x = blockIdx.x & 7u, q = (uint32_t)N >> 5, lo = 4u * q * x;
    // waves of the run (four a block), and this one's number
    const uint32_t n = gridDim.x >> 1, w = (blockIdx.x >> 3) * 4u + (threadIdx.x >> 6);
    return LabelRun{lab + lo, x == 7u ? (uint32_t)N - lo : 4u * q, (even ? spread(w, n) : w) * 64u + (threadIdx.x & 63u),
                    n * 64u};
}

// The first pass follows four links, so that no wave waits for the longest of
// its 256 paths; the second starts from entries that are all that much further
// on (4D labels 114 -> 72 us; three or six links are as good, and 5D and 6D,
// whose paths are short or bound by their bytes, stay as they were).  Both give
// a workgroup the same entries, so it leaves itself a note whether any are
// open: a flag for all of them, set by an atomic or a store of every wave, cost
// 90 to 290 us at one address.
constexpr int kFirstHops = 4;
__global__ __launch_bounds__(256) void k_final(int32_t* lab, int32_t N, uint32_t* __restrict__ ctr,
                                               uint32_t* __restrict__ open_flags, bool even)
{
    const LabelRun r = label_run(lab, N, even);
    const int open = __syncthreads_or(sweep(r.lab, r.n, lab, lab, N, kFirstHops, r.t, r.stride, false));
    if (threadIdx.x == 0) open_flags[blockIdx.x] = open != 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) ctr[C_PASSES] = 1;
}

__global__ __launch_bounds__(256) void k_final_rest(int32_t* lab, int32_t N, uint32_t* __restrict__ ctr,
                                                    const uint32_t* __restrict__ open_flags, int hops, int sweeps,
                                                    bool even)
{
    if (open_flags[blockIdx.x] == 0) return;
    const LabelRun r = label_run(lab, N, even);
    bool open = true;
    int k = 0;
    for (; __ballot(open) != 0 && k < sweeps; ++k)
        open = sweep(r.lab, r.n, lab, lab, N, hops, r.t, r.stride, k > 0);
    const bool left = __ballot(open) != 0;
    if (__lane_id() != 0) return;
    if (left) atomicOr(&ctr[C_OPEN], 1u);
    // a diagnostic: waves that needed one sweep need not queue at the counter
    if (k > 1 || (blockIdx.x == 0 && threadIdx.x == 0)) atomicMax(&ctr[C_PASSES], 1u + (uint32_t)k);
}

hipError_t launch_labels(const Grid& g, int32_t* lab, const Work& w, const Tuning& tu, hipStream_t s)
{
    const int32_t N = g.N;
    if (reinterpret_cast<uintptr_t>(lab) & 15u) return hipErrorInvalidValue;
    const int sweeps = sweeps_for(tu, N);
    if (g.ndim == 2 || g.ndim == 3) {
        if ((reinterpret_cast<uintptr_t>(w.exits) | reinterpret_cast<uintptr_t>(w.exres)) & 15u)
            return hipErrorInvalidValue;
        int ty, tz;
        tile_shape(tu, g.ndim, &ty, &tz);
        const TileArgs a = tile_args(nullptr, g, lab, nullptr, w, ty, tz);
        const int eblocks = all_blocks(w.cap_exit);
        // the jump reads entries that other threads have already advanced,
        // which shortens long chains: it needs every entry initialised first
        hipLaunchKernelGGL(k_exit_init, dim3(eblocks), dim3(256), 0, s, a, w.exres);
        // paths through thousands of tiles need an axis as long (or a field
        // made for it); elsewhere eight waves a SIMD in order are 2 to 3 us
        // faster (labels of 201 x 190 x 333 noise 46 and 49 us, 512^3 393 and 396)
        constexpr int kLongAxis = 1024;  // tiles
        const int axis = std::max({a.tiles_x, a.tiles_y, a.ntiles / (a.tiles_x * a.tiles_y)});
        const bool even = axis >= kLongAxis;
        const bool capped = exits_capped(w, N);
        const int slot = capped ? C_CODES : C_OPEN;
        hipLaunchKernelGGL(k_exit_jump, dim3(even ? even_blocks(w.cap_exit) : eblocks), dim3(256), 0, s, a, w.exres, N,
                           tu.hops, capped ? std::min(sweeps, kCappedSweeps) : sweeps, even, slot);
        const hipError_t e = launch_final_tiled(g, lab, w, tu, capped ? tu.hops : N, slot, s);
        if (e != hipSuccess || !capped) return e;
        hipLaunchKernelGGL(k_codes_rest, dim3(even_blocks(N)), dim3(256), 0, s, lab, w.exres, N, w.ctr, tu.hops, sweeps);
        return hipGetLastError();
    }
    // long paths whose vertices lie close together in memory need an axis as
    // long, and close to the last one (or a field made for it); elsewhere eight
    // waves a SIMD in order are the better trade (labels of 16^6 46.8 and 47.6
    // us, 24^6 773 and 851; slopes along the last axis of 16 x 16 x 16 x 4000
    // 2.6 and 1.0 ms, of 16 x 16 x 16 x 1000 0.40 and 0.30, along the first of
    // 4000 x 16 x 16 x 16 0.30 and 0.45)
    bool even = false;
    int64_t stride = 1;
    for (int i = g.ndim - 1; i >= 0 && stride <= 256; --i) {
        even |= g.dims[i] >= 512;
        stride *= g.dims[i];
    }
    const int blocks = even ? even_blocks(N) : all_blocks(N);
    uint32_t* flags = w.bsum + kSumRow;  // free until stage (d)
    hipLaunchKernelGGL(k_final, dim3(blocks), dim3(256), 0, s, lab, N, w.ctr, flags, even);
    hipLaunchKernelGGL(k_final_rest, dim3(blocks), dim3(256), 0, s, lab, N, w.ctr, flags, tu.hops, sweeps, even);
    return hipGetLastError();
}

}  // namespace eg
