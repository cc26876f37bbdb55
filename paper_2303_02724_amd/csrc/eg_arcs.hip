// eg_arcs.hip -- stage (d) and the canonical outputs, for one field or a batch.
//
// Classification leaves the maxima and the saddles as two row-padded bitmasks.
// Here:
//   1. k_mask_count / k_mask_emit: an order-preserving compaction of each mask
//      (block counts, then every block adds up the counts before its own and
//      expands its words), so maxima[] and saddles[] come out in ascending
//      vertex order without a sort;
//   2. k_arc_count: for every saddle, the highest vertex of each upper-link
//      component (UpperLinkRep, Sec. 3.4), the label it reaches, and the
//      number of distinct labels: the saddle's arcs (arcs form a set,
//      Sec. 2); the smallest are kept in registers and stored (four in 2D
//      and 3D, eight from 4D on);
//   3. k_arc_write: the CSR offsets from the counts, then the arcs (a saddle
//      with more distinct arcs than were stored, rare, finds the rest in
//      ascending order by one more pass over its components per arc); the
//      last block, which has added up every count, writes the header.
// No step uses an atomic: every position comes from a scan, so results do
// not depend on scheduling.
//
// Every kernel is written against a field selector: OneField (the field is
// the kernel argument, blocks are blockIdx.x) or BatchFields (the plan lists
// the fields; a flat grid is split over them in proportion to their size).
#include <algorithm>

#include "eg_internal.h"
#include "eg_rows.h"
#include "eg_link.h"
#include "eg_sample.h"

namespace eg {

// ------------------------------------------------------------------ selectors

struct OneField {
    ArcArgs a;
    // the field of this block, the block's index among the field's blocks and
    // their number
    __device__ __forceinline__ const ArcArgs& locate(uint32_t& blk, uint32_t& nb) const
    {
        blk = blockIdx.x;
        nb = gridDim.x;
        return a;
    }
};

struct BatchFields {
    EG_GPTR(const BatchPlan) plan;
    __device__ __forceinline__ const ArcArgs& locate(uint32_t& blk, uint32_t& nb) const
    {
        const EG_GPTR(BatchField) fs = plan->fields;
        const int64_t b = blockIdx.x;
        int lo = 0, hi = plan->count - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (fs[mid].arc_base <= b)
                lo = mid;
            else
                hi = mid - 1;
        }
        const int f = __builtin_amdgcn_readfirstlane(lo);
        blk = (uint32_t)(b - fs[f].arc_base);
        nb = (uint32_t)fs[f].arc.arc_blocks;
        return fs[f].arc;
    }
};

// ------------------------------------------------------------------ helpers

// Contiguous chunk [lo, hi) of [0, n) for block blk of nb: whole rounds of
// 256 items, so every block but the last has full rounds.
__device__ __forceinline__ void chunk(uint32_t n, uint32_t nb, uint32_t blk, uint32_t& lo, uint32_t& hi)
{
    uint32_t per = (uint32_t)(((uint64_t)n + nb - 1u) / nb);
    per = (per + 255u) & ~255u;
    if (per == 0) per = 256u;
    const uint64_t l = (uint64_t)blk * per;
    lo = (uint32_t)(l < n ? l : n);
    const uint64_t h = (uint64_t)lo + per;
    hi = (uint32_t)(h < n ? h : n);
}

// The same with the blocks that have a chunk dealt to the XCDs in runs, so
// that neighbouring saddles' gathers meet in one L2; blk becomes the chunk's
// number.  Up to 4D (stage (d) of 201 x 190 x 333 noise 113 -> 101 us, 4D 94 ->
// 84); the runs of 5D and 6D grids span more planes than an L2 holds, and
// dealing the chunks round-robin evens them out better (5D 521 against 541).
template <int NDIM>
__device__ __forceinline__ void chunk_run(uint32_t n, uint32_t nb, uint32_t& blk, uint32_t& lo, uint32_t& hi)
{
    uint32_t per = (uint32_t)(((uint64_t)n + nb - 1u) / nb);
    per = (per + 255u) & ~255u;
    const uint32_t used = per ? (n + per - 1u) / per : 0u;
    if (NDIM <= 4 && blk < used) blk = (uint32_t)xcd_run((int)blk, (int)used);
    chunk(n, nb, blk, lo, hi);
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    const int lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    return x;
}

// Exclusive scan of x over the block's threads; total gets the sum.  Uses
// tmp[0 .. BT / 64); every thread must call it.
template <int BT = 256>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t* tmp, uint32_t& total)
{
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const uint32_t inc = wave_incl_scan(x);
    if (lane == 63) tmp[w] = inc;
    __syncthreads();
    uint32_t pre = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < BT / 64; ++k) {
        pre += k < w ? tmp[k] : 0u;
        total += tmp[k];
    }
    __syncthreads();
    return pre + inc - x;
}

// Sums over the block's threads, to every thread.  Uses tmp[0 .. BT / 32).
template <int BT = 256>
__device__ __forceinline__ void block_sum2(uint32_t& x, uint32_t& y, uint32_t* tmp)
{
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        x += __shfl_xor(x, o);
        y += __shfl_xor(y, o);
    }
    if ((threadIdx.x & 63) == 0) {
        tmp[2 * w] = x;
        tmp[2 * w + 1] = y;
    }
    __syncthreads();
    x = y = 0;
#pragma unroll
    for (int k = 0; k < BT / 64; ++k) {
        x += tmp[2 * k];
        y += tmp[2 * k + 1];
    }
    __syncthreads();
}

// Sums of the block counts before block blk in rows `row` and `row + 1`.  Every
// block adds them up for itself (at most kArcBlocks entries, two coalesced
// reads per 256): a kernel of its own for the scan costs more than the reads,
// 4.5 to 8.6 us on every field.
template <int BT = 256>
__device__ __forceinline__ void sums_before(const ArcArgs& A, int row, uint32_t blk, uint32_t* tmp, uint32_t& a,
                                            uint32_t& b)
{
    a = b = 0;
    const EG_GPTR(uint32_t) p = A.bsum + row * kSumRow;
    for (uint32_t i = threadIdx.x; i < blk; i += BT) {
        a += p[i];
        b += p[kSumRow + i];
    }
    block_sum2<BT>(a, b, tmp);
}

__device__ __forceinline__ uint32_t saddle_count(const ArcArgs& A)
{
    const uint32_t n = A.ctr[C_NSAD];
    return n < A.cap_sad ? n : A.cap_sad;
}

// ------------------------------------------------------------------ masks

// Set bits of both masks in the block's chunk of the words.
template <class Sel>
__global__ __launch_bounds__(256) void k_mask_count(Sel sel)
{
    __shared__ uint32_t tmp[8];
    uint32_t blk, nb;
    const ArcArgs A = sel.locate(blk, nb);  // a copy: loop loads cannot alias it
    uint32_t lo, hi;
    chunk((uint32_t)A.words, nb, blk, lo, hi);
    uint32_t cm = 0, cs = 0;
    for (uint32_t i = lo + threadIdx.x; i < hi; i += 256) {
        cm += (uint32_t)__popcll(A.mmask[i]);
        cs += (uint32_t)__popcll(A.smask[i]);
    }
    block_sum2(cm, cs, tmp);
    if (threadIdx.x == 0) {
        A.bsum[blk] = cm;
        A.bsum[kSumRow + blk] = cs;
    }
}

// The vertex ids of the set bits of a round of 256 words (one per thread), both
// masks at once: one scan of the packed counts (at most 16384 each), the ids
// staged in LDS so that the global stores are whole-wave and contiguous; a
// round with more ids than the stage (very dense masks) writes directly.
// Entries at or past a capacity are dropped.  The last block's totals are the
// field's counts.
constexpr int kStage = 6144;
template <class Sel>
__global__ __launch_bounds__(256) void k_mask_emit(Sel sel)
{
    __shared__ uint32_t tmp[8];
    __shared__ int32_t stage[kStage];
    uint32_t blk, nb;
    const ArcArgs A = sel.locate(blk, nb);  // a copy: loop loads cannot alias it
    uint32_t lo, hi;
    chunk((uint32_t)A.words, nb, blk, lo, hi);
    uint32_t rm, rs;
    sums_before(A, 0, blk, tmp, rm, rs);
    const uint32_t XW = (uint32_t)A.XW, X = (uint32_t)A.X;
    for (uint32_t base = lo; base < hi; base += 256) {
        const uint32_t i = base + threadIdx.x;
        uint64_t m = i < hi ? A.mmask[i] : 0ull;
        uint64_t sd = i < hi ? A.smask[i] : 0ull;
        uint32_t total;
        const uint32_t local =
            block_excl_scan((uint32_t)__popcll(m) | ((uint32_t)__popcll(sd) << 16), tmp, total);
        const uint32_t tm = total & 0xFFFFu, ts = total >> 16;
        uint32_t jm = local & 0xFFFFu, js = local >> 16;
        const uint32_t row = i / XW, xw = i - row * XW;
        const int32_t vbase = (int32_t)(row * X + xw * 64u);
        if (tm + ts <= (uint32_t)kStage) {
            for (; m; ++jm, m &= m - 1ull) stage[jm] = vbase + (__ffsll((unsigned long long)m) - 1);
            for (js += tm; sd; ++js, sd &= sd - 1ull) stage[js] = vbase + (__ffsll((unsigned long long)sd) - 1);
            __syncthreads();
            for (uint32_t j = threadIdx.x; j < tm; j += 256)
                if (rm + j < A.cap_max) A.maxima[rm + j] = stage[j];
            for (uint32_t j = threadIdx.x; j < ts; j += 256)
                if (rs + j < A.cap_sad) A.saddles[rs + j] = stage[tm + j];
            __syncthreads();
        } else {
            for (uint32_t p = rm + jm; m; ++p, m &= m - 1ull)
                if (p < A.cap_max) A.maxima[p] = vbase + (__ffsll((unsigned long long)m) - 1);
            for (uint32_t p = rs + js; sd; ++p, sd &= sd - 1ull)
                if (p < A.cap_sad) A.saddles[p] = vbase + (__ffsll((unsigned long long)sd) - 1);
        }
        rm += tm;
        rs += ts;
    }
    if (blk == nb - 1 && threadIdx.x == 0) {
        A.ctr[C_NMAX] = rm;
        A.ctr[C_NSAD] = rs;
    }
}

// ------------------------------------------------------------------ arcs

// Rows of the link as a mask: one bit per row.
template <int NDIM>
struct LinkMask {
    using type = uint32_t;
};
template <>
struct LinkMask<5> {
    using type = uint64_t;
};
template <>
struct LinkMask<6> {
    using type = unsigned __int128;
};
template <int NDIM>
using LMask = typename LinkMask<NDIM>::type;

__device__ __forceinline__ int low_row(uint32_t m) { return __ffs((int)m) - 1; }
__device__ __forceinline__ int low_row(uint64_t m) { return lowest_bit(m); }
__device__ __forceinline__ int low_row(unsigned __int128 m) { return lowest_bit(m); }

// 1D and 4D-6D classification stores every vertex's order key (already
// reversed for the minimum graph); 2D and 3D read the field.  Fields of other
// sample types (3D) are read in their own type: 32-bit keys for 8- and 16-bit
// integers, exact 64-bit keys for the wider types.
template <int SRC>
struct VertexKey {
    using type = uint32_t;
};
template <>
struct VertexKey<SRC_WIDE> {
    using type = uint64_t;
};
template <int SRC>
using VKey = typename VertexKey<SRC>::type;
template <int NDIM>
constexpr bool kStoredKeys = NDIM != 2 && NDIM != 3;
// Up to 5D a thread of k_arc_count parks the keys of its saddle's
// neighbourhood in its own column of LDS, so that a rep is found by visiting
// its component's rows only (registers cannot be indexed: there, every
// component costs a scan of all rows; a column is one bank, so the reads do
// not conflict).  Stage (d), before and after, with the stored lists' sort as
// minima and maxima: 201 x 190 x 333 noise (1.95 M saddles) 124 -> 110 us,
// 4D (0.92 M of 10 M vertices) 132 -> 95, 5D (3.8 M) 577 -> 523.  What bounds
// 5D now is the L2: a gather fetches 128 bytes for the 8 it uses.  6D (126
// rows, 32 KB a wave) reads the keys of a component's rows again instead, as
// k_arc_write does everywhere: they need the waves (the path kernels: kPathKeys).
template <int NDIM>
constexpr bool kKeysInLds = NDIM <= 5;
// Threads per block: a 5D wave's keys take 16 KB of LDS, and ten of them fit a
// compute unit in blocks of two, eight in blocks of four.
template <int NDIM>
constexpr int kArcThreads = NDIM == 5 ? 128 : 256;

// Most waves per SIMD that k_arc_count schedules its registers for: 6D is
// bound by the latency of its 126 gathers, and more of them in flight in fewer
// waves is the better trade.  Stage (d) with registers for eight waves and for
// two, us: smoothed noise of 16^6 290 and 209, smoother 101 and 93, 12^6 87 and
// 76, 9 x 10 x 11 x 12 x 13 x 14 81 and 71, 2^5 x 100 000 107 and 94, noise of
// 12^6 275 and 236; of ten fields one was slower (noise of 16^6, 713 and 730).
template <int NDIM>
constexpr int kArcWaves = NDIM == 6 ? 2 : 8;

template <int NDIM, bool MINMODE, int SRC>
__device__ __forceinline__ VKey<SRC> vertex_key(const ArcArgs& A, int v)
{
    if constexpr (SRC == SRC_WIDE)
        return exact_key<MINMODE>(A.f, A.dtype, v);
    else if constexpr (SRC == SRC_INT)
        return int_key<MINMODE>(A.f, A.dtype, v);
    else if constexpr (kStoredKeys<NDIM>)
        return A.keys[v];
    else
        return mode_key<MINMODE>(A.f[v]);
}

// Where a kernel has the keys of a neighbourhood once it is loaded.
enum : int {
    KEYS_AGAIN = 0,  // nowhere: those of a component are read again
    KEYS_LDS = 1,    // in the thread's column of LDS
    KEYS_REGS = 2,   // in registers: a rep takes a scan of all rows
};

// LDS of a block of the arc and path kernels: the rows' linear offsets, and
// the keys (row j of thread t at keys[j][t]) where they are parked.
template <int NDIM, int KEYS, int SRC_ = SRC_F32>
struct RowLds {
    static constexpr int K = Rows<NDIM>::K;
    static constexpr int N = NDIM;
    static constexpr int SRC = SRC_;
    static constexpr int kKeys = KEYS;
    VKey<SRC> keys[KEYS == KEYS_LDS ? K : 1][KEYS == KEYS_LDS ? kArcThreads<NDIM> : 1];
    int off[K];
};

// A saddle's neighbourhood: its upper-link mask, and the keys where they stay
// in registers.
template <class LDS>
struct Hood {
    LMask<LDS::N> up;
    VKey<LDS::SRC> us[LDS::kKeys == KEYS_REGS ? LDS::K : 1];
};

template <class LDS>
__device__ __forceinline__ void load_rows(const ArcArgs& A, LDS& T)
{
    constexpr int NDIM = LDS::N;
    constexpr Rows<NDIM> R = make_rows_ce<NDIM>();
    constexpr int K = Rows<NDIM>::K;
    int st[NDIM];
    st[NDIM - 1] = 1;
#pragma unroll
    for (int i = NDIM - 2; i >= 0; --i) st[i] = st[i + 1] * A.dims[i + 1];
    for (int j = threadIdx.x; j < K; j += kArcThreads<NDIM>) {
        int off = 0;
#pragma unroll
        for (int i = 0; i < NDIM; ++i) off += R.d[j][i] * st[i];
        T.off[j] = off;
    }
    __syncthreads();
}

// The upper-link mask of saddle v over the K Freudenthal rows (Alg. 1, Sec.
// 3.3), and the rows' keys into this thread's column (0 outside the grid,
// below every vertex).
template <int NDIM, bool MINMODE, class LDS>
__device__ __forceinline__ Hood<LDS> load_nbhd(const ArcArgs& A, int v, LDS& T)
{
    constexpr Rows<NDIM> R = make_rows_ce<NDIM>();
    constexpr int K = Rows<NDIM>::K;
    int c[NDIM], st[NDIM];
    {
        int rem = v, stride = 1;
#pragma unroll
        for (int i = NDIM - 1; i >= 0; --i) {
            const int d = A.dims[i];
            c[i] = rem % d;
            rem /= d;
            st[i] = stride;
            stride *= d;
        }
    }
    const VKey<LDS::SRC> uv = vertex_key<NDIM, MINMODE, LDS::SRC>(A, v);
    Hood<LDS> h;
    // 32 rows per word, pushed from the highest row down
    constexpr int NW = (K + 31) / 32;
    uint32_t wd[NW];
    static_for<0, K>([&](auto step) {
        constexpr int j = K - 1 - decltype(step)::value;
        bool in = true;
        int off = 0;
#pragma unroll
        for (int i = 0; i < NDIM; ++i) {
            const int d = R.d[j][i];
            if (d != 0) {
                in = in && (unsigned)(c[i] + d) < (unsigned)A.dims[i];
                off += d * st[i];
            }
        }
        // no branch around the load: every row's load is in flight at once
        const VKey<LDS::SRC> x = vertex_key<NDIM, MINMODE, LDS::SRC>(A, in ? v + off : v);
        const VKey<LDS::SRC> u = in ? x : 0;
        if constexpr (LDS::kKeys == KEYS_LDS) T.keys[j][threadIdx.x] = u;
        if constexpr (LDS::kKeys == KEYS_REGS) h.us[j] = u;
        constexpr bool wins = (j >= K / 2) != MINMODE;
        if constexpr (LDS::SRC == SRC_WIDE)  // a wide sample's key may be 0 itself
            wd[0] = (j == K - 1 ? 0u : 2u * wd[0]) | (in && (wins ? u >= uv : u > uv) ? 1u : 0u);
        else if constexpr (j == K - 1 || j % 32 == 31)
            wd[j / 32] = first_above<wins>(u, uv);
        else
            wd[j / 32] = push_above<wins>(wd[j / 32], u, uv);
    });
    LMask<NDIM> up = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) up |= LMask<NDIM>(wd[w]) << (w == 0 ? 0 : 32 * w);
    h.up = up;
    return h;
}

// The component of the lowest row of `rem`: a table of every mask up to 3D,
// set algebra on the link's rows (eg_link.h) above.
template <int NDIM>
struct CompTable {
    uint16_t c[1 << Rows<NDIM>::K];
};
template <int NDIM>
constexpr CompTable<NDIM> make_comps()
{
    constexpr Rows<NDIM> r = make_rows_ce<NDIM>();
    CompTable<NDIM> t{};
    for (uint32_t m = 1; m < (1u << Rows<NDIM>::K); ++m)
        t.c[m] = (uint16_t)closure_ce<NDIM>(r, m & (~m + 1u), m);
    return t;
}
__constant__ CompTable<1> c_comp1 = make_comps<1>();
__constant__ CompTable<2> c_comp2 = make_comps<2>();
__constant__ CompTable<3> c_comp3 = make_comps<3>();

template <int NDIM>
__device__ __forceinline__ LMask<NDIM> first_component(LMask<NDIM> rem)
{
    if constexpr (NDIM == 1)
        return c_comp1.c[rem];
    else if constexpr (NDIM == 2)
        return c_comp2.c[rem];
    else if constexpr (NDIM == 3)
        return c_comp3.c[rem];
    else
        return link_component<NDIM>(rem);
}

// The key of row j of saddle v's link (a row in the grid).
template <int NDIM, bool MINMODE, class LDS>
__device__ __forceinline__ VKey<LDS::SRC> key_at(const ArcArgs& A, int v, int j, const LDS& T)
{
    if constexpr (LDS::kKeys == KEYS_LDS)
        return T.keys[j][threadIdx.x];
    else
        return vertex_key<NDIM, MINMODE, LDS::SRC>(A, v + T.off[j]);
}

// The highest vertex of a component (UpperLinkRep, Sec. 3.4): its rows in
// ascending vertex order, the later of two equal vertices the higher one, the
// earlier in the minimum graph.
template <int NDIM, bool MINMODE, class LDS>
__device__ __forceinline__ int rep_of(const ArcArgs& A, int v, const Hood<LDS>& h, LMask<NDIM> comp, const LDS& T)
{
    if constexpr (LDS::kKeys == KEYS_REGS) {
        VKey<LDS::SRC> best_u = 0;
        int best = 0;
        static_for<0, LDS::K>([&](auto step) {
            constexpr int j = MINMODE ? LDS::K - 1 - decltype(step)::value : decltype(step)::value;
            if ((uint32_t)(comp >> j) & 1u && h.us[j] >= best_u) {
                best_u = h.us[j];
                best = j;
            }
        });
        return v + T.off[best];
    }
    // two rows a round (the second again the first when there is none left),
    // so that two reads are in flight
    VKey<LDS::SRC> best_u = 0;
    int best = low_row(comp);
    do {
        const int j0 = low_row(comp);
        comp &= comp - 1;
        const int j1 = comp != 0 ? low_row(comp) : j0;
        comp &= comp - 1;  // 0 & anything stays 0
        const VKey<LDS::SRC> u0 = key_at<NDIM, MINMODE>(A, v, j0, T);
        const VKey<LDS::SRC> u1 = key_at<NDIM, MINMODE>(A, v, j1, T);
        const bool w0 = MINMODE ? u0 > best_u : u0 >= best_u;
        best_u = w0 ? u0 : best_u;
        best = w0 ? j0 : best;
        const bool w1 = MINMODE ? u1 > best_u : u1 >= best_u;
        best_u = w1 ? u1 : best_u;
        best = w1 ? j1 : best;
    } while (comp != 0);
    return v + T.off[best];
}

// Calls f(rep) for every upper-link component of saddle v, in ascending order
// of the components' smallest vertices (rows are in linear-index order).
template <int NDIM, bool MINMODE, class LDS, class F>
__device__ __forceinline__ void for_each_rep(const ArcArgs& A, int v, const Hood<LDS>& h, const LDS& T, F&& f)
{
    LMask<NDIM> rem = h.up;
    while (rem != 0) {
        const LMask<NDIM> comp = first_component<NDIM>(rem);
        rem &= ~comp;
        f(rep_of<NDIM, MINMODE>(A, v, h, comp, T));
    }
}

// f(label) for every component: the label its rep reaches.  A label is used
// only after the next component's rep has been sought, so its load is not
// waited for on its own.
template <int NDIM, bool MINMODE, class LDS, class F>
__device__ __forceinline__ void for_each_arc_label(const ArcArgs& A, int v, const Hood<LDS>& h, const LDS& T, F&& f)
{
    uint32_t last = 0;
    bool have = false;
    for_each_rep<NDIM, MINMODE>(A, v, h, T, [&](int rep) {
        const uint32_t L = (uint32_t)A.lab[rep];
        if (have) f(last);
        last = L;
        have = true;
    });
    if (have) f(last);
}

// The S smallest distinct arc labels of a saddle, ascending (unused entries
// ~0u; labels are vertex ids below 2^31), and the number of distinct labels as
// far as it is known: `more` is set when there are further ones above lo[S-1].
// S = 4 in 2D/3D (at most 3 and 6 components), 8 from 4D on, where more
// components are common.
template <int NDIM>
struct ArcList {
    static constexpr int S = NDIM >= 4 ? 8 : 4;
    uint32_t lo[S];
    bool more;
};

__device__ __forceinline__ void order2(uint32_t& a, uint32_t& b)
{
    const uint32_t t = min(a, b);
    b = max(a, b);
    a = t;
}
// Ascending order of 6 or 8 values (Batcher's odd-even merge sort).
__device__ __forceinline__ void sort_few(uint32_t (&x)[6])
{
    order2(x[0], x[5]), order2(x[1], x[3]), order2(x[2], x[4]);
    order2(x[1], x[2]), order2(x[3], x[4]);
    order2(x[0], x[3]), order2(x[2], x[5]);
    order2(x[0], x[1]), order2(x[2], x[3]), order2(x[4], x[5]);
    order2(x[1], x[2]), order2(x[3], x[4]);
}
__device__ __forceinline__ void sort_few(uint32_t (&x)[8])
{
    order2(x[0], x[1]), order2(x[2], x[3]), order2(x[4], x[5]), order2(x[6], x[7]);
    order2(x[0], x[2]), order2(x[1], x[3]), order2(x[4], x[6]), order2(x[5], x[7]);
    order2(x[1], x[2]), order2(x[5], x[6]);
    order2(x[0], x[4]), order2(x[1], x[5]), order2(x[2], x[6]), order2(x[3], x[7]);
    order2(x[2], x[4]), order2(x[3], x[5]);
    order2(x[1], x[2]), order2(x[3], x[4]), order2(x[5], x[6]);
}

template <int NDIM, bool MINMODE, class LDS>
__device__ __forceinline__ ArcList<NDIM> first_arcs(const ArcArgs& A, int v, const Hood<LDS>& h, const LDS& T, int& beta)
{
    constexpr int S = ArcList<NDIM>::S;
    // every component of a saddle up to 3D, nearly every saddle's above, has a
    // place in x: its labels go in by one pass of minima and maxima each,
    // equal ones drop out afterwards
    constexpr int X = NDIM >= 4 ? 8 : 6;
    uint32_t x[X];
#pragma unroll
    for (int k = 0; k < X; ++k) x[k] = ~0u;
    beta = 0;
    for_each_arc_label<NDIM, MINMODE>(A, v, h, T, [&](uint32_t L) {
        ++beta;
#pragma unroll
        for (int k = 0; k < X; ++k) order2(x[k], L);
    });
    ArcList<NDIM> r;
    bool dup = false;
#pragma unroll
    for (int k = X - 1; k > 0; --k) {
        const bool same = x[k] == x[k - 1] && x[k] != ~0u;
        dup |= same;
        x[k] = same ? ~0u : x[k];
    }
    if (dup) sort_few(x);
#pragma unroll
    for (int k = 0; k < S; ++k) r.lo[k] = x[k];
    r.more = false;
    if constexpr (X > S) {
        r.more = x[S] != ~0u;
    } else if (beta > X) {
        // more components than places: the list again, label by label
#pragma unroll
        for (int k = 0; k < S; ++k) r.lo[k] = ~0u;
        for_each_arc_label<NDIM, MINMODE>(A, v, h, T, [&](uint32_t L) {
            bool known = false;
#pragma unroll
            for (int k = 0; k < S; ++k) known |= L == r.lo[k];
            if (known) return;
#pragma unroll
            for (int k = 0; k < S; ++k) order2(r.lo[k], L);
            r.more |= L != ~0u;  // the largest moved out
        });
    }
    return r;
}

// Distinct labels above `last`, ascending, one pass over the components
// each: for saddles with more distinct arcs than the list holds (rare).  Calls
// emit(k, label) for the k-th of them and returns their number.
template <int NDIM, bool MINMODE, class LDS, class E>
__device__ __forceinline__ uint32_t labels_above(const ArcArgs& A, int v, const Hood<LDS>& h, const LDS& T, uint32_t last,
                                                 E&& emit)
{
    uint32_t k = 0;
    for (;;) {
        uint32_t next = ~0u;
        for_each_arc_label<NDIM, MINMODE>(A, v, h, T, [&](uint32_t L) {
            if (L > last && L < next) next = L;
        });
        if (next == ~0u) return k;
        emit(k, next);
        ++k;
        last = next;
    }
}

// Distinct-arc count, beta and the first four (eight from 4D on) arcs of every
// saddle of the block's chunk; the block's sums of both counts go to rows 2
// and 3.
template <int NDIM, bool MINMODE, class LDS>
__device__ __forceinline__ void arc_count_body(const ArcArgs& A, uint32_t blk_, uint32_t nb, LDS& T, uint32_t* tmp)
{
    load_rows(A, T);
    uint32_t lo, hi;
    uint32_t blk = blk_;
    chunk_run<NDIM>(saddle_count(A), nb, blk, lo, hi);
    const int tid = threadIdx.x;
    uint32_t sc = 0, sb = 0;
    for (uint32_t i = lo + tid; i < hi; i += kArcThreads<NDIM>) {
        // saddle ids come from the compaction; the check keeps a stage run
        // on a workspace without classification inside the grid
        const int v = min(max(A.saddles[i], 0), A.N - 1);
        const auto h = load_nbhd<NDIM, MINMODE>(A, v, T);
        int beta;
        const ArcList<NDIM> r = first_arcs<NDIM, MINMODE>(A, v, h, T, beta);
        constexpr int S = ArcList<NDIM>::S;
        uint32_t n = 0;
#pragma unroll
        for (int k = 0; k < S; ++k) n += r.lo[k] != ~0u;
        if (r.more) n += labels_above<NDIM, MINMODE>(A, v, h, T, r.lo[S - 1], [](uint32_t, uint32_t) {});
        if (A.beta) A.beta[i] = beta;
        A.offsets[i + 1] = (int32_t)n;  // the count until k_arc_write turns it into an offset
        A.atmp[i] = make_uint4(r.lo[0], r.lo[1], r.lo[2], r.lo[3]);
        if constexpr (S > 4) A.atmp[A.cap_sad + i] = make_uint4(r.lo[4], r.lo[5], r.lo[6], r.lo[7]);
        sc += n;
        sb += (uint32_t)beta;
    }
    block_sum2<kArcThreads<NDIM>>(sc, sb, tmp);
    if (tid == 0) {
        A.bsum[2 * kSumRow + blk] = sc;
        A.bsum[3 * kSumRow + blk] = sb;
    }
}

// Status and counts.
__device__ __forceinline__ void write_header(const ArcArgs& A, uint32_t narc, uint32_t npairs)
{
    const uint32_t* c = A.ctr;
    const uint32_t nmax = c[C_NMAX], nsad = c[C_NSAD];
    const bool sad_over = nsad > A.cap_sad;
    int status = EG_OK;
    if (c[C_NAN])
        status = EG_ERR_NAN;
    else if (A.last_flag && *A.last_flag)
        status = EG_ERR_UNRESOLVED;
    else if (nmax > A.cap_max || sad_over || narc > A.cap_arc)
        status = EG_ERR_CAPACITY;
    int32_t* h = A.header;
    h[EG_H_STATUS] = status;
    h[EG_H_NMAX] = (int32_t)nmax;
    h[EG_H_NSAD] = (int32_t)nsad;
    // with saddles cut off at the capacity, the arc and pair totals cover
    // only the first cap_sad saddles: unknown
    h[EG_H_NARC] = sad_over ? -1 : (int32_t)narc;
    h[EG_H_NPAIRS] = sad_over ? -1 : (int32_t)npairs;
    h[EG_H_PASSES] = (int32_t)c[C_PASSES];
    uint32_t exits = 0;  // counters behind row 0 (zero on grids without tiles)
    for (int r = 0; r < kRegions; ++r) exits += A.bsum[kArcBlocks + kRegionStride * r];
    h[EG_H_EXITS] = (int32_t)exits;
}

// Four saddles per thread and round: their counts and stored arcs are all
// loaded before the one scan of the round (the counts packed by 16 bits: a
// saddle has at most 63 arcs).
template <int NDIM, bool MINMODE, class LDS>
__device__ __forceinline__ void arc_write_body(const ArcArgs& A, uint32_t blk_, uint32_t nb, LDS& T, uint32_t* tmp)
{
    constexpr int S = ArcList<NDIM>::S;
    constexpr int R = 4, BT = kArcThreads<NDIM>;
    uint32_t lo, hi;
    uint32_t blk = blk_;
    chunk_run<NDIM>(saddle_count(A), nb, blk, lo, hi);
    const int tid = threadIdx.x;
    if (blk == 0 && tid == 0) A.offsets[0] = 0;
    if (lo >= hi && blk != nb - 1) return;  // nothing to write, and not the last block
    uint32_t run, pairs;
    sums_before<BT>(A, 2, blk, tmp, run, pairs);
    const uint32_t first = run;
    bool big = false;
    for (uint32_t base = lo; base < hi; base += BT * R) {
        uint32_t n[R];
        uint4 t[R], u[S > 4 ? R : 1];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t i = base + BT * r + tid;
            const uint32_t at = i < hi ? i : lo;
            n[r] = i < hi ? (uint32_t)A.offsets[at + 1] : 0u;
            t[r] = A.atmp[at];
        }
        if constexpr (S > 4) {
            // the next four stored arcs
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (n[r] > 4) u[r] = A.atmp[A.cap_sad + base + BT * r + tid];
        }
        uint32_t t01, t23;
        const uint32_t e01 = block_excl_scan<BT>(n[0] | (n[1] << 16), tmp, t01);
        const uint32_t e23 = block_excl_scan<BT>(n[2] | (n[3] << 16), tmp, t23);
        const uint32_t tot[R] = {t01 & 0xFFFFu, t01 >> 16, t23 & 0xFFFFu, t23 >> 16};
        const uint32_t ex[R] = {e01 & 0xFFFFu, e01 >> 16, e23 & 0xFFFFu, e23 >> 16};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t i = base + BT * r + tid;
            const uint32_t pos = run + ex[r];
            run += tot[r];
            if (i >= hi) continue;
            const uint32_t a4[4] = {t[r].x, t[r].y, t[r].z, t[r].w};
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if (k < n[r] && pos + k < A.cap_arc) A.arcs[pos + k] = (int32_t)a4[k];
            if constexpr (S > 4) {
                if (n[r] > 4) {
                    const uint32_t b4[4] = {u[r].x, u[r].y, u[r].z, u[r].w};
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k)
                        if (4 + k < n[r] && pos + 4 + k < A.cap_arc) A.arcs[pos + 4 + k] = (int32_t)b4[k];
                }
            }
            big |= n[r] > (uint32_t)S;
            A.offsets[i + 1] = (int32_t)(pos + n[r]);
        }
    }
    if constexpr (NDIM >= 3) {  // at most three arcs in 1D and 2D
        // saddles with arcs past the stored ones: ascending selection over
        // their components, in a loop of its own (whose registers the loop
        // above then does not carry)
        if (__syncthreads_or(big)) {
            load_rows(A, T);
            for (uint32_t i = lo + tid; i < hi; i += BT) {
                const uint32_t pos = i == lo ? first : (uint32_t)A.offsets[i];
                if ((uint32_t)A.offsets[i + 1] - pos <= (uint32_t)S) continue;
                const int v = min(max(A.saddles[i], 0), A.N - 1);
                const uint32_t last = S > 4 ? A.atmp[A.cap_sad + i].w : A.atmp[i].w;
                const auto h = load_nbhd<NDIM, MINMODE>(A, v, T);
                labels_above<NDIM, MINMODE>(A, v, h, T, last, [&](uint32_t k, uint32_t L) {
                    if (pos + S + k < A.cap_arc) A.arcs[pos + S + k] = (int32_t)L;
                });
            }
        }
    }
    // the last block has seen every count
    if (blk == nb - 1 && tid == 0) write_header(A, run, pairs + A.bsum[3 * kSumRow + blk]);
}

template <int NDIM, bool MINMODE, int SRC = SRC_F32>
__global__ __launch_bounds__(kArcThreads<NDIM>)
    __attribute__((amdgpu_waves_per_eu(1, kArcWaves<NDIM>))) void k_arc_count(OneField sel)
{
    __shared__ RowLds<NDIM, kKeysInLds<NDIM> ? KEYS_LDS : KEYS_AGAIN, SRC> T;
    __shared__ uint32_t tmp[8];
    uint32_t blk, nb;
    const ArcArgs A = sel.locate(blk, nb);  // a copy: loop loads cannot alias it
    arc_count_body<NDIM, MINMODE>(A, blk, nb, T, tmp);
}

template <int NDIM, bool MINMODE, int SRC = SRC_F32>
__global__ __launch_bounds__(kArcThreads<NDIM>) void k_arc_write(OneField sel)
{
    __shared__ RowLds<NDIM, KEYS_AGAIN, SRC> T;
    __shared__ uint32_t tmp[8];
    uint32_t blk, nb;
    const ArcArgs A = sel.locate(blk, nb);  // a copy: loop loads cannot alias it
    arc_write_body<NDIM, MINMODE>(A, blk, nb, T, tmp);
}

// Batches hold 2D and 3D fields of either graph: the body is chosen per
// field (a uniform branch).
template <bool WRITE>
__global__ __launch_bounds__(256) void k_arc_batched(BatchFields sel)
{
    __shared__ uint32_t tmp[8];
    uint32_t blk, nb;
    const ArcArgs A = sel.locate(blk, nb);  // a copy: loop loads cannot alias it
    const int kind = __builtin_amdgcn_readfirstlane((A.ndim == 3 ? 2 : 0) + (A.minima ? 1 : 0));
    using L3 = RowLds<3, WRITE ? KEYS_AGAIN : KEYS_LDS>;
    using L2 = RowLds<2, WRITE ? KEYS_AGAIN : KEYS_LDS>;
    __shared__ L3 T3;
    L2& T2 = reinterpret_cast<L2&>(T3);
#define EG_BODY(ND, MM)                               \
    if (WRITE)                                        \
        arc_write_body<ND, MM>(A, blk, nb, T##ND, tmp); \
    else                                              \
        arc_count_body<ND, MM>(A, blk, nb, T##ND, tmp);
    switch (kind) {
        case 0: EG_BODY(2, false) break;
        case 1: EG_BODY(2, true) break;
        case 2: EG_BODY(3, false) break;
        default: EG_BODY(3, true) break;
    }
#undef EG_BODY
}

// ------------------------------------------------------------------ paths

// The walk of Alg. 2 from rep: visit(r) for rep and every vertex after it, up
// to the maximum (ptr(m) = m).  Every step must stay in the grid and rise in
// the order; a pointer that does not (out->ptr not holding this field's
// pointers) ends the walk and returns false, so no input can make it leave
// the grid or loop.
template <int NDIM, bool MINMODE, int SRC, class V>
__device__ __forceinline__ bool walk(const ArcArgs& A, EG_GPTR(const int32_t) const ptr, int r, V&& visit)
{
    visit(r);
    VKey<SRC> ur = vertex_key<NDIM, MINMODE, SRC>(A, r);
    for (;;) {
        const int q = ptr[r];
        if (q == r) return true;
        if ((unsigned)q >= (unsigned)A.N) return false;
        const VKey<SRC> uq = vertex_key<NDIM, MINMODE, SRC>(A, q);
        if (!(uq > ur || (uq == ur && (MINMODE ? q < r : q > r)))) return false;
        visit(q);
        r = q;
        ur = uq;
    }
}

// The count pass records the vertices it meets: step t of path c (c < kRecPaths)
// of saddle i at rec[(t kRecPaths + c) n + i], n saddles, for as many steps as
// the scratch holds.  The write pass then copies a saddle's paths, all of whose
// loads are independent, instead of walking them a second time, one dependent
// load a step (17 k paths in 256^3: 155 us for the two walks, 100 with the
// copy; 35 k in 512^3: 261 and 165).  Saddles with more or longer paths are
// walked again.
constexpr uint32_t kRecPaths = 3;
// Keys of the path kernels.  Walking wants waves, so 5D has no room to park
// them, and reading a component's keys again costs more than scanning
// registers at four waves per SIMD (32^5, in blocks of 128 threads: 2.96 ms
// again, 3.9 parked, 2.6 in registers).
template <int NDIM>
constexpr int kPathKeys = NDIM <= 4 ? KEYS_LDS : NDIM == 5 ? KEYS_REGS : KEYS_AGAIN;
// Threads per block of the path kernels.  A chunk is whole rounds of 256
// saddles, one round on most fields: blocks of 128 threads, as k_arc_count has
// in 5D, walk a round's paths in two turns (noise of 12^5 87 us, of 16 x 17 x 18 x
// 19 x 5 93, of 25 x 24 x 26 x 27 x 23 536; 56, 63 and 520 in blocks of 256).
constexpr int kPathThreads = 256;
constexpr uint32_t kRecSteps = 128;
__device__ __forceinline__ uint32_t recorded_steps(const PathArgs& P, uint32_t n)
{
    const int64_t s = P.cap_rec / ((int64_t)kRecPaths * (n > 0 ? n : 1));
    // with little room few saddles' paths fit, and recording costs more than
    // it saves.  Walked twice and recorded, us, over 25 fields of 1D to 4D: 16
    // steps and more 158 and 105, 270 and 156; 4 to 15 steps gain on large
    // fields (256^3 251 and 196, 2000^2 109 and 94) and lose on small ones (17 x
    // 300 x 300 40 and 47, 300^2 30 and 36); 1 to 3 steps 608 and 680, 140 and 143
    return s < 16 ? 0u : (uint32_t)(s < (int64_t)kRecSteps ? s : (int64_t)kRecSteps);
}

// Paths and path vertices of every saddle of the block's chunk (kept for the
// write pass in the workspace); the block's sums go to rows 1 and 2, and whether
// a walk met a pointer that leaves the grid or does not rise to row 3 (row 0
// also holds the exit list's counters).
template <int NDIM, bool MINMODE, int SRC = SRC_F32>
__global__ __launch_bounds__(kPathThreads) __attribute__((amdgpu_waves_per_eu(NDIM == 5 ? 4 : 1, 8))) void k_path_count(OneField sel, PathArgs P)
{
    constexpr int BT = kPathThreads;
    __shared__ RowLds<NDIM, kPathKeys<NDIM>, SRC> T;
    __shared__ uint32_t tmp[8];
    uint32_t blk, nb;
    const ArcArgs A = sel.locate(blk, nb);  // a copy: loop loads cannot alias it
    load_rows(A, T);
    uint32_t lo, hi;
    const uint32_t n = saddle_count(A), steps = recorded_steps(P, n);
    chunk(n, nb, blk, lo, hi);
    uint32_t sp = 0, sv = 0;
    bool bad = false;
    for (uint32_t i = lo + threadIdx.x; i < hi; i += BT) {
        const int v = A.saddles[i];
        uint32_t np = 0, nv = 0;
        uint32_t len0 = 0, len1 = 0, longest = 0;
        if ((unsigned)v < (unsigned)A.N) {
            const auto h = load_nbhd<NDIM, MINMODE>(A, v, T);
            for_each_rep<NDIM, MINMODE>(A, v, h, T, [&](int rep) {
                uint32_t len = 0;
                int64_t at = (int64_t)np * n + i;
                const uint32_t room = np < kRecPaths ? steps : 0;
                bad |= !walk<NDIM, MINMODE, SRC>(A, P.ptr, rep, [&](int r) {
                    if (len < room) P.rec[at] = r;
                    at += (int64_t)kRecPaths * n;
                    ++len;
                });
                len0 = np == 0 ? len : len0;
                len1 = np == 1 ? len : len1;
                longest = max(longest, len);
                ++np;
                nv += len + 1;  // the saddle, then rep .. maximum
            });
        } else {
            bad = true;
        }
        // the first two paths' lengths (three paths: the third is the rest);
        // none when the saddle has to be walked again
        const bool copied = np <= kRecPaths && longest <= steps;
        A.atmp[i] = make_uint4(np, nv, copied ? len0 : 0u, len1);
        sp += np;
        sv += nv;
    }
    block_sum2<BT>(sp, sv, tmp);
    const int any_bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) {
        A.bsum[kSumRow + blk] = sp;
        A.bsum[2 * kSumRow + blk] = sv;
        A.bsum[3 * kSumRow + blk] = any_bad != 0;
    }
}

template <int NDIM, bool MINMODE, int SRC = SRC_F32>
__global__ __launch_bounds__(kPathThreads) __attribute__((amdgpu_waves_per_eu(NDIM == 5 ? 4 : 1, 8))) void k_path_write(OneField sel, PathArgs P)
{
    constexpr int BT = kPathThreads;
    __shared__ RowLds<NDIM, kPathKeys<NDIM>, SRC> T;
    __shared__ uint32_t tmp[8];
    uint32_t blk, nb;
    const ArcArgs A = sel.locate(blk, nb);  // a copy: loop loads cannot alias it
    load_rows(A, T);
    uint32_t lo, hi;
    const uint32_t n = saddle_count(A);
    chunk(n, nb, blk, lo, hi);
    if (lo >= hi && blk != nb - 1) return;  // nothing to write, and not the last block
    uint32_t runp, runv;
    sums_before<BT>(A, 1, blk, tmp, runp, runv);
    for (uint32_t base = lo; base < hi; base += BT) {
        const uint32_t i = base + threadIdx.x;
        const bool valid = i < hi;
        const uint4 c = valid ? A.atmp[i] : make_uint4(0u, 0u, 0u, 0u);
        uint32_t tp, tv;
        uint32_t pk = runp + block_excl_scan<BT>(c.x, tmp, tp);
        uint32_t at = runv + block_excl_scan<BT>(c.y, tmp, tv);
        const int v = valid ? A.saddles[i] : 0;
        if (valid) P.pair_offsets[i] = (int32_t)pk;
        if (valid && (unsigned)v < (unsigned)A.N && c.z != 0) {
            // every path of the saddle is on record (a path has a vertex at least)
            uint32_t left = c.y - c.x;  // recorded vertices of the paths to come
            for (uint32_t k = 0; k < c.x; ++k) {
                const uint32_t len = k == 0 ? c.z : k == 1 ? c.w : left;
                left -= len;
                if (pk <= P.cap_paths) P.path_offsets[pk] = (int32_t)at;
                ++pk;
                if (at < P.cap_vertices) P.vertices[at] = v;
                ++at;
                EG_GPTR(const int32_t) from = P.rec + ((int64_t)k * n + i);
                for (uint32_t t = 0; t < len; t += 8) {
                    int r[8];
#pragma unroll
                    for (uint32_t j = 0; j < 8; ++j)
                        r[j] = from[(int64_t)min(t + j, len - 1) * (kRecPaths * (int64_t)n)];
#pragma unroll
                    for (uint32_t j = 0; j < 8; ++j)
                        if (t + j < len && at + t + j < P.cap_vertices) P.vertices[at + t + j] = r[j];
                }
                at += len;
            }
        } else if (valid && (unsigned)v < (unsigned)A.N) {
            const auto h = load_nbhd<NDIM, MINMODE>(A, v, T);
            for_each_rep<NDIM, MINMODE>(A, v, h, T, [&](int rep) {
                if (pk <= P.cap_paths) P.path_offsets[pk] = (int32_t)at;
                ++pk;
                if (at < P.cap_vertices) P.vertices[at] = v;
                ++at;
                walk<NDIM, MINMODE, SRC>(A, P.ptr, rep, [&](int r) {
                    if (at < P.cap_vertices) P.vertices[at] = r;
                    ++at;
                });
            });
        }
        runp += tp;
        runv += tv;
    }
    // the last block has seen every count: closing entries of both offset
    // arrays, and the header
    if (blk != nb - 1) return;
    uint32_t bad = 0;
    for (uint32_t i = threadIdx.x; i < nb; i += BT) bad |= A.bsum[3 * kSumRow + i];
    const int any_bad = __syncthreads_or((int)bad);
    if (threadIdx.x != 0) return;
    const uint32_t nsad = A.ctr[C_NSAD];
    P.pair_offsets[saddle_count(A)] = (int32_t)runp;
    if (runp <= P.cap_paths) P.path_offsets[runp] = (int32_t)runv;
    const bool short_ = nsad > A.cap_sad || runp > P.cap_paths || runv > P.cap_vertices;
    P.header[EG_P_STATUS] = A.ctr[C_NAN] ? EG_ERR_NAN : any_bad ? EG_ERR_ARG : short_ ? EG_ERR_CAPACITY : EG_OK;
    P.header[EG_P_PATHS] = (int32_t)runp;
    P.header[EG_P_VERTICES] = (int32_t)runv;
}

template <int NDIM, bool MINMODE, int SRC = SRC_F32>
static void launch_paths_t(const OneField& sel, const PathArgs& p, uint32_t nb, hipStream_t s)
{
    hipLaunchKernelGGL((k_path_count<NDIM, MINMODE, SRC>), dim3(nb), dim3(kPathThreads), 0, s, sel, p);
    hipLaunchKernelGGL((k_path_write<NDIM, MINMODE, SRC>), dim3(nb), dim3(kPathThreads), 0, s, sel, p);
}

hipError_t launch_paths(const ArcArgs& a, const PathArgs& p, hipStream_t s)
{
    // walks are chains of dependent loads: one block per 256 saddle slots
    // keeps as many in flight as there are saddles, and evens out their lengths
    // (1.95 M saddles in noise: 1.36 ms in 8192 blocks, 1.52 in 4096)
    ArcArgs ap = a;
    const int64_t want = ((int64_t)a.cap_sad + 255) / 256;
    const int64_t nbp = want < kSumRow ? want : kSumRow;
    if (nbp > ap.arc_blocks) ap.arc_blocks = (int32_t)nbp;
    const OneField sel{ap};
    const uint32_t nb = (uint32_t)ap.arc_blocks;
    if (a.dtype != EG_F32) {
        if (a.ndim != 3) return hipErrorInvalidValue;
        const bool wide = sample_source(a.dtype) == SRC_WIDE;
        if (a.minima) {
            if (wide)
                launch_paths_t<3, true, SRC_WIDE>(sel, p, nb, s);
            else
                launch_paths_t<3, true, SRC_INT>(sel, p, nb, s);
        } else {
            if (wide)
                launch_paths_t<3, false, SRC_WIDE>(sel, p, nb, s);
            else
                launch_paths_t<3, false, SRC_INT>(sel, p, nb, s);
        }
        return hipGetLastError();
    }
#define EG_CASE(N)                                    \
    case N:                                           \
        if (a.minima)                                 \
            launch_paths_t<N, true>(sel, p, nb, s);   \
        else                                          \
            launch_paths_t<N, false>(sel, p, nb, s);  \
        break;
    switch (a.ndim) {
        EG_CASE(1)
        EG_CASE(2)
        EG_CASE(3)
        EG_CASE(4)
        EG_CASE(5)
        EG_CASE(6)
        default:
            return hipErrorInvalidValue;
    }
#undef EG_CASE
    return hipGetLastError();
}

// ------------------------------------------------------------------ launchers

// Blocks per field of the stage (d) kernels: one per kArcVertsPerBlock
// vertices; a small field still gets up to 64 blocks (one per 1024 vertices),
// so that its saddles spread over the GPU instead of queueing in a few blocks.
uint32_t arc_blocks(int64_t N)
{
    int64_t b = (N + kArcVertsPerBlock - 1) / kArcVertsPerBlock;
    if (b < 64) b = std::min<int64_t>(64, (N + 1023) / 1024);
    return (uint32_t)(b < 1 ? 1 : b > kArcBlocks ? kArcBlocks : b);
}

ArcArgs arc_args(const float* f, const Grid& g, const eg_out& o, const Work& w)
{
    ArcArgs a{};
    a.f = gptr(f);
    a.keys = gptr<const uint32_t>(w.keys);
    a.lab = gptr<const int32_t>(o.labels);
    a.mmask = gptr<const uint64_t>(w.mmask);
    a.smask = gptr<const uint64_t>(w.smask);
    a.bsum = gptr(w.bsum);
    a.atmp = gptr(w.atmp);
    a.ctr = gptr(w.ctr);
    a.header = gptr(o.header);
    a.maxima = gptr(o.maxima);
    a.saddles = gptr(o.saddles);
    a.beta = gptr(o.saddle_beta);
    a.offsets = gptr(o.arc_offsets);
    a.arcs = gptr(o.arc_maxima);
    a.ndim = g.ndim;
    a.minima = (o.flags & EG_MINIMA) ? 1 : 0;
    a.N = g.N;
    a.X = g.dims[g.ndim - 1];
    a.XW = (a.X + 63) / 64;
    a.words = (int32_t)w.words;
    for (int i = 0; i < EG_MAX_NDIM; ++i) a.dims[i] = i < g.ndim ? g.dims[i] : 1;
    a.cap_max = (uint32_t)o.cap_max;
    a.cap_sad = (uint32_t)o.cap_sad;
    a.cap_arc = (uint32_t)o.cap_arc;
    a.arc_blocks = (int32_t)arc_blocks(g.N);
    return a;
}

template <int NDIM, bool MINMODE, int SRC = SRC_F32>
static void launch_arc_pair(const OneField& sel, uint32_t nb, hipStream_t s)
{
    hipLaunchKernelGGL((k_arc_count<NDIM, MINMODE, SRC>), dim3(nb), dim3(kArcThreads<NDIM>), 0, s, sel);
    hipLaunchKernelGGL((k_arc_write<NDIM, MINMODE, SRC>), dim3(nb), dim3(kArcThreads<NDIM>), 0, s, sel);
}

hipError_t launch_arcs(const ArcArgs& a, hipStream_t s)
{
    const OneField sel{a};
    const uint32_t nb = (uint32_t)a.arc_blocks;
    hipLaunchKernelGGL(k_mask_count<OneField>, dim3(nb), dim3(256), 0, s, sel);
    hipLaunchKernelGGL(k_mask_emit<OneField>, dim3(nb), dim3(256), 0, s, sel);
    if (a.dtype != EG_F32) {
        if (a.ndim != 3) return hipErrorInvalidValue;
        const bool wide = sample_source(a.dtype) == SRC_WIDE;
        if (a.minima) {
            if (wide)
                launch_arc_pair<3, true, SRC_WIDE>(sel, nb, s);
            else
                launch_arc_pair<3, true, SRC_INT>(sel, nb, s);
        } else {
            if (wide)
                launch_arc_pair<3, false, SRC_WIDE>(sel, nb, s);
            else
                launch_arc_pair<3, false, SRC_INT>(sel, nb, s);
        }
        return hipGetLastError();
    }
#define EG_CASE(N)                                  \
    case N:                                         \
        if (a.minima)                               \
            launch_arc_pair<N, true>(sel, nb, s);   \
        else                                        \
            launch_arc_pair<N, false>(sel, nb, s);  \
        break;
    switch (a.ndim) {
        EG_CASE(1)
        EG_CASE(2)
        EG_CASE(3)
        EG_CASE(4)
        EG_CASE(5)
        EG_CASE(6)
        default:
            return hipErrorInvalidValue;
    }
#undef EG_CASE
    return hipGetLastError();
}

hipError_t launch_arcs_batched(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s)
{
    const BatchFields sel{gptr(dplan)};
    const unsigned grid = (unsigned)hplan.total_arc_blocks;
    hipLaunchKernelGGL(k_mask_count<BatchFields>, dim3(grid), dim3(256), 0, s, sel);
    hipLaunchKernelGGL(k_mask_emit<BatchFields>, dim3(grid), dim3(256), 0, s, sel);
    hipLaunchKernelGGL(k_arc_batched<false>, dim3(grid), dim3(256), 0, s, sel);
    hipLaunchKernelGGL(k_arc_batched<true>, dim3(grid), dim3(256), 0, s, sel);
    return hipGetLastError();
}

}  // namespace eg
