// eg_sample.h -- keys of the sample types other than float32 (eg_dtype).
//
// Two orders of a sample are used.  exact_key is an unsigned integer with
// exactly the order of the samples.  tile_key is a 32-bit key whose order
// never contradicts it but may make different samples equal: 8- and 16-bit
// integers keep all of theirs, 32-bit integers all but those at the ends (the key
// 0 is taken by positions outside the grid, the keys from kKeyTop up would not
// be finite numbers in the tiles' 64-bit maxima), and the 64-bit types go
// through their nearest float32 (a monotone rounding).  A tile compares the
// 32-bit keys and looks at the samples themselves only where two of them meet
// and some key of the tile is not exact.  Tiles whose samples lie close
// together (plateaus, a large offset with small differences) take the distances
// of the exact keys from one of them as their keys.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "eg_internal.h"

namespace eg {

// Where a kernel's samples come from.
enum : int {
    SRC_F32 = 0,   // float32, or the stored order keys
    SRC_INT = 1,   // 8- and 16-bit integers: the 32-bit key is exact
    SRC_WIDE = 2,  // 32- and 64-bit integers and float64
};

__host__ __device__ inline int sample_source(int dtype)
{
    return dtype == EG_F32 ? SRC_F32 : dtype >= EG_I8 && dtype <= EG_U16 ? SRC_INT : SRC_WIDE;
}
__host__ __device__ inline int sample_size(int dtype)
{
    return dtype == EG_I8 || dtype == EG_U8     ? 1
           : dtype == EG_I16 || dtype == EG_U16 ? 2
           : dtype == EG_F32 || dtype == EG_I32 || dtype == EG_U32 ? 4
                                                                   : 8;
}

// Tile keys lie in [1, kKeyTop - 1]; in the minimum graph a key k becomes
// kKeyTop - k, or the key of the negated number.
constexpr uint32_t kKeyTop = 0xFFE00000u;

// An order-preserving key of the bit pattern of a float32, in four or five
// instructions: negative values map to -b, the others to b | 2^31, so -0 and
// +0 meet at 2^31 and the order of the numbers is kept (keys of the same value
// are equal, the index decides); the top is clamped, so every vertex key is
// below kKeyTop and the key 0 of positions outside the grid stays below all of
// them, NaN included: no pointer can leave the grid.  The minimum graph takes
// the key of the negated number.
template <bool MINMODE>
__device__ __forceinline__ uint32_t bits_key(uint32_t b)
{
    if (MINMODE) b ^= 0x80000000u;
    const uint32_t m = (uint32_t)((int32_t)b >> 31);
    return min((b ^ (m | 0x80000000u)) - m, kKeyTop - 1u);
}

template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(double x)
{
    return bits_key<MINMODE>(__float_as_uint((float)x));
}
template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(int64_t x)
{
    return bits_key<MINMODE>(__float_as_uint((float)x));
}
template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(uint64_t x)
{
    return bits_key<MINMODE>(__float_as_uint((float)x));
}
template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(uint32_t x)
{
    const uint32_t k = min(max(x, 1u), kKeyTop - 1u);
    return MINMODE ? kKeyTop - k : k;
}
template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(int32_t x)
{
    return tile_key<MINMODE>((uint32_t)x ^ 0x80000000u);
}
// 8- and 16-bit integers
template <bool MINMODE, class T>
__device__ __forceinline__ uint32_t tile_key_int(T x)
{
    const uint32_t k = (uint32_t)((int)x + 32769);
    return MINMODE ? kKeyTop - k : k;
}
template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(int8_t x) { return tile_key_int<MINMODE>(x); }
template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(uint8_t x) { return tile_key_int<MINMODE>(x); }
template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(int16_t x) { return tile_key_int<MINMODE>(x); }
template <bool MINMODE>
__device__ __forceinline__ uint32_t tile_key(uint16_t x) { return tile_key_int<MINMODE>(x); }

// The 32-bit key of vertex v of a field of 8- or 16-bit integers.
template <bool MINMODE>
__device__ __forceinline__ uint32_t int_key(EG_GPTR(const float) f, int dtype, int64_t v)
{
    int x;
    if (dtype == EG_U8)
        x = ((EG_GPTR(const uint8_t))f)[v];
    else if (dtype == EG_I8)
        x = ((EG_GPTR(const int8_t))f)[v];
    else if (dtype == EG_U16)
        x = ((EG_GPTR(const uint16_t))f)[v];
    else
        x = ((EG_GPTR(const int16_t))f)[v];
    return tile_key_int<MINMODE>(x);
}

// Unsigned integers with exactly the order of the samples (-0 meets +0).
__device__ __forceinline__ uint64_t exact_of(double x)
{
    const uint64_t k = (uint64_t)__double_as_longlong(x + 0.0);
    return k ^ ((uint64_t)((int64_t)k >> 63) | (uint64_t(1) << 63));
}
__device__ __forceinline__ uint64_t exact_of(int64_t x) { return (uint64_t)x ^ (uint64_t(1) << 63); }
__device__ __forceinline__ uint64_t exact_of(uint64_t x) { return x; }
__device__ __forceinline__ uint64_t exact_of(int32_t x) { return (uint32_t)x ^ 0x80000000u; }
__device__ __forceinline__ uint64_t exact_of(uint32_t x) { return x; }

// The zero of a tile's distance keys (x - base, in [1, kKeyTop - 1]) for a tile
// whose first sample is `first`: 2^31 below it, so that samples on either side
// of it are in reach, but kept inside the range of 64 bits.  No distance in
// reach then wraps: from 2^64 - 1 (one below 0) every x but the largest keeps
// its order as x + 1, and 2^64 - 1 itself becomes 0, out of reach; from at most
// 2^64 - kKeyTop, an x below the base is at least kKeyTop away.
__host__ __device__ constexpr uint64_t near_base(uint64_t first)
{
    constexpr uint64_t half = uint64_t(1) << 31, top = uint64_t(0) - kKeyTop;
    return first < half ? ~uint64_t(0) : first - half < top ? first - half : top;
}

// Whether samples with this sample's tile_key are all equal to it (a
// sufficient test for the integers).
__device__ __forceinline__ bool key_is_exact(double x) { return (double)(float)x == x; }
__host__ __device__ constexpr bool key_is_exact(int64_t x)
{
    return (uint64_t)x + (uint64_t(1) << 24) <= (uint64_t(1) << 25);
}
__device__ __forceinline__ bool key_is_exact(uint64_t x) { return x <= (uint64_t(1) << 24); }
__device__ __forceinline__ bool key_is_exact(uint32_t x) { return x - 2u <= kKeyTop - 4u; }
__device__ __forceinline__ bool key_is_exact(int32_t x) { return key_is_exact((uint32_t)x ^ 0x80000000u); }

// The exact key of vertex v of a field of a wide type; the minimum graph takes
// the complement.
template <bool MINMODE>
__device__ __forceinline__ uint64_t exact_key(EG_GPTR(const float) f, int dtype, int64_t v)
{
    uint64_t k;
    if (dtype == EG_F64)
        k = exact_of(((EG_GPTR(const double))f)[v]);
    else if (dtype == EG_I64)
        k = exact_of(((EG_GPTR(const int64_t))f)[v]);
    else if (dtype == EG_U64)
        k = ((EG_GPTR(const uint64_t))f)[v];
    else
        k = ((EG_GPTR(const uint32_t))f)[v] ^ (dtype == EG_I32 ? 0x80000000u : 0u);
    return MINMODE ? ~k : k;
}

}  // namespace eg
