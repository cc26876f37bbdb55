// eg_classify_typed.hip -- classification of 3D fields of the other sample types.
//
// The tile kernel of eg_classify_tiled.hip with the samples read in their own
// type and turned into 32-bit keys on the way into LDS (eg_sample.h).  8- and
// 16-bit integers need nothing else.  A tile of a 32- or 64-bit type whose
// keys cannot be made exact (see stage_samples) notes the vertices whose keys
// leave the order open and classifies those again on the samples.  Ranking the
// whole field into a float32 order surrogate first (eg_order_field, which the
// other dimensions and batches still take) sorts it: 5.8 of 6.6 ms of a build
// of 301 x 384 x 449 smooth float64 samples, which now takes 0.57 ms.  The
// exact tiles matter where the sort had few passes: 256^3 equal float64
// samples 0.32 ms ranked, 0.57 with every vertex looked at again, 0.20 as it
// is; small int64 plateaus 0.48, 0.65 and 0.29.
#include "eg_tile.h"

namespace eg {

template <bool MINMODE, bool PTR, int SRC>
__global__ __launch_bounds__(256) void k_classify3d_typed(TileArgs a)
{
    __shared__ __align__(8) Tile3Lds<kTile3Y, kTile3Z> s;
    tile3d<MINMODE, kTile3Y, kTile3Z, PTR, SRC>(a, xcd_run(blockIdx.x, a.ntiles), s);
}

hipError_t launch_classify_typed(int dtype, const void* f, const Grid& g, bool minima, int32_t* lab, int32_t* ptr,
                                 const Work& w, hipStream_t s)
{
    if (g.ndim != 3 || dtype == EG_F32) return hipErrorInvalidValue;
    TileArgs a = tile_args((const float*)f, g, lab, ptr, w, kTile3Y, kTile3Z);
    a.dtype = (uint32_t)dtype;
    const bool wide = sample_source(dtype) == SRC_WIDE;
#define EG_LAUNCH(MM, SRC)                                                                                 \
    if (ptr)                                                                                               \
        hipLaunchKernelGGL((k_classify3d_typed<MM, true, SRC>), dim3(a.ntiles), dim3(256), 0, s, a);       \
    else                                                                                                   \
        hipLaunchKernelGGL((k_classify3d_typed<MM, false, SRC>), dim3(a.ntiles), dim3(256), 0, s, a);
    if (minima) {
        if (wide) {
            EG_LAUNCH(true, SRC_WIDE)
        } else {
            EG_LAUNCH(true, SRC_INT)
        }
    } else {
        if (wide) {
            EG_LAUNCH(false, SRC_WIDE)
        } else {
            EG_LAUNCH(false, SRC_INT)
        }
    }
#undef EG_LAUNCH
    return hipGetLastError();
}

}  // namespace eg
