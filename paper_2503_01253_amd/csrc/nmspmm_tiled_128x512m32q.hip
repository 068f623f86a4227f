// Instantiations of the tiled kernel for 128 x 512 tiles on the 32x32x2 fp32
// MFMA, 1 x 16 waves of 128 x 32, four per SIMD: the levels of at most 8 compressed
// rows in 128 columns (N/M <= 1/16), whose stages would leave the split
// kernel's K steps of 16 rows half empty.
#include "nmspmm_tiled.h"
#include "nmspmm_tiles.h"

namespace nmspmm {

using Tile_128x512m32q = TileCfg<128, 512, 128, 32, 32>;

hipError_t launch_tiled_128x512m32q(int BV, int KA, int NQ, const TiledArgs &a, hipStream_t stream)
{
    if (BV != 1 || KA != 128) return hipErrorInvalidValue;
    return NQ == 1   ? launch_tiled<Tile_128x512m32q, 1, 128, 1>(a, stream)
           : NQ == 2 ? launch_tiled<Tile_128x512m32q, 1, 128, 2>(a, stream)
                     : hipErrorInvalidValue;
}

bool tiled_fits_128x512m32q(int BV, int KA, int NQ)
{
    static_assert(Shape<Tile_128x512m32q, 1, 128, 1>::FITS && Shape<Tile_128x512m32q, 1, 128, 2>::FITS, "LDS");
    return BV == 1 && KA == 128 && (NQ == 1 || NQ == 2);
}

}  // namespace nmspmm
