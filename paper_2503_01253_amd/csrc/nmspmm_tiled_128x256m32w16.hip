// Instantiations of the split kernel for 128 x 256 tiles, 2 x 8 waves of 64 x 32
// (16 waves, four per SIMD: while some wait on their loads or split operands
// the others keep the matrix pipe busy; at most 64 accumulators per lane fit
// the 128 VGPRs).
#include "nmspmm_split.h"
#include "nmspmm_tiles.h"

namespace nmspmm {

using Tile_128x256m32w16 = SplitTile<128, 256, 64>;

hipError_t launch_tiled_128x256m32w16(int BV, int KA, int NQ, const TiledArgs &a, hipStream_t stream)
{
    return BV == 1 ? launch_split_any<Tile_128x256m32w16>(KA, NQ, a, stream) : hipErrorInvalidValue;
}

bool tiled_fits_128x256m32w16(int BV, int KA, int NQ) { return split_fits<Tile_128x256m32w16>(BV, KA, NQ); }

}  // namespace nmspmm
