// Layers over few pixels, their fragments straight from global memory into registers (see conv_igemm_direct).
#pragma once
#include "conv.h"

namespace iodf {

// Kernels of one tile, by epilogue (EPI_ANY, EPI_FAST, EPI_FAST_RELU of conv_dev.h).
struct DirectTile {
    int bc, bp;       // channels x pixels of a workgroup
    int waves;        // which share the reduction
    size_t lds;       // dynamic LDS bytes
    void (*kern[3])(const ConvArgs);
    const char* name;
};
// How the tiles of a launch with `bp` pixels a tile go round the XCDs. Over few pixels the weights are the larger operand
// by far: the channel blocks go round, so that each L2 takes a part of the weights and not all of them. Else whole pixel blocks.
__host__ __device__ inline bool direct_by_pixels(const ConvArgs& a, int bp) {
    return a.npix > 8 * bp && a.npix >= a.n_pad * (int)a.taps;
}
constexpr int kDirectTiles = 3;
extern const DirectTile kDirect[kDirectTiles];

}  // namespace iodf
