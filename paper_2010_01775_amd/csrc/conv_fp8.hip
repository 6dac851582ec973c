// The FP8 (e4m3) convolution tiles (conv_tile.h).
#include <algorithm>

#include "conv_tile.h"

hipError_t launch_tile_fp8(TileArgs a, TileShape t, int kc, TileIn in, hipStream_t s) {
  return launch_tile_any<TileFP8>(a, t, kc, in, s);
}
