// The BF16 convolution tiles (conv_tile.h).
#include <algorithm>

#include "conv_tile.h"

hipError_t launch_tile_bf16(TileArgs a, TileShape t, int kc, TileIn in, hipStream_t s) {
  return launch_tile_any<TileBF16>(a, t, kc, in, s);
}
