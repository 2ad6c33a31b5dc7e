// Rules that choose between forms of a kernel, as plain functions of sizes: no runtime, no device, so that they can be checked anywhere.
#pragma once
#include <cstddef>

namespace br {
namespace rule {

// bf16 outputs of the kernels with one tile of 128x128 or more per workgroup, which take products of any size whose K the persistent
// kernel does not (hidden sizes of an odd multiple of 64).  Up to 160 MB they are stored plainly and the launch that reads them finds
// a part in the memory-side cache; larger ones go past the caches.  Velocity calls of hidden 192, 320, 576, 960, 1344 and 2880, samples of 93
// and 1101 rows, past the caches against plain, by the bytes of the MLP's first layer: 25 to 90 MB 0.960 to 1.066, mean 1.007; 130 and 170 MB
// 0.955 to 1.010, mean 0.996; 250 and 400 MB 0.951 to 1.000, mean 0.975.  (fp32 outputs, the gated residual: the same either way.)
inline bool tile_output_streams(size_t bytes) { return bytes > (size_t)160 << 20; }

}  // namespace rule
}  // namespace br
