// RMSNorm + projection bias instantiations of the restoration kernel; the translation unit of the tiles
// of 128 rows and of those of 288 and 320 tokens.
#include "restore_kernel.inc"
#include "restore_mid.inc"
#include "restore_wide.inc"

namespace hc {

hipError_t launch_mode1(const RestoreArgs& a, const TileGrid& g, unsigned grid, const LayerBatch* mb,
                        const SplitPlan* sp, hipStream_t stream) {
  return launch_mode<1>(a, g, grid, mb, sp, stream);
}
hipError_t configure_mode1() { return configure_mode<1>(); }

}  // namespace hc
