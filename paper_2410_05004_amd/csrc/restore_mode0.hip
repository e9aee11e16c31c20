// RMSNorm instantiations of the restoration kernel, and the launch-shape selection shared by
// all variants.
#include <mutex>
#include <set>

#include "restore_kernel.inc"

namespace hc {

hipError_t launch_mode0(const RestoreArgs& a, const TileGrid& g, unsigned grid, const LayerBatch* mb,
                        const SplitPlan* sp, hipStream_t stream) {
  return launch_mode<0>(a, g, grid, mb, sp, stream);
}
hipError_t configure_mode0() { return configure_mode<0>(); }

// Function attributes are a device's, not a context's: set once per device (84 kernels, some 90 us).
hipError_t configure_kernels() {
  static std::mutex mutex;
  static std::set<int> done;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mutex);
  if (done.count(dev)) return hipSuccess;
  e = configure_mode0();
  if (e == hipSuccess) e = configure_mode1();
  if (e == hipSuccess) e = configure_mode2();
  if (e == hipSuccess) e = configure_mid();
  if (e == hipSuccess) e = configure_stream();
  if (e == hipSuccess) e = configure_wide();
  if (e == hipSuccess) done.insert(dev);
  return e;
}

hipError_t launch_restore(const RestoreArgs& a, const Route& route, LayerBatch* batch, int n_layers, hipStream_t stream) {
  if (route.kind == Route::kMid) return launch_restore_mid(a, route.nb, batch, n_layers, stream);
  if (route.kind == Route::kStream) return launch_restore_stream(a, route.nb, batch, n_layers, stream);
  if (route.kind == Route::kWide) return launch_restore_wide(a, route.nb, batch, n_layers, stream);
  if (route.kind == Route::kSmall) return launch_restore_small(a, route.nb, stream);
  TileGrid g = route.grid;
  const SplitPlan* use_split = route.split ? &route.split_plan : nullptr;
  unsigned grid = 0;
  if (!use_split) {
    grid = (unsigned)choose_tile_grid(2 * a.d_kv_pad / kTileF, (a.n_tok + kTileT - 1) / kTileT, g);
    if (batch) {
      batch->slots_per_layer = (int32_t)grid;
      grid *= (unsigned)n_layers;
    }
  }
  if (a.mode == 0) return launch_mode0(a, g, grid, batch, use_split, stream);
  if (a.mode == 1) return launch_mode1(a, g, grid, batch, use_split, stream);
  return launch_mode2(a, g, grid, batch, use_split, stream);
}

}  // namespace hc
