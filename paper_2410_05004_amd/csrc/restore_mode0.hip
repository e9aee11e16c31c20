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

// Function attributes are a device's, not a context's: set once per device (56 kernels, some 60 us).
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
  if (e == hipSuccess) done.insert(dev);
  return e;
}

bool restore_would_split(const RestoreArgs& a, SplitPlan& sp, TileGrid& g_main) {
  if (!a.split_ws || a.n_tok <= 0 || restore_route(a, 1).kind != Route::kTiles) return false;
  return plan_split(2 * a.d_kv_pad / kTileF, (a.n_tok + kTileT - 1) / kTileT, a.d_model / (2 * kTileK), a.split_force != 0, sp, g_main);
}

hipError_t launch_restore(const RestoreArgs& a, LayerBatch* batch, int n_layers, hipStream_t stream) {
  if (a.n_tok <= 0) return hipSuccess;
  const Route route = restore_route(a, batch ? n_layers : 1);
  if (route.kind == Route::kMid) return launch_restore_mid(a, route.nb, batch, n_layers, stream);
  if (!batch && route.kind == Route::kSmall) return launch_restore_small(a, route.nb, stream);
  TileGrid g;
  SplitPlan sp;
  const SplitPlan* use_split = nullptr;
  unsigned grid = 0;
  if (!batch && restore_would_split(a, sp, g)) {
    sp.ws = a.split_ws;
    use_split = &sp;
  } else {
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
