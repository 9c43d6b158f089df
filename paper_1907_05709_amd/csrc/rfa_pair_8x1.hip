// rfa_pair_8x1.hip -- two-step kernel, 8 waves of 1 voxel per lane, nz <= 128.
#include "rfa_pair_kernel.h"

namespace rfa {

RFA_PAIR_LAUNCH(launch_pair_8x1) {
  return launch_store<512, 1, 128>(s, g, b, mode, hi_mid, store, st);
}

RFA_PAIR_BATCH(launch_batch_8x1) {
  return launch_batch<512, 1, 128>(inst, items, first_item, n_items, perf, parity, partials,
                                  st);
}

}  // namespace rfa
