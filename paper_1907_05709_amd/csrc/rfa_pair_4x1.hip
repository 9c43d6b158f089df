// rfa_pair_4x1.hip -- two-step kernel, 4 waves of 1 voxel per lane, nz <= 96.
#include "rfa_pair_kernel.h"

namespace rfa {

RFA_PAIR_LAUNCH(launch_pair_4x1) {
  return launch_store<256, 1, 96>(s, g, b, mode, hi_mid, store, st);
}

RFA_PAIR_BATCH(launch_batch_4x1) {
  return launch_batch<256, 1, 96>(inst, items, first_item, n_items, perf, parity, partials,
                                  st);
}

}  // namespace rfa
