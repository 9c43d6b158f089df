// rfa_pair_16x2.hip -- two-step kernel, 16 waves of 2 voxels per lane, nz <= 256.
#include "rfa_pair_kernel.h"

namespace rfa {

RFA_PAIR_LAUNCH(launch_pair_16x2) {
  return launch_store<1024, 2, 256>(s, g, b, mode, hi_mid, store, st);
}

RFA_PAIR_BATCH(launch_batch_16x2) {
  return launch_batch<1024, 2, 256>(inst, items, first_item, n_items, perf, parity, partials,
                                  st);
}

}  // namespace rfa
