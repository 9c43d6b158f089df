// rfa_pair_8x1.hip -- two-step kernel, 8 waves of 1 voxel per lane, nz <= 128.
#include "rfa_pair_kernel.h"

namespace rfa {

RFA_PAIR_LAUNCH(launch_pair_8x1) {
  return launch_store<512, 1, 128>(s, g, b, K, mode, hi_mid, store, st);
}

}  // namespace rfa
