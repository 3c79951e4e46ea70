// Stage 1 with ordinary score stores: few scores, which the next kernel reads.
// The kernel is in index_kernel.h.
#include "index_kernel.h"

int ess_idx::launch_index_kept(const ess_config& c, int T, dim3 grid, hipStream_t st, const IdxArgs& a, hipEvent_t ev_start, hipEvent_t ev_stop) {
  return launch_series<DENSE_KEPT>(c, T, grid, st, a, ev_start, ev_stop);
}
