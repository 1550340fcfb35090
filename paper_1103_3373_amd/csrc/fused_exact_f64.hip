// Instantiations of the fused kernels with the exact Riemann solver for double:
// hydro_solve_groups only (ghosted groups, one group or a part of one per work
// item), limiter and mode chosen at run time.
#include "fused_exact.hpp"

namespace hy {

hipError_t launch_exact_f64(const FusedArgs<double>& a, int scheme, int recon, const FusedCfg& cfg, hipStream_t st) {
  return exact_launch::launch(a, scheme, recon, cfg, st);
}

}  // namespace hy
