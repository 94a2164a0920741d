// The expert system's entry point (expert.h).
#include <cmath>

#include "expert.h"

extern "C" cgs_status cgs_expert_system(const double *pc, const cgs_expert_params *ep,
                                        double *b_out, double *delta_out,
                                        double *delta_threads) {
  if (!pc || !b_out || !delta_out) return CGS_EINVAL;
  cgs_expert_params def;
  cgs_default_expert_params(&def);
  const cgs_expert_params &e = ep ? *ep : def;
  if (!(e.inst_reaction >= 0.0 && e.inst_reaction < 1.0) || !(e.cores > 0.0)) return CGS_EINVAL;
  for (int i = 0; i < 24; ++i)
    if (!std::isfinite(pc[i])) return CGS_EINVAL;

  cgs::expert::evaluate(pc, e, b_out, delta_out);
  if (delta_threads) *delta_threads = b_out[17];
  return CGS_OK;
}
