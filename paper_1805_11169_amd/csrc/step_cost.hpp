// Estimated device time of one step, for the server's turns.
#pragma once

#include <algorithm>

#include "../../include/icwf.h"

namespace icwf {

// Milliseconds: a launch-bound floor plus the step's flops at a sustained 40
// TFLOP/s (the two-body contraction by the route the simulation takes, with
// `rank` terms; the single-species products and velocities; two complex
// factorisations).  Only ratios between simulations matter: the scheduler
// gives every simulation turns of about the same device time.
inline double step_cost_ms(const icwf_config &c, int route, int rank) {
    const double N = (double)((c.n_traj + 63) / 64 * 64), nr = c.n_r, nR = c.n_R;
    const double pairs = 0.5 * N * (N + 1.0);
    const double table = 4.0 * pairs * nr * nR, products = 4.0 * pairs * (nr + nR) * ((rank + 15) / 16 * 16);
    double contraction = 0.0;
    if (route == ICWF_CONTRACTION_TABLE) contraction = table;
    if (route == ICWF_CONTRACTION_PRODUCTS) contraction = products;
    if (route == ICWF_CONTRACTION_FP32) contraction = 0.5 * table + products;
    const double rest = 28.0 * N * N * (nr + nR) + 2.0 * (8.0 / 3.0) * N * N * N;
    return 0.4 + (contraction + rest) / 4e10;
}

// Steps of a turn: `steps` for the costliest resident simulation (ref_cost),
// proportionally more for cheaper ones, never past the last step.
inline int turn_steps(int steps, double ref_cost, double cost, int left) {
    const double k = std::min(steps * std::max(1.0, ref_cost / cost), 1e6);
    return std::max(1, std::min((int)k, left));
}

}  // namespace icwf
