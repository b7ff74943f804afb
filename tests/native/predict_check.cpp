// Host check of the run prediction (csrc/group.cpp): it ends however long the predicted run is, at
// a time that follows from the launches' own.  Two queues, launches that ask for more than the GPU
// together.  Prints one line per failure; exit status 0 if none.
#include <cmath>
#include <cstdio>
#include <memory>

#include "group.hpp"

namespace psc {
std::unique_ptr<CostModel> mlp_cost_model(const psc_mlp *) { return make_heuristic_cost(); }
}  // namespace psc

using namespace psc;

int main() {
  int failures = 0;
  // launch times of 1 us to 1000 s: where the time so far resolves no better than what is left of a
  // launch, subtracting must not decide whether it has ended
  for (double us = 1.0; us < 2e9; us *= 1.7)
    for (int n : {1, 2, 7, 50}) {
      GroupedPlan gp;
      gp.plan.n_streams = gp.plan.total_streams = 2;
      std::vector<UnitCost> cost;
      double sum[2] = {0, 0};
      for (int i = 0; i < n; ++i)
        for (int q = 0; q < 2; ++q) {
          Op op;
          op.type = PSC_OP_KERNEL;
          op.kernel = int32_t(cost.size());
          op.stream = q;
          gp.plan.ops.push_back(op);
          gp.units.push_back({op.kernel});
          cost.push_back(UnitCost{us * (1.0 + 0.37 * q + 0.011 * i), 0.55 + 0.2 * q});
          sum[q] += cost.back().us;
        }
      assign_waits(gp.plan, std::vector<std::vector<int32_t>>(gp.plan.ops.size()));
      const double got = predict_plan_us(gp, cost, 1.0, 3.0);
      // no faster than each queue alone, no slower than both at their joint rate throughout
      const double least = std::fmax(sum[0], sum[1]), most = 1.3 * (sum[0] + sum[1]) + 10.0 * n;
      if (!(got >= least * (1 - 1e-9) && got <= most)) {
        ++failures;
        std::printf("us %g n %d: %g not in [%g, %g]\n", us, n, got, least, most);
      }
    }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
