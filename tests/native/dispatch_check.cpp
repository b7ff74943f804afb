// Host check of a Dispatcher that holds two plans (csrc/dispatch.cpp): runs alternate between a plan
// of one stream, which the caller enqueues by itself, and one of four, with a backend that records
// calls and one that throws in the middle.  One line per failure; exit status 0 if none.
#include <atomic>
#include <cstdio>
#include <memory>
#include <mutex>
#include <set>
#include <vector>

#include "dispatch.hpp"

namespace psc {
std::unique_ptr<CostModel> mlp_cost_model(const psc_mlp *) { return make_heuristic_cost(); }
}  // namespace psc

using namespace psc;

static int failures = 0;
static void check(bool ok, const char *what, int run) {
  if (ok) return;
  ++failures;
  std::printf("run %d: %s\n", run, what);
}

static SchedPlan plan_of(int streams, int n) {
  SchedPlan p;
  p.n_streams = p.total_streams = streams;
  std::vector<std::vector<int32_t>> deps;
  for (int i = 0; i < n; ++i) {
    Op op;
    op.type = PSC_OP_KERNEL;
    op.kernel = i;
    op.stream = i % streams;
    p.ops.push_back(op);
    deps.push_back(i > 2 ? std::vector<int32_t>{i - 3, i - 1} : std::vector<int32_t>{});
  }
  assign_waits(p, deps);
  return p;
}

struct Recorder final : Backend {
  const SchedPlan &plan;
  int throw_at;
  std::mutex mu;
  std::set<int32_t> execed, recorded;
  std::vector<int32_t> done;
  std::vector<int32_t> last;
  bool ordered = true;
  Recorder(const SchedPlan &p, int t) : plan(p), throw_at(t), last(size_t(p.total_streams), -1) {}
  void wait(int32_t op, int32_t awaited) override {
    std::lock_guard<std::mutex> lk(mu);
    ordered = ordered && recorded.count(awaited) == 1 && execed.count(op) == 0;
  }
  void exec(int32_t op) override {
    std::lock_guard<std::mutex> lk(mu);
    if (op == throw_at) throw Error{PSC_ERR_HIP, "planted"};
    ordered = ordered && last[size_t(plan.ops[size_t(op)].stream)] < op && execed.insert(op).second;
    last[size_t(plan.ops[size_t(op)].stream)] = op;
  }
  void record(int32_t op) override {
    std::lock_guard<std::mutex> lk(mu);
    ordered = ordered && execed.count(op) == 1;
    recorded.insert(op);
  }
  void stream_done(int32_t s) override {
    std::lock_guard<std::mutex> lk(mu);
    done.push_back(s);
  }
};

int main() {
  const SchedPlan one = plan_of(1, 40), four = plan_of(4, 60);
  for (int threads : {1, 2, 4}) {
    Dispatcher d(std::vector<const SchedPlan *>{&one, &four}, threads);
    check(d.threads() == threads, "thread count", -threads);
    for (int run = 0; run < 300; ++run) {
      const int which = (run / 2) % 2 ? run % 2 : 1 - run % 2;
      const SchedPlan &p = which ? four : one;
      const int throw_at = run % 7 == 3 ? int(p.ops.size()) / 2 : -1;
      Recorder r(p, throw_at);
      bool thrown = false;
      try {
        d.run(r, which);
      } catch (const Error &e) {
        thrown = true;
        check(e.status == PSC_ERR_HIP, "another error", run);
      }
      check(thrown == (throw_at >= 0), "error lost or made up", run);
      check(r.ordered, "calls out of order", run);
      check(r.execed.count(throw_at) == 0, "an op that failed counts as enqueued", run);
      if (throw_at < 0) {
        check(r.execed.size() == p.ops.size(), "ops lost", run);
        check(r.done.size() == size_t(p.total_streams), "streams not closed", run);
      }
    }
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
