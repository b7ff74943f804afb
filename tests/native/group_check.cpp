// Host check of launch groups (csrc/group.cpp): random DAGs, every mapper, with and without copies.
// Prints one line per failure; exit status 0 if none.
#include <cstdio>
#include <memory>
#include <random>
#include <set>

#include "group.hpp"

namespace psc {
std::unique_ptr<CostModel> mlp_cost_model(const psc_mlp *) { return make_heuristic_cost(); }
}  // namespace psc

using namespace psc;

static int failures = 0;
static void check(bool ok, const char *what, int seed) {
  if (ok) return;
  ++failures;
  std::printf("seed %d: %s\n", seed, what);
}

// Layered DAG of adds over n x n buffers; some operands are windows of a shared host buffer.
static void build(Dag &g, int seed) {
  std::mt19937 r(seed);
  const int nk = 5 + int(r() % 60), span = 1 + int(r() % 12);
  auto buffer = [&](const std::string &name, int64_t rows, int64_t cols, int32_t parent, int64_t c0) {
    Buffer b{};
    b.name = name;
    b.dtype = PSC_F32;
    b.rows = rows;
    b.cols = cols;
    b.parent = parent;
    b.root = parent >= 0 ? parent : int32_t(g.bufs.size());
    b.r0 = 0;
    b.c0 = c0;
    g.bufs.push_back(b);
    g.buf_by_name[name] = int32_t(g.bufs.size()) - 1;
    return int32_t(g.bufs.size()) - 1;
  };
  const int32_t wide = buffer("W", 4, 8 * nk, -1, 0);
  std::vector<int32_t> out;
  for (int k = 0; k < nk; ++k) {
    Kernel ker{};
    ker.name = "k" + std::to_string(k);
    ker.kind = PSC_ADD;
    ker.alpha = 1.0f;
    for (int i = 0; i < 2; ++i) {
      const int src = out.empty() || r() % 3 == 0 ? -1 : int(out.size()) - 1 - int(r() % std::min<size_t>(out.size(), size_t(span)));
      int32_t in;
      if (src >= 0) {
        in = out[size_t(src)];
        if (i == 0 || ker.ins[0] != in) g.edges.push_back(Edge{src, in, k, in});
      } else if (r() % 2) {
        in = buffer("w" + std::to_string(k) + "_" + std::to_string(i), 4, 4, wide, 4 * int64_t(2 * k + i));
      } else {
        in = buffer("h" + std::to_string(k) + "_" + std::to_string(i), 4, 4, -1, 0);
      }
      ker.ins.push_back(in);
    }
    ker.outs.push_back(buffer("o" + std::to_string(k), 4, 4, -1, 0));
    ker.component = int(r() % 5);
    out.push_back(ker.outs[0]);
    g.kers.push_back(ker);
    g.ker_by_name[ker.name] = k;
  }
  g.validate();
}

static void run_all() {
  for (int seed = 0; seed < 400; ++seed) {
    Dag g;
    build(g, seed);
    std::mt19937 r(seed + 10000);
    const int32_t nk = int32_t(g.kers.size());
    std::vector<int32_t> key(nk);
    std::vector<int64_t> blocks(nk);
    for (int32_t k = 0; k < nk; ++k) key[k] = int32_t(r() % 4) - 1, blocks[k] = 1 + int64_t(r() % 40);
    for (int mapper : {int(PSC_MAP_RR), int(PSC_MAP_EFT), int(PSC_MAP_COMPONENT)})
      for (int cs = 0; cs < 2; ++cs)
        for (int roots = 0; roots < 2; ++roots)
          for (int copies = 0; copies < 2; ++copies) {
            psc_sched_opts o{};
            o.n_streams = 1 + int32_t(r() % 5);
            o.mapper = mapper;
            o.copy_stream = cs;
            o.copy_roots = roots;
            const SchedPlan plan = build_plan(g, PSC_FINE, o);
            const int64_t cap = 60;
            const int32_t queues = 1 + int32_t(r() % unsigned(o.n_streams));
            auto queue_of = [&](int32_t st) { return st < o.n_streams ? st % queues : st - o.n_streams + queues; };
            const GroupedPlan gp = group_plan(g, plan, key, blocks, cap, copies != 0, roots != 0, queues);
            const std::vector<Op> &ops = gp.plan.ops;
            const size_t n = ops.size();
            // every kernel once, on its stream; members alike and within the cap
            std::vector<int32_t> at(nk, -1);
            size_t launches = 0;
            for (size_t i = 0; i < n; ++i) {
              if (ops[i].type != PSC_OP_KERNEL) continue;
              ++launches;
              int64_t before_last = 0;
              const auto &u = gp.units[size_t(ops[i].kernel)];
              for (size_t m = 0; m < u.size(); ++m) {
                check(at[u[m]] < 0, "kernel launched twice", seed);
                at[u[m]] = int32_t(i);
                check(queue_of(plan.ops[size_t(plan.kernel_op[u[m]])].stream) == ops[i].stream, "kernel on another stream", seed);
                check(u.size() == 1 || (key[u[m]] == key[u[0]] && key[u[m]] >= 0), "unlike kernels together", seed);
                if (m + 1 < u.size()) before_last += blocks[u[m]];
              }
              check(u.size() == 1 || before_last < cap, "launch above its cap", seed);
            }
            check(launches == gp.units.size(), "units and launches differ", seed);
            for (int32_t k = 0; k < nk; ++k) check(at[k] >= 0, "kernel missing", seed);
            // happens-before of the enqueued structure: stream order and waits, all on earlier ops
            std::vector<std::set<int32_t>> past(n);
            std::vector<int32_t> last(size_t(gp.plan.total_streams), -1);
            auto after = [&](size_t i, int32_t w) {
              past[i].insert(w);
              past[i].insert(past[size_t(w)].begin(), past[size_t(w)].end());
            };
            for (size_t i = 0; i < n; ++i) {
              if (last[size_t(ops[i].stream)] >= 0) after(i, last[size_t(ops[i].stream)]);
              for (int32_t w : ops[i].waits) {
                check(w < int32_t(i), "wait on a later op", seed);
                check(ops[size_t(w)].recorded, "awaited op records no event", seed);
                if (w < int32_t(i)) after(i, w);
              }
              last[size_t(ops[i].stream)] = int32_t(i);
            }
            for (int32_t k = 0; k < nk; ++k)
              for (int32_t q : g.succ[k]) check(past[size_t(at[q])].count(at[k]) == 1, "edge not enforced", seed);
            size_t n_copies = 0;
            const std::vector<int32_t> as = upload_buffers(g, roots != 0);
            std::vector<int32_t> up(g.bufs.size(), -1);
            for (size_t i = 0; i < n; ++i) {
              if (ops[i].type == PSC_OP_KERNEL) continue;
              ++n_copies;
              const Op &orig = plan.ops[size_t(gp.op_of[i])];
              check(orig.type == ops[i].type && orig.buffer == ops[i].buffer && queue_of(orig.stream) == ops[i].stream,
                    "copy changed", seed);
              if (ops[i].type == PSC_OP_H2D) up[size_t(ops[i].buffer)] = int32_t(i);
            }
            size_t want = 0;
            for (const Op &op : plan.ops) want += op.type != PSC_OP_KERNEL;
            check(n_copies == (copies ? want : 0), "copies lost or added", seed);
            if (!copies) {
              // the prediction ends, and counts at least the longest launch and every queue's sum
              std::vector<UnitCost> cost(gp.units.size());
              std::vector<double> sum(size_t(queues), 0.0);
              double least = 0;
              for (size_t u = 0; u < cost.size(); ++u) cost[u] = UnitCost{1.0 + double(r() % 20), 0.1 * (1 + double(r() % 10))};
              for (size_t i = 0; i < n; ++i) sum[size_t(ops[i].stream)] += cost[size_t(ops[i].kernel)].us;
              for (double x : sum) least = std::max(least, x);
              const double us = predict_plan_us(gp, cost, 1.0, 3.0);
              check(us >= least - 1e-6 && us < 1e6, "prediction out of bounds", seed);
              continue;
            }
            for (int32_t k = 0; k < nk; ++k)
              for (int32_t b : g.iso_in[k])
                check(past[size_t(at[k])].count(up[size_t(as[size_t(b)])]) == 1, "kernel not after its upload", seed);
            for (size_t i = 0; i < n; ++i)
              if (ops[i].type == PSC_OP_D2H)
                for (int32_t k = 0; k < nk; ++k)
                  for (int32_t b : g.iso_out[k])
                    if (b == ops[i].buffer) check(past[i].count(at[k]) == 1, "read-back before its kernel", seed);
          }
  }
}

int main() {
  try {
    run_all();
  } catch (const Error &e) {
    check(false, e.msg.c_str(), -1);
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
