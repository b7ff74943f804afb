// Launch groups; see group.hpp.
#include "group.hpp"

#include <algorithm>
#include <map>
#include <tuple>

namespace psc {

GroupedPlan group_plan(const Dag &g, const SchedPlan &plan, const std::vector<int32_t> &key,
                       const std::vector<int64_t> &blocks, int64_t max_blocks, bool copies, bool copy_roots,
                       int32_t queues) {
  GroupedPlan gp;
  gp.plan.n_streams = queues;
  gp.plan.total_streams = queues + (plan.total_streams - plan.n_streams);
  auto queue_of = [&](int32_t s) { return s < plan.n_streams ? s % queues : s - plan.n_streams + queues; };
  const size_t n = plan.ops.size(), nk = g.kers.size();
  const std::vector<int32_t> upload_as = upload_buffers(g, copy_roots);
  std::vector<int32_t> h2d_op(g.bufs.size(), -1);
  for (size_t o = 0; o < n; ++o)
    if (plan.ops[o].type == PSC_OP_H2D) h2d_op[plan.ops[o].buffer] = int32_t(o);
  // what an op of the original plan depends on (ids, all smaller than its own)
  std::vector<int32_t> producer(n, -1);  // read-backs: the kernel op that writes their buffer
  for (size_t k = 0; k < nk; ++k)
    for (size_t i = 0, o = size_t(plan.kernel_op[k]) + 1; i < g.iso_out[k].size() && o < n; ++o)
      if (plan.ops[o].type == PSC_OP_D2H && plan.ops[o].buffer == g.iso_out[k][i]) producer[o] = plan.kernel_op[k], ++i;
  auto deps_of = [&](size_t o, std::vector<int32_t> &d) {
    d.clear();
    const Op &op = plan.ops[o];
    if (op.type == PSC_OP_KERNEL) {
      for (int32_t p : g.pred[op.kernel]) d.push_back(plan.kernel_op[p]);
      if (copies)
        for (int32_t b : g.iso_in[op.kernel]) d.push_back(h2d_op[upload_as[b]]);
    } else if (op.type == PSC_OP_D2H) {
      d.push_back(producer[o]);
    }
  };
  struct Open {
    int32_t op;  // the launch's op in gp.plan
    size_t first;
    int64_t blocks;
  };
  std::map<std::tuple<int32_t, int32_t, int32_t>, Open> open;  // (stream, level, key)
  std::vector<int32_t> level(nk, 0);  // longest path from a root
  for (int32_t k : g.bfs_order())
    for (int32_t q : g.succ[k]) level[q] = std::max(level[q], level[k] + 1);
  std::vector<int32_t> new_of(n, -1), d;
  std::vector<std::vector<int32_t>> deps;
  auto emit = [&](const Op &op, size_t o, int32_t kernel) {
    Op x;
    x.type = op.type;
    x.kernel = kernel;
    x.buffer = op.buffer;
    x.stream = queue_of(op.stream);
    x.pos = 0;
    x.host_order = int32_t(gp.plan.ops.size());
    gp.plan.ops.push_back(std::move(x));
    gp.op_of.push_back(int32_t(o));
    deps.emplace_back();
    return new_of[o] = int32_t(gp.plan.ops.size()) - 1;
  };
  for (size_t o = 0; o < n; ++o) {
    const Op &op = plan.ops[o];
    if (op.type != PSC_OP_KERNEL) {
      if (!copies) continue;
      deps_of(o, d);
      const int32_t x = emit(op, o, -1);
      for (int32_t w : d) deps[x].push_back(new_of[w]);
      continue;
    }
    deps_of(o, d);
    const int32_t last = d.empty() ? -1 : *std::max_element(d.begin(), d.end());
    int32_t x = -1;
    const int32_t ky = key[op.kernel];
    if (ky >= 0) {
      auto it = open.find({queue_of(op.stream), level[op.kernel], ky});
      if (it != open.end() && last < int32_t(it->second.first) && it->second.blocks < max_blocks) {
        x = it->second.op;
        it->second.blocks += blocks[op.kernel];
        gp.units[gp.plan.ops[x].kernel].push_back(op.kernel);
        new_of[o] = x;
      }
    }
    if (x < 0) {
      gp.units.push_back({op.kernel});
      x = emit(op, o, int32_t(gp.units.size()) - 1);
      if (ky >= 0) open[{queue_of(op.stream), level[op.kernel], ky}] = Open{x, o, blocks[op.kernel]};
    }
    for (int32_t w : d) deps[x].push_back(new_of[w]);
  }
  assign_waits(gp.plan, deps);
  return gp;
}

double predict_plan_us(const GroupedPlan &gp, const std::vector<UnitCost> &cost, double gap_us, double wait_us) {
  const std::vector<Op> &ops = gp.plan.ops;
  const int32_t T = gp.plan.total_streams;
  std::vector<std::vector<int32_t>> queue(T);
  for (size_t o = 0; o < ops.size(); ++o) queue[ops[o].stream].push_back(int32_t(o));
  std::vector<double> end(ops.size(), -1), left(T, 0), until(T, 0);
  std::vector<double> from(T, 0);  // the queue's next start by its own order
  std::vector<size_t> at(T, 0);
  std::vector<char> running(T, 0);
  for (int32_t q = 1; q < T; ++q) from[q] = wait_us;
  double now = 0, finish = 0;
  for (;;) {
    // start what can start; otherwise the time at which the next one may
    double next = 1e300, asked = 0;
    bool any = false;
    for (int32_t q = 0; q < T; ++q) {
      if (!running[q] && at[q] < queue[q].size()) {
        any = true;
        const int32_t o = queue[q][at[q]];
        double start = from[q];
        for (int32_t w : ops[o].waits) start = end[w] < 0 ? 1e300 : std::max(start, end[w] + wait_us);
        if (start <= now + 1e-9) {
          running[q] = 1;
          left[q] = cost[ops[o].kernel].us;
        } else {
          next = std::min(next, start);
        }
      }
      if (running[q]) {
        any = true;
        asked += cost[ops[queue[q][at[q]]].kernel].share;
      }
    }
    if (!any) return finish;
    const double slow = std::max(1.0, asked);
    // what ends by `next` is decided on the sums themselves: what is left after subtracting can
    // round to a little more than nothing, less than `now` resolves, and time would stand still
    for (int32_t q = 0; q < T; ++q)
      if (running[q]) next = std::min(next, until[q] = now + left[q] * slow);
    if (next > 1e299) return 1e300;  // (not reached: the plan's waits name earlier ops)
    for (int32_t q = 0; q < T; ++q) {
      if (!running[q]) continue;
      left[q] -= (next - now) / slow;
      if (until[q] > next && left[q] > 1e-9) continue;
      running[q] = 0;
      end[queue[q][at[q]++]] = next;
      from[q] = next + gap_us;
      finish = std::max(finish, next + (q ? wait_us : 0.0));
    }
    now = next;
  }
}

}  // namespace psc
