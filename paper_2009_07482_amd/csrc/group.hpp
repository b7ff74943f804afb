// Launch groups of a fine schedule: mutually independent kernels of one stream that share a kernel
// function run as one launch.  A queue runs one launch at a time, and the kernels of an attention
// head or a small instance fill a fraction of the GPU for a few microseconds each, so their number
// set a schedule's time.  Measured when they came in, with groups (and the tiles they allow) against
// one launch per kernel: 4-layer 1024 BF16 attention on AQL queues 622 against 1092 us (410 now, with
// the kernels and queue counts since), 1-layer 512 FP32 104 against 161 us (64 now), a batch of
// sixteen BF16 DAGs on HIP streams 1.58 against 3.70 ms (1.10 now).
#pragma once

#include <cstdint>
#include <vector>

#include "core.hpp"

namespace psc {

// A plan whose kernel ops are launch units: op.kernel is an index into `units`, each the kernels
// (ids) one launch runs.
struct GroupedPlan {
  SchedPlan plan;
  std::vector<std::vector<int32_t>> units;
  std::vector<int32_t> op_of;  // per op: the op of the original plan (a unit: its first kernel's)
};

// The launch groups of `plan` (an in-order PSC_FINE plan of `g`).  Two kernels may
// share a launch if they lie on one stream, have the same key (>= 0; -1 = never) and the same level
// (longest path from a root: a kernel of a later level would run ahead of what the plan puts before
// it), and a launch takes no further kernel once its kernels have `max_blocks` workgroups
// (`blocks`, per kernel).  A kernel joins the latest open launch of its stream, level and key if
// every op it depends on comes before that launch's first kernel in host order.  Each launch then stands at its first
// kernel's place, where everything any of its kernels depends on has been enqueued: the order
// stays topological, so no wait can close a cycle, and no two kernels of a launch depend on each
// other.  copies = false leaves the uploads and read-backs out (a run without host memory), so
// that a kernel is not held back by an upload that is skipped.  queues (1 .. plan.n_streams): the
// kernel streams are carried by this many, stream s by s mod queues in host order; copy streams
// follow them.
GroupedPlan group_plan(const Dag &g, const SchedPlan &plan, const std::vector<int32_t> &key,
                       const std::vector<int64_t> &blocks, int64_t max_blocks, bool copies, bool copy_roots,
                       int32_t queues);

// What one launch needs, for the prediction below: microseconds alone on the GPU and the share of
// the GPU it then fills (0, 1].
struct UnitCost {
  double us = 0, share = 1;
};
// Predicted microseconds of a grouped plan without copies: each queue runs its launches one after
// the other `gap_us` apart, a wait for another queue's launch (the run's start and end among them)
// takes wait_us, and launches in flight together that ask for more than the whole GPU slow each
// other down in proportion.
double predict_plan_us(const GroupedPlan &gp, const std::vector<UnitCost> &cost, double gap_us, double wait_us);

}  // namespace psc
