// The gather slices of a plan as the kernels walk them: which kernel, how many lanes a row
// takes, and every worker's queues of chunks.  Pure host code (no HIP calls).
#pragma once

#include <cstdint>
#include <string>
#include <utility>
#include <vector>

#include "../../include/embx.h"
#include "device_types.hpp"
#include "planner.hpp"

namespace embx {

int lanes_per_row(int32_t R);
bool gather_only(const PlanOut& P);
// lanes of a row in every kernel this plan launches
int plan_lanes(const PlanOut& P);
// the plan runs gather_kernel (else lookup_kernel)
bool runs_gather_kernel(const PlanOut& P);

struct QueueIn {
  const PlanOut* plan;
  const emb_table_stats_t* stats;   // per table
  const int64_t* rows;
  const int32_t* mean;              // per table: 1 = mean pooling
  int32_t max_batch;
  bool wave_gather;                 // runs_gather_kernel
  int64_t run_cap;                  // records a worker's slot may take in LDS
};

struct GatherQueues {
  bool slots = false;               // the records hold the division for matrix slots (launch_slots)
  int wave_lanes = 0;               // lanes of a row in lookup_kernel's wave mode
  int ksteps = 0;                   // gather_kernel: row loads in flight per lane per step
  int slot = 1;                     // records per worker: a GatherSlotHeader, then its runs
  std::vector<GatherRun> records;   // [K * slot]; table pointers are set at bind
  std::vector<std::pair<size_t, int32_t>> run_at;   // (record, table) of every run
  int32_t n_runs[3] = {0, 0, 0};    // over all workers: wave mode, single-lookup bags, the rest
};

// Whether a launch of such a plan sums its multi-lookup bags in matrix slots.  fp32 rows always.
// fp16 rows of 16 and 32 bytes where they carry weights (12 tables at 8000 to 24000 queries, bags
// of 4 to 20, in shares of the time before slots: 0.50-0.66 and 0.67-0.79 in slots, 0.65-0.80 and
// 0.87-0.94 by SWs; without weights the two are within a tenth of each other) and the batch is at
// least half of the largest, below which the slices run out of bags (26 tables of 8 planned for
// 8192 queries, 32-byte rows with weights: at 1024 queries 18.2 us in slots, 16.0 by SWs; at 4096
// 20.9 and 25.1).
inline bool launch_slots(bool slots, bool f16, bool weighted, int32_t batch, int32_t max_batch) {
  return slots && (!f16 || (weighted && batch >= max_batch - batch));
}

// 0 on success, otherwise an emb_status_t code.
int gather_queues(const QueueIn& in, GatherQueues* out);

// One line of kernel, lanes, walker, steps and lanes in wave mode, then one per run: worker, queue, table, batch
// slice, slices, bags per chunk (of the walker that the line names), and in matrix slots.
std::string queues_text(const PlanOut& P, bool wave_gather, bool slots, int wave_lanes, int ksteps, int slot,
                        const std::vector<GatherRun>& records);

}  // namespace embx
