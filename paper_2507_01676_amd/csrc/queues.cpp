// Kernel choice and run queues of a plan's gather slices (queues.hpp).
#include "queues.hpp"

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

namespace embx {

int lanes_per_row(int32_t R) {
  int g = 1;
  while (g * 16 < R) g <<= 1;
  return g;
}

bool gather_only(const PlanOut& P) {
  for (const PSlice& x : P.slices)
    if (x.strat != S_GATHER) return false;
  return true;
}

// Gather-only plans take at least two lanes per row (of a 16-byte row the second idles).
// Alone, a lane would hold all the ids, weights and bag ends that a SW's lanes share: such
// kernels spilled 300-500 registers, and their scratch costs each launch several us.  One
// lane against two: 8 tables of 4332 one-lookup fp16 bags 10.8 -> 5.0 us, 12 weighted tables
// at batch 1 24.1 -> 13.4, 8M lookups in bags of 40 75.0 -> 72.3, 49.6 in fp32 (73.3); fp16
// bags of 8, 1.7M lookups, 26.2 -> 23.4; slower only for 1.7M bags of one lookup whose maximum
// is not stated, 25.2 -> 28.4 and 32.0 -> 35.0 in fp16.  (Long bags: see wave_lanes.)  Staged
// plans keep one lane: their LDS rows lose more by half the SWs (all-LDS fp32 8.3 -> 9.5 ms,
// HOT 62 -> 71 us).
int plan_lanes(const PlanOut& P) {
  return gather_only(P) ? std::max(2, lanes_per_row(P.R)) : lanes_per_row(P.R);
}

bool runs_gather_kernel(const PlanOut& P) {
  const char* env_kernel = std::getenv("EMBX_GATHER_KERNEL");
  const int G = lanes_per_row(P.R);
  // (the kernel offsets a few samples' outputs in 32 bits)
  return (G == 16 || G == 32 || G == 64) && gather_only(P) &&
         static_cast<int64_t>(P.T) * P.E < (int64_t(1) << 28) &&
         !(env_kernel && std::strcmp(env_kernel, "classic") == 0);
}

namespace {

// a slice of the plan, as far as the queues go
struct Item {
  int32_t table, strat, j, k;
  int32_t mode;     // gather: 1 = a wavefront per bag
  int64_t bags;     // at the max batch
  double lookups;   // at the max batch, one per bag at least (divided out once: the rules below
                    // pass over the slices about ten times)
  bool multi;       // gather: more than one lookup per bag may occur
};

}  // namespace

int gather_queues(const QueueIn& in, GatherQueues* q) {
  const PlanOut& P = *in.plan;
  const emb_table_stats_t* stats = in.stats;
  const int64_t* rows = in.rows;
  const int32_t* mean = in.mean;
  const int32_t max_batch = in.max_batch;
  const bool wave_gather = in.wave_gather;
  const bool f16 = P.f16;
  const bool staged = !gather_only(P);
  const int K = P.K, G = plan_lanes(P), block = kBlock;

  // slices in worker order
  std::vector<Item> items;
  std::vector<int32_t> wg_ptr(K + 1, 0);
  items.reserve(P.slices.size());
  for (const PSlice& x : P.slices) {
    const int64_t bags = (static_cast<int64_t>(x.j + 1) * max_batch) / x.k - (static_cast<int64_t>(x.j) * max_batch) / x.k;
    items.push_back(Item{x.t, x.strat, x.j, x.k, 0, bags, static_cast<double>(bags) * std::max(1.0, stats[x.t].mean_pooling),
                         x.strat == S_GATHER && stats[x.t].max_pooling != 1});
    wg_ptr[x.wg + 1] += 1;
  }
  for (int w = 0; w < K; ++w) wg_ptr[w + 1] += wg_ptr[w];
  // Gather slices share their worker's SW pool, so for them a bag is long when it
  // holds more lookups than one SW's share of the worker's gather lookups.
  for (int w = 0; w < K; ++w) {
    double Wg = 0.0;
    for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i) {
      const Item& d = items[i];
      if (d.strat != S_GATHER) continue;
      Wg += d.lookups;
    }
    for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i) {
      Item& d = items[i];
      if (d.strat != S_GATHER) continue;
      const double s_t = stats[d.table].mean_pooling;
      d.mode = (s_t >= 4.0 * (64 / G) && s_t * (kBlock / G) > Wg) ? 1 : 0;
    }
  }

  // Long bags of 16-byte rows are walked with one lane per row, 64 rows per load of a wavefront,
  // where most of the wave-mode lookups are in bags of 256 or more (5000 lookups: 20.9 us on two
  // lanes, 13.7 on one; 1000: 7.0 and 5.8; 300: 5.2 and 4.9; 9.75M lookups in bags of 150: 65 and
  // 70).  These are kernels of their own: with both walkers in one, the two-lane bags of 100
  // fp16 lookups ran 82.5 us instead of 72.5.
  q->wave_lanes = G;
  if (!staged && P.R <= 16) {
    double in_wave = 0.0, in_long = 0.0;
    for (const Item& d : items)
      if (d.mode) {
        in_wave += d.lookups;
        if (stats[d.table].mean_pooling >= 256.0) in_long += d.lookups;
      }
    if (in_long > 0.0 && in_long >= 0.5 * in_wave) q->wave_lanes = 1;
  }

  // gather run queues per worker, slices in plan order: wave-mode runs, then runs of
  // tables whose bags hold at most one lookup (kChunkSingle bags per chunk: one step
  // of a SW), then the other runs.  Of these, chunks that SWs walk carry about sqrt(5 W / NSW)
  // expected lookups (W: the worker's lookups in this queue at the max batch), at least one full
  // step (8) and at most 128; chunks for matrix slots see narrow_chunks.  Wave-mode chunks carry
  // about four wavefront steps of lookups, fewer when that leaves some of the 16 wavefronts
  // without one.
  //
  // The wave-uniform gather kernel's queues are single-lookup bags (chunks of one wavefront
  // step: ksteps S bags) and all other bags, in chunks of a wavefront's share of what is left
  // (wave_chunks): from half a step to 128 expected lookups, 192 when the worker's queue gives
  // each wavefront at least 64 chunks (W / 16 >= 64 * 192), or two steps if that is more, and
  // at most 64 bags (EMBX_WAVE_CHUNK overrides the share).  The cap, measured on workload 5
  // when every chunk had its size: 4358 us at 64 lookups, 4042 at 192, 4170 at 512 -- shorter
  // chunks keep a worker's wavefronts on fewer tables at a time, so their rows share L2; much
  // shorter ones pay the per-chunk start.
  const char* env_chunk = std::getenv("EMBX_WAVE_CHUNK");
  const double wave_chunk_override = env_chunk ? std::atof(env_chunk) : 0.0;
  // Rows in flight per step of the wave-uniform gather kernel (one build per choice): the
  // choice with the fewest row rounds -- a chunk of c expected lookups takes ceil(c / N)
  // steps of N = ks S lookups -- over the plan's multi-lookup chunks, ties to the larger
  // (more rows in flight for the same rounds); plans without such chunks keep 12 (their
  // single-lookup chunks are one step each, and larger steps make fewer of them).  Measured
  // (12 / 13 / 16): workload 4's 100-lookup chunks (two bags of 50) take 3 / 2 / 2 steps and
  // ran 14.36 / 14.03 / 13.92 us and, in a second session, 14.08 / 13.86 / 13.75 us; workload 5
  // (chunks of ~180 lookups, N = 2 ks) 3966 / 3949 / 3929 us; workload 3 119.3 / 119.9 /
  // 119.1 us; workload 2, single-lookup bags only, 5.30 / 5.36 / 5.51 us.
  // EMBX_GATHER_STEPS = 12, 13 or 16 overrides it.
  int ksteps = 12;
  // Bags per chunk of worker w's multi-lookup items for steps of N lookups (item_cb): as many
  // lookups as each wavefront's share of what is left of the queue, so that a queue shorter
  // than 16 full chunks still occupies all 16 wavefronts and a longer one ends in small
  // chunks; not below half a step (or the share of the whole queue), where a chunk's start
  // costs more than it evens out, nor above the cap described above; at most 64 bags, the bag
  // ends a wavefront holds.  Measured against the cap alone: 60k lookups of 1-KB rows (15 per
  // wavefront) 19.5 -> 12.6 us, 717k lookups of 384-byte rows 34.2 -> 33.6 us, 3.4M lookups of
  // 256-byte rows 108.9 -> 107.5 us; half or twice the share: within 2% of it.
  std::vector<int32_t> item_cb(items.size(), 1);
  // (lookup_kernel's wave-mode slices have a queue of their own)
  auto multi_lookup = [&](const Item& d) { return d.multi && (wave_gather || !d.mode); };
  auto bag_lookups = [&](const Item& d) { return std::max(1.0, stats[d.table].mean_pooling); };
  auto wave_chunks = [&](int w, double N) {
    const int nwaves = block / 64;
    double W = 0.0;
    for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i)
      if (multi_lookup(items[i])) W += items[i].lookups;
    const double cap = std::max(2.0 * N, W / nwaves >= 64.0 * 192.0 ? 192.0 : 128.0);
    const double least = std::min(0.5 * N, W / nwaves);
    double left = W;
    for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i) {
      const Item& d = items[i];
      if (!multi_lookup(d)) continue;
      const double target = wave_chunk_override > 0.0 ? wave_chunk_override
                                                      : std::min(cap, std::max(least, left / nwaves));
      item_cb[i] = static_cast<int32_t>(std::min(64.0, std::max(1.0, std::floor(target / bag_lookups(d)))));
      left -= d.lookups;
    }
  };
  // Narrow rows are summed in matrix slots by whole wavefronts or by SWs one by one: fp32 rows of
  // 2 to 8 lanes, fp16 rows of 2 (see launch_slots).  In slots a chunk is bags of one slice, one
  // or more per SW, so the slices must hold bags for half of a wavefront's S SWs (1.6M lookups in
  // bags of 8, 30 per slice: 18.1 us against 25.0; bags of 30, 3 per slice of 800 queries: 19.9
  // against 15.6).  fp16 rows of 64 and 128 bytes stay with the SWs: in slots they also pay
  // conversions, which cost more than the slots save (26 tables: bags of 2 at 1000 to 3000 queries
  // 5.0-10.4 us by SWs, 6.4-15.0 in slots; bags of 8 at 8192 queries 27.6 against 27.3 and 38.2
  // against 40.7, and 11.9-12.4 against 14.8-15.2 where such a plan is called with 64 queries).
  if (!wave_gather && !staged && (G == 2 || (!f16 && (G == 4 || G == 8)))) {
    const double S = 64.0 / G;
    double bags = 0.0, lookups = 0.0, filled = 0.0;
    for (const Item& d : items)
      if (multi_lookup(d)) {
        const double n = d.lookups, nb = n / bag_lookups(d);
        bags += nb;
        lookups += n;
        filled += n * std::min(1.0, nb / S);
      }
    q->slots = bags > 0.0 && filled >= 0.5 * lookups;
  }
  // The same for the rows that lookup_kernel walks in matrix slots, whose chunks are S = 64 / G SWs
  // of 1 to min(4, G) bags each: the wavefront's share of what is left of the queue, and at least
  // the bags that one step of kSlotStep lookups per SW holds, which cost no more than one bag (26
  // tables at 2500 queries, 128-byte rows: bags of 1 9.4 -> 5.9 us, of 2 9.9 -> 6.2, 5.8 and 6.7 by
  // SWs; 64-byte rows, 8 tables at 24000 queries: bags of 2 10.2 -> 7.3, 7.8 by SWs).  Bags of one
  // lookup on 32-byte rows fill two of a step's eight rows: 624k of them 15.4 us, 13.8 by SWs (where
  // lengths vary about a mean of 1, 0.6 of the SWs' time).
  auto narrow_chunks = [&](int w) {
    const int S = 64 / G, M = std::min(4, G), nwaves = block / 64;
    double left = 0.0;
    for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i)
      if (multi_lookup(items[i])) left += items[i].lookups;
    for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i) {
      const Item& d = items[i];
      if (!multi_lookup(d)) continue;
      const double share = std::floor(left / (nwaves * S * bag_lookups(d)));
      const double step = std::max(1.0, std::floor(kSlotStep / bag_lookups(d)));
      item_cb[i] = S * static_cast<int32_t>(std::min(static_cast<double>(M), std::max(step, share)));
      left -= d.lookups;
    }
  };
  if (wave_gather) {
    const char* env_steps = std::getenv("EMBX_GATHER_STEPS");
    if (env_steps && *env_steps) {
      ksteps = std::atoi(env_steps);
      bool known = false;
      for (int c : kGatherStepChoices) known = known || c == ksteps;
      if (!known) {
        return EMB_ERR_INVALID_ARGUMENT;
      }
    } else {
      double best = -1.0;
      for (int cand : kGatherStepChoices) {
        const double N = static_cast<double>(cand) * (64 / G);
        double rounds = 0.0;
        for (int w = 0; w < K; ++w) {
          wave_chunks(w, N);
          for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i) {
            const Item& d = items[i];
            if (!multi_lookup(d)) continue;
            const double s_t = bag_lookups(d), cb = item_cb[i];
            const double nc = std::ceil(static_cast<double>((static_cast<int64_t>(max_batch) + d.k - 1) / d.k) / cb);
            rounds += nc * std::ceil(cb * s_t / N);
          }
        }
        if (best < 0.0 || rounds <= best) {   // candidates ascend: ties go to the larger
          best = rounds;
          ksteps = cand;
        }
      }
      if (best == 0.0) ksteps = 12;   // no multi-lookup chunks
    }
  }
  std::vector<GatherRun> gr;                       // runs, worker-major
  std::vector<int32_t> gr_ptr(K + 1, 0);
  std::vector<GatherSlotHeader> gr_head(K);
  int max_runs = 0;
  {
    const int nsw = kBlock / G;
    const int nwaves = block / 64;
    const double wave_chunk = 4.0 * 8.0 * (64 / q->wave_lanes);
    // Slice j of k holds floor((j+1)B/k) - floor(jB/k) bags at the runtime batch B, which
    // for some B < max_batch is one more than at max_batch (e.g. k = 256, j = 10: 3 bags at
    // B = 1000, 4 at B = 792).  Every B <= max_batch gives at most ceil(max_batch / k), so a
    // run gets chunks for that many; chunks past the slice at the runtime batch are empty
    // and skipped by the kernel's queue.
    auto slice_bags_any = [&](const Item& d) -> int64_t {
      return (static_cast<int64_t>(max_batch) + d.k - 1) / d.k;
    };
    for (int w = 0; w < K; ++w) {
      double Ws = 0.0, Ww = 0.0;
      // classes, in queue order: 0 wave mode, 1 single-lookup bags, 2 SW mode.  Only a
      // table whose statistics state a maximum of one lookup per bag is single-lookup; an
      // unknown maximum (0) walks in SW mode
      auto class_of = [&](const Item& d) -> int {
        if (d.mode && !wave_gather) return 0;
        return stats[d.table].max_pooling == 1 ? 1 : 2;
      };
      for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i) {
        if (items[i].strat != S_GATHER) continue;
        const double lk = items[i].lookups;
        const int cls = class_of(items[i]);
        if (cls == 0)
          Ww += lk;
        else if (cls == 2)
          Ws += lk;
      }
      // SW-mode chunks are claimed dynamically: a chunk boundary costs about five lookups
      // of a SW's time and the worker's tail is up to one chunk, so ~sqrt(5 W / NSW)
      // lookups per chunk balances the two; measured, chunks past ~128 lookups lose again
      // (the SWs then work on fewer tables at a time), hence the cap
      const double target = std::min(128.0, std::max(8.0, std::floor(std::sqrt(5.0 * Ws / nsw))));
      if (wave_gather) wave_chunks(w, static_cast<double>(ksteps) * (64 / G));
      else if (q->slots) narrow_chunks(w);
      const double wtarget = std::min(wave_chunk, std::max(1.0, std::floor(Ww / nwaves)));
      gr_ptr[w] = static_cast<int32_t>(gr.size());
      int64_t base[3] = {0, 0, 0}, slot_base = 0;
      int32_t nrun[3] = {0, 0, 0};
      for (int cls = 0; cls < 3; ++cls) {
        for (int32_t i = wg_ptr[w]; i < wg_ptr[w + 1]; ++i) {
          const Item& d = items[i];
          if (d.strat != S_GATHER || class_of(d) != cls) continue;
          const double s_t = std::max(1.0, stats[d.table].mean_pooling);
          const int32_t cb = cls == 1 ? (wave_gather ? ksteps * (64 / G) : kChunkSingle)
                             : cls == 2 && (wave_gather || (q->slots && !f16)) ? item_cb[i]
                                      : static_cast<int32_t>(std::max(1.0, std::floor((cls == 0 ? wtarget : target) / s_t)));
          const int64_t nc = (slice_bags_any(d) + cb - 1) / cb;
          if (nc == 0) continue;
          GatherRun r{};
          r.w = nullptr;
          r.rows = rows[d.table];
          r.table = d.table;
          r.j = d.j;
          r.k = d.k;
          r.cb = cb;
          r.chunk_base = static_cast<int32_t>(base[cls]);
          r.mean = mean[d.table];
          if (cls == 2 && q->slots) {
            r.slot_cb = item_cb[i];
            r.slot_base = static_cast<int32_t>(slot_base);
            slot_base += (slice_bags_any(d) + r.slot_cb - 1) / r.slot_cb;
          }
          gr.push_back(r);
          base[cls] += nc;
          nrun[cls] += 1;
        }
      }
      // the worker's header and runs are copied into LDS (all of a workgroup's LDS but
      // the kernel's own static variables)
      if (base[0] > INT32_MAX || base[1] > INT32_MAX || base[2] > INT32_MAX || slot_base > INT32_MAX ||
          nrun[0] + nrun[1] + nrun[2] > in.run_cap - 1) {
        return EMB_ERR_UNSUPPORTED;
      }
      max_runs = std::max(max_runs, nrun[0] + nrun[1] + nrun[2]);
      for (int cls = 0; cls < 3; ++cls) q->n_runs[cls] += nrun[cls];
      GatherSlotHeader& hd = gr_head[w];
      std::memset(&hd, 0, sizeof hd);
      hd.n_wave = nrun[0];
      hd.wave_chunks = static_cast<int32_t>(base[0]);
      hd.n_single = nrun[1];
      hd.single_chunks = static_cast<int32_t>(base[1]);
      hd.sw_chunks = static_cast<int32_t>(base[2]);
      hd.n_runs = nrun[0] + nrun[1] + nrun[2];
      hd.slot_chunks = static_cast<int32_t>(slot_base);
    }
    gr_ptr[K] = static_cast<int32_t>(gr.size());
  }
  // fixed-size slots, so that a worker fetches its header and runs in one round trip
  q->slot = max_runs + 1;
  q->records.assign(static_cast<size_t>(K) * q->slot, GatherRun{});
  for (int w = 0; w < K; ++w) {
    const size_t s0 = static_cast<size_t>(w) * q->slot;
    std::memcpy(&q->records[s0], &gr_head[w], sizeof(GatherSlotHeader));
    for (int32_t i = gr_ptr[w]; i < gr_ptr[w + 1]; ++i) {
      q->records[s0 + 1 + (i - gr_ptr[w])] = gr[i];
      q->run_at.emplace_back(s0 + 1 + (i - gr_ptr[w]), gr[i].table);
    }
  }
  q->ksteps = wave_gather ? ksteps : 0;
  return EMB_OK;
}

std::string queues_text(const PlanOut& P, bool wave_gather, bool slots, int wave_lanes, int ksteps, int slot,
                        const std::vector<GatherRun>& records) {
  static const char* const names[] = {"wave", "single", "multi"};
  char line[160];
  std::snprintf(line, sizeof line, "kernel %s lanes %d walker %s weighted %s steps %d wave_lanes %d\n",
                wave_gather ? "gather_kernel" : "lookup_kernel", plan_lanes(P),
                wave_gather ? "wavefront" : slots && !P.f16 ? "slots" : "sw",
                wave_gather ? "wavefront" : slots ? "slots" : "sw", ksteps, wave_lanes);
  std::string s = line;
  for (int w = 0; w < P.K; ++w) {
    const GatherRun* const r = &records[static_cast<size_t>(w) * slot];
    GatherSlotHeader hd;
    std::memcpy(&hd, r, sizeof hd);
    for (int i = 0; i < hd.n_runs; ++i) {
      const int cls = i < hd.n_wave ? 0 : i < hd.n_wave + hd.n_single ? 1 : 2;
      std::snprintf(line, sizeof line, "%d %s %d %d %d %d %d\n", w, names[cls], r[1 + i].table, r[1 + i].j, r[1 + i].k,
                    r[1 + i].cb, r[1 + i].slot_cb);
      s += line;
    }
  }
  return s;
}

}  // namespace embx
