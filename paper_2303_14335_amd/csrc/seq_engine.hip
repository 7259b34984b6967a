// seq_engine.hip - the sequence engine's lists (seq_types.h): the kernel that
// moves every component's list on after a round, and the host side that
// drives the rounds.  The tasks themselves run in the tiers' own files.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "runtime.h"
#include "seq_types.h"
#include "trace.h"

namespace mpld {

static constexpr int kFoldThreads = 256;
// LDS bytes up to which a component keeps the one-wave tier's layout.
static constexpr int64_t kSeqSmallLds = 16 * 1024;
// The arena that the engine does not start without (bytes).
static constexpr int64_t kSeqLeastArena = 1 << 20;

// Every component starts as one task, its root.
__global__ __launch_bounds__(256) void seq_init_kernel(SeqArgs a) {
  const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i == 0) {
    a.head->arena = 0;
    a.head->tasks = a.ncomps;
    a.head->lost = a.head->ticket = a.head->rounds = 0;
    for (int t = 0; t < kSeqTiers; ++t) {
      a.head->active[t] = a.head->next[t] = a.head->run[1][t] = a.head->pop[0][t] = a.head->pop[1][t] = 0;
      a.head->share[t] = a.least[t];
    }
  }
  if (i >= a.ncomps) return;
  a.results[i].status = kSeqWaiting;
  SeqTask t{};
  t.comp = i;
  t.kind = kSeqRoot;
  t.col = -1;
  a.tasks[i] = t;
  a.lists[(int64_t)i * a.list_cap] = i;
}

struct FoldShared {
  uint64_t sum[kFoldThreads / 64], hash[kFoldThreads / 64];
  int32_t isum[kFoldThreads / 64];
  int32_t stop, cross, cut;
  uint64_t acc, h;
};

__device__ __forceinline__ uint64_t shfl_up64(uint64_t x, int d) {
  return ((uint64_t)(uint32_t)__shfl_up((int)(uint32_t)(x >> 32), d, 64) << 32) |
         (uint32_t)__shfl_up((int)(uint32_t)x, d, 64);
}
__device__ __forceinline__ uint64_t shfl_down64(uint64_t x, int d) {
  return ((uint64_t)(uint32_t)__shfl_down((int)(uint32_t)(x >> 32), d, 64) << 32) |
         (uint32_t)__shfl_down((int)(uint32_t)x, d, 64);
}

// One workgroup per component, a few instructions per list entry; a round's
// lists are some thousands of entries, so the launch is about as long as one.
__global__ __launch_bounds__(kFoldThreads) void seq_fold_kernel(SeqArgs a, const DevDesc* __restrict__ descs,
                                                                int32_t parity) {
  __shared__ FoldShared sh;
  const int32_t tid = (int32_t)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t ci = (int32_t)blockIdx.x;
  SeqComp* cp = a.comps + ci;
  SeqHead* head = a.head;
  if (cp->running) {
    const int32_t* L = a.lists + ((int64_t)parity * a.ncomps + ci) * a.list_cap;
    int32_t* N = a.lists + ((int64_t)(parity ^ 1) * a.ncomps + ci) * a.list_cap;
    const int32_t count = cp->count, tier = cp->tier, share = head->share[tier];
    const uint64_t budget = (uint64_t)descs[cp->pos].budget;
    if (tid == 0) {
      sh.acc = cp->acc;
      sh.h = cp->hash;
      sh.stop = sh.cross = sh.cut = INT32_MAX;
    }
    __syncthreads();
    // ---- the front: counts add up to the first task that has no final count
    int32_t stop = count;
    for (int32_t base = 0; base < count; base += kFoldThreads) {
      const int32_t i = base + tid, t = i < count ? L[i] : -1;
      const int32_t st = t >= 0 ? a.results[t].status : MPLD_INFEASIBLE;
      const bool ran = t >= 0 && st != kSeqWaiting && st != kSeqLost;
      if (t >= 0 && st != MPLD_INFEASIBLE) atomicMin(&sh.stop, i);
      __syncthreads();
      stop = sh.stop;
      const bool in = ran && i <= stop;
      const uint64_t n = in ? a.results[t].nodes : 0;
      uint64_t incl = n;
      for (int off = 1; off < 64; off <<= 1) {
        const uint64_t x = shfl_up64(incl, off);
        if (lane >= off) incl += x;
      }
      if (lane == 63) sh.sum[wave] = incl;
      __syncthreads();
      uint64_t before = sh.acc, total = 0;
      for (int w = 0; w < kFoldThreads / 64; ++w) {
        before += w < wave ? sh.sum[w] : 0;
        total += sh.sum[w];
      }
      incl += before;
      if (in && incl > budget) atomicMin(&sh.cross, i);
      __syncthreads();
      const int32_t cross = sh.cross;
      if (a.trace) {   // traces appended in order: T after S is h(S) B^|T| + h(T)
        uint64_t hn = in && i < cross ? n : 0, h = in && i < cross ? a.results[t].hash : 0;
        for (int off = 1; off < 64; off <<= 1) {
          const uint64_t n2 = shfl_down64(hn, off), h2 = shfl_down64(h, off);
          if ((lane & (2 * off - 1)) == 0) {
            h = trace_concat(h, h2, n2);
            hn += n2;
          }
        }
        if (lane == 0) {
          sh.hash[wave] = h;
          sh.sum[wave] = hn;
        }
        __syncthreads();
        if (tid == 0)
          for (int w = 0; w < kFoldThreads / 64; ++w) sh.h = trace_concat(sh.h, sh.hash[w], sh.sum[w]);
      }
      if (i == cross) {
        cp->cross = t;
        cp->left = budget - (incl - n);
      }
      __syncthreads();
      if (cross != INT32_MAX) break;
      if (tid == 0) sh.acc += total;
      __syncthreads();
      if (stop != INT32_MAX) break;
    }
    const int32_t cross = sh.cross;
    const int32_t front = stop < count ? L[stop] : -1;
    const int32_t fst = front >= 0 ? a.results[front].status : MPLD_INFEASIBLE;
    bool done = true;
    if (cross != INT32_MAX) {
      if (tid == 0) {
        cp->status = MPLD_BUDGET_EXHAUSTED;
        cp->acc = budget;
        cp->hash = sh.h;
      }
    } else if (fst == MPLD_INFEASIBLE || fst == MPLD_FEASIBLE || fst == MPLD_BUDGET_EXHAUSTED) {
      // the end of the list, a solution, or a root that met the whole budget
      if (tid == 0) {
        cp->status = fst;
        cp->acc = sh.acc;
        cp->hash = sh.h;
        cp->depth = fst == MPLD_BUDGET_EXHAUSTED ? a.results[front].depth : 0;
        if (fst == MPLD_FEASIBLE) cp->sol = a.results[front].sol;
      }
    } else {
      // ---- the new list: from the front's task on, pieces in their task's place
      done = false;
      int32_t out = 0;
      bool full = fst == kSeqLost;
      for (int32_t base = stop; base < count && !full; base += kFoldThreads) {
        const int32_t i = base + tid, t = i < count ? L[i] : -1;
        const SeqResult r = t >= 0 ? a.results[t] : SeqResult{MPLD_INFEASIBLE, 0, 0, 0, 0, 0, 0};
        if (t >= 0 && r.status == MPLD_FEASIBLE) atomicMin(&sh.cut, i);   // nothing counts behind it
        __syncthreads();
        const int32_t cut = sh.cut;
        // a cut task's own count stays as an entry, unless the front has just taken it
        const bool self = t >= 0 && i <= cut && !(i == stop && r.status == kSeqCapped);
        const int32_t kids = t >= 0 && i < cut && r.status == kSeqCapped ? r.nchild : 0;
        const int32_t mine = (self ? 1 : 0) + kids;
        int32_t incl = mine;
        for (int off = 1; off < 64; off <<= 1) {
          const int32_t x = __shfl_up(incl, off, 64);
          if (lane >= off) incl += x;
        }
        if (lane == 63) sh.isum[wave] = incl;
        __syncthreads();
        int32_t at = out, total = 0;
        for (int w = 0; w < kFoldThreads / 64; ++w) {
          at += w < wave ? sh.isum[w] : 0;
          total += sh.isum[w];
        }
        at += incl - mine;
        full = out + total > a.list_cap;
        if (!full) {
          const auto put = [&](int32_t task, bool waits) {
            N[at] = task;
            if (waits && at < share) {
              const int32_t s = atomicAdd(&head->run[parity ^ 1][tier], 1);
              if (s < a.run_cap)
                a.runs[(int64_t)((parity ^ 1) * kSeqTiers + tier) * a.run_cap + s] =
                    task | kSeqCut | (at == 0 ? kSeqForce : 0);
            }
            ++at;
          };
          if (self) put(t, r.status == kSeqWaiting);
          for (int32_t j = 0; j < kids; ++j) put(r.child + j, true);
          if (kids || (t >= 0 && r.status == kSeqCapped)) a.results[t].status = MPLD_INFEASIBLE;   // a count now
        }
        out += total;
        __syncthreads();
        if (cut != INT32_MAX) break;
      }
      if (full) {
        done = true;
        if (tid == 0) {
          cp->status = kSeqLost;
          atomicAdd(&head->lost, 1);
        }
      } else if (tid == 0) {
        cp->acc = sh.acc;
        cp->hash = sh.h;
        cp->count = out;
        atomicAdd(&head->next[tier], 1);
      }
    }
    __syncthreads();
    if (done && tid == 0) cp->running = 0;
  }
  if (tid == 0) {
    __threadfence();
    if (atomicAdd(&head->ticket, 1) == a.ncomps - 1) {   // the round's last workgroup
      for (int t = 0; t < kSeqTiers; ++t) {
        const int32_t left = atomicExch(&head->next[t], 0);
        head->active[t] = left;
        head->share[t] = max(a.least[t], left ? a.slots[t] / left : 0);
        head->run[parity][t] = head->pop[parity][t] = 0;
      }
      head->ticket = 0;
      head->rounds += 1;
    }
  }
}

// ---- host side ------------------------------------------------------------------

static size_t seq_up(size_t x) { return (x + 255) & ~(size_t)255; }

bool seq_solve(DeviceBatch& db, const std::vector<int32_t>& positions, bool trace) {
  if (positions.empty()) return true;
  mpld_context* ctx = db.ctx;
  hipStream_t s = ctx->stream;
  const int32_t H = (int32_t)positions.size();
  SeqArgs a{};
  a.ncomps = H;
  a.trace = trace ? 1 : 0;
  a.cap[kSeqReg] = db.tune.heavy_round_cap;
  a.cap[kSeqCsr] = db.tune.heavy_round_cap;
  for (int32_t t = 0; t < kSeqTiers; ++t) a.least[t] = 64;
  std::vector<SeqComp> comps((size_t)H);
  int32_t nt[kSeqTiers] = {0, 0};
  int64_t tasks = 0, piece = 0;   // tasks, and their bytes of a piece, summed over what the budgets may need
  int64_t cut = 0, cuts = 0, cut_bytes = 0;   // largest cut; cuts that the budgets may need, and their bytes
  int32_t lds = 0;
  int64_t stack_words = 0;
  for (int32_t i = 0; i < H; ++i) {
    const int32_t pos = positions[(size_t)i];
    const DevDesc& d = db.host_desc[(size_t)pos];
    SeqComp& c = comps[(size_t)i];
    c = SeqComp{};
    c.pos = pos;
    c.tier = pos < db.n_reg ? kSeqReg : kSeqCsr;
    c.running = 1;
    c.count = 1;
    c.sol = -1;
    c.cross = -1;
    ++nt[c.tier];
    if (c.tier == kSeqCsr) {
      // the wide layout keeps headers and log in global memory: 20 to 25%
      // slower a node, but a third of the LDS from a few hundred nodes on, so
      // three times the tasks at once (48 traced components of 65 to 2048
      // nodes: 24 ms a solve with each tier's own layout, two launches a round,
      // 12 so)
      const CsrShape& sh = db.csr_shape[(size_t)(pos - db.n_reg)];
      c.wide = sh.wide_bytes >= 0 && (sh.small_bytes > kSeqSmallLds || pos >= db.n_reg + db.n_lds);
      lds = std::max<int32_t>(lds, (int32_t)(c.wide ? sh.wide_bytes : sh.small_bytes));
      if (c.wide) stack_words = std::max(stack_words, sh.stack_words);
    }
    // about one piece for 16 nodes of the budget, in search order
    const int64_t bytes = c.tier == kSeqReg ? 1024 : 16 * (int64_t)((d.n + 31) / 32) * (d.k < 4 ? 1 : 2) + 512;
    const int64_t most = std::min<int64_t>(d.budget / 16 + 64, 1 << 16);
    tasks += most;
    piece += most * bytes + 64 * (int64_t)d.n;
    // a cut keeps the stack's planes once a piece, its headers, log (about
    // three entries a node) and colors once
    const int64_t each = c.tier == kSeqReg ? 4096 : kSeqPieces * (bytes - 448) + (8 + 12 + 1) * (int64_t)d.n;
    cut = std::max(cut, each);
    cuts += d.budget / 32 + 64;
    cut_bytes += (d.budget / 32 + 64) * each;
  }
  a.slots[kSeqReg] = ctx->num_cus * 16;
  a.slots[kSeqCsr] = std::max(1, std::min(16, 160 * 1024 / std::max(lds, 1))) * ctx->num_cus;
  // and what a few rounds of all slots cut, which is soon more than small
  // budgets come to (three components of 1200 to 2800 nodes, 43,000 nodes each:
  // 52 MB and 22,000 tasks; with the 14 MB and 8,000 of their budgets alone
  // the front went on by itself, 25 ms as root-row tasks, 65 so, 5.8 now)
  const int64_t slots = a.slots[kSeqReg] * (nt[kSeqReg] ? 1 : 0) + a.slots[kSeqCsr] * (nt[kSeqCsr] ? 1 : 0);
  tasks = std::max(tasks, kSeqPieces * std::min(cuts, 2 * slots));
  piece = std::max(piece, std::min(cut_bytes, 2 * slots * cut));
  a.task_cap = (int32_t)std::min<int64_t>(tasks, 1 << 18) + H;
  a.list_cap = std::max(1024, std::min(1 << 17, (1 << 21) / H));
  a.run_cap = 1 << 15;
  a.arena_cap = std::min<int64_t>(std::max<int64_t>(piece, 4 << 20), 1ll << 30);
  if (H > a.run_cap) return false;
  // the workspace, or what there is of it: with less of it more of the search
  // is done by the tasks at the front, down to where the callers' own ways are
  // the better ones
  size_t o_comps, o_tasks, o_res, o_lists, o_runs, o_stack, o_arena;
  for (;;) {
    o_comps = seq_up(sizeof(SeqHead));
    o_tasks = o_comps + seq_up(sizeof(SeqComp) * (size_t)H);
    o_res = o_tasks + seq_up(sizeof(SeqTask) * (size_t)a.task_cap);
    o_lists = o_res + seq_up(sizeof(SeqResult) * (size_t)a.task_cap);
    o_runs = o_lists + seq_up(8 * (size_t)H * (size_t)a.list_cap);
    o_stack = o_runs + seq_up(8 * (size_t)kSeqTiers * (size_t)a.run_cap);
    o_arena = o_stack + seq_up(8 * (size_t)stack_words * (size_t)(stack_words ? a.slots[kSeqCsr] : 0));
    if (ctx->seq_take(o_arena + (size_t)a.arena_cap)) break;
    if (a.arena_cap / 4 < kSeqLeastArena) return false;
    a.arena_cap /= 4;
    a.task_cap = std::max(a.task_cap / 4, 1 << 10) + H;
    a.list_cap = std::max(a.list_cap / 4, 1 << 10);
    a.slots[kSeqCsr] = std::max(a.slots[kSeqCsr] / 2, ctx->num_cus);
  }
  struct Use {   // not given back before the last launch is enqueued
    mpld_context* ctx;
    ~Use() {
      std::lock_guard<std::mutex> lk(ctx->seq_mu);
      ctx->seq_used = false;
    }
  } use{ctx};
  uint8_t* m = static_cast<uint8_t*>(ctx->seq_mem);
  a.head = reinterpret_cast<SeqHead*>(m);
  a.comps = reinterpret_cast<SeqComp*>(m + o_comps);
  a.tasks = reinterpret_cast<SeqTask*>(m + o_tasks);
  a.results = reinterpret_cast<SeqResult*>(m + o_res);
  a.lists = reinterpret_cast<int32_t*>(m + o_lists);
  a.runs = reinterpret_cast<int32_t*>(m + o_runs);
  auto* stack = reinterpret_cast<uint64_t*>(m + o_stack);
  a.arena = m + o_arena;
  // the first run lists: every root
  std::vector<int32_t> first;
  int32_t run0[kSeqTiers] = {0, 0};
  for (int32_t t = 0; t < kSeqTiers; ++t)
    for (int32_t i = 0; i < H; ++i)
      if (comps[(size_t)i].tier == t) {
        first.push_back(i | kSeqCut | kSeqForce);
        ++run0[t];
      }
  const size_t b_comps = sizeof(SeqComp) * (size_t)H, b_first = 4 * (size_t)H;
  if (!db.sp_host_tasks.reserve(seq_up(b_comps) + seq_up(b_first) + 256) || !db.sp_host_out.reserve(sizeof(SeqHead)))
    fail(MPLD_E_NOMEM, "sequence engine: pinned host memory");
  uint8_t* up = db.sp_host_tasks.as<uint8_t>();
  std::memcpy(up, comps.data(), b_comps);
  std::memcpy(up + seq_up(b_comps), first.data(), b_first);
  std::memcpy(up + seq_up(b_comps) + seq_up(b_first), run0, sizeof(run0));
  check_hip(hipMemcpyAsync(a.comps, up, b_comps, hipMemcpyHostToDevice, s), "sequence engine: components");
  hipLaunchKernelGGL(seq_init_kernel, dim3((unsigned)((H + 255) / 256)), dim3(256), 0, s, a);
  check_hip(hipMemcpyAsync(a.head->run[0], up + seq_up(b_comps) + seq_up(b_first), sizeof(run0),
                           hipMemcpyHostToDevice, s), "sequence engine: first round");
  for (int32_t t = 0, at = 0; t < kSeqTiers; at += run0[t++])
    if (run0[t])
      check_hip(hipMemcpyAsync(a.runs + (size_t)t * (size_t)a.run_cap, up + seq_up(b_comps) + 4 * (size_t)at,
                               4 * (size_t)run0[t], hipMemcpyHostToDevice, s), "sequence engine: first round");
  const auto* desc = db.desc.as<DevDesc>();
  const auto* adj = db.adj32.as<uint32_t>();
  SeqHead h{};
  int32_t parity = 0;
  const auto run_tiers = [&](bool finish) {
    if (nt[kSeqReg])
      check_hip(launch_seq_reg(trace, db.k, std::min(a.slots[kSeqReg] / 4, finish ? (nt[kSeqReg] + 3) / 4 : 1 << 30),
                               a, db.reg_items(), parity, finish, db.recs.as<DevRecord>(), db.colors.as<int8_t>(), s),
                "sequence engine: register tier");
    if (nt[kSeqCsr])
      check_hip(launch_seq_csr(trace, db.k, std::min(a.slots[kSeqCsr], finish ? nt[kSeqCsr] : 1 << 30), lds, a, desc,
                               adj, stack, (uint64_t)stack_words, parity, finish, db.recs.as<DevRecord>(),
                               db.colors.as<int8_t>(), s),
                "sequence engine: CSR tiers");
  };
  for (int32_t round = 0;;) {
    // (many components are colored in their first descent: a look after that)
    for (int32_t i = round == 0 ? kSeqRoundsPerCheck - 1 : 0; i < kSeqRoundsPerCheck; ++i, ++round, parity ^= 1) {
      run_tiers(false);
      hipLaunchKernelGGL(seq_fold_kernel, dim3((unsigned)H), dim3(kFoldThreads), 0, s, a, desc, parity);
    }
    check_hip(hipMemcpyAsync(db.sp_host_out.p, a.head, sizeof(SeqHead), hipMemcpyDeviceToHost, s),
              "sequence engine: head");
    check_hip(hipStreamSynchronize(s), "sequence engine: rounds");
    std::memcpy(&h, db.sp_host_out.p, sizeof(h));
    if (h.active[0] + h.active[1] == 0) break;
    if (round >= kSeqMaxRounds) return false;
  }
  db.sp_rounds += h.rounds;
  db.sp_tasks_run += std::min(h.tasks, a.task_cap);
  run_tiers(true);
  return h.lost == 0;
}

}  // namespace mpld
