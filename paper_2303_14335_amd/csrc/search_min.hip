// search_min.hip - Eq. 1 minimisation of register-tier components (at most
// 64 nodes), one 64-lane wavefront per component.
//
// Eq. 1 (Sec. 2.1) asks for a coloring of least conflicts + alpha x
// stitches (alpha = 0.1).  The exact-cover search of Algorithm 1 stops at
// the first exact cover or reports that none exists; Algorithm 1's conflict
// candidates (a column left with no related row) give a coloring with
// conflicts but no claim of least cost.  Here the exact cover is relaxed:
// a row (v, c) whose secondary columns are already covered may still be
// taken, each covered (edge, color) column counting one conflict, and a row
// whose node's stitch partner holds another color counts one stitch.  A
// depth-first branch and bound over the rows, started from the incumbent
// coloring the search (or the conflict marking) left, finds a coloring of
// least cost = 10 conflicts + stitches (Eq. 1 scaled by 10, integers):
//   - penalty of (u, c) for an uncolored node u: 10 x (colored neighbours
//     of color c) + 1 if u's partner is colored with a color other than c;
//   - bound = cost so far + the sum over uncolored u of u's least penalty
//     (each term charges edges to colored nodes only, so the terms are
//     disjoint and only grow);
//   - a node entry passing the budget test counts one node; with every node
//     colored it replaces the incumbent when cheaper; otherwise it returns
//     when the bound reaches the incumbent's cost, else branches on the
//     uncolored node with the fewest conflict-free colors (lowest index on
//     ties) and tries the colors in ascending order, skipping a color whose
//     child bound (bound - least(v) + penalty(v, c)) reaches the incumbent's
//     cost when it is tried.
// Lane u holds u's neighbour mask, its stitch partner, its color and the
// penalties of all colors.  The recursion is an explicit stack in VGPRs, lane
// d holding frame d: the node and color taken at depth d, the bound and the
// node's least penalty at that depth, and the cost before the row was taken.
// Undoing a row restores that frame.
//
// Components of more than kMinAlone nodes are searched again by a workgroup:
// what is left of a search is a list of pieces in the search's order, each a
// path, the next color at its end and the depth above which the piece ends.
// The waves of a round take pieces in order, each up to its share of nodes;
// one that is stopped there is replaced by the pieces of its own stack.  All
// run with the incumbent of the pieces committed before; a piece that finds a
// cheaper coloring counts only as the first one left, and then everything
// after it starts over with the new incumbent (pieces cut out of a piece
// behind it go back into that one).  So the pieces committed in order add up
// to the sequential search's nodes, and its coloring is the one found.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_types.h"
#include "mpld.h"
#include "min_core.h"
#include "reg_items.h"
#include "wave_ops.h"

namespace mpld {

// Nodes that one wave searches before the component goes to a workgroup.
// Of 220 components of 30,000 rects (k = 4, stitches) 40 need a search, 4 to
// 10 of them more than 128 nodes and one or two 1,000 to 10,000: alone on its
// wave at 0.46 us a node, that one is the whole kernel's time.
constexpr uint32_t kMinAlone = 64;
constexpr int kMinWaves = 8, kMinItems = 192, kMinPieces = 8;
constexpr uint32_t kMinShare = 16, kMinShareMost = 128;   // nodes of a wave's round: 16, 18, ... 128

// One wave per workgroup, register-tier items taken grid-stride; every
// item's incumbent colors are in `colors` (the search's solution or the
// conflict marking).  min_out[comp] receives the node count (negated when
// the budget stopped the item), 0 when the incumbent costs nothing.  Items
// not done after kMinAlone nodes are listed instead.
template <int K>
__global__ __launch_bounds__(64) void min_reg_kernel(const RegItems items, int32_t qlen,
                                                     const uint8_t* __restrict__ partners,
                                                     int8_t* __restrict__ colors,
                                                     int32_t* __restrict__ min_out, uint32_t budget,
                                                     int32_t* __restrict__ list_len, int32_t* __restrict__ list) {
  for (int32_t i = (int32_t)uniform(blockIdx.x); i < qlen; i += (int32_t)gridDim.x) {
    const DevDesc d = item_desc(items, i);
    const int32_t comp = (int32_t)uniform((uint32_t)d.comp);
    const int32_t r = minimize_core<K>(d, item_mask(items, i, __lane_id()), partners, colors, budget, kMinAlone);
    if (__lane_id() == 0) {
      if (budget > kMinAlone && r == -(int32_t)kMinAlone) list[atomicAdd(list_len, 1)] = i;
      else min_out[comp] = r;
    }
  }
}

enum : uint8_t { kMinUnrun, kMinDone, kMinHead, kMinBetter, kMinGone };
constexpr uint8_t kMinNone = 0xff;
// MinPieces.finished.  A round takes at least the first piece off the list
// (the first one left always runs, and runs to its end where it finds no room);
// one that did not would be followed by the same again, so the search is then
// done by one wave instead.
enum : int32_t { kMinComplete = 1, kMinStuck = 2 };

// A component's pieces.  An item is a piece not searched yet, one searched to
// its end, or the searched front (head) of one whose rest became pieces.
struct MinPieces {
  uint32_t fb[kMinItems][64];   // path: bound | cost << 16
  uint16_t fr[kMinItems][64];   // path: node | color << 6 | least byte << 9
  uint32_t nodes[kMinItems];
  uint8_t hi[kMinItems], lo[kMinItems], next[kMinItems];   // next = kMinNone: the root
  uint8_t state[kMinItems], parent[kMinItems], pieces[kMinItems];
  uint8_t piece[kMinItems][kMinPieces];
  uint8_t seq[2][kMinItems];    // items in the search's order
  uint8_t spare[kMinItems], run[kMinItems];
  int32_t nseq, nspare, nrun, taken, side;
  uint32_t best, better, committed, round;
  int32_t best_col[64], better_col[64];
  int32_t improved, stopped, finished, result;
};
static_assert(kMinItems < kMinNone, "item ids are bytes");

__device__ __forceinline__ void min_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

// Number of the lower lanes whose bit is set in m.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The front of the `want` spare ids taken off the top (a call by one lane), -1
// if there are not as many.  In one step: taken with a subtraction that is given
// back when it was too much, a third wave in between would find a count too low
// but enough for it, and take ids from below the top that are spare still, or
// in use already once the count is whole again.  No ids come back before the
// round ends, so a try fails only for another's success.
__device__ __forceinline__ int32_t min_take(int32_t* nspare, int32_t want) {
  int32_t have = __hip_atomic_load(nspare, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  while (have >= want) {
    const int32_t seen = atomicCAS(nspare, have, have - want);
    if (seen == have) return have - want;
    have = seen;
  }
  return -1;
}

// Exclusive sum over the wave; `total` the whole.
__device__ __forceinline__ uint32_t min_excl_sum(uint32_t x, uint32_t& total) {
  uint32_t sum = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)sum, o);
    if (__lane_id() >= (uint32_t)o) sum += y;
  }
  total = rdlane(sum, 63u);
  return sum - x;
}

// The pieces of a round that have been searched, in order: what is known to
// be the sequential search's is counted and dropped, cut pieces take their
// parts, and the next round's list is made.  One wave.
__device__ void min_fold(MinPieces& p, uint32_t budget) {
  const uint32_t lane = __lane_id();
  const int32_t n0 = (int32_t)uniform((uint32_t)p.nseq);
  int32_t side = (int32_t)uniform((uint32_t)p.side);
  const bool improved = uniform((uint32_t)p.improved) != 0u;
  // cut pieces: the head, then its parts
  uint32_t len = 0;
  for (int32_t at = 0; at < n0; at += 64) {
    const bool in = at + (int32_t)lane < n0;
    const uint32_t i = in ? p.seq[side][at + (int32_t)lane] : 0u;
    const uint32_t parts = in && p.state[i] == kMinHead ? p.pieces[i] : 0u;
    uint32_t total;
    const uint32_t to = len + min_excl_sum(in ? 1u + parts : 0u, total);
    if (in) {
      p.seq[side ^ 1][to] = (uint8_t)i;
      for (uint32_t j = 0; j < parts; ++j) p.seq[side ^ 1][to + 1u + j] = p.piece[i][j];
      if (parts) p.pieces[i] = 0;
    }
    len += total;
  }
  side ^= 1;
  min_wave_sync();
  // the front that counts: the first piece alone if it found a cheaper
  // coloring, else all up to the first one not searched
  int32_t front = 0;
  uint32_t total = 0;
  for (int32_t at = 0; at < (int32_t)len; at += 64) {
    const bool in = at + (int32_t)lane < (int32_t)len;
    const uint32_t i = in ? p.seq[side][at + (int32_t)lane] : 0u;
    const bool ok = in && (p.state[i] == kMinDone || p.state[i] == kMinHead) && !(improved && at + lane > 0u);
    const uint64_t bad = ~__ballot(ok);
    const uint32_t ahead = bad ? low_bit(bad) : 64u;
    total += wave_sum_u32(lane < ahead ? p.nodes[i] : 0u);
    front += (int32_t)ahead;
    if (ahead < 64u) break;
  }
  const uint32_t committed = uniform(p.committed) + total;
  const bool over = uniform((uint32_t)p.stopped) != 0u || committed > budget;
  int32_t spare = (int32_t)uniform((uint32_t)p.nspare);
  for (int32_t at = (int32_t)lane; at < front; at += 64) {
    const uint8_t i = p.seq[side][at];
    p.state[i] = kMinGone;
    p.spare[spare + at] = i;
  }
  spare += front;
  min_wave_sync();
  // what is left; a cheaper coloring starts all of it over
  int32_t left = 0;
  for (int32_t at = front; at < (int32_t)len; at += 64) {
    const bool in = at + (int32_t)lane < (int32_t)len;
    const uint32_t i = in ? p.seq[side][at + (int32_t)lane] : 0u;
    uint32_t up = in ? p.parent[i] : (uint32_t)kMinNone;
    if (up != kMinNone && p.state[up] == kMinGone) {
      up = kMinNone;
      p.parent[i] = kMinNone;
    }
    const bool keep = in && (!improved || up == kMinNone);
    const uint64_t kept = __ballot(keep), dropped = __ballot(in && !keep);
    if (keep) {
      p.seq[side ^ 1][left + (int32_t)lanes_below(kept)] = (uint8_t)i;
      if (improved) {
        p.state[i] = kMinUnrun;
        p.pieces[i] = 0;
      }
    }
    if (in && !keep) p.spare[spare + (int32_t)lanes_below(dropped)] = (uint8_t)i;
    left += (int32_t)__builtin_popcountll(kept);
    spare += (int32_t)__builtin_popcountll(dropped);
  }
  side ^= 1;
  min_wave_sync();
  // the next round: pieces not searched, up to one that is known to find a
  // cheaper coloring; that one alone once it is the first
  int32_t run = 0;
  const bool first_better = left > 0 && p.state[p.seq[side][0]] == kMinBetter;
  for (int32_t at = 0; at < left; at += 64) {
    const bool in = at + (int32_t)lane < left;
    const uint32_t i = in ? p.seq[side][at + (int32_t)lane] : 0u;
    uint64_t stop = __ballot(in && p.state[i] == kMinBetter);
    if (first_better) stop = 2ull;
    const bool before = stop == 0ull || lane < low_bit(stop);
    const bool take = in && before && (p.state[i] == kMinUnrun || first_better);
    const uint64_t m = __ballot(take);
    if (take) {
      p.run[run + (int32_t)lanes_below(m)] = (uint8_t)i;
      p.state[i] = kMinUnrun;
    }
    run += (int32_t)__builtin_popcountll(m);
    if (stop != 0ull) break;
  }
  if (improved) p.best_col[lane] = p.better_col[lane];
  if (lane == 0) {
    if (improved) p.best = p.better;
    p.committed = committed;
    p.nseq = left;
    p.side = side;
    p.nspare = spare;
    p.nrun = run;
    p.taken = 0;
    p.improved = 0;
    ++p.round;
    if (over || left == 0) {
      p.finished = kMinComplete;
      p.result = over ? -(int32_t)budget : (int32_t)committed;
    } else if (front == 0) {
      p.finished = kMinStuck;
    }
  }
}

// One piece on one wave; `front`: the first of all that is left.  Returns the
// nodes it took of the wave's share.
template <int K>
__device__ __forceinline__ uint32_t min_piece(MinPieces& p, MinSearch<K>& s, uint32_t i, bool front,
                                              uint32_t share, uint32_t budget) {
  const uint32_t lane = __lane_id();
  const uint32_t hi = uniform(p.hi[i]), lo = uniform(p.lo[i]), next = uniform(p.next[i]);
  const uint32_t best = uniform(p.best), rest = budget - uniform(p.committed);
  s.root();
  s.best = best;
  bool enter = true;
  uint32_t v = 0, least = 0, lb = 0;
  if (next != kMinNone) {   // color the path again
    const uint32_t f16 = p.fr[i][lane];
    s.fr = (f16 & 63u) | (((f16 >> 6) & 7u) << 8) | ((f16 >> 9) << 16);
    s.fb = p.fb[i][lane];
    for (uint32_t d = 0; d < hi; ++d) {
      const uint32_t f = uniform(rdlane(s.fr, d)), c = (f >> 8) & 0xffu;
      s.color(f & 0xffu, c, true);
      s.col = wrlane(s.col, f & 0xffu, c);
      s.unc &= ~(1ull << (f & 0xffu));
    }
    const uint32_t f = uniform(rdlane(s.fr, hi)), b = uniform(rdlane(s.fb, hi));
    v = f & 0xffu;
    least = f >> 16;
    lb = b & 0xffffu;
    s.cost = b >> 16;
    s.depth = hi;
    enter = false;
  }
  const uint32_t limit = uniform(front && rest < share ? rest : share);
  bool stopped = s.explore(lo, limit, enter, v, next, least, lb);
  if (!front && s.best < best) {   // counts only as the first
    if (lane == 0) p.state[i] = kMinBetter;
    return s.nodes;
  }
  uint32_t parts = 0, ids = 0;
  const bool end = front && stopped && s.nodes == rest;
  if (stopped && !end) {
    const uint32_t levels = s.depth - lo;
    parts = levels < (uint32_t)kMinPieces ? levels : (uint32_t)kMinPieces;
    int32_t at = 0;
    if (lane == 0) at = min_take(&p.nspare, (int32_t)parts);
    at = (int32_t)uniform((uint32_t)at);
    if (at < 0) {   // no room for its parts
      if (!front) return s.nodes;  // searched again in a later round
      stopped = s.explore(lo, rest, true, 0, 0, 0, 0);
      parts = 0;
    } else {
      ids = (uint32_t)at;
    }
  }
  if (front && s.best < best) {
    p.better_col[lane] = s.best_col;
    if (lane == 0) {
      p.better = s.best;
      p.improved = 1;
    }
  }
  if (parts) {
    // the pieces of its stack, deepest first: one level each but the deepest
    // (at most 8 levels in a piece)
    const uint32_t levels = s.depth - lo, each = levels / (uint32_t)kMinPieces > 1u ? levels / (uint32_t)kMinPieces : 1u;
    const uint32_t f16 = (s.fr & 63u) | (((s.fr >> 8) & 7u) << 6) | (((s.fr >> 16) & 127u) << 9);
    uint32_t top = s.depth - 1u, from = (uniform(rdlane(s.fr, top)) >> 8) & 0xffu;
    for (uint32_t j = 0; j < parts; ++j) {
      const uint32_t id = uniform(p.spare[ids + j]), base = lo + each * (parts - 1u - j);
      p.fr[id][lane] = (uint16_t)f16;
      p.fb[id][lane] = s.fb;
      if (lane == 0) {
        p.hi[id] = (uint8_t)top;
        p.lo[id] = (uint8_t)base;
        p.next[id] = (uint8_t)from;
        p.state[id] = kMinUnrun;
        p.parent[id] = (uint8_t)i;
        p.pieces[id] = 0;
        p.piece[i][j] = (uint8_t)id;
      }
      if (base > lo) {
        top = base - 1u;
        from = ((uniform(rdlane(s.fr, top)) >> 8) & 0xffu) + 1u;
      }
    }
  }
  if (lane == 0) {
    p.nodes[i] = s.nodes;
    p.pieces[i] = (uint8_t)parts;
    p.state[i] = parts ? kMinHead : kMinDone;
    if (front && stopped && !parts) p.stopped = 1;
  }
  return s.nodes;
}

// The listed items, one per workgroup.  What bounds it: the rounds, each a
// share of nodes long (0.46 us a node on a SIMD of its own), and the pieces,
// which are of very different sizes: 8 waves do the work of three to four in a
// search of 10^4 nodes.  So from four items per workgroup on, every wave takes
// an item of its own.  A component of 10^4 nodes (k = 4): 4.6 ms on one wave,
// 1.3 here; with 4 waves 2.0, 6 1.7, 12 2.3 and 16 2.5 (a SIMD's waves share
// its issue slots, and more pieces run ahead for nothing); with shares from 8
// or 32 nodes on 1.4 and 1.7.
template <int K>
__global__ __launch_bounds__(64 * kMinWaves) void min_pieces_kernel(const RegItems items,
                                                                    const uint8_t* __restrict__ partners,
                                                                    int8_t* __restrict__ colors,
                                                                    int32_t* __restrict__ min_out, uint32_t budget,
                                                                    int32_t* __restrict__ list_len,
                                                                    const int32_t* __restrict__ list) {
  __shared__ MinPieces p;
  const int32_t count = *list_len;
  const uint32_t lane = __lane_id(), wave = uniform(threadIdx.x >> 6);
  if (count > 4 * (int32_t)gridDim.x) {
    for (int32_t t = (int32_t)(blockIdx.x * kMinWaves + wave); t < count; t += (int32_t)(gridDim.x * kMinWaves)) {
      const int32_t i = (int32_t)uniform((uint32_t)list[t]);
      const DevDesc d = item_desc(items, i);
      const int32_t r = minimize_core<K>(d, item_mask(items, i, lane), partners, colors, budget);
      if (lane == 0) min_out[d.comp] = r;
    }
  } else {
    for (int32_t t = (int32_t)blockIdx.x; t < count; t += (int32_t)gridDim.x) {
      const int32_t item = (int32_t)uniform((uint32_t)list[t]);
      const DevDesc d = item_desc(items, item);
      const uint32_t n = uniform((uint32_t)d.n);
      const bool in = lane < n;
      MinSearch<K> s;
      s.init(n, item_mask(items, item, lane), in ? (uint32_t)partners[d.nbr_off + lane] : 0xffu,
             in ? (int32_t)colors[d.out_off + lane] : 0);
      __syncthreads();   // the item before is written
      if (wave == 0) {
        p.best_col[lane] = s.best_col;
        for (int32_t j = (int32_t)lane; j < kMinItems - 1; j += 64) p.spare[j] = (uint8_t)(j + 1);
        if (lane == 0) {
          p.hi[0] = p.lo[0] = 0;
          p.next[0] = p.parent[0] = kMinNone;
          p.state[0] = kMinUnrun;
          p.pieces[0] = 0;
          p.seq[0][0] = p.run[0] = 0;
          p.nseq = p.nrun = 1;
          p.nspare = kMinItems - 1;
          p.taken = p.side = 0;
          p.best = s.best;
          p.committed = p.round = 0;
          p.improved = p.stopped = p.finished = p.result = 0;
        }
      }
      __syncthreads();
      // every round takes pieces off the front or is the last, so the rounds end
      for (;;) {
        const uint32_t share = kMinShare + 2u * uniform(p.round);
        const uint32_t most = share < kMinShareMost ? share : kMinShareMost;
        const int32_t nrun = (int32_t)uniform((uint32_t)p.nrun);
        for (uint32_t used = 0; used < most;) {
          int32_t t2 = 0;
          if (lane == 0) t2 = atomicAdd(&p.taken, 1);
          t2 = (int32_t)uniform((uint32_t)t2);
          if (t2 >= nrun) break;
          used = uniform(used + 1u + min_piece<K>(p, s, uniform(p.run[t2]), t2 == 0, most - used, budget));
        }
        __syncthreads();
        if (wave == 0) min_fold(p, budget);
        __syncthreads();
        if (uniform((uint32_t)p.finished) != 0u) break;
      }
      if (wave == 0) {
        int32_t r = (int32_t)uniform((uint32_t)p.result);
        if (uniform((uint32_t)p.finished) == (uint32_t)kMinStuck)
          r = minimize_core<K>(d, item_mask(items, item, lane), partners, colors, budget);
        else if (in)
          colors[d.out_off + lane] = (int8_t)p.best_col[lane];
        if (lane == 0) min_out[d.comp] = r;
      }
    }
  }
  // the last workgroup leaves the list empty for the next call
  __syncthreads();
  if (threadIdx.x == 0) {
    if (atomicAdd(list_len + 1, 1) == (int32_t)gridDim.x - 1) {
      list_len[0] = 0;
      list_len[1] = 0;
    }
  }
}

template <class F>
static void with_colors(int k, F&& f) {
  switch (k) {
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 5: f(std::integral_constant<int, 5>()); break;
    case 6: f(std::integral_constant<int, 6>()); break;
    case 7: f(std::integral_constant<int, 7>()); break;
    default: f(std::integral_constant<int, 8>()); break;
  }
}

hipError_t launch_min_reg(int k, int grid, int num_cus, RegItems items, int32_t qlen, const uint8_t* partners,
                          int8_t* colors, int32_t* min_out, uint32_t budget, int32_t* list_len, int32_t* list,
                          hipStream_t s) {
  if (qlen <= 0) return hipSuccess;
  if (k < 2 || k > 8 || grid < 1 || num_cus < 1 || budget < 1) return hipErrorInvalidValue;
  with_colors(k, [&](auto kp) {
    constexpr int K = decltype(kp)::value;
    hipLaunchKernelGGL((min_reg_kernel<K>), dim3(grid), dim3(64), 0, s, items, qlen, partners,
                       colors, min_out, budget, list_len, list);
    if (budget > kMinAlone)
      hipLaunchKernelGGL((min_pieces_kernel<K>), dim3(std::min(qlen, num_cus)), dim3(64 * kMinWaves), 0, s, items,
                         partners, colors, min_out, budget, list_len, list);
  });
  return hipGetLastError();
}

}  // namespace mpld
