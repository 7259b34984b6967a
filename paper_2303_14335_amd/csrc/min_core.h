// min_core.h - the Eq. 1 branch and bound of one register-tier component
// on one wavefront (the method is described in search_min.hip), shared by
// the batched minimisation kernel and the serving tick.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_types.h"
#include "wave_ops.h"

namespace mpld {

// What bounds it: one wave's chain of dependent instructions, a node after
// another.  A lane's penalties of all colors are bytes of one word (two for
// k > 4): byte c = 2 x (colored neighbours of color c) + 1 if the stitch
// partner has another color, at most 127 and in the order of the penalties
// 10 conflicts + stitches; colors past k hold 127.  So the least penalty is a
// minimum of bytes, the open colors are counted with one addition, coloring a
// node is one conditional addition in its neighbours' lanes (the mask comes
// from the node's own lane), the bound's sum is population counts of ballots
// and the branching node three steps of narrowing them; the colors of the
// branching node are tried side by side in lanes.  With counters and partner
// colors apart, the sums and minima over the wave in DPP steps and the colors
// one after another a node took 0.79 us (k = 4, components that run to 10^4
// nodes), this way 0.46 us.
template <int K>
struct MinWords {
  static constexpr int N = (K + 3) / 4;
  uint32_t w[N];
};

// on ? x : 0 in the lanes of `mask`.
__device__ __forceinline__ uint32_t lanes_of(uint64_t mask, uint32_t x) {
  uint32_t r;
  asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(x), "s"(mask));
  return r;
}

// The branch and bound of one component on one wave: lane u holds node u's
// neighbour mask, partner and penalties, lane d frame d of the path.
template <int K>
struct MinSearch {
  static constexpr int N = MinWords<K>::N;
  uint32_t lane, n, part, nb_lo, nb_hi;
  MinWords<K> X;
  uint32_t ones[N];        // 1 in every color's byte
  uint64_t unc;            // uncolored nodes
  uint32_t col;            // lane u: u's color on the path
  int32_t best_col;
  uint32_t best, cost, depth, nodes;
  uint32_t fr, fb;         // lane = depth: node | color << 8 | least byte << 16; bound | cost << 16

  static __device__ __forceinline__ uint32_t penalty(uint32_t b) { return 10u * (b >> 1) + (b & 1u); }

  // inc: each lane's color of the incumbent, whose cost becomes `best`.
  __device__ __forceinline__ void init(uint32_t nodes_of, uint64_t nb, uint32_t partner, int32_t inc) {
    lane = __lane_id();
    n = nodes_of;
    part = partner;
    nb_lo = (uint32_t)nb;
    nb_hi = (uint32_t)(nb >> 32);
    const bool in = lane < n;
    // incumbent cost: conflict ends of each lane (each edge twice) and the
    // stitch pairs seen from their lower end
    uint64_t same = 0;
#pragma unroll
    for (int c = 0; c < K; ++c) {
      const uint64_t m = __ballot(in && inc == c);
      if (in && inc == c) same = m;
    }
    const uint32_t pinc = (uint32_t)__shfl(inc, (int)(part & 63u));
    const uint32_t ends = in ? (uint32_t)__popcll(nb & same) : 0u;
    const uint32_t st = (in && part != 0xffu && part > lane && pinc != (uint32_t)inc) ? 1u : 0u;
    best = uniform(10u * (wave_sum_u32(ends) / 2u) + wave_sum_u32(st));
    best_col = inc;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      ones[j] = 0;
      for (int c = 0; c < 4; ++c)
        if (4 * j + c < K) ones[j] |= 1u << (8 * c);
    }
  }

  // The root: nothing colored.
  __device__ __forceinline__ void root() {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      X.w[j] = 0;
      for (int c = 0; c < 4; ++c)
        if (4 * j + c >= K) X.w[j] |= 127u << (8 * c);
    }
    unc = n >= 64u ? ~0ull : (1ull << n) - 1ull;
    col = cost = depth = nodes = fr = fb = 0;
  }

  // Node v takes color c (or gives it back): its neighbours' byte c by 2, its
  // partner's other bytes by 1.
  __device__ __forceinline__ void color(uint32_t v, uint32_t c, bool on) {
    const uint64_t nv = rdlane64(nb_lo, nb_hi, v);
    const uint32_t p = rdlane(part, v), byte = 1u << (8u * (c & 3u));
    const uint64_t pm = p < 64u ? 1ull << p : 0ull;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const uint32_t mine = (c >> 2) == (uint32_t)j ? byte : 0u;
      const uint32_t x = lanes_of(nv, 2u * mine) + lanes_of(pm, ones[j] & ~mine);
      X.w[j] = on ? X.w[j] + x : X.w[j] - x;
    }
  }

  // The search from here until it has backed up to depth `base`, or until the
  // next node would be one more than `limit` (true).  enter: a node is
  // entered first; otherwise node v at the current depth goes on with its
  // first color from c0 on (least byte `least`, bound `lb`).
  __device__ __forceinline__ bool explore(uint32_t base, uint32_t limit, bool enter, uint32_t v, uint32_t c0,
                                          uint32_t least, uint32_t lb) {
    for (;;) {
      bool down = !enter;
      if (enter) {
        // ---- one node
        if (nodes == limit) return true;
        ++nodes;
        v = c0 = least = lb = 0;
        if (unc == 0ull) {   // every node colored: cheaper than the incumbent?
          if (cost < best) {
            best = cost;
            best_col = (int32_t)col;
          }
        } else {
          uint32_t x = 127u, shut = 0;
#pragma unroll
          for (int j = 0; j < N; ++j) {
#pragma unroll
            for (int c = 0; c < 4; ++c) x = min(x, (X.w[j] >> (8 * c)) & 0xffu);
            shut += (uint32_t)__popc((X.w[j] + 0x7e7e7e7eu) & 0x80808080u);   // bytes of 2 and more
          }
          const uint32_t open = 4u * (uint32_t)N - shut;   // colors without a conflict: 0 .. K
          uint32_t sum = (uint32_t)__builtin_popcountll(__ballot((x & 1u) != 0u) & unc) +
                         10u * (uint32_t)__builtin_popcountll(__ballot((x & 2u) != 0u) & unc) +
                         20u * (uint32_t)__builtin_popcountll(__ballot((x & 4u) != 0u) & unc);
          const uint64_t more = __ballot(x >= 8u) & unc;   // four conflicts at least: rare
          if (more != 0ull) sum += 10u * uniform(wave_sum_u32(lanes_of(more, x >> 3 << 2)));
          uint64_t cand = unc;
#pragma unroll
          for (int b = K < 4 ? 1 : (K < 8 ? 2 : 3); b >= 0; --b) {
            const uint64_t less = cand & ~__ballot(((open >> b) & 1u) != 0u);
            cand = less != 0ull ? less : cand;
          }
          lb = cost + sum;
          if (lb < best) {
            v = low_bit(cand);
            least = rdlane(x, v);
            down = true;
          }
        }
      }
      enter = true;
      for (;;) {
        if (down) {
          // the next color of v whose child bound stays below the incumbent
          const uint32_t w0 = rdlane(X.w[0], v), w1 = rdlane(X.w[N - 1], v);
          const uint32_t word = lane >= 4u ? w1 : w0;
          const uint32_t pen = penalty((word >> (8u * (lane & 3u))) & 0xffu);
          const uint64_t fits = __ballot(lane >= c0 && lane < (uint32_t)K && lb - penalty(least) + pen < best);
          if (fits != 0ull) {
            const uint32_t c = low_bit(fits);
            fr = wrlane(fr, depth, v | (c << 8) | (least << 16));
            fb = wrlane(fb, depth, lb | (cost << 16));
            color(v, c, true);
            col = wrlane(col, v, c);
            unc &= ~(1ull << v);
            cost += rdlane(pen, c);
            ++depth;
            break;
          }
        }
        // back up one level: undo its row, go on with its next color
        if (depth == base) return false;
        --depth;
        const uint32_t f = uniform(rdlane(fr, depth)), b = uniform(rdlane(fb, depth));
        v = f & 0xffu;
        least = f >> 16;
        lb = b & 0xffffu;
        cost = b >> 16;
        color(v, (f >> 8) & 0xffu, false);
        unc |= 1ull << v;
        c0 = ((f >> 8) & 0xffu) + 1u;
        down = true;
      }
    }
  }
};

// Minimises the component of descriptor d (lane u holding u's neighbour
// mask in nb; partners[d.nbr_off + u] its stitch partner, 0xff none) from
// the incumbent colors at colors_base + d.out_off.  Returns the
// branch-and-bound nodes, negated when the budget stopped it; 0 when the
// incumbent costs nothing.  Writes the best coloring, unless it was stopped
// at `limit` nodes below the budget.
template <int K>
__device__ int32_t minimize_core(const DevDesc& d, const uint64_t nb,
                                 const uint8_t* __restrict__ partners,
                                 int8_t* __restrict__ colors_base, uint32_t budget, uint32_t limit = ~0u) {
  const uint32_t lane = __lane_id();
  const uint32_t n = uniform((uint32_t)d.n);
  const bool in = lane < n;
  MinSearch<K> s;
  s.init(n, nb, in ? (uint32_t)partners[d.nbr_off + lane] : 0xffu,
         in ? (int32_t)colors_base[d.out_off + lane] : 0);
  if (s.best == 0u) return 0;
  s.root();
  const uint32_t until = budget < limit ? budget : limit;
  const bool stopped = s.explore(0, until, true, 0, 0, 0, 0);
  if (in && !(stopped && until < budget)) colors_base[d.out_off + lane] = (int8_t)s.best_col;
  return stopped ? -(int32_t)s.nodes : (int32_t)s.nodes;
}

}  // namespace mpld
