// flow_device.hip - the whole-layout flow of Sec. 2.2 around the search, on
// the device: a caller's pairs become the CSR layout graph (validated), the
// graph is simplified and split (graph_device.hip), the components are
// packed for the search, and after it the removed nodes are recovered and
// the Eq. 1 tallies taken.  The host copies the pairs in, places the
// components (tiers, launch order, offsets: a few words each) and copies
// colors, components and records out.
//
// Every kernel here is bound by dependent loads and launches, not by
// bandwidth: a 200k-node layout is 2 to 6 MB in and out.  On one CPU core the
// same passes (validation and CSR, pairs and masks of each component,
// recovery, tallies) walk those arrays with a cache miss per entry: one
// decomposition of 200k rectangles took 6.1 ms at k = 3 and 15.4 ms at k = 4
// with 0.26 and 1.1 ms of it in kernels.
//
// What does not come out of the ordinary (a fault in the caller's graph, a
// node of very many neighbours, a recovery whose chain of dependencies is
// very long) is left to the host path, which reports the fault or does the
// work: the flow only says that it did not.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "graph_builder.h"

namespace mpld {

#define FLOW_FOR(v, n)                                                                  \
  for (int32_t v = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); v < (n);          \
       v += (int32_t)(gridDim.x * blockDim.x))

static constexpr int kFlowGrid = 2048;   // grid-stride kernels: blocks of 256
static unsigned flow_grid(int64_t n) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, kFlowGrid));
}

// Faults found on the device (FlowHead.flags).
enum : int32_t {
  kFlowBadPair = 1,      // id out of range, self loop, duplicate, stitch pair fault
  kFlowDegree = 2,       // a node of more than kFlowMaxDegree neighbours
  kFlowNoColor = 4,      // recovery found no free color
  kFlowChain = 8,        // recovery gave up waiting
};
// An entry's rank in its list is counted against the whole list: d^2 reads
// for a node of d neighbours (layout graphs have a few dozen at most).
static constexpr int32_t kFlowMaxDegree = 2048;

struct FlowHead {
  int32_t flags, removed, ncomp, ticket;
  unsigned long long stitches, conflicts, uncolored;
};
static_assert(sizeof(FlowHead) == 40, "head is 40 bytes");

// ---- the CSR graph of the caller's pairs -----------------------------------

__global__ __launch_bounds__(256) void flow_init_kernel(int32_t n, FlowHead* head, int32_t* deg,
                                                        int32_t* partner, int32_t* cmax) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *head = FlowHead{};
  FLOW_FOR(v, n) {
    deg[v] = 0;
    partner[v] = -1;
    cmax[v] = 0;
  }
}

__device__ __forceinline__ bool flow_pair_ok(int2 e, int32_t n) {
  return e.x >= 0 && e.y >= 0 && e.x < n && e.y < n && e.x != e.y;
}

// Degrees; each pair's places in the two lists are the counts it found, so
// that the scatter needs no atomics of its own.
__global__ __launch_bounds__(256) void flow_count_kernel(int32_t n, int32_t m, const int2* ce,
                                                         int32_t* deg, int2* place, FlowHead* head) {
  FLOW_FOR(i, m) {
    const int2 e = ce[i];
    if (!flow_pair_ok(e, n)) {
      atomicOr(&head->flags, kFlowBadPair);
      continue;
    }
    place[i] = int2{atomicAdd(deg + e.x, 1), atomicAdd(deg + e.y, 1)};
  }
}

// Both directions of every pair into its node's list, in any order; src is
// the list's node, so that the ranking below has one thread per entry.
__global__ __launch_bounds__(256) void flow_scatter_kernel(int32_t n, int32_t m, const int2* ce,
                                                           const int32_t* ptr, const int2* place,
                                                           int32_t* tmp, int32_t* src) {
  FLOW_FOR(i, m) {
    const int2 e = ce[i];
    if (!flow_pair_ok(e, n)) continue;
    const int2 at = place[i];
    const int32_t a = ptr[e.x] + at.x, b = ptr[e.y] + at.y;
    tmp[a] = e.y;
    src[a] = e.x;
    tmp[b] = e.x;
    src[b] = e.y;
  }
}

// Ascending lists: an entry's place is the number of smaller entries of its
// list (of equal ones, those before it: a duplicate pair is a fault, but
// every slot is written).
__global__ __launch_bounds__(256) void flow_rank_kernel(int32_t n, const int32_t* ptr,
                                                        const int32_t* tmp, const int32_t* src,
                                                        int32_t* adj, FlowHead* head) {
  const int32_t total = ptr[n];
  FLOW_FOR(t, total) {
    const int32_t u = src[t], x = tmp[t], t0 = ptr[u], t1 = ptr[u + 1];
    if (t1 - t0 > kFlowMaxDegree) {
      if (t == t0) atomicOr(&head->flags, kFlowDegree);
      adj[t] = x;
      continue;
    }
    int32_t r = 0;
    bool dup = false;
    for (int32_t j = t0; j < t1; ++j) {
      const int32_t y = tmp[j];
      r += y < x || (y == x && j < t) ? 1 : 0;
      dup |= y == x && j != t;
    }
    if (dup) atomicOr(&head->flags, kFlowBadPair);
    adj[t0 + r] = x;
  }
}

__global__ __launch_bounds__(256) void flow_partner_kernel(int32_t n, int32_t m, const int2* se,
                                                           const int32_t* ptr, const int32_t* adj,
                                                           int32_t* partner, FlowHead* head) {
  FLOW_FOR(i, m) {
    const int2 e = se[i];
    bool bad = !flow_pair_ok(e, n);
    if (!bad) {
      bad = atomicCAS(partner + e.x, -1, e.y) != -1;
      bad |= atomicCAS(partner + e.y, -1, e.x) != -1;
      int32_t lo = ptr[e.x], hi = ptr[e.x + 1];
      while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (adj[mid] < e.y) lo = mid + 1;
        else hi = mid;
      }
      bad |= lo < ptr[e.x + 1] && adj[lo] == e.y;
    }
    if (bad) atomicOr(&head->flags, kFlowBadPair);
  }
}

// ---- components ---------------------------------------------------------------

// Degree within the core of every core node, by its place in `order`; the
// largest of each component.
__global__ __launch_bounds__(256) void flow_core_kernel(int32_t n, const int32_t* counts,
                                                        const int32_t* ptr, const int32_t* adj,
                                                        const int32_t* comp_of, const int32_t* order,
                                                        int32_t* cdeg, int32_t* cmax) {
  const int32_t core = n - counts[0];
  FLOW_FOR(p, n) {
    int32_t d = 0;
    if (p < core) {
      const int32_t x = order[p], c = comp_of[x];
      for (int32_t t = ptr[x]; t < ptr[x + 1]; ++t) d += comp_of[adj[t]] >= 0 ? 1 : 0;
      // a wave within one component asks once (40k nodes of one component
      // asking one by one took 464 us)
      if (__ballot(c == __builtin_amdgcn_readfirstlane(c)) == __ballot(true)) {
        int32_t most = d;
        for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, 64));
        if ((threadIdx.x & 63u) == (unsigned)__builtin_ctzll(__ballot(true))) atomicMax(cmax + c, most);
      } else {
        atomicMax(cmax + c, d);
      }
    }
    cdeg[p] = d;
  }
}

__global__ __launch_bounds__(256) void flow_summary_kernel(const int32_t* counts, const int32_t* comp_ptr,
                                                           const int32_t* order, const int32_t* cpre,
                                                           const int32_t* cmax, FlowHead* head,
                                                           FlowComp* out) {
  const int32_t nc = counts[1];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    head->removed = counts[0];
    head->ncomp = nc;
  }
  FLOW_FOR(c, nc) {
    const int32_t b = comp_ptr[c], e = comp_ptr[c + 1];
    out[c] = FlowComp{e - b, cpre[e] - cpre[b], cmax[c], order[b]};
  }
}

// ---- packing --------------------------------------------------------------------

// One wave per register-tier item (launch order): descriptor, neighbour
// masks (zero past n), stitch partners.  Lane v gathers node v's mask.
__global__ __launch_bounds__(256) void flow_pack_reg_kernel(RegItems items, const DevDesc* descs,
                                                            int32_t count, const int32_t* ptr,
                                                            const int32_t* adj, const int32_t* partner,
                                                            const int32_t* comp_of, const int32_t* order,
                                                            const int32_t* comp_ptr, const int32_t* local,
                                                            uint8_t* partners) {
  const int32_t i = (int32_t)(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = (int32_t)(threadIdx.x & 63);
  if (i >= count) return;
  const DevDesc d = descs[i];
  uint8_t* it = const_cast<uint8_t*>(items.base) + (uint64_t)items.stride * (uint64_t)i;
  if (lane < 4) reinterpret_cast<uint64_t*>(it)[lane] = reinterpret_cast<const uint64_t*>(descs + i)[lane];
  uint64_t m = 0;
  uint32_t mate = 0xffu;
  if (lane < d.n) {
    const int32_t x = order[comp_ptr[d.comp] + lane];
    for (int32_t t = ptr[x]; t < ptr[x + 1]; ++t) {
      const int32_t l = local[adj[t]];   // -1: removed
      if (l >= 0) m |= 1ull << l;
    }
    const int32_t q = partner[x];
    if (q >= 0 && comp_of[q] == d.comp) mate = (uint32_t)local[q];
  }
  if (lane < (int32_t)items.width) reinterpret_cast<uint64_t*>(it + kRegItemHead)[lane] = m;
  if (items.part_off && lane < (int32_t)((items.width + 7u) & ~7u))
    it[items.part_off + lane] = lane < (int32_t)items.width ? (uint8_t)mate : (uint8_t)0;
  if (partners && lane < d.n) partners[d.nbr_off + lane] = (uint8_t)mate;
}

// CSR components (LDS, big and device-wide tiers): blockIdx.x is the item,
// the waves of its gridDim.y blocks take one node each in turn.  A node's
// list is its core neighbours' local ids, each at its rank (lists are
// compared chunk by chunk through the wave's lanes).
__global__ __launch_bounds__(256) void flow_pack_csr_kernel(const DevDesc* descs, const int32_t* ptr,
                                                            const int32_t* adj, const int32_t* partner,
                                                            const int32_t* comp_of, const int32_t* order,
                                                            const int32_t* comp_ptr, const int32_t* local,
                                                            const int32_t* cpre, const int32_t* cmax,
                                                            bool stitch, uint32_t* adj32) {
  const DevDesc d = descs[blockIdx.x];
  const int32_t lane = (int32_t)(threadIdx.x & 63), base = comp_ptr[d.comp], pre = cpre[base];
  uint32_t* rows = adj32 + d.nbr_off;
  uint32_t* ids = rows + d.n + 1;
  const int32_t m2 = cpre[base + d.n] - pre;
  if (blockIdx.y == 0 && threadIdx.x == 0) {
    rows[d.n] = (uint32_t)m2;
    ids[m2] = (uint32_t)cmax[d.comp];
  }
  for (int32_t v = (int32_t)(blockIdx.y * 4 + (threadIdx.x >> 6)); v < d.n; v += (int32_t)gridDim.y * 4) {
    const int32_t x = order[base + v], t0 = ptr[x], t1 = ptr[x + 1], at = cpre[base + v] - pre;
    if (lane == 0) {
      rows[v] = (uint32_t)at;
      if (stitch) {
        const int32_t q = partner[x];
        ids[m2 + 1 + v] = q >= 0 && comp_of[q] == d.comp ? (uint32_t)local[q] : 0xffffffffu;
      }
    }
    for (int32_t a = t0; a < t1; a += 64) {
      const int32_t l = a + lane < t1 ? local[adj[a + lane]] : -1;
      int32_t r = 0;
      for (int32_t b = t0; b < t1; b += 64) {
        const int32_t o = b == a ? l : (b + lane < t1 ? local[adj[b + lane]] : -1);
        const int32_t cnt = t1 - b < 64 ? t1 - b : 64;
        for (int32_t j = 0; j < cnt; ++j) {
          const int32_t y = __builtin_amdgcn_readlane(o, j);
          r += y >= 0 && y < l ? 1 : 0;
        }
      }
      if (l >= 0) ids[at + r] = (uint32_t)l;
    }
  }
}

// ---- recovery and tallies -----------------------------------------------------

static constexpr int32_t kPending = -2;      // a removed node not colored yet

__device__ __forceinline__ int32_t ld_color(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Core nodes take their local color, removed ones wait; each removed node's
// place in the removal order (-1: core).
__global__ __launch_bounds__(256) void flow_colors_kernel(int32_t n, int32_t removed, FlowHead* head,
                                                          const int32_t* queue, const int32_t* comp_of,
                                                          const int32_t* comp_ptr, const int32_t* local,
                                                          const int8_t* lcol, int32_t* col, int32_t* qpos,
                                                          int2* cstat, int32_t ncomp) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *head = FlowHead{};
  FLOW_FOR(v, n) {
    const int32_t c = comp_of[v];
    col[v] = c >= 0 ? (int32_t)lcol[comp_ptr[c] + local[v]] : kPending;
    if (c >= 0) qpos[v] = -1;
  }
  FLOW_FOR(i, removed) qpos[queue[i]] = i;
  FLOW_FOR(c, ncomp) cstat[c] = int2{0, 0};
}

// Recovery: the removed nodes in reverse order, each taking its color from
// the nodes colored before it (core nodes and nodes removed later).  A
// thread waits for exactly those neighbours (and its stitch partner).
// Blocks take their place in the order by a ticket, so a block only ever
// waits for blocks that already run; a chain of dependencies longer than
// `rounds` (ids that run along a path of thousands of nodes) is given up
// and left to the host.
__global__ __launch_bounds__(256) void flow_recover_kernel(int32_t removed, int32_t k, int32_t rounds,
                                                           FlowHead* head,
                                                           const int32_t* ptr, const int32_t* adj,
                                                           const int32_t* partner, const int32_t* queue,
                                                           const int32_t* qpos, int32_t* col) {
  __shared__ int32_t base;
  if (threadIdx.x == 0) base = atomicAdd(&head->ticket, 1) * 256;
  __syncthreads();
  const int32_t i = removed - 1 - (base + (int32_t)threadIdx.x);
  bool done = i < 0;
  int32_t x = 0, t = 0, t1 = 0, q = -1, w = -1, q_col = -1;
  uint32_t used = 0;
  // the next node whose color x needs, from its list, then its partner
  auto next = [&] {
    for (w = -1; t < t1 && w < 0; ++t) {
      const int32_t y = adj[t], py = qpos[y];
      if (py < 0 || py > i) w = y;
    }
    if (w < 0) {
      w = q;
      q = -1;
      t = t1 + 1;   // w, if any, is the partner
    }
  };
  if (!done) {
    x = queue[i];
    t = ptr[x];
    t1 = ptr[x + 1];
    q = partner[x];
    if (q >= 0) {
      const int32_t pq = qpos[q];
      if (pq >= 0 && pq < i) q = -1;   // removed before x: not colored yet
    }
    next();
  }
  // A lane keeps what it has read and asks for one color a round.  It stores
  // its own inside the loop, not on its way out: lanes of its own wave may
  // be waiting for it.
  for (int32_t spin = 0; spin < rounds; ++spin) {
    while (!done) {
      if (w >= 0) {
        const int32_t c = ld_color(col + w);
        if (c == kPending) break;
        if (t > t1) q_col = c;
        else if (c >= 0) used |= 1u << c;
        if (t <= t1) {
          next();
          continue;
        }
      }
      int32_t c = q_col;
      if (c < 0 || ((used >> c) & 1u)) {
        const uint32_t free_mask = ~used & ((1u << k) - 1u);
        if (!free_mask) atomicOr(&head->flags, kFlowNoColor);
        c = free_mask ? (int32_t)__builtin_ctz(free_mask) : 0;
      }
      __hip_atomic_store(col + x, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      done = true;
    }
    if (__ballot(!done) == 0ull) break;
    if ((spin & 15) == 15 && (ld_color(&head->flags) & kFlowChain)) break;
  }
  if (!done) atomicOr(&head->flags, kFlowChain);
}

// Final colors, Eq. 1 tallies of the layout, and each component's conflicts
// and stitches (cstat: same-colored pairs seen from both ends, stitches).
__global__ __launch_bounds__(256) void flow_tally_kernel(int32_t n, const int32_t* ptr, const int32_t* adj,
                                                         const int32_t* partner, const int32_t* comp_of,
                                                         const int32_t* col, int8_t* colors, int2* cstat,
                                                         FlowHead* head) {
  uint32_t st = 0, cn = 0, un = 0;
  FLOW_FOR(v, n) {
    const int32_t cv = col[v] < 0 ? -1 : col[v], cc = comp_of[v];
    colors[v] = (int8_t)cv;
    const int32_t p = partner[v];
    if (p > v) {
      const int32_t cp = col[p] < 0 ? -1 : col[p];
      st += cv >= 0 && cp >= 0 && cp != cv ? 1 : 0;
      if (cc >= 0 && cp != cv && comp_of[p] == cc) atomicAdd(&cstat[cc].y, 1);
    }
    if (cv < 0) {
      ++un;
      continue;
    }
    int32_t same = 0;
    for (int32_t t = ptr[v]; t < ptr[v + 1]; ++t) {
      const int32_t w = adj[t];
      if (col[w] != cv) continue;
      cn += w > v ? 1 : 0;
      same += cc >= 0 && comp_of[w] == cc ? 1 : 0;
    }
    if (same) atomicAdd(&cstat[cc].x, same);
  }
  for (int off = 32; off > 0; off >>= 1) {
    st += __shfl_down(st, off, 64);
    cn += __shfl_down(cn, off, 64);
    un += __shfl_down(un, off, 64);
  }
  // one addition a block: thousands of waves adding to one address had taken
  // most of this kernel's time (82 us on 296k nodes)
  __shared__ uint32_t sum[3][4];
  if ((threadIdx.x & 63) == 0) {
    sum[0][threadIdx.x >> 6] = st;
    sum[1][threadIdx.x >> 6] = cn;
    sum[2][threadIdx.x >> 6] = un;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const uint32_t* s = sum[threadIdx.x];
    const unsigned long long v = (unsigned long long)s[0] + s[1] + s[2] + s[3];
    if (v) atomicAdd(&head->stitches + threadIdx.x, v);
  }
}

// ---- host side ------------------------------------------------------------------

// Components whose summary comes with the head in one copy.
static constexpr int32_t kSummaryFirst = 4096;

bool flow_build(FlowGraph& f, GraphBuilder& gb, const mpld_graph& in, int32_t k, bool simplify) {
  const int64_t m = in.num_ce, ns = in.num_se;
  const int32_t n = in.num_nodes;
  if (n <= 0 || m < 0 || ns < 0 || (m > 0 && !in.ce) || (ns > 0 && !in.se)) return false;
  // 32-bit offsets; two entries a pair
  if (n > (1 << 28) || 2 * m >= (1ll << 30) || 2 * ns > (int64_t)n) return false;
  std::lock_guard<std::mutex> lk(gb.mu);
  mpld_context* ctx = gb.ctx;
  hipStream_t st = gb.stream;
  const size_t nn = (size_t)n, mm = (size_t)m;
  f.n = n;
  f.m = m;
  f.simplify = simplify;
  // what a later collection reads stays with the graph ...
  const size_t keep = (nn + 1) + 2 * mm + nn + split_out_words(n) + 2 * (nn + 1);
  // ... the rest is the builder's
  const size_t head_words = (sizeof(FlowHead) + 24) / 4;   // the summary behind it, 16-byte aligned
  const size_t pair_words = 2 * (mm + (size_t)ns);
  const size_t scratch =
      head_words + 4 * (nn + 1) + pair_words + 2 * mm + 2 * (nn + 1) + 4 * mm + split_scratch_words(n);
  try {   // all of it, before the first launch
    if (f.keep.bytes < 4 * keep) f.keep.alloc(ctx, 4 * keep);
    grow(gb.flow_ws, ctx, 4 * scratch);
    scan_reserve(gb, n);
  } catch (const NoMemory&) {
    f.keep.release();
    return false;
  }
  if (!grow_pinned(gb.hin, std::max<size_t>(4 * pair_words, 4)) ||
      !grow_pinned(gb.hout, sizeof(FlowHead) + 24 + sizeof(FlowComp) * nn + 5 * nn + 256))
    return false;
  f.ptr = f.keep.as<int32_t>();
  f.adj = f.ptr + nn + 1;
  f.partner = f.adj + 2 * mm;
  f.cpre = f.partner + nn;       // n + 1
  f.cmax = f.cpre + nn + 1;      // n + 1
  int32_t* out = f.cmax + nn + 1;
  int32_t* w = gb.flow_ws.as<int32_t>();
  auto* head = reinterpret_cast<FlowHead*>(w);
  w += head_words;
  auto* summary = reinterpret_cast<FlowComp*>(w);
  w += 4 * (nn + 1);
  auto* ce = reinterpret_cast<int2*>(w);
  auto* se = ce + mm;
  w += pair_words;
  auto* place = reinterpret_cast<int2*>(w);
  w += 2 * mm;
  int32_t* deg = w;
  int32_t* cdeg = deg + nn + 1;
  int32_t* tmp = cdeg + nn + 1;
  int32_t* src = tmp + 2 * mm;
  int32_t* split_scratch = src + 2 * mm;
  const unsigned gn = flow_grid(n);
  hipLaunchKernelGGL(flow_init_kernel, dim3(gn), dim3(256), 0, st, n, head, deg, f.partner, f.cmax);
  if (m) {
    std::memcpy(gb.hin.p, in.ce, 8 * mm);
    check_hip(hipMemcpyAsync(ce, gb.hin.p, 8 * mm, hipMemcpyHostToDevice, st), "layout flow: pairs");
    hipLaunchKernelGGL(flow_count_kernel, dim3(flow_grid(m)), dim3(256), 0, st, n, (int32_t)m, ce, deg, place,
                       head);
  }
  scan(gb, deg, n, f.ptr);
  if (m) {
    hipLaunchKernelGGL(flow_scatter_kernel, dim3(flow_grid(m)), dim3(256), 0, st, n, (int32_t)m, ce, f.ptr,
                       place, tmp, src);
    hipLaunchKernelGGL(flow_rank_kernel, dim3(flow_grid(2 * m)), dim3(256), 0, st, n, f.ptr, tmp, src, f.adj,
                       head);
  }
  if (ns) {
    uint8_t* hs = gb.hin.as<uint8_t>() + 8 * mm;
    std::memcpy(hs, in.se, 8 * (size_t)ns);
    check_hip(hipMemcpyAsync(se, hs, 8 * (size_t)ns, hipMemcpyHostToDevice, st), "layout flow: stitch pairs");
    hipLaunchKernelGGL(flow_partner_kernel, dim3(flow_grid(ns)), dim3(256), 0, st, n, (int32_t)ns, se, f.ptr,
                       f.adj, f.partner, head);
  }
  const SplitArgs a = enqueue_split(gb, n, f.ptr, f.adj, 2 * m, k, simplify, out, split_scratch, &head->flags,
                                    f.ptr);
  f.queue = a.queue;
  f.comp_of = a.comp_of;
  f.order = a.order;
  f.comp_ptr = a.comp_ptr;
  f.local = a.local;
  hipLaunchKernelGGL(flow_core_kernel, dim3(gn), dim3(256), 0, st, n, a.counts, f.ptr, f.adj, f.comp_of,
                     f.order, cdeg, f.cmax);
  scan(gb, cdeg, n, f.cpre);
  hipLaunchKernelGGL(flow_summary_kernel, dim3(gn), dim3(256), 0, st, a.counts, f.comp_ptr, f.order, f.cpre,
                     f.cmax, head, summary);
  check_hip(hipGetLastError(), "layout flow: front-end");
  uint8_t* ho = gb.hout.as<uint8_t>();
  const size_t first = std::min<size_t>(nn, (size_t)kSummaryFirst), at = 4 * head_words;
  check_hip(hipMemcpyAsync(ho, head, at + sizeof(FlowComp) * first, hipMemcpyDeviceToHost, st),
            "layout flow: summary");
  check_hip(hipStreamSynchronize(st), "layout flow: front-end");
  FlowHead h;
  std::memcpy(&h, ho, sizeof(h));
  if (h.ncomp == -1) ++ctx->splits_left;
  if (h.flags || h.ncomp == -1) return false;   // a fault or a hub; a split that the device gave up
  if (h.removed < 0 || h.removed > n || h.ncomp < 0 || h.ncomp > n - h.removed)
    fail(MPLD_E_INTERNAL, "layout flow: bad counts");
  f.removed = h.removed;
  f.ncomp = h.ncomp;
  if ((size_t)h.ncomp > first) {
    check_hip(hipMemcpyAsync(ho + at + sizeof(FlowComp) * first, summary + first,
                             sizeof(FlowComp) * ((size_t)h.ncomp - first), hipMemcpyDeviceToHost, st),
              "layout flow: summary");
    check_hip(hipStreamSynchronize(st), "layout flow: summary");
  }
  f.comps.resize((size_t)h.ncomp);
  if (h.ncomp) std::memcpy(f.comps.data(), ho + at, sizeof(FlowComp) * (size_t)h.ncomp);
  f.active = true;
  return true;
}

void flow_pack(FlowGraph& f, DeviceBatch& db, hipStream_t st) {
  const auto* desc = db.desc.as<DevDesc>();
  if (db.n_reg)
    hipLaunchKernelGGL(flow_pack_reg_kernel, dim3((unsigned)((db.n_reg + 3) / 4)), dim3(256), 0, st,
                       db.reg_items(), desc, db.n_reg, f.ptr, f.adj, f.partner, f.comp_of, f.order,
                       f.comp_ptr, f.local, db.partners.as<uint8_t>());
  const int32_t ncsr = (int32_t)db.host_desc.size() - db.n_reg;
  if (ncsr) {
    int32_t most = 1;
    for (size_t i = (size_t)db.n_reg; i < db.host_desc.size(); ++i) most = std::max(most, db.host_desc[i].n);
    const unsigned slices = (unsigned)std::max(1, std::min((most + 15) / 16, 1024));
    hipLaunchKernelGGL(flow_pack_csr_kernel, dim3((unsigned)ncsr, slices), dim3(256), 0, st, desc + db.n_reg,
                       f.ptr, f.adj, f.partner, f.comp_of, f.order, f.comp_ptr, f.local, f.cpre, f.cmax,
                       db.csr_stitch, db.adj32.as<uint32_t>());
  }
  check_hip(hipGetLastError(), "layout flow: packing");
}

// Looks at a neighbour's color, 1 us each, after which a recovery is the
// host's: as long as the host takes for its own (about 10 ns a node).  The
// longest chain is 10 to 20 nodes where ids are in no order.
static int32_t recover_rounds(int32_t removed) { return 32 + std::min(removed / 128, 1024 - 32); }

bool flow_collect(FlowGraph& f, GraphBuilder& gb, const mpld_options& opt, DeviceBatch& db,
                  mpld_result* r) {
  std::lock_guard<std::mutex> lk(gb.mu);
  mpld_context* ctx = gb.ctx;
  hipStream_t st = gb.stream;
  const size_t nn = (size_t)f.n, nc = (size_t)f.ncomp;
  // scratch: head, component tallies, colors being recovered, places, bytes
  const size_t head_words = (sizeof(FlowHead) + 24) / 4;
  try {
    grow(gb.flow_ws, ctx, 4 * (head_words + 2 * nc + 2 * nn + (nn + 3) / 4));
  } catch (const NoMemory&) {
    return false;
  }
  int32_t* w = gb.flow_ws.as<int32_t>();
  auto* head = reinterpret_cast<FlowHead*>(w);
  auto* cstat = reinterpret_cast<int2*>(w + head_words);
  int32_t* col = w + head_words + 2 * nc;
  int32_t* qpos = col + nn;
  auto* colors = reinterpret_cast<int8_t*>(qpos + nn);
  const unsigned gn = flow_grid(f.n);
  hipLaunchKernelGGL(flow_colors_kernel, dim3(gn), dim3(256), 0, st, f.n, f.removed, head, f.queue, f.comp_of,
                     f.comp_ptr, f.local, db.colors.as<int8_t>(), col, qpos, cstat, f.ncomp);
  const int32_t rounds = ctx->recover_rounds >= 0 ? ctx->recover_rounds : recover_rounds(f.removed);
  if (f.simplify && f.removed)
    hipLaunchKernelGGL(flow_recover_kernel, dim3((unsigned)((f.removed + 255) / 256)), dim3(256), 0, st,
                       f.removed, opt.k, rounds, head, f.ptr, f.adj, f.partner, f.queue, qpos, col);
  hipLaunchKernelGGL(flow_tally_kernel, dim3(std::min(gn, 512u)), dim3(256), 0, st, f.n, f.ptr, f.adj, f.partner, f.comp_of,
                     col, colors, cstat, head);
  check_hip(hipGetLastError(), "layout flow: recovery");
  // page-locked staging: components of the nodes, head and tallies, records,
  // minimisation counts, colors
  const bool minimize = (opt.flags & MPLD_MINIMIZE) && db.min_out.p;
  const size_t b_comp = 4 * nn, b_head = 4 * head_words + 8 * nc, b_rec = sizeof(DevRecord) * nc,
               b_min = minimize ? 4 * nc : 0;
  auto up = [](size_t x) { return (x + 63) & ~(size_t)63; };
  const size_t o_head = up(b_comp), o_rec = o_head + up(b_head), o_min = o_rec + up(b_rec), o_col = o_min + up(b_min);
  if (!grow_pinned(gb.hout, o_col + nn)) fail(MPLD_E_NOMEM, "layout flow: pinned host memory");
  uint8_t* ho = gb.hout.as<uint8_t>();
  auto down = [&](size_t at, const void* p, size_t bytes) {
    if (bytes) check_hip(hipMemcpyAsync(ho + at, p, bytes, hipMemcpyDeviceToHost, st), "layout flow: results");
  };
  down(0, f.comp_of, b_comp);
  down(o_head, head, b_head);
  down(o_rec, db.recs.p, b_rec);
  down(o_min, db.min_out.p, b_min);
  down(o_col, colors, nn);
  check_hip(hipStreamSynchronize(st), "layout flow: results");
  device_time(db);
  FlowHead h;
  std::memcpy(&h, ho + o_head, sizeof(h));
  if (h.flags & kFlowChain) {
    ++ctx->recoveries_left;
    return false;
  }
  if (h.flags & kFlowNoColor) fail(MPLD_E_INTERNAL, "recovery found no free color");
  const auto* recs = reinterpret_cast<const DevRecord*>(ho + o_rec);
  const auto* stat = reinterpret_cast<const int32_t*>(ho + o_head + 4 * head_words);
  const auto* mins = reinterpret_cast<const int32_t*>(ho + o_min);
  r->colors.assign(reinterpret_cast<const int8_t*>(ho + o_col), reinterpret_cast<const int8_t*>(ho + o_col) + nn);
  r->comp_of.assign(reinterpret_cast<const int32_t*>(ho), reinterpret_cast<const int32_t*>(ho) + nn);
  r->comps.resize(nc);
  const bool trace = opt.flags & MPLD_TRACE_HASH;
  const bool marked = opt.flags & (MPLD_MARK_CONFLICTS | MPLD_MINIMIZE);
  for (size_t c = 0; c < nc; ++c) {
    if (recs[c].status < 0 || recs[c].status > MPLD_BUDGET_EXHAUSTED)
      fail(MPLD_E_INTERNAL, "search reported a broken state");
    mpld_comp_record& o = r->comps[c];
    o.size = f.comps[c].n;
    o.status = recs[c].status;
    o.nodes = (int64_t)recs[c].nodes;
    o.trace_hash = trace ? recs[c].hash : 0;
    o.depth_at_stop = recs[c].depth;
    o.stitches = o.status == MPLD_FEASIBLE || marked ? stat[2 * c + 1] : -1;
    o.first_node = f.comps[c].first;
    o.num_edges = f.comps[c].m2 / 2;
    o.conflicts = stat[2 * c] / 2;
    o.min_nodes = 0;
  }
  if (minimize)   // only register-tier items write their entry
    for (int32_t i = 0; i < db.n_reg; ++i) {
      const int32_t c = db.host_queue[(size_t)i];
      r->comps[(size_t)c].min_nodes = mins[c];
    }
  r->stitches = (int64_t)h.stitches;
  r->conflicts = (int64_t)h.conflicts;
  r->uncolored = (int64_t)h.uncolored;
  return true;
}

FlowGraph::~FlowGraph() {
  if (keep.p && keep.ctx) (void)hipStreamSynchronize(keep.ctx->stream);
}

void FlowGraph::drop() {
  if (keep.p && keep.ctx) (void)hipStreamSynchronize(keep.ctx->stream);
  keep.release();
  comps.clear();
  active = false;
}

void flow_split_out(FlowGraph& f, GraphBuilder& gb, int32_t* removal, int32_t* comp_of, int32_t* order,
                    int32_t* comp_ptr) {
  std::lock_guard<std::mutex> lk(gb.mu);
  hipStream_t st = gb.stream;
  const size_t nn = (size_t)f.n, nrem = (size_t)f.removed, nptr = (size_t)f.ncomp + 1;
  if (!grow_pinned(gb.hout, 4 * (2 * nn + nptr))) fail(MPLD_E_NOMEM, "layout flow: pinned host memory");
  int32_t* h = gb.hout.as<int32_t>();
  auto down = [&](int32_t* to, const int32_t* p, size_t count) {
    if (count) check_hip(hipMemcpyAsync(to, p, 4 * count, hipMemcpyDeviceToHost, st), "layout flow: split");
  };
  down(h, f.comp_of, nn);
  down(h + nn, f.queue, nrem);
  down(h + nn + nrem, f.order, nn - nrem);
  down(h + 2 * nn, f.comp_ptr, nptr);
  check_hip(hipStreamSynchronize(st), "layout flow: split");
  std::memcpy(comp_of, h, 4 * nn);
  std::memcpy(removal, h + nn, 4 * nrem);
  std::memcpy(order, h + nn + nrem, 4 * (nn - nrem));
  std::memcpy(comp_ptr, h + 2 * nn, 4 * nptr);
}

void flow_to_host(FlowGraph& f, GraphBuilder& gb, Graph& g, Split& s) {
  std::lock_guard<std::mutex> lk(gb.mu);
  const size_t nn = (size_t)f.n, words = (size_t)(f.local - f.ptr) + nn;
  // everything that is kept, in one copy: eight apart took longer than the
  // host's recovery of a small layout
  if (!grow_pinned(gb.hout, 4 * words)) fail(MPLD_E_NOMEM, "layout flow: pinned host memory");
  check_hip(hipMemcpyAsync(gb.hout.p, f.ptr, 4 * words, hipMemcpyDeviceToHost, gb.stream), "layout flow: download");
  check_hip(hipStreamSynchronize(gb.stream), "layout flow: download");
  const auto at = [&](const int32_t* p) { return gb.hout.as<int32_t>() + (p - f.ptr); };
  g = Graph();
  s = Split();
  g.n = f.n;
  g.num_ce = f.m;
  g.ptr.assign(at(f.ptr), at(f.ptr) + nn + 1);
  g.adj.assign(at(f.adj), at(f.adj) + 2 * (size_t)f.m);
  g.partner.assign(at(f.partner), at(f.partner) + nn);
  s.removal.assign(at(f.queue), at(f.queue) + f.removed);
  s.comp_of.assign(at(f.comp_of), at(f.comp_of) + nn);
  s.order.assign(at(f.order), at(f.order) + (nn - (size_t)f.removed));
  s.comp_ptr.assign(at(f.comp_ptr), at(f.comp_ptr) + f.ncomp + 1);
  s.local.assign(at(f.local), at(f.local) + nn);
}

}  // namespace mpld
