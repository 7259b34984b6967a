// graph_device.hip - the layout graph (Sec. 2.1: a conflict edge joins two
// features closer than d_min) built on the device, for requests large
// enough that the host's pair search dominates their front-end latency.
//
// The host copies the rectangles in; the device then
//   1. validates them, applies the midpoint stitch split (a scan gives the
//      nodes' ids) and takes the bounds, from which the host picks the search
//      grid;
//   2. counts the nodes per grid cell (atomics), scans the counts into cell
//      starts, and scatters ids and boxes into cell order;
//   3. gives every node one thread that tests the nodes of its 3x3 cell
//      neighbourhood (three contiguous runs of the cell order) with the
//      closed-box gap test, skipping its own stitch partner, and counts its
//      neighbours; a scan of the counts gives the row offsets;
//   4. writes the neighbour ids, each node's list sorted in place (lists are
//      short: the graph is a unit-disk-like geometric graph).
// The result is the CSR the rest of the front-end consumes: adjacency
// ascending per node, symmetric, no self loops or duplicates by
// construction.
//
// The simplification and sub-graph split that follow (Sec. 2.2; Algorithm 1
// splits the graph into sub-graphs) can run here too, on the CSR while it is
// still on the device: the split kernels reproduce the host's FIFO peeling
// order, components ordered by smallest id and BFS local numbering exactly,
// level by level (see the comment above them).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "graph_builder.h"

namespace mpld {

struct GridParams {
  int64_t minx, miny, cell;
  int32_t gx, gy;
};

__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t* __restrict__ p, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// ---- scans --------------------------------------------------------------------
//
// One launch a scan: a block takes the next tile by a ticket, publishes the
// tile's sum, and its first wave looks back over the published tiles, 64 at
// a time, to the nearest one that already knows its prefix.  Blocks only
// wait for tiles with smaller tickets, whose blocks run.  A published word
// holds an epoch (one per launch, so that nothing is cleared between
// launches), a state and a value, written and read whole.  Three launches a
// scan (tile sums, their scan, the tiles again) took 9 to 13 us of a split
// of 50k to 300k nodes, one takes 4 to 5.
static constexpr int kScanBlock = 256;               // threads per scan block
static constexpr int kScanItems = 8;                 // elements per thread
static constexpr int kScanTile = kScanBlock * kScanItems;

enum : uint64_t { kTileSum = 1, kTilePrefix = 2 };
__device__ __forceinline__ uint64_t tile_word(uint32_t epoch, uint64_t state, int32_t value) {
  return ((uint64_t)epoch << 34) | (state << 32) | (uint32_t)value;
}

// Exclusive prefix of tile `tile` (its sum: `sum`), by the lanes of one
// wave; every lane gets it.  -1: quit() said to wait no longer for the tiles
// before (where blocks take tiles by ticket there is no need to).
struct NeverQuit {
  __device__ __forceinline__ bool operator()() const { return false; }
};
template <class Q>
__device__ int32_t look_back(uint64_t* status, uint32_t epoch, int32_t tile, int32_t sum, Q&& quit) {
  const int32_t lane = (int32_t)(threadIdx.x & 63u);
  if (lane == 0)
    __hip_atomic_store(status + tile, tile_word(epoch, tile == 0 ? kTilePrefix : kTileSum, sum),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tile == 0) return 0;
  int32_t prefix = 0;
  for (int32_t end = tile - 1;; end -= 64) {
    const int32_t at = end - lane;
    uint64_t w = tile_word(epoch, kTilePrefix, 0);   // before tile 0: nothing
    for (;;) {
      if (at >= 0) w = __hip_atomic_load(status + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__ballot((uint32_t)(w >> 34) != epoch || ((w >> 32) & 3u) == 0) == 0ull) break;
      if (__ballot(quit()) != 0ull) return -1;
    }
    const uint64_t known = __ballot(((w >> 32) & 3u) == kTilePrefix);
    const int32_t stop = known ? (int32_t)__builtin_ctzll(known) : 63;
    int32_t v = lane <= stop ? (int32_t)(uint32_t)w : 0;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    prefix += v;
    if (known) break;
  }
  if (lane == 0)
    __hip_atomic_store(status + tile, tile_word(epoch, kTilePrefix, prefix + sum), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  return prefix;
}

// Exclusive prefix of x over a block of THREADS; `total` = the sum.
template <int THREADS>
__device__ __forceinline__ int32_t block_excl_scan(int32_t x, int32_t* wsum, int32_t& total) {
  const int32_t lane = (int32_t)(threadIdx.x & 63u), w = (int32_t)(threadIdx.x >> 6);
  int32_t incl = x;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t t = __shfl_up(incl, off, 64);
    if (lane >= off) incl += t;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  int32_t before = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < THREADS / 64; ++i) {
    const int32_t v = wsum[i];
    before += i < w ? v : 0;
    tot += v;
  }
  __syncthreads();   // wsum is reused by the next scan
  total = tot;
  return before + incl - x;
}

// What a scanning block shares.
struct ScanShared {
  int32_t wsum[kScanBlock / 64];
  int32_t tile, prefix;
};

// The block's tile: the next ticket past `base` (every thread gets it).
__device__ __forceinline__ int32_t take_tile(int32_t* ticket, uint32_t base, ScanShared& sh) {
  __syncthreads();   // the last tile's users are done
  if (threadIdx.x == 0) sh.tile = (int32_t)((uint32_t)atomicAdd(ticket, 1) - base);
  __syncthreads();
  return sh.tile;
}

// Exclusive prefix, over the whole launch, of this thread's x; `end` =
// prefix behind the block's last thread.  sh.prefix = -1: quit() ended it.
template <class Q = NeverQuit>
__device__ __forceinline__ int32_t device_excl_scan(int32_t x, uint64_t* status, uint32_t epoch, int32_t tile,
                                                    ScanShared& sh, int32_t& end, Q&& quit = Q()) {
  int32_t total;
  const int32_t ex = block_excl_scan<kScanBlock>(x, sh.wsum, total);
  if (threadIdx.x < 64) {
    const int32_t p = look_back(status, epoch, tile, total, quit);
    if (threadIdx.x == 0) sh.prefix = p;
  }
  __syncthreads();
  end = sh.prefix + total;
  return sh.prefix + ex;
}

__global__ __launch_bounds__(kScanBlock) void scan_kernel(const int32_t* __restrict__ in, int64_t n,
                                                          int32_t* __restrict__ out, int32_t* ticket,
                                                          uint32_t ticket_base, uint64_t* status,
                                                          uint32_t epoch) {
  __shared__ ScanShared sh;
  const int32_t tile = take_tile(ticket, ticket_base, sh);
  const int64_t base = (int64_t)tile * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int32_t v[kScanItems], s = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    v[j] = base + j < n ? in[base + j] : 0;
    s += v[j];
  }
  int32_t end;
  int32_t run = device_excl_scan(s, status, epoch, tile, sh, end);
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    if (base + j < n) out[base + j] = run;
    run += v[j];
  }
  if (tile == (int32_t)gridDim.x - 1 && threadIdx.x == 0) out[n] = end;
}

// ---- the layout graph ---------------------------------------------------------

struct LayoutHead {
  int32_t bad, splits;                     // a box with x1 < x0 or y1 < y0; rectangles cut in two
  int32_t minx, miny, maxx, maxy;          // of the nodes' lower-left corners
  uint32_t ext;                            // largest side
  int32_t pad;
};

// Rectangles to nodes, as prepare_layout on the host: a rectangle whose long
// side exceeds split_len becomes two nodes, cut at floor(L / 2), lower or left
// first; a node's id is its rectangle's plus the cuts before it.  The bounds
// for the search grid on the way.
__global__ __launch_bounds__(kScanBlock) void layout_nodes_kernel(const int4* __restrict__ rects, int32_t n,
                                                                  int32_t split_len, int4* __restrict__ box,
                                                                  int32_t* __restrict__ partner,
                                                                  int2* __restrict__ se, LayoutHead* head,
                                                                  int32_t* ticket, uint32_t ticket_base,
                                                                  uint64_t* status, uint32_t epoch) {
  __shared__ ScanShared sh;
  const int32_t tile = take_tile(ticket, ticket_base, sh);
  const int64_t base = (int64_t)tile * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t cut = 0;
  bool bad = false;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j)
    if (base + j < n) {
      const int4 r = rects[base + j];
      bad |= r.z < r.x || r.w < r.y;
      const int32_t len = max((int32_t)((uint32_t)r.z - (uint32_t)r.x), (int32_t)((uint32_t)r.w - (uint32_t)r.y));
      if (split_len > 0 && len > split_len) cut |= 1u << j;
    }
  int32_t end;
  int32_t before = device_excl_scan(__builtin_popcount(cut), status, epoch, tile, sh, end);
  int32_t minx = INT32_MAX, miny = INT32_MAX, maxx = INT32_MIN, maxy = INT32_MIN;
  uint32_t ext = 0;
  auto put = [&](int32_t id, const int4 r, int32_t mate) {
    box[id] = r;
    partner[id] = mate;
    minx = min(minx, r.x);
    miny = min(miny, r.y);
    maxx = max(maxx, r.x);
    maxy = max(maxy, r.y);
    ext = max(ext, max((uint32_t)r.z - (uint32_t)r.x, (uint32_t)r.w - (uint32_t)r.y));
  };
#pragma unroll
  for (int j = 0; j < kScanItems; ++j)
    if (base + j < n) {
      const int4 r = rects[base + j];
      const int32_t id = (int32_t)(base + j) + before;
      if ((cut >> j) & 1u) {
        const int32_t w = (int32_t)((uint32_t)r.z - (uint32_t)r.x), h = (int32_t)((uint32_t)r.w - (uint32_t)r.y);
        int4 lo = r, up = r;
        if (w >= h) up.x = lo.z = r.x + max(w, h) / 2;
        else up.y = lo.w = r.y + max(w, h) / 2;
        put(id, lo, id + 1);
        put(id + 1, up, id);
        se[before++] = int2{id, id + 1};
      } else {
        put(id, r, -1);
      }
    }
  for (int off = 32; off > 0; off >>= 1) {
    minx = min(minx, __shfl_xor(minx, off, 64));
    miny = min(miny, __shfl_xor(miny, off, 64));
    maxx = max(maxx, __shfl_xor(maxx, off, 64));
    maxy = max(maxy, __shfl_xor(maxy, off, 64));
    ext = max(ext, (uint32_t)__shfl_xor((int)ext, off, 64));
  }
  const bool any_bad = __ballot(bad) != 0ull;
  if ((threadIdx.x & 63) == 0) {
    if (any_bad) atomicOr(&head->bad, 1);
    atomicMin(&head->minx, minx);
    atomicMin(&head->miny, miny);
    atomicMax(&head->maxx, maxx);
    atomicMax(&head->maxy, maxy);
    atomicMax(&head->ext, ext);
  }
  if (tile == (int32_t)gridDim.x - 1 && threadIdx.x == 0) head->splits = end;
}

__global__ void layout_head_kernel(LayoutHead* head) {
  *head = LayoutHead{0, 0, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, 0, 0};
}

// Nodes per cell; a node's place within its cell is the count it found.
__global__ __launch_bounds__(256) void cell_count_kernel(const int4* __restrict__ box, int32_t nn,
                                                         GridParams g, int2* __restrict__ cell_of,
                                                         int32_t* __restrict__ cnt) {
  const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= nn) return;
  const int4 b = box[i];
  const int64_t cx = ((int64_t)b.x - g.minx) / g.cell, cy = ((int64_t)b.y - g.miny) / g.cell;
  const int32_t c = (int32_t)(cy * g.gx + cx);
  cell_of[i] = int2{c, atomicAdd(&cnt[c], 1)};
}

// Boxes, ids and stitch partners in cell order ({id, partner, cell}: one
// 16-byte word).
__global__ __launch_bounds__(256) void cell_scatter_kernel(const int4* __restrict__ box,
                                                           const int32_t* __restrict__ partner,
                                                           int32_t nn, const int2* __restrict__ cell_of,
                                                           const int32_t* __restrict__ start,
                                                           int4* __restrict__ sbox, int4* __restrict__ sid) {
  const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= nn) return;
  const int2 c = cell_of[i];
  const int32_t pos = start[c.x] + c.y;
  sbox[pos] = box[i];
  sid[pos] = int4{i, partner[i], c.x, 0};
}

// Tests the node at place p of the cell order against its 3x3 cell
// neighbourhood: three contiguous runs of the cell order.  f(id) for every
// conflict partner, in no order.
template <class F>
__device__ __forceinline__ void for_partners(const int4* __restrict__ sbox, const int4* __restrict__ sid,
                                             const int32_t* __restrict__ start, int32_t p, const int4 me,
                                             const GridParams& g, int64_t d2, F&& f) {
  const int4 a = sbox[p];
  const int32_t cy = me.z / g.gx, cx = me.z - cy * g.gx;
  const int32_t x0 = cx > 0 ? cx - 1 : 0, x1 = cx + 1 < g.gx ? cx + 1 : g.gx - 1;
  const int32_t y0 = cy > 0 ? cy - 1 : 0, y1 = cy + 1 < g.gy ? cy + 1 : g.gy - 1;
  for (int32_t yy = y0; yy <= y1; ++yy) {
    const int32_t q0 = start[yy * g.gx + x0], q1 = start[yy * g.gx + x1 + 1];
    for (int32_t q = q0; q < q1; ++q) {
      const int4 b = sbox[q];
      const int64_t dx = max(max((int64_t)0, (int64_t)b.x - a.z), (int64_t)a.x - b.z);
      const int64_t dy = max(max((int64_t)0, (int64_t)b.y - a.w), (int64_t)a.y - b.w);
      if (q == p || dx * dx + dy * dy >= d2) continue;
      const int32_t id = sid[q].x;
      if (id != me.y) f(id);   // not the other half of a split feature
    }
  }
}

// Neighbour lists up to this long stay in the scratch that the counting pass
// writes them to; the writing pass searches again for longer ones only.
// 16 entries hold every list of the sparse layouts (mean degree 1 to 3); the
// second search of all nodes had made the writing pass 41 us at 296k nodes.
static constexpr int kKeptNeighbours = 16;

// One thread per node (cell order): counts its neighbours into deg[id], and
// keeps the first ones (kept[j * nn + p]).  UP: only neighbours of larger id.
template <bool UP>
__global__ __launch_bounds__(256) void neighbour_count_kernel(
    const int4* __restrict__ sbox, const int4* __restrict__ sid, const int32_t* __restrict__ start,
    int32_t nn, GridParams g, int64_t d2, int32_t* __restrict__ deg, int32_t* __restrict__ kept) {
  const int32_t p = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (p >= nn) return;
  const int4 me = sid[p];
  int32_t k = 0;
  for_partners(sbox, sid, start, p, me, g, d2, [&](int32_t id) {
    if (UP && id < me.x) return;
    if (k < kKeptNeighbours) kept[(int64_t)k * nn + p] = id;
    ++k;
  });
  deg[me.x] = k;
}

// Each node's list, ascending.  UP: as pairs (id, larger id); out then holds
// two words an entry.
template <bool UP>
__global__ __launch_bounds__(256) void neighbour_write_kernel(
    const int4* __restrict__ sbox, const int4* __restrict__ sid, const int32_t* __restrict__ start,
    int32_t nn, GridParams g, int64_t d2, const int32_t* __restrict__ ptr,
    const int32_t* __restrict__ kept, int32_t* __restrict__ out, int64_t room) {
  const int32_t p = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (p >= nn) return;
  const int4 me = sid[p];
  const int64_t t0 = ptr[me.x];
  const int32_t k = (int32_t)(ptr[me.x + 1] - t0);
  if (k == 0 || t0 + k > room) return;   // no room: the host sees the total and asks again
  constexpr int S = UP ? 2 : 1;
  int32_t* list = out + S * t0 + (S - 1);
  int32_t have = 0;
  auto insert = [&](int32_t id) {   // insertion sort of the short list
    int32_t j = have++;
    for (; j > 0 && list[S * (j - 1)] > id; --j) list[S * j] = list[S * (j - 1)];
    list[S * j] = id;
  };
  if (k <= kKeptNeighbours) {
    for (int32_t i = 0; i < k; ++i) {
      // the place of an entry is the number of smaller ones
      const int32_t id = kept[(int64_t)i * nn + p];
      int32_t r = 0;
      for (int32_t j = 0; j < k; ++j) r += kept[(int64_t)j * nn + p] < id ? 1 : 0;
      list[S * r] = id;
    }
  } else {
    for_partners(sbox, sid, start, p, me, g, d2, [&](int32_t id) {
      if (!UP || id > me.x) insert(id);
    });
  }
  if (UP)
    for (int32_t i = 0; i < k; ++i) list[2 * i - 1] = me.x;
}

// ---- simplification and sub-graph split ------------------------------------
//
// The sequential definitions (FIFO peeling of nodes of conflict degree < k,
// queue seeded in ascending id, a popped node lowering its neighbours'
// degrees in ascending id; components of the rest ordered by smallest id;
// local numbering by BFS from that node, neighbours in ascending id) are
// reproduced exactly, in level-synchronous form:
//
// Peeling.  Node w of d = deg(w) neighbours is queued when its
// (d - k + 1)-th neighbour is popped, and pops follow the queue: a popped
// node u at place p queues exactly those neighbours w of which d(w) - k
// neighbours have a place before p.  That needs no levels and no order
// within one: it holds for one u alone (the count grows along w's popped
// neighbours), and places given at the same time are behind p and do not
// count.  So a level of the queue (the nodes queued while the level before
// it is popped) is one launch: count each node's children, scan over the
// level in queue order, write the children in the node's ascending list
// order.  Level 0 is the seed in id order.  The first levels, which hold
// nearly every node, take the whole device; what is left, usually small, goes
// on in one workgroup whose levels are separated by barriers.
//
// Components: union-find over the whole device, the larger root hooked
// under the smaller (so each root is its component's smallest id), numbered
// by root id with a scan.  BFS: one wave per component of at most 64 nodes
// (ranks by id, neighbour masks over the ranks, the queue kept in a lane
// register), a workgroup per larger component, several for the largest.
constexpr int kSplitThreads = 1024;   // the one-workgroup kernels
constexpr int kSplitGrid = 2048;      // grid-stride kernels: blocks of 256
// BFS of the components above 64 nodes: those above kGiantNodes by several
// workgroups, one component after another, the others by one workgroup each;
// those above kBigNodes by several too where there are no more than kFewBigs
// (dense components of 2000 and 4000 nodes: 0.3 against 0.9 and 1.2 ms).
constexpr int kMidThreads = 512;
constexpr int kMidGrid = 512;
constexpr int32_t kBigNodes = 512, kFewBigs = 3, kGiantNodes = 4096;
constexpr int kGiantBlocks = 128;
constexpr int32_t kMeetSpin = 1 << 22;   // looks at a word before a wait is given up: some seconds
constexpr int kLevelGrid = 1024;      // level kernels: blocks of 256 taking tiles by ticket

// Levels 1 .. kWideLevels are found by launches over the device.
constexpr int kWideLevels = 5;
// SplitArgs.ctl: [2L], [2L + 1] the queue range of level L, [kCtlTicket + L]
// the ticket of the launch that pops level L.
constexpr int kCtlTicket = 2 * (kWideLevels + 2);
// ... then the lengths of the lists of larger components, and the meetings of
// the workgroups that number the largest.
constexpr int kCtlMids = kCtlTicket + kWideLevels + 2, kCtlBigs = kCtlMids + 1, kCtlGiants = kCtlMids + 2,
              kCtlMeet = kCtlMids + 3, kCtlOver = kCtlMids + 4;
constexpr int kCtlWords = kCtlMids + 5;
static_assert(kCtlWords <= 64, "ctl is 64 words at least");

#define SPLIT_FOR(v, n)                                                                 \
  for (int32_t v = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); v < (n);          \
       v += (int32_t)(gridDim.x * blockDim.x))

// The split is left to the host (kCtlOver): the launches behind find nothing
// to do, and the counts say so.
__device__ __forceinline__ bool left_to_host(const SplitArgs& a) { return a.ctl[kCtlOver] != 0; }
__device__ __forceinline__ void leave_to_host(const SplitArgs& a) {
  a.ctl[kCtlOver] = 1;
  a.counts[0] = a.n;
  a.counts[1] = -1;
}

// fault (may be null): a nonzero word makes the graph one without pairs (the
// kernels behind take ascending, symmetric lists for granted).
__global__ __launch_bounds__(256) void split_init_kernel(SplitArgs a, const int32_t* fault, int32_t* ptr) {
  if (blockIdx.x == 0 && threadIdx.x < kCtlWords) a.ctl[threadIdx.x] = 0;
  const bool none = fault && *fault;
  SPLIT_FOR(v, a.n) {
    if (none) {
      ptr[v] = 0;
      if (v == 0) ptr[a.n] = 0;
    }
    a.csize[v] = 0;
    a.fill[v] = 0;
    a.qpos[v] = -1;
    a.parent[v] = v;
    a.words[v] = 0;
    a.local[v] = -1;
    a.comp_of[v] = -1;
  }
}

// Level 0: the nodes of degree < k in id order.
__global__ __launch_bounds__(kScanBlock) void split_seed_kernel(SplitArgs a, int32_t* ticket,
                                                                uint32_t ticket_base, uint64_t* status,
                                                                uint32_t epoch) {
  __shared__ ScanShared sh;
  const int32_t tile = take_tile(ticket, ticket_base, sh);
  const int64_t base = (int64_t)tile * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t seeds = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j)
    if (base + j < a.n) {
      const int32_t deg = a.ptr[base + j + 1] - a.ptr[base + j];
      if (a.simplify && deg < a.k) seeds |= 1u << j;
      if (deg > a.limits.degree) a.ctl[kCtlOver] = 1;
    }
  int32_t end;
  int32_t run = device_excl_scan(__builtin_popcount(seeds), status, epoch, tile, sh, end);
#pragma unroll
  for (int j = 0; j < kScanItems; ++j)
    if ((seeds >> j) & 1u) {
      a.queue[run] = (int32_t)(base + j);
      a.qpos[base + j] = run++;
    }
  if (tile == (int32_t)gridDim.x - 1 && threadIdx.x == 0) a.ctl[1] = end;   // level 0 = [0, end)
}

// Whether the node popped at place p queues its neighbour w.
__device__ __forceinline__ bool queues(const SplitArgs& a, int32_t w, int32_t p) {
  const int32_t t0 = a.ptr[w], t1 = a.ptr[w + 1], want = t1 - t0 - a.k;
  if (want < 0) return false;   // a seed
  int32_t r = 0;
  for (int32_t t = t0; t < t1; ++t) r += (uint32_t)a.qpos[a.adj[t]] < (uint32_t)p ? 1 : 0;   // -1: no place
  return r == want;
}

// One node per group of G lanes, which share its list chunk by chunk: how
// many neighbours w have test(w) (every lane of the group gets it), then
// put(w, place) for them in list order from place `at` on.  `hit` keeps the
// first 64 neighbours' answers.
template <int G, class F>
__device__ __forceinline__ int32_t group_count(const SplitArgs& a, int32_t u, uint64_t& hit, F&& test) {
  const int32_t j = (int32_t)threadIdx.x & (G - 1), shift = (int32_t)(threadIdx.x & 63u) - j;
  const int32_t t0 = u >= 0 ? a.ptr[u] : 0, t1 = u >= 0 ? a.ptr[u + 1] : 0;
  int32_t c = 0;
  hit = 0;
  for (int32_t t = t0, ch = 0; t < t1; t += G, ch += G) {
    const bool h = t + j < t1 && test(a.adj[t + j]);
    const uint64_t b = (__ballot(h) >> shift) & ((1ull << G) - 1);
    c += __builtin_popcountll(b);
    if (ch < 64) hit |= b << ch;
  }
  return c;
}
template <int G, class F, class P>
__device__ __forceinline__ void group_put(const SplitArgs& a, int32_t u, uint64_t hit, int32_t at, F&& test, P&& put) {
  const int32_t j = (int32_t)threadIdx.x & (G - 1), shift = (int32_t)(threadIdx.x & 63u) - j;
  const int32_t t0 = a.ptr[u], t1 = a.ptr[u + 1];
  for (int32_t t = t0, ch = 0; t < t1; t += G, ch += G) {
    uint64_t b = (hit >> (ch & 63)) & ((1ull << G) - 1);
    if (ch >= 64) b = (__ballot(t + j < t1 && test(a.adj[t + j])) >> shift) & ((1ull << G) - 1);
    if ((b >> j) & 1u) put(a.adj[t + j], at + __builtin_popcountll(b & ((1ull << j) - 1)));
    at += __builtin_popcountll(b);
  }
}
// `at` of the group's first lane.
template <int G>
__device__ __forceinline__ int32_t of_group(int32_t at) {
  return G > 1 ? __shfl(at, (int32_t)(threadIdx.x & 63u) & ~(G - 1), 64) : at;
}
template <int G>
__device__ __forceinline__ bool leads_group() {
  return ((int32_t)threadIdx.x & (G - 1)) == 0;
}

// The children of the node at place p, and their places.
template <int G>
__device__ __forceinline__ int32_t count_children(const SplitArgs& a, int32_t u, int32_t p, uint64_t& hit) {
  return group_count<G>(a, u, hit, [&](int32_t w) { return queues(a, w, p); });
}
template <int G>
__device__ __forceinline__ void write_children(const SplitArgs& a, int32_t u, int32_t p, uint64_t hit, int32_t at) {
  group_put<G>(a, u, hit, at, [&](int32_t w) { return queues(a, w, p); },
               [&](int32_t w, int32_t q) {
                 if (q < a.n) {   // always: places are a permutation
                   a.queue[q] = w;
                   a.qpos[w] = q;
                 }
               });
}

// Pops level L: level L + 1 behind it.  Groups of G lanes share a node (one
// lane each on level 0, whose nodes have fewer than k neighbours).
template <int G>
__global__ __launch_bounds__(kScanBlock) void split_level_kernel(SplitArgs a, int32_t L, uint64_t* status,
                                                                 uint32_t epoch) {
  __shared__ ScanShared sh;
  constexpr int32_t kNodes = kScanBlock / G;
  const int32_t lo = a.ctl[2 * L], hi = a.ctl[2 * L + 1];
  const int32_t tiles = left_to_host(a) ? 0 : (hi - lo + kNodes - 1) / kNodes;
  if (tiles == 0 && blockIdx.x == 0 && threadIdx.x == 0) {
    a.ctl[2 * L + 2] = hi;
    a.ctl[2 * L + 3] = hi;
  }
  for (;;) {
    if (tiles <= (int32_t)blockIdx.x) break;   // no tile can be left for this block
    const int32_t tile = take_tile(a.ctl + kCtlTicket + L, 0, sh);
    if (tile >= tiles) break;
    const int32_t p = lo + tile * kNodes + (int32_t)threadIdx.x / G;
    const int32_t u = p < hi ? a.queue[p] : -1;
    uint64_t hit;
    const int32_t c = count_children<G>(a, u, p, hit);
    int32_t end;
    const int32_t at =
        of_group<G>(hi + device_excl_scan(leads_group<G>() ? c : 0, status, epoch, tile, sh, end));
    if (c) write_children<G>(a, u, p, hit, at);
    if (tile == tiles - 1 && threadIdx.x == 0) {
      a.ctl[2 * L + 2] = hi;
      a.ctl[2 * L + 3] = hi + end;
    }
  }
}

// The remaining levels on one workgroup.
__global__ __launch_bounds__(kSplitThreads) void split_peel_kernel(SplitArgs a) {
  __shared__ int32_t wsum[kSplitThreads / 64];
  constexpr int32_t G = 8, kNodes = kSplitThreads / G;
  int32_t lo = a.ctl[2 * (kWideLevels + 1)], hi = a.ctl[2 * (kWideLevels + 1) + 1];
  bool over = left_to_host(a);
  for (int32_t levels = 0; lo < hi && !over; ++levels) {
    if (levels == a.limits.peel) {
      over = true;
      break;
    }
    int32_t next = hi;
    for (int32_t base = lo; base < hi; base += kNodes) {
      const int32_t p = base + (int32_t)threadIdx.x / G;
      const int32_t u = p < hi ? a.queue[p] : -1;
      uint64_t hit;
      const int32_t c = count_children<G>(a, u, p, hit);
      int32_t total;
      const int32_t at =
          of_group<G>(next + block_excl_scan<kSplitThreads>(leads_group<G>() ? c : 0, wsum, total));
      if (c) write_children<G>(a, u, p, hit, at);
      next += total;
    }
    __syncthreads();   // the next level reads what this one wrote
    lo = hi;
    hi = next;
  }
  __syncthreads();   // (all have looked at the word)
  if (threadIdx.x == 0) {
    if (over) leave_to_host(a);
    else a.counts[0] = hi;
  }
}

__device__ __forceinline__ int32_t ld_agent(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of x with path halving (parent[x] < x for every non-root, so every
// rewrite points x at one of its ancestors and the loop ends).
__device__ int32_t uf_find(int32_t* parent, int32_t x) {
  for (;;) {
    const int32_t p = ld_agent(parent + x);
    if (p == x) return x;
    const int32_t g = ld_agent(parent + p);
    if (g == p) return p;
    __hip_atomic_store(parent + x, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x = g;
  }
}

// Hooks the larger of two roots under the smaller; a failed CAS means that
// root was just hooked elsewhere: find again.  G lanes share a node's list:
// 4 on sparse graphs, where the time is each node's chain of loads (24 us with
// one lane on 296k nodes of 2.5 neighbours); one on dense graphs, whose pairs
// soon all ask for the same few roots' words (872k entries over one component
// took 0.17 ms with one lane a node, 1.7 ms with 16).
template <int G>
__global__ __launch_bounds__(256) void uf_unite_kernel(SplitArgs a) {
  if (left_to_host(a)) return;
  const int32_t groups = (int32_t)(gridDim.x * blockDim.x) / G;
  for (int32_t v = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x) / G; v < a.n; v += groups) {
    if (a.qpos[v] >= 0) continue;
    for (int32_t t = a.ptr[v] + ((int32_t)threadIdx.x & (G - 1)); t < a.ptr[v + 1]; t += G) {
      const int32_t w = a.adj[t];
      if (w < v || a.qpos[w] >= 0) continue;
      for (;;) {
        const int32_t ra = uf_find(a.parent, v), rb = uf_find(a.parent, w);
        if (ra == rb) break;
        const int32_t hi = ra > rb ? ra : rb, lo = ra > rb ? rb : ra;
        if (atomicCAS(a.parent + hi, hi, lo) == hi) break;
      }
    }
  }
}

// Every core node's root (read-only walks: the forest is final here), the
// roots numbered in id order.
__global__ __launch_bounds__(kScanBlock) void uf_root_kernel(SplitArgs a, int32_t* ticket, uint32_t ticket_base,
                                                             uint64_t* status, uint32_t epoch) {
  __shared__ ScanShared sh;
  const int32_t tile = take_tile(ticket, ticket_base, sh);
  // a thread's nodes are kScanBlock apart: neighbouring threads read
  // neighbouring parents, and the tile's order is kept by its rounds
  const bool none = left_to_host(a);
  int32_t carry = 0;
  int32_t num[kScanItems];
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    const int64_t v = (int64_t)tile * kScanTile + j * kScanBlock + threadIdx.x;
    int32_t r = -1;   // (removed nodes have no parent)
    if (v < a.n && a.qpos[v] < 0 && !none) {
      r = (int32_t)v;
      for (int32_t p = a.parent[r]; p != r; p = a.parent[r]) r = p;
    }
    if (v < a.n) a.root[v] = r;
    const int32_t flag = v < a.n && r == (int32_t)v ? 1 : 0;
    int32_t total;
    const int32_t ex = block_excl_scan<kScanBlock>(flag, sh.wsum, total);
    num[j] = flag ? carry + ex : -1;
    carry += total;
  }
  if (threadIdx.x < 64) {
    const int32_t p = look_back(status, epoch, tile, carry, NeverQuit());
    if (threadIdx.x == 0) sh.prefix = p;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kScanItems; ++j)
    if (num[j] >= 0) a.cid[(int64_t)tile * kScanTile + j * kScanBlock + threadIdx.x] = sh.prefix + num[j];
  if (tile == (int32_t)gridDim.x - 1 && threadIdx.x == 0) a.cid[a.n] = sh.prefix + carry;
}

// Component of every core node (roots numbered in id order), its size, and
// the root of every component.  A wave whose nodes are all of one component
// adds them at once: a component of 40k nodes is one address.
__global__ __launch_bounds__(256) void comp_kernel(SplitArgs a) {
  SPLIT_FOR(v, a.n) {
    const int32_t r = a.root[v];
    if (r < 0) continue;
    const int32_t c = a.cid[r];
    a.comp_of[v] = c;
    if (r == v) a.parent[c] = v;   // parent[] is free now: root of component c
    const uint64_t active = __ballot(true);
    if (__ballot(c == __builtin_amdgcn_readfirstlane(c)) == active) {
      if ((threadIdx.x & 63u) == (unsigned)__builtin_ctzll(active))
        atomicAdd(a.csize + c, __builtin_popcountll(active));
    } else {
      atomicAdd(a.csize + c, 1);
    }
  }
}

// Core nodes of the components of at most 64 nodes listed per component (any
// order within it); the larger components in two lists, by who numbers them.
__global__ __launch_bounds__(256) void comp_list_kernel(SplitArgs a) {
  if (blockIdx.x == 0 && threadIdx.x == 0) a.counts[1] = left_to_host(a) ? -1 : a.cid[a.n];
  SPLIT_FOR(v, a.n) {
    const int32_t c = a.comp_of[v];
    if (c < 0) continue;
    const int32_t base = a.comp_ptr[c], sz = a.comp_ptr[c + 1] - base;
    if (sz <= 64)
      a.list[base + atomicAdd(a.fill + c, 1)] = v;
    else if (a.root[v] == v && sz <= kBigNodes)
      a.mids[atomicAdd(a.ctl + kCtlMids, 1)] = c;
    else if (a.root[v] == v && sz <= kGiantNodes)
      a.bigs[atomicAdd(a.ctl + kCtlBigs, 1)] = c;
    else if (a.root[v] == v)
      a.giants[atomicAdd(a.ctl + kCtlGiants, 1)] = c;
  }
}

__device__ __forceinline__ uint64_t rdlane64(uint64_t x, uint32_t l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, (int)l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), (int)l);
  return ((uint64_t)hi << 32) | lo;
}

// BFS numbering of the components of at most 64 nodes, one wave each.
// Lane i holds node x_i of the component; its rank by id is its index in
// the neighbour masks (rank 0 is the smallest id: the root).
__global__ __launch_bounds__(256) void bfs_small_kernel(SplitArgs a) {
  const int32_t lane = (int32_t)(threadIdx.x & 63u);
  const int32_t ncomp = a.cid[a.n];
  const int32_t waves = (int32_t)(gridDim.x * (blockDim.x >> 6));
  for (int32_t c = (int32_t)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); c < ncomp;
       c += waves) {
    const int32_t base = a.comp_ptr[c], sz = a.comp_ptr[c + 1] - base;
    if (sz > 64) continue;
    const bool in = lane < sz;
    const int32_t x = in ? a.list[base + lane] : INT32_MAX;
    int32_t r = 0;
    for (int32_t j = 0; j < sz; ++j) r += __builtin_amdgcn_readlane(x, j) < x ? 1 : 0;
    if (in) a.rank[x] = r;
    __threadfence_block();
    uint64_t m = 0;
    if (in)
      for (int32_t t = a.ptr[x]; t < a.ptr[x + 1]; ++t) {
        const int32_t w = a.adj[t];
        if (a.comp_of[w] == c) m |= 1ull << a.rank[w];
      }
    // lane i's mask is indexed by its rank: mk[rank] via a lane shuffle
    const int32_t src = [&] {
      // the lane whose rank equals this lane's index
      int32_t s = 0;
      for (int32_t j = 0; j < sz; ++j)
        if (__builtin_amdgcn_readlane(r, j) == lane) s = j;
      return s;
    }();
    const uint32_t mlo = (uint32_t)__shfl((int)(uint32_t)m, src, 64);
    const uint32_t mhi = (uint32_t)__shfl((int)(uint32_t)(m >> 32), src, 64);
    const uint64_t mk = ((uint64_t)mhi << 32) | mlo;   // mask of rank `lane`
    // sequential BFS over ranks; q: lane t holds the rank at queue position t
    int32_t q = 0;
    uint64_t seen = 1ull;
    int32_t tail = 1;
    for (int32_t head = 0; head < tail; ++head) {
      const int32_t u = __builtin_amdgcn_readlane(q, head);
      uint64_t nb = rdlane64(mk, (uint32_t)u) & ~seen;
      seen |= nb;
      while (nb) {
        const int32_t b = (int32_t)__builtin_ctzll(nb);
        nb &= nb - 1;
        q = lane == tail ? b : q;
        ++tail;
      }
    }
    // the lane of rank q[t] is numbered t
    int32_t pos = -1;
    for (int32_t t = 0; t < sz; ++t)
      if (__builtin_amdgcn_readlane(q, t) == r) pos = t;
    if (in && pos >= 0) {
      a.local[x] = pos;
      a.order[base + pos] = x;
    }
  }
}

// BFS numbering of larger components.  As in the peeling, no levels are
// marked: the node u at position p numbers its unnumbered neighbour w exactly
// when no neighbour of w has a position before p, positions given meanwhile
// being behind p.  A level of the queue is counted, scanned and written.
// AGENT: positions are written and read across workgroups.
template <bool AGENT>
__device__ __forceinline__ int32_t ld_local(const SplitArgs& a, int32_t v) {
  return AGENT ? ld_agent(a.local + v) : a.local[v];
}
template <bool AGENT>
__device__ __forceinline__ bool numbers(const SplitArgs& a, int32_t w, int32_t p) {
  const int32_t gone = a.qpos[w], at = ld_local<AGENT>(a, w), t0 = a.ptr[w], t1 = a.ptr[w + 1];
  bool before = gone >= 0 || (uint32_t)at <= (uint32_t)p;   // removed, or numbered by then
  if (before || p == 0) return !before;   // (nothing is before the root)
  if (t1 - t0 <= 64) {
#pragma unroll 4
    for (int32_t t = t0; t < t1; ++t) before |= (uint32_t)ld_local<AGENT>(a, a.adj[t]) < (uint32_t)p;
    return !before;
  }
  // of a dense component's lists only the front is read: most nodes have a
  // neighbour there that is (one component of 1200 nodes, all pairs: 31 -> 9 ms)
  for (int32_t t = t0; t < t1 && !before; t += 16) {
#pragma unroll
    for (int32_t j = 0; j < 16; ++j)
      before |= (uint32_t)ld_local<AGENT>(a, a.adj[t + j < t1 ? t + j : t1 - 1]) < (uint32_t)p;
  }
  return !before;
}

// A workgroup each.
__global__ __launch_bounds__(kMidThreads) void bfs_mid_kernel(SplitArgs a) {
  __shared__ int32_t wsum[kMidThreads / 64];
  constexpr int32_t G = 8, kNodes = kMidThreads / G;
  const int32_t mids = a.ctl[kCtlMids], bigs = a.ctl[kCtlBigs];
  const int32_t first = bigs > kFewBigs ? bigs : 0;   // the larger ones first
  int32_t levels = 0;   // of all its components
  for (int32_t i = (int32_t)blockIdx.x; i < first + mids; i += (int32_t)gridDim.x) {
    const int32_t c = i < first ? a.bigs[i] : a.mids[i - first], sz = a.comp_ptr[c + 1] - a.comp_ptr[c];
    int32_t* order = a.order + a.comp_ptr[c];
    if (threadIdx.x == 0) {
      order[0] = a.parent[c];
      a.local[a.parent[c]] = 0;
    }
    __syncthreads();
    for (int32_t lo = 0, hi = 1; lo < hi;) {
      if (++levels > a.limits.mid) {
        if (threadIdx.x == 0) leave_to_host(a);
        return;
      }
      int32_t next = hi;
      for (int32_t base = lo; base < hi; base += kNodes) {
        const int32_t p = base + (int32_t)threadIdx.x / G;
        const int32_t u = p < hi ? order[p] : -1;
        const auto test = [&](int32_t w) { return numbers<false>(a, w, p); };
        uint64_t hit;
        const int32_t found = group_count<G>(a, u, hit, test);
        int32_t total;
        const int32_t at =
            of_group<G>(next + block_excl_scan<kMidThreads>(leads_group<G>() ? found : 0, wsum, total));
        if (found)
          group_put<G>(a, u, hit, at, test, [&](int32_t w, int32_t q) {
            if (q < sz) {
              order[q] = w;
              a.local[w] = q;
            }
          });
        next += total;
      }
      __syncthreads();   // the next level reads what this one wrote
      lo = hi;
      hi = next;
    }
  }
}

// Larger ones, one after another on kGiantBlocks workgroups that meet after
// each level: a level of some 400 nodes of 22 neighbours (a packed window)
// is 50 blocks' work of one wave-wide step, and one workgroup took 140 us for
// it.  Positions and order go past the caches of one compute unit (agent
// scope).  All blocks of this launch fit the device at once; should others'
// kernels keep some out, every wait ends all the same: a block that has waited
// far too long sets kMeetLost in the word that counts the meetings, every wait
// looks at that bit, and a meeting counts only if the word is read without it.
// So a block that leaves is waited for by nobody, and the graph is then split
// on the host.
constexpr int32_t kMeetLost = 1 << 30;
__global__ __launch_bounds__(kScanBlock) void bfs_giant_kernel(SplitArgs a) {
  __shared__ ScanShared sh;
  __shared__ int32_t lost;
  constexpr int32_t G = 32, kNodes = kScanBlock / G;
  int32_t* const word = a.ctl + kCtlMeet;
  const int32_t giants = a.ctl[kCtlGiants], bigs = a.ctl[kCtlBigs];
  const int32_t count = left_to_host(a) ? 0 : giants + (bigs > kFewBigs ? 0 : bigs);
  // tiles' words of even and of odd levels: a block that has met the others
  // after a level may write the next level's before a slow one has read the
  // last of this level's, so they are apart (a block is never two levels ahead)
  uint64_t* const words = reinterpret_cast<uint64_t*>(((uintptr_t)a.words + 7) & ~(uintptr_t)7);
  const int32_t level_words = a.n / kNodes + 1;
  uint32_t tag = 0;
  int32_t met = 0;
  const auto meet = [&] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);   // this wave's stores are out
    __syncthreads();
    if (threadIdx.x == 0) {
      met += (int32_t)gridDim.x;
      int32_t have = atomicAdd(word, 1) + 1;
      for (int32_t spin = 0; have < met; ++spin) {
        if (spin < a.limits.spin) {
          have = ld_agent(word);
        } else {   // only while the meeting is incomplete: then nobody has passed it
          const int32_t seen = atomicCAS(word, have, have | kMeetLost);
          have = seen == have ? have | kMeetLost : seen;
        }
      }
      lost = have & kMeetLost;
      if (lost) leave_to_host(a);
    }
    __syncthreads();
    asm volatile("" ::: "memory");
    return lost == 0;
  };
  // in a level this block has not met the others yet: the meeting is incomplete
  int32_t waited = 0;
  const auto quit = [&] {
    if (ld_agent(word) & kMeetLost) return true;
    if (++waited < a.limits.spin) return false;
    atomicOr(word, kMeetLost);
    return true;
  };
  for (int32_t g = 0; g < count; ++g) {
    const int32_t c = g < giants ? a.giants[g] : a.bigs[g - giants], sz = a.comp_ptr[c + 1] - a.comp_ptr[c];
    int32_t* order = a.order + a.comp_ptr[c];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      __hip_atomic_store(order, a.parent[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(a.local + a.parent[c], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!meet()) return;
    // a component that is growing so slowly that it will not get there: one as
    // wide as it is long has a sixteenth of its nodes after a quarter of its levels
    const uint32_t quarter = tag + (uint32_t)a.limits.giant / 4u;
    for (int32_t lo = 0, hi = 1; lo < hi;) {
      if (++tag > (uint32_t)a.limits.giant || (tag == quarter && hi < sz / 12)) {   // all workgroups count alike
        if (threadIdx.x == 0) leave_to_host(a);
        return;
      }
      waited = 0;
      uint64_t* const status = words + (tag & 1u ? level_words : 0);
      const int32_t tiles = (hi - lo + kNodes - 1) / kNodes;
      for (int32_t tile = (int32_t)blockIdx.x; tile < tiles; tile += (int32_t)gridDim.x) {
        const int32_t p = lo + tile * kNodes + (int32_t)threadIdx.x / G;
        const int32_t u = p < hi ? ld_agent(order + p) : -1;
        const auto test = [&](int32_t w) { return numbers<true>(a, w, p); };
        uint64_t hit;
        const int32_t found = group_count<G>(a, u, hit, test);
        int32_t end;
        const int32_t at =
            of_group<G>(hi + device_excl_scan(leads_group<G>() ? found : 0, status, tag, tile, sh, end, quit));
        if (sh.prefix < 0) {
          if (threadIdx.x == 0) leave_to_host(a);
          return;
        }
        if (found)
          group_put<G>(a, u, hit, at, test, [&](int32_t w, int32_t q) {
            if (q < sz) {
              __hip_atomic_store(order + q, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              __hip_atomic_store(a.local + w, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
          });
      }
      if (!meet()) return;
      const uint64_t last = __hip_atomic_load(status + tiles - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      lo = hi;
      hi += (int32_t)(uint32_t)last;   // the last tile's prefix with its own: the level's total
    }
  }
}

// ---- host side --------------------------------------------------------------

GraphBuilder* graph_builder_create(mpld_context* ctx, bool own_stream) {
  auto* gb = new GraphBuilder();
  gb->ctx = ctx;
  if (own_stream) {
    hipStream_t s = nullptr;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) {
      delete gb;
      fail(MPLD_E_DEVICE, "hipStreamCreateWithFlags failed for the graph builder");
    }
    gb->stream = s;
    gb->own_stream = true;
  } else {
    gb->stream = ctx->stream;
  }
  return gb;
}

void graph_builder_destroy(GraphBuilder* gb) { delete gb; }


// What a scanning launch of `tiles` tiles works with: the ticket and the
// value it starts from, the tiles' words and the launch's epoch.
struct ScanArgs {
  int32_t* ticket;
  uint32_t base;
  uint64_t* status;
  uint32_t epoch;
};

constexpr uint32_t kLastEpoch = (1u << 30) - 1;   // of a tile's word
// tickets: how many the launch takes (one a block), 0 when it has its own.
static ScanArgs scan_args(GraphBuilder& gb, int64_t tiles, int64_t tickets) {
  const size_t bytes = 64 + 8 * (size_t)tiles;
  if (gb.tiles.bytes < bytes || gb.epoch >= kLastEpoch) {
    // launches on the way still use the words that go back
    if (gb.tiles.p) check_hip(hipStreamSynchronize(gb.stream), "graph builder: scan");
    grow(gb.tiles, gb.ctx, bytes);
    gb.epoch = 0;
    gb.tickets = 0;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(256), dim3(256), 0, gb.stream, gb.tiles.as<int32_t>(),
                       (int64_t)(gb.tiles.bytes / 4), 0);
  }
  ScanArgs a{gb.tiles.as<int32_t>(), gb.tickets, gb.tiles.as<uint64_t>() + 8, ++gb.epoch};
  gb.tickets += (uint32_t)tickets;
  return a;
}

void scan_reserve(GraphBuilder& gb, int64_t n) { (void)scan_args(gb, std::max<int64_t>(1, (n + 31) / 32), 0); }

// Checks the launches so far.  One that failed took no tickets: the counts start
// anew with the next scan, or its workgroups would look for tiles that are not
// theirs.
static void check_launches(GraphBuilder& gb, const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) gb.epoch = kLastEpoch;
  check_hip(e, what);
}

void scan(GraphBuilder& gb, const int32_t* in, int64_t n, int32_t* out) {
  const int64_t tiles = std::max<int64_t>(1, (n + kScanTile - 1) / kScanTile);
  const ScanArgs sa = scan_args(gb, tiles, tiles);
  hipLaunchKernelGGL(scan_kernel, dim3((unsigned)tiles), dim3(kScanBlock), 0, gb.stream, in, n, out, sa.ticket,
                     sa.base, sa.status, sa.epoch);
  check_launches(gb, "graph builder: scan");
}

// What a split may take on the device before the host is to do it (identical
// results).  A level of the peeling's tail takes some 2.5 us, one of the
// numbering 1.5 to 2 us in a workgroup and 10 us by many, whatever is in it, so
// a deep graph would take as long as it is deep: lines with two neighbours on
// either side (k = 3) peel from their two ends, 100,000 in 50,000 levels, over
// 100 ms where the host's whole path takes 2 to 6.  Layouts of 8,000 to 200,000
// rectangles have at most 8 levels in the tail, packed windows of 1,500, 5,000
// and 40,000 (16,600, 57,000 and 476,000 nodes and pairs) at most 21, 34 and 96
// in the numbering: these go through (26, 43 and 210 are allowed), and what is
// given up has taken a fifth of the host's time at most.  A node of very many
// neighbours takes 0.65 us for each over all passes, one load after another (one
// of 1500 in 91,500 nodes and pairs: 1.4 ms a decomposition, 0.75 on the host).
static SplitLimits split_limits(int64_t n, int64_t adj_entries) {
  const int64_t size = n + adj_entries / 2;
  const auto levels = [&](int64_t least, int64_t per) { return (int32_t)std::min<int64_t>(least + size / per, 1 << 20); };
  return SplitLimits{levels(24, 4000), levels(32, 1000), levels(20, 2500), std::min(levels(256, 100), 2048), kMeetSpin};
}

SplitArgs enqueue_split(GraphBuilder& gb, int32_t n, const int32_t* dptr, const int32_t* dadj,
                        int64_t adj_entries, int32_t k, bool simplify, int32_t* out, int32_t* scratch_at, const int32_t* fault,
                        int32_t* ptr_w) {
  const size_t nn = (size_t)n;
  SplitArgs a{};
  a.limits = split_limits(n, adj_entries);
  if (gb.ctx->split_levels >= 0)
    a.limits.peel = a.limits.mid = a.limits.giant = gb.ctx->split_levels;
  a.n = n;
  a.k = k;
  a.simplify = simplify ? 1 : 0;
  a.ptr = dptr;
  a.adj = dadj;
  a.counts = out;
  a.queue = out + 2;
  a.comp_of = a.queue + nn;
  a.order = a.comp_of + nn;
  a.comp_ptr = a.order + nn;
  a.local = a.comp_ptr + nn + 1;
  const size_t stride = split_scratch_words(n) / kSplitScratch;
  int32_t* q = scratch_at;
  int32_t** scratch[kSplitScratch] = {&a.qpos, &a.parent, &a.root, &a.cid,  &a.csize,  &a.fill,
                                      &a.list, &a.rank,   &a.mids, &a.bigs, &a.giants, &a.words,
                                      &a.ctl};
  for (int32_t** d : scratch) {
    *d = q;
    q += stride;
  }
  hipStream_t st = gb.stream;
  const unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, kSplitGrid);
  auto wide = [&](void (*kern)(SplitArgs)) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, a);
  };
  const int64_t tiles = (n + kScanTile - 1) / kScanTile;
  hipLaunchKernelGGL(split_init_kernel, dim3(grid), dim3(256), 0, st, a, fault, ptr_w);
  ScanArgs sa = scan_args(gb, tiles, tiles);
  hipLaunchKernelGGL(split_seed_kernel, dim3((unsigned)tiles), dim3(kScanBlock), 0, st, a, sa.ticket, sa.base,
                     sa.status, sa.epoch);
  for (int32_t L = 0; simplify && L <= kWideLevels; ++L) {
    const int64_t most = L == 0 ? (n + kScanBlock - 1) / kScanBlock : (n + 31) / 32;
    sa = scan_args(gb, most, 0);
    const dim3 lg((unsigned)std::min<int64_t>(most, kLevelGrid));
    if (L == 0)
      hipLaunchKernelGGL(split_level_kernel<1>, lg, dim3(kScanBlock), 0, st, a, L, sa.status, sa.epoch);
    else
      hipLaunchKernelGGL(split_level_kernel<8>, lg, dim3(kScanBlock), 0, st, a, L, sa.status, sa.epoch);
  }
  hipLaunchKernelGGL(split_peel_kernel, dim3(1), dim3(kSplitThreads), 0, st, a);
  if (adj_entries > 8 * (int64_t)n)
    wide(uf_unite_kernel<1>);
  else
    hipLaunchKernelGGL(uf_unite_kernel<4>, dim3((unsigned)std::min<int64_t>((n + 63) / 64, 2 * kSplitGrid)), dim3(256),
                       0, st, a);
  sa = scan_args(gb, tiles, tiles);     // component ids; cid[n] = components
  hipLaunchKernelGGL(uf_root_kernel, dim3((unsigned)tiles), dim3(kScanBlock), 0, st, a, sa.ticket, sa.base,
                     sa.status, sa.epoch);
  wide(comp_kernel);
  scan(gb, a.csize, n, a.comp_ptr);
  wide(comp_list_kernel);
  wide(bfs_small_kernel);
  hipLaunchKernelGGL(bfs_mid_kernel, dim3((unsigned)std::min<int64_t>(kMidGrid, n / 65 + 1)), dim3(kMidThreads), 0,
                     st, a);
  if (n > kBigNodes)
    hipLaunchKernelGGL(bfs_giant_kernel, dim3(kGiantBlocks), dim3(kScanBlock), 0, st, a);
  check_launches(gb, "device split");
  return a;
}

// The same in the builder's own workspace: outputs at its front.
static void enqueue_split(GraphBuilder& gb, int32_t n, const int32_t* dptr, const int32_t* dadj,
                          int64_t adj_entries, int32_t k, bool simplify) {
  grow(gb.split_ws, gb.ctx, sizeof(int32_t) * (split_out_words(n) + split_scratch_words(n)));
  int32_t* w = gb.split_ws.as<int32_t>();
  enqueue_split(gb, n, dptr, dadj, adj_entries, k, simplify, w, w + split_out_words(n), nullptr, nullptr);
}

// Split from the copied-back words of split_ws; false if the device gave up.
static bool collect_split(const int32_t* h, int32_t n, Split& s) {
  const size_t nn = (size_t)n;
  const int32_t removed = h[0], ncomp = h[1];
  const int32_t* queue = h + 2;
  const int32_t* comp_of = queue + nn;
  const int32_t* order = comp_of + nn;
  const int32_t* comp_ptr = order + nn;
  const int32_t* local = comp_ptr + nn + 1;
  if (ncomp == -1) return false;
  if (removed < 0 || removed > n || ncomp < 0 || ncomp > n)
    fail(MPLD_E_INTERNAL, "device split returned bad counts");
  s = Split();
  s.removal.assign(queue, queue + removed);
  s.comp_of.assign(comp_of, comp_of + nn);
  s.comp_ptr.assign(comp_ptr, comp_ptr + ncomp + 1);
  s.order.assign(order, order + s.comp_ptr.back());
  s.local.assign(local, local + nn);
  return true;
}

void graph_builder_reserve(GraphBuilder& gb, int32_t nodes) {
  // sizes as a build and split of `nodes` nodes with up to 8 adjacency
  // entries and 4 grid cells per node would ask for
  std::lock_guard<std::mutex> lk(gb.mu);
  mpld_context* ctx = gb.ctx;
  const size_t n = (size_t)std::max(nodes, 1), cells = 4 * n, adj = 8 * n;
  grow(gb.rects, ctx, 16 * n + sizeof(LayoutHead));
  for (DevBuf* b : {&gb.partner, &gb.se}) grow(*b, ctx, 4 * n);
  grow(gb.cell_of, ctx, 8 * n);
  for (DevBuf* b : {&gb.box, &gb.sbox, &gb.sid}) grow(*b, ctx, 16 * n);
  for (DevBuf* b : {&gb.cnt, &gb.start}) grow(*b, ctx, 4 * (cells + 1));
  grow(gb.kept, ctx, 4 * n * kKeptNeighbours);
  for (DevBuf* b : {&gb.deg, &gb.ptr}) grow(*b, ctx, 4 * (n + 1));
  grow(gb.adj, ctx, 4 * adj);
  (void)scan_args(gb, (int64_t)std::max(cells / kScanTile, n / 32) + 1, 0);
  grow(gb.split_ws, ctx, 4 * (split_out_words((int64_t)n) + split_scratch_words((int64_t)n)));
  for (int i = 0; i < GraphBuilder::kStagings; ++i) {
    std::unique_ptr<Staging> sg(new Staging());
    if (!grow_pinned(sg->in, 16 * n) ||
        !grow_pinned(sg->out, 4 * (2 * n + 1 + adj + split_out_words((int64_t)n))))
      fail(MPLD_E_NOMEM, "graph builder: pinned host memory");
    std::lock_guard<std::mutex> sl(gb.smu);
    if (gb.stagings == GraphBuilder::kStagings) break;
    gb.spare.push_back(std::move(sg));
    ++gb.stagings;
  }
}

// Copies the rectangles to the staging (before the builder's lock).
static void stage_rects(Staging& sg, const mpld_rect* rects, int32_t n) {
  const size_t bytes = sizeof(mpld_rect) * (size_t)n;
  if (!grow_pinned(sg.in, bytes)) fail(MPLD_E_NOMEM, "graph builder: pinned host memory");
  std::memcpy(sg.in.p, rects, bytes);
}

// Nodes, stitch pairs and search grid of a staged layout, on the device, and
// its nodes in cell order; waits once, for the grid's bounds.  Returns the
// number of nodes.  Caller holds the lock.
struct LayoutGrid {
  GridParams g{};
  int32_t nn = 0, nse = 0;
  int64_t d2 = 0;
};
static LayoutGrid layout_cells(GraphBuilder& gb, Staging& sg, const mpld_rect* rects, int32_t n, int32_t dmin,
                               int32_t split_len) {
  mpld_context* ctx = gb.ctx;
  hipStream_t s = gb.stream;
  check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (2 * (int64_t)n >= INT32_MAX)
    fail(MPLD_E_INVALID, "layout too large for the device graph builder");
  const size_t nr = (size_t)n, most = nr * (split_len > 0 ? 2 : 1);
  grow(gb.rects, ctx, sizeof(int4) * nr + sizeof(LayoutHead));
  grow(gb.box, ctx, sizeof(int4) * most);
  grow(gb.partner, ctx, sizeof(int32_t) * most);
  grow(gb.se, ctx, sizeof(int32_t) * most);
  if (!grow_pinned(sg.out, sizeof(LayoutHead))) fail(MPLD_E_NOMEM, "graph builder: pinned host memory");
  auto* head = gb.rects.as<LayoutHead>();
  auto* drects = reinterpret_cast<int4*>(gb.rects.as<uint8_t>() + sizeof(LayoutHead));
  hipLaunchKernelGGL(layout_head_kernel, dim3(1), dim3(1), 0, s, head);
  check_hip(hipMemcpyAsync(drects, sg.in.p, sizeof(int4) * nr, hipMemcpyHostToDevice, s),
            "graph builder: upload rectangles");
  const int64_t tiles = (n + kScanTile - 1) / kScanTile;
  const ScanArgs sa = scan_args(gb, tiles, tiles);
  hipLaunchKernelGGL(layout_nodes_kernel, dim3((unsigned)tiles), dim3(kScanBlock), 0, s, drects, n, split_len,
                     gb.box.as<int4>(), gb.partner.as<int32_t>(), gb.se.as<int2>(), head, sa.ticket, sa.base,
                     sa.status, sa.epoch);
  check_launches(gb, "graph builder: nodes");
  check_hip(hipMemcpyAsync(sg.out.p, head, sizeof(LayoutHead), hipMemcpyDeviceToHost, s),
            "graph builder: bounds");
  check_hip(hipStreamSynchronize(s), "graph builder: bounds");
  LayoutHead h;
  std::memcpy(&h, sg.out.p, sizeof(h));
  if (h.bad) {   // the host names the rectangle
    LayoutPrep lp;
    prepare_layout(rects, n, dmin, split_len, lp);
    fail(MPLD_E_INTERNAL, "the device refused a layout that the host takes");
  }
  LayoutGrid out;
  if (2 * ((int64_t)n + h.splits) >= INT32_MAX)
    fail(MPLD_E_INVALID, "layout too large for the device graph builder");
  out.nn = n + h.splits;
  out.nse = h.splits;
  out.d2 = (int64_t)dmin * dmin;
  LayoutPrep lp;
  layout_grid(h.minx, h.miny, h.maxx, h.maxy, std::max<int64_t>(1, h.ext), out.nn, dmin, lp);
  const int64_t ncell = lp.gx * lp.gy;
  if (ncell >= INT32_MAX) fail(MPLD_E_INVALID, "layout too large for the device graph builder");
  const GridParams g{lp.minx, lp.miny, lp.cell, (int32_t)lp.gx, (int32_t)lp.gy};
  out.g = g;
  const int32_t nn = out.nn;
  const size_t nb = (size_t)nn;
  grow(gb.cell_of, ctx, sizeof(int2) * nb);
  grow(gb.cnt, ctx, sizeof(int32_t) * (size_t)(ncell + 1));
  grow(gb.start, ctx, sizeof(int32_t) * (size_t)(ncell + 1));
  grow(gb.sbox, ctx, sizeof(int4) * nb);
  grow(gb.sid, ctx, sizeof(int4) * nb);
  grow(gb.kept, ctx, sizeof(int32_t) * nb * kKeptNeighbours);
  grow(gb.deg, ctx, sizeof(int32_t) * (nb + 1));
  grow(gb.ptr, ctx, sizeof(int32_t) * (nb + 1));
  const dim3 blocks((unsigned)((nn + 255) / 256));
  const unsigned cblocks = (unsigned)std::min<int64_t>((ncell + 255) / 256, 4096);
  hipLaunchKernelGGL(fill_i32_kernel, dim3(cblocks), dim3(256), 0, s, gb.cnt.as<int32_t>(), ncell, 0);
  hipLaunchKernelGGL(cell_count_kernel, blocks, dim3(256), 0, s, gb.box.as<int4>(), nn, g,
                     gb.cell_of.as<int2>(), gb.cnt.as<int32_t>());
  scan(gb, gb.cnt.as<int32_t>(), ncell, gb.start.as<int32_t>());
  hipLaunchKernelGGL(cell_scatter_kernel, blocks, dim3(256), 0, s, gb.box.as<int4>(),
                     gb.partner.as<int32_t>(), nn, gb.cell_of.as<int2>(), gb.start.as<int32_t>(),
                     gb.sbox.as<int4>(), gb.sid.as<int4>());
  check_hip(hipGetLastError(), "graph builder: cells");
  return out;
}

// Neighbour lists (CSR, or with UP the pairs of smaller and larger id) of the
// nodes in cell order: offsets in gb.ptr, lists in gb.adj; waits for their
// total, which it returns.
template <bool UP>
static int32_t layout_lists(GraphBuilder& gb, Staging& sg, const LayoutGrid& L) {
  hipStream_t s = gb.stream;
  const dim3 blocks((unsigned)((L.nn + 255) / 256));
  constexpr int64_t kWords = UP ? 2 : 1;
  hipLaunchKernelGGL(neighbour_count_kernel<UP>, blocks, dim3(256), 0, s, gb.sbox.as<int4>(), gb.sid.as<int4>(),
                     gb.start.as<int32_t>(), L.nn, L.g, L.d2, gb.deg.as<int32_t>(), gb.kept.as<int32_t>());
  scan(gb, gb.deg.as<int32_t>(), L.nn, gb.ptr.as<int32_t>());
  int32_t total = 0;
  check_hip(hipMemcpyAsync(sg.out.p, gb.ptr.as<int32_t>() + L.nn, sizeof(int32_t), hipMemcpyDeviceToHost, s),
            "graph builder: edge total");
  // the lists go where the last layouts' went while the total is on its way;
  // a longer one is written again once its room is known
  for (int pass = 0; pass < 2; ++pass) {
    const int64_t room = (int64_t)(gb.adj.bytes / (4 * kWords));
    if (room > 0)
      hipLaunchKernelGGL(neighbour_write_kernel<UP>, blocks, dim3(256), 0, s, gb.sbox.as<int4>(),
                         gb.sid.as<int4>(), gb.start.as<int32_t>(), L.nn, L.g, L.d2, gb.ptr.as<int32_t>(),
                         gb.kept.as<int32_t>(), gb.adj.as<int32_t>(), room);
    check_hip(hipGetLastError(), "graph builder: neighbours");
    if (pass == 0) {
      check_hip(hipStreamSynchronize(s), "graph builder: counts");
      std::memcpy(&total, sg.out.p, sizeof(total));
      if (total <= room) break;
      grow(gb.adj, gb.ctx, 4 * (size_t)kWords * (size_t)total);
    }
  }
  return total;
}

bool build_layout_graph_device(GraphBuilder& gb, const mpld_rect* rects, int32_t n, int32_t dmin,
                               int32_t split_len, Graph& g, Split* split, int32_t k, bool simplify) {
  g = Graph();
  if (n <= 0 || !rects || dmin < 0 || split_len < 0) {   // a fault, or nothing to do
    LayoutPrep lp;
    prepare_layout(rects, n, dmin, split_len, lp);
    g.ptr.assign(1, 0);
    if (split) {
      *split = Split();
      split->comp_ptr.push_back(0);
    }
    return split != nullptr;
  }
  StagingUse use(gb);
  Staging& sg = *use;
  stage_rects(sg, rects, n);
  int32_t nn = 0, total = 0;
  size_t nb = 0;
  {
    std::lock_guard<std::mutex> lk(gb.mu);
    const LayoutGrid L = layout_cells(gb, sg, rects, n, dmin, split_len);
    hipStream_t s = gb.stream;
    nn = L.nn;
    nb = (size_t)nn;
    total = layout_lists<false>(gb, sg, L);
    if (split && !device_split_pays(nn, total, k)) split = nullptr;   // the caller splits on the host
    if (split) enqueue_split(gb, nn, gb.ptr.as<int32_t>(), gb.adj.as<int32_t>(), total, k, simplify);
    const size_t split_words = split ? split_out_words(nn) : 0;
    const size_t out_bytes = sizeof(int32_t) * ((nb + 1) + nb + (size_t)total + split_words);
    if (!grow_pinned(sg.out, out_bytes)) fail(MPLD_E_NOMEM, "graph builder: pinned host memory");
    int32_t* h = sg.out.as<int32_t>();
    const auto down = [&](int32_t* to, const void* p, size_t words) {
      if (words)
        check_hip(hipMemcpyAsync(to, p, sizeof(int32_t) * words, hipMemcpyDeviceToHost, s),
                  "graph builder: download");
    };
    down(h, gb.ptr.p, nb + 1);
    down(h + nb + 1, gb.partner.p, nb);
    down(h + 2 * nb + 1, gb.adj.p, (size_t)total);
    down(h + 2 * nb + 1 + total, gb.split_ws.p, split_words);
    check_hip(hipStreamSynchronize(s), "graph builder");
  }
  const int32_t* hptr = sg.out.as<int32_t>();
  const int32_t* hmate = hptr + nb + 1;
  const int32_t* hadj = hmate + nb;
  g.n = nn;
  g.ptr.assign(hptr, hptr + nb + 1);
  g.partner.assign(hmate, hmate + nb);
  g.adj.assign(hadj, hadj + total);
  g.num_ce = total / 2;
  if (!split) return false;
  const bool done = collect_split(hadj + total, nn, *split);
  if (!done) ++gb.ctx->splits_left;
  return done;
}

void build_layout_pairs_device(GraphBuilder& gb, const mpld_rect* rects, int32_t n, int32_t dmin,
                               int32_t split_len, DevicePairs& out) {
  out = DevicePairs();
  if (n <= 0 || !rects || dmin < 0 || split_len < 0) {   // a fault, or nothing to do
    LayoutPrep lp;
    prepare_layout(rects, n, dmin, split_len, lp);
    return;
  }
  StagingUse use(gb);
  Staging& sg = *use;
  stage_rects(sg, rects, n);
  size_t total = 0, nse = 0;
  {
    std::lock_guard<std::mutex> lk(gb.mu);
    const LayoutGrid L = layout_cells(gb, sg, rects, n, dmin, split_len);
    hipStream_t s = gb.stream;
    total = (size_t)layout_lists<true>(gb, sg, L);
    nse = (size_t)L.nse;
    out.num_nodes = L.nn;
    if (!grow_pinned(sg.out, 8 * (total + nse) + 8)) fail(MPLD_E_NOMEM, "graph builder: pinned host memory");
    int32_t* h = sg.out.as<int32_t>();
    if (total)
      check_hip(hipMemcpyAsync(h, gb.adj.p, 8 * total, hipMemcpyDeviceToHost, s), "graph builder: download pairs");
    if (nse)
      check_hip(hipMemcpyAsync(h + 2 * total, gb.se.p, 8 * nse, hipMemcpyDeviceToHost, s),
                "graph builder: download stitch pairs");
    out.ce.reset(new int32_t[2 * (total + nse) + 1]);
    check_hip(hipStreamSynchronize(s), "graph builder");
  }
  out.num_ce = (int64_t)total;
  out.num_se = (int64_t)nse;
  std::memcpy(out.ce.get(), sg.out.p, 8 * (total + nse));
}

}  // namespace mpld
