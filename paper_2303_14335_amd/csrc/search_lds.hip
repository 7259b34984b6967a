// search_lds.hip - LDS tier of the exact-cover search (components of more
// than 64 nodes), one 64-lane wavefront per component.
//
// Same matrix and rules as the register tier (Sec. 2.3, Algorithm 1), with
// the state spread over W = ceil(n/64) words per bit-plane:
//   PL[c][w]  (c < k) color plane: bit v set while color c is open at v,
//             i.e. while row (v, c) is active;
//   PL[k][w]  uncovered primary columns P.
// Column choice (count + select): lane l takes words l, l+64, ...; a
// bit-sliced adder over the k planes gives per-word count-bit planes,
// narrowing P from the top count bit leaves the lowest-count columns of the
// word, and the key (count << 24 | index) of its lowest one goes into a
// DPP min-reduction over the wave: the global minimum is the fewest-rows,
// lowest-index column.  All-ones means P is empty (a solution).
// Cover of row (v, c) (Eq. 2): P loses v, and each neighbour u of v loses
// color c through an LDS atomic AND that returns the old word, so a lane
// knows whether it removed an active row; those rows go to an undo log of
// 32-bit entries (plane << 26 | node), after one entry for v's P bit.
// Uncover (Eq. 2) ORs entries back.  Because OR commutes and the removed
// bits of different levels are disjoint, a backtrack over several levels is
// one lane-parallel pass over the log suffix: a per-depth bit set marks
// levels whose column still has untried rows, and the deepest such level
// is found with a word scan instead of popping level by level.
//
// Placement: the planes always live in LDS.  Small components run on one
// wave and also keep their neighbour lists, level headers and undo log in
// LDS (the per-depth bit set in lane registers); "big" components run on a
// workgroup of up to 16 waves that share the column scan, and keep the
// per-depth bit set in LDS and the rest in global memory (header and log in
// a per-worker scratch area).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_types.h"
#include "mpld.h"
#include "seq_reserve.h"
#include "seq_types.h"
#include "trace.h"
#include "wave_ops.h"

namespace mpld {

static constexpr uint32_t kNoneL = 0xffffffffu;
static constexpr uint32_t kNoKey = 0xffffffffu;
static constexpr uint32_t kEntryNodeBits = 26;   // undo entry: plane << 26 | node

__device__ __forceinline__ uint32_t uni(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}
__device__ __forceinline__ uint64_t uni64(uint64_t x) {
  return ((uint64_t)uni((uint32_t)(x >> 32)) << 32) | uni((uint32_t)x);
}

constexpr int bits_for(int x) { return x == 0 ? 0 : 1 + bits_for(x >> 1); }

__device__ __forceinline__ uint32_t wave_min(uint32_t m) { return wave_min_u32(m); }

// Key of the lowest-count, lowest-index uncovered column in word w:
// (count << 24) | (64 w + bit), or kNoKey when the word has none.
template <int K>
__device__ __forceinline__ uint32_t word_key(const uint64_t* PL, uint32_t W, uint32_t w) {
  constexpr int NB = bits_for(K);
  uint64_t a[K];
#pragma unroll
  for (int c = 0; c < K; ++c) a[c] = PL[(uint32_t)c * W + w];
  const uint64_t p = PL[(uint32_t)K * W + w];
  uint64_t cnt[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) cnt[b] = 0;
#pragma unroll
  for (int c = 0; c < K; ++c) {
    uint64_t carry = a[c];
#pragma unroll
    for (int b = 0; b < bits_for(c + 1); ++b) {
      const uint64_t t = cnt[b] & carry;
      cnt[b] ^= carry;
      carry = t;
    }
  }
  uint64_t cand = p;
  uint32_t t = 0;
#pragma unroll
  for (int b = NB - 1; b >= 0; --b) {
    const uint64_t x = cand & ~cnt[b];
    if (x) cand = x;
    else t |= 1u << b;
  }
  const uint32_t key = (t << 24) | (w << 6) | (uint32_t)__builtin_ctzll(cand | (1ull << 63));
  return p ? key : kNoKey;
}

// Byte layout of the LDS area of one component.
struct LdsLayout {
  uint32_t W, E, pl_off, a_off, adj_off, hdr_off, ent_off, ctl_off, col_off, total;
};

// Undo-log capacity: one entry per level (its P bit) plus the removed rows,
// at most one per (neighbour, color) pair and at most one per incidence.
__host__ __device__ inline uint32_t lds_log_entries(int32_t n, int32_t k, int64_t adj_words) {
  const int64_t incid = adj_words - n - 1;   // 2m
  const int64_t nk = (int64_t)n * k;
  return (uint32_t)(n + (incid < nk ? incid : nk));
}

__host__ __device__ inline LdsLayout lds_layout(int32_t n, int32_t k, int64_t adj_words, bool big,
                                               bool stitch = false) {
  LdsLayout L;
  L.W = (uint32_t)((n + 63) / 64);
  L.E = lds_log_entries(n, k, adj_words);
  uint32_t off = big ? 16u : 0u;   // big: the workgroup's queue pop result first
  L.pl_off = off;
  off += 8u * (uint32_t)(k + 1) * L.W;
  L.a_off = off;
  if (big) off += 8u * L.W;   // one bit per depth 0 .. n-1 (small: in registers)
  L.ctl_off = off;
  if (big) off += 128u;       // per-wave minima, loop status, final depth
  L.col_off = off;            // stitch-aware order: each covered node's color
  if (big && stitch) off += (uint32_t)n;
  L.adj_off = off;
  if (!big) off += 4u * (uint32_t)adj_words;
  off = (off + 7u) & ~7u;
  L.hdr_off = off;
  if (!big) off += 8u * (uint32_t)n;
  L.ent_off = off;
  if (!big) off += 4u * L.E;
  L.total = (off + 7u) & ~7u;
  return L;
}

// Level header: v | c << 24 | rows << 28 | log start << 36.
__device__ __forceinline__ uint64_t make_hdr(uint32_t v, uint32_t c, uint32_t rows, uint32_t est) {
  return (uint64_t)v | ((uint64_t)c << 24) | ((uint64_t)rows << 28) | ((uint64_t)est << 36);
}

// put(i, get(i)) for i < count over the wave, eight reads in flight: one at
// a time, a component's lists came to LDS at about one memory latency per 64
// words (some 80 us at n = 1800).
template <class G, class P>
__device__ __forceinline__ void load_words(uint32_t count, G&& get, P&& put) {
  const uint32_t lane = __lane_id();
  for (uint32_t i0 = lane; i0 < count; i0 += 64u * 8u) {
    uint32_t x[8];
#pragma unroll
    for (uint32_t q = 0; q < 8u; ++q) x[q] = i0 + 64u * q < count ? get(i0 + 64u * q) : 0u;
#pragma unroll
    for (uint32_t q = 0; q < 8u; ++q)
      if (i0 + 64u * q < count) put(i0 + 64u * q, x[q]);
  }
}

// A sequence-engine task on a CSR tier (the *_seq forms of the one-wave
// solvers): where it starts, how far it may go, and what becomes of it.
struct SeqIo {
  SeqArgs a;
  SeqTask task;
  int32_t id;          // its result: a.results[id]
  uint64_t stop;       // nodes it counts before it is cut, if it may be
  uint64_t limit;      // nodes after which the search's budget is out
  bool load;           // the component's lists are not in LDS yet
  bool cuts;           // at `stop` it is cut (false: saved whole, one piece)
  bool force;          // without room for that it goes on to `limit` (false: it is left as it was)
};

// Room for `pieces` pieces of a stack of `depth` levels and `ents` log entries;
// the first task and arena byte, false when there is none.
__device__ __forceinline__ bool seq_reserve(const SeqIo& io, uint32_t pieces, uint32_t n, uint32_t plane_bytes,
                                            uint32_t depth, uint32_t ents, int32_t& child, int64_t& at) {
  const uint64_t bytes =
      ((uint64_t)pieces * (plane_bytes + 64u) + 8ull * depth + 4ull * ents + n + 127u) & ~63ull;
  return seq_take_room(io.a, bytes, (int32_t)pieces, child, at);
}
// Pieces that a stack with `open` untried levels is cut into.
__device__ __forceinline__ uint32_t seq_pieces(const SeqIo& io, uint32_t open) {
  if (!io.cuts || open <= (uint32_t)kSeqFirstLevels) return 1u;
  const uint32_t singles = open - (uint32_t)kSeqFirstLevels;
  return 1u + (singles < (uint32_t)kSeqPieces - 1u ? singles : (uint32_t)kSeqPieces - 1u);
}
// Room for n colors; -1: none.
__device__ __forceinline__ int64_t seq_reserve_colors(const SeqIo& io, uint32_t n) {
  const uint64_t bytes = (n + 63u) & ~63u;
  int32_t none;
  int64_t at;
  return seq_take_room(io.a, bytes, 0, none, at) ? at : -1;
}
// Colors of the nodes below the piece, from its predecessor's array.
__device__ __forceinline__ void seq_copy_colors(const SeqIo& io, int64_t to, uint32_t n) {
  if (io.task.col < 0) return;
  const uint4* src = reinterpret_cast<const uint4*>(io.a.arena + io.task.col);
  uint4* dst = reinterpret_cast<uint4*>(io.a.arena + to);
  for (uint32_t i = __lane_id(); i < (n + 15u) / 16u; i += 64u) dst[i] = src[i];
}
// Every lane writes the same record.
__device__ __forceinline__ void seq_put_piece(const SeqIo& io, int32_t id, int32_t kind, uint32_t dbase,
                                              uint32_t levels, uint32_t nent, uint32_t row_in, int64_t at,
                                              int64_t col) {
  SeqTask t;
  t.comp = io.task.comp;
  t.kind = kind;
  t.dbase = dbase;
  t.levels = levels;
  t.nent = nent;
  t.row_in = row_in;
  t.at = at;
  t.col = col;
  t.open = 0;
  io.a.tasks[id] = t;
  io.a.results[id].status = kSeqWaiting;
}
__device__ __forceinline__ void seq_put_result(const SeqIo& io, int32_t status, uint32_t depth, uint64_t nodes,
                                               uint64_t hash, int64_t sol, int32_t child, int32_t nchild) {
  SeqResult r;
  r.status = status;
  r.depth = (int32_t)depth;
  r.nodes = nodes;
  r.hash = hash;
  r.sol = sol;
  r.child = child;
  r.nchild = nchild;
  io.a.results[io.id] = r;
}

// ---- one-wave tier --------------------------------------------------------
//
// Components of at most kLds1MaxN nodes: one wave, 32-bit plane words, one
// node word per lane (lane l holds nodes 32l .. 32l+31), everything in LDS:
//   planes   64 node words x S dwords: word w of plane c (c < k) at w*S + c,
//            P at w*S + k, so a lane reads all of its word's planes with
//            S/4 ds_read_b128 (S = k+1 rounded up to 4, 8 or 16);
//   offs     per node: first neighbour (low 16 bits) | degree << 16;
//   ids      16-bit neighbour ids;
//   hdr      per depth: {offs of the level's column, est | untried << 16 |
//            c << 24} (est: the level's first log entry, which holds the
//            column's P bit, so the column itself is read back from the log;
//            untried: the column's rows not tried yet at this level);
//   ent      the undo log;
//   (stitch-aware order) each node's stitch partner and the color of each
//            covered node.
// The per-depth "untried rows" bit set is one 32-bit word per lane (depth d
// in lane d >> 5).  Per node the dependent chain is: the plane words (read
// at the end of the previous node, behind its cover atomics), the count and
// narrowing in each lane, a wave minimum, then the winner's row set and
// offs word (each lane reads the offs word of its own candidate before the
// minimum, so the winner's is already in a register), one read of the
// neighbour ids, and one atomic AND per neighbour (lane 0 clears the
// column's P bit in the same instruction).
__host__ __device__ constexpr uint32_t lds1_stride(int32_t k) {
  return k + 1 <= 4 ? 4u : (k + 1 <= 8 ? 8u : 16u);
}

struct Lds1Layout {
  uint32_t offs_off, ids_off, hdr_off, ent_off, part_off, col_off, total;
};

// stitch: also each node's stitch partner (16 bits, 0xffff none) and the
// color of each covered node (one byte).
__host__ __device__ inline Lds1Layout lds1_layout(int32_t n, int32_t k, int64_t adj_words,
                                                 bool stitch = false) {
  Lds1Layout L;
  const uint32_t m2 = (uint32_t)(adj_words - n - 1);
  L.offs_off = 64u * 4u * lds1_stride(k);
  L.ids_off = L.offs_off + 4u * (uint32_t)(n > 0 ? n : 1);   // one offs word at least
  L.hdr_off = (L.ids_off + 2u * m2 + 7u) & ~7u;
  L.ent_off = L.hdr_off + 8u * (uint32_t)n;
  L.part_off = L.ent_off + 4u * lds_log_entries(n, k, adj_words);
  L.col_off = L.part_off + (stitch ? 2u * (uint32_t)(n > 0 ? n : 1) : 0u);
  L.total = (L.col_off + (stitch ? (uint32_t)n : 0u) + 15u) & ~15u;
  return L;
}

template <int K>
struct Lds1Words {
  static constexpr int S = (int)lds1_stride(K);
  uint32_t a[S];
  __device__ __forceinline__ void load(const uint32_t* PL, uint32_t lane) {
    const uint4* q = reinterpret_cast<const uint4*>(PL + lane * (uint32_t)S);
#pragma unroll
    for (int j = 0; j < S / 4; ++j) {
      const uint4 x = q[j];
      a[4 * j] = x.x;
      a[4 * j + 1] = x.y;
      a[4 * j + 2] = x.z;
      a[4 * j + 3] = x.w;
    }
  }
};

// solve_lds itself is in lds_one_wave.inc, included below.

// ---- one-wave wide tier ---------------------------------------------------
//
// Big components whose planes and neighbour lists fit in LDS: one wave, as
// the one-wave tier, but up to kWideMaxWords 32-bit node words per lane
// (word w in lane w & 63), so no barrier per node, and the column choice
// reads a cache of per-word keys instead of recounting every word: key(w) =
// count << 28 | node << 8 | rows of the lowest-count, lowest-index
// uncovered column of word w (kNoKey when w has none).  A cover changes
// only the words of the column and of its neighbours, so after the cover
// atomics each lane that made one reads its word's planes back and
// rewrites that word's key; after a backtrack (the undo log touches any
// words) every key is recomputed.  Per node a lane reads its keys (at most
// eight, two ds_read_b128), takes their minimum, and the wave minimum is
// the column with its count and rows.  LDS: the planes, the keys, the
// per-depth "untried rows" bit set, offs (first neighbour | degree << 17),
// 16-bit neighbour ids, and for the stitch-aware order the partners and the
// color of each covered node.  Level headers {log start, v | untried << 16
// | c << 24} and the undo log go to the worker's global area: the forward
// path only stores to it (nothing waits for those stores), and a backtrack
// - rare on components this large - reads it back after a fence.
__host__ __device__ inline uint32_t wide_words(int32_t n) {
  const uint32_t w = (uint32_t)((n + 2047) / 2048);   // 64 lanes x 32 nodes
  return w < 1u ? 1u : w;
}

struct WideLayout {
  uint32_t pl_off, key_off, bits_off, offs_off, ids_off, part_off, col_off, total;
};

__host__ __device__ inline WideLayout wide_layout(int32_t n, int32_t k, int64_t adj_words,
                                                  bool stitch) {
  WideLayout L;
  const uint32_t m2 = (uint32_t)(adj_words - n - 1);
  const uint32_t n1 = (uint32_t)(n > 0 ? n : 1);   // one offs word at least
  L.pl_off = 16u;   // the workgroup's queue pop result first
  L.key_off = L.pl_off + 64u * wide_words(n) * 4u * lds1_stride(k);
  L.bits_off = L.key_off + 64u * 4u * (uint32_t)kWideMaxWords;
  L.offs_off = L.bits_off + ((4u * (((uint32_t)n + 31u) / 32u) + 15u) & ~15u);
  L.ids_off = L.offs_off + 4u * n1;
  L.part_off = (L.ids_off + 2u * m2 + 15u) & ~15u;
  L.col_off = L.part_off + (stitch ? 2u * n1 : 0u);
  L.total = (L.col_off + (stitch ? (uint32_t)n : 0u) + 15u) & ~15u;
  return L;
}

// Key of word w (planes in W): count << 28 | node << 8 | rows (count <= k <= 8,
// node < 2^20).
template <int K>
__device__ __forceinline__ uint32_t wide_key(const Lds1Words<K>& W, uint32_t w) {
  constexpr int NB = bits_for(K);
  uint32_t cnt[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) cnt[b] = 0u;
#pragma unroll
  for (int c = 0; c < K; ++c) {
    uint32_t carry = W.a[c];
#pragma unroll
    for (int b = 0; b < bits_for(c + 1); ++b) {
      const uint32_t t = cnt[b] & carry;
      cnt[b] ^= carry;
      carry = t;
    }
  }
  const uint32_t p = W.a[K];
  uint32_t cand = p, t = 0u;
#pragma unroll
  for (int b = NB - 1; b >= 0; --b) {
    const uint32_t x = cand & ~cnt[b];
    if (x) cand = x;
    else t |= 1u << b;
  }
  const uint32_t bit = (uint32_t)__builtin_ctz(cand | 0x80000000u);
  uint32_t r = 0;
#pragma unroll
  for (int c = 0; c < K; ++c) r |= __builtin_amdgcn_ubfe(W.a[c], bit, 1u) << c;
  return p ? (t << 28) | (((w << 5) | bit) << 8) | r : kNoKey;
}

#define LDS_SEQ 0
#include "lds_one_wave.inc"
#undef LDS_SEQ
#define LDS_SEQ 1
#include "lds_one_wave.inc"
#undef LDS_SEQ

// Big components: one workgroup of nw waves (nw = blockDim.x / 64).  Every
// wave scans its share of the plane words; the per-wave minima meet in LDS
// and each wave folds them, so all waves hold the same column choice.  The
// rest of the node (cover, backtrack, bookkeeping) is a few lanes of work
// and runs on wave 0 alone; a barrier ends the node, and wave 0 publishes
// the loop status (and the final depth) in LDS for the others.  Adjacency,
// level headers and the undo log are in global memory.
// root_row / task_budget: a subtree task, as for solve_lds.  STITCH: the
// stitch-aware row order, as for solve_lds (partners from the CSR block,
// the color of each covered node in LDS).  Level headers hold the rows
// not tried yet.
template <bool TRACE, int K, bool STITCH>
__device__ void solve_lds_wg(const DevDesc& d, const uint32_t* __restrict__ adj, char* lds,
                             uint64_t* gstack, int8_t* __restrict__ colors,
                             DevRecord* __restrict__ rec, int32_t root_row = -1,
                             uint64_t task_budget = 0) {
  const uint32_t tid = threadIdx.x, lane = __lane_id(), nthr = blockDim.x;
  const uint32_t wid = uni(tid >> 6), nw = nthr >> 6;
  const uint32_t n = (uint32_t)d.n;
  const uint32_t adj_words = uni(adj[n]) + n + 1u;
  const LdsLayout L = lds_layout((int32_t)n, K, adj_words, true, STITCH);
  const uint32_t W = L.W;
  uint64_t* PL = reinterpret_cast<uint64_t*>(lds + L.pl_off);
  uint64_t* A = reinterpret_cast<uint64_t*>(lds + L.a_off);
  uint8_t* scol = reinterpret_cast<uint8_t*>(lds + L.col_off);
  const uint32_t* gpart = adj + adj_words + 1u;   // STITCH: partner of each node
  uint32_t* red = reinterpret_cast<uint32_t*>(lds + L.ctl_off);   // per-wave minima
  int32_t* ctl = reinterpret_cast<int32_t*>(lds + L.ctl_off + 64);  // status, depth
  uint64_t* hdr = gstack;
  uint32_t* ent = reinterpret_cast<uint32_t*>(gstack + n);
  const uint32_t* ids = adj + n + 1;
  for (uint32_t w = tid; w < W; w += nthr) {
    const uint32_t cnt = n - w * 64u >= 64u ? 64u : n - w * 64u;
    const uint64_t val = cnt == 64u ? ~0ull : ((1ull << cnt) - 1ull);
#pragma unroll
    for (int c = 0; c <= K; ++c) PL[(uint32_t)c * W + w] = val;
    A[w] = 0ull;
  }
  if (tid == 0) ctl[0] = -1;   // budget >= 1: the root always counts
  __syncthreads();

  // search state, kept by wave 0
  uint32_t depth = 0, row_in = kNoneL, esp = 0;
  uint64_t nodes = 1, h = 0;
  int32_t status = -1;
  const uint64_t budget = root_row >= 0 ? task_budget : (uint64_t)d.budget;
  if (root_row >= 0) {
    // wave 0 takes row (0, root_row) at depth 0 (A's bit for level 0 stays
    // clear); `nodes` = 1 then counts the first node below it
    if (wid == 0u) {
      const uint32_t c = (uint32_t)root_row;
      const uint32_t beg = uni(adj[0]), deg = uni(adj[1]) - beg;
      if (lane == 63u) {
        ent[0] = (uint32_t)K << kEntryNodeBits;
        atomicAnd(reinterpret_cast<unsigned long long*>(&PL[(uint32_t)K * W]), ~1ull);
        hdr[0] = make_hdr(0u, c, 0u, 0u);   // no other row at this level
        if (STITCH) scol[0] = (uint8_t)c;
      }
      esp = 1u;
      unsigned long long* plane = reinterpret_cast<unsigned long long*>(PL + c * W);
      for (uint32_t ch = 0; ch < deg; ch += 64u) {
        bool hit = false;
        uint32_t u = 0;
        if (ch + lane < deg) {
          u = ids[beg + ch + lane];
          const uint64_t bit = 1ull << (u & 63u);
          hit = (atomicAnd(&plane[u >> 6], ~bit) & bit) != 0ull;
        }
        const uint64_t bal = __ballot(hit);
        if (hit) {
          const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
          ent[esp + rank] = (c << kEntryNodeBits) | u;
        }
        esp += (uint32_t)__popcll(bal);
      }
      depth = 1u;
      row_in = c;
    }
    __syncthreads();
  }

  while (ctl[0] < 0) {
    uint32_t key = kNoKey;
    for (uint32_t w = tid; w < W; w += nthr) key = min(key, word_key<K>(PL, W, w));
    key = wave_min(key);
    if (nw > 1u) {
      if (lane == 63u) red[wid] = key;
      __syncthreads();
      key = wave_min(lane < nw ? red[lane] : kNoKey);
    }
    if (wid == 0u) {
      if (key == kNoKey) {   // no uncovered column: the levels hold a solution
        if (TRACE) h = trace_node(h, depth, row_in, kNoneL, 0);
        status = MPLD_FEASIBLE;
      } else {
        uint32_t v = key & 0xffffffu;
        const uint32_t size = key >> 24;
        if (TRACE) h = trace_node(h, depth, row_in, v, size);
        uint32_t c = 0, rows = 0, est = 0, beg = 0, deg = 0;
        if (size != 0) {
          const uint32_t b0 = adj[v], b1 = adj[v + 1];
          uint32_t r = 0;
#pragma unroll
          for (int j = 0; j < K; ++j) r |= (uint32_t)((PL[(uint32_t)j * W + (v >> 6)] >> (v & 63u)) & 1ull) << j;
          beg = uni(b0);
          deg = uni(b1) - beg;
          rows = uni(r);
          c = (uint32_t)__builtin_ctz(rows);
          if (STITCH) {
            // the partner's color first when the partner is covered and
            // that row of v is open
            const uint32_t p = uni(gpart[v]);
            if (p < n && !((uni64(PL[(uint32_t)K * W + (p >> 6)]) >> (p & 63u)) & 1ull)) {
              const uint32_t cp = uni((uint32_t)scol[p]);
              if ((rows >> cp) & 1u) c = cp;
            }
          }
          rows &= ~(1u << c);   // the level's untried rows
          est = esp;
          if (lane == 63u) {
            ent[est] = ((uint32_t)K << kEntryNodeBits) | v;
            atomicAnd(reinterpret_cast<unsigned long long*>(&PL[(uint32_t)K * W + (v >> 6)]),
                      ~(1ull << (v & 63u)));
          }
          esp = est + 1u;
        } else {
          // dead end: back to the deepest level whose column has an untried row
          uint32_t f = kNoneL;
          if (depth != 0) {
            const uint32_t d1 = depth - 1u;
            uint32_t aw = d1 >> 6;
            uint64_t bits = uni64(A[aw]) & (~0ull >> (63u - (d1 & 63u)));
            while (bits == 0ull && aw != 0u) bits = uni64(A[--aw]);
            if (bits) f = aw * 64u + 63u - (uint32_t)__builtin_clzll(bits);
          }
          if (f == kNoneL) {
            status = MPLD_INFEASIBLE;
          } else {
            const uint64_t hd = uni64(hdr[f]);
            v = (uint32_t)hd & 0xffffffu;
            rows = (uint32_t)(hd >> 28) & 0xffu;   // untried rows, next in ascending order
            est = (uint32_t)(hd >> 36);
            beg = uni(adj[v]);
            deg = uni(adj[v + 1]) - beg;
            // uncover every level above f, and the rows level f removed
            for (uint32_t i = est + 1u + lane; i < esp; i += 64) {
              const uint32_t e = ent[i];
              const uint32_t u = e & ((1u << kEntryNodeBits) - 1u);
              atomicOr(reinterpret_cast<unsigned long long*>(&PL[(e >> kEntryNodeBits) * W + (u >> 6)]),
                       1ull << (u & 63u));
            }
            c = (uint32_t)__builtin_ctz(rows);
            rows &= rows - 1u;
            depth = f;
            esp = est + 1u;
          }
        }
        if (status < 0) {
          // include row (v, c) at this depth
          if (lane == 63u) {
            hdr[depth] = make_hdr(v, c, rows, est);
            if (STITCH) scol[v] = (uint8_t)c;
            const uint64_t bit = 1ull << (depth & 63u);
            if (rows != 0u) atomicOr(reinterpret_cast<unsigned long long*>(&A[depth >> 6]), bit);
            else atomicAnd(reinterpret_cast<unsigned long long*>(&A[depth >> 6]), ~bit);
          }
          unsigned long long* plane = reinterpret_cast<unsigned long long*>(PL + c * W);
          for (uint32_t ch = 0; ch < deg; ch += 64u) {
            bool hit = false;
            uint32_t u = 0;
            if (ch + lane < deg) {
              u = ids[beg + ch + lane];
              const uint64_t bit = 1ull << (u & 63u);
              hit = (atomicAnd(&plane[u >> 6], ~bit) & bit) != 0ull;
            }
            const uint64_t bal = __ballot(hit);
            if (hit) {
              const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
              ent[esp + rank] = (c << kEntryNodeBits) | u;
            }
            esp += (uint32_t)__popcll(bal);
          }
          ++depth;
          row_in = v * (uint32_t)K + c;
          // the next node, if the budget allows it
          if (nodes == budget) status = MPLD_BUDGET_EXHAUSTED;
          else ++nodes;
        }
      }
      if (lane == 63u) {
        ctl[0] = status;
        ctl[1] = (int32_t)depth;
      }
    }
    __syncthreads();
  }
  const int32_t fin = ctl[0];
  const uint32_t fdepth = (uint32_t)ctl[1];
  if (fin == MPLD_FEASIBLE) {
    for (uint32_t f = tid; f < fdepth; f += nthr) {
      const uint64_t hd = hdr[f];
      colors[(uint32_t)hd & 0xffffffu] = (int8_t)((hd >> 24) & 0xfu);
    }
  } else {
    for (uint32_t v = tid; v < n; v += nthr) colors[v] = -1;
  }
  if (wid == 0u) {   // uniform record from every lane of wave 0
    rec->status = status;
    rec->depth = status == MPLD_INFEASIBLE ? 0 : (int32_t)depth;
    rec->nodes = nodes;
    rec->hash = h;
  }
  __syncthreads();
}

template <bool TRACE, bool BIG, bool STITCH>
__device__ __forceinline__ void solve_lds_k(const DevDesc& d, const uint32_t* gadj, char* lds,
                                            uint64_t* gstack, int8_t* colors, DevRecord* rec,
                                            uint32_t wide, int32_t root_row = -1,
                                            uint64_t task_budget = 0) {
#define MPLD_LDS_CASE(KK)                                                                     \
  case KK:                                                                                    \
    if (BIG && KK <= kWideMaxK && wide) solve_lds_wide<TRACE, (KK <= kWideMaxK ? KK : 2), STITCH>(d, gadj, lds, gstack, colors, rec, root_row, task_budget); \
    else if (BIG) solve_lds_wg<TRACE, KK, STITCH>(d, gadj, lds, gstack, colors, rec, root_row, task_budget); \
    else solve_lds<TRACE, KK, STITCH>(d, gadj, lds, colors, rec, root_row, task_budget);     \
    break;
  switch (d.k) {
    MPLD_LDS_CASE(2)
    MPLD_LDS_CASE(3)
    MPLD_LDS_CASE(4)
    MPLD_LDS_CASE(5)
    MPLD_LDS_CASE(6)
    MPLD_LDS_CASE(7)
    default:
      if (BIG && wide) solve_lds_wide<TRACE, 8, STITCH>(d, gadj, lds, gstack, colors, rec, root_row, task_budget);
      else if (BIG) solve_lds_wg<TRACE, 8, STITCH>(d, gadj, lds, gstack, colors, rec, root_row, task_budget);
      else solve_lds<TRACE, 8, STITCH>(d, gadj, lds, colors, rec, root_row, task_budget);
      break;
  }
#undef MPLD_LDS_CASE
}

// Persistent kernel, one workgroup per component (one wave for small
// components, nw waves for big ones); work distribution as in the register
// tier: static first item, then atomic pops by one thread, the last pop
// resets the counter.
template <bool TRACE, bool BIG, bool STITCH>
__global__ __launch_bounds__(BIG ? 1024 : 64) void lds_batched_kernel(
    const DevDesc* __restrict__ descs, const uint32_t* __restrict__ adj32, int32_t qlen,
    int32_t* __restrict__ counter, uint64_t* gstack, uint64_t stack_words_per_wave,
    DevRecord* __restrict__ recs, int8_t* __restrict__ colors, uint32_t wide) {
  extern __shared__ __align__(16) char lds[];
  uint64_t* my_stack = BIG ? gstack + (uint64_t)blockIdx.x * stack_words_per_wave : nullptr;
  const int32_t gw = (int32_t)gridDim.x;
  int32_t item = (int32_t)uni(blockIdx.x);
  while (item < qlen) {
    const DevDesc d = descs[item];
    solve_lds_k<TRACE, BIG, STITCH>(d, adj32 + d.nbr_off, lds, my_stack, colors + d.out_off, recs + d.comp,
                                    wide);
    if (gw >= qlen) break;
    int32_t r = 0;
    if constexpr (BIG) {   // one pop per workgroup, shared through LDS
      int32_t* popped = reinterpret_cast<int32_t*>(lds);
      if (threadIdx.x == 0) *popped = atomicAdd(counter, 1);
      __syncthreads();
      r = (int32_t)uni((uint32_t)*popped);
      __syncthreads();
    } else {
      if (__lane_id() == 0) r = atomicAdd(counter, 1);
      r = (int32_t)uni((uint32_t)r);
    }
    item = gw + r;
    if (r == qlen - 1 && threadIdx.x == 0) atomicExch(counter, 0);
  }
}

template <bool TRACE, bool BIG, bool STITCH>
__global__ __launch_bounds__(BIG ? 1024 : 64) void lds_single_kernel(
    const DevDesc* __restrict__ descs, const uint32_t* __restrict__ adj32, int32_t item,
    uint64_t* gstack, DevRecord* __restrict__ recs, int8_t* __restrict__ colors, uint32_t wide) {
  extern __shared__ __align__(16) char lds[];
  const DevDesc d = descs[item];
  solve_lds_k<TRACE, BIG, STITCH>(d, adj32 + d.nbr_off, lds, gstack, colors + d.out_off, recs + d.comp,
                                  wide);
}

// Subtree tasks of the heavy-component split: task t searches the subtree
// of root row tasks[t].row of component tasks[t].item with its own budget,
// and writes its record (with TRACE, the trace hash of its own nodes) to
// task_recs[t] and its colors to task_colors + tasks[t].col_off.  Grid-stride over the tasks, one
// workgroup each (one wave small, nw waves big; big ones use the block's
// stack area).
template <bool TRACE, bool BIG, bool STITCH>
__global__ __launch_bounds__(BIG ? 1024 : 64) void lds_task_kernel(
    const DevDesc* __restrict__ descs, const uint32_t* __restrict__ adj32,
    const LdsTask* __restrict__ tasks, int32_t ntasks, uint64_t* gstack,
    uint64_t stack_words_per_block, DevRecord* __restrict__ task_recs,
    int8_t* __restrict__ task_colors, uint32_t wide) {
  extern __shared__ __align__(16) char lds[];
  uint64_t* my_stack = BIG ? gstack + (uint64_t)blockIdx.x * stack_words_per_block : nullptr;
  for (int32_t t = (int32_t)uni(blockIdx.x); t < ntasks; t += (int32_t)gridDim.x) {
    const LdsTask task = tasks[t];
    const DevDesc d = descs[task.item];
    solve_lds_k<TRACE, BIG, STITCH>(d, adj32 + d.nbr_off, lds, my_stack, task_colors + task.col_off,
                                    task_recs + t, wide, task.row, (uint64_t)task.budget);
  }
}

// Sequence-engine tasks of the CSR tiers: one wave per workgroup over a
// round's run list, or, FINISH, over the tiers' components: a component cut by
// its budget searches its last task once more with what was left, then record
// and colors are written.  A component keeps the layout that it was given.
template <bool TRACE, int K, bool FINISH>
__global__ __launch_bounds__(64) void seq_csr_kernel(const SeqArgs a, const DevDesc* __restrict__ descs,
                                                     const uint32_t* __restrict__ adj32, uint64_t* stack,
                                                     uint64_t stack_words, int32_t parity,
                                                     DevRecord* __restrict__ recs, int8_t* __restrict__ colors) {
  extern __shared__ __align__(16) char lds[];
  uint64_t* my_stack = stack + (uint64_t)blockIdx.x * stack_words;
  const auto run = [&](SeqIo& io, const DevDesc& d, bool wide) {
    const uint32_t* g = adj32 + d.nbr_off;
    if constexpr (K <= kWideMaxK) {
      if (wide) {
        solve_lds_wide_seq<TRACE, K, false>(d, g, lds, my_stack, &io);
        return;
      }
    }
    solve_lds_seq<TRACE, K, false>(d, g, lds, &io);
  };
  if constexpr (!FINISH) {
    const int32_t* list = a.runs + (int64_t)(parity * kSeqTiers + kSeqCsr) * a.run_cap;
    const int32_t count = min((int32_t)uni((uint32_t)a.head->run[parity][kSeqCsr]), a.run_cap);
    int32_t loaded = -1;
    for (int32_t r = (int32_t)uni(blockIdx.x); r < count;) {
      SeqIo io;
      io.a = a;
      const uint32_t entry = uni((uint32_t)list[r]);
      io.id = (int32_t)(entry & (uint32_t)kSeqTaskMask);
      io.task = a.tasks[io.id];
      const int32_t pos = (int32_t)uni((uint32_t)a.comps[io.task.comp].pos);
      const bool wide = uni((uint32_t)a.comps[io.task.comp].wide) != 0;
      const DevDesc d = descs[pos];
      io.limit = (uint64_t)d.budget;
      // a root first goes all the way down
      const uint64_t cap = (uint64_t)a.cap[kSeqCsr] + (io.task.kind == kSeqRoot ? (uint64_t)d.n : 0ull);
      io.stop = cap < io.limit ? cap : io.limit;
      io.load = io.task.comp != loaded;
      io.cuts = (entry & (uint32_t)kSeqCut) != 0;
      io.force = (entry & (uint32_t)kSeqForce) != 0;
      loaded = io.task.comp;
      run(io, d, wide);
      if ((int32_t)gridDim.x >= count) break;
      int32_t q = 0;
      if (__lane_id() == 0) q = atomicAdd(&a.head->pop[parity][kSeqCsr], 1);
      r = (int32_t)gridDim.x + (int32_t)uni((uint32_t)q);
    }
  } else {
    for (int32_t ci = (int32_t)uni(blockIdx.x); ci < a.ncomps; ci += (int32_t)gridDim.x) {
      const SeqComp c = a.comps[ci];
      if (c.tier != kSeqCsr || c.status == kSeqLost) continue;
      const DevDesc d = descs[c.pos];
      int32_t depth = c.status == MPLD_FEASIBLE ? d.n : (c.status == MPLD_INFEASIBLE ? 0 : c.depth);
      uint64_t hash = c.hash;
      if (c.cross >= 0) {
        SeqIo io;
        io.a = a;
        io.id = c.cross;
        io.task = a.tasks[c.cross];
        io.stop = io.limit = c.left;
        io.load = true;
        io.cuts = io.force = false;   // (it stops at `limit`)
        run(io, d, uni((uint32_t)c.wide) != 0);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        const SeqResult r = a.results[c.cross];
        depth = r.depth;
        if (TRACE) hash = trace_concat(hash, r.hash, c.left);
      }
      int8_t* out = colors + d.out_off;
      const int8_t* sol = reinterpret_cast<const int8_t*>(a.arena + (c.status == MPLD_FEASIBLE ? c.sol : 0));
      for (int32_t v = (int32_t)__lane_id(); v < d.n; v += 64)
        out[v] = c.status == MPLD_FEASIBLE ? sol[v] : (int8_t)-1;
      DevRecord* rec = recs + d.comp;
      rec->status = c.status;
      rec->depth = depth;
      rec->nodes = c.acc;
      rec->hash = TRACE ? hash : 0;
    }
  }
}

// Conflict marking (Algorithm 1: a column left with no related row is a
// conflict candidate (cl, cl'), cl' the column whose cover removed cl's
// final row) for a component whose search ended without a solution: one
// descent of the search that never backtracks.  Same column rule and plane
// scan as the search; the column takes its lowest open color, or, with no
// row left, the color it lost last (last[u] in LDS, written by the lane
// whose atomic AND removed u's row).  One wave; adjacency from global
// memory; LDS holds the planes and last[].  Every node is colored.
template <int K>
__device__ void mark_csr(const DevDesc& d, const uint32_t* __restrict__ adj, char* lds,
                         int8_t* __restrict__ colors) {
  const uint32_t lane = __lane_id();
  const uint32_t n = (uint32_t)d.n, W = (n + 63u) / 64u;
  uint64_t* PL = reinterpret_cast<uint64_t*>(lds);
  uint8_t* last = reinterpret_cast<uint8_t*>(PL + (uint32_t)(K + 1) * W);
  const uint32_t* ids = adj + n + 1;
  for (uint32_t w = lane; w < W; w += 64) {
    const uint32_t cnt = n - w * 64u >= 64u ? 64u : n - w * 64u;
    const uint64_t val = cnt == 64u ? ~0ull : ((1ull << cnt) - 1ull);
#pragma unroll
    for (int c = 0; c <= K; ++c) PL[(uint32_t)c * W + w] = val;
  }
  __syncthreads();
  for (;;) {
    uint32_t key = kNoKey;
    for (uint32_t w = lane; w < W; w += 64) key = min(key, word_key<K>(PL, W, w));
    key = wave_min(key);
    if (key == kNoKey) break;
    const uint32_t v = key & 0xffffffu;
    uint32_t c;
    if ((key >> 24) != 0u) {
      uint32_t r = 0;
#pragma unroll
      for (int j = 0; j < K; ++j) r |= (uint32_t)((PL[(uint32_t)j * W + (v >> 6)] >> (v & 63u)) & 1ull) << j;
      c = (uint32_t)__builtin_ctz(uni(r));
    } else {
      c = uni(last[v]);
    }
    if (lane == 63u) {
      colors[v] = (int8_t)c;
      atomicAnd(reinterpret_cast<unsigned long long*>(&PL[(uint32_t)K * W + (v >> 6)]),
                ~(1ull << (v & 63u)));
    }
    const uint32_t beg = uni(adj[v]), deg = uni(adj[v + 1]) - beg;
    unsigned long long* plane = reinterpret_cast<unsigned long long*>(PL + c * W);
    for (uint32_t j = lane; j < deg; j += 64u) {
      const uint32_t u = ids[beg + j];
      const uint64_t bit = 1ull << (u & 63u);
      if (atomicAnd(&plane[u >> 6], ~bit) & bit) last[u] = (uint8_t)c;
    }
    __syncthreads();
  }
  __syncthreads();
}

// One wave per workgroup over the components of the LDS, big and
// device-wide tiers; components whose record is FEASIBLE keep the search's
// colors.
__global__ __launch_bounds__(64) void mark_lds_kernel(const DevDesc* __restrict__ descs,
                                                      const uint32_t* __restrict__ adj32,
                                                      int32_t qlen,
                                                      const DevRecord* __restrict__ recs,
                                                      int8_t* __restrict__ colors) {
  extern __shared__ __align__(16) char lds[];
  for (int32_t i = (int32_t)uni(blockIdx.x); i < qlen; i += (int32_t)gridDim.x) {
    const DevDesc d = descs[i];
    if ((int32_t)uni((uint32_t)recs[d.comp].status) == MPLD_FEASIBLE) continue;
    const uint32_t* adj = adj32 + d.nbr_off;
    int8_t* out = colors + d.out_off;
    switch (d.k) {
      case 2: mark_csr<2>(d, adj, lds, out); break;
      case 3: mark_csr<3>(d, adj, lds, out); break;
      case 4: mark_csr<4>(d, adj, lds, out); break;
      case 5: mark_csr<5>(d, adj, lds, out); break;
      case 6: mark_csr<6>(d, adj, lds, out); break;
      case 7: mark_csr<7>(d, adj, lds, out); break;
      default: mark_csr<8>(d, adj, lds, out); break;
    }
  }
}

// ---- host side --------------------------------------------------------------

int64_t lds_bytes_for(int32_t n, int32_t k, int64_t adj_words, int32_t max_deg, bool big,
                      bool stitch) {
  // adj_words: row offsets + neighbour ids (n + 1 + 2m)
  (void)max_deg;
  return big ? (int64_t)lds_layout(n, k, adj_words, true, stitch).total
             : (int64_t)lds1_layout(n, k, adj_words, stitch).total;
}

int64_t lds_wide_bytes(int32_t n, int32_t k, int64_t adj_words, int32_t max_deg, bool stitch) {
  // -1: the one-wave wide layout does not apply (too many nodes, or ids or
  // degrees beyond its offs fields)
  const int64_t m2 = adj_words - n - 1;
  if (k > kWideMaxK || n > kWideMaxN || m2 >= (int64_t)1 << kWideBegBits ||
      (int64_t)max_deg >= (int64_t)1 << (32 - kWideBegBits))
    return -1;
  return (int64_t)wide_layout(n, k, adj_words, stitch).total;
}

int64_t lds_stack_words(int32_t n, int32_t k, int64_t adj_words) {
  // level headers (one u64 per depth) and the undo log (u32 entries)
  return (int64_t)n + ((int64_t)lds_log_entries(n, k, adj_words) + 1) / 2;
}
template <bool TRACE, bool BIG, bool STITCH>
static void lds_attr(int bytes) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&lds_batched_kernel<TRACE, BIG, STITCH>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&lds_single_kernel<TRACE, BIG, STITCH>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&lds_task_kernel<TRACE, BIG, STITCH>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

int64_t mark_lds_bytes(int32_t n, int32_t k) {
  // planes (k + 1 words of 64 nodes each) and one byte per node
  const int64_t W = ((int64_t)n + 63) / 64;
  return (8 * (int64_t)(k + 1) * W + (int64_t)n + 7) & ~(int64_t)7;
}

hipError_t launch_mark_lds(int grid, int lds_bytes, const DevDesc* descs, const uint32_t* adj32,
                           int32_t qlen, const DevRecord* recs, int8_t* colors, hipStream_t s) {
  if (qlen <= 0) return hipSuccess;
  hipLaunchKernelGGL(mark_lds_kernel, dim3(grid), dim3(64), (size_t)lds_bytes, s, descs, adj32,
                     qlen, recs, colors);
  return hipGetLastError();
}

// Calls f(trace, K, finish) with each as a std::integral_constant.
template <typename F>
static hipError_t seq_dispatch(bool trace, int k, bool finish, F&& f) {
  const auto with_k = [&](auto t, auto fin) {
    switch (k) {
      case 2: f(t, std::integral_constant<int, 2>(), fin); break;
      case 3: f(t, std::integral_constant<int, 3>(), fin); break;
      case 4: f(t, std::integral_constant<int, 4>(), fin); break;
      case 5: f(t, std::integral_constant<int, 5>(), fin); break;
      case 6: f(t, std::integral_constant<int, 6>(), fin); break;
      case 7: f(t, std::integral_constant<int, 7>(), fin); break;
      default: f(t, std::integral_constant<int, 8>(), fin); break;
    }
  };
  const auto with_f = [&](auto t) {
    if (finish) with_k(t, std::true_type{});
    else with_k(t, std::false_type{});
  };
  if (trace) with_f(std::true_type{});
  else with_f(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_seq_csr(bool trace, int k, int grid, int lds_bytes, const SeqArgs& a, const DevDesc* descs,
                          const uint32_t* adj32, uint64_t* stack, uint64_t stack_words, int32_t parity,
                          bool finish, DevRecord* recs, int8_t* colors, hipStream_t s) {
  if (grid < 1) return hipErrorInvalidValue;
  return seq_dispatch(trace, k, finish, [&](auto t, auto kk, auto fin) {
    hipLaunchKernelGGL((seq_csr_kernel<decltype(t)::value, decltype(kk)::value, decltype(fin)::value>),
                       dim3(grid), dim3(64), (size_t)lds_bytes, s, a, descs, adj32, stack, stack_words, parity,
                       recs, colors);
  });
}

static void seq_attr(int bytes) {
  for (int k = 2; k <= 8; ++k)
    for (int m = 0; m < 4; ++m)
      (void)seq_dispatch(m & 1, k, m & 2, [&](auto t, auto kk, auto fin) {
        (void)hipFuncSetAttribute(
            reinterpret_cast<const void*>(
                &seq_csr_kernel<decltype(t)::value, decltype(kk)::value, decltype(fin)::value>),
            hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
      });
}

void lds_configure(int bytes) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&mark_lds_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  lds_attr<true, true, false>(bytes);
  lds_attr<true, false, false>(bytes);
  lds_attr<false, true, false>(bytes);
  lds_attr<false, false, false>(bytes);
  lds_attr<true, true, true>(bytes);
  lds_attr<true, false, true>(bytes);
  lds_attr<false, true, true>(bytes);
  lds_attr<false, false, true>(bytes);
  seq_attr(bytes);
  (void)hipGetLastError();
}

int lds_big_waves(int32_t max_n) {
  // one plane word per lane of the workgroup, at most 16 waves
  const int32_t words = (max_n + 63) / 64;
  const int32_t w = (words + 63) / 64;
  return w < 1 ? 1 : (w > 16 ? 16 : w);
}

// Calls f(trace, big, stitch) with each flag as a std::integral_constant,
// so that the launch names the matching kernel instantiation.
template <typename F>
static hipError_t lds_dispatch(bool trace, bool big, bool stitch, F&& f) {
  auto with_stitch = [&](auto t, auto g) {
    if (stitch) f(t, g, std::true_type{});
    else f(t, g, std::false_type{});
  };
  auto with_big = [&](auto t) {
    if (big) with_stitch(t, std::true_type{});
    else with_stitch(t, std::false_type{});
  };
  if (trace) with_big(std::true_type{});
  else with_big(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_lds_batched(bool trace, bool big, bool stitch, int waves, int grid,
                              int lds_bytes, const DevDesc* descs, const uint32_t* adj32,
                              int32_t qlen, int32_t* counter, uint64_t* gstack,
                              uint64_t stack_words, DevRecord* recs, int8_t* colors,
                              hipStream_t s) {
  if (qlen <= 0) return hipSuccess;
  if (waves < 0 || waves > 16 || (!big && waves != 1)) return hipErrorInvalidValue;
  const uint32_t wide = waves == 0 ? 1u : 0u;   // big tier, one wave, wide layout
  return lds_dispatch(trace, big, stitch, [&](auto t, auto g, auto st) {
    hipLaunchKernelGGL((lds_batched_kernel<decltype(t)::value, decltype(g)::value, decltype(st)::value>),
                       dim3(grid), dim3(64 * (wide ? 1 : waves)), (size_t)lds_bytes, s, descs, adj32,
                       qlen, counter, gstack, stack_words, recs, colors, wide);
  });
}

hipError_t launch_lds_tasks(bool trace, bool big, bool stitch, int waves, int grid, int lds_bytes,
                            const DevDesc* descs, const uint32_t* adj32, const LdsTask* tasks,
                            int32_t ntasks, uint64_t* gstack, uint64_t stack_words,
                            DevRecord* task_recs, int8_t* task_colors, hipStream_t s) {
  if (ntasks <= 0) return hipSuccess;
  if (waves < 0 || waves > 16 || (!big && waves != 1) || grid < 1) return hipErrorInvalidValue;
  const uint32_t wide = waves == 0 ? 1u : 0u;   // big tier, one wave, wide layout
  return lds_dispatch(trace, big, stitch, [&](auto t, auto g, auto st) {
    hipLaunchKernelGGL((lds_task_kernel<decltype(t)::value, decltype(g)::value, decltype(st)::value>),
                       dim3(grid), dim3(64 * (wide ? 1 : waves)), (size_t)lds_bytes, s, descs, adj32,
                       tasks, ntasks, gstack, stack_words, task_recs, task_colors, wide);
  });
}

// One workgroup per resolved component: its colors and record.
__global__ __launch_bounds__(256) void csr_writeback_kernel(const LdsResolved* __restrict__ w,
                                                            int32_t count, const int8_t* __restrict__ src,
                                                            DevRecord* __restrict__ recs,
                                                            int8_t* __restrict__ colors) {
  for (int32_t i = (int32_t)blockIdx.x; i < count; i += (int32_t)gridDim.x) {
    const LdsResolved r = w[i];
    for (int32_t v = (int32_t)threadIdx.x; v < r.n; v += (int32_t)blockDim.x)
      colors[r.out_off + v] = r.src_off >= 0 ? src[r.src_off + v] : (int8_t)-1;
    if (threadIdx.x == 0) recs[r.comp] = r.rec;
  }
}

hipError_t launch_csr_writeback(const LdsResolved* w, int32_t count, const int8_t* src,
                                DevRecord* recs, int8_t* colors, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(csr_writeback_kernel, dim3(count < 1024 ? count : 1024), dim3(256), 0, s, w,
                     count, src, recs, colors);
  return hipGetLastError();
}

hipError_t launch_lds_single(bool trace, bool big, bool stitch, int waves, int lds_bytes,
                             const DevDesc* descs, const uint32_t* adj32, int32_t item,
                             uint64_t* gstack, DevRecord* recs, int8_t* colors, hipStream_t s) {
  if (waves < 0 || waves > 16 || (!big && waves != 1)) return hipErrorInvalidValue;
  const uint32_t wide = waves == 0 ? 1u : 0u;   // big tier, one wave, wide layout
  return lds_dispatch(trace, big, stitch, [&](auto t, auto g, auto st) {
    hipLaunchKernelGGL((lds_single_kernel<decltype(t)::value, decltype(g)::value, decltype(st)::value>),
                       dim3(1), dim3(64 * (wide ? 1 : waves)), (size_t)lds_bytes, s, descs, adj32,
                       item, gstack, recs, colors, wide);
  });
}

}  // namespace mpld
