// graph_builder.h - the device front-end's workspace and the pieces that its
// two files share: scans, the simplification and split of a CSR graph
// (graph_device.hip) and the whole-layout flow (flow_device.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <condition_variable>
#include <memory>
#include <mutex>
#include <vector>

#include "internal.h"
#include "runtime.h"

namespace mpld {

// Page-locked copies of one layout's rectangles and graph.
struct Staging {
  PinnedBuf in, out;
};

struct GraphBuilder {
  mpld_context* ctx = nullptr;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  std::mutex mu;
  DevBuf rects, box, partner, se, cell_of, cnt, start, sbox, sid, kept, deg, ptr, adj;
  DevBuf tiles;            // scans: the ticket, then a word per tile
  uint32_t epoch = 0, tickets = 0;   // launches so far, tickets they took
  DevBuf split_ws;   // split outputs then scratch (int32)
  DevBuf flow_ws;    // scratch of the whole-layout flow
  PinnedBuf hin, hout;
  // Layouts are copied in before and out after the builder's lock, from
  // staging of their own, so that the device works for one caller while the
  // others copy: kStagings layouts at most are on the way (four took the same
  // 5.2 ms for a burst of 48 layouts, and twice the pinned memory).
  static constexpr int kStagings = 2;
  std::mutex smu;
  std::condition_variable scv;
  std::vector<std::unique_ptr<Staging>> spare;
  int stagings = 0;   // made so far
  ~GraphBuilder() {
    if (own_stream && stream) (void)hipStreamDestroy(stream);
  }
};

// A staging taken from a builder, given back at the end of the scope.
class StagingUse {
 public:
  explicit StagingUse(GraphBuilder& gb) : gb_(gb) {
    std::unique_lock<std::mutex> lk(gb.smu);
    gb.scv.wait(lk, [&] { return !gb.spare.empty() || gb.stagings < GraphBuilder::kStagings; });
    if (gb.spare.empty()) {
      gb.spare.emplace_back(new Staging());
      ++gb.stagings;
    }
    st_ = std::move(gb.spare.back());
    gb.spare.pop_back();
  }
  ~StagingUse() {
    {
      std::lock_guard<std::mutex> lk(gb_.smu);
      gb_.spare.push_back(std::move(st_));
    }
    gb_.scv.notify_one();
  }
  StagingUse(const StagingUse&) = delete;
  StagingUse& operator=(const StagingUse&) = delete;
  Staging& operator*() { return *st_; }

 private:
  GraphBuilder& gb_;
  std::unique_ptr<Staging> st_;
};

// Buffers grow geometrically: a reallocation (and, for pinned host memory,
// hipHostMalloc) costs milliseconds, so it should happen rarely.
inline void grow(DevBuf& b, mpld_context* ctx, size_t bytes) {
  if (b.bytes < bytes) b.alloc(ctx, std::max(bytes + bytes / 4, 2 * b.bytes));
}
inline bool grow_pinned(PinnedBuf& b, size_t bytes) {
  return bytes <= b.bytes || b.reserve(std::max(bytes + bytes / 4, 2 * b.bytes));
}

// The tiles' words for scans and splits of up to n entries.
void scan_reserve(GraphBuilder& gb, int64_t n);
// Exclusive scan of in[0 .. n) into out[0 .. n], out[n] = the total.
void scan(GraphBuilder& gb, const int32_t* in, int64_t n, int32_t* out);

// Past one of these the device leaves a split to the host.
struct SplitLimits {
  int32_t peel, mid, giant;   // levels of the peeling's tail and of the numbering: of the components that
                              // a workgroup takes, and of those that several number together
  int32_t degree;             // a node's neighbours
  int32_t spin;               // looks at a word before a wait among workgroups is given up
};

struct SplitArgs {
  int32_t n, k, simplify;
  const int32_t* ptr;   // n + 1 CSR offsets
  const int32_t* adj;   // ascending neighbour lists
  // outputs (one contiguous region)
  int32_t* counts;      // [0] removed, [1] components
  int32_t* queue;       // n: removal order
  int32_t* comp_of;     // n: component, -1 if removed
  int32_t* order;       // n: core nodes by component, local order
  int32_t* comp_ptr;    // n + 1
  int32_t* local;       // n: local index, -1 if removed
  // scratch: n + 1 each (mids, bigs, giants: components of more than 64 nodes;
  // words: the giants' scans)
  int32_t *qpos, *parent, *root, *cid, *csize, *fill, *list, *rank, *mids, *bigs, *giants, *words;
  int32_t* ctl;         // the peeling's level ranges and tickets
  SplitLimits limits;
};

// int32 words of the split's outputs (counts (2), queue, comp_of, order (n
// each), comp_ptr (n + 1), local (n)) and of its scratch.
inline size_t split_out_words(int64_t n) { return 2 + 5 * (size_t)n + 1; }
constexpr int kSplitScratch = 13;
inline size_t split_scratch_words(int64_t n) {   // ctl needs up to 64
  return kSplitScratch * std::max<size_t>((size_t)n + 1, 64);
}

// Enqueues the split of the CSR at dptr / dadj (device, int32) on the
// builder's stream, outputs at `out`; no host synchronisation.  Returns the
// addresses it used.  adj_entries: about how many dadj holds.  fault (may be
// null): a device word that, nonzero, makes the graph one without pairs (dptr,
// as ptr_w, is cleared).  counts[1] = -1 afterwards: the host is to split it.
SplitArgs enqueue_split(GraphBuilder& gb, int32_t n, const int32_t* dptr, const int32_t* dadj, int64_t adj_entries,
                        int32_t k, bool simplify, int32_t* out, int32_t* scratch, const int32_t* fault,
                        int32_t* ptr_w);

}  // namespace mpld
