// runtime.h - device context, device buffers, packed batches and kernel
// launchers of the decomposer library (host side).
#pragma once

#include <hip/hip_runtime_api.h>

#include <atomic>
#include <memory>
#include <mutex>
#include <vector>

#include "device_types.h"
#include "internal.h"

namespace mpld {

// kernel launchers (defined with the kernels)
// k: the batch's mask count (every component of a batch shares it).
// wpb: waves per workgroup (1..4); cap < budget stops components after cap
// nodes (status -1, for the heavy-component engine).
// heavy > 0: root split of items 0 .. heavy-1 (cap = ~0, wpb = 4,
// grid >= heavy + ceil((qlen - heavy) / 4)).  mark (cap = ~0 only): a
// component whose search ends without a solution is colored by the
// conflict marking in the same wave.
hipError_t launch_reg_batched(bool trace, int k, int grid, int wpb, RegItems items,
                              int32_t qlen, int32_t* counter, DevRecord* recs, int8_t* colors,
                              uint64_t cap, int32_t heavy, uint32_t chunk, bool mark,
                              hipStream_t s);
// Heavy-component engine: explore / split subtree tasks.
// Task t writes its output block at out + t * kSplitBlockBytes and its
// split items to pool at an offset taken from *pool_count (zero before the
// launch).
hipError_t launch_reg_split(int k, int grid, const SplitTask* tasks, int32_t ntasks,
                            int32_t* counter, RegItems regitems, uint64_t cap,
                            uint32_t levels, uint8_t* out, SplitItem* pool,
                            int32_t* pool_count, hipStream_t s);
// Device-resident heavy engine: move the round window on (one thread), and
// run the current round's tasks (persistent grid; the window comes from
// head).  hc_nodes / hc_limit: per heavy component, explored nodes and the
// limit past which its tasks stop splitting.  trace: tasks and split items
// also carry the trace hashes of their nodes.
hipError_t launch_engine_advance(EngineHead* head, int32_t task_cap, hipStream_t s);
hipError_t launch_engine_round(int k, int grid, EngineHead* head, EngineTask* tasks,
                               int32_t task_cap, uint8_t* blocks, EngineItem* pool,
                               int32_t pool_cap, RegItems regitems,
                               unsigned long long* hc_nodes, const uint64_t* hc_limit,
                               uint64_t cap, uint32_t levels, bool trace, hipStream_t s);
// Scatters `count` resolved heavy components (records and colors).
hipError_t launch_heavy_writeback(const HeavyWrite* w, int32_t count, DevRecord* recs,
                                  int8_t* colors, hipStream_t s);
hipError_t launch_reg_single(bool trace, int k, RegItems items, int32_t item,
                             DevRecord* recs, int8_t* colors, hipStream_t s);
int reg_batched_blocks_per_cu(bool trace);
// Serving tick over register-tier components (see the kernel).
hipError_t launch_reg_tick(bool trace, bool stitch, int k, int grid, const int32_t* list,
                           int32_t len, int32_t* counter, const DevDesc* slot_desc,
                           uint8_t* slot_state, DevRecord* slot_rec, const uint64_t* arena64,
                           int8_t* arena8, const uint8_t* part8, const uint32_t* slot_minb,
                           int32_t* slot_min, uint64_t slice, DevRecord* tick_out, hipStream_t s);
// stitch: the stitch-aware row order (the CSR blocks end with the partners).
hipError_t launch_lds_batched(bool trace, bool big, bool stitch, int waves, int grid,
                              int lds_bytes, const DevDesc* descs, const uint32_t* adj32,
                              int32_t qlen, int32_t* counter, uint64_t* gstack,
                              uint64_t stack_words, DevRecord* recs, int8_t* colors,
                              hipStream_t s);
hipError_t launch_lds_single(bool trace, bool big, bool stitch, int waves, int lds_bytes,
                             const DevDesc* descs, const uint32_t* adj32, int32_t item,
                             uint64_t* gstack, DevRecord* recs, int8_t* colors, hipStream_t s);
// Subtree tasks of LDS-tier (big = false) or big-tier components (trace:
// each task record holds the trace hash of its own nodes).
hipError_t launch_lds_tasks(bool trace, bool big, bool stitch, int waves, int grid, int lds_bytes, const DevDesc* descs,
                            const uint32_t* adj32, const LdsTask* tasks, int32_t ntasks,
                            uint64_t* gstack, uint64_t stack_words, DevRecord* task_recs,
                            int8_t* task_colors, hipStream_t s);
// Writes resolved components' records (rec[i] to recs[comp[i]]) and colors
// (n[i] bytes from src + src_off[i], or -1 when src_off[i] < 0, to colors +
// out_off[i]).
hipError_t launch_csr_writeback(const LdsResolved* w, int32_t count, const int8_t* src,
                                DevRecord* recs, int8_t* colors, hipStream_t s);
// The sequence engine's tasks (seq_types.h): a round's run list of one tier,
// or with `finish` the results of the tier's components (records, colors).
struct SeqArgs;
hipError_t launch_seq_reg(bool trace, int k, int grid, const SeqArgs& a, RegItems items, int32_t parity,
                          bool finish, DevRecord* recs, int8_t* colors, hipStream_t s);
hipError_t launch_seq_csr(bool trace, int k, int grid, int lds_bytes, const SeqArgs& a,
                          const DevDesc* descs, const uint32_t* adj32, uint64_t* stack, uint64_t stack_words,
                          int32_t parity, bool finish, DevRecord* recs, int8_t* colors, hipStream_t s);
// Waves per workgroup for big LDS-tier components of at most max_n nodes.
// The big-tier launchers take waves = 0 for the one-wave wide layout
// (lds_wide_bytes of LDS).
int lds_big_waves(int32_t max_n);
// Conflict marking (MPLD_MARK_CONFLICTS) of the components whose record is
// not FEASIBLE: register-tier items, and CSR components (LDS, big and
// device-wide tiers, one wave each, mark_lds_bytes of LDS).
hipError_t launch_mark_reg(int k, int grid, RegItems items, int32_t qlen, const DevRecord* recs,
                           int8_t* colors, hipStream_t s);
hipError_t launch_mark_lds(int grid, int lds_bytes, const DevDesc* descs, const uint32_t* adj32,
                           int32_t qlen, const DevRecord* recs, int8_t* colors, hipStream_t s);
int64_t mark_lds_bytes(int32_t n, int32_t k);
// Eq. 1 minimisation (MPLD_MINIMIZE) of the register-tier items from the
// incumbent colors in `colors`; partners: stitch partner byte per node
// (indexed like the masks, 0xff none); min_out[comp]: nodes, negated when
// stopped by `budget`, 0 when the incumbent costs nothing.
hipError_t launch_min_reg(int k, int grid, int num_cus, RegItems items, int32_t qlen, const uint8_t* partners,
                          int8_t* colors, int32_t* min_out, uint32_t budget, int32_t* list_len, int32_t* list,
                          hipStream_t s);
// LDS bytes of one LDS-tier component (adj_words = n + 1 + 2m) and the
// global stack words of a big one.
int64_t lds_bytes_for(int32_t n, int32_t k, int64_t adj_words, int32_t max_deg, bool big,
                      bool stitch = false);
int64_t lds_stack_words(int32_t n, int32_t k, int64_t adj_words);
// LDS bytes of a big component on one wave with its neighbour lists in LDS
// (the wide layout), or -1 when that layout does not apply to it.
int64_t lds_wide_bytes(int32_t n, int32_t k, int64_t adj_words, int32_t max_deg, bool stitch);
// Device-wide tier (cooperative launch over `grid` workgroups, one per CU).
hipError_t launch_device_tier(bool trace, int grid, int lds_bytes, const DevDesc* desc,
                              const uint32_t* adj32, unsigned long long* keys, uint64_t* stacks,
                              DevRecord* recs, int8_t* colors, hipStream_t s);
int device_tier_lds_bytes(int32_t n, int grid);
int64_t device_tier_stack_words(int32_t n, int32_t max_deg);
// Allows every LDS-tier kernel up to `bytes` of dynamic LDS (once per context).
void lds_configure(int bytes);

void check_hip(hipError_t e, const char* what);

}  // namespace mpld

namespace mpld {
struct GraphBuilder;
}

struct mpld_context {
  int device = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  mpld_allocator alloc{};
  bool has_alloc = false;
  int num_cus = 0;
  int reg_blocks_per_cu = 1;
  int lds_per_block = 0;
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
  mpld::GraphBuilder* graph_builder = nullptr;   // device layout-graph builder (lazy)
  // page-locked staging of the calls on this context, one copy up and one
  // down at a time (stage_up, stage_down): at most kStageMax bytes each
  void *up = nullptr, *down = nullptr;
  size_t up_bytes = 0, down_bytes = 0;
  // for tests: levels after which a split and rounds after which a recovery are
  // left to the host, nodes and pairs from which a graph goes to the device
  // (-1: the rules), and how often the host took one back
  int32_t split_levels = -1, recover_rounds = -1;
  int64_t flow_from = -1;
  std::atomic<int64_t> splits_left{0}, recoveries_left{0};

  // The sequence engine's workspace, one per context: up to 1.5 GiB where
  // budgets are large, taken by a solve and given back when the call that
  // asked for it ends (one-shot calls), with a batch, or when the context's
  // memory runs out.  Without an allocator of the caller's, up to kSeqKeep bytes
  // stay for the next call (hipMalloc and hipFree of 100 MiB take 0.3 ms, as
  // long as a component of 600 nodes that is colored at once).
  static constexpr size_t kSeqKeep = (size_t)512 << 20;
  void* seq_mem = nullptr;
  size_t seq_bytes = 0;
  bool seq_used = false;   // a solve is between its launches
  std::mutex seq_mu;

  void* try_alloc(size_t bytes);   // null: there is not as much
  void* dev_alloc(size_t bytes);
  void dev_free(void* p);
  // At least `bytes` of workspace for the launches to come on the stream;
  // false: there is not as much.
  bool seq_take(size_t bytes);
  // Gives the workspace back, once the stream has passed its launches.
  void seq_give_back();
  // The call that used it ends.
  void seq_done() {
    if (has_alloc || seq_bytes > kSeqKeep) seq_give_back();
  }
};

namespace mpld {

// Device memory owned through the context's allocator.
struct DevBuf {
  mpld_context* ctx = nullptr;
  void* p = nullptr;
  size_t bytes = 0;
  DevBuf() = default;
  DevBuf(const DevBuf&) = delete;
  DevBuf& operator=(const DevBuf&) = delete;
  ~DevBuf() { release(); }
  void release() {
    if (p && ctx) ctx->dev_free(p);
    p = nullptr;
    bytes = 0;
  }
  void alloc(mpld_context* c, size_t n) {
    release();
    ctx = c;
    p = c->dev_alloc(n ? n : 256);
    bytes = n ? n : 256;   // (none if that threw)
  }
  // `n` bytes of `of` from byte `at` on; not owned
  void view(const DevBuf& of, size_t at, size_t n) {
    release();
    ctx = nullptr;
    bytes = n ? n : 256;
    p = of.as<uint8_t>() + at;
  }
  template <class T>
  T* as() const { return static_cast<T*>(p); }
};

// Page-locked host memory (hipHostMalloc), for small transfers that the
// host waits on.
struct PinnedBuf {
  void* p = nullptr;
  size_t bytes = 0;
  PinnedBuf() = default;
  PinnedBuf(const PinnedBuf&) = delete;
  PinnedBuf& operator=(const PinnedBuf&) = delete;
  ~PinnedBuf() { release(); }
  void release() {
    if (p) (void)hipHostFree(p);
    p = nullptr;
    bytes = 0;
  }
  // grows (never shrinks); false if the allocation failed
  bool reserve(size_t n) {
    if (n <= bytes) return true;
    release();
    if (hipHostMalloc(&p, n, hipHostMallocDefault) != hipSuccess) {
      p = nullptr;
      return false;
    }
    bytes = n;
    return true;
  }
  template <class T>
  T* as() const { return static_cast<T*>(p); }
};

// Page-locked memory of at least n bytes for one copy on the context's
// stream: the context's own staging up to kStageMax bytes, `own` beyond.
// Allocating and freeing a page-locked buffer takes some 45 us, as long as a
// small batch's search and copies together; the context keeps its staging
// until it is destroyed.  stage_up waits for the stream, so that the copy
// before has been read; what is staged down is taken out before the next use.
constexpr size_t kStageMin = 256 << 10, kStageMax = 4 << 20;
uint8_t* stage_up(mpld_context* ctx, size_t n, PinnedBuf& own);
uint8_t* stage_down(mpld_context* ctx, size_t n, PinnedBuf& own);

// What a CSR component takes in the one-wave layouts (-1: not in that one).
struct CsrShape {
  int64_t small_bytes = -1, wide_bytes = -1, stack_words = 0;
};

// Host-side packed exact-cover image of a set of components.
struct Image {
  std::vector<DevDesc> desc;       // by component id
  std::vector<uint64_t> masks;     // register tier: one neighbour mask per node
  std::vector<uint8_t> partner8;   // register tier: local stitch partner per node (0xff none)
  bool stitch = false;             // MPLD_STITCH_ORDER: items carry the partners
  bool csr_stitch = false;         // MPLD_STITCH_ORDER: CSR blocks end with the partners
  bool minimize = false;           // MPLD_MINIMIZE: partner8 holds the partners
  std::vector<uint32_t> adj32;     // LDS tiers: row offsets, ids, max degree
  int64_t mask_words = 0, adj_words = 0;   // sizes of masks and adj32 (which stay empty when the
                                           // device packs the components)
  std::vector<int32_t> q_reg, q_lds, q_big, q_dev;   // component ids per tier
  int32_t total_nodes = 0;
  int32_t max_size = 0;
  int64_t core_edges = 0;
  int64_t lds_bytes_small = 0;     // largest footprint on the LDS tier
  int64_t lds_bytes_big = 0;       // largest footprint on the big tier
  std::vector<CsrShape> csr_shape;   // by component id, CSR tiers
  // per component id, big tier: its LDS bytes in the workgroup layout and
  // in the one-wave layout (-1: that layout does not take it)
  std::vector<int64_t> big_bytes_wg, big_bytes_wide;
  int64_t big_stack_words = 0;     // largest global stack of the big tier
  int32_t big_max_n = 0;           // largest component of the big tier
  int64_t mark_lds = 0;            // LDS of the conflict marking of CSR components
  int64_t dev_stack_words = 0;     // largest per-workgroup stack of the device tier
  int32_t dev_max_n = 0;
};

// LDS byte limit for a component to keep its lists and stack in LDS.
constexpr int64_t kLdsSmallLimit = 64 * 1024;

// Launch parameters of a batch (chosen by the autotuner or defaults).
struct Tune {
  int32_t waves_per_block = 4;   // register tier workgroup = 64 * waves
  int32_t max_blocks = 0;        // register tier grid cap; 0 = one wave per component
  int32_t use_graph = 0;         // replay a captured HIP graph (off: direct launches are cheaper for the usual one or two kernels)
  int32_t order = 0;             // 0 largest first, 1 smallest first
  int32_t giant_device = 0;      // giants on the device-wide tier instead of the big tier
  int32_t giant_min_nodes = 4096;
  int32_t heavy_first_cap = 128;   // heavy-component engine: first-pass node cap
  int32_t heavy_round_cap = 256;   // nodes per subtree task and round
  int32_t heavy_levels = 0;        // levels per split; 0 = by k (4, 3 or 2)
  int32_t heavy_device = 1;        // 1: rounds chained on the device; 0: host-driven rounds
  int32_t root_split = 1;          // root split of the largest register-tier items
  int32_t root_split_min_n = 4;    // smallest item that gets one
  int32_t root_split_max = 0;      // most items that get one; 0 = all
  int32_t root_split_chunk = 16;   // helper nodes between release checks
  int32_t big_one_wave = 1;        // big tier on one wave (wide layout) when every component fits
};

// Adds one component (local numbering, pairs i < j or j < i) to the image.
// Throws MPLD_E_UNSUPPORTED when a forced tier cannot take it or it does
// not fit any tier.
// partner: local stitch partner per node (-1 none), for MPLD_STITCH_ORDER.
void image_add(Image& im, mpld_context* ctx, int32_t n, const int32_t* pairs, int64_t m,
               int32_t k, int64_t budget, uint32_t flags, const int32_t* partner = nullptr);
// The same for a component whose data the device packs: its shape alone.
void image_place(Image& im, mpld_context* ctx, int32_t n, int64_t m, int32_t max_deg, int32_t k,
                 int64_t budget, uint32_t flags);
// Sorts each tier's queue by size (descending, or ascending when order = 1),
// ties by id.
void image_finish(Image& im, int order = 0);

// Device copy of an image plus its outputs and queue counters.
struct DeviceBatch {
  mpld_context* ctx = nullptr;
  // one block of device memory: counters | desc | regitems | adj32, filled by
  // one copy where they fit the staging, then recs | colors | min_out, read
  // back by one
  DevBuf mem;
  DevBuf desc, regitems, adj32, counters, recs, colors;  // views of mem; desc in launch order
  DevBuf gstack;
  std::vector<uint8_t> got;   // recs | colors of the last solve, where its check for
                              // heavy components has read them already
  size_t result_bytes(bool with_min) const {
    return (size_t)((with_min ? min_out : colors).as<uint8_t>() - recs.as<uint8_t>()) +
           (with_min ? min_out : colors).bytes;
  }
  uint32_t reg_width = 1;   // masks per register-tier item
  bool reg_stitch = false;  // items carry stitch partners
  bool csr_stitch = false;  // CSR blocks end with stitch partners (LDS and big tiers)
  RegItems reg_items() const {
    const uint32_t pb = reg_stitch ? (reg_width + 7u) & ~7u : 0u;
    return RegItems{regitems.as<uint8_t>(), reg_width, kRegItemHead + 8u * reg_width + pb,
                    reg_stitch ? kRegItemHead + 8u * reg_width : 0u};
  }
  DevBuf dev_keys, dev_stacks;      // device-wide tier
  DevBuf partners, min_out;         // MPLD_MINIMIZE: stitch partners, per-component node counts (views)
  DevBuf min_list;                  // MPLD_MINIMIZE: items that one wave leaves to a workgroup (view)
  uint32_t min_budget = 10000;      // MPLD_MINIMIZE: nodes per component
  DevBuf sp_tasks, sp_out, sp_pool, sp_writes;      // heavy-component engine
  PinnedBuf sp_host_tasks, sp_host_out, sp_host_pool, sp_host_writes, sp_host_recs;
  DevBuf en_meta, en_tasks, en_blocks, en_pool;     // device-resident rounds
  DevBuf ct_tasks, ct_recs, ct_colors, ct_resolved; // LDS/big-tier subtree tasks
  PinnedBuf ct_host;
  std::vector<uint8_t> sp_host_copy;                // engine results in ordinary memory
  int64_t sp_rounds = 0, sp_tasks_run = 0, sp_heavy = 0, sp_reruns = 0;  // last solve's stats
  Tune tune;
  int32_t n_reg = 0, n_lds = 0, n_big = 0, n_dev = 0;
  // the first n_wide big-tier components take the one-wave layout
  // (lds_wide bytes, grid_wide workgroups), the rest the workgroup layout
  // (lds_big bytes, big_waves waves, grid_big workgroups)
  int32_t n_wide = 0;
  int lds_wide = 0, grid_wide = 1;
  int grid_dev = 1, lds_dev = 0;
  int32_t num_comps = 0, total_nodes = 0;
  int32_t k = 3;
  int grid_reg = 1, grid_lds = 1, grid_big = 1;
  int grid_big_tasks = 1;   // big-tier subtree tasks (stack areas allocated for this many blocks)
  int lds_small = 0, lds_big = 0;
  int big_waves = 1;   // waves per workgroup on the big tier
  int32_t reg_heavy = 0;   // register-tier items (a launch-order prefix) with a root split
  int64_t mark_lds = 0;   // LDS bytes of the CSR conflict marking
  uint64_t big_stack_words = 0;
  float last_search_ms = 0.f, last_total_ms = 0.f;
  int32_t launches = 0;
  hipGraphExec_t graph = nullptr;
  uint32_t graph_flags = 0xffffffffu;
  bool timed = false;               // events of the last solve not read yet
  std::vector<uint8_t> host_items;  // register-tier items as uploaded
  bool device_packed = false;       // items and adjacency were packed on the device
  // MPLD_ROUNDTRIP: page-locked copies of the image and the results, and
  // the two events around the whole solve
  PinnedBuf rt_up, rt_down;
  bool rt_ready = false, rt_timed = false;
  hipEvent_t rt_ev[2] = {nullptr, nullptr};
  float last_roundtrip_ms = 0.f;
  std::vector<int32_t> host_queue;  // component ids in launch order (all tiers)
  std::vector<DevDesc> host_desc;   // descriptors in launch order
  std::vector<CsrShape> csr_shape;  // by launch position past the register tier
  ~DeviceBatch();
};

// A layout graph on the device (flow_device.hip): the CSR of the caller's
// pairs and its split, kept for the packing and for collecting results.
struct FlowComp {
  int32_t n, m2, max_deg, first;   // nodes, adjacency entries, largest degree, smallest id
};
struct FlowGraph {
  bool active = false;
  bool host_form = false;   // the host has the graph and its split too, and collects
  int32_t n = 0, removed = 0, ncomp = 0;
  int64_t m = 0;
  bool simplify = true;
  DevBuf keep;   // everything below
  int32_t *ptr = nullptr, *adj = nullptr, *partner = nullptr, *queue = nullptr, *comp_of = nullptr,
          *order = nullptr, *comp_ptr = nullptr, *local = nullptr;
  int32_t *cpre = nullptr, *cmax = nullptr;   // core degrees' prefix over `order`; largest per component
  std::vector<FlowComp> comps;
  ~FlowGraph();   // waits for the stream: its memory may be in use
  void drop();    // gives it back: the host path has the graph
};
struct GraphBuilder;
// Validates and splits a caller's graph on the device.  False: the host path
// is to take it (a fault to report, nothing that the flow is made for, or no
// memory for it).
bool flow_build(FlowGraph& f, GraphBuilder& gb, const mpld_graph& in, int32_t k, bool simplify);
// Enqueues the packing of the batch's components (db laid out from their
// shapes, its descriptors on the device).
void flow_pack(FlowGraph& f, DeviceBatch& db, hipStream_t st);
// Recovery, tallies and the result of a solved batch; waits.  False: the
// recovery was given up, or there is no memory for it (nothing in *r): the host
// does it.
bool flow_collect(FlowGraph& f, GraphBuilder& gb, const mpld_options& opt, DeviceBatch& db,
                  mpld_result* r);
// The split in a caller's arrays (n, n, n, n + 1 entries; as many as it has are written); waits.
void flow_split_out(FlowGraph& f, GraphBuilder& gb, int32_t* removal, int32_t* comp_of, int32_t* order,
                    int32_t* comp_ptr);
// The host forms of the graph and its split.
void flow_to_host(FlowGraph& f, GraphBuilder& gb, Graph& g, Split& s);

// flow: the components' data are packed by the device from that graph (im
// then holds their shapes only); the copies are not waited for.
void device_upload(mpld_context* ctx, const Image& im, DeviceBatch& db, const Tune& tune = Tune(),
                   FlowGraph* flow = nullptr);
// Enqueues the search of every component on the context stream (no wait).
void device_solve(DeviceBatch& db, uint32_t flags);
// Result of a decomposition from the device records and local colors: maps
// local colors to nodes, fills the component records, recovers the removed
// nodes and computes the Eq. 1 tallies.
void assemble_result(const Graph& g, const Split& s, const Image& im, const mpld_options& opt,
                     const std::vector<DevRecord>& recs, const std::vector<int8_t>& lcol,
                     mpld_result* r, const std::vector<int32_t>* min_nodes = nullptr);

// The whole device solve: image H2D from page-locked memory, the search
// (device_solve with `flags`), records and local colors D2H, between two
// events (read by device_time into last_roundtrip_ms).
void device_roundtrip(DeviceBatch& db, const Image& im, uint32_t flags);
// Searches the components at these launch positions (register tier, LDS tier,
// one-wave big tier) with the sequence engine and writes their records and
// colors; waits for the rounds.  False: there was no memory for it, or for some
// of them (their records are not written).
bool seq_solve(DeviceBatch& db, const std::vector<int32_t>& positions, bool trace);
constexpr int32_t kSeqRoundsPerCheck = 3;      // rounds enqueued between looks at the head
constexpr int32_t kSeqMaxRounds = 1 << 16;     // then the callers search one component after another
// Reads the last solve's event time if the stream has passed it.
bool device_time(DeviceBatch& db);
// Waits, then copies records and colors back (and, when the batch was
// packed for MPLD_MINIMIZE and min_nodes is given, the minimisation's node
// counts per component: 0 for components off the register tier).
void device_fetch(DeviceBatch& db, std::vector<DevRecord>& recs, std::vector<int8_t>& colors,
                  std::vector<int32_t>* min_nodes = nullptr);

}  // namespace mpld

struct mpld_batch {
  mpld_context* ctx = nullptr;
  mpld::Graph g;
  mpld::Split s;
  mpld::FlowGraph flow;   // active: the graph and its split are on the device
                          // instead (s.comp_ptr is filled all the same)
  mpld_options opt{};
  mpld::Image im;
  mpld::DeviceBatch db;
  bool solved = false;
  bool tuned_from_cache = false;
  // its buffers go back while nothing on the stream uses them
  ~mpld_batch() {
    if (!ctx) return;
    (void)hipStreamSynchronize(ctx->stream);
    ctx->seq_done();
  }
};

namespace mpld {
// Packs the batch's components with tune `t` (tier of giants, queue order)
// and uploads them (launch geometry).
void batch_pack(mpld_batch* b, const Tune& t);
// Looks the batch's shape up in the tuning cache (path, else $MPLD_TUNE_CACHE);
// true and *t filled on a hit.
bool tune_from_cache(mpld_batch* b, const char* path, Tune* t);
// Device layout-graph builder (graph_device.hip).  own_stream: a stream of
// its own (server front-end workers), else the context's stream.
GraphBuilder* graph_builder_create(mpld_context* ctx, bool own_stream);
void graph_builder_destroy(GraphBuilder* gb);
// Allocates the builder's device and pinned buffers for layouts of up to
// about `nodes` nodes ahead of use (they still grow beyond).
void graph_builder_reserve(GraphBuilder& gb, int32_t nodes);
// Builds the CSR layout graph of `rects` on the device.  With `split`, the
// simplification and sub-graph split (identical to simplify_and_split(g, k,
// simplify)) run on the device too when device_split_pays for the graph;
// returns whether *split was filled.
bool build_layout_graph_device(GraphBuilder& gb, const mpld_rect* rects, int32_t n, int32_t dmin,
                               int32_t split_len, Graph& g, Split* split = nullptr, int32_t k = 0,
                               bool simplify = true);
// The same graph as pairs, u < v, sorted: conflict pairs, then stitch pairs.
void build_layout_pairs_device(GraphBuilder& gb, const mpld_rect* rects, int32_t n, int32_t dmin,
                               int32_t split_len, DevicePairs& out);
// Whether a server splits a device-built graph of n nodes with `adj_entries`
// (= 2 |CE|) adjacency entries on the device too: below an average conflict
// degree of k the peeling leaves small components.  Above it they can be large,
// whose numbering goes level by level, and their lists come back to the host
// either way.  Six packed layouts (degree 22) at once, split on the host / on
// the device: 4200 rects 3.9 / 5.3 ms, 8000 5.6 / 7.4, 16000 9.6 / 12.1.
inline bool device_split_pays(int64_t n, int64_t adj_entries, int32_t k) {
  return adj_entries < (int64_t)k * n;
}

}  // namespace mpld
