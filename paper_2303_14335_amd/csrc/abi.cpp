// abi.cpp - the C ABI of include/mpld.h: argument checks, error mapping,
// and the flow of Sec. 2.2 (front-end -> device search -> recovery).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <new>

#include "graph_builder.h"
#include "runtime.h"

namespace mpld {
const char* last_error_cstr();
}

using namespace mpld;

namespace {

template <class F>
int32_t guard(F&& f) {
  try {
    f();
    set_last_error("");
    return MPLD_OK;
  } catch (const Error& e) {
    set_last_error(e.what);
    return e.code;
  } catch (const std::bad_alloc&) {
    set_last_error("host allocation failed");
    return MPLD_E_NOMEM;
  } catch (const std::exception& e) {
    set_last_error(e.what());
    return MPLD_E_INTERNAL;
  } catch (...) {
    set_last_error("unknown exception");
    return MPLD_E_INTERNAL;
  }
}

void check_options(const mpld_options* opt) {
  if (!opt) fail(MPLD_E_INVALID, "options are NULL");
  if (opt->struct_size != sizeof(mpld_options))
    fail(MPLD_E_INVALID, "options.struct_size does not match this library's mpld_options");
  if (opt->k < 2 || opt->k > MPLD_MAX_K) fail(MPLD_E_INVALID, "k must be in [2, 8]");
  if (opt->node_budget < 1) fail(MPLD_E_INVALID, "node_budget must be >= 1");
  const uint32_t forced =
      opt->flags & (MPLD_FORCE_WAVE | MPLD_FORCE_LDS | MPLD_FORCE_GLOBAL | MPLD_FORCE_DEVICE);
  if (forced & (forced - 1)) fail(MPLD_E_INVALID, "at most one MPLD_FORCE_* flag");
  if (opt->min_budget < 0) fail(MPLD_E_INVALID, "min_budget must be >= 0 (0 = 10000)");
}

// Graphs of at least this many nodes and pairs together go through the
// device's flow: some 35 launches, 0.3 ms whatever the size, where the host's
// passes take time in proportion to both, 20 to 25 ns each where a node's
// neighbours lie anywhere in memory.  Host against device, ms: k = 3, 13,300
// together 0.30 / 0.30, 19,800 0.44 / 0.31, 32,900 0.69 / 0.34, 82,700 1.5 /
// 0.37; k = 4 with stitches, 19,800 0.92 / 0.74.
// Where ids follow the layout the host takes 7 ns: a path of 40,000 together
// 0.28 / 0.42, of 80,000 0.63 / 0.60, of 200,000 1.25 / 1.17.  That is told from
// 64 of the pairs: in such a graph most join near ids.  A node without pairs
// costs the host a quarter of a pair (14,000 / 30,000 / 60,000 of them 0.10 /
// 0.16 / 0.41, on the device 0.2), so there have to be 8,000 by that measure.
// A graph that the device gives up (split_limits in graph_device.hip: deep
// peelings, long narrow components; a recovery that is one long chain) costs
// the front of the flow besides.  Host alone / both, ms: lines with two
// neighbours on either side (k = 3), ids in order, 60,000 0.43 / 0.43 (the host's
// at once), 300,000 2.0 / 2.4, ids in no order, 24,000 0.39 / 0.62, 60,000 1.0 /
// 1.3, 300,000 6.1 / 6.4; a packed window of 1:100, 50,000 2.0 / 2.4, 106,000
// 4.0 / 4.4, 455,000 17.1 / 20.1.
constexpr int64_t kFlowMinSize = 14000, kFlowMinOrdered = 60000, kFlowMinPairs = 8000;

bool flow_pays(const mpld_context& ctx, const mpld_graph& g) {
  const int64_t size = (int64_t)g.num_nodes + g.num_ce;
  if (ctx.flow_from >= 0) return size >= ctx.flow_from;
  if (size < kFlowMinSize || (int64_t)g.num_nodes / 4 + g.num_ce < kFlowMinPairs) return false;
  if (size >= kFlowMinOrdered || g.num_ce <= 0 || !g.ce) return true;
  int near = 0;
  for (int64_t i = 0; i < 64; ++i) {
    const int32_t* e = g.ce + 2 * (i * g.num_ce / 64);
    near += std::abs((int64_t)e[0] - e[1]) <= 64 ? 1 : 0;
  }
  return near < 48;
}

void use_device(mpld_context* ctx) {
  if (!ctx) fail(MPLD_E_INVALID, "context is NULL");
  check_hip(hipSetDevice(ctx->device), "hipSetDevice");
}

// Builds the batch: front-end, then packing and upload with the batch's
// launch parameters (from the tuning cache when one is configured).
void batch_build(mpld_context* ctx, const mpld_graph* g, const mpld_options* opt, mpld_batch* b) {
  if (!g) fail(MPLD_E_INVALID, "graph is NULL");
  check_options(opt);
  b->ctx = ctx;
  b->opt = *opt;
  const bool simplify = opt->flags & MPLD_SIMPLIFY;
  // large graphs are validated, simplified, split and packed on the
  // device (identical results)
  if (flow_pays(*ctx, *g)) {
    if (!ctx->graph_builder) ctx->graph_builder = graph_builder_create(ctx, false);
    (void)flow_build(b->flow, *ctx->graph_builder, *g, opt->k, simplify);
  }
  if (b->flow.active) {
    b->s.comp_ptr.assign(1, 0);
    for (const FlowComp& c : b->flow.comps) b->s.comp_ptr.push_back(b->s.comp_ptr.back() + c.n);
  }
  Tune t;
  if (b->flow.active) {
    tune_from_cache(b, nullptr, &t);
    try {
      batch_pack(b, t);
      return;
    } catch (const NoMemory&) {
    }
    // the components themselves may fit where they and the graph do not
    b->flow.drop();
    ctx->graph_builder->flow_ws.release();
    t = Tune();
  }
  b->g = make_graph(*g);
  b->s = simplify_and_split(b->g, opt->k, simplify);
  tune_from_cache(b, nullptr, &t);
  batch_pack(b, t);
}

uint32_t min_budget_of(const mpld_options* opt) {
  return opt->min_budget > 0 ? (uint32_t)opt->min_budget : 10000u;
}

void batch_collect(mpld_batch* b, mpld_result* r) {
  if (b->flow.active && !b->flow.host_form) {
    if (flow_collect(b->flow, *b->ctx->graph_builder, b->opt, b->db, r)) return;
    // a recovery that the device gave up: this batch's host form from now on
    // (the packed components stay as they are)
    flow_to_host(b->flow, *b->ctx->graph_builder, b->g, b->s);
    b->flow.host_form = true;
  }
  std::vector<DevRecord> recs;
  std::vector<int8_t> lcol;
  std::vector<int32_t> mins;
  const bool minimize = b->opt.flags & MPLD_MINIMIZE;
  device_fetch(b->db, recs, lcol, minimize ? &mins : nullptr);
  assemble_result(b->g, b->s, b->im, b->opt, recs, lcol, r, minimize ? &mins : nullptr);
}

}  // namespace

extern "C" {

uint32_t mpld_abi_version(void) { return MPLD_ABI_VERSION; }

const char* mpld_error_string(int32_t err) {
  switch (err) {
    case MPLD_OK: return "ok";
    case MPLD_E_INVALID: return "invalid argument";
    case MPLD_E_NOMEM: return "out of memory";
    case MPLD_E_DEVICE: return "device error";
    case MPLD_E_NOT_READY: return "not ready";
    case MPLD_E_CANCELLED: return "cancelled";
    case MPLD_E_INTERNAL: return "internal error";
    case MPLD_E_UNSUPPORTED: return "unsupported";
    default: return "unknown error code";
  }
}

const char* mpld_last_error(void) { return last_error_cstr(); }

int32_t mpld_build_graph(const mpld_rect* rects, int32_t n, int32_t dmin_nm, int32_t split_len_nm,
                         mpld_owned_graph** out) {
  return guard([&] {
    if (!out) fail(MPLD_E_INVALID, "out is NULL");
    *out = nullptr;
    auto* g = new mpld_owned_graph();
    try {
      build_layout_graph(rects, n, dmin_nm, split_len_nm, g->g);
    } catch (...) {
      delete g;
      throw;
    }
    *out = g;
  });
}

int32_t mpld_build_graph_device(mpld_context* ctx, const mpld_rect* rects, int32_t n,
                                int32_t dmin_nm, int32_t split_len_nm, mpld_owned_graph** out) {
  return guard([&] {
    if (!out) fail(MPLD_E_INVALID, "out is NULL");
    *out = nullptr;
    use_device(ctx);
    if (!ctx->graph_builder) ctx->graph_builder = graph_builder_create(ctx, false);
    std::unique_ptr<mpld_owned_graph> og(new mpld_owned_graph());
    og->from_device = true;
    build_layout_pairs_device(*ctx->graph_builder, rects, n, dmin_nm, split_len_nm, og->d);
    *out = og.release();
  });
}

int32_t mpld_split_graph_device(mpld_context* ctx, const mpld_graph* g, int32_t k, uint32_t flags,
                                int32_t* removal_order, int32_t* num_removed, int32_t* comp_of,
                                int32_t* bfs_order, int32_t* comp_ptr, int32_t* num_comps) {
  return guard([&] {
    if (!g || !removal_order || !num_removed || !comp_of || !bfs_order || !comp_ptr || !num_comps)
      fail(MPLD_E_INVALID, "NULL argument");
    if (k < 2 || k > MPLD_MAX_K) fail(MPLD_E_INVALID, "k outside [2, MPLD_MAX_K]");
    use_device(ctx);
    if (!ctx->graph_builder) ctx->graph_builder = graph_builder_create(ctx, false);
    FlowGraph f;
    if (flow_build(f, *ctx->graph_builder, *g, k, flags & MPLD_SIMPLIFY)) {
      flow_split_out(f, *ctx->graph_builder, removal_order, comp_of, bfs_order, comp_ptr);
      *num_removed = f.removed;
      *num_comps = f.ncomp;
      return;
    }
    const Split s = simplify_and_split(make_graph(*g), k, flags & MPLD_SIMPLIFY);
    std::copy(s.removal.begin(), s.removal.end(), removal_order);
    *num_removed = (int32_t)s.removal.size();
    std::copy(s.comp_of.begin(), s.comp_of.end(), comp_of);
    std::copy(s.order.begin(), s.order.end(), bfs_order);
    std::copy(s.comp_ptr.begin(), s.comp_ptr.end(), comp_ptr);
    *num_comps = (int32_t)s.comp_ptr.size() - 1;
  });
}

// For tests, and not declared in the header: levels after which a split and
// rounds after which a recovery are left to the host, and nodes and pairs from
// which a graph goes to the device (-1: the rules); left: how often the host has
// taken a split and a recovery back on this context.
int32_t mpld_test_flow_limits(mpld_context* ctx, int32_t levels, int32_t rounds, int64_t from, int64_t* left) {
  return guard([&] {
    if (!ctx || !left) fail(MPLD_E_INVALID, "NULL argument");
    ctx->split_levels = levels;
    ctx->recover_rounds = rounds;
    ctx->flow_from = from;
    left[0] = ctx->splits_left;
    left[1] = ctx->recoveries_left;
  });
}

int32_t mpld_owned_graph_view(const mpld_owned_graph* g, mpld_graph* view) {
  return guard([&] {
    if (!g || !view) fail(MPLD_E_INVALID, "NULL argument");
    view->reserved = 0;
    if (g->from_device) {
      view->num_nodes = g->d.num_nodes;
      view->num_ce = g->d.num_ce;
      view->ce = g->d.ce.get();
      view->num_se = g->d.num_se;
      view->se = g->d.ce ? g->d.ce.get() + 2 * g->d.num_ce : nullptr;
      return;
    }
    view->num_nodes = g->g.num_nodes;
    view->num_ce = (int64_t)g->g.ce.size() / 2;
    view->ce = g->g.ce.data();
    view->num_se = (int64_t)g->g.se.size() / 2;
    view->se = g->g.se.data();
  });
}

void mpld_owned_graph_free(mpld_owned_graph* g) { delete g; }

int32_t mpld_context_create(int32_t device, const mpld_allocator* alloc, void* hip_stream,
                            mpld_context** out) {
  return guard([&] {
    if (!out) fail(MPLD_E_INVALID, "out is NULL");
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count == 0)
      fail(MPLD_E_DEVICE, "no HIP device is visible");
    if (device < 0 || device >= count) fail(MPLD_E_DEVICE, "device ordinal out of range");
    check_hip(hipSetDevice(device), "hipSetDevice");
    hipDeviceProp_t prop;
    check_hip(hipGetDeviceProperties(&prop, device), "hipGetDeviceProperties");
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
      fail(MPLD_E_DEVICE, std::string("device is ") + prop.gcnArchName + ", this library is built for gfx950");
    if (alloc && (!alloc->alloc || !alloc->free)) fail(MPLD_E_INVALID, "allocator lacks alloc or free");
    auto* ctx = new mpld_context();
    ctx->device = device;
    ctx->num_cus = prop.multiProcessorCount;
    ctx->lds_per_block = (int)prop.sharedMemPerBlock;
    if (alloc) {
      ctx->alloc = *alloc;
      ctx->has_alloc = true;
    }
    try {
      if (hip_stream) {
        ctx->stream = static_cast<hipStream_t>(hip_stream);
      } else {
        check_hip(hipStreamCreateWithFlags(&ctx->stream, hipStreamNonBlocking), "stream");
        ctx->own_stream = true;
      }
      for (auto& e : ctx->ev) check_hip(hipEventCreate(&e), "event");
      ctx->reg_blocks_per_cu = reg_batched_blocks_per_cu(false);
      lds_configure(ctx->lds_per_block);
    } catch (...) {
      mpld_context_destroy(ctx);
      throw;
    }
    *out = ctx;
  });
}

int32_t mpld_context_destroy(mpld_context* ctx) {
  if (!ctx) return MPLD_OK;
  (void)hipSetDevice(ctx->device);
  if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
  if (ctx->graph_builder) graph_builder_destroy(ctx->graph_builder);
  ctx->seq_give_back();
  for (auto& e : ctx->ev)
    if (e) (void)hipEventDestroy(e);
  if (ctx->up) (void)hipHostFree(ctx->up);
  if (ctx->down) (void)hipHostFree(ctx->down);
  if (ctx->own_stream && ctx->stream) (void)hipStreamDestroy(ctx->stream);
  delete ctx;
  return MPLD_OK;
}

int32_t mpld_batch_create(mpld_context* ctx, const mpld_graph* g, const mpld_options* opt,
                          mpld_batch** out) {
  return guard([&] {
    if (!out) fail(MPLD_E_INVALID, "out is NULL");
    *out = nullptr;
    use_device(ctx);
    auto* b = new mpld_batch();
    try {
      batch_build(ctx, g, opt, b);
      // a batch is ready when the call returns
      check_hip(hipStreamSynchronize(ctx->stream), "batch");
    } catch (...) {
      delete b;
      throw;
    }
    *out = b;
  });
}

int32_t mpld_batch_solve(mpld_batch* b, uint32_t flags) {
  return guard([&] {
    if (!b) fail(MPLD_E_INVALID, "batch is NULL");
    use_device(b->ctx);
    const uint32_t how = MPLD_PLAIN | MPLD_DIRECT;
    const uint32_t f = (b->opt.flags & ~how) | (flags & (how | MPLD_SPLIT_HEAVY | MPLD_UNTIMED));
    if (flags & MPLD_ROUNDTRIP)
      device_roundtrip(b->db, b->im, f);
    else
      device_solve(b->db, f);
    b->solved = true;
  });
}

int32_t mpld_batch_result(mpld_batch* b, mpld_result** out) {
  return guard([&] {
    if (!b || !out) fail(MPLD_E_INVALID, "NULL argument");
    *out = nullptr;
    if (!b->solved) fail(MPLD_E_INVALID, "batch was not solved");
    use_device(b->ctx);
    auto* r = new mpld_result();
    try {
      batch_collect(b, r);
    } catch (...) {
      delete r;
      throw;
    }
    *out = r;
  });
}

int32_t mpld_batch_get_info(mpld_batch* b, mpld_batch_info* info) {
  return guard([&] {
    if (!b || !info) fail(MPLD_E_INVALID, "NULL argument");
    use_device(b->ctx);
    device_time(b->db);
    std::memset(info, 0, sizeof(*info));
    info->num_components = b->db.num_comps;
    info->num_wave = b->db.n_reg;
    info->num_lds = b->db.n_lds;
    info->num_global = b->db.n_big;
    info->core_nodes = b->im.total_nodes;
    info->max_size = b->im.max_size;
    info->image_bytes = (int64_t)(b->db.desc.bytes + b->db.regitems.bytes + b->db.adj32.bytes);
    info->core_edges = b->im.core_edges;
    info->last_search_ms = b->db.last_search_ms;
    info->last_total_ms = b->db.last_total_ms;
    info->launches = b->db.launches;
    info->num_device = b->db.n_dev;
    info->heavy_components = (int32_t)b->db.sp_heavy;
    info->split_rounds = (int32_t)b->db.sp_rounds;
    info->split_tasks = (int32_t)b->db.sp_tasks_run;
    info->split_reruns = (int32_t)b->db.sp_reruns;
    info->last_roundtrip_ms = b->db.last_roundtrip_ms;
    info->big_waves = b->db.n_big > b->db.n_wide ? b->db.big_waves : 0;
  });
}

void mpld_batch_free(mpld_batch* b) {
  if (!b) return;
  if (b->ctx) {
    (void)hipSetDevice(b->ctx->device);
    (void)hipStreamSynchronize(b->ctx->stream);
  }
  delete b;
}

int32_t mpld_decompose(mpld_context* ctx, const mpld_graph* g, const mpld_options* opt,
                       mpld_result** out) {
  return guard([&] {
    if (!out) fail(MPLD_E_INVALID, "out is NULL");
    *out = nullptr;
    use_device(ctx);
    mpld_batch b;
    batch_build(ctx, g, opt, &b);
    // one-shot: no graph to capture; it waits anyway, so heavy components
    // always go to the subtree engine
    device_solve(b.db, opt->flags | MPLD_DIRECT | MPLD_SPLIT_HEAVY);
    b.solved = true;
    auto* r = new mpld_result();
    try {
      batch_collect(&b, r);
    } catch (...) {
      delete r;
      throw;
    }
    *out = r;
  });
}

int32_t mpld_solve_components(mpld_context* ctx, const mpld_component* comps, int32_t count,
                              const mpld_options* opt, mpld_comp_record* out, int8_t* colors_out) {
  return guard([&] {
    use_device(ctx);
    check_options(opt);
    if (count < 0 || (count > 0 && (!comps || !out || !colors_out)))
      fail(MPLD_E_INVALID, "bad component array");
    Image im;
    std::vector<int32_t> pairs;
    for (int32_t c = 0; c < count; ++c) {
      const mpld_component& cp = comps[c];
      if (cp.n < 0 || cp.m < 0 || (cp.m > 0 && !cp.edges))
        fail(MPLD_E_INVALID, "component " + std::to_string(c) + " has a bad size or edge array");
      std::vector<uint64_t> keys((size_t)cp.m);
      for (int64_t e = 0; e < cp.m; ++e) {
        int32_t a = cp.edges[2 * e], b = cp.edges[2 * e + 1];
        if (a < 0 || b < 0 || a >= cp.n || b >= cp.n || a == b)
          fail(MPLD_E_INVALID, "component " + std::to_string(c) + " edge " + std::to_string(e) +
                                   " is out of range or a self loop");
        if (a > b) std::swap(a, b);
        keys[e] = ((uint64_t)(uint32_t)a << 32) | (uint32_t)b;
      }
      std::sort(keys.begin(), keys.end());
      if (std::adjacent_find(keys.begin(), keys.end()) != keys.end())
        fail(MPLD_E_INVALID, "component " + std::to_string(c) + " has a duplicate edge");
      pairs.resize(2 * keys.size());
      for (size_t e = 0; e < keys.size(); ++e) {
        pairs[2 * e] = (int32_t)(keys[e] >> 32);
        pairs[2 * e + 1] = (int32_t)(keys[e] & 0xffffffffu);
      }
      image_add(im, ctx, cp.n, pairs.data(), cp.m, opt->k, opt->node_budget, opt->flags);
    }
    image_finish(im);
    DeviceBatch db;
    struct GiveBack {   // before db's memory, also after an error: nothing on the stream uses either
      mpld_context* ctx;
      ~GiveBack() {
        (void)hipStreamSynchronize(ctx->stream);
        ctx->seq_done();
      }
    } give_back{ctx};
    device_upload(ctx, im, db);
    db.min_budget = min_budget_of(opt);
    device_solve(db, opt->flags | MPLD_DIRECT | MPLD_SPLIT_HEAVY);
    std::vector<DevRecord> recs;
    std::vector<int8_t> lcol;
    std::vector<int32_t> mins;
    device_fetch(db, recs, lcol, &mins);
    const bool trace = opt->flags & MPLD_TRACE_HASH;
    for (int32_t c = 0; c < count; ++c) {
      mpld_comp_record& r = out[c];
      r.size = comps[c].n;
      r.status = recs[c].status;
      r.nodes = (int64_t)recs[c].nodes;
      r.trace_hash = trace ? recs[c].hash : 0;
      r.depth_at_stop = recs[c].depth;
      r.stitches = r.status == MPLD_FEASIBLE || (opt->flags & (MPLD_MARK_CONFLICTS | MPLD_MINIMIZE))
                       ? 0 : -1;
      r.first_node = -1;
      r.num_edges = (int32_t)comps[c].m;
      r.conflicts = 0;
      r.min_nodes = (opt->flags & MPLD_MINIMIZE) ? mins[(size_t)c] : 0;
      const int8_t* cc = lcol.data() + im.desc[c].out_off;
      for (int64_t e = 0; e < comps[c].m; ++e) {
        const int8_t a = cc[comps[c].edges[2 * e]];
        r.conflicts += a >= 0 && a == cc[comps[c].edges[2 * e + 1]];
      }
    }
    if (!lcol.empty()) std::memcpy(colors_out, lcol.data(), lcol.size());
  });
}

const int8_t* mpld_result_colors(const mpld_result* r, int32_t* num_nodes) {
  if (!r) return nullptr;
  if (num_nodes) *num_nodes = (int32_t)r->colors.size();
  return r->colors.data();
}

const int32_t* mpld_result_component_of(const mpld_result* r) {
  return r ? r->comp_of.data() : nullptr;
}

int32_t mpld_result_num_components(const mpld_result* r) {
  return r ? (int32_t)r->comps.size() : 0;
}

const mpld_comp_record* mpld_result_components(const mpld_result* r) {
  return r ? r->comps.data() : nullptr;
}

void mpld_result_totals(const mpld_result* r, int64_t* stitches, int64_t* conflicts,
                        int64_t* uncolored) {
  if (!r) return;
  if (stitches) *stitches = r->stitches;
  if (conflicts) *conflicts = r->conflicts;
  if (uncolored) *uncolored = r->uncolored;
}

void mpld_result_timing(const mpld_result* r, double* queue_us, double* total_us) {
  if (!r) return;
  if (queue_us) *queue_us = r->queue_us;
  if (total_us) *total_us = r->total_us;
}

void mpld_result_free(mpld_result* r) { delete r; }

}  // extern "C"
