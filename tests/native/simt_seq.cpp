// The sequence engine's host side and list kernel on the CPU
// (simt/hip/hip_runtime.h), with stand-ins for the searches: every task is
// exhausted after one node.  The device memory comes from a pool of a limited
// size, and launches are on the way until the stream is waited for.
//   run CAP: solves components of growing workspaces, each with the register
//   tier's and then the CSR tiers', from a pool of CAP MiB.  Prints how many
//   solves there was memory for; fails when memory goes back or is handed out
//   while launches that use it are on the way, or when any is lost.
#include "seq_engine.hip"

static size_t g_cap = 0, g_used = 0;
static int g_pending = 0;      // launches on the way
static int g_bad = 0;
static std::vector<std::pair<void*, size_t>> g_live;

namespace mpld {
void fail(int32_t code, const std::string& what) { throw Error{code, what}; }
void check_hip(hipError_t e, const char* what) {
  if (e) fail(MPLD_E_DEVICE, what);
}
DeviceBatch::~DeviceBatch() {}

// What the searches' launches leave: every listed task has counted one node.
static void exhaust(const SeqArgs& a, int32_t tier, int32_t parity) {
  ++g_pending;
  const int32_t* list = a.runs + (int64_t)(parity * kSeqTiers + tier) * a.run_cap;
  for (int32_t i = 0; i < a.head->run[parity][tier]; ++i) {
    SeqResult& r = a.results[list[i] & kSeqTaskMask];
    r = SeqResult{};
    r.status = MPLD_INFEASIBLE;
    r.nodes = 1;
    r.sol = -1;
  }
}
static void finish_all(const SeqArgs& a, DevRecord* recs, int32_t tier) {
  ++g_pending;
  for (int32_t i = 0; i < a.ncomps; ++i)
    if (a.comps[i].tier == tier) {
      g_bad |= a.comps[i].running || a.comps[i].acc != 1;
      recs[a.comps[i].pos].status = a.comps[i].status;
    }
}
hipError_t launch_seq_reg(bool, int, int, const SeqArgs& a, RegItems, int32_t parity, bool finish, DevRecord* recs,
                          int8_t*, hipStream_t) {
  if (finish) finish_all(a, recs, kSeqReg);
  else exhaust(a, kSeqReg, parity);
  return hipSuccess;
}
hipError_t launch_seq_csr(bool, int, int, int, const SeqArgs& a, const DevDesc*, const uint32_t*, uint64_t*, uint64_t,
                          int32_t parity, bool finish, DevRecord* recs, int8_t*, hipStream_t) {
  if (finish) finish_all(a, recs, kSeqCsr);
  else exhaust(a, kSeqCsr, parity);
  return hipSuccess;
}
}  // namespace mpld

int main(int argc, char** argv) {
  using namespace mpld;
  if (argc != 2) return 2;
  g_cap = (size_t)std::atoi(argv[1]) << 20;
  simt::on_sync = [] { g_pending = 0; };
  mpld_context ctx;
  ctx.num_cus = 256;
  ctx.has_alloc = true;
  ctx.alloc.alloc = [](size_t n, void*) -> void* {
    if (g_used + n > g_cap) return nullptr;
    g_used += n;
    g_live.emplace_back(std::aligned_alloc(256, (n + 255) & ~(size_t)255), n);
    std::memset(g_live.back().first, 0xa5, std::min<size_t>(n, 16 << 20));
    return g_live.back().first;
  };
  ctx.alloc.free = [](void* p, void*) {
    g_bad |= g_pending != 0;
    for (auto& b : g_live)
      if (b.first == p) {
        g_used -= b.second;
        std::free(p);
        b = g_live.back();
        g_live.pop_back();
        return;
      }
    g_bad = 1;
  };
  int solved = 0;
  for (int32_t count : {1, 3, 9, 24}) {
    DeviceBatch db;
    db.ctx = &ctx;
    db.k = 3;
    db.n_reg = count;
    db.n_lds = count;
    std::vector<DevDesc> desc;
    for (int32_t i = 0; i < 2 * count; ++i) {
      DevDesc d{};
      d.n = i < count ? 60 : 2000;
      d.k = 3;
      d.budget = 100000;
      d.comp = i;
      desc.push_back(d);
    }
    db.host_desc = desc;
    db.csr_shape.resize((size_t)count);
    for (CsrShape& s : db.csr_shape) s = CsrShape{40000, 20000, 9000};
    std::vector<DevRecord> recs(desc.size());
    DevBuf d, r;
    d.p = desc.data();
    r.p = recs.data();
    db.desc.view(d, 0, sizeof(DevDesc) * desc.size());
    db.recs.view(r, 0, sizeof(DevRecord) * recs.size());
    std::vector<int32_t> reg, csr;
    for (int32_t i = 0; i < count; ++i) {
      reg.push_back(i);
      csr.push_back(count + i);
    }
    // the register tier's last launches are still on the way when the other
    // tiers ask for more
    solved += seq_solve(db, reg, false) ? 1 : 0;
    solved += seq_solve(db, csr, false) ? 1 : 0;
    // few components: room for what the device's 2,048 places cut in a round or
    // two (66 KB a cut of 2,000 nodes), not for the budgets' share alone
    if (count == 3 && g_cap > (1ull << 30)) g_bad |= ctx.seq_bytes < (2ull * 2048 * 60000);
    if (solved == 8)
      for (const DevRecord& x : recs) g_bad |= x.status != MPLD_INFEASIBLE;
  }
  // memory that something else needs is given back by the workspace
  if (ctx.seq_bytes) {
    const size_t most = g_cap - 4096;
    ctx.dev_free(ctx.dev_alloc(most));
    g_bad |= ctx.seq_bytes != 0;
  }
  ctx.seq_give_back();
  g_bad |= g_used != 0;
  std::printf("%d\n", solved);
  return g_bad;
}
