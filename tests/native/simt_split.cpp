// The device's simplification and split on the CPU (simt/hip/hip_runtime.h),
// against the host's.
//   run SHAPE N K SIMPLIFY SEED HOLD LEVELS: the graph (see make); HOLD >= 0: one
//   workgroup of the giants' numbering sleeps before its HOLD-th atomic
//   operation; LEVELS: what the device may take, -1 by size.  A ninth word: the
//   launch of a split before it that fails.  Prints "same", "given up" or what differs.
#include <atomic>
#include <chrono>

#include "graph_device.hip"

namespace mpld {
void check_hip(hipError_t e, const char* what) {
  if (e) fail(MPLD_E_DEVICE, what);
}
}  // namespace mpld
void* mpld_context::dev_alloc(size_t bytes) { return std::aligned_alloc(256, (bytes + 255) & ~(size_t)255); }
void mpld_context::dev_free(void* p) { std::free(p); }

static std::atomic<int> g_atomics{0};
static int g_hold = -1;
static void slow_block(unsigned block, unsigned thread) {
  if (simt::grid_now != (unsigned)mpld::kGiantBlocks || block != 2 || thread != 0) return;
  if (g_atomics++ == g_hold) std::this_thread::sleep_for(std::chrono::milliseconds(400));
}

// line: node i and i + 1, i + 2; grid: a square lattice; strip: a lattice 4 wide;
// random: about 2.6 pairs a node.
static std::vector<int32_t> make(const std::string& shape, int32_t n, uint64_t seed) {
  std::mt19937_64 rng(seed);
  std::vector<int32_t> ids((size_t)n), e;
  for (int32_t i = 0; i < n; ++i) ids[(size_t)i] = i;
  if (seed) std::shuffle(ids.begin(), ids.end(), rng);
  const auto put = [&](int32_t a, int32_t b) {
    if (b >= n) return;
    e.push_back(ids[(size_t)a]);
    e.push_back(ids[(size_t)b]);
  };
  int32_t side = 4;
  if (shape == "grid")
    while (side * side < n) ++side;
  for (int32_t i = 0; i < n; ++i) {
    if (shape == "line") {
      put(i, i + 1);
      put(i, i + 2);
    } else if (shape == "grid" || shape == "strip") {
      if (i % side != side - 1) put(i, i + 1);
      put(i, i + side);
    } else if (i > 0) {
      int32_t had[3];
      const int m = 1 + (int)(rng() % 3) + (i % 5 == 0);
      for (int j = 0; j < std::min(m, 3); ++j) {
        had[j] = (int32_t)(rng() % (uint64_t)std::min(i, 40)) + std::max(0, i - 40);
        bool dup = false;
        for (int q = 0; q < j; ++q) dup |= had[q] == had[j];
        if (!dup) put(had[j], i);
      }
    }
  }
  return e;
}

int main(int argc, char** argv) {
  using namespace mpld;
  if (argc != 8 && argc != 9) return 2;
  const std::string shape = argv[1];
  const int32_t n = std::atoi(argv[2]), k = std::atoi(argv[3]);
  const bool simplify = std::atoi(argv[4]) != 0;
  const std::vector<int32_t> e = make(shape, n, std::strtoull(argv[5], nullptr, 10));
  g_hold = std::atoi(argv[6]);
  mpld_graph mg{};
  mg.num_nodes = n;
  mg.num_ce = (int64_t)e.size() / 2;
  mg.ce = e.data();
  const Graph g = make_graph(mg);
  const Split want = simplify_and_split(g, k, simplify);
  mpld_context ctx;
  ctx.split_levels = std::atoi(argv[7]);
  GraphBuilder gb;
  gb.ctx = &ctx;
  std::vector<int32_t> ptr(g.ptr.begin(), g.ptr.end()), out(split_out_words(n)), scratch(split_scratch_words(n) + 2);
  simt::concurrent = (unsigned)kGiantBlocks;
  simt::on_atomic = slow_block;
  // one of the split's launches has failed before
  if (argc == 9) {
    simt::fail_launch = std::atoi(argv[8]);
    try {
      enqueue_split(gb, n, ptr.data(), g.adj.data(), (int64_t)g.adj.size(), k, simplify, out.data(), scratch.data(),
                    nullptr, nullptr);
      return 2;
    } catch (const Error&) {
    }
  }
  enqueue_split(gb, n, ptr.data(), g.adj.data(), (int64_t)g.adj.size(), k, simplify, out.data(), scratch.data(),
                nullptr, nullptr);
  Split got;
  if (!collect_split(out.data(), n, got)) {
    std::puts("given up");
    return 0;
  }
  std::puts(got.removal != want.removal     ? "removal differs"
            : got.comp_of != want.comp_of   ? "components differ"
            : got.comp_ptr != want.comp_ptr ? "sizes differ"
            : got.order != want.order       ? "order differs"
            : got.local != want.local       ? "numbering differs"
                                            : "same");
  return 0;
}
