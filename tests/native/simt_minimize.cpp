// The Eq. 1 minimisation kernels on the CPU (simt/hip/hip_runtime.h).
//   run ids N SEED: eight waves take pieces' ids off a stack of N until each
//   has been refused four times; fails when an id is taken twice or the stack
//   does not hold what is left.
//   run: reads components, writes each one's node count and colors;
//   input:  K budget seed count, then per component: n, its n masks, n
//           partners (255 none), n incumbent colors
#include <cinttypes>

#include "search_min.hip"

namespace mpld {
int mpld_writelane(int val, int lane, int old) { return (int)__lane_id() == (lane & 63) ? val : old; }
}  // namespace mpld

static int take_ids(int count, uint64_t seed) {
  int bad = 0;
  for (uint64_t s = 0; s < 200 && !bad; ++s) {
    simt::seed = seed * 1000 + s;
    simt::hold = 1 + s % 5;
    int32_t spare = count;
    std::vector<int> taken((size_t)count, 0);
    simt::launch(dim3(1), dim3(64 * 8), [&] {
      std::mt19937 rng((unsigned)(simt::seed * 64 + threadIdx.x));
      if ((threadIdx.x & 63) != 0) return;
      for (int refused = 0; refused < 4;) {
        const int want = 1 + (int)(rng() % 8);
        const int32_t at = mpld::min_take(&spare, want);
        if (at < 0) ++refused;
        for (int i = 0; at >= 0 && i < want; ++i) bad |= at + i >= count || ++taken[(size_t)(at + i)] > 1;
      }
    });
    for (int i = 0; i < count; ++i) bad |= taken[(size_t)i] != (i >= spare ? 1 : 0);
  }
  return bad;
}

int main(int argc, char** argv) {
  using namespace mpld;
  if (argc == 4 && !std::strcmp(argv[1], "ids")) return take_ids(std::atoi(argv[2]), std::strtoull(argv[3], nullptr, 10));
  int k = 0, count = 0;
  unsigned budget = 0;
  if (std::scanf("%d %u %" SCNu64 " %d", &k, &budget, &simt::seed, &count) != 4) return 2;
  simt::hold = 1500;
  struct Comp { int n; std::vector<uint64_t> nb; std::vector<int> part, col; };
  std::vector<Comp> comps((size_t)count);
  int width = 1, total = 0;
  for (Comp& c : comps) {
    if (std::scanf("%d", &c.n) != 1) return 2;
    c.nb.resize((size_t)c.n);
    c.part.resize((size_t)c.n);
    c.col.resize((size_t)c.n);
    for (auto& x : c.nb) if (std::scanf("%" SCNu64, &x) != 1) return 2;
    for (int& x : c.part) if (std::scanf("%d", &x) != 1) return 2;
    for (int& x : c.col) if (std::scanf("%d", &x) != 1) return 2;
    width = std::max(width, c.n);
    total += c.n;
  }
  const uint32_t stride = kRegItemHead + 8u * (uint32_t)width;
  std::vector<uint64_t> items((size_t)stride / 8 * comps.size(), 0);
  std::vector<uint8_t> part((size_t)total);
  std::vector<int8_t> colors((size_t)total);
  int at = 0;
  for (size_t i = 0; i < comps.size(); ++i) {
    const Comp& c = comps[i];
    auto* it = reinterpret_cast<uint8_t*>(items.data()) + stride * i;
    DevDesc d{};
    d.n = c.n;
    d.k = k;
    d.nbr_off = d.out_off = at;
    d.comp = (int32_t)i;
    std::memcpy(it, &d, sizeof(d));
    std::memcpy(it + kRegItemHead, c.nb.data(), 8 * c.nb.size());
    for (int v = 0; v < c.n; ++v) {
      part[(size_t)(at + v)] = (uint8_t)c.part[(size_t)v];
      colors[(size_t)(at + v)] = (int8_t)c.col[(size_t)v];
    }
    at += c.n;
  }
  std::vector<int32_t> out(comps.size(), 0), list(comps.size(), -1);
  int32_t len[2] = {0, 0};
  const RegItems ri{reinterpret_cast<const uint8_t*>(items.data()), (uint32_t)width, stride, 0u};
  if (launch_min_reg(k, count, count, ri, count, part.data(), colors.data(), out.data(), budget, len, list.data(),
                     nullptr) != hipSuccess)
    return 2;
  if (len[0] || len[1]) return 2;   // left empty for the next call
  at = 0;
  for (size_t i = 0; i < comps.size(); ++i) {
    std::printf("%d", out[i]);
    for (int v = 0; v < comps[i].n; ++v) std::printf(" %d", colors[(size_t)at++]);
    std::printf("\n");
  }
  return 0;
}
