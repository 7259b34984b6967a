// The sequence engine's reservations on the CPU (simt/hip/hip_runtime.h): 32
// waves ask for tasks and arena until each has been refused 200 times; fails
// when a place is given twice or past the end, or when the counts go on.
#include <mutex>

#include "seq_reserve.h"

namespace mpld {
int mpld_writelane(int val, int lane, int old) { return (int)__lane_id() == (lane & 63) ? val : old; }
}  // namespace mpld

int main(int argc, char** argv) {
  using namespace mpld;
  if (argc != 4) return 2;
  simt::seed = std::strtoull(argv[3], nullptr, 10);
  simt::concurrent = 8;
  simt::hold = 3;
  SeqHead head{};
  SeqArgs a{};
  a.head = &head;
  a.task_cap = std::atoi(argv[1]);
  a.arena_cap = std::atoi(argv[2]);
  std::vector<int> task((size_t)a.task_cap, 0), unit((size_t)a.arena_cap / 64, 0);
  std::mutex mu;
  int bad = 0;
  simt::launch(dim3(8), dim3(256), [&] {
    std::mt19937 rng((unsigned)(simt::seed * 4099 + blockIdx.x * 4 + (threadIdx.x >> 6)));   // alike in a wave
    for (int refused = 0; refused < 200;) {
      const int pieces = (int)(rng() % 25);
      const uint64_t bytes = 64 * (1 + rng() % 40);
      int32_t child;
      int64_t at;
      const bool got = seq_take_room(a, bytes, pieces, child, at);
      refused += got ? 0 : 1;
      if (!got || (threadIdx.x & 63) != 0) continue;
      std::lock_guard<std::mutex> lk(mu);
      bad |= at < 0 || at + (int64_t)bytes > a.arena_cap || (pieces && (child < 0 || child + pieces > a.task_cap));
      for (uint64_t b = 0; !bad && b < bytes / 64; ++b) bad |= ++unit[(size_t)at / 64 + b] > 1;
      for (int i = 0; !bad && i < pieces; ++i) bad |= ++task[(size_t)(child + i)] > 1;
    }
  });
  bad |= head.tasks > a.task_cap + 32 * 24 || head.arena > (uint64_t)a.arena_cap + 32 * 64 * 40;
  std::printf("%d tasks, %llu bytes\n", head.tasks, head.arena);
  return bad;
}
