// The walk kernels' launches (walk_shape.hpp) under AddressSanitizer /
// UndefinedBehaviorSanitizer: every vector of every destination chunk, and every
// byte of every receive row, belongs to exactly one lane of one workgroup, over
// sizes on both sides of every rule; operations of several launches too.
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <vector>

#include "walk_shape.hpp"

using namespace pat;

static int failures = 0;
static long checked = 0;
#define EXPECT(cond)                                                                    \
  do {                                                                                  \
    if (!(cond)) {                                                                      \
      if (++failures < 20) std::fprintf(stderr, "%s:%d: expected %s\n", __FILE__, __LINE__, #cond); \
    }                                                                                   \
  } while (0)

// Every block of an operation once, over its launches; f(block) for each.
template <class F>
static void all_blocks(const Blocks& all, int threads, F f) {
  std::vector<bool> seen(all.count);
  each_launch(all, threads, [&](const Blocks& b, uint32_t grid) {
    EXPECT(grid > 0 && uint64_t(grid) * threads <= (uint64_t(1) << 31) + 8ull * all.grain * threads);
    EXPECT(b.first % (8 * b.grain) == 0 && b.count == all.count);
    for (uint32_t i = 0; i < grid; ++i) {
      const uint32_t blk = block_of(b, i);
      if (blk >= all.count) continue;
      EXPECT(!seen[blk]);
      seen[blk] = true;
      f(blk);
    }
  });
  for (uint32_t i = 0; i < all.count; ++i) EXPECT(seen[i]);
}

static void check_reduce(int N, int64_t count, int elem, const WalkRows& rows) {
  const int64_t V = (count + 3) / 4, back = V * 4 - count, chunk = count * elem;
  ReduceShape sh;
  EXPECT(reduce_shape(N, V, chunk, elem, rows, &sh));
  const int G = walk_group(elem, sh.S);
  // the parts cover the positions; a part's groups fit its slots, the parts the first group's five
  EXPECT(sh.S <= kWalkMostGroups && sh.threads == sh.lanes * sh.S && sh.lanes % 64 == 0);
  EXPECT(sh.threads <= (sh.S <= 4 ? 256 : 1024) && (sh.w & (sh.w - 1)) == 0);
  EXPECT(int64_t(sh.w) * sh.S >= N && (N + sh.w - 1) / sh.w <= sh.S);
  EXPECT((std::min(N, sh.w) + G - 1) / G <= 1 << (walk_slots(sh.S) - 1));
  // a key permutes the groups of whole, equal parts
  if (sh.keyed && sh.S > 1) EXPECT(N % sh.w == 0 && sh.w % G == 0);
  EXPECT(back < 4 && count >= 4);  // a partial vector's start is inside its chunk
  EXPECT(sh.uni || V < 8 * sh.lanes);
  std::vector<uint8_t> seen(size_t(N) * V);
  all_blocks(sh.blocks, sh.threads, [&](uint32_t blk) {
    for (int lane = 0; lane < sh.lanes; ++lane) {
      int R;
      int64_t v;
      if (!(sh.uni ? own_vector(blk, lane, sh.lanes, sh.tiles, V, &R, &v)
                   : shared_vector(blk, lane, sh.lanes, N, V, &R, &v)))
        continue;
      EXPECT(R >= 0 && R < N && v >= 0 && v < V);
      EXPECT(!seen[size_t(R) * V + v]++);
    }
  });
  for (uint8_t s : seen) EXPECT(s == 1);
  ++checked;
}

// Rows of `elem`-byte elements that start `at` bytes past a line, `stride` apart.
static void check_gather(int N, int64_t row_bytes, int64_t at, int64_t stride) {
  auto cover = [&](std::vector<uint8_t>& seen, int r, uint32_t tile, uint64_t align) {
    // the kernels' tiles start at the (first) receiver's line
    for (int lane = 0; lane < kGatherThreads; ++lane) {
      const int64_t o = int64_t(tile) * kGatherTile - int64_t(align) + lane * 16;
      for (int64_t i = std::max<int64_t>(o, 0); i < std::min(o + 16, row_bytes); i += 2)
        EXPECT(!seen[(size_t(r) * row_bytes + i) / 2]++);
    }
  };
  auto offset = [&](int r) { return uint64_t(at + r * stride) & 127; };
  GatherShape g;
  EXPECT(gather_shape(N, row_bytes, stride, &g));
  EXPECT(g.run >= 1 && g.run <= kGatherRun && g.period >= 1);
  std::vector<uint8_t> seen(size_t(N) * row_bytes / 2);  // per two bytes: every size and offset is even
  all_blocks(g.blocks, kGatherThreads, [&](uint32_t blk) {
    const uint32_t group = blk / g.tiles, tile = blk - group * g.tiles;  // as walk_ag_kernel takes them apart
    const int turn = (int)group / g.period, r0 = (int)group - turn * g.period + turn * g.run * g.period;
    EXPECT(tile < g.tiles && r0 >= 0);
    for (int k = 0, r = r0; k < g.run && r < N; ++k, r += g.period) cover(seen, r, tile, offset(r0));
  });
  for (uint8_t s : seen) EXPECT(s == 1);
  CopyShape c;
  EXPECT(copy_shape(N, row_bytes, &c));
  std::fill(seen.begin(), seen.end(), 0);
  all_blocks(c.blocks, kGatherThreads, [&](uint32_t blk) {
    uint32_t tile, r;
    copy_block(blk, c.panel, N, &tile, &r);
    EXPECT(r < (uint32_t)N);
    cover(seen, (int)r, tile, offset((int)r));
  });
  for (uint8_t s : seen) EXPECT(s == 1);
  ++checked;
}

int main() {
  auto at_stride = [](int64_t stride, bool aligned8 = true) {
    WalkRows w{};
    w.send_stride = stride;
    w.spaced = true;
    w.aligned8 = aligned8;
    return w;
  };
  std::srand(5);
  auto any = [](int64_t lo, int64_t hi) { return lo + std::rand() % (hi - lo + 1); };
  const int ns[] = {2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 127, 128, 129, 256, 257, 512, 513, 1000, 1024, 1025, 2048, 2049, 4096};
  const int64_t counts[] = {16, 17, 18, 19, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 4096, 8187, 8188, 9213, 16384, 70001};
  for (int n : ns)
    for (int64_t c : counts)
      for (int elem : {2, 4}) {
        if (int64_t(n) * c > 1 << 20) continue;
        check_reduce(n, c, elem, at_stride(n * c * elem));
        check_reduce(n, c, elem, at_stride(n * c * elem + elem, false));
        WalkRows table = at_stride(0);
        table.spaced = false;
        check_reduce(n, c, elem, table);
      }
  for (int k = 0; k < 400; ++k) {
    const int n = (int)any(2, k % 2 ? 4096 : 150), elem = k % 3 ? 4 : 2;
    const int64_t c = any(16, std::max<int64_t>(17, std::min<int64_t>((1 << 20) / n, 40000)));
    check_reduce(n, c, elem, at_stride(n * c * elem, c * elem % 8 == 0));
  }
  const int rn[] = {2, 3, 7, 13, 33, 64, 130, 300, 1025};
  const int64_t rb[] = {4, 30, 128, 4000, 4096, 4098, 8192, 12346, 65536, 1048576, 1052670, 2097152, 2097154, 2101250};
  for (int n : rn)
    for (int64_t b : rb)
      for (int64_t at : {0, 2, 96, 126}) {
        if (n * b > 5 << 20 || (n * b > 1 << 20 && at % 4)) continue;
        check_gather(n, b, at, b);
        check_gather(n, b, at, b + 2);
        check_gather(n, b, at, -b - 32);
      }
  // several launches: 2^31 lanes each, all but the last a multiple of the XCD runs
  for (uint32_t grain : {1u, 4u, 64u, 256u})
    for (int threads : {256, 1024})
      for (uint64_t count : {uint64_t(1) << 21, (uint64_t(1) << 23) + 5, (uint64_t(1) << 24) - 1, uint64_t(1) << 31}) {
        uint64_t next = 0;
        each_launch(Blocks{(uint32_t)count, grain, 0}, threads, [&](const Blocks& b, uint32_t grid) {
          EXPECT(b.first == next && grid % (8 * grain) == 0 && uint64_t(grid) * threads <= uint64_t(1) << 31);
          next += grid;
        });
        EXPECT(next >= count && next - count < 8 * grain);
        ++checked;
      }
  std::printf("%ld launches checked, %d failures\n", checked, failures);
  return failures != 0;
}
