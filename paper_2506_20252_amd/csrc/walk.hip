// Walk kernels for gfx950 (CDNA4): a whole operation as one launch, every
// tree walked in its linear order with the intermediate buffers in registers.
//
// The step kernels run the schedule one step of all trees at a time, and a
// partial or a forwarded chunk goes through memory between two steps: about
// three transfers of a chunk per edge, where each input has to be read only
// once.  The far-first linear walk of one tree (section "The PAT algorithm")
// needs one chunk of intermediate buffer per distance, ceil(log2 N) in all;
// over one 4-element vector of the chunk that is a few registers, so a lane can
// walk its vector's whole tree by itself.
//
// Reduce-scatter: lane (R, v) owns vector v of destination chunk R.  It reads
// the tree's positions q = 0 .. N - 1 (rank R + q) in order and adds them as
// the reversed binomial tree does: the partial S(lo, w) of the sub-tree that
// starts at position lo and spans w positions is S(lo, w/2), or, where
// position lo + w/2 exists, S(lo, w/2) + S(lo + w/2, w/2) -- the order in
// which the schedule adds children, nearest first, whatever the number of
// parallel sub-trees, pieces or chunks per step.

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstring>
#include <type_traits>

#include "device_access.hpp"
#include "walk.hpp"
#include "walk_shape.hpp"

namespace pat {
namespace {

// How a kernel finds rank r's buffers: at base + r * stride (SPACED kernels),
// else in a pointer table, which is in device memory or comes with the launch
// (RowPointers, read from the kernel-argument segment).
struct RowsArg {
  uint64_t send0, recv0;
  int64_t send_stride, recv_stride;
  uint64_t send_table, recv_table;  // 0: RowPointers
};
struct RowPointers {
  uint64_t send[kWalkInlineRanks], recv[kWalkInlineRanks];
};

// Pointer tables do not change during a launch: constant memory, which scalar
// loads serve where the rank is uniform.
#define PAT_CONSTANT __attribute__((address_space(4)))
typedef const PAT_CONSTANT uint64_t* RowTable;

// A kernel's one argument: the pointers' place in the argument segment is
// then known.
template <class Ctx, bool SPACED>
struct WalkArgs {
  Ctx cx;
};
template <class Ctx>
struct WalkArgs<Ctx, false> {
  Ctx cx;
  RowPointers ptrs;
};

template <class Ctx>
__device__ __forceinline__ RowTable row_table(uint64_t table, size_t member) {
  using IndexedArgs = WalkArgs<Ctx, false>;
  if (table) return (RowTable)table;
  return (RowTable)((const PAT_CONSTANT char*)__builtin_amdgcn_kernarg_segment_ptr() +
                    offsetof(IndexedArgs, ptrs) + member);
}
template <bool SPACED, class Ctx>
__device__ __forceinline__ const char* send_row(const Ctx& cx, int r) {
  if constexpr (SPACED) return (const char*)(cx.rows.send0 + (uint64_t)(r * cx.rows.send_stride));
  return (const char*)row_table<Ctx>(cx.rows.send_table, offsetof(RowPointers, send))[r];
}
template <bool SPACED, class Ctx>
__device__ __forceinline__ char* recv_row(const Ctx& cx, int r) {
  if constexpr (SPACED) return (char*)(cx.rows.recv0 + (uint64_t)(r * cx.rows.recv_stride));
  return (char*)row_table<Ctx>(cx.rows.recv_table, offsetof(RowPointers, recv))[r];
}

// Launches the blocks of cx, in as many launches as it takes.
template <class Arg, class Ctx>
void launch_blocks(void (*kernel)(Arg), int threads, Arg& arg, Ctx& cx, hipStream_t stream) {
  each_launch(cx.blocks, threads, [&](const Blocks& b, uint32_t grid) {
    cx.blocks = b;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, stream, arg);
  });
}

template <class Ctx, bool SPACED>
void launch_kernel(void (*kernel)(WalkArgs<Ctx, SPACED>), int threads, const Ctx& cx, const WalkRows& rows,
                   hipStream_t stream) {
  WalkArgs<Ctx, SPACED> a;
  a.cx = cx;
  if constexpr (!SPACED) {
    if (!rows.table) {
      std::memcpy(a.ptrs.send, rows.send, cx.N * sizeof(void*));
      std::memcpy(a.ptrs.recv, rows.recv, cx.N * sizeof(void*));
    }
  }
  launch_blocks(kernel, threads, a, a.cx, stream);
}

// What a kernel's context says about `rows` (device tables: kx's).
RowsArg rows_arg(const KCtx& kx, const WalkRows& rows) {
  return RowsArg{(uint64_t)rows.send[0], (uint64_t)rows.recv[0], rows.send_stride, rows.recv_stride,
                 rows.table ? (uint64_t)kx.send : 0, rows.table ? (uint64_t)kx.recv : 0};
}

struct WalkCtx {
  RowsArg rows;
  int64_t chunk_bytes;      // of a user chunk
  int64_t V;                // 4-element vectors per chunk, a partial last one among them
  int32_t N;
  int32_t back;             // a partial last vector begins this many elements inside the one before (0: none)
  int32_t w;                // positions per lane group, a power of two
  int32_t lanes;            // vectors per workgroup, a multiple of 64
  uint32_t tiles;           // workgroups per chunk (a workgroup's vectors in one chunk)
  Blocks blocks;
};

// A chunk's vectors are read at element alignment (see Access); the last one
// may be moved back to end where the chunk ends.
struct WI32 {
  using in_t = v4u;
  static constexpr int kElem = 4;
  struct acc_t {
    v4u a;
  };
  __device__ static acc_t widen(const in_t& x) { return {x}; }
  __device__ static in_t narrow(const acc_t& x) { return x.a; }
  __device__ static acc_t add(const acc_t& x, const acc_t& y) { return {x.a + y.a}; }  // wraps
};

struct WF32 {
  using in_t = v4f;
  static constexpr int kElem = 4;
  struct acc_t {
    v4f a;
  };
  __device__ static acc_t widen(const in_t& x) { return {x}; }
  __device__ static in_t narrow(const acc_t& x) { return x.a; }
  __device__ static acc_t add(const acc_t& x, const acc_t& y) { return {x.a + y.a}; }
};

// 8-byte vectors: 4 float32 partials per slot, as for float32, leave 64 VGPRs
// and 8 waves per SIMD, where 16-byte vectors take 108 and 4 (measured on
// MI355X, 16-byte / 8-byte: N=128 4 MiB 12.3 / 11.0 ms, N=64 2 MiB 1568 / 1402
// us, N=24 64 KiB 10.0 / 8.4 us).
struct WB16 {
  using in_t = v2u;  // 4 bf16, element 2j in the low half of word j
  static constexpr int kElem = 2;
  struct acc_t {
    v4f a;
  };
  __device__ static acc_t widen(const in_t& x) {
    return {v4f{bf16_lo(x.x), bf16_hi(x.x), bf16_lo(x.y), bf16_hi(x.y)}};
  }
  __device__ static in_t narrow(const acc_t& x) {
    return v2u{bf16_rne(x.a.x) | (bf16_rne(x.a.y) << 16), bf16_rne(x.a.z) | (bf16_rne(x.a.w) << 16)};
  }
  __device__ static acc_t add(const acc_t& x, const acc_t& y) { return {x.a + y.a}; }
};

// Partials of complete sub-trees, one per distance, like the schedule's slots:
// entry l holds a sub-tree of 2^l leaves (a leaf being whatever push() is
// given).  Every index is a compile-time constant and every branch uniform,
// so the entries stay in registers.
template <class T, int LV>
struct WalkSlots {
  typename T::acc_t st[LV];

  // Leaf number b (0, 1, ...): merges with the sub-trees it completes.  With a
  // key, the leaves come in the order b ^ key, which fills the same sub-trees,
  // a level's right one first where the key has its bit.
  template <int L = 0>
  __device__ __forceinline__ void push(int b, const typename T::acc_t& x, int key = 0) {
    if constexpr (L < LV) {
      if ((b >> L) & 1)
        push<L + 1>(b, (key >> L) & 1 ? T::add(x, st[L]) : T::add(st[L], x), key);
      else
        st[L] = x;
    }
  }

  // The tree of nb >= 1 leaves: the truncated tree's complete sub-trees, the
  // smallest (last) first.
  template <int L = 0>
  __device__ __forceinline__ typename T::acc_t total(int nb, typename T::acc_t x = {}, bool any = false) const {
    if constexpr (L < LV) {
      if ((nb >> L) & 1) {
        x = any ? T::add(st[L], x) : st[L];
        any = true;
      }
      return total<L + 1>(nb, x, any);
    } else {
      return x;
    }
  }
};

// Tree sum of the group's first m leaves (1 <= m <= G).
template <class T, int G>
__device__ __forceinline__ typename T::acc_t group_sum(const typename T::in_t (&x)[G], int m) {
  typename T::acc_t a[G];
  if (m == G) {
#pragma unroll
    for (int j = 0; j < G; ++j) a[j] = T::widen(x[j]);
#pragma unroll
    for (int d = 1; d < G; d *= 2)
#pragma unroll
      for (int j = 0; j < G; j += 2 * d) a[j] = T::add(a[j], a[j + d]);
  } else {
#pragma unroll
    for (int j = 0; j < G; ++j)
      if (j < m) a[j] = T::widen(x[j]);
#pragma unroll
    for (int d = 1; d < G; d *= 2)
#pragma unroll
      for (int j = 0; j < G; j += 2 * d)
        if (j + d < m) a[j] = T::add(a[j], a[j + d]);
  }
  return a[0];
}

// Reduce-scatter.  A workgroup owns `lanes` vectors, blockDim / lanes = S
// lane groups to each: group s walks positions [s w, (s + 1) w), the sub-tree
// of span w (a power of two) that starts there, and the first group adds the S
// partials by the same rule through LDS.  `lanes` is a multiple of 64, so a
// wave's lanes share s and every loop below is uniform.  UNI: a workgroup's
// vectors belong to one chunk, whose senders' addresses are then scalar; else
// they are consecutive vectors of consecutive chunks.
//
// A lane reads G positions at a time and asks for the next G before it adds.
// Where those loads have a condition (a last group may be partial) the compiler
// waits for all in flight before it adds: other waves, not the lane's own next
// loads, cover most of the latency.  The bound of a large operation is HBM's
// read rate.  Measured on MI355X, step schedule -> walk: N=64 float32 1 MiB 1992 -> 650 us, N=128 bf16 4 MiB 52.6 -> 10.8 ms
// (6.6 and 6.4 TB/s of input), N=1000 float32 256 B 139 -> 42 us a call.
//
// KEYED (power-of-two parts only): a workgroup reads its groups of positions in
// the order g ^ key, a key of its own.  See walk_keyed().
template <class T, int G, int MAXT, int LV, bool SPLIT, bool UNI, bool SPACED, bool KEYED, bool NT>
__global__ __launch_bounds__(MAXT) void walk_rs_kernel(WalkArgs<WalkCtx, SPACED> args) {
  const WalkCtx& cx = args.cx;
  using in_t = typename T::in_t;
  using acc_t = typename T::acc_t;
  const int N = cx.N;
  const int lanes = SPLIT ? cx.lanes : MAXT;
  int s = 0, lane = threadIdx.x;
  if constexpr (SPLIT) {
    s = __builtin_amdgcn_readfirstlane(threadIdx.x / lanes);
    lane = threadIdx.x - s * lanes;
  }
  const uint32_t blk = block_of(cx.blocks, blockIdx.x);
  if (blk >= cx.blocks.count) return;
  int R;
  int64_t v;
  const bool live = UNI ? own_vector(blk, lane, lanes, cx.tiles, cx.V, &R, &v)
                        : shared_vector(blk, lane, lanes, cx.N, cx.V, &R, &v);
  const bool part = cx.back && v == cx.V - 1;
  const int64_t voff = v * (int64_t)sizeof(in_t) - (part ? cx.back * T::kElem : 0);
  const int64_t soff = (int64_t)R * cx.chunk_bytes + voff;

  acc_t sum;
  const int p0 = SPLIT ? s * cx.w : 0;
  const int n = SPLIT && N - p0 > cx.w ? cx.w : N - p0;  // positions of this lane group
  if (live && n > 0) {
    // The send buffer of position q (rank R + q, mod N).
    const char* const row0 = SPACED ? send_row<SPACED>(cx, R) : nullptr;
    auto row = [&](int q) -> const char* {
      if constexpr (SPACED) return row0 + (R >= N - q ? (q - N) * cx.rows.send_stride : q * cx.rows.send_stride);
      return send_row<SPACED>(cx, wrap_add(R, q, N));
    };
    auto load = [&](in_t(&x)[G], int q, int m) {
      const char* p[G];
#pragma unroll
      for (int j = 0; j < G; ++j)
        if (j < m) p[j] = row(p0 + q + j);
#pragma unroll
      for (int j = 0; j < G; ++j)
        if (j < m) x[j] = ldg<in_t, NT, T::kElem>(p[j] + soff);
    };
    const int groups = (n + G - 1) / G;
    auto size = [&](int g) { return n - g * G < G ? n - g * G : G; };
    WalkSlots<T, LV> slots;
    in_t x[G], y[G];
    if constexpr (!SPACED && !UNI) {
      // Every lane looks its own rank up in the pointer table, a load that the
      // data load waits for.  So the addresses come two groups ahead of their
      // data, and each load is issued before an older one is waited for: the
      // loop's loads have no condition (it runs while two more whole groups
      // follow), since over one that may not have been issued the compiler
      // waits for all in flight.  Measured on MI355X, float32 rows in
      // shuffled order, address and data in turn / ahead (step schedule):
      // N=1025 96 B 108 / 52 us (63), N=513 512 B 98 / 40 us (66), N=2049 64 B
      // 213 / 99 us (159).
      const char *t[G], *u[G];
      auto find = [&](const char*(&p)[G], int g) {
#pragma unroll
        for (int j = 0; j < G; ++j) p[j] = row(p0 + min(g * G + j, n - 1));
      };
      auto read = [&](in_t(&x)[G], const char* const(&p)[G]) {
#pragma unroll
        for (int j = 0; j < G; ++j) x[j] = ldg<in_t, NT, T::kElem>(p[j] + soff);
      };
      find(t, 0);
      find(u, 1);
      read(x, t);
      int g = 0;
      for (; g + 3 < groups; g += 2) {
        find(t, g + 2);
        read(y, u);
        slots.push(g, group_sum<T, G>(x, G));
        find(u, g + 3);
        read(x, t);
        slots.push(g + 1, group_sum<T, G>(y, G));
      }
      const bool two = g + 1 < groups, three = g + 2 < groups;
      if (three) find(t, g + 2);
      if (two) read(y, u);
      slots.push(g, group_sum<T, G>(x, size(g)));
      if (three) read(x, t);
      if (two) slots.push(g + 1, group_sum<T, G>(y, size(g + 1)));
      if (three) slots.push(g + 2, group_sum<T, G>(x, size(g + 2)));
    } else {
      const int key = KEYED ? (int)(blk * 2654435761u >> 24) & (groups - 1) : 0;
      load(x, key * G, size(key));
      for (int g = 0; g < groups; g += 2) {
        const bool two = g + 1 < groups;
        if (two) load(y, ((g + 1) ^ key) * G, size((g + 1) ^ key));
        slots.push(g, group_sum<T, G>(x, size(g ^ key)), key);
        if (two) {
          if (g + 2 < groups) load(x, ((g + 2) ^ key) * G, size((g + 2) ^ key));
          slots.push(g + 1, group_sum<T, G>(y, size((g + 1) ^ key)), key);
        }
      }
    }
    sum = slots.total(groups);
  }
  if constexpr (SPLIT) {
    __shared__ acc_t partial[MAXT];
    if (live && n > 0) partial[threadIdx.x] = sum;
    __syncthreads();
    if (s > 0 || !live) return;
    const int parts = (N + cx.w - 1) / cx.w;
    WalkSlots<T, 5> top;  // at most 16 partials
    top.push(0, sum);
    for (int u = 1; u < parts; ++u) top.push(u, partial[u * lanes + lane]);
    sum = top.total(parts);
  } else {
    if (!live) return;
  }
  const in_t out = T::narrow(sum);
  char* const dst = recv_row<SPACED>(cx, R) + voff;
  if (part)
    stg_from<NT, T::kElem>(dst, out, cx.back);
  else
    stg<NT, T::kElem>(dst, out);
}

template <class T, int G, int MAXT, int LV, bool SPLIT, bool NT>
void launch_walk_rs_k(const WalkCtx& cx, const WalkRows& rows, bool uni, bool keyed, int threads, hipStream_t stream) {
  if constexpr (SPLIT && T::kElem == 4) {
    if (keyed && uni)
      return launch_kernel(walk_rs_kernel<T, G, MAXT, LV, true, true, true, true, NT>, threads, cx, rows, stream);
    if (keyed)
      return launch_kernel(walk_rs_kernel<T, G, MAXT, LV, true, false, true, true, NT>, threads, cx, rows, stream);
  }
  if (rows.spaced && uni)
    launch_kernel(walk_rs_kernel<T, G, MAXT, LV, SPLIT, true, true, false, NT>, threads, cx, rows, stream);
  else if (rows.spaced)
    launch_kernel(walk_rs_kernel<T, G, MAXT, LV, SPLIT, false, true, false, NT>, threads, cx, rows, stream);
  else if (uni)
    launch_kernel(walk_rs_kernel<T, G, MAXT, LV, SPLIT, true, false, false, NT>, threads, cx, rows, stream);
  else
    launch_kernel(walk_rs_kernel<T, G, MAXT, LV, SPLIT, false, false, false, NT>, threads, cx, rows, stream);
}

template <class T, bool NT>
hipError_t launch_walk_rs_t(WalkCtx cx, const WalkRows& rows, hipStream_t stream) {
  ReduceShape sh;
  if (!reduce_shape(cx.N, cx.V, cx.chunk_bytes, T::kElem, rows, &sh)) return hipErrorInvalidValue;
  const int S = sh.S, threads = sh.threads;
  const bool uni = sh.uni, keyed = sh.keyed;
  cx.lanes = sh.lanes;
  cx.w = sh.w;
  cx.tiles = sh.tiles;
  cx.blocks = sh.blocks;
  if (S == 1)
    launch_walk_rs_k<T, walk_group(T::kElem, 1), 256, walk_slots(1), false, NT>(cx, rows, uni, keyed, threads, stream);
  else if (S <= 4)
    launch_walk_rs_k<T, walk_group(T::kElem, 4), 256, walk_slots(4), true, NT>(cx, rows, uni, keyed, threads, stream);
  else
    launch_walk_rs_k<T, walk_group(T::kElem, 16), 1024, walk_slots(16), true, NT>(cx, rows, uni, keyed, threads, stream);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// All-gather
// ---------------------------------------------------------------------------

// Every receive row is the same concatenation of the N chunks, and every node
// of a chunk's tree forwards the bytes it received: a workgroup takes 256
// 16-byte vectors of the concatenation (a tile) and a few receivers, reads the
// tile once, into registers, and stores it to each receiver in turn.
struct GatherCtx {
  RowsArg rows;
  int64_t chunk_bytes;
  int64_t row_bytes;        // N * chunk_bytes
  int32_t N;
  int32_t period;           // rows r and r + period start at the same offset from a 128-byte line
  int32_t run;              // receivers per workgroup, `period` apart
  uint32_t tiles;           // tiles per row
  Blocks blocks;
};

// The bound is HBM's write rate.  A tile's vectors start where the
// workgroup's first receiver has a 128-byte line, so that its stores write
// whole lines also where rows start in the middle of one (then the first tile
// begins before the row): N=1000 ranks of 63 float32, rows 96 bytes past the
// line before's end, 39 us against 56 us with every tile at a multiple of 4096
// bytes from its row's start.  Vectors that hold bytes of several chunks, and
// the row's ends, are read and where necessary stored element by element.
// ES: bytes per element.
// Measured on MI355X, step schedule -> walk, a call, in place: N=128 float32 1
// MiB 6982 -> 2762 us, N=1000 float32 252 B 134 -> 39 us, N=13 bf16 2002 B 11.6 ->
// 4.5 us; rows in shuffled order: 7149 -> 2818, 137 -> 58, 11.5 -> 4.4 us.  (The
// timings above and at the launch are of one tensor's rows through this kernel,
// which have one of their own below, where they do not say in place.)
template <int ES, bool SPACED>
__global__ __launch_bounds__(kGatherThreads) void walk_ag_kernel(WalkArgs<GatherCtx, SPACED> args) {
  const GatherCtx& cx = args.cx;
  constexpr int kElems = 16 / ES;
  using elem_t = typename std::conditional<ES == 4, uint32_t, uint16_t>::type;
  const uint32_t blk = block_of(cx.blocks, blockIdx.x);
  if (blk >= cx.blocks.count) return;
  const uint32_t g = blk / cx.tiles, tile = blk - g * cx.tiles;
  // receivers r0, r0 + period, ...: `run` of them
  const int turn = (int)g / cx.period, r0 = (int)g - turn * cx.period + turn * cx.run * cx.period;
  if (r0 >= cx.N) return;
  const int64_t C = cx.chunk_bytes;
  const int64_t tile0 = (int64_t)tile * kGatherTile - (int64_t)((uintptr_t)recv_row<SPACED>(cx, r0) & 127);  // may be negative
  if (tile0 >= cx.row_bytes) return;
  const int64_t start = tile0 > 0 ? tile0 : 0;
  const int x0 = cx.row_bytes < (int64_t(1) << 32) ? (int)((uint32_t)start / (uint32_t)C) : (int)(start / C);

  const int off = (int)threadIdx.x * 16;
  const int64_t o = tile0 + off;               // first byte in the row
  const int64_t left = cx.row_bytes - o;
  const int lo = o < 0 ? (o > -16 ? (int)-o : 16) : 0;  // bytes [lo, hi) are the row's
  const int hi = left < 16 ? (int)left : 16;
  const int64_t t = tile0 - x0 * C + off;      // first byte from chunk x0's start; negative before the row
  const int q = C >= kGatherTile ? (t >= C ? 1 : 0) : t > 0 ? (int)((uint32_t)t / (uint32_t)C) : 0;
  const int first = x0 + q;                    // chunks the vector holds bytes of
  const int64_t at = t - q * C;                // its first byte in chunk `first`
  const bool whole = lo == 0 && hi == 16;
  int last = first;
  v4u val = {};
  if (whole && at + 16 <= C) {
    val = ldg<v4u, false, ES>(send_row<SPACED>(cx, first) + at);
  } else if (lo < hi) {
    int64_t i = at;
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < kElems; ++e) {
      if (e * ES >= lo && e * ES < hi) {
        if (i >= C) i -= C, ++last;
        const uint32_t b = ldg<elem_t, false>(send_row<SPACED>(cx, last) + i);
        w[e * ES / 4] |= b << (e * ES % 4 * 8);
      }
      i += ES;
    }
    val = v4u{w[0], w[1], w[2], w[3]};
  }
  for (int k = 0, r = r0; k < cx.run && r < cx.N; ++k, r += cx.period) {
    char* const row = recv_row<SPACED>(cx, r);
    const bool inplace = send_row<SPACED>(cx, r) == row + r * C;  // rank r's chunk is there already
    char* const dst = row + tile0 + off;
    if (whole && !(inplace && first <= r && r <= last)) {
      stg<true, ES>(dst, val);
    } else if (lo < hi) {
      int x = first;
      int64_t i = at;
#pragma unroll
      for (int e = 0; e < kElems; ++e) {
        if (e * ES >= lo && e * ES < hi) {
          if (i >= C) i -= C, ++x;
          if (!(inplace && x == r)) stg<false>(dst + e * ES, (elem_t)(val[e * ES / 4] >> (e * ES % 4 * 8)));
        }
        i += ES;
      }
    }
  }
}

hipError_t launch_walk_ag(GatherCtx cx, const WalkRows& rows, int esize, hipStream_t stream) {
  GatherShape sh;
  if (!gather_shape(cx.N, cx.row_bytes, rows.recv_stride, &sh)) return hipErrorInvalidValue;
  cx.period = sh.period;
  cx.run = sh.run;
  cx.tiles = sh.tiles;
  cx.blocks = sh.blocks;
  if (rows.spaced)
    launch_kernel(esize == 2 ? walk_ag_kernel<2, true> : walk_ag_kernel<4, true>, kGatherThreads, cx, rows, stream);
  else
    launch_kernel(esize == 2 ? walk_ag_kernel<2, false> : walk_ag_kernel<4, false>, kGatherThreads, cx, rows, stream);
  return hipGetLastError();
}

// Send buffers that follow each other (the rows of one tensor): the
// concatenation is in memory already, and a receiver's row is a copy of it.  A
// lane copies one vector to one receiver: with nothing to look up and no vector
// across chunks, short workgroups stream best, and the receivers of a tile
// come by the order of the workgroups instead of in a loop.  Tiles start at
// the receiver's 128-byte lines as above.
struct CopyCtx {
  uint64_t send0, recv0;
  int64_t recv_stride, row_bytes;
  uint32_t N;
  uint32_t panel;  // tiles that every receiver takes before the next ones
  Blocks blocks;
};

template <int ES>
__global__ __launch_bounds__(kGatherThreads) void walk_ag_rows_kernel(CopyCtx cx) {
  using elem_t = typename std::conditional<ES == 4, uint32_t, uint16_t>::type;
  const uint32_t blk = block_of(cx.blocks, blockIdx.x);
  if (blk >= cx.blocks.count) return;
  uint32_t tile, receiver;
  copy_block(blk, cx.panel, cx.N, &tile, &receiver);
  char* const row = (char*)(cx.recv0 + (uint64_t)((int64_t)receiver * cx.recv_stride));
  const char* const src = (const char*)cx.send0;
  const int64_t tile0 = (int64_t)tile * kGatherTile - (int64_t)((uintptr_t)row & 127);  // may be negative
  const int64_t o = tile0 + (int)threadIdx.x * 16;
  if (o >= 0 && o + 16 <= cx.row_bytes) {
    stg<true, ES>(row + o, ldg<v4u, false, ES>(src + o));
  } else {  // the row's ends
    for (int64_t i = o < 0 ? 0 : o; i < o + 16 && i < cx.row_bytes; i += ES)
      stg<false>(row + i, ldg<elem_t, false>(src + i));
  }
}

hipError_t launch_walk_ag_rows(const GatherCtx& gx, const WalkRows& rows, int esize, hipStream_t stream) {
  CopyShape sh;
  if (!copy_shape(gx.N, gx.row_bytes, &sh)) return hipErrorInvalidValue;
  CopyCtx cx{(uint64_t)rows.send[0], (uint64_t)rows.recv[0], rows.recv_stride, gx.row_bytes, (uint32_t)gx.N, sh.panel,
             sh.blocks};
  launch_blocks(esize == 2 ? walk_ag_rows_kernel<2> : walk_ag_rows_kernel<4>, kGatherThreads, cx, cx, stream);
  return hipGetLastError();
}

}  // namespace

template <class T>
hipError_t launch_walk_rs(const WalkCtx& cx, const WalkRows& rows, bool streaming, hipStream_t stream) {
  return streaming ? launch_walk_rs_t<T, true>(cx, rows, stream) : launch_walk_rs_t<T, false>(cx, rows, stream);
}

hipError_t launch_walk(Variant v, bool streaming, const KCtx& cx, const WalkRows& rows, hipStream_t stream) {
  if (!rows.spaced && !rows.table && cx.N > kWalkInlineRanks) return hipErrorInvalidValue;
  if (v == kAgVec || v == kAgVecU || v == kAgS4 || v == kAgS2) {
    GatherCtx gx{};
    gx.rows = rows_arg(cx, rows);
    gx.chunk_bytes = cx.count * cx.esize;
    gx.row_bytes = cx.N * gx.chunk_bytes;
    gx.N = cx.N;
    if (rows.spaced && rows.send_stride == gx.chunk_bytes) return launch_walk_ag_rows(gx, rows, (int)cx.esize, stream);
    return launch_walk_ag(gx, rows, (int)cx.esize, stream);
  }
  if (cx.count < kWalkLeastElems || cx.N > kWalkMostRanks) return hipErrorInvalidValue;
  WalkCtx wx{};
  wx.rows = rows_arg(cx, rows);
  wx.N = cx.N;
  wx.chunk_bytes = cx.count * cx.esize;
  wx.V = (cx.count + 3) / 4;
  wx.back = (int32_t)(wx.V * 4 - cx.count);
  switch (v) {  // whichever path the plan's pieces take: a walk has none
    case kRsI32S:
    case kRsI32Vec:
    case kRsI32VecU: return launch_walk_rs<WI32>(wx, rows, streaming, stream);
    case kRsF32S:
    case kRsF32Vec:
    case kRsF32VecU: return launch_walk_rs<WF32>(wx, rows, streaming, stream);
    case kRsB16S:
    case kRsB16Vec:
    case kRsB16VecU: return launch_walk_rs<WB16>(wx, rows, streaming, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pat
