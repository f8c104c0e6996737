// Walk kernels (walk.hip): whole operations in one launch, every tree walked
// in its linear order with the intermediate buffers in registers.
#pragma once

#include "kernels.hpp"

namespace pat {

// Most ranks a reduce-scatter's walk holds slots for: 16 lane groups, each
// with slots for 128 groups of 2 positions.
constexpr int kWalkMostRanks = 4096;
// Fewest elements of a chunk a walk is taken for.  Under that a tree is too
// few vectors for a walk: N = 1000 float32 on MI355X, steps / walk, 4
// elements 52 / 92 us, 8 elements 55 / 59 us, 16 elements 64 / 51 us (bf16 16
// elements 66 / 56 us; N = 16 and 100, 16 elements: the walk 2-15% faster).
constexpr int64_t kWalkLeastElems = 16;

// Where the ranks' buffers are, for one call.  The caller's host arrays
// (`send`, `recv`) are read during the call only.
struct WalkRows {
  const void* const* send;
  void* const* recv;
  int64_t send_stride, recv_stride;  // bytes from rank 0's buffer to rank 1's
  bool spaced;                       // every rank's buffers follow at those strides: the launch carries
                                     // two addresses and two strides
  bool aligned8;                     // every send buffer is 8-byte aligned
  bool table;                        // neither spaced nor few enough for the launch to carry the pointers:
                                     // the kernel reads the device tables of its context
};

// Most ranks whose pointers a launch carries as arguments (1 KiB of them).
constexpr int kWalkInlineRanks = 64;

inline WalkRows walk_rows(const void* const* send, void* const* recv, int N) {
  WalkRows w{send, recv, 0, 0, true, true, false};
  if (N > 1) {
    const uintptr_t s0 = (uintptr_t)send[0], r0 = (uintptr_t)recv[0];
    const uintptr_t ds = (uintptr_t)send[1] - s0, dr = (uintptr_t)recv[1] - r0;
    uintptr_t off = 0, bits = s0 | (uintptr_t)send[1];
    for (int r = 2; r < N; ++r) {
      off |= ((uintptr_t)send[r] - s0 - r * ds) | ((uintptr_t)recv[r] - r0 - r * dr);  // distances from their places
      bits |= (uintptr_t)send[r];
    }
    w.send_stride = (int64_t)ds;
    w.recv_stride = (int64_t)dr;
    w.spaced = off == 0;
    w.aligned8 = bits % 8 == 0;
  }
  w.table = !w.spaced && N > kWalkInlineRanks;
  return w;
}

// The operation of variant v over the buffers of `rows` (rows.table: of
// cx.send and cx.recv).  streaming: nontemporal accesses (reduce-scatter).
hipError_t launch_walk(Variant v, bool streaming, const KCtx& cx, const WalkRows& rows, hipStream_t stream);

}  // namespace pat
