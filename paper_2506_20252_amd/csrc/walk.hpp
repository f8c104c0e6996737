// Walk kernels (walk.hip): whole operations in one launch, every tree walked
// in its linear order with the intermediate buffers in registers.
#pragma once

#include "kernels.hpp"

namespace pat {

// Most ranks a reduce-scatter's walk holds slots for: 16 lane groups, each
// with slots for 128 groups of 2 positions (bf16: 64 of 4).
constexpr int kWalkMostRanks = 4096;
// Fewest elements of a chunk a walk is taken for.  Under that a tree is too
// few vectors for a walk: N = 1000 float32 on MI355X, steps / walk, 4
// elements 52 / 92 us, 8 elements 55 / 59 us, 16 elements 64 / 51 us (bf16 16
// elements 66 / 56 us; N = 16 and 100, 16 elements: the walk 2-15% faster).
constexpr int64_t kWalkLeastElems = 16;

// The operation of variant v over the buffers of cx.send and cx.recv.
// streaming: nontemporal accesses (reduce-scatter).  recv_stride: the bytes
// from one rank's receive buffer to the next one's, where that is the same for
// all (all-gather: how its receivers share workgroups follows from it; any
// value gives the same result).
hipError_t launch_walk(Variant v, bool streaming, const KCtx& cx, int64_t recv_stride, hipStream_t stream);

}  // namespace pat
