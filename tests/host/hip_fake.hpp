// A stand-in for the HIP runtime and for the kernels' launch entry points, so
// that whole calls of the C-ABI layer (api.cpp) run on the CPU: which launch an
// operation takes, and which buffer addresses that launch finds.
//
// Device memory is host memory.  Queued work -- copies, event records,
// launches -- waits in one queue, in order, until something waits for it, as
// late as the runtime may run it: a copy from pinned memory reads its source
// then, one from pageable memory has read it when the call returns, and a
// launch reads its pointer tables then.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <vector>

#include "kernels.hpp"
#include "walk.hpp"

namespace fake {

struct Launch {
  char kind;  // 's' step, 't' fused steps, 'w' walk, 'p' persistent, 'd' dataflow
  bool streaming;
  std::vector<const void*> send;  // the addresses the kernel finds when it runs
  std::vector<void*> recv;
};

inline std::deque<std::function<void()>> queue;
inline uint64_t queued = 0, done = 0;  // entries, in all
inline std::map<void*, uint64_t> recorded;  // event -> the queue position that completes it
inline std::map<char*, size_t> pinned;
inline std::vector<Launch> launches;  // in launch order; addresses are filled in as they run

inline void push(std::function<void()> f) {
  queue.push_back(std::move(f));
  ++queued;
}
inline void run_until(uint64_t position) {
  while (done < position && !queue.empty()) {
    queue.front()();
    queue.pop_front();
    ++done;
  }
}
inline void drain() { run_until(queued); }
inline void forget() {  // the launches so far
  drain();
  launches.clear();
}

inline void launch(char kind, bool streaming, const pat::KCtx& cx, const pat::WalkRows* rows = nullptr) {
  const size_t i = launches.size();
  launches.push_back({kind, streaming, {}, {}});
  if (rows && !rows->table) {  // the launch carries the addresses
    launches[i].send.assign(rows->send, rows->send + cx.N);
    launches[i].recv.assign(rows->recv, rows->recv + cx.N);
    push([] {});
    return;
  }
  push([i, cx] {
    launches[i].send.assign(cx.send, cx.send + cx.N);
    launches[i].recv.assign(cx.recv, cx.recv + cx.N);
  });
}

}  // namespace fake

extern "C" {

hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) {
  fake::drain();
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::malloc(n);
  fake::pinned[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  fake::drain();
  fake::pinned.erase((char*)p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) {
  fake::drain();
  std::memset(p, v, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) {
  fake::drain();
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyDeviceToDevice) return fake::push([] {}), hipSuccess;  // of user buffers, which do not exist
  auto it = fake::pinned.upper_bound((char*)src);
  if (it != fake::pinned.begin() && (char*)src < std::prev(it)->first + std::prev(it)->second) {
    fake::push([=] { std::memcpy(dst, src, n); });
  } else {
    std::vector<char> bytes((const char*)src, (const char*)src + n);
    fake::push([dst, bytes = std::move(bytes)] { std::memcpy(dst, bytes.data(), bytes.size()); });
  }
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)std::malloc(1);
  fake::recorded[*e] = 0;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  fake::recorded.erase(e);
  std::free((void*)e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  fake::push([] {});
  fake::recorded[e] = fake::queued;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  fake::run_until(fake::recorded[e]);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return fake::drain(), hipSuccess; }
hipError_t hipDeviceSynchronize() { return fake::drain(), hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipErrorNotSupported; }  // no graph mode here
hipError_t hipStreamDestroy(hipStream_t) { return hipErrorNotSupported; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipErrorNotSupported; }

}  // extern "C"

namespace pat {

// The sizes of kernels.hip's variants: they shape the launch-level steps.
int variant_in_bytes(Variant v) {
  if (v == kRsB16Vec || v == kRsB16VecU) return 8;
  if (v == kAgS4 || v == kRsI32S || v == kRsF32S) return 4;
  return v == kAgS2 || v == kRsB16S ? 2 : 16;
}
bool variant_partial(Variant v) { return v == kAgVecU || v == kRsI32VecU || v == kRsF32VecU || v == kRsB16VecU; }
bool variant_partial_items(Variant v) { return v == kRsB16VecU; }
int variant_tile(Variant v) { return variant_in_bytes(v) < 8 ? 2048 : variant_in_bytes(v) == 8 ? 1024 : 512; }
int variant_pack_tile(Variant v) { return variant_in_bytes(v) < 16 ? 1024 : 512; }

hipError_t launch_step(Variant, bool nt, int64_t, const KCtx& cx, const DevStep&, hipStream_t) {
  return fake::launch('s', nt, cx), hipSuccess;
}
hipError_t launch_step2(Variant, bool nt, int64_t, const KCtx& cx, int, const DevStep&, int, const DevStep&,
                        hipStream_t) {
  return fake::launch('s', nt, cx), hipSuccess;
}
hipError_t launch_tree(Variant, bool nt, const KCtx& cx, const TreeRange&, hipStream_t) {
  return fake::launch('t', nt, cx), hipSuccess;
}
hipError_t launch_walk(Variant, bool nt, const KCtx& cx, const WalkRows& rows, hipStream_t) {
  return fake::launch('w', nt, cx, &rows), hipSuccess;
}
hipError_t launch_persistent(Variant, bool nt, const KCtx& cx, int, hipStream_t) {
  return fake::launch('p', nt, cx), hipSuccess;
}
hipError_t launch_dataflow(Variant, bool nt, const KCtx& cx, bool, int, hipStream_t) {
  return fake::launch('d', nt, cx), hipSuccess;
}
hipError_t persistent_capacity(Variant, bool, int* blocks) { return *blocks = 1024, hipSuccess; }

size_t scratch_bytes() { return size_t(256) << 20; }
hipError_t scratch_base(int, char** base) {
  static std::vector<char> scratch(scratch_bytes());
  return *base = scratch.data(), hipSuccess;
}

}  // namespace pat
