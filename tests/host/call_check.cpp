// Whole calls of the C-ABI layer over the stand-in runtime of hip_fake.hpp,
// under AddressSanitizer / UndefinedBehaviorSanitizer.  The argument names the
// check.
#include <unistd.h>

#include <cmath>
#include <string>

#include "../../include/pat.h"
#include "hip_fake.hpp"

static int failures = 0;
#define EXPECT(cond)                                                        \
  do {                                                                      \
    if (!(cond)) {                                                          \
      std::fprintf(stderr, "%s:%d: expected %s\n", __FILE__, __LINE__, #cond); \
      ++failures;                                                           \
    }                                                                       \
  } while (0)

// Buffer addresses (never followed): n rows of `bytes`, `gap` apart.
template <class P>
static std::vector<P> rows(uintptr_t base, int n, size_t bytes, size_t gap = 0) {
  std::vector<P> v(n);
  for (int i = 0; i < n; ++i) v[i] = (P)(base + uintptr_t(i) * (bytes + gap));
  return v;
}

struct Buffers {
  std::vector<const void*> send;
  std::vector<void*> recv;
};
static Buffers buffers(int coll, int n, size_t chunk, uintptr_t base = uintptr_t(1) << 40) {
  return {rows<const void*>(base, n, coll == 0 ? chunk : chunk * n),
          rows<void*>(base + (uintptr_t(1) << 44), n, coll == 0 ? chunk * n : chunk)};
}
static pat_status_t call(int coll, const Buffers& b, size_t count, pat_dtype_t dt) {
  const int n = (int)b.send.size();
  return coll == 0 ? pat_allgather(b.send.data(), b.recv.data(), count, dt, n, nullptr)
                   : pat_reducescatter(b.send.data(), b.recv.data(), count, dt, PAT_SUM, n, nullptr);
}

// No environment at all (clearenv() leaves a null environ): the default path.
static void check_no_environment() {
  EXPECT(clearenv() == 0 && environ == nullptr);
  for (int coll = 0; coll < 2; ++coll) {
    fake::launches.clear();
    EXPECT(call(coll, buffers(coll, 6, 4096), 1024, PAT_FLOAT32) == PAT_OK);
    EXPECT(fake::launches.size() == 1 && fake::launches[0].kind == 'w');
  }
  const Buffers b = buffers(1, 6, 4096);
  EXPECT(pat_reducescatter_noalloc(b.send.data(), b.recv.data(), 1024, PAT_FLOAT32, PAT_SUM, 6, nullptr) == PAT_OK);
}

// What a trace changes and records: pat_trace_start the step schedule,
// pat_trace_start_as_run what an untraced operation launches.
static void check_trace() {
  for (int coll = 0; coll < 2; ++coll) {
    const int n = 24;
    const size_t count = 1000;
    const Buffers b = buffers(coll, n, count * 4);
    pat_plan_info_t info;
    EXPECT(pat_plan_info((pat_collective_t)coll, n, count, PAT_FLOAT32, &info) == PAT_OK);
    for (bool steps : {false, true}) {
      EXPECT((steps ? pat_trace_start(100) : pat_trace_start_as_run(100)) == PAT_OK);
      fake::launches.clear();
      EXPECT(call(coll, b, count, PAT_FLOAT32) == PAT_OK && call(coll, b, count, PAT_FLOAT32) == PAT_OK);
      float ms[100];
      double bytes[100];
      int32_t kind[100], step[100];
      int used = 0;
      EXPECT(pat_trace_read(ms, bytes, kind, step, 100, &used) == PAT_OK);
      EXPECT((int)fake::launches.size() == used && used == 2 * (steps ? info.launches_per_op : 1));
      double sum = 0;
      for (int j = 0; j < used; ++j) {
        EXPECT(fake::launches[j].kind == "stw"[kind[j]] && (steps ? kind[j] < 2 : kind[j] == 2 && step[j] == 0));
        sum += bytes[j];
      }
      const double needed = 4.0 * count * n * (n + 1);
      EXPECT(steps ? std::abs(sum / 2 / info.alg_bytes - 1) < 1e-9 : sum == 2 * needed);
      EXPECT(pat_trace_read(ms, bytes, kind, step, 100, &used) == PAT_ERR_INVALID_ARGUMENT);  // disarmed
    }
    fake::launches.clear();
    EXPECT(call(coll, b, count, PAT_FLOAT32) == PAT_OK);
    EXPECT(fake::launches.size() == 1 && fake::launches[0].kind == 'w');
    EXPECT(pat_trace_start_as_run(1) == PAT_OK);  // room for one launch: the second call records nothing
    EXPECT(call(coll, b, count, PAT_FLOAT32) == PAT_OK && call(coll, b, count, PAT_FLOAT32) == PAT_OK);
    int used = 0;
    EXPECT(pat_trace_read(nullptr, nullptr, nullptr, nullptr, 1, &used) == PAT_OK && used == 1);
  }
  EXPECT(pat_trace_start_as_run(0) == PAT_ERR_INVALID_ARGUMENT);
}

int main(int argc, char** argv) {
  const std::string which = argc > 1 ? argv[1] : "";
  if (which == "no_environment") check_no_environment();
  else if (which == "trace") check_trace();
  else return std::fprintf(stderr, "no check named '%s'\n", which.c_str()), 2;
  EXPECT(pat_finalize() == PAT_OK);
  std::printf("%s: %d failures\n", which.c_str(), failures);
  return failures != 0;
}
