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
    fake::forget();
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
      fake::forget();
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
    fake::forget();
    EXPECT(call(coll, b, count, PAT_FLOAT32) == PAT_OK);
    EXPECT(fake::launches.size() == 1 && fake::launches[0].kind == 'w');
    EXPECT(pat_trace_start_as_run(1) == PAT_OK);  // room for one launch: the second call records nothing
    EXPECT(call(coll, b, count, PAT_FLOAT32) == PAT_OK && call(coll, b, count, PAT_FLOAT32) == PAT_OK);
    int used = 0;
    EXPECT(pat_trace_read(nullptr, nullptr, nullptr, nullptr, 1, &used) == PAT_OK && used == 1);
  }
  EXPECT(pat_trace_start_as_run(0) == PAT_ERR_INVALID_ARGUMENT);
}

// pat_launch_info says what a call launches, on both sides of every limit of
// the choice, in every mode (a graph's capture aside) and at every setting
// that it depends on.
static void check_routes() {
  struct Case {
    int coll, n;
    size_t count;
    pat_dtype_t dt;
    bool walk;  // at the default settings
  };
  const Case cases[] = {
      {1, 6, 15, PAT_FLOAT32, false},   {1, 6, 16, PAT_FLOAT32, true},      {1, 6, 16, PAT_BFLOAT16, true},
      {1, 6, 15, PAT_INT32, false},     {1, 4096, 16, PAT_BFLOAT16, true},  {1, 4097, 16, PAT_BFLOAT16, false},
      {1, 2, 16, PAT_FLOAT32, true},    {0, 2, 1, PAT_BFLOAT16, true},      {0, 5000, 3, PAT_FLOAT32, true},
      {1, 70, 5098, PAT_FLOAT32, true}, {1, 70, 5103, PAT_FLOAT32, true},  // 0.999e8 and 1.0002e8 bytes
      {1, 64, 262144, PAT_FLOAT32, true}, {0, 64, 262144, PAT_FLOAT32, true}, {1, 1, 64, PAT_FLOAT32, false},
  };
  auto agrees = [](const Case& c, bool walk) {
    pat_launch_info_t li;
    EXPECT(pat_launch_info((pat_collective_t)c.coll, c.n, c.count, c.dt, &li) == PAT_OK);
    fake::forget();
    EXPECT(call(c.coll, buffers(c.coll, c.n, c.count * (c.dt == PAT_BFLOAT16 ? 2 : 4)), c.count, c.dt) == PAT_OK);
    EXPECT((li.walk == 1) == walk);
    EXPECT(li.launches == (int)fake::launches.size());
    for (const auto& l : fake::launches) EXPECT((l.kind == 'w') == walk && l.streaming == (li.nontemporal == 1));
  };
  for (const Case& c : cases) {
    agrees(c, c.walk);
    if (c.n > 1000) continue;  // the settings: at small plans
    for (int mode : {PAT_EXEC_PERSISTENT, PAT_EXEC_DATAFLOW}) {
      EXPECT(pat_set_exec_mode(mode) == PAT_OK);
      agrees(c, false);
    }
    EXPECT(pat_set_exec_mode(PAT_EXEC_STREAM) == PAT_OK);
    for (int fusion : {PAT_FUSION_OFF, PAT_FUSION_ON}) {
      EXPECT(pat_set_top_fusion(fusion) == PAT_OK);
      agrees(c, false);
    }
    EXPECT(pat_set_top_fusion(PAT_FUSION_AUTO) == PAT_OK);
    EXPECT(pat_set_linear_order(PAT_LINEAR_CLOSE_FIRST) == PAT_OK);
    agrees(c, c.walk && c.coll == 0);
    EXPECT(pat_set_linear_order(PAT_LINEAR_FAR_FIRST) == PAT_OK);
    EXPECT(pat_set_buffer_bytes(1024) == PAT_OK);  // pieces: no part of a walk
    agrees(c, c.walk);
    EXPECT(pat_set_buffer_bytes(0) == PAT_OK);
    EXPECT(pat_trace_start(1) == PAT_OK);
    agrees(c, false);
    EXPECT(pat_trace_start_as_run(1) == PAT_OK);
    agrees(c, c.walk);
    int used = 0;
    EXPECT(pat_trace_read(nullptr, nullptr, nullptr, nullptr, 1, &used) == PAT_OK && used == (c.n > 1));
    for (const char* name : {"PAT_WALK", "PAT_TREE_TILE", "PAT_TREE_FUSE_VECS", "PAT_TREE_FUSE_BYTES",
                             "PAT_TREE_EDGE_CACHE", "PAT_STREAMING", "PAT_XCD_GRAIN", "PAT_PIECE_PIPELINE",
                             "PAT_STEP_CLOCK"}) {
      EXPECT(pat_finalize() == PAT_OK);  // some are a plan's
      setenv(name, std::strcmp(name, "PAT_STEP_CLOCK") ? "0" : "1", 1);
      agrees(c, false);
      unsetenv(name);
    }
    EXPECT(pat_finalize() == PAT_OK);
    setenv("PAT_WALK", "1", 1);
    agrees(c, c.walk);
    unsetenv("PAT_WALK");
  }
  pat_launch_info_t li;
  EXPECT(pat_launch_info(PAT_ALLGATHER, 0, 1, PAT_FLOAT32, &li) == PAT_ERR_INVALID_ARGUMENT);
  EXPECT(pat_launch_info(PAT_ALLGATHER, 2, 1, PAT_FLOAT32, nullptr) == PAT_ERR_INVALID_ARGUMENT);
}

// Calls with buffers of their own, none waited for: every launch must find its
// own call's addresses when it runs, also where the staging sets have come
// round several times, and where calls that upload nothing come in between.
static void check_staging() {
  const int n = 70;  // more than a launch carries
  const size_t count = 200;
  for (int coll = 0; coll < 2; ++coll)
    for (int mode : {PAT_EXEC_STREAM, PAT_EXEC_PERSISTENT, PAT_EXEC_DATAFLOW})
      for (int fusion : {PAT_FUSION_AUTO, PAT_FUSION_OFF}) {
        EXPECT(pat_set_exec_mode(mode) == PAT_OK && pat_set_top_fusion(fusion) == PAT_OK);
        fake::forget();
        std::vector<Buffers> made;
        std::vector<size_t> first;
        for (int k = 0; k < 23; ++k) {
          made.push_back(buffers(coll, n, count * 4, (uintptr_t(1) << 40) + (uintptr_t(k) << 32)));
          Buffers& b = made.back();
          if (k % 5 != 3) {  // no spacing: the table has to be uploaded
            std::swap(b.send[k + 1], b.send[k + 2]);
            std::swap(b.recv[k + 3], b.recv[k + 40]);
          }
          if (k % 7 == 6) b = made[k - 1];  // the set of the call before
          first.push_back(fake::launches.size());
          EXPECT(call(coll, b, count, PAT_FLOAT32) == PAT_OK);
        }
        first.push_back(fake::launches.size());
        fake::drain();
        for (size_t k = 0; k < made.size(); ++k) {
          EXPECT(first[k + 1] > first[k]);
          for (size_t j = first[k]; j < first[k + 1]; ++j)
            EXPECT(fake::launches[j].send == made[k].send && fake::launches[j].recv == made[k].recv);
        }
      }
  EXPECT(pat_set_exec_mode(PAT_EXEC_STREAM) == PAT_OK && pat_set_top_fusion(PAT_FUSION_AUTO) == PAT_OK);
}

int main(int argc, char** argv) {
  const std::string which = argc > 1 ? argv[1] : "";
  if (which == "no_environment") check_no_environment();
  else if (which == "trace") check_trace();
  else if (which == "routes") check_routes();
  else if (which == "staging") check_staging();
  else return std::fprintf(stderr, "no check named '%s'\n", which.c_str()), 2;
  EXPECT(pat_finalize() == PAT_OK);
  std::printf("%s: %d failures\n", which.c_str(), failures);
  return failures != 0;
}
