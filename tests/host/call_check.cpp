// Whole calls of the C-ABI layer over the stand-in runtime of hip_fake.hpp,
// under AddressSanitizer / UndefinedBehaviorSanitizer.  The argument names the
// check.
#include <unistd.h>

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

int main(int argc, char** argv) {
  const std::string which = argc > 1 ? argv[1] : "";
  if (which == "no_environment") check_no_environment();
  else return std::fprintf(stderr, "no check named '%s'\n", which.c_str()), 2;
  EXPECT(pat_finalize() == PAT_OK);
  std::printf("%s: %d failures\n", which.c_str(), failures);
  return failures != 0;
}
