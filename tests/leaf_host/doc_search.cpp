// The document search (sources.hpp) on the CPU over M documents of which only
// the last holds tokens, M near 2^31: offsets are M zeros (untouched pages of a
// private mapping between two inaccessible ones) and N.
//
//   doc_search M N FIRST ...   the documents found for tokens FIRST .. FIRST + 63
#include "hip/hip_runtime.h"

#include <sys/mman.h>

#include "sources.hpp"

int main(int argc, char **argv) {
  using namespace LDA_NS;
  const int64_t M = atoll(argv[1]), N = atoll(argv[2]);
  const size_t page = 4096, body = ((size_t)(M + 1) * 8 + page - 1) / page * page;
  // (far enough that an index wrapped past 2^31 lands in the first guard)
  const size_t guard = (size_t)1 << 35;
  char *p = static_cast<char *>(mmap(nullptr, guard + body + page, PROT_NONE,
                                     MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
  if (p == MAP_FAILED || mprotect(p + guard, body, PROT_READ | PROT_WRITE) != 0) return 2;
  int64_t *offsets = reinterpret_cast<int64_t *>(p + guard);
  offsets[M] = N;
  const DocSource docs{nullptr, offsets, (int)M, N};
  for (int i = 3; i < argc; ++i) {
    const int64_t first = atoll(argv[i]);
    int64_t low = M, high = -1;
    emu::wavefront(0, [&] {
      const int64_t d = docs.wave_doc(first + lane_id(), first, first + kWave - 1);
      low = std::min(low, d);
      high = std::max(high, d);
    });
    printf("%lld %lld\n", (long long)low, (long long)high);
    fflush(stdout);
  }
  return 0;
}
