// The leaf-group kernel built for the CPU, every access bounds-checked: global
// arrays and LDS by the address sanitizer (arrays of their exact sizes; of LDS
// only the running wavefront's region is accessible), table loads by emu (a
// load must stay inside its row).
//
//   leaf_host INPUT OUTPUT G H C KEEP TOK SPREAD FIRST STEP
//
// INPUT: int64 N, M, V, K, form (0 doc ids, 1 offsets), then theta, phi, doc_id
// or offsets, word_id and u.  Workgroups FIRST, FIRST + STEP, ... and the last
// one are run (STEP 0: FIRST alone); OUTPUT gets z (-1: not drawn).
#include "hip/hip_runtime.h"

#include <sanitizer/asan_interface.h>

#include <vector>

#include "leaf_group.hpp"

namespace LDA_NS {
namespace {

alignas(16) float lds[1 << 16];

template <class T>
T *read_array(FILE *f, size_t n) {
  T *p = static_cast<T *>(malloc(n * sizeof(T)));
  if (fread(p, sizeof(T), n, f) != n) emu::fail("short input");
  return p;
}

struct Input {
  int64_t N, M, V, K, form;
  float *theta, *phi, *u;
  int32_t *ids, *word, *z;
  int64_t *offsets;
  int spread, first, step;
};

template <int G, int H, int C, bool KEEP, int TOK, bool PAD>
void run(const Input &in) {
  constexpr size_t region = (size_t)group_lds_bytes<G, H>();
  const DocSource docs{in.ids, in.offsets, (int)in.M, in.N};
  const UniformSource us{in.u, 0, 0, 0};
  const int64_t per = kWavesPerBlock * TOK;
  const int64_t blocks = (in.N + per - 1) / per;
  emu::grid_dim.x = (unsigned)blocks;
  std::vector<int64_t> run_these{in.first};
  if (in.step > 0) {
    for (int64_t b = in.first + in.step; b < blocks - 1; b += in.step) run_these.push_back(b);
    if (in.first < blocks - 1) run_these.push_back(blocks - 1);
  }
  for (const int64_t b : run_these) {
    emu::block_idx.x = (unsigned)b;
    for (int w = 0; w < kWavesPerBlock; ++w) {
      char *base = reinterpret_cast<char *>(lds);
      __asan_poison_memory_region(base, sizeof(lds));
      __asan_unpoison_memory_region(base + w * region, region);
      emu::wavefront((unsigned)w * kWave, [&] {
        leaf_group_kernel<G, H, C, 1, KEEP, PAD, TOK>(
            in.theta, in.phi, docs, in.word, us, in.z, in.N, (int)in.K,
            table_extent(in.M, (int32_t)in.K), table_extent(in.V, (int32_t)in.K), in.spread);
      });
    }
  }
}

struct Shape {
  int G, H, C, keep, tok;
  void (*full)(const Input &);
  void (*padded)(const Input &);
};
#define SHAPE(G, H, C, KEEP, TOK) \
  {G, H, C, KEEP, TOK, run<G, H, C, KEEP, TOK, false>, run<G, H, C, KEEP, TOK, true>}
// the launch shapes of the dispatch
const Shape kShapes[] = {
    SHAPE(4, 1, 4, false, 64),
    SHAPE(8, 1, 8, false, 64),
    SHAPE(16, 1, 8, true, 64),
    SHAPE(32, 1, 8, true, 64),
    SHAPE(32, 1, 4, false, 64),
    SHAPE(64, 1, LDA_GROUP64_WINDOW, false, 64),
    SHAPE(64, 1, LDA_GROUP64_WINDOW, false, 16),
    SHAPE(64, 2, LDA_LEAF8_WINDOW, false, 64),
    SHAPE(64, 2, LDA_LEAF8_WINDOW, false, 16),
    SHAPE(4, 2, 4, false, 64),
    SHAPE(8, 2, 4, false, 64),
    SHAPE(16, 2, 4, false, 64),
    SHAPE(32, 2, 4, false, 64),
};

}  // namespace
}  // namespace LDA_NS

int main(int argc, char **argv) {
  using namespace LDA_NS;
  if (argc != 11) return 2;
  Input in{};
  FILE *f = fopen(argv[1], "rb");
  if (!f || fread(&in.N, 8, 5, f) != 5) return 2;
  in.theta = read_array<float>(f, (size_t)(in.M * in.K));
  in.phi = read_array<float>(f, (size_t)(in.V * in.K));
  if (in.form == 0)
    in.ids = read_array<int32_t>(f, (size_t)in.N);
  else
    in.offsets = read_array<int64_t>(f, (size_t)in.M + 1);
  in.word = read_array<int32_t>(f, (size_t)in.N);
  in.u = read_array<float>(f, (size_t)in.N);
  fclose(f);
  in.z = static_cast<int32_t *>(malloc((size_t)in.N * 4));
  for (int64_t i = 0; i < in.N; ++i) in.z[i] = -1;
  const int G = atoi(argv[3]), H = atoi(argv[4]), C = atoi(argv[5]), keep = atoi(argv[6]);
  const int tok = atoi(argv[7]);
  in.spread = atoi(argv[8]);
  in.first = atoi(argv[9]);
  in.step = atoi(argv[10]);
  emu::row_bytes = (uint64_t)in.K * 4;
  for (const Shape &s : kShapes)
    if (s.G == G && s.H == H && s.C == C && s.keep == keep && s.tok == tok) {
      (in.K == 4 * H * G ? s.full : s.padded)(in);
      f = fopen(argv[2], "wb");
      if (!f || fwrite(in.z, 4, (size_t)in.N, f) != (size_t)in.N) return 2;
      fclose(f);
      return 0;
    }
  fprintf(stderr, "leaf_host: no such shape\n");
  return 2;
}
