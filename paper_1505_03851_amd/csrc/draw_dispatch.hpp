// Launches of the draw kernels and the choice among them by K (gfx950):
// lda_draw_butterfly, lda_draw_docs and lda_draw_butterfly_philox draw
// through dispatch_butterfly.  Included by each build of the kernels (the
// default one, and the one for tables past 4 GiB: see config.hpp).
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "tuning.hpp"
#include "sources.hpp"
#include "tile.hpp"
#include "one_topic.hpp"
#include "leaf_eighths.hpp"
#include "leaf_group.hpp"

namespace LDA_NS {
namespace {

int width_for(int32_t K) { return K >= 64 ? 64 : 32; }

// The rebuilt block's table goes to LDS only for block counts up to
// LDA_LDS_TABLE_MAX_BLOCKS.  Measured on MI355X, the register table searched
// with the search-assist shuffle loop is faster at every K (the LDS table
// costs 16 KiB per wavefront and with it occupancy), so the default is 0 and
// the LDS variant is kept for comparison builds.
bool lds_table_for(int32_t K) {
  const int nb = (K + width_for(K) - 1) / width_for(K);
  return nb <= LDA_LDS_TABLE_MAX_BLOCKS;
}

// The half-block tail (W = 64) for block counts up to LDA_HALF_MAX_BLOCKS:
// it doubles the LDS rows of the block prefixes.
bool half_tail_for(int32_t K) {
  const int nb = (K + 63) / 64;
  return nb >= 2 && nb <= LDA_HALF_MAX_BLOCKS;
}

dim3 wave_grid(int64_t N, int wpb = kWavesPerBlock, int tokens = kWave) {
  const int64_t waves = (N + tokens - 1) / tokens;
  return dim3((unsigned)((waves + wpb - 1) / wpb));
}

// 256-topic blocks of the eighths kernel (the remnant of K mod 256 included).
int eighths_blocks(int32_t K) { return (K + kBlock4 - 1) / kBlock4; }

// Wavefronts per workgroup of the eighths kernel: 4 while three such
// workgroups fit in a CU's LDS (8 rows of 64 floats per block and wavefront),
// else 2.
bool eighths_wide_groups(int32_t K) {
  return 3LL * 4 * 8 * eighths_blocks(K) * kWave * (int64_t)sizeof(float) <= 160 * 1024;
}
// Whether one-document wavefronts stage their theta row in LDS for the
// rebuild: while three 4-wavefront workgroups still fit with it.
bool eighths_stage_theta(int32_t K) {
  return 3LL * 4 * eighths_lds_floats(eighths_blocks(K), true) * (int64_t)sizeof(float) <=
         160 * 1024;
}

template <int C, int WPEU, bool PAD>
void launch_eighths(const float *theta, const float *phi, DocSource d, const int32_t *wd,
                    UniformSource u, int32_t *z, int64_t N, int32_t M, int32_t V, int32_t K,
                    hipStream_t s) {
  const uint32_t tb = table_extent(M, K);
  const uint32_t pb = table_extent(V, K);
  const int NB = eighths_blocks(K);
  const size_t rows = (size_t)eighths_lds_floats(NB, false) * sizeof(float);
  const size_t staged = (size_t)eighths_lds_floats(NB, true) * sizeof(float);
  if (eighths_stage_theta(K))
    leaf_eighths_kernel<C, 4, WPEU, PAD, true><<<wave_grid(N, 4), 4 * kWave, 4 * staged, s>>>(
        theta, phi, d, wd, u, z, N, K, tb, pb);
  else if (eighths_wide_groups(K))
    leaf_eighths_kernel<C, 4, WPEU, PAD, false><<<wave_grid(N, 4), 4 * kWave, 4 * rows, s>>>(
        theta, phi, d, wd, u, z, N, K, tb, pb);
  else
    leaf_eighths_kernel<C, 2, WPEU, PAD, false><<<wave_grid(N, 2), 2 * kWave, 2 * rows, s>>>(
        theta, phi, d, wd, u, z, N, K, tb, pb);
}

template <int C, int WPEU>
void launch_eighths(const float *theta, const float *phi, DocSource d, const int32_t *wd,
                    UniformSource u, int32_t *z, int64_t N, int32_t M, int32_t V, int32_t K,
                    hipStream_t s) {
  if (K % kBlock4 == 0)
    launch_eighths<C, WPEU, false>(theta, phi, d, wd, u, z, N, M, V, K, s);
  else
    launch_eighths<C, WPEU, true>(theta, phi, d, wd, u, z, N, M, V, K, s);
}

// The leaf-group kernel: K from 4 to LDA_GROUP_MAX_K (at most 256) topics, N >=
// 64; groups of 4, 8, 16, 32 or 64 lanes for K up to 16, 32, 64, 128, 256.
// Measured on MI355X against the kernels it replaces there: 2.0x to 2.6x faster
// than the one-topic kernel for K = 10 ... 128 (K = 50 on 1M tokens: 40.9 ->
// 15.7 us; 10 on 8M: 150 -> 49; 101 on 8M: 406 -> 197), 5-8% faster than the
// eighths kernel for K = 144 ... 256.
bool groups_for(int64_t N, int32_t K) {
  return N >= kWave && K >= kLeaf && K <= LDA_GROUP_MAX_K && K <= kLeaf * kWave;
}

// Documents long enough that a 32-lane group's 32 consecutive tokens mostly
// share one: there the sums are kept in registers (118 VGPRs, 4 wavefronts per
// SIMD), else more wavefronts run (5 per SIMD).  Measured on MI355X on 4M tokens,
// not kept -> kept, documents of 64 tokens on average, of 96, 128 and 400: K = 80
// 88 -> 89 us, 86 -> 86, 85 -> 86, 80 -> 81; K = 112 101 -> 101, 100 -> 96, 98 -> 93,
// 97 -> 88; K = 128 102 -> 101, 102 -> 98, 102 -> 95, 99 -> 90; with offsets 3-4%
// less is gained (K = 112 104 -> 108, 101 -> 102, 100 -> 100, 99 -> 96).  Shuffled
// tokens, whatever the documents' lengths: 0-3% (K = 128 on 2M tokens by document
// class: 148 -> 142).  The line could lie at 96 with document ids; it stands where
// neither form loses.
bool long_docs(int64_t N, int32_t M) { return N >= 128 * (int64_t)M; }

// Where the kernel looks for scattered documents (spread_draw), and log2 of the
// tokens of a wavefront's share: documents as ids, theta past an XCD's 4 MiB of
// L2, tokens enough that every eighth wavefront's windows fill the chip, and
// enough of them per document that an XCD reads a row again before it has lost
// it.  Measured on MI355X: with theta of 4 MiB at 1M tokens 63 -> 75 us, of 8 MiB
// 85 -> 83, of 16 MiB 189 -> 139; 2M tokens, without -> with, at 64 tokens per
// document 131 -> 132 (K = 80), 195 -> 167 (128), 411 -> 345 (256), at 40 144 ->
// 144, 205 -> 195, 417 -> 395, at 30 150 -> 158, 210 -> 215, 424 -> 417, at 10 162
// -> 199, 222 -> 262, 432 -> 474.  Shares of 2^11 (four windows of 64 on
// average): 142 us at 2M tokens, K = 128; of 2^10 235 (a last window that is
// mostly empty), of 2^12 153 (too few wavefronts; at 1M tokens 207 against 139).
int spread_for(const DocSource &d, int64_t N, int32_t M, int32_t K) {
  const bool pays = d.ids && N >= (1 << 20) && (int64_t)M * K * 4 >= (6 << 20) &&
                    N >= 40 * (int64_t)M;
  return pays ? 11 : 0;
}

// Whether 64-lane groups draw 16 tokens per wavefront (one tile) instead of 64:
// where wavefronts of 64 would be about one per SIMD (1,024) or fewer, a
// wavefront's chain of four tiles is the whole launch; and with 8-topic leaves,
// of which a SIMD holds three wavefronts, where their second round would be a
// rest.  Measured on MI355X, 64 -> 16 tokens (documents of 128 tokens to 3, and
// shuffled): 65,536 tokens K = 208 7.4-10.3 -> 7.2-8.0 us, K = 300 9.7-13.5 ->
// 8.5-13.1; 98,304 at K = 300 10.8-17.4 -> 10.6-16.8; 4,096 at K = 448 7.9-10.1 ->
// 7.2-7.6; 229,376 at K = 300 21.6-37.9 -> 20.9-33.9.  Elsewhere more wavefronts
// only cost: 131,072 tokens at K = 208 8.0-14.1 -> 8.5-14.1, at K = 300 12.2-21.9
// -> 13.5-21.4; 1M at K = 300 (documents of 128) 74.0 -> 81.7.
template <int H>
bool fewer_tokens(int64_t N) {
  const int64_t waves = (N + kWave - 1) / kWave, simds = 1024;
  if (H == 1) return waves <= simds;
  const int64_t round = LDA_LEAF8_WAVES_PER_EU * simds;
  return waves <= round / 2 || (waves > round && waves < 2 * round);
}

template <int G, int H, int C, int WPEU, bool KEEP, int TOK = kWave>
void launch_groups_as(const float *theta, const float *phi, DocSource d, const int32_t *wd,
                      UniformSource u, int32_t *z, int64_t N, int32_t M, int32_t V, int32_t K,
                      hipStream_t s) {
  const uint32_t tb = table_extent(M, K);
  const uint32_t pb = table_extent(V, K);
  const size_t lds = (size_t)kWavesPerBlock * group_lds_bytes<G, H>();
  const int spread = kSpread<G, H> ? spread_for(d, N, M, K) : 0;
  if (K == kLeaf * H * G)
    leaf_group_kernel<G, H, C, WPEU, KEEP, false, TOK>
        <<<wave_grid(N, kWavesPerBlock, TOK), kBlockThreads, lds, s>>>(theta, phi, d, wd, u, z, N,
                                                                       K, tb, pb, spread);
  else
    leaf_group_kernel<G, H, C, WPEU, KEEP, true, TOK>
        <<<wave_grid(N, kWavesPerBlock, TOK), kBlockThreads, lds, s>>>(theta, phi, d, wd, u, z, N,
                                                                       K, tb, pb, spread);
}

// Launch shapes by group and leaf (tuning.hpp).
template <int G, int H>
void launch_groups(const float *theta, const float *phi, DocSource d, const int32_t *wd,
                   UniformSource u, int32_t *z, int64_t N, int32_t M, int32_t V, int32_t K,
                   hipStream_t s) {
  if constexpr (G == kWave) {
    if (fewer_tokens<H>(N)) {
      launch_groups_as<G, H, (H > 1 ? LDA_LEAF8_WINDOW : LDA_GROUP64_WINDOW),
                       (H > 1 ? LDA_LEAF8_WAVES_PER_EU : LDA_GROUP64_WAVES_PER_EU), false, 16>(
          theta, phi, d, wd, u, z, N, M, V, K, s);
      return;
    }
  }
  if constexpr (H > 1) {
    launch_groups_as<G, H, (LDA_LEAF8_WINDOW < G ? LDA_LEAF8_WINDOW : G), LDA_LEAF8_WAVES_PER_EU,
                     false>(theta, phi, d, wd, u, z, N, M, V, K, s);
  } else if constexpr (G == kWave) {
    launch_groups_as<G, H, LDA_GROUP64_WINDOW, LDA_GROUP64_WAVES_PER_EU, false>(
        theta, phi, d, wd, u, z, N, M, V, K, s);
  } else if constexpr (G == 32) {
    if (long_docs(N, M))
      launch_groups_as<G, H, 8, 4, true>(theta, phi, d, wd, u, z, N, M, V, K, s);
    else  // (the wide build's 64-bit addresses do not fit 5 wavefronts' registers: padded
          // rows at 5 spilled, K = 112 on 3M tokens 82.3 us, at 4 77.4)
      launch_groups_as<G, H, 4, 5 - LDA_WIDE_TABLES, false>(theta, phi, d, wd, u, z, N, M, V, K, s);
  } else if constexpr (G == 16) {
    launch_groups_as<G, H, 8, 5, true>(theta, phi, d, wd, u, z, N, M, V, K, s);
  } else {
    launch_groups_as<G, H, G, 6, false>(theta, phi, d, wd, u, z, N, M, V, K, s);
  }
}

// Groups of 64 lanes with 8-topic leaves for K from 257 to 512: the whole row
// in one tile, as the leaf groups do up to 256.  Measured on MI355X against
// the eighths kernel, which pads such K to two 256-topic blocks (4M tokens, V =
// 50,000): 282 against 350 us at K = 260 (18% with the butterfly search it had
// before), 347 at 384, 409 against 419 at 448, 470 against 479 at 512; against
// the one-topic kernel 304 against 380 at K = 301, 491 against 609 at 501.
// (Shuffled tokens at K = 448, 480 and 512 would be 4-18% faster by the eighths
// kernel up to 1M tokens, as fast at 2M; documents in order are 3-40% slower
// there, the shorter the more, and the order is not known on the host.)
bool leaf8_for(int64_t N, int32_t K) {
  return N >= kWave && K > kLeaf * kWave && K <= LDA_LEAF8_MAX_K && K <= 2 * kLeaf * kWave;
}

// The eighths kernel takes K divisible by 4 (16-byte leaves) up to
// LDA_EIGHTHS_MAX_BLOCKS blocks, N >= 64.  Measured on MI355X against the
// one-topic kernel: 4% faster at K = 1024, 5% at K = 2048.  The dispatch gives K
// up to 512 to the leaf-group kernel first; LDA_EIGHTHS_MIN_K bounds it in builds
// that lower LDA_GROUP_MAX_K or LDA_LEAF8_MAX_K (there it was 15-30% faster than the
// one-topic kernel from K = 144, 3-4% slower at K = 80 and 112, whose padding fills
// most of the block).
bool eighths_for(int64_t N, int32_t K) {
  return N >= kWave && K % kLeaf == 0 && K >= LDA_EIGHTHS_MIN_K &&
         eighths_blocks(K) <= LDA_EIGHTHS_MAX_BLOCKS;
}

template <int W, bool LDS_TABLE, bool ALT = false, bool HALF = false, int WPB = kWavesPerBlock>
void launch_butterfly(const float *theta, const float *phi, DocSource d,
                      const int32_t *wd, UniformSource u, int32_t *z, int64_t N,
                      int32_t M, int32_t V, int32_t K, hipStream_t s) {
  const int nb = (K + W - 1) / W;  // blocks, the remnant included
  const size_t lds = (size_t)WPB * region_rows(nb, W, LDS_TABLE, HALF) * kWave * sizeof(float);
  const uint32_t tb = table_extent(M, K);
  const uint32_t pb = table_extent(V, K);
  if (N < kWave)
    butterfly_kernel<W, LDS_TABLE, true, ALT, HALF, WPB><<<wave_grid(N, WPB), WPB * kWave, lds, s>>>(
        theta, phi, d, wd, u, z, N, K, tb, pb);
  else
    butterfly_kernel<W, LDS_TABLE, false, ALT, HALF, WPB><<<wave_grid(N, WPB), WPB * kWave, lds, s>>>(
        theta, phi, d, wd, u, z, N, K, tb, pb);
}

// The leaf-group kernel with groups just wide enough for K: K up to 16, 32, 64,
// 128, 256 topics take 4, 8, 16, 32, 64 lanes with 4-topic leaves (H = 1), half
// as many, at least 4, with 8-topic leaves (H = 2).
template <int H>
void dispatch_groups(const float *theta, const float *phi, DocSource d, const int32_t *word_id,
                     UniformSource u, int32_t *z, int64_t N, int32_t M, int32_t V, int32_t K,
                     hipStream_t s) {
  if (H == 1 && K <= kLeaf * 4)
    launch_groups<4, 1>(theta, phi, d, word_id, u, z, N, M, V, K, s);
  else if (K <= kLeaf * 8)
    launch_groups<8 / H, H>(theta, phi, d, word_id, u, z, N, M, V, K, s);
  else if (K <= kLeaf * 16)
    launch_groups<16 / H, H>(theta, phi, d, word_id, u, z, N, M, V, K, s);
  else if (K <= kLeaf * 32)
    launch_groups<32 / H, H>(theta, phi, d, word_id, u, z, N, M, V, K, s);
  else
    launch_groups<64 / H, H>(theta, phi, d, word_id, u, z, N, M, V, K, s);
}

// The butterfly draw for either document source (kernel choice by K); with
// H = 2 the leaf groups take 8-topic leaves.
template <int H = LDA_GROUP_LEAF / kLeaf>
void dispatch_butterfly(const float *theta, const float *phi, DocSource d,
                        const int32_t *word_id, UniformSource u, int32_t *z, int64_t N,
                        int32_t M, int32_t V, int32_t K, hipStream_t s) {
  if (groups_for(N, K)) {
    dispatch_groups<H>(theta, phi, d, word_id, u, z, N, M, V, K, s);
    return;
  }
  if constexpr (LDA_LEAF8_MAX_K > 0) {
    if (leaf8_for(N, K)) {
      launch_groups<kWave, 2>(theta, phi, d, word_id, u, z, N, M, V, K, s);
      return;
    }
  }
  if (eighths_for(N, K)) {
    // launch shapes measured on MI355X: up to five blocks, 16 tokens in
    // flight per wavefront at 2 wavefronts per SIMD (1-2% faster than 8 at 3
    // or 4 at 4); six to eight, 4 at 4 (3-5% faster than 16 at 2 or 8 at 3;
    // 2 in flight: 30% slower)
    if (eighths_blocks(K) <= LDA_EIGHTHS_SPLIT)
      launch_eighths<LDA_EIGHTHS_WINDOW, LDA_EIGHTHS_WAVES_PER_EU>(theta, phi, d, word_id, u, z,
                                                                   N, M, V, K, s);
    else
      launch_eighths<LDA_EIGHTHS_WINDOW_LARGE, LDA_EIGHTHS_WAVES_PER_EU_LARGE>(
          theta, phi, d, word_id, u, z, N, M, V, K, s);
    return;
  }
  const bool lt = lds_table_for(K);
  if (width_for(K) == 64) {
    if (lt)
      launch_butterfly<64, true>(theta, phi, d, word_id, u, z, N, M, V, K, s);
    else if (half_tail_for(K))
      launch_butterfly<64, false, false, true>(theta, phi, d, word_id, u, z, N, M, V, K, s);
    else
      launch_butterfly<64, false>(theta, phi, d, word_id, u, z, N, M, V, K, s);
  } else {
    if (lt)
      launch_butterfly<32, true>(theta, phi, d, word_id, u, z, N, M, V, K, s);
    else
      launch_butterfly<32, false>(theta, phi, d, word_id, u, z, N, M, V, K, s);
  }
}

}  // namespace
}  // namespace LDA_NS
