// Build-time tuning of the draw kernels (chosen by measurement on MI355X).
#pragma once

//   LDA_LDS_TABLE_MAX_BLOCKS  largest K / W whose rebuilt table goes to LDS
//                             (see lds_table_for);
//   LDA_WAVES_PER_EU          wavefronts per SIMD the register budget targets;
//   LDA_WAVES_PER_BLOCK       wavefronts per workgroup (for the leaf-group
//                             kernel, 1 and 4 were within 2% of 2 at
//                             K = 16 ... 256).
#ifndef LDA_LDS_TABLE_MAX_BLOCKS
#define LDA_LDS_TABLE_MAX_BLOCKS 0
#endif
#ifndef LDA_WAVES_PER_EU
#define LDA_WAVES_PER_EU 3
#endif
#ifndef LDA_WAVES_PER_BLOCK
#define LDA_WAVES_PER_BLOCK 2
#endif
//   LDA_DOC_LANES_TARGET_WAVES wavefronts the document-per-lane driver aims
//                             for by splitting each group's master loop.
#ifndef LDA_DOC_LANES_TARGET_WAVES
#define LDA_DOC_LANES_TARGET_WAVES 16384
#endif
//   LDA_HALF_MAX_BLOCKS       largest K / 64 for which the W = 64 kernel
//                             rebuilds only the chosen half-block (its 2 K/64
//                             LDS rows per wavefront keep 12 wavefronts per CU
//                             up to 26 blocks, 10 at 32 blocks).
#ifndef LDA_HALF_MAX_BLOCKS
#define LDA_HALF_MAX_BLOCKS 32
#endif
//   LDA_EIGHTHS_MAX_BLOCKS    largest number of 256-topic blocks for which the
//                             leaf kernel with 32-topic prefix rows draws
//                             (8 rows of LDS per block and wavefront; 0: never);
//   LDA_EIGHTHS_SPLIT         largest block count drawn with the first of its
//                             two launch shapes;
//   LDA_EIGHTHS_WINDOW{,_LARGE}, LDA_EIGHTHS_WAVES_PER_EU{,_LARGE}
//                             tokens in flight per wavefront (16-byte loads)
//                             and wavefronts per SIMD of the two shapes.
#ifndef LDA_EIGHTHS_MAX_BLOCKS
#define LDA_EIGHTHS_MAX_BLOCKS 8
#endif
//   LDA_GROUP_MAX_K           largest K drawn by the leaf-group kernel with
//                             4-topic leaves (K >= 4, at most 256; 0: never).
#ifndef LDA_GROUP_MAX_K
#define LDA_GROUP_MAX_K 256
#endif
//   LDA_GROUP64_WINDOW, LDA_GROUP64_WAVES_PER_EU  tokens in flight per
//                             wavefront and wavefronts per SIMD of its 64-lane
//                             groups (K from 129 to 256): 8 at 4 (128 VGPRs)
//                             took 133 us on the paper-shaped corpus at K =
//                             208, 8 at 3 took 147; even at K = 256 on 1M
//                             tokens (51 us).  Narrower groups: see
//                             launch_groups.
#ifndef LDA_GROUP64_WINDOW
#define LDA_GROUP64_WINDOW 8
#endif
#ifndef LDA_GROUP64_WAVES_PER_EU
#define LDA_GROUP64_WAVES_PER_EU 4
#endif
//   LDA_GROUP_LEAF            topics per lane of the leaf-group kernel (4 or
//                             8: groups of K / 4 or K / 8 lanes, rounded up
//                             to a power of two).
#ifndef LDA_GROUP_LEAF
#define LDA_GROUP_LEAF 4
#endif
//   LDA_LEAF8_MAX_K           largest K above 256 drawn by groups of 64 lanes
//                             with 8-topic leaves, the whole row in one tile
//                             (at most 512; 0: none); the eighths kernel draws
//                             the rest (see leaf8_for).
//   LDA_LEAF8_WINDOW, LDA_LEAF8_WAVES_PER_EU  tokens in flight per wavefront
//                             and wavefronts per SIMD of 8-topic leaves: 4 at
//                             3 (158 VGPRs) took 282-470 us at K = 260 ... 512
//                             on 4M tokens, 2 at 4 305-467, 8 at 3 340-545.
#ifndef LDA_LEAF8_MAX_K
#define LDA_LEAF8_MAX_K 512
#endif
#ifndef LDA_LEAF8_WINDOW
#define LDA_LEAF8_WINDOW 4
#endif
#ifndef LDA_LEAF8_WAVES_PER_EU
#define LDA_LEAF8_WAVES_PER_EU 3
#endif
//   LDA_EIGHTHS_MIN_K         smallest K it takes where the leaf groups leave it
//                             (LDA_GROUP_MAX_K or LDA_LEAF8_MAX_K lowered; K
//                             divisible by 4; the first block is padded with
//                             empty topics up to a multiple of 256).
#ifndef LDA_EIGHTHS_MIN_K
#define LDA_EIGHTHS_MIN_K 132
#endif
#ifndef LDA_EIGHTHS_SPLIT
#define LDA_EIGHTHS_SPLIT 5
#endif
#ifndef LDA_EIGHTHS_WINDOW
#define LDA_EIGHTHS_WINDOW 16
#endif
#ifndef LDA_EIGHTHS_WAVES_PER_EU
#define LDA_EIGHTHS_WAVES_PER_EU 2
#endif
#ifndef LDA_EIGHTHS_WINDOW_LARGE
#define LDA_EIGHTHS_WINDOW_LARGE 4
#endif
#ifndef LDA_EIGHTHS_WAVES_PER_EU_LARGE
#define LDA_EIGHTHS_WAVES_PER_EU_LARGE 4
#endif
//   LDA_ROUTED_FEW_WINDOW, LDA_ROUTED_FEW_THETA  tokens in flight per
//                             wavefront (phi loads) and theta leaves read
//                             ahead from LDS when a routed wavefront's tokens
//                             form a few runs of documents.
#ifndef LDA_ROUTED_FEW_WINDOW
#define LDA_ROUTED_FEW_WINDOW 16
#endif
#ifndef LDA_ROUTED_FEW_THETA
#define LDA_ROUTED_FEW_THETA 4
#endif
//   LDA_COUNT_SPLIT_MIN_N     smallest number of tokens whose word counts are
//                             taken by partition of the cells (count_cells in
//                             lda_draw.hip).
#ifndef LDA_COUNT_SPLIT_MIN_N
#define LDA_COUNT_SPLIT_MIN_N 524288
#endif
