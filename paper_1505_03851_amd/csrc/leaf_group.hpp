// Leaf-group kernel for K from 4 to 256, and with 8-topic leaves up to 512
// (gfx950).
#pragma once

#include "tile.hpp"

namespace LDA_NS {
namespace {

// Leaf groups for 4 <= K <= 4 H G topics (groups of G = 4, 8, 16, 32 or 64
// lanes, leaves of 4 H topics: H quads).  Sections 3 and 4 with a leaf in the
// place of a topic: a wavefront holds 64 / G groups of G tokens, lane r of a
// group owns token r of the group and, in the tile, leaf r of every token of
// its group.  Load k brings leaf r of token k of every group into lane r of
// that group, so each load instruction reads the whole rows (16 G bytes for H
// = 1) of 64 / G tokens, and the lane sums its leaf's products (dot4).
//
// The leaf sums go through LDS to the lanes that search them: every NLD loads
// make a tile of T = 64 NLD / G tokens, P = 64 / T lanes then share a token,
// each taking G / P consecutive leaf sums (16-byte reads), and the quad's
// lanes learn each other's totals by DPP.  The search is a descent with
// nested thresholds: the lane whose leaves hold u * S (prefixes of the lane
// totals), the quad of leaves in it (prefixes of quad sums), the leaf, then
// the topic by a scan of the leaf's products.  At K = 64 that is 195 vector
// instructions per wavefront where Algorithm 8's butterfly over the leaf sums
// with Algorithm 10's search-assist loop took 275, and one chain of LDS round
// trips instead of one per level.  What bounds a draw here is the sum of
// latencies of a wavefront (ids, rows, search) over the wavefronts that a CU
// holds, then the L1's 64 bytes per clock; misses past L2 take over from about
// K = 200.  Measured on MI355X (1M tokens, documents of 128): K = 64 17.2 ->
// 14.8 us, K = 128 28.1 -> 25.8, K = 256 53.9 -> 51.0; on the paper-shaped
// corpus K = 208 152 -> 136 us; K not divisible by 4, which one topic per lane
// drew before: K = 50 41.0 -> 15.7, K = 250 82.7 -> 54.7.
//
// The topics of a row are padded in front to a whole number of leaves: index
// i of the padded row (i < 0: empty leaves) is topic i for K divisible by 4;
// else the first quad (0 <= i < 4) holds topics 0 .. K mod 4 - 1 in its first
// components and none in the others, and i >= 4 is topic i - (4 - K mod 4).
// No load leaves the token's row, whatever its alignment (a row needs K >= 4).
// Empty components have a theta of zero, hence a prefix equal to the one
// before them, and a search that skips every prefix <= u * S never ends in
// front of the first topic.
//
// How the theta leaves of a group's tokens are found: every group's tokens in
// one document (one leaf per lane, loaded once), in at most kMaxGroupRuns<G>
// runs of documents (each run's leaf loaded once per lane; token k takes the
// leaf of its run: for groups of 64 lanes, up to 4 runs, from LDS where the
// leaves are staged, read a few tokens ahead; below, up to 2 runs, by a
// select in registers), or any mix (a leaf per token, loaded with its phi
// leaf).  In the first two cases every run's leaves are also staged in LDS,
// and the final reload takes its theta leaf from there (one LDS read in the
// place of a gather from memory).
enum GroupTheta : int { kGroupOne = 0, kGroupRuns = 1, kGroupAny = 2 };
template <int G>
constexpr int kMaxGroupRuns = G == kWave ? 4 : 2;
constexpr int kRunAhead = 4;  // tokens whose staged theta leaves are read ahead
// Runs read from LDS in the tile (measured: 5-15% faster for 64-lane groups
// than four selects per token; for 32-lane groups, up to 12% slower than one
// select)
template <int G>
constexpr bool kStageRuns = G == kWave;

// Shape of a tile and the layout of its leaf sums in LDS (see above).  Rows
// are padded so that the 16-byte reads of eight consecutive lanes, and the
// 4-byte writes of 32, fall on different banks.
template <int G>
struct GroupTile {
  static constexpr int kLoads = G < 16 ? G : 16;       // loads per tile (NLD)
  static constexpr int kTiles = G / kLoads;            // tiles per 64 tokens
  static constexpr int kTokens = kLoads * (kWave / G);  // T
  static constexpr int kParts = kWave / kTokens;       // lanes per token (P)
  static constexpr int kLeaves = G / kParts;           // leaves per lane
  static constexpr int kQuads = kLeaves / 4;           // 16-byte reads per lane
  // floats between the rows of consecutive tokens (16-byte multiples)
  static constexpr int kRow = G == 4 ? 4 : (G == kWave ? G + 8 : G + 4);
  // floats between the tokens of consecutive groups
  static constexpr int kGroup =
      kLoads * kRow + (G == 4 ? 4 : (G == 8 ? 8 : (G == 16 ? 16 : 0)));
  static constexpr int kFloats = (kWave / G) * kGroup;
  // leaf r of a row: 64-leaf rows skip 4 floats after the first 32
  __device__ static __forceinline__ int leaf(int r) {
    return G == kWave ? r + 4 * (r >> 5) : r;
  }
};

// How the last four topics of a draw are told apart.  Reload: the lane that
// found the leaf reads it again (one cache line per token, against G / 8 per
// token for the tile).  Groups of 4 and 8 lanes with 4-topic leaves (K <= 32)
// write each leaf's running sums after one, two and three topics to LDS in the
// tile and read the chosen leaf's there.  With KEEP, groups of 16 and 32 keep
// them in registers until the tile has been searched, and the lane that holds
// the leaf hands them over through LDS (in the modes that have the registers:
// one document; for groups of 16 also any).
enum GroupLast : int { kReload = 0, kKeepInLds = 1, kKeepInRegs = 2 };
template <int G, int H, bool KEEP, int MODE>
constexpr int kGroupLast =
    H != 1 ? kReload
           : (G <= 8 ? kKeepInLds
                     : (KEEP && (MODE == kGroupOne || (G == 16 && MODE == kGroupAny))
                            ? kKeepInRegs
                            : kReload));

// LDS bytes per wavefront: the tile's leaf sums (and in their place, once
// searched, the leaves and sums handed over), then the kept sums (12 bytes per
// token and leaf, rows padded by one leaf against bank conflicts) or, where
// leaves are reloaded, the staged theta leaves of up to kMaxGroupRuns<G> runs.
// Groups of 8 lanes transpose their leaf sums in registers.
template <int G>
constexpr int kSumFloats = G == 8 ? 0 : GroupTile<G>::kFloats;
// Tokens whose documents are scattered (see spread_draw): groups that take
// them by document class, the classes (XCDs), and the doc ids read at a time.
template <int G, int H>
constexpr bool kSpread = G >= 32 && H == 1;
constexpr int kSpreadClasses = 8;
constexpr int kSpreadBatch = 4;
constexpr int kSpreadRing = (kSpreadBatch + 1) * kWave;  // listed tokens, 16 bits each
constexpr int kSpreadNear = 16;   // documents apart that count as near
constexpr int kSpreadFalls = 24;  // of 64 tokens, far falls of ordered ones at most
constexpr int kSpreadShare = 2;   // of 64 tokens, those of one class's document at most
template <int G, int H>
constexpr int group_lds_bytes() {
  constexpr bool lds = kGroupLast<G, H, false, kGroupOne> == kKeepInLds;
  return (kSumFloats<G> + (lds ? kWave * (G + 1) * 3 : 0)) * (int)sizeof(float) +
         (lds ? 0 : kMaxGroupRuns<G> * H * kWave * (int)sizeof(f4)) +
         (kSpread<G, H> ? kSpreadRing * (int)sizeof(uint16_t) : 0);
}

using f3 = float __attribute__((ext_vector_type(3)));

// A leaf of L = 4 H consecutive topics: H 16-byte quads.
template <int H>
struct Leaf {
  f4 q[H];
};

// Sum of the leaf's L theta-phi products, in topic order (the first a
// product, the others fused multiply-adds onto the running sum).
template <int H>
__device__ __forceinline__ float leaf_dot(const Leaf<H> &t, const Leaf<H> &p) {
  float s = dot4(t.q[0], p.q[0]);
#pragma unroll
  for (int h = 1; h < H; ++h) {
    s = __builtin_fmaf(t.q[h].x, p.q[h].x, s);
    s = __builtin_fmaf(t.q[h].y, p.q[h].y, s);
    s = __builtin_fmaf(t.q[h].z, p.q[h].z, s);
    s = __builtin_fmaf(t.q[h].w, p.q[h].w, s);
  }
  return s;
}

// Value of x in lane J of this lane's quad (J = 0 .. 3) or pair (PARTS = 2, J
// = 0, 1), by a DPP quad permutation.
template <int PARTS, int J>
__device__ __forceinline__ float part_value(float x) {
  constexpr int ctrl = PARTS == 4 ? J * 0x55 : (J == 0 ? 0xA0 : 0xF5);
  return as_float(__builtin_amdgcn_mov_dpp(as_int(x), ctrl, 0xF, 0xF, true));
}

// Exchange between lanes l and l xor BIT (1 or 2, inside a quad): lanes with
// BIT clear receive the partner's x in y, lanes with BIT set the partner's y in
// x (half_swap for the bits that DPP bank masks cannot pick).
template <int BIT>
__device__ __forceinline__ void quad_swap(float &x, float &y) {
  const bool hi = (lane_id() & BIT) != 0;
  const float got = xor_lane<BIT>(hi ? x : y);
  x = hi ? got : x;
  y = hi ? y : got;
}

// x moved by one DPP control.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
}

// Lane J of each half row of 8 lanes: row_newbcast of lane J, then of lane 8 +
// J into the upper two banks.
template <int J>
__device__ __forceinline__ uint32_t half_row_bcast(uint32_t x) {
  const int lo = __builtin_amdgcn_mov_dpp((int)x, 0x150 + J, 0xF, 0xF, true);
  return (uint32_t)__builtin_amdgcn_update_dpp(lo, (int)x, 0x158 + J, 0xF, 0xC, false);
}

// Value held by lane k mod 16 of this lane's row of 16 (G = 16, 32), or by lane
// k of this lane's group of G < 16, in every lane: DPP row broadcasts, for G =
// 8 one per half row (bank masks), for G = 4 one per quad.
template <int G>
__device__ __forceinline__ uint32_t group_row(uint32_t x, int k) {
  if constexpr (G == 4) {
    switch (k & 3) {
      case 0: return dpp_u32<0x00>(x);
      case 1: return dpp_u32<0x55>(x);
      case 2: return dpp_u32<0xAA>(x);
      default: return dpp_u32<0xFF>(x);
    }
  } else if constexpr (G == 8) {
    switch (k & 7) {
      case 0: return half_row_bcast<0>(x);
      case 1: return half_row_bcast<1>(x);
      case 2: return half_row_bcast<2>(x);
      case 3: return half_row_bcast<3>(x);
      case 4: return half_row_bcast<4>(x);
      case 5: return half_row_bcast<5>(x);
      case 6: return half_row_bcast<6>(x);
      default: return half_row_bcast<7>(x);
    }
  } else {
    switch (k & 15) {
      case 0: return dpp_u32<0x150>(x);
      case 1: return dpp_u32<0x151>(x);
      case 2: return dpp_u32<0x152>(x);
      case 3: return dpp_u32<0x153>(x);
      case 4: return dpp_u32<0x154>(x);
      case 5: return dpp_u32<0x155>(x);
      case 6: return dpp_u32<0x156>(x);
      case 7: return dpp_u32<0x157>(x);
      case 8: return dpp_u32<0x158>(x);
      case 9: return dpp_u32<0x159>(x);
      case 10: return dpp_u32<0x15A>(x);
      case 11: return dpp_u32<0x15B>(x);
      case 12: return dpp_u32<0x15C>(x);
      case 13: return dpp_u32<0x15D>(x);
      case 14: return dpp_u32<0x15E>(x);
      default: return dpp_u32<0x15F>(x);
    }
  }
}

// What every token of the wavefront brings: handles of its rows, its uniform
// and the run of documents it belongs to, in the lane that owns the token.
struct GroupTokens {
  uint32_t ph_lane, th_lane;
  float u;
  int run;
  bool store;
  int at;      // the token's place after the window's first (its lane, unless
               // the tokens are listed)
};

// A token whose leaf is known and whose leaf's factors are on their way.
template <int H>
struct GroupFound {
  Leaf<H> th, ph;
  float low, stop;
  int leaf;         // the leaf (of the row)
  int first;        // padded index of the leaf's first topic
  int slot;         // the token's place in the tile
  bool who;         // this lane's part of the token holds u * S
  int32_t *z;       // where the draw goes
  bool mine;        // this lane stores it
  uint32_t ph_row, th_row;  // the token's rows, run and lane (for the reload)
  int run, owner;
};

// Search of one tile: the P lanes of each token agree on the lane, quad and
// leaf that hold u * S.  `sums`: the tile's leaf sums in LDS.
template <int G, int H, int MODE, bool LISTED>
__device__ __forceinline__ GroupFound<H> group_search(const GroupTokens &tok, const float *sums,
                                                      int tile, int c0, int32_t *z) {
  using S = GroupTile<G>;
  constexpr int P = S::kParts;
  const int lane = lane_id();
  const int t = lane / P, p = lane % P;       // token of the tile, part
  const int g = t / S::kLoads, j = t % S::kLoads;
  const int owner = g * G + tile * S::kLoads + j;  // lane that owns the token
  // the token's values, from the lane that owns it (this one with P = 1)
  GroupTokens my = tok;
  if constexpr (P > 1) {
    const int a = owner << 2;
    my.ph_lane = (uint32_t)__builtin_amdgcn_ds_bpermute(a, (int)tok.ph_lane);
    my.u = as_float(__builtin_amdgcn_ds_bpermute(a, as_int(tok.u)));
    if constexpr (MODE == kGroupAny)
      my.th_lane = (uint32_t)__builtin_amdgcn_ds_bpermute(a, (int)tok.th_lane);
    if constexpr (MODE == kGroupRuns) my.run = __builtin_amdgcn_ds_bpermute(a, tok.run);
    const uint64_t stores = __builtin_amdgcn_ballot_w64(tok.store);
    my.store = (stores >> owner) & 1;
    my.at = LISTED ? __builtin_amdgcn_ds_bpermute(a, tok.at) : owner;
  }
  const float *row = sums + g * S::kGroup + j * S::kRow + S::leaf(p * S::kLeaves);
  float q[S::kQuads];
#pragma unroll
  for (int i = 0; i < S::kQuads; ++i) {
    const f4 x = *reinterpret_cast<const f4 *>(row + 4 * i);
    q[i] = (x.x + x.y) + (x.z + x.w);
  }
  // prefixes of the quads inside this lane's part, then of the parts
  float pre[S::kQuads + 1];
  pre[0] = 0.0f;
#pragma unroll
  for (int i = 0; i < S::kQuads; ++i) pre[i + 1] = i == 0 ? q[0] : pre[i] + q[i];
  const float part = pre[S::kQuads];
  GroupFound<H> f;
  float base = 0.0f, total;
  int who = 0;  // the part that holds u * S: the last if none is above it
  if constexpr (P == 1) {
    total = part;
    f.stop = total * my.u;
  } else if constexpr (P == 2) {
    const float e0 = part_value<2, 0>(part);
    total = e0 + part_value<2, 1>(part);
    f.stop = total * my.u;
    who = f.stop < e0 ? 0 : 1;
    base = p ? e0 : 0.0f;
  } else {
    const float e0 = part_value<4, 0>(part);
    const float e1 = e0 + part_value<4, 1>(part);
    const float e2 = e1 + part_value<4, 2>(part);
    total = e2 + part_value<4, 3>(part);
    f.stop = total * my.u;
    who = f.stop < e0 ? 0 : f.stop < e1 ? 1 : f.stop < e2 ? 2 : 3;
    base = p == 0 ? 0.0f : p == 1 ? e0 : p == 2 ? e1 : e2;
  }
  f.who = p == who;
  f.mine = my.store && f.who;
  // the quad of leaves, then the leaf
  f.low = base;
  int quad = 0;
#pragma unroll
  for (int i = 1; i < S::kQuads; ++i) {
    const float at = base + pre[i];
    const bool past = !(f.stop < at);
    f.low = past ? at : f.low;
    quad = past ? i : quad;
  }
  const f4 x = *reinterpret_cast<const f4 *>(row + 4 * quad);
  const float a1 = f.low + x.x, a2 = f.low + (x.x + x.y), a3 = f.low + ((x.x + x.y) + x.z);
  int leaf = p * S::kLeaves + 4 * quad;
  const bool p1 = !(f.stop < a1), p2 = !(f.stop < a2), p3 = !(f.stop < a3);
  f.low = p3 ? a3 : p2 ? a2 : p1 ? a1 : f.low;
  leaf += p3 ? 3 : p2 ? 2 : p1 ? 1 : 0;
  f.leaf = leaf;
  f.first = c0 + kLeaf * H * leaf;
  f.slot = t;
  f.z = z + my.at;
  f.ph_row = my.ph_lane;
  f.th_row = my.th_lane;
  f.run = MODE == kGroupRuns ? my.run : 0;
  f.owner = owner;
  return f;
}

// The same for groups of 8 lanes: a[k] is this lane's leaf sum of token k of
// its group.  Three exchanges across lane bits 2, 1 and 0 transpose the 8 x 8
// sums in registers, so that each lane scans its own token's.
template <int H>
__device__ __forceinline__ GroupFound<H> group8_search(const GroupTokens &tok, float (&a)[8],
                                                       int c0, int32_t *z) {
  const int lane = lane_id();
#pragma unroll
  for (int k = 0; k < 4; ++k) half_swap<4>(a[k], a[k + 4]);
#pragma unroll
  for (int k = 0; k < 8; k += 4) {
    quad_swap<2>(a[k], a[k + 2]);
    quad_swap<2>(a[k + 1], a[k + 3]);
  }
#pragma unroll
  for (int k = 0; k < 8; k += 2) quad_swap<1>(a[k], a[k + 1]);
  // prefixes at the leaves' ends; an end that is not above u * S is passed
  float end[8];
  end[0] = a[0];
#pragma unroll
  for (int i = 1; i < 8; ++i) end[i] = end[i - 1] + a[i];
  GroupFound<H> f;
  f.stop = end[7] * tok.u;
  f.low = 0.0f;
  f.leaf = 0;
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    const bool past = !(f.stop < end[i]);
    f.low = past ? end[i] : f.low;
    f.leaf = past ? i + 1 : f.leaf;
  }
  f.first = c0 + kLeaf * H * f.leaf;
  f.slot = lane;
  f.who = true;
  f.mine = tok.store;
  f.z = z + tok.at;
  f.ph_row = tok.ph_lane;
  f.th_row = tok.th_lane;
  f.run = tok.run;
  f.owner = lane;
  return f;
}

// The factors of a found leaf, in the lane that found it: phi reloaded, theta
// from the staged leaves or reloaded.
template <int G, int H, int MODE, bool PAD>
__device__ __forceinline__ void group_reload(GroupFound<H> &f, const Table &th_t,
                                             const Table &ph_t, const f4 *stage, int drop) {
  if (!f.mine) return;
  const int gb = (f.owner & ~(G - 1)) + f.leaf;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int i = f.first + kLeaf * h;
    const int topic = PAD ? (i >= kLeaf ? i - drop : 0) : i;
    const uint32_t off = (uint32_t)topic * 4u;
    f.ph.q[h] = ph_t.ld4v(off, f.ph_row);
    if constexpr (MODE == kGroupAny) {
      f.th.q[h] = th_t.ld4v(off, f.th_row);
      if constexpr (PAD) {
        // components past the topics the quad holds (see above)
        const int real = i < 0 ? 0 : (i < kLeaf ? kLeaf - drop : kLeaf);
#pragma unroll
        for (int e = 0; e < kLeaf; ++e)
          if (e >= real) f.th.q[h][e] = 0.0f;
      }
    } else {
      f.th.q[h] = stage[((MODE == kGroupRuns ? f.run : 0) * H + h) * kWave + gb];
    }
  }
}

// Topic of padded index i.  The first quad's empty components hold a draw only
// by rounding: its last topic.  The empty leaves before it (i < 0) hold none,
// unless u or a weight is negative, which is no draw at all: topic 0, so that
// what is stored always indexes a topic.
template <bool PAD>
__device__ __forceinline__ int group_topic(int i, int drop) {
  return PAD ? max(max(i - drop, min(i, kLeaf - 1 - drop)), 0) : i;
}

// The topic of a found token: the first of its leaf's L topics whose running
// sum exceeds u * S, else the last.
template <int H, bool PAD>
__device__ __forceinline__ void group_finish(const GroupFound<H> &f, int drop) {
  constexpr int L = kLeaf * H;
  if (!f.mine) return;
  float sum = f.low;
  int i = L - 1;
#pragma unroll
  for (int h = 0; h < H; ++h) {
#pragma unroll
    for (int e = 0; e < kLeaf; ++e) {
      const int idx = kLeaf * h + e;
      if (idx == L - 1) break;  // the leaf's last topic needs no comparison
      sum = __builtin_fmaf(f.th.q[h][e], f.ph.q[h][e], sum);
      if (i == L - 1 && f.stop < sum) i = idx;
    }
  }
  *f.z = group_topic<PAD>(f.first + i, drop);
}

// The topic of a found token from its leaf's running sums after one, two and
// three topics (nondecreasing: the products are not negative).
template <bool PAD>
__device__ __forceinline__ void group_store_kept(const GroupFound<1> &f, float s0, float s1,
                                                 float s2, int drop) {
  const int i = f.stop < f.low + s0 ? 0 : f.stop < f.low + s1 ? 1 : f.stop < f.low + s2 ? 2 : 3;
  if (f.mine) *f.z = group_topic<PAD>(f.first + i, drop);
}

// The running sums kept in registers: lane r of group g holds those of
// leaf r for the tile's tokens g NLD + k in kept[k]; the lane whose leaf a
// token ended in writes them for the lane that searched the token.
template <int G, bool PAD>
__device__ __forceinline__ void group_finish_kept(const GroupFound<1> &f,
                                                  const f3 (&kept)[GroupTile<G>::kLoads],
                                                  float *sums, int drop) {
  using S = GroupTile<G>;
  static_assert(kWave + 4 * S::kTokens <= kSumFloats<G>, "leaves and slots take the sums' place");
  const int lane = lane_id(), r = lane & (G - 1), g = lane / G;
  int *leaves = reinterpret_cast<int *>(sums);
  f3 *slots = reinterpret_cast<f3 *>(sums + kWave);  // (16 bytes each)
  if (f.who) leaves[f.slot] = f.leaf;
  lds_order();
#pragma unroll
  for (int i = 0; i < S::kLoads / 4; ++i) {
    const int4 q = *reinterpret_cast<const int4 *>(leaves + g * S::kLoads + 4 * i);
    const int at = g * S::kLoads + 4 * i;
    if (q.x == r) slots[at] = kept[4 * i];
    if (q.y == r) slots[at + 1] = kept[4 * i + 1];
    if (q.z == r) slots[at + 2] = kept[4 * i + 2];
    if (q.w == r) slots[at + 3] = kept[4 * i + 3];
  }
  lds_order();
  const f3 s = slots[f.slot];
  group_store_kept<PAD>(f, s.x, s.y, s.z, drop);
}

// The tiles of a wavefront: leaf sums, search and topics of its 64 tokens.
// voff[h]: byte offset of quad h of this lane's leaf in a row; real[h]: the
// topics it holds, in its first components (0: front padding).  NK: the tokens
// of a group (its first NK lanes').
template <int G, int H, int C, bool KEEP, int MODE, bool PAD, bool LISTED = false, int NK = G>
__device__ __forceinline__ void group_tiles(const Table &th_t, const Table &ph_t,
                                            const uint32_t (&voff)[H], const int (&real)[H],
                                            const GroupTokens &tok, int gbase, uint64_t gstarts,
                                            float *sums, f4 *stage, int c0, int drop,
                                            int32_t *z) {
  using S = GroupTile<G>;
  static_assert(NK % C == 0 && NK % S::kLoads == 0, "the window size must divide NK");
  constexpr int LAST = kGroupLast<G, H, KEEP, MODE>;
  constexpr int R = MODE == kGroupRuns ? kMaxGroupRuns<G> : 1;
  const int lane = lane_id(), r = lane & (G - 1);
  // Leaf of token k of the group.  `rows` holds the row handles: with G = 64
  // this lane's token's (token k's is uniform and goes in the scalar offset),
  // with G = 8 and 16 too (token k's comes from its lane by a DPP row
  // broadcast, no LDS round trip before the load), with G = 32 those of the
  // tile's 16 tokens, in every row of 16 lanes of the group (rows_of_tile).
  const auto leaf_of = [&](const Table &t, uint32_t rows, int k) {
    Leaf<H> l;
    if constexpr (G == kWave) {
      const uint32_t srow = (uint32_t)__builtin_amdgcn_readlane((int)rows, k);
#pragma unroll
      for (int h = 0; h < H; ++h) l.q[h] = t.ld4(voff[h], srow);
    } else {
      const uint32_t vrow = group_row<G>(rows, k);
#pragma unroll
      for (int h = 0; h < H; ++h) l.q[h] = t.ld4v(voff[h], vrow);
    }
    return l;
  };
  constexpr int NT = G == 32 ? S::kTiles : 1;
  uint32_t ph_rows[NT], th_rows[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    ph_rows[i] = tok.ph_lane;
    th_rows[i] = tok.th_lane;
    if constexpr (G == 32) {
      const int from = (gbase + i * S::kLoads + (lane & 15)) << 2;
      ph_rows[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)tok.ph_lane);
      if constexpr (MODE != kGroupOne)
        th_rows[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)tok.th_lane);
    }
  }
  const auto ph_leaf = [&](int k) { return leaf_of(ph_t, ph_rows[G == 32 ? k / S::kLoads : 0], k); };
  const auto th_leaf = [&](int k) { return leaf_of(th_t, th_rows[G == 32 ? k / S::kLoads : 0], k); };
  const auto mask = [&](Leaf<H> l) {
    if constexpr (PAD) {
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int e = 0; e < kLeaf; ++e) l.q[h][e] = e < real[h] ? l.q[h][e] : 0.0f;
    }
    return l;
  };
  // kGroupRuns: gstarts bit p (0 < p < G) marks the group's token p as the
  // first of a run; run j's leaf is that of the token opening it
  Leaf<H> th[R];
  if constexpr (MODE == kGroupOne) {
    Leaf<H> l;
#pragma unroll
    for (int h = 0; h < H; ++h) l.q[h] = th_t.ld4v(voff[h], tok.th_lane);
    th[0] = mask(l);
  } else if constexpr (MODE == kGroupRuns) {
    uint64_t m = gstarts;
    th[0] = mask(th_leaf(0));
#pragma unroll
    for (int j = 1; j < R; ++j) {
      const int p = m ? (int)__builtin_ctzll(m) : 0;
      m &= m - 1;
      Leaf<H> l;
      const uint32_t row = (uint32_t)__builtin_amdgcn_ds_bpermute((gbase + p) << 2, (int)tok.th_lane);
#pragma unroll
      for (int h = 0; h < H; ++h) l.q[h] = th_t.ld4v(voff[h], row);
      th[j] = mask(l);
    }
  }
  Leaf<H> win[C];
#pragma unroll
  for (int k = 0; k < C; ++k) win[k] = ph_leaf(k);
  if constexpr (MODE != kGroupAny && LAST == kReload) {
    // stage the runs' leaves: quad h of run j at stage[(j H + h) 64 + lane]
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int h = 0; h < H; ++h) stage[(j * H + h) * kWave + lane] = th[j].q[h];
    lds_order();
  }
  const auto run_of = [&](int k) {
    // runs opened at the group's tokens 1 .. k
    const uint64_t upto = k == 63 ? ~0ull : ((2ull << k) - 1ull);
    return __builtin_popcountll(gstarts & upto);
  };
  const auto staged = [&](int k) {
    Leaf<H> l;
    const int base = run_of(k) * H * kWave + lane;
#pragma unroll
    for (int h = 0; h < H; ++h) l.q[h] = stage[base + h * kWave];
    return l;
  };
  constexpr bool STAGED = MODE == kGroupRuns && kStageRuns<G>;
  constexpr int CT = MODE == kGroupAny ? C : (STAGED ? kRunAhead : 1);
  Leaf<H> twin[CT];
  if constexpr (MODE == kGroupAny) {
#pragma unroll
    for (int k = 0; k < C; ++k) twin[k] = th_leaf(k);
  }
  if constexpr (STAGED) {
#pragma unroll
    for (int k = 0; k < CT; ++k) twin[k] = staged(k);
  }
  // this lane's place in the rows of its group's tokens
  float *put = sums + (gbase / G) * S::kGroup + S::leaf(r);
  GroupFound<H> found{};
  f3 kept[S::kLoads];  // kKeepInRegs: the running sums of this lane's leaf
  float a[G == 8 ? G : 1];  // G = 8: the leaf sums
  // kKeepInLds: the running sums after one and two topics, and three
  f2 *keep2 = reinterpret_cast<f2 *>(sums + kSumFloats<G>);
  float *keep1 = sums + kSumFloats<G> + 2 * kWave * (G + 1);
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    Leaf<H> tv;
    if constexpr (MODE == kGroupAny) {
      tv = mask(twin[k % C]);
    } else if constexpr (STAGED) {
      tv = twin[k % CT];
    } else if constexpr (MODE == kGroupRuns) {
      const int j = run_of(k);
      tv = th[0];
#pragma unroll
      for (int i = 1; i < R; ++i)
#pragma unroll
        for (int h = 0; h < H; ++h) tv.q[h] = j == i ? th[i].q[h] : tv.q[h];
    } else {
      tv = th[0];
    }
    float sum;
    if constexpr (LAST != kReload) {
      // leaf_dot's steps, every sum kept
      const f4 t = tv.q[0], x = win[k % C].q[0];
      f4 s;
      s.x = t.x * x.x;
      s.y = __builtin_fmaf(t.y, x.y, s.x);
      s.z = __builtin_fmaf(t.z, x.z, s.y);
      s.w = __builtin_fmaf(t.w, x.w, s.z);
      sum = s.w;
      if constexpr (LAST == kKeepInRegs) {
        kept[k % S::kLoads] = f3{s.x, s.y, s.z};
      } else {
        const int at = (gbase + k) * (G + 1) + r;
        keep2[at] = f2{s.x, s.y};
        keep1[at] = s.z;
      }
    } else {
      sum = leaf_dot(tv, win[k % C]);
    }
    if constexpr (G == 8)
      a[k] = sum;
    else
      put[(k % S::kLoads) * S::kRow] = sum;
    if (k + C < NK) {
      win[k % C] = ph_leaf(k + C);
      if constexpr (MODE == kGroupAny) twin[k % C] = th_leaf(k + C);
    }
    if constexpr (STAGED)
      if (k + CT < NK) twin[k % CT] = staged(k + CT);
    __builtin_amdgcn_sched_barrier(0);
    if ((k + 1) % S::kLoads == 0) {
      // The tile's search; its reload is in flight while the next tile's
      // leaves are summed (whose first C loads were issued before it).
      lds_order();
      GroupFound<H> now;
      if constexpr (G == 8)
        now = group8_search<H>(tok, a, c0, z);
      else
        now = group_search<G, H, MODE, LISTED>(tok, sums, k / S::kLoads, c0, z);
      if constexpr (LAST == kKeepInRegs) {
        lds_order();
        group_finish_kept<G, PAD>(now, kept, sums, drop);
      } else if constexpr (LAST == kKeepInLds) {
        const int at = lane * (G + 1) + now.leaf;
        const f2 s01 = keep2[at];
        group_store_kept<PAD>(now, s01.x, s01.y, keep1[at], drop);
      } else {
        group_reload<G, H, MODE, PAD>(now, th_t, ph_t, stage, drop);
        if (k >= S::kLoads) group_finish<H, PAD>(found, drop);
        found = now;
      }
      lds_order();
    }
  }
  if constexpr (LAST == kReload) group_finish<H, PAD>(found, drop);
}

// What a lane's leaf needs of a row: padded index of the first leaf's first
// topic, empty components of the first quad, and per quad of this lane's leaf
// its byte offset and the topics it holds.
template <int H>
struct GroupLeaf {
  int c0, drop;
  uint32_t voff[H];
  int real[H];
};
template <int G, int H, bool PAD>
__device__ __forceinline__ GroupLeaf<H> group_leaf(int K, int r) {
  GroupLeaf<H> l;
  l.drop = PAD ? (-K) & (kLeaf - 1) : 0;
  l.c0 = K + l.drop - kLeaf * H * G;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int i = l.c0 + kLeaf * H * r + kLeaf * h;
    l.real[h] = !PAD || i >= kLeaf ? kLeaf : (i < 0 ? 0 : kLeaf - l.drop);
    l.voff[h] = (uint32_t)(!PAD ? i : (i >= kLeaf ? i - l.drop : 0)) * 4u;
  }
  return l;
}

// Whether a stretch's documents are scattered, from its first 64 tokens' (d: this
// lane's token's): they fall far at two tokens of five (shuffled ones at every
// other).  Short documents in order change at every token but never fall, and
// the documents of a word, where tokens stand word by word, fall once a word:
// listed by class, such tokens took 1.2-1.4 times the plain draw's time (2M
// tokens, one per document, K = 100 ... 256) and 1.1-1.35 times (word by word, K =
// 100 ... 160).  Nor do shuffled tokens fall that often where one document has
// half of them, for which the plain draw is the faster one too.
__device__ __forceinline__ bool scattered(int d) {
  const int p = __builtin_amdgcn_update_dpp(d, d, 0x138, 0xF, 0xF, false);
  const bool fall = d < p && (uint32_t)p - (uint32_t)d > (uint32_t)kSpreadNear;
  return __builtin_popcountll(__builtin_amdgcn_ballot_w64(fall)) > kSpreadFalls;
}

// Up to two documents that more than kSpreadShare of those 64 tokens share (-1:
// none).  Their tokens go to all classes by turns: one class, and so one XCD,
// would otherwise draw a large document alone (20% of shuffled tokens in one
// document: 1.2-1.8 times the plain draw's time, by turns 0.8-1).  Ten bits of a
// hash tell documents apart: three of 64 agree by chance in one stretch of 25,
// which does no harm.
struct LargeDocs {
  int d0, d1;
};
__device__ __forceinline__ LargeDocs large_docs(int d) {
  const uint32_t h = (uint32_t)d * 2654435761u;
  uint64_t same = ~0ull;  // the lanes of this lane's document
#pragma unroll
  for (int b = 22; b < 32; ++b) {
    const bool bit = (h >> b) & 1u;
    const uint64_t set = __builtin_amdgcn_ballot_w64(bit);
    same &= bit ? set : ~set;
  }
  const uint64_t large = __builtin_amdgcn_ballot_w64(__builtin_popcountll(same) > kSpreadShare);
  LargeDocs l{-1, -1};
  if (large == 0) return l;
  l.d0 = __builtin_amdgcn_readlane(d, __builtin_ctzll(large));
  const uint64_t rest = large & ~__builtin_amdgcn_ballot_w64(d == l.d0);
  if (rest) l.d1 = __builtin_amdgcn_readlane(d, __builtin_ctzll(rest));
  return l;
}

// Tokens whose documents are scattered (shuffled tokens): theta rows, like phi
// rows, then come from all over their table in every XCD, and misses past L2
// bound the draw.  Eight workgroups, one per XCD (workgroup b runs on XCD b
// mod 8), share a stretch of tokens instead: each wavefront reads the doc ids
// of its share of the stretch, lists the tokens whose document's class is its
// workgroup's, and draws them 64 at a time, so that an XCD's L2 holds one
// eighth of theta.  Measured on MI355X, tokens shuffled: 2M tokens, V = 50,000,
// theta of 8 MiB at K = 128 172 -> 142 us, of 12.5 MiB at K = 200 317 -> 233;
// 1M tokens, 16 MiB at K = 256 189 -> 139; tokens in document order within 1%
// (the check's doc ids are loaded with the wavefront's own).  `ids`, `word_id`,
// `z`: from the share's first token on; `first`: its index, for `u`.
template <int G, int H, int C, bool KEEP, bool PAD>
__device__ __forceinline__ void spread_draw(const Table &th_t, const Table &ph_t,
                                            const int32_t *ids, const int32_t *word_id,
                                            const UniformSource &u, int64_t first, int tokens,
                                            uint32_t cls, LargeDocs large,
                                            const GroupLeaf<H> &leaf, float *sums, f4 *stage,
                                            uint16_t *ring, int32_t *z) {
  const int lane = lane_id(), gbase = lane & ~(G - 1);
  const uint64_t below = (1ull << lane) - 1ull;
  constexpr int step = kSpreadBatch * kWave;
  int32_t doc[kSpreadBatch];
  const auto load = [&](int from) {
#pragma unroll
    for (int i = 0; i < kSpreadBatch; ++i) {
      const int at = from + i * kWave + lane;
      doc[i] = at < tokens ? ids[at] : 0;
    }
  };
  load(0);
  int have = 0;  // listed tokens not yet drawn
  int from = 0;
  while (true) {
    while (have < kWave && from < tokens) {
#pragma unroll
      for (int i = 0; i < kSpreadBatch; ++i) {
        const int at = from + i * kWave + lane;
        uint32_t c = ((uint32_t)doc[i] * 2654435761u) >> 29;
        if (large.d0 >= 0 && (doc[i] == large.d0 || doc[i] == large.d1))
          c = (uint32_t)at % kSpreadClasses;
        const bool mine = at < tokens && c == cls;
        const uint64_t picks = __builtin_amdgcn_ballot_w64(mine);
        if (mine) ring[have + __builtin_popcountll(picks & below)] = (uint16_t)at;
        have += __builtin_popcountll(picks);
      }
      from += step;
      if (from < tokens) load(from);  // (in flight during the next window)
      lds_order();
    }
    if (have == 0) return;
    const int take = have < kWave ? have : kWave;
    have -= take;
    GroupTokens tok;
    tok.at = ring[have + (lane < take ? lane : take - 1)];
    tok.store = lane < take;
    tok.ph_lane = ph_t.row((uint32_t)word_id[tok.at]);
    tok.th_lane = th_t.row((uint32_t)ids[tok.at]);
    tok.u = u(first + tok.at);
    tok.run = 0;
    group_tiles<G, H, C, KEEP, kGroupAny, PAD, true>(th_t, ph_t, leaf.voff, leaf.real, tok, gbase,
                                                     0, sums, stage, leaf.c0, leaf.drop, z);
    lds_order();
  }
}

// L = 4 H topics per lane: groups of G lanes cover 4 H G topics.  A wavefront
// draws TOK tokens: 64, or for 64-lane groups 16, one tile (fewer_tokens).
template <int G, int H, int C, int WPEU, bool KEEP, bool PAD, int TOK = kWave>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(WPEU)))
void leaf_group_kernel(const float *__restrict__ theta, const float *__restrict__ phi,
                       DocSource docs, const int32_t *__restrict__ word_id,
                       UniformSource u, int32_t *__restrict__ z, int64_t N, int K,
                       uint32_t theta_extent, uint32_t phi_extent, int spread) {
  extern __shared__ __align__(16) float lds[];
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  float *sums = lds + wave * (group_lds_bytes<G, H>() / (int)sizeof(float));
  f4 *stage = reinterpret_cast<f4 *>(sums + kSumFloats<G>);
  const int64_t first = ((int64_t)blockIdx.x * kWavesPerBlock + wave) * TOK;
  const int r = lane & (G - 1), gbase = lane & ~(G - 1);
  // Window of TOK tokens as in butterfly_kernel (N >= 64 here); lanes past it
  // repeat the last token.
  static_assert(TOK == kWave || (G == kWave && TOK == GroupTile<G>::kTokens), "whole tiles");
  const int64_t t0 = first + TOK <= N ? first : N - TOK;
  GroupTokens tok;
  const int64_t n = t0 + (TOK == kWave ? lane : min(lane, TOK - 1));
  tok.at = lane;
  tok.store = n >= first && lane < TOK;
  int doc = docs.ids ? docs.ids[n] : 0;
  const int word = word_id[n];
  tok.u = u(n);
  // Windows of the modes that keep their sums in registers: for groups of 16
  // all 16 tokens in one document (the sums take the loaded leaves' place),
  // fewer where theta comes per token too.
  constexpr bool K16 = G == 16 && H == 1 && KEEP;
  constexpr int C1 = K16 ? G : C;
  constexpr int CA = K16 ? (PAD ? 2 : 4) : (G == kWave && H == 1 ? C / 2 : C);
  if constexpr (kSpread<G, H> && TOK == kWave) {
    // spread: log2 of the tokens per wavefront's share of a stretch (0: never).
    // A stretch of scattered documents is drawn by eight of its workgroups; the
    // others are done.
    const int64_t stretch = (int64_t)kWavesPerBlock << spread;
    const int shift = spread ? spread - 6 : 0;  // log2 of a stretch's workgroups
    const uint32_t index = blockIdx.x >> shift;
    const int64_t s0 = index * stretch;
    // (a last, incomplete stretch may have fewer than eight workgroups)
    if (spread && s0 + stretch <= N) {
      const int d = docs.ids[s0 + lane];
      if (scattered(d)) {
        // (a stretch's eight by turns: an XCD's CUs get workgroups round robin)
        const uint32_t part = blockIdx.x & ((1u << shift) - 1u);
        const uint32_t turns = (1u << shift) / kSpreadClasses;
        if (part / kSpreadClasses != (index & (turns - 1u))) return;
        const int64_t lo = s0 + ((int64_t)wave << spread);
        // (a window of 2 where 4 would not fit the registers)
        constexpr int CS = G == 32 && !KEEP && !PAD ? 2 : CA;
        spread_draw<G, H, CS, KEEP, PAD>(
            make_table(theta, theta_extent, K), make_table(phi, phi_extent, K), docs.ids + lo,
            word_id + lo, u, lo, 1 << spread, part % kSpreadClasses, large_docs(d),
            group_leaf<G, H, PAD>(K, r), sums, stage,
            reinterpret_cast<uint16_t *>(stage + kMaxGroupRuns<G> * H * kWave), z + lo);
        return;
      }
    }
  }
  if (first >= N) return;  // whole wavefront past the end
  if (!docs.ids) doc = docs.wave_doc(n, t0, t0 + TOK - 1);
  z += t0;

  const Table th_t = make_table(theta, theta_extent, K);
  const Table ph_t = make_table(phi, phi_extent, K);
  tok.ph_lane = ph_t.row((uint32_t)word);
  tok.th_lane = th_t.row((uint32_t)doc);
  const GroupLeaf<H> leaf = group_leaf<G, H, PAD>(K, r);
  // runs of documents inside each group: bit l of `starts` marks lane l's
  // token as the first of a run (not counting the group's first token)
  // (lane l's previous document by a DPP wavefront shift right by one lane:
  // no LDS round trip before the first loads; lane 0 keeps its own)
  const int prev = __builtin_amdgcn_update_dpp(doc, doc, 0x138, 0xF, 0xF, false);
  const uint64_t starts = __builtin_amdgcn_ballot_w64(r != 0 && doc != prev);
  const uint64_t gmask = G == kWave ? ~0ull : ((1ull << G) - 1ull);
  const uint64_t gstarts = (starts >> gbase) & gmask;  // this lane's group, bit p = token p
  tok.run = __builtin_popcountll(gstarts & ((2ull << r) - 1ull));
  // the most runs in any group (groups of G lanes: at most 64 / G of them)
  int most = 0;
#pragma unroll
  for (int g = 0; g < kWave / G; ++g)
    most = max(most, __builtin_popcountll((starts >> (g * G)) & gmask));

  constexpr int NK = TOK == kWave ? G : TOK;  // tokens of a group
  if (most == 0)
    group_tiles<G, H, C1, KEEP, kGroupOne, PAD, false, NK>(
        th_t, ph_t, leaf.voff, leaf.real, tok, gbase, 0, sums, stage, leaf.c0, leaf.drop, z);
  else if (most < kMaxGroupRuns<G>)
    group_tiles<G, H, C, KEEP, kGroupRuns, PAD, false, NK>(
        th_t, ph_t, leaf.voff, leaf.real, tok, gbase, gstarts, sums, stage, leaf.c0, leaf.drop, z);
  else
    group_tiles<G, H, CA, KEEP, kGroupAny, PAD, false, NK>(
        th_t, ph_t, leaf.voff, leaf.real, tok, gbase, 0, sums, stage, leaf.c0, leaf.drop, z);
}

}  // namespace
}  // namespace LDA_NS
