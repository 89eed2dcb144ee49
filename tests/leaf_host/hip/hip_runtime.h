// A wavefront on the CPU: what the leaf-group kernel uses of HIP and of the
// gfx950 builtins, for a bounds-checked host build (leaf_host.cpp).
//
// The 64 lanes are coroutines run in turn.  A cross-lane operation deposits
// its operand, lets every other lane reach the same operation and then reads
// the others' operands; lds_order's wave barrier is such a point too.  Between
// two of them the lanes run one after another, so LDS data that one lane hands
// to another without an ordering point in between is seen stale here.
#pragma once

#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <algorithm>

namespace emu {

struct Dim {
  unsigned x;
};
inline Dim thread_idx, block_idx, grid_dim;

[[noreturn]] inline void fail(const char *what) {
  fprintf(stderr, "leaf_host: %s (workgroup %u, thread %u)\n", what, block_idx.x, thread_idx.x);
  abort();
}

constexpr int kLanes = 64;
inline ucontext_t scheduler, lane_context[kLanes];
inline int lane_now;              // the lane that runs
inline uint32_t deposit[2][kLanes];
inline const char *reached[2][kLanes];
inline long steps[kLanes];        // cross-lane operations a lane has reached

// Deposit v, wait for the other lanes at the same operation; their deposits.
inline const uint32_t *exchange(uint32_t v, const char *op) {
  const int l = lane_now, b = (int)(steps[l]++ & 1);
  deposit[b][l] = v;
  reached[b][l] = op;
  swapcontext(&lane_context[l], &scheduler);
  for (int i = 0; i < kLanes; ++i)
    if (steps[i] < steps[l] || reached[b][i] != op) fail("lanes at different operations");
  return deposit[b];
}

inline int readlane(int v, int k) {
  if (k < 0 || k >= kLanes) fail("readlane of no lane");
  return (int)exchange((uint32_t)v, "readlane")[k];
}
inline int readfirstlane(int v) { return (int)exchange((uint32_t)v, "readfirstlane")[0]; }
inline int ds_bpermute(int addr, int v) {
  return (int)exchange((uint32_t)v, "ds_bpermute")[(addr >> 2) & (kLanes - 1)];
}
inline int ds_swizzle(int v, int mask) {
  const uint32_t *x = exchange((uint32_t)v, "ds_swizzle");
  const int l = lane_now;
  return (int)x[(l & 32) | (((l & mask & 31) | ((mask >> 5) & 31)) ^ ((mask >> 10) & 31))];
}
inline uint64_t ballot(bool p) {
  const uint32_t *x = exchange(p, "ballot");
  uint64_t m = 0;
  for (int i = 0; i < kLanes; ++i) m |= (uint64_t)(x[i] != 0) << i;
  return m;
}
inline int dpp(int old, int v, int ctrl, int rows, int banks, bool zero) {
  const uint32_t *x = exchange((uint32_t)v, "dpp");
  const int l = lane_now, row = l & ~15, in = l & 15;
  if (!((rows >> (l / 16)) & 1) || !((banks >> (in / 4)) & 1)) return old;
  int from = -1;
  if (ctrl <= 0xFF)
    from = (l & ~3) | ((ctrl >> (2 * (l & 3))) & 3);  // quad permutation
  else if (ctrl > 0x100 && ctrl <= 0x10F)
    from = in + (ctrl & 15) < 16 ? l + (ctrl & 15) : -1;  // row shift left
  else if (ctrl > 0x110 && ctrl <= 0x11F)
    from = in >= (ctrl & 15) ? l - (ctrl & 15) : -1;  // row shift right
  else if (ctrl == 0x138)
    from = l - 1;  // wavefront shift right
  else if (ctrl >= 0x150 && ctrl <= 0x15F)
    from = row + (ctrl & 15);  // row broadcast
  else
    fail("unknown DPP control");
  return from >= 0 ? (int)x[from] : (zero ? 0 : old);
}
inline void wave_barrier() { exchange(0, "wave barrier"); }

// A table read through a buffer resource.  Stricter than the hardware's range
// check: a 16-byte load must lie inside one row of the table.
struct Resource {
  const char *base;
  uint64_t bytes;
};
inline uint64_t row_bytes;
inline Resource make_rsrc(const void *p, int, uint64_t bytes, int) {
  return {static_cast<const char *>(p), bytes};
}
struct Bits128 {
  uint32_t w[4];
};
inline Bits128 load_b128(const Resource &r, uint32_t voff, uint32_t soff, int) {
  const uint64_t off = (uint64_t)voff + soff;
  if (off + 16 > r.bytes || off % row_bytes + 16 > row_bytes) fail("load leaves its row");
  Bits128 v;
  __builtin_memcpy(&v, r.base + off, 16);
  return v;
}
inline uint32_t load_b32(const Resource &, uint32_t, uint32_t, int) { fail("not used here"); }

struct Pair {
  int v[2];
  int operator[](int i) const { return v[i]; }
};
inline Pair permlane_swap(int, int, bool, bool) { fail("not used here"); }

// Run `lane_main` as the 64 lanes of a wavefront.
template <class F>
inline void wavefront(unsigned first_thread, const F &lane_main) {
  static char *stacks = static_cast<char *>(malloc((size_t)kLanes << 18));
  static const F *body;
  static bool done[kLanes];
  body = &lane_main;
  for (int l = 0; l < kLanes; ++l) {
    steps[l] = 0;
    done[l] = false;
    getcontext(&lane_context[l]);
    lane_context[l].uc_stack.ss_sp = stacks + ((size_t)l << 18);
    lane_context[l].uc_stack.ss_size = (size_t)1 << 18;
    lane_context[l].uc_link = &scheduler;
    makecontext(&lane_context[l], static_cast<void (*)()>([] {
                  (*body)();
                  done[lane_now] = true;
                }),
                0);
  }
  while (true) {
    int running = 0;
    for (int l = 0; l < kLanes; ++l)
      if (!done[l]) {
        lane_now = l;
        thread_idx.x = first_thread + (unsigned)l;
        swapcontext(&scheduler, &lane_context[l]);
        running += !done[l];
      }
    if (running == 0) return;
    if (running != kLanes) fail("lanes ended at different operations");
  }
}

}  // namespace emu

#define __device__
#define __host__
#define __global__
#define __shared__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define threadIdx ::emu::thread_idx
#define blockIdx ::emu::block_idx
#define gridDim ::emu::grid_dim
#define amdgpu_waves_per_eu(...) unused
using std::max;
using std::min;
struct alignas(16) int4 {
  int x, y, z, w;
};

#define __amdgpu_buffer_rsrc_t ::emu::Resource
#define __builtin_amdgcn_make_buffer_rsrc ::emu::make_rsrc
#define __builtin_amdgcn_raw_buffer_load_b128 ::emu::load_b128
#define __builtin_amdgcn_raw_buffer_load_b32 ::emu::load_b32
#define __builtin_amdgcn_readlane ::emu::readlane
#define __builtin_amdgcn_readfirstlane ::emu::readfirstlane
#define __builtin_amdgcn_ds_bpermute ::emu::ds_bpermute
#define __builtin_amdgcn_ds_swizzle ::emu::ds_swizzle
#define __builtin_amdgcn_ballot_w64 ::emu::ballot
#define __builtin_amdgcn_mov_dpp(v, ctrl, rows, banks, zero) \
  ::emu::dpp(0, v, ctrl, rows, banks, zero)
#define __builtin_amdgcn_update_dpp ::emu::dpp
#define __builtin_amdgcn_permlane32_swap ::emu::permlane_swap
#define __builtin_amdgcn_permlane16_swap ::emu::permlane_swap
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier ::emu::wave_barrier
#define __builtin_amdgcn_sched_barrier(...) ((void)0)
// (the one inline assembly of the headers keeps a value opaque)
#define asm
#define volatile(...) ((void)0)
