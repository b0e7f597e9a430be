// msa_sweep4.hip -- streaming fill of the four-sequence tensor.
//
// The computation waves of Section 3 (cells at equal distance from the
// origin are independent) swept in a pipeline instead of tile by tile, as the
// three-sequence streaming fill does, with one more dimension:
//
//   - Lines.  A line is the run of cells (v0, v1, v2, 0..n3) along dimension
//     3.  A workgroup owns a block of 4 x 16 x 16 lines: rows v0 = B0*4 + u, all
//     held by every compute lane, v1 = B1*16 + q1 and v2 = B2*16 + q2 (one
//     compute lane per (q1, q2), four waves).  At block step s a lane computes
//     cell t = s - q1 - q2 of each of its rows, top row first.  A neighbour in
//     another lane was computed one step (v1 - 1 or v2 - 1) or two steps (both)
//     earlier; a neighbour in the row above is a value this lane read or
//     computed for that row in the same or in the previous step.  So a cell
//     reads three neighbours from LDS instead of seven or more, and a step
//     needs no wait beyond one barrier.
//   - Exchange inside a workgroup: every lane writes its four outputs to an LDS
//     ring of 4 steps (17 x 17 positions: the block's lanes and the layers q1
//     = -1 and q2 = -1 of the workgroups before it), beside the row above the
//     block, which another workgroup computed.
//   - Exchange between workgroups, by block step, so that one step's values
//     are consecutive words: region X0 holds the last row of every lane, X1
//     the lanes q1 = 15 and X2 the lanes q2 = 15 of every row.  Each word
//     carries the launch's tag (1..15) in the key's 4 low bits, which are zero
//     in a stored key.  A storer wave copies them from the ring one step after
//     they were computed, 16 bytes a lane.  Loader waves load the neighbours'
//     values kS4Pf steps ahead, reload while a tag is stale, and write them to
//     LDS one step before they are read.  Compute waves issue no global access
//     but their direction bytes, and wait for none.
//   - Workgroups take blocks in the order of `order`, in which every block
//     follows the blocks before it in each dimension, so a workgroup only
//     waits for workgroups that are already running.
//
// What bounds it: vector issue for a little more than half of the time, and the
// chain of a step (ring write, barrier, ring reads) where two workgroups do not
// cover each other.  A step is about 150 vector instructions a compute wave (37 lane
// slots a cell; the tile kernel's took 129), 0.39 us for a workgroup alone on its
// compute unit and 0.67 for two of them side by side, of which issue is 0.46; in
// all 129^4 takes 247 M vector instructions, 0.40 of 0.75 ms, and moves 2.25 GB of
// exchange words and directions (3 TB/s).  Of the cell slots 60% are cells: all
// lanes wait for the last one's skew, and a last block along dimension 1 or 2 may
// hold few lanes.
// Measured (129^4): fill 0.76 ms against 1.61 with the tile kernel; 46 x 34 x 62
// x 39: 0.11 against 0.30.  On the way there: one workgroup of 8 rows, four
// compute waves and one loader, all LDS reads after the barrier 1.03 ms (the
// step took 0.95 us, more than half of it waiting); blocks of 8, 12 and 16 rows
// by two or three groups of compute waves, one workgroup a compute unit,
// 0.79-0.96.
//
// Per cell (Section 2, Eq. 1 for four sequences): 15 candidates key(v - b) +
// column(b), pre-shifted by 4 bits with the tie bits 15 - b in the low bits,
// as in the tile kernel.  Direction bytes are collected in registers (a lane's
// byte of each step is shifted into a word) and stored, 4 cells at a time, in
// the same tile-major blocks (edge 8) as the tile kernel's, so the traceback
// and the decision export read them unchanged.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "msa_internal.h"
#include "msa_plan.h"
#include "msa_runtime.h"

namespace msa {

namespace {

constexpr int kS4Ring = 4;                 // LDS ring slots (steps)
constexpr int kS4Pf = 2;                   // loader prefetch distance (steps)
constexpr int kS4Un = 8;                   // steps per unrolled group
constexpr int kS4E = 17;                   // ring edge: 16 lanes and the layer before them
constexpr int kS4Pos = kS4E * kS4E;        // ring positions
constexpr int kS4Skew = 30;                // largest q1 + q2
constexpr int kS4Front = 32;               // LDS bytes before the fourth sequence
constexpr int kS4T = 8;                    // tile edge of the direction blocks (k = 4)
constexpr int kS4Dbs = kS4T * kS4T * kS4T * kS4T;
constexpr int64_t kS4WaitTicks = 200000000;  // 2 s of waiting (WaitClock ticks)

static_assert(tile_edge_for_k(4) == kS4T, "same blocks as the tile kernel");
static_assert(kS4Un % 4 == 0 && kS4T % 4 == 0, "whole direction runs");
static_assert(kS4Un % kS4Ring == 0 && kS4Un % kS4Pf == 0, "ring slots fixed per group");

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// Four compute waves, three loader waves and the storer wave: two waves on
// each SIMD, so that two workgroups fit a compute unit (at up to 128 vector
// registers) and one's barriers and LDS reads overlap the other's arithmetic.
constexpr int kS4Threads = 8 * 64;
// Words of one step in a block's slice of X0, and of X1 or X2.
constexpr int kS4X0 = 256;
constexpr int kS4X1 = 16 * kS4Rows;
constexpr int kS4UpRow = 48, kS4UpOff = 4, kS4Up = kS4E * kS4UpRow;
constexpr int kS4SubRow = 33;  // (an odd stride spreads the rows over the banks)

struct S4Smem {
  // Position (q1 + 1) * kS4E + q2 + 1 of slot s % 4: the four rows at t = s - q1
  // - q2.
  i32x4 ring[kS4Ring][kS4Pos];
  // The row above the block, at t = s - q1 - q2 + 1: position (q1 + 1) * kS4UpRow
  // + kS4UpOff + q2.  A wave's four runs of 16 words fall in distinct quarters
  // of the 64 banks, and the loader writes 16 bytes a lane.
  alignas(16) int32_t up[kS4Ring][kS4Up];
  alignas(16) int32_t last[kS4Ring][kS4X0];  // the lanes' last rows, for the storer
  i32x4 p03[kS4SubMax];                      // sub(r0 of each row, c) << 4 by code c
  int32_t sub16[kS4SubMax * kS4SubRow];      // substitution matrix << 4
  uint8_t s3[kS4Front + kS4SeqMax + 64];
  int32_t late, pause;  // the loader's watchdog fired; longest pause it saw (ticks)
  int32_t item, job;
};
static_assert(kS4Front > kS4Skew, "cells t < 0 read residue codes of the padding");

// LDS accesses of this wave complete, then every wave of the workgroup meets.
// Global stores stay in flight: no wave waits on them.
__device__ __forceinline__ void s4_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ uint64_t s4_load2(const int32_t *p) {
  return __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t s4_load(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Four words, each of which a reader accepts by its own tag: a device-scope
// store of 16 bytes, for which there is no atomic (the s_nop keeps the data
// registers from being written in the next cycle).
__device__ __forceinline__ void s4_store4(int32_t *base, uint32_t off, i32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, %2 sc1\n\ts_nop 1" ::"v"(off * 4u), "v"(v), "s"(base)
               : "memory");
}

// Steps a block runs: lane (q1, q2) computes its last stored cell, the end of the
// last 4-cell run, at step 4 * ceil(n3 / 4) + q1 + q2; a ragged block (the last
// along dimension 1 or 2) stops after its last valid lane.
__device__ __forceinline__ int s4_steps(const Sweep4Dev &sd, int B1, int B2) {
  const int j1 = min(15, sd.n[1] - B1 * 16);
  const int j2 = min(15, sd.n[2] - B2 * 16);
  const int n = (sd.n[3] + 3) / 4 * 4 + 1 + j1 + j2;
  return (n + kS4Un - 1) / kS4Un * kS4Un;
}

// First word of a block's slice of an exchange region.
__device__ __forceinline__ int64_t s4_x0(const Sweep4Dev &sd, int b0, int b1, int b2) {
  return (((int64_t)b0 * sd.nb[1] + b1) * sd.nb[2] + b2) * sd.S * kS4X0;
}
__device__ __forceinline__ int64_t s4_x1(const Sweep4Dev &sd, int b0, int b1, int b2) {
  return (((int64_t)b0 * (sd.nb[1] - 1) + b1) * sd.nb[2] + b2) * sd.S * kS4X1;
}
__device__ __forceinline__ int64_t s4_x2(const Sweep4Dev &sd, int b0, int b1, int b2) {
  return (((int64_t)b0 * sd.nb[1] + b1) * (sd.nb[2] - 1) + b2) * sd.S * kS4X1;
}

// The loader waves.  During step s they write the halo of ring slot s, and
// issue the loads of step s + kS4Pf:
//   wave 0: the row above, block (B0-1, B1, B2), step s + 1 (4 words a lane);
//   wave 1: layer q1 = -1, block (B0, B1-1, B2), step s + 16 (4 rows of one
//      position a lane), and single words: the corner (-1, -1) of every row
//      (block (B0, B1-1, B2-1), step s + 32), and the row above's layers q1 =
//      -1, q2 = -1 and corner;
//   wave 2: layer q2 = -1, block (B0, B1, B2-1), step s + 16.
// (A layer's 64 words take 16 lanes; the other lanes repeat them, as do lanes
// without a single word of their own.)  Values of
// a workgroup that does not exist, or of steps it does not run, read -infinity;
// they belong to no cell of the tensor.  Both are decided per lane and group
// of kS4Un steps, as three masks (tag check, bits kept, bits set), so a step
// costs an and-or per word and no address or window test: a producer's steps
// are a multiple of kS4Un, it stores one more step of X0 (the step s + 1 after
// a group's last), and loads past its steps stay inside the padded regions.
template <int W>
struct S4Loader {
  using Sm = S4Smem;
  static constexpr int E = W == 1 ? 2 : 1;
  const int32_t *ptr[E];  // words of the next step to issue
  int32_t inc[E];         // words per step (no producer: 0, a dummy word)
  int32_t lim[E];         // steps with a word: s < lim (no producer: none)
  uint32_t chk[E], keep[E];
  int32_t neg[E];
  int32_t dst[E];         // LDS words from the ring's first, slot 0
  int32_t slot1;          // words per slot there, of the single words
  static constexpr int kUp = (int)(offsetof(Sm, up) - offsetof(Sm, ring)) / 4;

  __device__ __forceinline__ void set(int x, const int32_t *p, int words, int off, int steps) {
    ptr[x] = p + (int64_t)off * words;
    inc[x] = words;
    lim[x] = steps - off;
  }

  __device__ __forceinline__ S4Loader(const Sweep4Dev &sd, int B0, int B1, int B2, int lane) {
#pragma unroll
    for (int x = 0; x < E; ++x) {
      ptr[x] = sd.x0;
      inc[x] = 0;
      lim[x] = INT32_MIN;
    }
    const int here = s4_steps(sd, B1, B2);
    const int left1 = B1 > 0 ? s4_steps(sd, B1 - 1, B2) : 0;
    const int left2 = B2 > 0 ? s4_steps(sd, B1, B2 - 1) : 0;
    const int left12 = B1 > 0 && B2 > 0 ? s4_steps(sd, B1 - 1, B2 - 1) : 0;
    const int32_t *const x0 = sd.x0, *const x1 = sd.x1, *const x2 = sd.x2;
    const int q = lane % 16, lv = q * 4;
    if constexpr (W == 0) {
      // (X0: here + 1 steps are stored, the last for the check alone)
      if (B0 > 0) set(0, x0 + s4_x0(sd, B0 - 1, B1, B2) + lane * 4, kS4X0, 1, here + 1);
      dst[0] = kUp + (lane / 4 + 1) * kS4UpRow + kS4UpOff + lane % 4 * 4;
    } else if constexpr (W == 2) {
      if (B2 > 0) set(0, x2 + s4_x2(sd, B0, B1, B2 - 1) + lv, kS4X1, 16, left2);
      dst[0] = (q + 1) * kS4E * 4;
    } else {
      if (B1 > 0) set(0, x1 + s4_x1(sd, B0, B1 - 1, B2) + lv, kS4X1, 16, left1);
      dst[0] = (q + 1) * 4;
      const int l = min(lane, kS4Rows + 32);
      int pos = kS4UpOff - 1;  // in the row above
      if (l < kS4Rows) {
        if (B1 > 0 && B2 > 0)
          set(1, x1 + s4_x1(sd, B0, B1 - 1, B2 - 1) + 15 * kS4Rows + l, kS4X1, 32, left12);
      } else if (l < kS4Rows + 16) {
        const int q2 = l - kS4Rows;
        if (B0 > 0 && B1 > 0)
          set(1, x0 + s4_x0(sd, B0 - 1, B1 - 1, B2) + 15 * 16 + q2, kS4X0, 17, left1 + 1);
        pos += q2 + 1;
      } else if (l < kS4Rows + 32) {
        const int q1 = l - kS4Rows - 16;
        if (B0 > 0 && B2 > 0)
          set(1, x0 + s4_x0(sd, B0 - 1, B1, B2 - 1) + q1 * 16 + 15, kS4X0, 17, left2 + 1);
        pos += (q1 + 1) * kS4UpRow;
      } else {
        if (B0 > 0 && B1 > 0 && B2 > 0)
          set(1, x0 + s4_x0(sd, B0 - 1, B1 - 1, B2 - 1) + 255, kS4X0, 33, left12 + 1);
      }
      dst[1] = l < kS4Rows ? l : kUp + pos;
      slot1 = l < kS4Rows ? kS4Pos * 4 : kS4Up;
    }
  }

  // The masks of the steps of a group, from its first step: all of them have
  // a word, or none.
  __device__ __forceinline__ void masks(int s0, bool before = false) {
#pragma unroll
    for (int x = 0; x < E; ++x) {
      // (before: the row above's own cells have no step s + 1 < 0)
      const bool in = s0 < lim[x] && !(before && W == 0);
      chk[x] = in ? 15u : 0u;
      keep[x] = in ? ~15u : 0u;
      neg[x] = in ? 0 : kNegKey;
    }
  }
  // Back to step -3, the first halo a block needs.
  __device__ __forceinline__ void rewind() {
#pragma unroll
    for (int x = 0; x < E; ++x) ptr[x] -= 3 * inc[x];
  }

  struct Vals {
    uint64_t w[2];
    int32_t c;
  };
  __device__ __forceinline__ static void fetch(const int32_t *const (&p)[E], Vals &v) {
    v.w[0] = s4_load2(p[0]);
    v.w[1] = s4_load2(p[0] + 2);
    if constexpr (E > 1) v.c = s4_load(p[E - 1]);
  }
  __device__ __forceinline__ void issue(Vals &v) {
    fetch(ptr, v);
#pragma unroll
    for (int x = 0; x < E; ++x) ptr[x] += inc[x];
  }
  // some word of a step is a neighbour's and not yet this launch's
  __device__ __forceinline__ bool stale(const Vals &v, uint32_t tag) const {
    auto off = [&](uint64_t w) { return ((uint32_t)w ^ tag) | ((uint32_t)(w >> 32) ^ tag); };
    uint32_t st = (off(v.w[0]) | off(v.w[1])) & chk[0];
    if constexpr (E > 1) st |= ((uint32_t)v.c ^ tag) & chk[E - 1];
    return __builtin_amdgcn_ballot_w64(st != 0) != 0;
  }
  // Slow path: reloads until every word carries this launch's tag or the
  // watchdog fires (pauses of the queue do not count as waiting).  What it has
  // to report goes to LDS and from there to the control block at the block's
  // end, so that a loader issues no global store or atomic beside its loads
  // (one counter tracks both).
  __device__ __forceinline__ void respin(int back, Vals &v, uint32_t tag, Sm &sm, Ctrl *ctrl,
                                         int64_t wlim) {
    const int32_t *p[E];
#pragma unroll
    for (int x = 0; x < E; ++x) p[x] = ptr[x] - back * inc[x];
    Vals u;
    WaitClock wc;
    for (int it = 0;; ++it) {
      __builtin_amdgcn_s_sleep(1);
      fetch(p, u);
      if (!stale(u, tag)) break;
      if ((it & 15) == 15) {
        const int st = __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(&ctrl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const bool late = wc.tick() > wlim;
        if (late) sm.late = 1;
        if (late || st == -4) {  // (or another workgroup timed out)
          // give up: the rest of the block waits for nothing
#pragma unroll
          for (int x = 0; x < E; ++x) {
            lim[x] = INT32_MIN;
            chk[x] = 0;
          }
          break;
        }
      }
    }
    if (wc.pause > sm.pause) sm.pause = (int32_t)min(wc.pause, (int64_t)INT32_MAX);
    v = u;
  }
  // The values of step s (its group's masks are set), issued `back` steps
  // before the next one to issue.
  __device__ __forceinline__ void finish(int s, int back, Vals &v, uint32_t tag, Sm &sm,
                                         Ctrl *ctrl, int64_t wlim) {
    if (stale(v, tag)) respin(back, v, tag, sm, ctrl, wlim);
    auto key = [&](int x, uint32_t w) { return (int32_t)(w & keep[x]) | neg[x]; };
    int32_t *const rb = reinterpret_cast<int32_t *>(&sm.ring[0][0]);
    const int k = s & (kS4Ring - 1);
    const i32x4 r = {key(0, (uint32_t)v.w[0]), key(0, (uint32_t)(v.w[0] >> 32)),
                     key(0, (uint32_t)v.w[1]), key(0, (uint32_t)(v.w[1] >> 32))};
    *reinterpret_cast<i32x4 *>(rb + (dst[0] + k * (W == 0 ? kS4Up : kS4Pos * 4))) = r;
    if constexpr (E > 1) rb[dst[E - 1] + k * slot1] = key(E - 1, (uint32_t)v.c);
  }
  // The whole block.
  __device__ __forceinline__ void run(int total, uint32_t tag, Sm &sm, Ctrl *ctrl, int64_t wlim) {
    Vals q[kS4Pf];
    {
      // the halo of the steps before the first, then the first steps' loads
      Vals f[3];
      rewind();
#pragma unroll
      for (int i = 0; i < 3; ++i) issue(f[i]);
#pragma unroll
      for (int i = 0; i < kS4Pf; ++i) issue(q[i]);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        masks(-kS4Un, i < 2);
        finish(i - 3, 3 - i + kS4Pf, f[i], tag, sm, ctrl, wlim);
      }
    }
    s4_barrier();
    for (int s0 = 0; s0 < total; s0 += kS4Un) {
      masks(s0);
#pragma unroll
      for (int i = 0; i < kS4Un; ++i) {
        finish(i, kS4Pf, q[i % kS4Pf], tag, sm, ctrl, wlim);  // (slots depend on s % 4 alone)
        s4_barrier();
        issue(q[i % kS4Pf]);
      }
    }
  }
};

// The storer wave: the block's exchange words of one step, from the ring.
struct S4Storer {
  using Sm = S4Smem;
  int32_t *x0, *x1, *x2;      // this step's words (wave-uniform)
  bool wx0, wx1, wx2;
  int src1, src2;             // ring vectors
  uint32_t o0, o1;
  bool edge;  // the 16 lanes that store X1 and X2
  __device__ __forceinline__ S4Storer(const Sweep4Dev &sd, int B0, int B1, int B2, int lane) {
    wx0 = B0 < sd.nb[0] - 1;
    wx1 = B1 < sd.nb[1] - 1;
    wx2 = B2 < sd.nb[2] - 1;
    x0 = sd.x0 + s4_x0(sd, B0, B1, B2);
    x1 = sd.x1 + s4_x1(sd, B0, B1, B2);
    x2 = sd.x2 + s4_x2(sd, B0, B1, B2);
    o0 = (uint32_t)lane * 4;
    const int q = lane % 16;
    src1 = 16 * kS4E + q + 1;
    src2 = (q + 1) * kS4E + 16;
    o1 = (uint32_t)q * 4;
    edge = lane < 16;
  }
  __device__ __forceinline__ void step(int s, int tag, const Sm &sm) {
    const i32x4 *const rb = &sm.ring[s & (kS4Ring - 1)][0];
    if (wx0)
      s4_store4(x0, o0,
                *reinterpret_cast<const i32x4 *>(&sm.last[s & (kS4Ring - 1)][o0]) | tag);
    if (edge) {
      if (wx1) s4_store4(x1, o1, rb[src1] | tag);
      if (wx2) s4_store4(x2, o1, rb[src2] | tag);
    }
    x0 += kS4X0;
    x1 += kS4X1;
    x2 += kS4X1;
  }
  // the step of X0 after the last
  __device__ __forceinline__ void tail(int tag) {
    if (wx0) s4_store4(x0, o0, i32x4{tag, tag, tag, tag});
  }
};

// The compute waves' sweep of block (B0, B1, B2).
__device__ __forceinline__ void s4_sweep(const Sweep4Dev &sd, S4Smem &sm, int B0, int B1,
                                         int B2, int tid, int gap, int total) {
  using Sm = S4Smem;
  constexpr int R = kS4Rows;
  const int q1 = tid >> 4, q2 = tid & 15;
  const int sk = q1 + q2;
  const int vg = B0 * R;  // the first row
  const int v1 = B1 * 16 + q1, v2 = B2 * 16 + q2;
  const int n0 = sd.n[0], n3 = sd.n[3];
  const bool lane_ok = v1 <= sd.n[1] && v2 <= sd.n[2];
  const int r1 = v1 >= 1 && v1 <= sd.n[1] ? min((int)sd.seqs[n0 + v1 - 1], kS4SubMax - 1) : 0;
  const int r2 =
      v2 >= 1 && v2 <= sd.n[2] ? min((int)sd.seqs[n0 + sd.n[1] + v2 - 1], kS4SubMax - 1) : 0;
  // column scores: gap term of 1, 2 or 3 residues and the tie bits 15 - b
  const int g3 = gap * 48, g4 = gap * 64;
  const int32_t K1 = g3 + 14, K2 = g3 + 13, K4 = g3 + 11, K8 = g3 + 7, K9 = g4 + 6;
  int32_t K3 = g4 + 12, K5 = g4 + 10;
  const int32_t p12 = sm.sub16[r1 * kS4SubRow + r2];
  const int32_t K10 = g4 + 5, K11 = g3 + 4, K12 = g4 + 3, K13 = g3 + 2;  // (mask 15: 0)
  const int32_t P7 = p12 + g3 + 8;
  int32_t K6 = g4 + 9;
  int32_t p01[R], p02[R];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    p01[u] = sm.p03[r1][u];  // sub(r0 of row u, r1) << 4
    p02[u] = sm.p03[r2][u];
  }
  const int32_t *const sub1 = sm.sub16 + r1 * kS4SubRow;
  const int32_t *const sub2 = sm.sub16 + r2 * kS4SubRow;
  // The lane's ring vectors at position (q1 - 1, q2 - 1): + 1 is (q1 - 1, q2),
  // + kS4E (q1, q2 - 1), + kS4E + 1 the lane's own (the row above's rows:
  // kS4UpRow).
  i32x4 *const rp = &sm.ring[0][q1 * kS4E + q2];
  const int32_t *const up = &sm.up[0][q1 * kS4UpRow + kS4UpOff - 1 + q2];
  constexpr int RS = kS4Pos;
  // direction lines: tile (c0, c1, c2, c3), bytes ((q0*8 + q1)*8 + q2)*8 + q3
  auto tc = [](int v) { return v == 0 ? 0 : (v - 1) / kS4T + 1; };
  auto tq = [](int v) { return v == 0 ? 0 : (v - 1) % kS4T; };
  // byte offset of the lane's line in tile row c0 = 0 (below 2^32: sweep4_eligible)
  const uint32_t dlane =
      ((uint32_t)tc(v1) * (uint32_t)sd.ts[1] + (uint32_t)tc(v2) * (uint32_t)sd.ts[2]) * kS4Dbs +
      (uint32_t)((tq(v1) * kS4T + tq(v2)) * kS4T);
  // first byte of the tile rows along dimension 0: row u = 0, and rows u >= 1,
  // which all lie in one tile
  const int rows = min(R, n0 - vg + 1);
  auto drow = [&](int v0) {
    return sd.dir + (int64_t)tc(v0) * sd.ts[0] * kS4Dbs + tq(v0) * (kS4T * kS4T * kS4T);
  };
  uint8_t *const drow0 = drow(vg), *const drow1 = drow(vg + 1);
  const bool origin = vg == 0 && B1 == 0 && B2 == 0;
  // the score: the corner cell is row n0 % R of lane (n1 % 16, n2 % 16)
  const bool cw = vg / R == n0 / R && B1 == sd.n[1] / 16 && B2 == sd.n[2] / 16;
  const int cl1 = sd.n[1] & 15, cl2 = sd.n[2] & 15;
  const int sc = n3 + cl1 + cl2, uc = n0 % R, tcw = cl1 * 16 + cl2;

  // Direction bytes: every 4 steps the run of 4 cells (one aligned word of the
  // direction block) that ended at or before the lane's last cell is taken out
  // of the bytes of the last 8 steps; its place there is the same every time.
  const int xs = ((sk + 1) & 3) * 8;  // shift of the lane's run within two words
  const bool xz = xs == 0;
  const int cl = (n3 + 3) / 4;  // the last run (cells 4 cl - 3 .. n3)

  // m8[u]: the best of the row's candidates with dimension 3 (masks 8 .. 15),
  // which come from the cells of step s - 1.  They are taken at the end of step
  // s - 1, after its outputs went to LDS and before the barrier, so that a
  // step's path from the barrier to its outputs holds only masks 1 .. 7.  What
  // else step s reads from LDS but the values of step s - 1 itself (the cells
  // two steps back, the row above, residues and pair scores) is loaded in step
  // s - 1 as well.  (129^4 fill of 8-row blocks, all of it after the barrier:
  // 0.95 us a step, of which the vector instructions take 0.5.)
  int32_t m8[R];
  uint32_t w0[R], nw[R];  // direction bytes of the previous and the current 4 steps
  constexpr int RM = kS4Ring - 1;
#pragma unroll
  for (int u = 0; u < R; ++u) {
    m8[u] = kNegKey;
    w0[u] = nw[u] = 0;
  }
  i32x4 c = rp[(-2 & RM) * RS];  // (v1 - 1, v2 - 1)
  // the row above at (v1 - 1), (v2 - 1) and both
  int32_t na = up[(-2 & RM) * kS4Up + 1], nb = up[(-2 & RM) * kS4Up + kS4UpRow],
          nc = up[(-3 & RM) * kS4Up];
  const uint8_t *s3p = sm.s3 + kS4Front - 1 - sk;  // s3p[s]: residue of cell t of step s
  int r3 = s3p[1];

  auto group = [&](auto pro, int s0) __attribute__((always_inline)) {
    constexpr bool kPro = decltype(pro)::value;
#pragma unroll
    for (int i = 0; i < kS4Un; ++i) {
      const int s = s0 + i;
      const int t = s - sk;
      const i32x4 a = rp[((i - 1) & RM) * RS + 1];     // (v1 - 1)
      const i32x4 b = rp[((i - 1) & RM) * RS + kS4E];  // (v2 - 1)
      const int32_t no = up[((i - 1) & RM) * kS4Up + kS4UpRow + 1];
      __builtin_amdgcn_sched_barrier(0);  // (LDS returns in order: these first)
      // ---- for step s + 1 ----
      const i32x4 p03 = sm.p03[r3], cn = rp[((i - 1) & RM) * RS];
      const int32_t p13 = sub1[r3], p23 = sub2[r3];
      r3 = s3p[s + 2];
      const int32_t na1 = up[((i - 1) & RM) * kS4Up + 1];
      const int32_t nb1 = up[((i - 1) & RM) * kS4Up + kS4UpRow];
      const int32_t nc1 = up[((i - 2) & RM) * kS4Up];
      // Opaque at every step: the compiler would otherwise keep sums with them
      // in registers across the steps.
      asm volatile("" : "+s"(K3), "+s"(K5), "+s"(K6));
#pragma unroll
      for (int u = 0; u < R; ++u) asm volatile("" : "+v"(p01[u]), "+v"(p02[u]));
      const int32_t q15 = p13 + p23 + p12, q14 = q15 + g3 + 1;
      i32x4 out;
      int32_t x3[R], x5[R], x7[R];
      {
        // ---- masks 1 .. 7, and the cell ----
        // the row above at t: own, v1 - 1, v2 - 1, both
        int32_t ro = no, ra = na, rb = nb, rc = nc;
#pragma unroll
        for (int u = 0; u < R; ++u) {
          x3[u] = ra + p01[u];
          x5[u] = rb + p02[u];
          x7[u] = rc + (p01[u] + p02[u]);
          int32_t m = max(max(m8[u], c[u] + p12 + K6), x7[u] + P7);
          m = max(max(m, x3[u] + K3), x5[u] + K5);
          m = max(max(m, a[u] + K2), b[u] + K4);
          m = max(m, ro + K1);
          if constexpr (kPro) {
            m = t < 0 ? kNegKey : m;
            if (u == 0) m = origin && sk == 0 && t == 0 ? 15 : m;  // score 0, mask 0
          }
          nw[u] = __builtin_amdgcn_alignbyte((uint32_t)m, nw[u], 1);
          out[u] = m & ~15;
          ro = out[u];
          ra = a[u];
          rb = b[u];
          rc = c[u];
        }
      }
      rp[(i & RM) * RS + kS4E + 1] = out;
      sm.last[i & RM][tid] = out[R - 1];
      {
        // ---- masks 8 .. 15 of step s + 1 ----
        int32_t so = no;
#pragma unroll
        for (int u = 0; u < R; ++u) {
          const int32_t f = p03[u];
          int32_t m = max(out[u] + K8, so + f + K9);
          m = max(max(m, a[u] + p13 + K10), x3[u] + (f + p13 + K11));
          m = max(max(m, b[u] + p23 + K12), x5[u] + (f + p23 + K13));
          m8[u] = max(max(m, c[u] + q14), x7[u] + (f + q15));
          so = out[u];
        }
      }
      c = cn;
      na = na1;
      nb = nb1;
      nc = nc1;
      if (cw && s == sc) {  // wave-uniform
        int32_t o = out[0];
#pragma unroll
        for (int u = 1; u < R; ++u) o = uc == u ? out[u] : o;
        if (tid == tcw) *sd.score_out = (int64_t)(o >> 4);
      }
      s4_barrier();
      // ---- the direction run completed in the last 4 steps ----
      if (i % 4 == 3) {
        const int c3 = (s - sk) >> 2;  // run c3: cells 4 c3 - 3 .. 4 c3
        const uint32_t dl =
            dlane + (uint32_t)((c3 + 1) >> 1) * kS4Dbs + (uint32_t)((c3 - 1) & 1) * 4;
        const bool st = lane_ok && c3 >= 1 && c3 <= cl;
#pragma unroll
        for (int u = 0; u < R; ++u) {
          const uint32_t wv = __builtin_amdgcn_alignbit(nw[u], w0[u], xs);
          const uint32_t run = xz ? nw[u] : wv;
          w0[u] = nw[u];
          if (u < rows) {  // uniform
            uint8_t *const d = u == 0 ? drow0 : drow1 + (u - 1) * (kS4T * kS4T * kS4T);
            if (st) *reinterpret_cast<uint32_t *>(d + dl) = run;
            if constexpr (kPro)
              if (lane_ok && c3 == 0) d[dlane] = (uint8_t)(run >> 24);  // cell 0, its own block
          }
        }
      }
    }
  };
  int s0 = 0;
  // cells t < 0 and t = 0 fall in the first steps
  for (; s0 < total && s0 < 40; s0 += kS4Un) group(std::true_type{}, s0);
  for (; s0 < total; s0 += kS4Un) group(std::false_type{}, s0);
}

// One block: set-up by all waves, then every wave runs the same number of
// steps.  `status` takes MSA_EINVAL for a bad residue code.
__device__ __forceinline__ void s4_block(const Sweep4Dev &sd, S4Smem &sm, int item,
                                         int alpha, int gap, int tag, int32_t *status, Ctrl *ctrl,
                                         int64_t wlim) {
  constexpr int R = kS4Rows, NT = kS4Threads;
  // (opaque, so that nothing derived from it is kept across a batched launch's
  // blocks)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
  int rem = item;
  const int B2 = rem % sd.nb[2];
  rem /= sd.nb[2];
  const int B1 = rem % sd.nb[1];
  const int B0 = rem / sd.nb[1];
  bool bad = false;
  for (int e = tid; e < alpha * alpha; e += NT)
    sm.sub16[(e / alpha) * kS4SubRow + e % alpha] = (int32_t)sd.sub[e] * 16;
  for (int e = tid; e < alpha * R; e += NT) {
    const int cc = e / R, u = e % R;
    const int v0 = B0 * R + u;
    int r0 = v0 >= 1 && v0 <= sd.n[0] ? (int)sd.seqs[v0 - 1] : 0;
    bad = bad || r0 >= alpha;
    reinterpret_cast<int32_t *>(sm.p03)[e] = (int32_t)sd.sub[(r0 >= alpha ? 0 : r0) * alpha + cc] * 16;
  }
  const uint8_t *const s3 = sd.seqs + sd.n[0] + sd.n[1] + sd.n[2];
  for (int e = tid; e < kS4Front + sd.n[3] + 64; e += NT) {
    const int q = e - kS4Front;
    const int r = q >= 0 && q < sd.n[3] ? (int)s3[q] : 0;
    bad = bad || r >= alpha;
    sm.s3[e] = (uint8_t)(r >= alpha ? 0 : r);
  }
  if (tid < 32) {  // this block's residues of dimensions 1 and 2
    const int v = (tid < 16 ? B1 : B2) * 16 + (tid & 15);
    const int n = tid < 16 ? sd.n[1] : sd.n[2];
    const int o = tid < 16 ? sd.n[0] : sd.n[0] + sd.n[1];
    bad = bad || (v >= 1 && v <= n && (int)sd.seqs[o + v - 1] >= alpha);
  }
  if (bad) atomicCAS(status, 0, -1);
  // before step 0 the rings hold cells t < 0: -infinity
  for (int e = tid; e < kS4Ring * kS4Pos; e += NT)
    (&sm.ring[0][0])[e] = i32x4{kNegKey, kNegKey, kNegKey, kNegKey};
  for (int e = tid; e < kS4Ring * kS4Up; e += NT) (&sm.up[0][0])[e] = kNegKey;
  if (tid == 0) sm.late = sm.pause = 0;
  s4_barrier();
  const int total = s4_steps(sd, B1, B2);
  if (wave == 4) {
    S4Loader<0> ld(sd, B0, B1, B2, tid & 63);
    ld.run(total, tag, sm, ctrl, wlim);
  } else if (wave == 5) {
    S4Loader<1> ld(sd, B0, B1, B2, tid & 63);
    ld.run(total, tag, sm, ctrl, wlim);
  } else if (wave == 6) {
    S4Loader<2> ld(sd, B0, B1, B2, tid & 63);
    ld.run(total, tag, sm, ctrl, wlim);
  } else if (wave == 7) {
    S4Storer st(sd, B0, B1, B2, tid & 63);
    s4_barrier();
    s4_barrier();  // step 0
    for (int s = 1; s < total; ++s) {
      st.step(s - 1, tag, sm);
      s4_barrier();
    }
    st.step(total - 1, tag, sm);
    st.tail(tag);
  } else {
    s4_barrier();
    s4_sweep(sd, sm, B0, B1, B2, tid, gap, total);
    if (tid == 0) {
      if (sm.late) sweep_timed_out(ctrl, sm.job, item);
      if (sm.pause > 0)
        __hip_atomic_fetch_max(&ctrl->max_pause, (int64_t)sm.pause, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

}  // namespace

__global__ __launch_bounds__(kS4Threads) __attribute__((amdgpu_waves_per_eu(4)))
void sweep4_kernel(Sweep4Dev sd, Ctrl *ctrl) {
  __shared__ S4Smem sm;
  if (threadIdx.x == 0) {
    sm.item = atomicAdd(&ctrl->head, 1);
    sm.job = 0;
  }
  const int alpha = ctrl->alpha;
  const int gap = ctrl->gap;
  const int tag = sweep_tag(ctrl->sweeps, kSweepTags);
  s4_barrier();
  const int ticket = __builtin_amdgcn_readfirstlane(sm.item);
  // a ticket past the grid: the counter was not reset since the last fill
  if (ticket >= sd.nb[0] * sd.nb[1] * sd.nb[2]) return;
  if (ticket == 0 && threadIdx.x == 0) ctrl->swept = 1;
  s4_block(sd, sm, __builtin_amdgcn_readfirstlane(sd.order[ticket]), alpha, gap, tag,
                 &ctrl->status, ctrl, kS4WaitTicks);
}

// ---------------------------------------------------------------------------
// Batched launches: the blocks of all k = 4 jobs from one queue.
// ---------------------------------------------------------------------------

// Block b of job j goes to slot kbase_j[key] (where the host placed job j's
// blocks of that key) + its rank among them in the order of (b1 + b2, b1).
__global__ __launch_bounds__(256) void batch_s4queue_kernel(const BatchArgs *__restrict__ a) {
  const int total = a->s4total;
  const int32_t *__restrict__ pre = a->s4pre;
  int32_t *q = a->s4q;
  for (int g = blockIdx.x * (int)blockDim.x + threadIdx.x; g < total;
       g += (int)(gridDim.x * blockDim.x)) {
    int lo = 0, hi = a->s4n;  // pre[lo] <= g < pre[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (pre[mid] <= g) lo = mid; else hi = mid;
    }
    const Sweep4Dev &sd = a->s4jobs[lo];
    const int nb0 = sd.nb[0], nb1 = sd.nb[1], nb2 = sd.nb[2];
    const int b = g - pre[lo];
    const int b2 = b % nb2, b1 = b / nb2 % nb1, b0 = b / nb2 / nb1;
    const int key = sweep4_key(b0, b1, b2);
    int rank = b1 - max(0, b1 + b2 - (nb2 - 1));
    for (int m = 0; m < b1 + b2; ++m) {
      const int c0 = key - sweep4_key(0, m, 0);  // the b0 of a block with this m and key
      if (c0 >= 0 && c0 < nb0) rank += min(m, nb1 - 1) - max(0, m - (nb2 - 1)) + 1;
    }
    const int slot = sd.kbase[key] + rank;
    q[2 * slot] = lo;
    q[2 * slot + 1] = b;
  }
}

// Persistent workgroups take the queue's blocks in order; every block follows
// its job's lower neighbours there.
__global__ __launch_bounds__(kS4Threads) __attribute__((amdgpu_waves_per_eu(4)))
void batch_sweep4_kernel(const BatchArgs *__restrict__ a, Ctrl *ctrl) {
  __shared__ S4Smem sm;
  const int total = __builtin_amdgcn_readfirstlane(a->s4total);
  const int tag = __builtin_amdgcn_readfirstlane(a->s4tag);
  const int32_t *const q = as_global(a->s4q);
  const Sweep4Dev *const jobs = as_global(a->s4jobs);
  const int64_t wl =
      __hip_atomic_load(&ctrl->wait_limit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t wlim = wl > 0 ? wl : kS4WaitTicks;
  for (;;) {
    // every lane of the workgroup takes the same way: no divergent pop next to
    // the loop's back edge
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x) == 0) {
      const int got = atomicAdd(&ctrl->s4head, threadIdx.x == 0 ? 1 : 0);
      sm.item = __builtin_amdgcn_readfirstlane(got);
    }
    s4_barrier();  // also: every wave is done with the last block's LDS
    const int it = __builtin_amdgcn_readfirstlane(sm.item);
    if (it >= total) break;
    const int job = __builtin_amdgcn_readfirstlane(q[2 * it]);
    const int blk = __builtin_amdgcn_readfirstlane(q[2 * it + 1]);
    if (threadIdx.x == 0) sm.job = job;  // (read by the same thread)
    // the job's descriptor, kept in scalar registers
    Sweep4Dev sd;
    {
      const uint32_t *const src = reinterpret_cast<const uint32_t *>(jobs + job);
      uint32_t w[sizeof(Sweep4Dev) / 4];
#pragma unroll
      for (int i = 0; i < (int)(sizeof(Sweep4Dev) / 4); ++i)
        w[i] = __builtin_amdgcn_readfirstlane(src[i]);
      __builtin_memcpy(&sd, w, sizeof(sd));
    }
    sd.seqs = as_global(sd.seqs);
    sd.sub = as_global(sd.sub);
    sd.x0 = as_global(sd.x0);
    sd.x1 = as_global(sd.x1);
    sd.x2 = as_global(sd.x2);
    sd.dir = as_global(sd.dir);
    sd.score_out = as_global(sd.score_out);
    sd.status = as_global(sd.status);
    s4_block(sd, sm, blk, sd.alpha, sd.gap, tag, sd.status, ctrl, wlim);
  }
}

void launch_batch_sweep4(const BatchArgs *d_args, Ctrl *ctrl, hipStream_t s) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch_sweep4_kernel, kS4Threads, 0) !=
          hipSuccess ||
      nb < 1)
    nb = 1;
  hipLaunchKernelGGL(batch_s4queue_kernel, dim3(256), dim3(256), 0, s, d_args);
  hipLaunchKernelGGL(batch_sweep4_kernel, dim3((unsigned)(device_cu_count() * nb)),
                     dim3(kS4Threads), 0, s, d_args, ctrl);
}

int launch_sweep4(const Plan &p, char *ws, const JobDev &jd, Ctrl *ctrl, hipStream_t s) {
  Sweep4Dev sd;
  fill_sweep4dev(p, &sd);
  sd.seqs = jd.seqs;
  sd.sub = jd.sub;
  sd.dir = jd.dir;
  sd.score_out = jd.score_out;
  sd.x0 = reinterpret_cast<int32_t *>(ws + p.off_faces) + kS4PadFront;
  sd.x1 = sd.x0 + p.s4_x0;
  sd.x2 = sd.x1 + p.s4_x1;
  sd.order = reinterpret_cast<const int32_t *>(ws + p.off_s4order);
  const unsigned grid = (unsigned)(sd.nb[0] * sd.nb[1] * sd.nb[2]);
  launch_begin();
  hipLaunchKernelGGL(sweep4_kernel, dim3(grid), dim3(kS4Threads), 0, s, sd, ctrl);
  return launch_end();
}

}  // namespace msa
