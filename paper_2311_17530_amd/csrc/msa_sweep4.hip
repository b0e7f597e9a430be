// msa_sweep4.hip -- streaming fill of the four-sequence tensor.
//
// The computation waves of Section 3 (cells at equal distance from the
// origin are independent) swept in a pipeline instead of tile by tile, as the
// three-sequence streaming fill does, with one more dimension:
//
//   - Lines.  A line is the run of cells (v0, v1, v2, 0..n3) along dimension
//     3.  A workgroup owns a block of R x 16 x 16 lines: rows v0 = B0*R + u
//     (u < R, all of them held by every lane), v1 = B1*16 + q1 and v2 = B2*16
//     + q2 (one compute lane per (q1, q2), four waves).  At block step s a
//     lane computes cell t = s - q1 - q2 of each of its rows, top row first.
//     A neighbour in another lane was computed one step (v1 - 1 or v2 - 1) or
//     two steps (both) earlier; a neighbour in the row above is a value this
//     lane read or computed for that row in the same or in the previous step.
//     So a cell reads three neighbours from LDS instead of seven or more, and
//     a step needs no wait beyond one barrier.
//   - Exchange inside a workgroup: every lane writes its R outputs to an LDS
//     ring of 4 steps (17 x 17 positions: the block's lanes and the layers q1
//     = -1 and q2 = -1 of the workgroups before it; position (q1, q2) of step
//     s always holds cell t = s - q1 - q2).  The row above the block has a
//     ring of its own (up).
//   - Exchange between workgroups, by block step, so that one step's values
//     are consecutive words: region X0 holds the last row of every lane, X1
//     the lanes q1 = 15 and X2 the lanes q2 = 15 of every row.  Each word
//     carries the launch's tag (1..15) in the key's 4 low bits, which are zero
//     in a stored key.  A loader wave (wave 4) loads the neighbours' values
//     kS4Pf steps ahead, reloads while a tag is stale, and writes them to LDS
//     one step before they are read.  Compute waves issue no global load, and
//     no wave waits for its stores.
//   - Workgroups take blocks in the order of `order`, in which every block
//     follows the blocks before it in each dimension, so a workgroup only
//     waits for workgroups that are already running.
//
// Per cell (Section 2, Eq. 1 for four sequences): 15 candidates key(v - b) +
// column(b), pre-shifted by 4 bits with the tie bits 15 - b in the low bits,
// as in the tile kernel.  Direction bytes are collected in registers (a lane's
// byte of each step is shifted into a word) and stored, 8 cells at a time, in
// the same tile-major blocks (edge 8) as the tile kernel's, so the traceback
// and the decision export read them unchanged.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "msa_internal.h"
#include "msa_plan.h"

namespace msa {

namespace {

constexpr int kS4Ring = 4;                 // LDS ring slots (steps)
constexpr int kS4Pf = 2;                   // loader prefetch distance (steps)
constexpr int kS4Un = 8;                   // steps per unrolled group
constexpr int kS4E = 17;                   // ring edge: 16 lanes and the layer before them
constexpr int kS4Pos = kS4E * kS4E;        // ring positions
constexpr int kS4Waves = 4;                // compute waves
constexpr int kS4Threads = (kS4Waves + 1) * 64;
constexpr int kS4Skew = 30;                // largest q1 + q2
constexpr int kS4Front = 32;               // LDS bytes before the fourth sequence
constexpr int kS4T = 8;                    // tile edge of the direction blocks (k = 4)
constexpr int kS4Dbs = kS4T * kS4T * kS4T * kS4T;
constexpr int64_t kS4WaitTicks = 200000000;  // 2 s of waiting (WaitClock ticks)

static_assert(tile_edge_for_k(4) == kS4T, "same blocks as the tile kernel");
static_assert(kS4Un % 4 == 0 && kS4T % 4 == 0, "whole direction runs");
static_assert(kS4Un % kS4Ring == 0 && kS4Un % kS4Pf == 0, "ring slots fixed per group");
static_assert(kS4Front > kS4Skew, "cells t < 0 read residue codes of the padding");

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

template <int R>
struct S4Smem {
  alignas(16) int32_t ring[kS4Ring][R / 4][kS4Pos][4];  // outputs of a step, 4 rows a vector
  int32_t up[kS4Ring][kS4Pos];                          // the row above the block
  alignas(16) int32_t p03[kS4SubMax][R];                // sub(r0 of row u, c) << 4 by code c
  int32_t sub16[kS4SubMax * kS4SubMax];                 // substitution matrix << 4
  uint8_t s3[kS4Front + kS4SeqMax + 64];
  int32_t item;
};

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
__device__ __forceinline__ void s4_store(int32_t *p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void s4_store2(int32_t *p, int32_t a, int32_t b) {
  __hip_atomic_store(reinterpret_cast<uint64_t *>(p), (uint64_t)(uint32_t)a | ((uint64_t)(uint32_t)b << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Words of one step in a block's slice of X0, and of X1 or X2.
constexpr int kS4X0 = 256;
template <int R> constexpr int kS4X1 = 16 * R;

// Steps a block runs: lane (q1, q2) computes its last stored cell, the end of
// the last 4-cell run, at step 4 * ceil(n3 / 4) + q1 + q2; a ragged block (the
// last along dimension 1 or 2) stops after its last valid lane.
__device__ __forceinline__ int s4_steps(const Sweep4Dev &sd, int B1, int B2) {
  const int j1 = min(15, sd.n[1] - B1 * 16);
  const int j2 = min(15, sd.n[2] - B2 * 16);
  const int n = (sd.n[3] + 3) / 4 * 4 + 1 + j1 + j2;
  return (n + kS4Un - 1) / kS4Un * kS4Un;
}

// The loader wave.  During step s it writes the halo of ring slot s and row
// slot s + 1 of `up`, and issues the loads of step s + kS4Pf:
//   0: the row above, block (B0-1, B1, B2), step s + 1 (4 words a lane);
//   1: layer q1 = -1, block (B0, B1-1, B2), step s + 16 (lanes 0..31), and
//      layer q2 = -1, block (B0, B1, B2-1), step s + 16 (lanes 32..63): 4 rows
//      of one position a lane;
//   2: single words: the corner (-1, -1) of every row (block (B0, B1-1, B2-1),
//      step s + 32), and the row above's layers q1 = -1, q2 = -1 and corner.
// A lane without a word of its own repeats another lane's.  Values of a
// workgroup that does not exist, or of steps it does not run, read -infinity;
// they belong to no cell of the tensor.
template <int R>
struct S4Loader {
  const int32_t *base[3];
  // offset of the next step to issue within the producer's slice, its
  // increment and last value; no producer: offset -1, increment 0
  int32_t acc[3], inc[3], ohi[3];
  i32x4 *dst1;          // ring slot 0
  int32_t dst2[kS4Ring];  // word index from ring, per slot s % 4
  int32_t *dst0;        // up slot 0

  __device__ __forceinline__ void set(int x, const int32_t *p, int words, int off, int steps,
                                      int s_first) {
    base[x] = p;
    inc[x] = words;
    acc[x] = (s_first + off) * words;
    ohi[x] = (steps - 1) * words;
  }

  __device__ __forceinline__ S4Loader(const Sweep4Dev &sd, S4Smem<R> &sm, int B0, int B1, int B2,
                                      int lane, int s_first) {
    const int64_t S = sd.S;
    auto x0 = [&](int b0, int b1, int b2) {
      return sd.x0 + (((int64_t)b0 * sd.nb[1] + b1) * sd.nb[2] + b2) * S * kS4X0;
    };
    auto x1 = [&](int b0, int b1, int b2) {
      return sd.x1 + (((int64_t)b0 * (sd.nb[1] - 1) + b1) * sd.nb[2] + b2) * S * kS4X1<R>;
    };
    auto x2 = [&](int b0, int b1, int b2) {
      return sd.x2 + (((int64_t)b0 * sd.nb[1] + b1) * (sd.nb[2] - 1) + b2) * S * kS4X1<R>;
    };
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      base[x] = sd.x0;  // never empty (the region holds at least one slot)
      acc[x] = -1;
      inc[x] = 0;
      ohi[x] = 0;
    }
    const int here = s4_steps(sd, B1, B2);
    const int left1 = B1 > 0 ? s4_steps(sd, B1 - 1, B2) : 0;
    const int left2 = B2 > 0 ? s4_steps(sd, B1, B2 - 1) : 0;
    const int left12 = B1 > 0 && B2 > 0 ? s4_steps(sd, B1 - 1, B2 - 1) : 0;
    if (B0 > 0) set(0, x0(B0 - 1, B1, B2) + lane * 4, kS4X0, 1, here, s_first);
    dst0 = &sm.up[0][(lane / 4 + 1) * kS4E + lane % 4 * 4 + 1];
    {
      const int l = (lane & 31) % (4 * R);
      const int q = l * 4 / R, h = l * 4 % R / 4;
      if (lane < 32) {
        if (B1 > 0) set(1, x1(B0, B1 - 1, B2) + l * 4, kS4X1<R>, 16, left1, s_first);
        dst1 = reinterpret_cast<i32x4 *>(&sm.ring[0][h][q + 1][0]);
      } else {
        if (B2 > 0) set(1, x2(B0, B1, B2 - 1) + l * 4, kS4X1<R>, 16, left2, s_first);
        dst1 = reinterpret_cast<i32x4 *>(&sm.ring[0][h][(q + 1) * kS4E][0]);
      }
    }
    {
      const int l = min(lane, R + 32);
      const int32_t *const rb = &sm.ring[0][0][0][0];
      const int ub = (int)(&sm.up[0][0] - rb);
      int pos = 0;
      if (l < R) {
        if (B1 > 0 && B2 > 0)
          set(2, x1(B0, B1 - 1, B2 - 1) + 15 * R + l, kS4X1<R>, 32, left12, s_first);
      } else if (l < R + 16) {
        const int q2 = l - R;
        if (B0 > 0 && B1 > 0)
          set(2, x0(B0 - 1, B1 - 1, B2) + 15 * 16 + q2, kS4X0, 17, left1, s_first);
        pos = q2 + 1;
      } else if (l < R + 32) {
        const int q1 = l - R - 16;
        if (B0 > 0 && B2 > 0)
          set(2, x0(B0 - 1, B1, B2 - 1) + q1 * 16 + 15, kS4X0, 17, left2, s_first);
        pos = (q1 + 1) * kS4E;
      } else {
        if (B0 > 0 && B1 > 0 && B2 > 0)
          set(2, x0(B0 - 1, B1 - 1, B2 - 1) + 255, kS4X0, 33, left12, s_first);
      }
#pragma unroll
      for (int k = 0; k < kS4Ring; ++k)
        dst2[k] = l < R ? (int)(&sm.ring[k][l / 4][0][l % 4] - rb)
                        : ub + ((k + 1) & (kS4Ring - 1)) * kS4Pos + pos;
    }
  }

  __device__ __forceinline__ const int32_t *addr(int x, int32_t a) const {
    return base[x] + (uint32_t)min(max(a, 0), ohi[x]);
  }
  struct Vals {
    uint64_t a[2], b[2];
    int32_t c;
  };
  __device__ __forceinline__ void fetch(const int32_t (&o)[3], Vals &v) const {
    const int32_t *p0 = addr(0, o[0]);
    const int32_t *p1 = addr(1, o[1]);
    v.a[0] = s4_load2(p0);
    v.a[1] = s4_load2(p0 + 2);
    v.b[0] = s4_load2(p1);
    v.b[1] = s4_load2(p1 + 2);
    v.c = s4_load(addr(2, o[2]));
  }
  __device__ __forceinline__ void issue(Vals &v) {
    fetch(acc, v);
#pragma unroll
    for (int x = 0; x < 3; ++x) acc[x] += inc[x];
  }
  __device__ __forceinline__ bool in(int x, int32_t o) const {
    return (unsigned)o <= (unsigned)ohi[x];
  }
  // some word of a step is a neighbour's and not yet this launch's
  __device__ __forceinline__ bool stale(const int32_t (&o)[3], const Vals &v, int tag) const {
    auto off = [&](uint64_t w) {
      return ((uint32_t)w ^ (uint32_t)tag) | ((uint32_t)(w >> 32) ^ (uint32_t)tag);
    };
    // (no short circuit: straight-line code, so the waits count younger loads)
    const int s0 = (int)in(0, o[0]) & (int)(((off(v.a[0]) | off(v.a[1])) & 15u) != 0);
    const int s1 = (int)in(1, o[1]) & (int)(((off(v.b[0]) | off(v.b[1])) & 15u) != 0);
    const int s2 = (int)in(2, o[2]) & (int)(((v.c ^ tag) & 15) != 0);
    return __builtin_amdgcn_ballot_w64((s0 | s1 | s2) != 0) != 0;
  }
  // Slow path: reloads until every word carries this launch's tag or the
  // watchdog fires (pauses of the queue do not count as waiting).
  __device__ __forceinline__ void respin(const int32_t (&o)[3], Vals &v, int tag,
                                         Ctrl *ctrl) const {
    Vals u;
    WaitClock wc;
    for (int it = 0;; ++it) {
      __builtin_amdgcn_s_sleep(1);
      fetch(o, u);
      if (!stale(o, u, tag)) break;
      if ((it & 15) == 15) {
        const int st = __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(&ctrl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (st == -4) break;  // another workgroup timed out: stop waiting
        if (wc.tick() > kS4WaitTicks) {
          atomicCAS(&ctrl->status, 0, -4);
          break;
        }
      }
    }
    wc.report(ctrl);
    v = u;
  }
  // The values of step s, issued `back` steps before the next one to issue.
  __device__ __forceinline__ void finish(int s, int back, Vals &v, int tag, S4Smem<R> &sm,
                                         Ctrl *ctrl) const {
    int32_t o[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) o[x] = acc[x] - back * inc[x];
    if (stale(o, v, tag)) respin(o, v, tag, ctrl);
    const bool i0 = in(0, o[0]), i1 = in(1, o[1]), i2 = in(2, o[2]);
    auto key = [](bool ok, uint32_t w) { return ok ? (int32_t)(w & ~15u) : kNegKey; };
    int32_t *const u = dst0 + ((s + 1) & (kS4Ring - 1)) * kS4Pos;
    u[0] = key(i0, (uint32_t)v.a[0]);
    u[1] = key(i0, (uint32_t)(v.a[0] >> 32));
    u[2] = key(i0, (uint32_t)v.a[1]);
    u[3] = key(i0, (uint32_t)(v.a[1] >> 32));
    i32x4 r;
    r.x = key(i1, (uint32_t)v.b[0]);
    r.y = key(i1, (uint32_t)(v.b[0] >> 32));
    r.z = key(i1, (uint32_t)v.b[1]);
    r.w = key(i1, (uint32_t)(v.b[1] >> 32));
    dst1[(s & (kS4Ring - 1)) * (R / 4) * kS4Pos] = r;
    (&sm.ring[0][0][0][0])[dst2[s & (kS4Ring - 1)]] = key(i2, (uint32_t)v.c);
  }
};

// The compute waves' sweep of block (B0, B1, B2).
template <int R>
__device__ __forceinline__ void s4_sweep(const Sweep4Dev &sd, S4Smem<R> &sm, int B0, int B1,
                                         int B2, int tid, int gap, int tag, int total) {
  const int q1 = tid >> 4, q2 = tid & 15;
  const int sk = q1 + q2;
  const int v1 = B1 * 16 + q1, v2 = B2 * 16 + q2;
  const int n0 = sd.n[0], n3 = sd.n[3];
  const bool lane_ok = v1 <= sd.n[1] && v2 <= sd.n[2];
  const int r1 = v1 >= 1 && v1 <= sd.n[1] ? min((int)sd.seqs[n0 + v1 - 1], kS4SubMax - 1) : 0;
  const int r2 =
      v2 >= 1 && v2 <= sd.n[2] ? min((int)sd.seqs[n0 + sd.n[1] + v2 - 1], kS4SubMax - 1) : 0;
  // column scores: gap term of 1, 2 or 3 residues and the tie bits 15 - b
  const int g3 = gap * 48, g4 = gap * 64;
  const int32_t K1 = g3 + 14, K2 = g3 + 13, K4 = g3 + 11, K8 = g3 + 7, K9 = g4 + 6;
  int32_t K3 = g4 + 12, K5 = g4 + 10, K7 = g3 + 8;
  const int32_t p12 = sm.sub16[r1 * kS4SubMax + r2];
  const int32_t P6 = p12 + g4 + 9;
  // the same for the masks of three residues or more that hold dimension 3,
  // without the pair scores
  const int32_t K10 = g4 + 5, K11 = g3 + 4, K12 = g4 + 3, K13 = g3 + 2, K15 = 0;
  const int32_t P14 = p12 + g3 + 1;
  int32_t p01[R], p02[R], p7[R];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    p01[u] = sm.p03[r1][u];  // sub(r0 of row u, r1) << 4
    p02[u] = sm.p03[r2][u];
    p7[u] = p01[u] + p02[u] + p12;
  }
  const int32_t *const sub1 = sm.sub16 + r1 * kS4SubMax;
  const int32_t *const sub2 = sm.sub16 + r2 * kS4SubMax;
  // ring positions from that of (q1 - 1, q2 - 1): + 1 is (q1 - 1, q2), + kS4E
  // (q1, q2 - 1), + kS4E + 1 the lane's own
  i32x4 *const rp = reinterpret_cast<i32x4 *>(&sm.ring[0][0][q1 * kS4E + q2][0]);
  const int32_t *const up = &sm.up[0][q1 * kS4E + q2];
  constexpr int RS = R / 4 * kS4Pos;  // ring vectors per slot
  // direction lines: tile (c0, c1, c2, c3), bytes ((q0*8 + q1)*8 + q2)*8 + q3
  auto tc = [](int v) { return v == 0 ? 0 : (v - 1) / kS4T + 1; };
  auto tq = [](int v) { return v == 0 ? 0 : (v - 1) % kS4T; };
  // byte offset of the lane's line in tile row c0 = 0 (below 2^32: sweep4_eligible)
  const uint32_t dlane =
      ((uint32_t)tc(v1) * (uint32_t)sd.ts[1] + (uint32_t)tc(v2) * (uint32_t)sd.ts[2]) * kS4Dbs +
      (uint32_t)((tq(v1) * kS4T + tq(v2)) * kS4T);
  // first byte of the tile rows along dimension 0: row u = 0, and rows u >= 1,
  // which all lie in one tile
  const int rows = min(R, n0 - B0 * R + 1);
  auto drow = [&](int v0) {
    return sd.dir + (int64_t)tc(v0) * sd.ts[0] * kS4Dbs + tq(v0) * (kS4T * kS4T * kS4T);
  };
  uint8_t *const drow0 = drow(B0 * R), *const drow1 = drow(B0 * R + 1);
  // exchange stores: wave-uniform base of the step's words and a lane offset,
  // so that a store needs no vector address arithmetic
  const bool wx0 = B0 < sd.nb[0] - 1;
  const bool wx1 = B1 < sd.nb[1] - 1 && q1 == 15;
  const bool wx2 = B2 < sd.nb[2] - 1 && q2 == 15;
  int32_t *px0 = sd.x0 + ((((int64_t)B0 * sd.nb[1] + B1) * sd.nb[2] + B2) * sd.S) * kS4X0;
  int32_t *px1 =
      sd.x1 + ((((int64_t)B0 * (sd.nb[1] - 1) + B1) * sd.nb[2] + B2) * sd.S) * kS4X1<R>;
  int32_t *px2 =
      sd.x2 + ((((int64_t)B0 * sd.nb[1] + B1) * (sd.nb[2] - 1) + B2) * sd.S) * kS4X1<R>;
  // (lane (15, 15) stores to both at the same offset)
  const uint32_t ox = (uint32_t)((q1 == 15 ? q2 : q1) * R);
  const bool origin = B0 == 0 && B1 == 0 && B2 == 0;
  // the score: the corner cell is row n0 % R of lane (n1 % 16, n2 % 16)
  const bool cw = B0 == n0 / R && B1 == sd.n[1] / 16 && B2 == sd.n[2] / 16;
  const int cl1 = sd.n[1] & 15, cl2 = sd.n[2] & 15;
  const int sc = n3 + cl1 + cl2, uc = n0 % R, tcw = cl1 * 16 + cl2;

  // Direction bytes: every 4 steps the run of 4 cells (one aligned word of the
  // direction block) that ended at or before the lane's last cell is taken out
  // of the bytes of the last 8 steps; its place there is the same every time.
  const int xs = ((sk + 1) & 3) * 8;  // shift of the lane's run within two words
  const bool xz = xs == 0;
  const int cl = (n3 + 3) / 4;  // the last run (cells 4 cl - 3 .. n3)

  int32_t op[R], ap[R], bp[R], cp[R];  // own, v1 - 1, v2 - 1, both: at t - 1
  uint32_t w0[R], nw[R];  // direction bytes of the previous and the current 4 steps
#pragma unroll
  for (int u = 0; u < R; ++u) {
    op[u] = ap[u] = bp[u] = cp[u] = kNegKey;
    w0[u] = nw[u] = 0;
  }
  int32_t uo = kNegKey, ua = kNegKey, ub = kNegKey, uc7 = kNegKey;  // the row above at t - 1
  const uint8_t *s3p = sm.s3 + kS4Front - 1 - sk;  // s3p[s]: residue of cell t of step s
  int r3 = s3p[0], r3n = s3p[1];

  auto group = [&](auto pro, int s0) __attribute__((always_inline)) {
    constexpr bool kPro = decltype(pro)::value;
#pragma unroll
    for (int i = 0; i < kS4Un; ++i) {
      const int s = s0 + i;
      const int t = s - sk;
      constexpr int RM = kS4Ring - 1;
      const int32_t p13 = sub1[r3], p23 = sub2[r3];
      int32_t a[R], b[R], c[R], p03[R];
#pragma unroll
      for (int h = 0; h < R / 4; ++h) {
        const i32x4 va = rp[((i - 1) & RM) * RS + h * kS4Pos + 1];
        const i32x4 vb = rp[((i - 1) & RM) * RS + h * kS4Pos + kS4E];
        const i32x4 vc = rp[((i - 2) & RM) * RS + h * kS4Pos];
        const i32x4 vp = *reinterpret_cast<const i32x4 *>(&sm.p03[r3][4 * h]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[4 * h + e] = va[e];
          b[4 * h + e] = vb[e];
          c[4 * h + e] = vc[e];
          p03[4 * h + e] = vp[e];
        }
      }
      r3 = r3n;
      r3n = s3p[s + 2];
      const int32_t no = up[(i & RM) * kS4Pos + kS4E + 1];
      const int32_t na = up[((i - 1) & RM) * kS4Pos + 1];
      const int32_t nb = up[((i - 1) & RM) * kS4Pos + kS4E];
      const int32_t nc = up[((i - 2) & RM) * kS4Pos];
      // Opaque at every step: the compiler would otherwise keep sums with them
      // (p01 + K3 and the like, and the row above's keys plus p01, p02 and p7
      // for the next step) in six more registers per row, and spill.
      asm volatile("" : "+s"(K3), "+s"(K5), "+s"(K7));
#pragma unroll
      for (int u = 0; u < R; ++u) asm volatile("" : "+v"(p01[u]), "+v"(p02[u]), "+v"(p7[u]));
      const int32_t q10 = p13 + K10, q11 = p13 + K11, q12 = p23 + K12, q13 = p23 + K13;
      const int32_t q15 = p13 + p23 + K15, q14 = p13 + p23 + P14;
      // the row above: own, v1 - 1, v2 - 1, both, at t and at t - 1
      int32_t ro = no, ra = na, rb = nb, rc = nc, so = uo, sa = ua, sb = ub, scc = uc7;
      int32_t out[R];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int32_t f = p03[u];
        int32_t m = max(a[u] + K2, b[u] + K4);
        m = max(max(m, ra + p01[u] + K3), rb + p02[u] + K5);
        m = max(max(m, c[u] + P6), rc + p7[u] + K7);
        m = max(max(m, op[u] + K8), so + f + K9);
        m = max(max(m, ap[u] + q10), sa + p01[u] + (f + q11));
        m = max(max(m, bp[u] + q12), sb + p02[u] + (f + q13));
        m = max(max(m, cp[u] + q14), scc + p7[u] + (f + q15));
        m = max(m, ro + K1);
        if constexpr (kPro) {
          m = t < 0 ? kNegKey : m;
          if (u == 0) m = origin && sk == 0 && t == 0 ? 15 : m;  // score 0, mask 0
        }
        const int32_t o = m & ~15;
        nw[u] = __builtin_amdgcn_alignbyte((uint32_t)m, nw[u], 1);
        ro = o;
        ra = a[u];
        rb = b[u];
        rc = c[u];
        so = op[u];
        sa = ap[u];
        sb = bp[u];
        scc = cp[u];
        out[u] = o;
        op[u] = o;
        ap[u] = a[u];
        bp[u] = b[u];
        cp[u] = c[u];
      }
      uo = no;
      ua = na;
      ub = nb;
      uc7 = nc;
#pragma unroll
      for (int h = 0; h < R / 4; ++h) {
        i32x4 v = {out[4 * h], out[4 * h + 1], out[4 * h + 2], out[4 * h + 3]};
        rp[(i & RM) * RS + h * kS4Pos + kS4E + 1] = v;
      }
      if (wx0) s4_store(px0 + (uint32_t)tid, out[R - 1] | tag);
      if (wx1) {
#pragma unroll
        for (int u = 0; u < R; u += 2)
          s4_store2(px1 + (ox + u), out[u] | tag, out[u + 1] | tag);
      }
      if (wx2) {
#pragma unroll
        for (int u = 0; u < R; u += 2)
          s4_store2(px2 + (ox + u), out[u] | tag, out[u + 1] | tag);
      }
      // (opaque: kept as scalar bases)
      asm volatile("" : "+s"(px0), "+s"(px1), "+s"(px2));
      px0 += kS4X0;
      px1 += kS4X1<R>;
      px2 += kS4X1<R>;
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

// One block: set-up by all waves, then the loader and the compute waves run
// the same number of steps.  `status` takes MSA_EINVAL for a bad residue code.
template <int R>
__device__ __forceinline__ void s4_block(const Sweep4Dev &sd, S4Smem<R> &sm, int item, int alpha,
                                         int gap, int tag, int32_t *status, Ctrl *ctrl) {
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
  int rem = item;
  const int B2 = rem % sd.nb[2];
  rem /= sd.nb[2];
  const int B1 = rem % sd.nb[1];
  const int B0 = rem / sd.nb[1];
  bool bad = false;
  for (int e = tid; e < alpha * alpha; e += kS4Threads)
    sm.sub16[(e / alpha) * kS4SubMax + e % alpha] = (int32_t)sd.sub[e] * 16;
  for (int e = tid; e < alpha * R; e += kS4Threads) {
    const int cc = e / R, u = e % R;
    const int v0 = B0 * R + u;
    int r0 = v0 >= 1 && v0 <= sd.n[0] ? (int)sd.seqs[v0 - 1] : 0;
    bad = bad || r0 >= alpha;
    sm.p03[cc][u] = (int32_t)sd.sub[(r0 >= alpha ? 0 : r0) * alpha + cc] * 16;
  }
  const uint8_t *const s3 = sd.seqs + sd.n[0] + sd.n[1] + sd.n[2];
  for (int e = tid; e < kS4Front + sd.n[3] + 64; e += kS4Threads) {
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
  for (int e = tid; e < kS4Ring * R * kS4Pos; e += kS4Threads) (&sm.ring[0][0][0][0])[e] = kNegKey;
  for (int e = tid; e < kS4Ring * kS4Pos; e += kS4Threads) (&sm.up[0][0])[e] = kNegKey;
  s4_barrier();
  const int total = s4_steps(sd, B1, B2);
  if (wave == kS4Waves) {
    S4Loader<R> ld(sd, sm, B0, B1, B2, tid & 63, -3);
    typename S4Loader<R>::Vals q[kS4Pf];
    {
      // ring slots -2 and -1 and the row above's slots -2 .. 0
      typename S4Loader<R>::Vals f[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) ld.issue(f[i]);
#pragma unroll
      for (int i = 0; i < 3; ++i) ld.finish(i - 3, 3 - i, f[i], tag, sm, ctrl);
    }
#pragma unroll
    for (int i = 0; i < kS4Pf; ++i) ld.issue(q[i]);
    s4_barrier();
    for (int s0 = 0; s0 < total; s0 += kS4Un) {
#pragma unroll
      for (int i = 0; i < kS4Un; ++i) {
        ld.finish(i, kS4Pf, q[i % kS4Pf], tag, sm, ctrl);  // (slots depend on s % 4 alone)
        s4_barrier();
        ld.issue(q[i % kS4Pf]);
      }
    }
  } else {
    s4_barrier();
    s4_sweep<R>(sd, sm, B0, B1, B2, tid, gap, tag, total);
  }
}

}  // namespace

template <int R>
__global__ __launch_bounds__(kS4Threads) __attribute__((amdgpu_waves_per_eu(R == 8 ? 3 : 4)))
void sweep4_kernel(Sweep4Dev sd, Ctrl *ctrl) {
  __shared__ S4Smem<R> sm;
  if (threadIdx.x == 0) sm.item = atomicAdd(&ctrl->head, 1);
  const int alpha = ctrl->alpha;
  const int gap = ctrl->gap;
  const int tag = ctrl->sweeps % 15 + 1;
  s4_barrier();
  const int ticket = __builtin_amdgcn_readfirstlane(sm.item);
  // a ticket past the grid: the counter was not reset since the last fill
  if (ticket >= sd.nb[0] * sd.nb[1] * sd.nb[2]) return;
  if (ticket == 0 && threadIdx.x == 0) ctrl->swept = 1;
  s4_block<R>(sd, sm, __builtin_amdgcn_readfirstlane(sd.order[ticket]), alpha, gap, tag,
              &ctrl->status, ctrl);
}

int launch_sweep4(const Plan &p, char *ws, const JobDev &jd, Ctrl *ctrl, hipStream_t s) {
  Sweep4Dev sd;
  fill_sweep4dev(p, &sd);
  sd.seqs = jd.seqs;
  sd.sub = jd.sub;
  sd.dir = jd.dir;
  sd.score_out = jd.score_out;
  sd.x0 = reinterpret_cast<int32_t *>(ws + p.off_s4x);
  sd.x1 = sd.x0 + p.s4_x0;
  sd.x2 = sd.x1 + p.s4_x1;
  sd.order = reinterpret_cast<const int32_t *>(ws + p.off_s4order);
  const unsigned grid = (unsigned)(sd.nb[0] * sd.nb[1] * sd.nb[2]);
  launch_begin();
  if (p.s4_rows == 8)
    hipLaunchKernelGGL(sweep4_kernel<8>, dim3(grid), dim3(kS4Threads), 0, s, sd, ctrl);
  else
    hipLaunchKernelGGL(sweep4_kernel<4>, dim3(grid), dim3(kS4Threads), 0, s, sd, ctrl);
  return launch_end();
}

}  // namespace msa
