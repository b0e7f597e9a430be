// msa_sweep5.hip -- streaming fill of the five-sequence tensor.
//
// The tile kernel sweeps 4^5 cells at a time: more than half of its vector
// instructions go to halo and face addresses, pair tables and lanes that wait
// for their turn in the tile's skew (464 lane slots a cell, of which the 31
// candidates need about 70).  Here a workgroup owns the lines of one tile
// column along dimension 4: 4 x 4 x 4 x 4 lines (v0 .. v3), one to a lane, swept
// over the whole length.
//
//   - At step s the lane at (q0, q1, q2, q3) computes the cell t = s - q0 - q1 -
//     q2 - q3 of its line.  The neighbour at lane q - b, for a mask b over the
//     lane dimensions, was computed |b| steps earlier; its values are kept in an
//     LDS ring of 8 steps (5^4 positions: the lanes and the layers q_i = -1).
//     The 16 candidates with dimension 4 come from values this lane read or
//     computed one step earlier, so they are taken before the step's barrier.
//   - Between workgroups the 175 lanes on an upper edge of the block pass their
//     values through one exchange region, [block][step][word], each word with
//     the launch's tag (1..15) in the key's 5 low bits, which are zero in a stored
//     key.  The lanes with the same edges are consecutive words, so that a layer
//     is a few runs (by lane order, every layer touched each line of a step:
//     1.96 GB of fetch for 41^5 cells, 1.32 now).  A fifth wave loads the 369
//     words of the layers q_i = -1 kS5Pf steps ahead, again while a tag is stale.
//     A position with the dimensions N at -1 lies in the block one lower along
//     them, ahead of this one by the sum of that block's extents along N in steps.
//   - Workgroups take blocks in the order of the sum of their coordinates, so a
//     workgroup only waits for workgroups that are already running.
//
// What bounds it: a step's latency and issue together.  A step takes 0.5 us for a
// workgroup alone on its compute unit and 0.7 for four of them; its vector
// instructions are about half of the fill's time (279 M for 41^5 cells, 0.45 of
// 0.92 ms), beside 3.42 GB of exchange words and directions (3.7 TB/s).  Measured: 40^5 2.50 ms with
// the tile kernel, 0.92 now; 28^5 0.66 and 0.32.  On the way there: halo words
// loaded by the compute waves 1.47 ms (every step waited for memory); one
// workgroup a block 1.47; waiting several steps ahead after a stall, 1.78 against
// 1.70; prefetch 4 steps ahead, 3.1; 3 workgroups a compute unit (128 registers),
// 1.17 against 1.00.
//
// Per cell (Section 2, Eq. 1 for five sequences): 31 candidates key(v - b) +
// column(b), shifted by 5 bits with the tie bits 31 - b below, as in the tile
// kernel; the direction bytes go to the same blocks (edge 4), a lane's run of 4
// cells as one word.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "msa_internal.h"
#include "msa_plan.h"
#include "msa_runtime.h"

namespace msa {

namespace {

constexpr int kS5T = 4;         // lanes along dimensions 0..3, tile edge (k = 5)
constexpr int kS5Dbs = 1024;    // bytes of a direction block
constexpr int kS5Ring = 8;      // LDS ring slots (steps)
constexpr int kS5Un = 8;        // steps per unrolled group
constexpr int kS5Pf = 2;        // prefetch distance (steps)
constexpr int kS5Pos = 5 * 5 * 5 * 5;
// Ring word of position (d0, d1, d2, d3) (d_i = q_i + 1) of a slot: the strides of
// dimensions 1 and 2 are 16 and 4 modulo the 64 banks, so that a wave's 64 lanes
// (q1, q2, q3) fall in distinct banks; the slots and d0 lie in the gaps.  (Row-major
// positions: 1.1e8 bank-conflict cycles for 41^5 cells.)
constexpr int kS5Str0 = 5, kS5Str1 = 1296, kS5Str2 = 260, kS5Slot = 25;
constexpr int kS5Words = 4 * (kS5Str0 + kS5Str1 + kS5Str2 + 1) + (kS5Ring - 1) * kS5Slot + 1;
static_assert(kS5Str1 % 64 == 16 && kS5Str2 % 64 == 4 && kS5Slot >= 5 * kS5Str0 &&
                  kS5Str2 >= kS5Ring * kS5Slot && kS5Str1 >= 4 * kS5Str2 + kS5Ring * kS5Slot,
              "distinct words and banks");
constexpr int kS5Halo = kS5Pos - 256;
constexpr int kS5Front = 16;    // table entries before cell 0 (largest skew 12)
constexpr int kS5Row = kS5Front + kS5SeqMax + 41;
constexpr int kS5Threads = 5 * 64;  // four compute waves and the one for the exchange
constexpr int32_t kS5WaitTicks = 200000000;  // 2 s of waiting (WaitClock ticks)
static_assert(tile_edge_for_k(5) == kS5T, "same blocks as the tile kernel");
static_assert(kS5Un == kS5Ring && kS5Un % kS5Pf == 0, "slots fixed per group");

struct S5Smem {
  int32_t ring[kS5Words];
  int32_t pk[4 * kS5T][kS5Row];  // sub(r_i(q), r_4(t)) << 5, row i * 4 + q, entry t + kS5Front
  int8_t sub[kS4SubMax * kS4SubMax];
  uint8_t s4[kS5SeqMax];
  uint16_t halo[kS5Halo];        // the tables below
  uint8_t word[256], lane[192];
  int32_t job, item;             // the next block
};

// The ring positions with some q_i = -1: digits q_i + 1, 3 bits each.
struct S5HaloList {
  uint16_t v[kS5Halo];
  constexpr S5HaloList() : v() {
    int p = 0;
    for (int x = 0; x < kS5Pos; ++x) {
      const int d0 = x / 125, d1 = x / 25 % 5, d2 = x / 5 % 5, d3 = x % 5;
      if (d0 == 0 || d1 == 0 || d2 == 0 || d3 == 0)
        v[p++] = (uint16_t)(d0 << 9 | d1 << 6 | d2 << 3 | d3);
    }
  }
};
__device__ const S5HaloList kS5HaloList{};

// Exchange word of a lane, by the digits q_i (2 bits each, q_0 highest; 3 for the
// edge lane of a block one cell thick): lanes with the same set of q_i = 3 side by
// side, the 81 without any last (they have no word).
struct S5Words {
  uint8_t v[256];
  uint8_t lane[256];  // and back
  constexpr S5Words() : v(), lane() {
    int p = 0;
    for (int set = 15; set >= 0; --set)  // (bit 3: q_3 .. bit 0: q_0)
      for (int x = 0; x < 256; ++x) {
        const int have = ((x & 3) == 3 ? 8 : 0) | ((x >> 2 & 3) == 3 ? 4 : 0) |
                         ((x >> 4 & 3) == 3 ? 2 : 0) | ((x >> 6) == 3 ? 1 : 0);
        if (have == set) {
          lane[p] = (uint8_t)x;
          v[x] = (uint8_t)p++;
        }
      }
  }
};
__device__ const S5Words kS5WordOf{};

// Ring strides, and the offset from a position to its neighbour at q - b.
__device__ constexpr int s5_stride(int i) {
  return i == 0 ? kS5Str0 : i == 1 ? kS5Str1 : i == 2 ? kS5Str2 : 1;
}
__device__ constexpr int s5_off(int b) {
  int o = 0;
  for (int i = 0; i < 4; ++i)
    if (b >> i & 1) o += s5_stride(i);
  return o;
}

__device__ __forceinline__ void s5_tables(S5Smem &sm) {
  for (int e = threadIdx.x; e < kS5Halo; e += kS5Threads) sm.halo[e] = kS5HaloList.v[e];
  if (threadIdx.x < 256) sm.word[threadIdx.x] = kS5WordOf.v[threadIdx.x];
  if (threadIdx.x < 192) sm.lane[threadIdx.x] = kS5WordOf.lane[threadIdx.x];
}

// LDS accesses of this wave complete, then every wave of the workgroup meets.
__device__ __forceinline__ void s5_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ int s5_lane() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
}

// status takes `code` unless it has one.  (The constants are formed here, not kept
// in registers across the persistent loop.)
__device__ __forceinline__ void s5_report(int32_t *status, int code) {
  int none = 0;
  asm volatile("" : "+v"(none), "+v"(code));
  atomicCAS(status, none, code);
}

// A ticket, by one lane of a wave that stays together.
__device__ __forceinline__ int s5_take(int32_t *head) {
  const int got = atomicAdd(head, s5_lane() == 0 ? 1 : 0);
  return __builtin_amdgcn_readfirstlane(got);
}

// The wave beside the compute waves.  During step s it writes the halo of ring
// slot s (six words a lane, loaded kS5Pf steps before), stores the exchange words
// of step s - 1, and issues the loads of step s + kS5Pf.  (In the compute waves, two
// words a lane: every step waited for memory, 0.97 us a step of a workgroup alone.)
struct S5Aux {
  static constexpr int E = (kS5Halo + 63) / 64;
  static constexpr int W = (kS5Step + 63) / 64;
  const char *x0;
  uint32_t hoff[E];  // byte offset of the word of step 0 in the exchange region
  int hlo[E];        // the word is there in the steps hlo .. hlo + n4 (1 << 30: never)
  int hdst[E];       // ring words
  int n4, lane;
  int32_t *xp;       // the block's slice
  const int32_t *src[W];
  bool dead = false;  // given up waiting (a time-out)

  __device__ __forceinline__ S5Aux(const Sweep5Dev &sd, S5Smem &sm, int item, const int (&c)[4],
                                   const int (&ext)[4], int lane_)
      : x0(reinterpret_cast<const char *>(sd.x)), n4(sd.n[4]), lane(lane_),
        xp(sd.x + (int64_t)item * sd.S * kS5Step) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      int x = lane + 64 * e;
      x = x < kS5Halo ? x : x - 64;  // (no word left: the one before once more)
      const int w = sm.halo[x];
      bool there = true;
      int pos = 0, sum = 0, off = 0, blk = 0, ln = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int d = w >> (9 - 3 * i) & 7;  // q_i + 1
        const bool low = d == 0;
        const int e1 = c[i] - 1 <= 0 ? 1 : kS5T;  // the lower block's extent
        // (a lane past the block's extent holds no cell, and its last steps may not run)
        there = there && !(low && c[i] == 0) && d <= ext[i];
        pos += d * s5_stride(i);
        sum += d - 1;
        off += low ? e1 : 0;
        blk = blk * sd.nb[i] + c[i] - (low ? 1 : 0);
        ln = ln * 4 + (low ? 3 : ext[i] == 1 ? 3 : d - 1);
      }
      hdst[e] = pos;
      hlo[e] = there ? sum : 1 << 30;
      hoff[e] = there ? (((uint32_t)blk * (uint32_t)sd.S + (uint32_t)off) * (uint32_t)kS5Step +
                         (uint32_t)sm.word[ln & 255]) * 4u
                      : 0u;
      asm volatile("" ::: "memory");  // (one word after the other: fewer registers)
    }
    // the ring words of the lanes in the order of their exchange words
#pragma unroll
    for (int y = 0; y < W; ++y) {
      const int x = sm.lane[lane + 64 * y];
      src[y] = sm.ring;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int d = x >> (6 - 2 * i) & 3;
        src[y] += ((ext[i] == 1 ? d ^ 3 : d) + 1) * s5_stride(i);
      }
    }
  }
  __device__ __forceinline__ void issue(int32_t (&w)[E], int s) const {
    const char *const p = x0 + (int64_t)s * (kS5Step * 4);
#pragma unroll
    for (int e = 0; e < E; ++e)
      w[e] = __hip_atomic_load(reinterpret_cast<const int32_t *>(p + hoff[e]), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
  }
  // some word of step s is not yet this launch's
  __device__ __forceinline__ bool stale(const int32_t (&w)[E], int s, int tag) const {
    uint32_t st = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const uint32_t off = (uint32_t)(w[e] ^ tag) & 31u;
      st |= (uint32_t)(s - hlo[e]) <= (uint32_t)n4 ? off : 0u;
    }
    return __builtin_amdgcn_ballot_w64(st != 0) != 0;
  }
  __device__ __forceinline__ void settle(int32_t (&w)[E], int s, int slot, int tag, S5Smem &sm,
                                         Ctrl *ctrl, int32_t wlim) {
    if (stale(w, s, tag) && !dead) {
      // (WaitClock in 32 bits, its bounds formed here)
      uint32_t last = (uint32_t)wall_clock64(), waited = 0, pause = 0;
      uint32_t most = (uint32_t)kPauseTicks;
      asm volatile("" : "+s"(most));
      for (int it = 0;; ++it) {
        __builtin_amdgcn_s_sleep(1);
        issue(w, s);
        if (!stale(w, s, tag)) break;
        if ((it & 15) == 15) {
          const int st = __builtin_amdgcn_readfirstlane(
              __hip_atomic_load(&ctrl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
          const uint32_t now = (uint32_t)wall_clock64(), d = now - last;
          last = now;
          if (d < most) waited += d;
          else pause = d > pause ? d : pause;
          if (waited > (uint32_t)wlim || st == -4) {  // (or another workgroup timed out)
            dead = true;           // the rest of the block waits for nothing
            break;
          }
        }
      }
      if (pause > 0)
        __hip_atomic_fetch_max(&ctrl->max_pause, (int64_t)pause, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
      sm.ring[slot * kS5Slot + hdst[e]] =
          (uint32_t)(s - hlo[e]) <= (uint32_t)n4 ? w[e] & ~31 : kNegKey;
  }
  // The exchange words of the step in `slot`, in the order of the words.  (Stored
  // by the lanes that computed them, in 11 lines of which each wave writes parts:
  // 1.35 GB of writes for 41^5 cells against 0.76, and a fill of 1.9 ms against 1.5.)
  __device__ __forceinline__ void pass_on(int slot, int tag) {
#pragma unroll
    for (int y = 0; y < W; ++y)
      if (lane + 64 * y < kS5Step)
        __hip_atomic_store(xp + lane + 64 * y, src[y][slot * kS5Slot] | tag, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    xp += kS5Step;
  }
  // next(ticket) leaves the block of a ticket in sm (-1: none); `head` counts
  // them.  more: there are blocks beyond each workgroup's first.
  template <class Next>
  __device__ __forceinline__ void run(int total, int tag, S5Smem &sm, Ctrl *ctrl, int32_t wlim,
                                      int32_t *head, bool more, Next next) {
    int ticket = -1;
    int32_t q[kS5Pf][E];
    {
      int32_t f[4][E];  // the halo of the steps before the first
#pragma unroll
      for (int i = 0; i < 4; ++i) issue(f[i], i - 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        settle(f[i], i - 4, i + 4, tag, sm, ctrl, wlim);
        if (i < kS5Pf) issue(q[i], i);
      }
    }
    s5_barrier();
    for (int s0 = 0; s0 < total; s0 += kS5Un) {
      // the next block is taken early (it waits for lower tickets alone, this
      // block's among them)
      if (more && s0 + kS5Un >= total) ticket = s5_take(head);
#pragma unroll
      for (int i = 0; i < kS5Un; ++i) {
        settle(q[i % kS5Pf], s0 + i, i, tag, sm, ctrl, wlim);
        if (i > 0 || s0 > 0) pass_on((i - 1) & (kS5Ring - 1), tag);
        s5_barrier();
        issue(q[i % kS5Pf], s0 + i + kS5Pf);
      }
    }
    pass_on(kS5Ring - 1, tag);
    if (dead) sweep_timed_out(ctrl, sm.job, sm.item);  // (here, where few registers are in use)
    next(ticket);
  }
};

template <class Next>
__device__ __forceinline__ void s5_block(const Sweep5Dev &sd_, S5Smem &sm, int item, int alpha,
                                         int gap, int tag, int32_t *status, Ctrl *ctrl,
                                         int32_t wlim, int wave, int32_t *head, bool more,
                                         Next next) {
  // (the thread index from the wave's and the lane's, so that none of it, nor what
  // follows from it, is kept in vector registers across blocks)
  int tid = wave * 64 + s5_lane();
  asm volatile("" : "+v"(tid));
  // (the sizes are opaque for the same reason)
  Sweep5Dev sd = sd_;
#pragma unroll
  for (int i = 0; i < 4; ++i) asm volatile("" : "+s"(sd.n[i]), "+s"(sd.nb[i]), "+s"(sd.ts[i]));
  asm volatile("" : "+s"(sd.n[4]), "+s"(sd.S), "+s"(alpha), "+s"(gap), "+s"(tag), "+s"(wlim));
  const int n4 = sd.n[4];
  // ---- the block: coordinates c_i, first cells lo_i, extents ext_i ----
  int c[4], lo[4], ext[4];
  {
    int rem = item;
#pragma unroll
    for (int i = 3; i >= 0; --i) {
      // (the quotient of a uniform division is formed in vector registers)
      const int up = __builtin_amdgcn_readfirstlane(rem / sd.nb[i]);
      c[i] = rem - up * sd.nb[i];
      rem = up;
      lo[i] = c[i] == 0 ? 0 : (c[i] - 1) * kS5T + 1;
      ext[i] = c[i] == 0 ? 1 : min(kS5T, sd.n[i] - (c[i] - 1) * kS5T);
    }
  }
  int tail = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) tail += ext[i] - 1;
  // the last run of 4 cells ends at cell 4 * ceil(n4 / 4)
  const int total = ((n4 + 3) / 4 * 4 + 1 + tail + kS5Un - 1) / kS5Un * kS5Un;

  // ---- before step 0 the ring holds cells t < 0: -infinity ----
#pragma unroll 1
  for (int e = tid; e < kS5Words; e += kS5Threads) sm.ring[e] = kNegKey;
  if (wave == 4) {
    s5_barrier();  // the ring is set
    S5Aux aux(sd, sm, item, c, ext, tid & 63);
    aux.run(total, tag, sm, ctrl, wlim, head, more, next);
    return;
  }
  // ---- matrix and fifth sequence in LDS, residues, pair scores ----
  bool bad = false;
  {
    const uint8_t *const s4 = sd.seqs + sd.n[0] + sd.n[1] + sd.n[2] + sd.n[3];
#pragma unroll 1
    for (int e = tid; e < alpha * alpha; e += 256) sm.sub[e] = sd.sub[e];
    if (tid < n4) {
      const int x = (int)s4[tid];
      bad = x >= alpha;
      sm.s4[tid] = (uint8_t)(x >= alpha ? 0 : x);
    }
  }
  int q[4], r[4], sk = 0;
  bool lane_ok = true;
  {
    int so = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      q[i] = tid >> (6 - 2 * i) & 3;
      sk += q[i];
      lane_ok = lane_ok && q[i] < ext[i];
      const int v = lo[i] + q[i];
      r[i] = v >= 1 && v <= sd.n[i] ? (int)sd.seqs[so + v - 1] : 0;
      bad = bad || r[i] >= alpha;
      r[i] = r[i] >= alpha ? 0 : r[i];
      so += sd.n[i];
    }
  }
  const int row = tid >> 4;  // row of pair scores this lane fills with 15 others
  int rrow;
  {
    const int i = row >> 2;
    int so = 0, vi = 0, ni = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      so += x < i ? sd.n[x] : 0;
      vi = x == i ? lo[x] + (row & 3) : vi;
      ni = x == i ? sd.n[x] : ni;
    }
    rrow = vi >= 1 && vi <= ni ? (int)sd.seqs[so + vi - 1] : 0;
    rrow = (rrow >= alpha ? 0 : rrow) * alpha;
  }
  s5_barrier();
#pragma unroll 1
  for (int e = tid & 15; e < kS5Front + n4 + 41; e += 16) {
    const int t = e - kS5Front;
    const int r4 = sm.s4[t >= 1 && t <= n4 ? t - 1 : 0];
    sm.pk[row][e] = (int32_t)sm.sub[rrow + (t >= 1 && t <= n4 ? r4 : 0)] * 32;
  }
  if (bad) s5_report(status, -1);
  // column scores of the lane dimensions' masks: pairs, gap term, tie bits
  int32_t lc[16];
  const int32_t g1 = gap * 4 * 32, g2 = gap * 6 * 32;  // 1 or 4, 2 or 3 residues (5: 0)
  {
    int32_t pr[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = i + 1; j < 4; ++j) pr[i][j] = (int32_t)sm.sub[r[i] * alpha + r[j]] * 32;
#pragma unroll
    for (int b = 1; b < 16; ++b) {
      const int cb = __builtin_popcount(b);
      int32_t x = (cb == 1 || cb == 4 ? g1 : g2) + 31 - b;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = i + 1; j < 4; ++j)
          if ((b >> i & 1) && (b >> j & 1)) x += pr[i][j];
      lc[b] = x;
    }
  }
  // what dimension 4 adds to the constant, by the number of lane residues
  const int32_t D1 = g2 - g1 - 16, D2 = -16, D3 = g1 - g2 - 16, D4 = -g1 - 16;
  const int32_t K16 = g1 + 31 - 16;

  s5_barrier();  // the tables and the halo of the steps before the first are there

  // ---- the sweep ----
  const int32_t *const pkp = &sm.pk[0][0] + kS5Front - sk;
  const int32_t *const pk0 = pkp + q[0] * kS5Row, *const pk1 = pkp + (4 + q[1]) * kS5Row,
                *const pk2 = pkp + (8 + q[2]) * kS5Row, *const pk3 = pkp + (12 + q[3]) * kS5Row;
  int32_t *const own = &sm.ring[s5_off(15) + q[0] * kS5Str0 + q[1] * kS5Str1 + q[2] * kS5Str2 + q[3]];
  const bool origin = item == 0;
  const bool cw = c[0] == sd.nb[0] - 1 && c[1] == sd.nb[1] - 1 && c[2] == sd.nb[2] - 1 &&
                  c[3] == sd.nb[3] - 1;
  const int sc = n4 + tail;
  const int tcw = ((ext[0] - 1) * 64) + ((ext[1] - 1) * 16) + ((ext[2] - 1) * 4) + ext[3] - 1;
  uint8_t *const dbase =
      sd.dir + ((int64_t)c[0] * sd.ts[0] + (int64_t)c[1] * sd.ts[1] + (int64_t)c[2] * sd.ts[2] +
                (int64_t)c[3] * sd.ts[3]) * kS5Dbs;
  const int xs = ((sk + 1) & 3) * 8;
  const bool xz = xs == 0;
  const int cl = (n4 + 3) / 4;
  uint32_t dw0 = 0, dnw = 0;
  int32_t m16 = kNegKey;  // the best candidate with dimension 4, taken one step ahead
  int32_t nv[16];         // neighbours at q - b
  auto far_reads = [&](int i) __attribute__((always_inline)) {  // for step i: two steps back and more
#pragma unroll
    for (int b = 1; b < 16; ++b) {
      const int lag = __builtin_popcount(b);
      if (lag >= 2) nv[b] = own[((i - lag) & (kS5Ring - 1)) * kS5Slot - s5_off(b)];
    }
  };
  far_reads(0);
  auto group = [&](auto pro, int s0) __attribute__((always_inline)) {
    constexpr bool kPro = decltype(pro)::value;
#pragma unroll
    for (int i = 0; i < kS5Un; ++i) {
      const int s = s0 + i;
      const int t = s - sk;
#pragma unroll
      for (int x = 0; x < 4; ++x)
        nv[1 << x] = own[((i - 1) & (kS5Ring - 1)) * kS5Slot - s5_off(1 << x)];
      const int32_t p0 = pk0[s + 1], p1 = pk1[s + 1], p2 = pk2[s + 1], p3 = pk3[s + 1];
      int32_t m = m16;
#pragma unroll
      for (int y = 0; y < 15; ++y) {
        // (masks of two and more first: their values are here already)
        constexpr int kOrder[15] = {3, 5, 6, 9, 10, 12, 7, 11, 13, 14, 15, 1, 2, 4, 8};
        const int b = kOrder[y];
        m = max(m, nv[b] + lc[b]);
      }
      if constexpr (kPro) {
        m = t < 0 ? kNegKey : m;
        m = origin && sk == 0 && t == 0 ? 31 : m;  // score 0, mask 0
      }
      const int32_t out = m & ~31;
      own[i * kS5Slot] = out;
      dnw = __builtin_amdgcn_alignbyte((uint32_t)m, dnw, 1);
      {
        // ---- candidates with dimension 4 of step s + 1 ----
        const int32_t p01 = p0 + p1 + D2, p23 = p2 + p3 + D2;
        const int32_t ps[16] = {0,
                                p0 + D1,
                                p1 + D1,
                                p01,
                                p2 + D1,
                                p0 + p2 + D2,
                                p1 + p2 + D2,
                                p01 + p2 + (D3 - D2),
                                p3 + D1,
                                p0 + p3 + D2,
                                p1 + p3 + D2,
                                p01 + p3 + (D3 - D2),
                                p23,
                                p23 + p0 + (D3 - D2),
                                p23 + p1 + (D3 - D2),
                                p01 + p23 + (D4 - 2 * D2)};
        int32_t x = out + K16;
#pragma unroll
        for (int b = 1; b < 16; ++b) x = max(x, nv[b] + lc[b] + ps[b]);
        m16 = x;
      }
      far_reads(i + 1);
      if (cw && s == sc) {  // wave-uniform
        if (tid == tcw) *sd.score_out = (int64_t)(out >> 5);
      }
      s5_barrier();
      if (i % 4 == 3) {
        const int c4 = (s - sk) >> 2;  // run c4: cells 4 c4 - 3 .. 4 c4
        const uint32_t wv = __builtin_amdgcn_alignbit(dnw, dw0, xs);
        const uint32_t run = xz ? dnw : wv;
        dw0 = dnw;
        if (lane_ok && c4 >= 1 && c4 <= cl)
          *reinterpret_cast<uint32_t *>(dbase + ((uint32_t)c4 * kS5Dbs + (uint32_t)tid * 4)) = run;
        if constexpr (kPro)
          if (lane_ok && c4 == 0) dbase[(uint32_t)tid * 4] = (uint8_t)(run >> 24);  // cell 0
      }
    }
  };
  int s0 = 0;
  // cells t < 0 and t = 0 fall in the first steps (largest skew 12)
  for (; s0 < total && s0 < 16; s0 += kS5Un) group(std::true_type{}, s0);
  for (; s0 < total; s0 += kS5Un) group(std::false_type{}, s0);
}

}  // namespace

// Persistent workgroups: a block is short (57 steps for 40 residues), and a
// workgroup a block cost 50 ns a block, in a row, beside the steps (14641 blocks of
// 41^5 cells: 1.47 ms).
__global__ __launch_bounds__(kS5Threads) __attribute__((amdgpu_waves_per_eu(5)))
void sweep5_kernel(Sweep5Dev sd, Ctrl *ctrl) {
  __shared__ S5Smem sm;
  const int alpha = ctrl->alpha;
  const int gap = ctrl->gap;
  const int tag = sweep_tag(ctrl->sweeps, kSweepTags);
  const int total = sd.nb[0] * sd.nb[1] * sd.nb[2] * sd.nb[3];
  const bool more = total > (int)gridDim.x;
  auto next = [&](int ticket) {
    sm.job = 0;
    sm.item = ticket >= 0 && ticket < total ? sd.order[ticket] : -1;
  };
  s5_tables(sm);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x) >> 6;
  if (wave == 0) {
    const int ticket = s5_take(&ctrl->head);
    if (ticket == 0) ctrl->swept = 1;
    next(ticket);
  }
  for (;;) {
    s5_barrier();  // the next block is known, the last one's LDS read no more
    const int item = __builtin_amdgcn_readfirstlane(sm.item);
    if (item < 0) break;
    s5_block(sd, sm, item, alpha, gap, tag, &ctrl->status, ctrl, kS5WaitTicks, wave, &ctrl->head, more,
             next);
  }
}

// ---------------------------------------------------------------------------
// Batched launches: the blocks of all k = 5 jobs from one queue.
// ---------------------------------------------------------------------------

// A block goes to the next slot of its coordinate sum's (kbase: where the host
// placed the job's blocks of that sum; their order there does not matter).
__global__ __launch_bounds__(256) void batch_s5queue_kernel(const BatchArgs *__restrict__ a) {
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
    const Sweep5Dev &sd = a->s5jobs[lo];
    const int b = g - pre[lo];
    int rem = b, key = 0;
    for (int i = 3; i >= 0; --i) {
      key += rem % sd.nb[i];
      rem /= sd.nb[i];
    }
    const int slot = atomicAdd(sd.kbase + key, 1);
    q[2 * slot] = lo;
    q[2 * slot + 1] = b;
  }
}

__global__ __launch_bounds__(kS5Threads) __attribute__((amdgpu_waves_per_eu(5)))
void batch_sweep5_kernel(const BatchArgs *__restrict__ a, Ctrl *ctrl) {
  __shared__ S5Smem sm;
  const int total = __builtin_amdgcn_readfirstlane(a->s4total);
  const int tag = __builtin_amdgcn_readfirstlane(a->s4tag);
  const int32_t *const q = as_global(a->s4q);
  const Sweep5Dev *const jobs = as_global(a->s5jobs);
  const int64_t wl =
      __hip_atomic_load(&ctrl->wait_limit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int32_t wlim =
      __builtin_amdgcn_readfirstlane(wl > 0 ? (int)min(wl, (int64_t)INT32_MAX) : kS5WaitTicks);
  auto next = [&](int ticket) {
    const bool some = ticket >= 0 && ticket < total;
    sm.job = some ? q[2 * ticket] : 0;
    sm.item = some ? q[2 * ticket + 1] : -1;
  };
  if (total == 0) return;
  s5_tables(sm);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x) >> 6;
  if (wave == 0) next(s5_take(&ctrl->s4head));
  for (;;) {
    s5_barrier();
    const int item = __builtin_amdgcn_readfirstlane(sm.item);
    if (item < 0) break;
    const int job = __builtin_amdgcn_readfirstlane(sm.job);
    // the job's descriptor, kept in scalar registers
    Sweep5Dev sd;
    {
      const uint32_t *const src = reinterpret_cast<const uint32_t *>(jobs + job);
      uint32_t w[sizeof(Sweep5Dev) / 4];
#pragma unroll
      for (int i = 0; i < (int)(sizeof(Sweep5Dev) / 4); ++i)
        w[i] = __builtin_amdgcn_readfirstlane(src[i]);
      __builtin_memcpy(&sd, w, sizeof(sd));
    }
    sd.seqs = as_global(sd.seqs);
    sd.sub = as_global(sd.sub);
    sd.x = as_global(sd.x);
    sd.dir = as_global(sd.dir);
    sd.score_out = as_global(sd.score_out);
    sd.status = as_global(sd.status);
    s5_block(sd, sm, item, sd.alpha, sd.gap, tag, sd.status, ctrl, wlim, wave, &ctrl->s4head,
             total > (int)gridDim.x, next);
  }
}

// Four workgroups fit a compute unit.
void launch_batch_sweep5(const BatchArgs *d_args, Ctrl *ctrl, hipStream_t s) {
  hipLaunchKernelGGL(batch_s5queue_kernel, dim3(256), dim3(256), 0, s, d_args);
  hipLaunchKernelGGL(batch_sweep5_kernel, dim3((unsigned)(device_cu_count() * 4)),
                     dim3(kS5Threads), 0, s, d_args, ctrl);
}

int launch_sweep5(const Plan &p, char *ws, const JobDev &jd, Ctrl *ctrl, hipStream_t s) {
  Sweep5Dev sd;
  fill_sweep5dev(p, &sd);
  sd.seqs = jd.seqs;
  sd.sub = jd.sub;
  sd.dir = jd.dir;
  sd.score_out = jd.score_out;
  sd.x = reinterpret_cast<int32_t *>(ws + p.off_faces) + kS5PadFront;
  sd.order = reinterpret_cast<const int32_t *>(ws + p.off_s4order);
  const int blocks = sd.nb[0] * sd.nb[1] * sd.nb[2] * sd.nb[3];
  const int fit = device_cu_count() * 4;
  launch_begin();
  hipLaunchKernelGGL(sweep5_kernel, dim3((unsigned)(blocks < fit ? blocks : fit)),
                     dim3(kS5Threads), 0, s, sd, ctrl);
  return launch_end();
}

}  // namespace msa
