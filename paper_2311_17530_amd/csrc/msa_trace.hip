// msa_trace.hip -- traceback by several walkers, the co-optimal list built on
// it, and the near-optimal list.
//
// The walk from the far corner (Section 2) is a chain of dependent reads, one
// per column: a single wave took 0.13 us a column and 0.5 us a tile crossing.
// But the walk from a cell depends on the cell alone, so two walks that meet in
// a cell are one walk from there on, and walks that start near an optimal path
// meet it soon.  So one workgroup walks the alignment in pieces at once: wave
// 0 from the end cell, the others from guessed cells on the way to the origin.
// Cells are told apart by their coordinate sum h, which every step lowers.  A
// guessed walker owns the sums from its start down to the next guess's, where
// it records its cells and masks by h; below, it compares its cell with the
// next owner's record at the same h and stops when they are equal.  The
// alignment is the end cell's walk up to its meeting with a guessed walk, that
// one's up to its meeting with the next, and so on.  A walk that met nobody
// within the next range is continued by wave 0 alone, so the result is the
// single walk's whatever the guesses were worth.
//
// The guesses lie on the straight line to the origin; where the lengths are
// far apart (a path of such sequences runs along the diagonal and has its
// gaps at one end), on three lines: the straight one, the diagonal from the
// origin and the diagonal from the end cell, each a family with ranges and
// records of its own, and wave 0 watches for all of them.
//
// What bounds it: the latency of a tile crossing (a walker waits 1 to 2 us for
// the next tile's directions, at every fourth column or so) times the columns
// of the longest piece.  Measured, single walk and walkers: related sequences
// 384^3 94 and 25 us, 128^4 69 and 29, 40^5 57 and 16; unrelated ones, whose walks
// meet late, 384^3 106 and 78, 128^4 68 and 66, 40^5 76 and 32.  Short walks, and
// those of many jobs at once, keep the single wave (trace_by_walkers).
//
// Co-optimal alignments (co-optimal mode, k <= 3): the depth-first enumeration
// takes at every new cell the lowest mask of its tie set, so below a cell of
// the first alignment (the one the walkers found) a new alignment goes on like
// the first one.  Only the columns between a tie and the meeting are walked;
// the rest of the stack is copied.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "msa_internal.h"
#include "msa_runtime.h"

namespace msa {

namespace {

enum { ST_OK = 0, ST_EINVAL = -1, ST_EDEVICE = -4 };

constexpr int kTrWalkers = 16;
constexpr int kTrThreads = kTrWalkers * 64;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int K>
struct TrCfg {
  static constexpr int T = tile_edge_for_k(K);
  static constexpr int M = (1 << K) - 1;
  static constexpr int DBS = (ipow(T, K) + 15) / 16 * 16;
  static constexpr int dstride(int i) { return ipow(T, K - 1 - i); }
};

// The lane, and the thread index from the wave's (a scalar) and it, opaque: what
// follows from them is formed where it is used instead of being kept in vector
// registers across a batched launch's jobs, as is the kernel's own index.
__device__ __forceinline__ int tr_lane() {
  int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
  asm volatile("" : "+v"(lane));
  return lane;
}
__device__ __forceinline__ int tr_wave() {
  return __builtin_amdgcn_readfirstlane((int)threadIdx.x) >> 6;
}

// How a walk ended.
enum { kTrMerged = 0, kTrOpen = 1, kTrEnd = 2, kTrBad = 3 };

// Families of guesses (k = 5, whose sequences are short and whose walk takes
// the most registers: the straight line alone).
template <int K> constexpr int kTrFam = K <= 4 ? 3 : 1;
// LDS bytes of the records: per sum and family a cell (8 bytes), the owner's
// mask and the overlap's, and per sum the path's mask.
constexpr int kTrRec = 92 * 1024;
constexpr int tr_rec_bytes(int fam, int total) { return (total + 1) * (10 * fam + 1); }
static_assert(tr_rec_bytes(1, kTrMaxTotal) <= kTrRec, "records of one family fit");

template <int K>
struct TrSmem {
  alignas(16) uint8_t dirb[kTrWalkers][TrCfg<K>::DBS];  // each walker's tile
  alignas(16) uint8_t rec[kTrRec];
  int32_t state[kTrWalkers], hstop[kTrWalkers], hstart[kTrWalkers];
  int32_t vstop[kTrWalkers][K];
  int32_t hend, status;
  int32_t seg[kTrWalkers][3], ns;  // the path's stretches: lowest and highest walker, first sum
  int32_t done, never;  // the path is known; 0 for wave 0's own walks
  int32_t vend[K];  // the walk's last cell
  int32_t cnt[kTrWalkers][K + 1];
};

// The records of families f < F for sums 0 .. H.
struct TrRec {
  uint64_t *pos;  // [f][h]: the owner's cell (v_0 .. v_{k-2}, 16 bits each)
  uint8_t *own;   // [f][h]: its mask there (0: it has no cell with that sum)
  uint8_t *ov;    // [f][h]: the mask of the walker from the range above
  uint8_t *path;  // [h]: the path's mask
  int n;          // H + 1
  template <int K>
  __device__ __forceinline__ TrRec(TrSmem<K> &sm, int F, int H) : n(H + 1) {
    pos = reinterpret_cast<uint64_t *>(sm.rec);
    own = sm.rec + (size_t)F * n * 8;
    ov = own + F * n;
    path = ov + F * n;
  }
};

// One walk from cell v (sum h), wave-uniform.  Above sum h_own it records its
// cells and masks in family `fam`; from there down it watches the families f0
// .. f0 + nf - 1, writes its masks to `to` and stops where it meets one (met),
// or at a sum h_stop or less (-1: never), or at a tile's entry once `done` is
// set.  On return v, h is the cell where it stopped.
//
// Wave 0 (main: h_own is the end cell's sum, no records) watches only where it
// enters a tile: walks that met stay together, and its steps are the longest
// chain where the guesses are worth little.  The others watch one family at
// every step, since a range may be shorter than a tile.  (Wave 0 watching at
// every step, three families: unrelated sequences 40^3 21.7 us against 15.4, 96^3
// 46 and 29; the others watching at entries alone: related sequences 128^3 27 us
// against 15.)
template <int K, bool egf, bool coopt, bool main>
__device__ __forceinline__ int tr_walk(const JobDev &jd, const TrRec &rc, uint8_t *dirb, int (&v)[K], int &h,
                       int h_own, int h_stop, int fam, int f0, int nf, uint8_t *to, int &met,
                       const int32_t &done) {
  using C = TrCfg<K>;
  constexpr int T = C::T;
  constexpr int M = C::M;
  constexpr int NQ = C::DBS / 16;      // 16-byte chunks per direction block
  constexpr int CPL = (NQ + 63) / 64;  // chunks per lane
  const int lane = tr_lane();
  u32x4 *const lds4 = reinterpret_cast<u32x4 *>(dirb);
  uint8_t *const own = rc.own + fam * rc.n;
  int c[K], q[K];
  int64_t t = 0;
  {
    bool all = true, any = false;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      all = all && v[i] == 0;
      any = any || v[i] == 0;
      c[i] = v[i] == 0 ? 0 : (v[i] - 1) / T + 1;
      t += (int64_t)c[i] * jd.tstride[i];
    }
    if (egf ? any : all) return kTrEnd;
  }
  {
    const u32x4 *src = reinterpret_cast<const u32x4 *>(jd.dir + t * C::DBS);
    for (int idx = lane; idx < NQ; idx += 64) lds4[idx] = src[idx];
  }
  u32x4 pf[K][CPL];
  // Per lane l, what a step by mask l subtracts: of the byte offset in the
  // tile, of the cell packed in two words, of the tile position packed with a
  // guard bit per dimension (cleared when the position leaves the tile) and of
  // h.  A step reads them by readlane instead of forming them bit by bit.
  constexpr int QW = K == 5 ? 6 : 8;  // bits per packed tile position
  static_assert(K * QW <= 32 && T <= 1 << (QW - 1), "packed tile positions");
  uint32_t guards = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) guards |= 1u << (QW * i + QW - 1);
  int loff = 0, lh = 0;
  uint32_t llo = 0, lhi = 0, lq = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const uint32_t bit = (uint32_t)(lane & M) >> i & 1u;
    loff += (int)bit * C::dstride(i);
    lh += (int)bit;
    lq |= bit << (QW * i);
    if (i < K - 1) (i < 2 ? llo : lhi) |= bit << (16 * (i & 1));
  }
  // the watched records of sums w0 - lane, read again every kTrWin sums (an
  // owner may be writing them: what is not there yet is no meeting)
  constexpr int kTrWin = 16;
  uint64_t win = 0;
  int w0 = INT32_MAX;
  for (;;) {
    if (h <= h_own && h > 0 && __hip_atomic_load(&done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
      return kTrOpen;  // the path is known without this walk
    int d = 0;
    uint32_t Q = guards, plo = 0, phi = 0;
    int base[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      base[i] = c[i] == 0 ? 0 : (c[i] - 1) * T + 1;
      q[i] = v[i] - base[i];
      d += q[i] * C::dstride(i);
      Q |= (uint32_t)q[i] << (QW * i);
      if (i < K - 1) (i < 2 ? plo : phi) |= (uint32_t)v[i] << (16 * (i & 1));
    }
    uint64_t seen[kTrFam<K>];  // (main: the watched records here)
    if constexpr (main) {
#pragma unroll
      for (int f = 0; f < kTrFam<K>; ++f)
        seen[f] = rc.pos[(f0 + min(f, max(nf - 1, 0))) * rc.n + h];
    }
    // prefetch the face neighbours' blocks (an absent neighbour: this tile's)
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const int64_t tn = c[s] > 0 ? t - jd.tstride[s] : t;
      const u32x4 *src = reinterpret_cast<const u32x4 *>(jd.dir + tn * C::DBS);
#pragma unroll
      for (int x = 0; x < CPL; ++x) {
        const int idx = lane + x * 64;
        pf[s][x] = src[idx < NQ ? idx : NQ - 1];
      }
    }
    // Each lane reads one candidate next byte, so that a step's byte is a
    // register read of what was loaded a step earlier.  (The end of the walk,
    // a cell with v_i = 0, lies in a tile of its own: no test here.)
    int cand = dirb[max(d - loff, 0)];
    int byte = __builtin_amdgcn_readlane(cand, 0);
    if constexpr (main) {
      const uint64_t cell = ((uint64_t)phi << 32) | plo;
      int mf = -1;
#pragma unroll
      for (int f = kTrFam<K> - 1; f >= 0; --f)
        mf = __builtin_amdgcn_ballot_w64(f < nf && seen[f] == cell) ? f : mf;
      if (mf >= 0) {
        met = f0 + mf;
        return kTrMerged;
      }
    }
    int how = -1;
    for (;;) {
      if constexpr (!main) {
        if (h <= h_own) {
          if (h <= h_stop) {
            how = kTrOpen;
            break;
          }
          if (w0 - h >= kTrWin) {
            w0 = h;
            win = rc.pos[f0 * rc.n + max(h - lane, 0)];
          }
          if (__ballot(lane == w0 - h && (uint32_t)win == plo && (uint32_t)(win >> 32) == phi)) {
            met = f0;
            how = kTrMerged;
            break;
          }
        }
      }
      int b;
      if constexpr (coopt) {  // the lowest mask of the tie set
        const int ties = byte & ((1 << M) - 1);
        b = ties ? __builtin_ctz(ties) + 1 : 0;
      } else {
        b = M - (byte & M);
      }
      if (b == 0) {  // a cell without a move: corrupt decision data
        how = kTrBad;
        break;
      }
      byte = __builtin_amdgcn_readlane(cand, b);
      d -= __builtin_amdgcn_readlane(loff, b);
      cand = dirb[max(d - loff, 0)];
      // (every lane stores the same values)
      if constexpr (main) {
        to[h] = (uint8_t)b;
      } else {
        if (h > h_own) rc.pos[fam * rc.n + h] = ((uint64_t)phi << 32) | plo;
        (h > h_own ? own : to)[h] = (uint8_t)b;
        plo -= __builtin_amdgcn_readlane(llo, b);
        if constexpr (K > 3) phi -= __builtin_amdgcn_readlane(lhi, b);
      }
      Q -= __builtin_amdgcn_readlane(lq, b);
      h -= __builtin_amdgcn_readlane(lh, b);
      if ((Q & guards) != guards) break;  // left the tile
    }
    bool allz = true, anyz = false, bad = false;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      v[i] = base[i] + (int)((Q >> (QW * i)) & ((1u << QW) - 1)) - (1 << (QW - 1));
      bad = bad || v[i] < 0;  // a step below v_i = 0: corrupt decision data
      allz = allz && v[i] == 0;
      anyz = anyz || v[i] == 0;
    }
    if (how >= 0) return how;
    if (bad) return kTrBad;
    if (egf ? anyz : allz) return kTrEnd;
    int S = 0;
    t = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const int ci = v[i] == 0 ? 0 : (v[i] - 1) / T + 1;
      if (ci != c[i]) S |= 1 << i;
      c[i] = ci;
      t += (int64_t)ci * jd.tstride[i];
    }
    bool hit = false;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      if (S == 1 << s) {
#pragma unroll
        for (int x = 0; x < CPL; ++x) {
          const int idx = lane + x * 64;
          if (idx < NQ) lds4[idx] = pf[s][x];
        }
        hit = true;
      }
    }
    if (!hit) {
      const u32x4 *src = reinterpret_cast<const u32x4 *>(jd.dir + t * C::DBS);
      for (int idx = lane; idx < NQ; idx += 64) lds4[idx] = src[idx];
    }
  }
}

// Guess g of G (0: the origin, G: the end cell) of family f.
template <int K>
__device__ __forceinline__ int tr_guess(const int (&end)[K], int most, int f, int g, int G,
                                        int (&v)[K]) {
  int h = 0;
  const int up = (int)((int64_t)most * g / G), down = (int)((int64_t)most * (G - g) / G);
#pragma unroll
  for (int i = 0; i < K; ++i) {
    v[i] = f == 0 ? (int)((int64_t)end[i] * g / G) : f == 1 ? min(end[i], up) : max(0, end[i] - down);
    h += v[i];
  }
  return h;
}

// Families of guesses for an end cell with coordinate sum H: one where the
// lengths are within a sixteenth of the longest, or where three families'
// records do not fit.  (Traceback with one family and with three: 512^3 38 and
// 50 us, 300 x 257 x 281 51 and 42, 401 x 365 x 512 114 and 85, 157 x 93 x 201 63
// and 39.)
template <int K>
__device__ __forceinline__ int tr_families(const int (&end)[K], int &H) {
  int most = 0, least = INT32_MAX;
  H = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    most = max(most, end[i]);
    least = min(least, end[i]);
    H += end[i];
  }
  return 16 * (most - least) <= most || most < 24 || tr_rec_bytes(kTrFam<K>, H) > kTrRec
             ? 1
             : kTrFam<K>;
}

// The walk from cell end[] by all waves of the workgroup: sm.status, sm.vend
// and sm.hend (its last cell) and rc.path[h], the mask of its cell with sum
// h (0: none), for every sum above hend.
template <int K, bool egf, bool coopt>
__device__ __forceinline__ void tr_walk_all(const JobDev &jd, TrSmem<K> &sm, const int (&end)[K], const TrRec &rc,
                            int F, int wave) {
  const int lane = tr_lane();
  const int tid = wave * 64 + lane;
  const int H = rc.n - 1;
  int most = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) most = max(most, end[i]);
  // G guesses a family, the last of them the end cell: strictly ascending sums
  // (the longest dimension rises at each), and at least 4 cells apart
  const int G = max(1, min(1 + (kTrWalkers - 1) / F, most / 4));
  for (int x = tid; x < F * rc.n; x += kTrThreads) {
    rc.pos[x] = ~0ull;
    rc.own[x] = 0;
    rc.ov[x] = 0;
  }
  for (int x = tid; x < rc.n; x += kTrThreads) rc.path[x] = 0;
  if (tid < kTrWalkers) sm.state[tid] = -1;
  if (tid == 0) sm.done = sm.never = sm.ns = 0;
  __syncthreads();
  int v[K], h = 0, met = 0;
  // (the sums of all guesses are known to wave 0 before it looks)
  if (wave > 0 && wave <= F * (G - 1))
    sm.hstart[wave] =
        tr_guess<K>(end, most, (wave - 1) / (G - 1), (wave - 1) % (G - 1) + 1, G, v);
  __syncthreads();
  if (wave > 0 && wave <= F * (G - 1)) {
    const int f = (wave - 1) / (G - 1), g = (wave - 1) % (G - 1) + 1;
    const int hp = g > 1 ? sm.hstart[wave - 1] : -1, hpp = g > 2 ? sm.hstart[wave - 2] : -1;
    h = tr_guess<K>(end, most, f, g, G, v);
    const int how = tr_walk<K, egf, coopt, false>(
        jd, rc, sm.dirb[wave], v, h, __builtin_amdgcn_readfirstlane(hp),
        __builtin_amdgcn_readfirstlane(hpp), f, f, 1, rc.ov + f * rc.n, met, sm.done);
    sm.hstop[wave] = h;
#pragma unroll
    for (int i = 0; i < K; ++i) sm.vstop[wave][i] = v[i];
    __hip_atomic_store(&sm.state[wave], how, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  } else if (wave == 0) {
    __builtin_amdgcn_s_setprio(3);  // the others' work may be of no use, this wave's always is
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] = end[i];
    h = H;
    int how = tr_walk<K, egf, coopt, true>(jd, rc, sm.dirb[0], v, h, H, -1, 0, 0, G > 1 ? F : 0, rc.path,
                                     met, sm.never);
    // From a meeting the path goes down the family's walkers, each up to its own
    // meeting with the next, to the first that met nobody: as soon as those
    // walkers are done, the stretch is known.
    int ns = 0;
    while (how == kTrMerged) {
      const int first = met * (G - 1) + 1;  // the family's lowest walker
      const int st = lane < kTrWalkers ? sm.hstart[lane] : 0;
      // the owner of sum h: the lowest walker of the family that starts at h or above
      const uint64_t from =
          __ballot(lane >= first && lane < first + G - 1 && lane < kTrWalkers && st >= h);
      const int o = (int)__builtin_ctzll(from);
      uint64_t stay;  // of the walkers from the lowest to o: those that met nobody
      for (;;) {
        const int x = lane >= first && lane <= o
                          ? __hip_atomic_load(&sm.state[lane], __ATOMIC_ACQUIRE,
                                              __HIP_MEMORY_SCOPE_WORKGROUP)
                          : kTrMerged;
        stay = __ballot(x != kTrMerged);
        if (__ballot(x < 0) == 0) break;
        __builtin_amdgcn_s_sleep(1);
      }
      const int low = 63 - __builtin_clzll(stay);  // (the lowest never meets anybody)
      how = __builtin_amdgcn_readfirstlane(sm.state[low]);
      sm.seg[ns][0] = low;
      sm.seg[ns][1] = o;
      sm.seg[ns][2] = h;
      ++ns;
      h = __builtin_amdgcn_readfirstlane(sm.hstop[low]);
#pragma unroll
      for (int i = 0; i < K; ++i) v[i] = __builtin_amdgcn_readfirstlane(sm.vstop[low][i]);
      if (how == kTrOpen)  // go on alone until the walk meets someone
        how = tr_walk<K, egf, coopt, true>(jd, rc, sm.dirb[0], v, h, H, -1, 0, 0, F, rc.path, met,
                                     sm.never);
    }
    sm.ns = ns;
    __hip_atomic_store(&sm.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    sm.status = how == kTrEnd ? ST_OK : ST_EDEVICE;
    sm.hend = h;
#pragma unroll
    for (int i = 0; i < K; ++i) sm.vend[i] = v[i];
  }
  __syncthreads();
  // every walker of a stretch copies its part: its own sums from the meeting
  // above it, and the ones below down to its meeting
  for (int x = 0; x < sm.ns; ++x) {
    const int low = sm.seg[x][0], top = sm.seg[x][1];
    if (wave < low || wave > top) continue;
    const int f = (wave - 1) / (G - 1), g = (wave - 1) % (G - 1) + 1;
    const int hx = wave == top ? sm.seg[x][2] : sm.hstop[wave + 1];
    const int hp = g > 1 ? sm.hstart[wave - 1] : 0, hpp = g > 2 ? sm.hstart[wave - 2] : 0;
    const int h1 = max(sm.hstop[wave], hpp);
    for (int y = max(h1, hp) + 1 + lane; y <= hx; y += 64) rc.path[y] = rc.own[f * rc.n + y];
    for (int y = h1 + 1 + lane; y <= min(hp, hx); y += 64) rc.path[y] = rc.ov[f * rc.n + y];
  }
  __syncthreads();
}

// Rows of the alignment: unaligned prefixes (end gaps free; sequence 0 first),
// the path's columns in ascending order of h, unaligned suffixes.
template <int K>
__device__ __forceinline__ void tr_rows(const JobDev &jd, TrSmem<K> &sm, const int (&end)[K],
                                        const TrRec &rc, int wave) {
  const int lane = tr_lane();
  const int tid = wave * 64 + lane;
  int H = 0, pre = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    H += end[i];
    pre += sm.vend[i];
  }
  const int hend = sm.hend;
  // wave w takes the sums (w, w + 1] * per
  const int per = (H + kTrThreads - 1) / kTrThreads * 64;
  const int first = wave * per + 1, last = min(H, (wave + 1) * per);
  int cnt[K + 1];  // columns, and columns with a residue of sequence i
#pragma unroll
  for (int i = 0; i <= K; ++i) cnt[i] = 0;
  for (int h0 = first; h0 <= last; h0 += 64) {
    const int m = h0 + lane <= last && h0 + lane > hend ? rc.path[h0 + lane] : 0;
    cnt[K] += __builtin_popcountll(__ballot(m != 0));
#pragma unroll
    for (int i = 0; i < K; ++i) cnt[i] += __builtin_popcountll(__ballot((m >> i) & 1));
  }
#pragma unroll
  for (int i = 0; i <= K; ++i) sm.cnt[wave][i] = cnt[i];
  __syncthreads();
  int at[K + 1], total = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) at[i] = sm.vend[i];
  at[K] = pre;
  for (int w = 0; w < kTrWalkers; ++w) {
#pragma unroll
    for (int i = 0; i <= K; ++i) at[i] += w < wave ? sm.cnt[w][i] : 0;
    total += sm.cnt[w][K];
  }
  const uint64_t below = (1ull << lane) - 1;
  for (int h0 = first; h0 <= last; h0 += 64) {
    const int m = h0 + lane <= last && h0 + lane > hend ? rc.path[h0 + lane] : 0;
    const uint64_t cols = __ballot(m != 0);
    const int64_t col = at[K] + __builtin_popcountll(cols & below);
    at[K] += __builtin_popcountll(cols);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const uint64_t bits = __ballot((m >> i) & 1);
      const int pos = at[i] + __builtin_popcountll(bits & below);
      at[i] += __builtin_popcountll(bits);
      if (m != 0)
        jd.aln_out[(int64_t)i * jd.aln_cap + col] =
            (m >> i) & 1 ? jd.seqs[jd.seq_off[i] + pos] : (uint8_t)0xFF;
    }
  }
  // one-residue columns of the unaligned prefixes and suffixes
  int64_t c0 = 0, c1 = pre + total;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    for (int x = tid; x < sm.vend[s]; x += kTrThreads)
#pragma unroll
      for (int i = 0; i < K; ++i)
        jd.aln_out[(int64_t)i * jd.aln_cap + c0 + x] =
            i == s ? jd.seqs[jd.seq_off[s] + x] : (uint8_t)0xFF;
    c0 += sm.vend[s];
    for (int x = tid; x < jd.n[s] - end[s]; x += kTrThreads)
#pragma unroll
      for (int i = 0; i < K; ++i)
        jd.aln_out[(int64_t)i * jd.aln_cap + c1 + x] =
            i == s ? jd.seqs[jd.seq_off[s] + end[s] + x] : (uint8_t)0xFF;
    c1 += jd.n[s] - end[s];
  }
  if (tid == 0) *jd.aln_len_out = c1;
}

template <int K, bool egf, bool coopt>
__device__ __forceinline__ void tr_job(const JobDev &jd, TrSmem<K> &sm, int status, int64_t best,
                                       int wave) {
  int end[K];
  if constexpr (egf) {  // the end cell from its row-major index
    int64_t lin = (int64_t)(uint32_t)best;
#pragma unroll
    for (int i = K - 1; i >= 0; --i) {
      end[i] = (int)(lin % ((int64_t)jd.n[i] + 1));
      lin /= (int64_t)jd.n[i] + 1;
    }
  } else {
#pragma unroll
    for (int i = 0; i < K; ++i) end[i] = jd.n[i];
  }
  if (status == ST_OK) {
    int H = 0;
    const int F = tr_families<K>(end, H);
    const TrRec rc(sm, F, H);
    tr_walk_all<K, egf, coopt>(jd, sm, end, rc, F, wave);
    status = sm.status;
    if (status == ST_OK) tr_rows<K>(jd, sm, end, rc, wave);
  }
  if (wave * 64 + tr_lane() == 0) {
    *jd.status_out = status;
    if (status != ST_OK) {
      *jd.aln_len_out = 0;
      *jd.score_out = 0;
    } else if (egf) {
      *jd.score_out = best >> 32;
    }
  }
}

}  // namespace

template <int K>
__global__ __launch_bounds__(kTrThreads) void trace_kernel(JobDev jd, Ctrl *ctrl) {
  __shared__ TrSmem<K> sm;
  const int wave = tr_wave();
  const int mode = __builtin_amdgcn_readfirstlane(ctrl->flags);
  const int st = __builtin_amdgcn_readfirstlane(
      __hip_atomic_load(&ctrl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  if (mode & kEndGapsFree) {
    tr_job<K, true, false>(
        jd, sm, st, __hip_atomic_load(&ctrl->best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
        wave);
  } else if (mode & kCoOptimal) {
    if constexpr (K <= kCoMaxK) tr_job<K, false, true>(jd, sm, st, 0, wave);
  } else {
    tr_job<K, false, false>(jd, sm, st, 0, wave);
  }
  __syncthreads();
  if (threadIdx.x == 0) finish_launch(ctrl);
}

__device__ __forceinline__ int64_t tr_uni(int64_t x) {
  return (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)x) |
         (int64_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32;
}
template <class T>
__device__ __forceinline__ T *tr_uni(T *p) {
  return as_global(reinterpret_cast<T *>(tr_uni(reinterpret_cast<int64_t>(p))));
}

// What the walk reads of a job's descriptor, in scalar registers.
__device__ __forceinline__ JobDev tr_desc(const JobDev &jd) {
  JobDev r;
#pragma unroll
  for (int i = 0; i < kTrMaxK; ++i) {
    r.n[i] = __builtin_amdgcn_readfirstlane(jd.n[i]);
    r.tstride[i] = __builtin_amdgcn_readfirstlane(jd.tstride[i]);
    r.seq_off[i] = __builtin_amdgcn_readfirstlane(jd.seq_off[i]);
  }
  r.dir = tr_uni(jd.dir);
  r.seqs = tr_uni(jd.seqs);
  r.aln_out = tr_uni(jd.aln_out);
  r.aln_cap = tr_uni(jd.aln_cap);
  r.aln_len_out = tr_uni(jd.aln_len_out);
  r.status_out = tr_uni(jd.status_out);
  r.score_out = tr_uni(jd.score_out);
  return r;
}

// A batched launch's jobs, one workgroup each at a time; the others are left to
// the single walk's kernel.
template <int KLO, int KHI>
__global__ __launch_bounds__(kTrThreads) void batch_trace_kernel(const BatchArgs *__restrict__ a,
                                                                 const JobDev *__restrict__ jobs,
                                                                 Ctrl *ctrl) {
  constexpr size_t kBytes =
      sizeof(TrSmem<KHI>) > sizeof(TrSmem<KLO>) ? sizeof(TrSmem<KHI>) : sizeof(TrSmem<KLO>);
  __shared__ alignas(16) char mem[kBytes];
  const int wave = tr_wave();
  const int njobs = __builtin_amdgcn_readfirstlane(a->njobs);
  const int gst = __builtin_amdgcn_readfirstlane(
      __hip_atomic_load(&ctrl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  for (int j = blockIdx.x; j < njobs; j += gridDim.x) {
    if (!__builtin_amdgcn_readfirstlane(jobs[j].walkers)) continue;
    const JobDev jd = tr_desc(jobs[j]);
    const int jst = __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(jobs[j].jstatus, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const int st = gst != ST_OK ? gst : jst;
    __syncthreads();  // the last job's records are read no more
    switch (__builtin_amdgcn_readfirstlane(jobs[j].k)) {
      case 2:
        if constexpr (KLO <= 2 && 2 <= KHI)
          tr_job<2, false, false>(jd, *reinterpret_cast<TrSmem<2> *>(mem), st, 0, wave);
        break;
      case 3:
        if constexpr (KLO <= 3 && 3 <= KHI)
          tr_job<3, false, false>(jd, *reinterpret_cast<TrSmem<3> *>(mem), st, 0, wave);
        break;
      case 4:
        if constexpr (KLO <= 4 && 4 <= KHI)
          tr_job<4, false, false>(jd, *reinterpret_cast<TrSmem<4> *>(mem), st, 0, wave);
        break;
      case 5:
        if constexpr (KLO <= 5 && 5 <= KHI)
          tr_job<5, false, false>(jd, *reinterpret_cast<TrSmem<5> *>(mem), st, 0, wave);
        break;
      default: break;
    }
  }
}

// One workgroup per compute unit holds the walkers' LDS.
void launch_batch_trace(int kclass, const BatchArgs *d_args, const JobDev *d_jobs, Ctrl *ctrl,
                        hipStream_t s) {
  const dim3 grid((unsigned)device_cu_count()), block(kTrThreads);
  if (kclass == 0)
    hipLaunchKernelGGL((batch_trace_kernel<2, 4>), grid, block, 0, s, d_args, d_jobs, ctrl);
  else if (kclass == 1)
    hipLaunchKernelGGL((batch_trace_kernel<5, 5>), grid, block, 0, s, d_args, d_jobs, ctrl);
}

// ---------------------------------------------------------------------------
// Co-optimal alignments.
// ---------------------------------------------------------------------------
constexpr int kMoreTies = 0x80;  // stack entry flag: the cell has tied masks above the one taken

// Records over the first alignment's walk, in the memory of its walkers' cells.
struct CoRec {
  uint32_t *cell;   // [h]: the first alignment's cell (v_0, v_1), ~0: none
  uint16_t *level;  // [h]: its column, counted from the last one
  uint8_t *first;   // [level]: its stack (mask and kMoreTies)
  uint8_t *stack;   // [level]: the current alignment's
  uint8_t *seq;     // the sequences
  __device__ __forceinline__ explicit CoRec(const TrRec &rc)
      : cell(reinterpret_cast<uint32_t *>(rc.pos)),
        level(reinterpret_cast<uint16_t *>(cell + rc.n)),
        first(reinterpret_cast<uint8_t *>(level + rc.n)),
        stack(first + rc.n),
        seq(rc.own) {}
};

// The tie set of cell v, from its tile's block in `blk` (tile cur).
template <int K>
__device__ __forceinline__ int co_ties(const JobDev &jd, uint8_t *blk, int &cur,
                                       const int (&v)[K]) {
  using C = TrCfg<K>;
  constexpr int T = C::T;
  const int lane = threadIdx.x & 63;
  int t = 0, dl = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const int ci = v[i] == 0 ? 0 : (v[i] - 1) / T + 1;
    t += ci * jd.tstride[i];
    dl += (v[i] - (ci == 0 ? 0 : (ci - 1) * T + 1)) * C::dstride(i);
  }
  if (t != cur) {
    const u32x4 *src = reinterpret_cast<const u32x4 *>(jd.dir + (int64_t)t * C::DBS);
    u32x4 *dst = reinterpret_cast<u32x4 *>(blk);
#pragma unroll
    for (int x = 0; x < (C::DBS / 16 + 63) / 64; ++x) {
      const int idx = lane + x * 64;
      if (idx < C::DBS / 16) dst[idx] = src[idx];
    }
    cur = t;
  }
  return __builtin_amdgcn_readfirstlane(blk[dl]) & ((1 << C::M) - 1);
}

// Alignment p goes to aln_out + p * k * aln_cap.  Wave 0 enumerates and leaves
// each alignment's masks in its first row; all waves expand them afterwards.
template <int K>
__global__ __launch_bounds__(kTrThreads) void coopt_trace_kernel(JobDev jd, Ctrl *ctrl,
                                                                 int32_t max_paths,
                                                                 uint8_t *aln_out,
                                                                 int64_t *len_out,
                                                                 int32_t *npaths_out) {
  using C = TrCfg<K>;
  __shared__ TrSmem<K> sm;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
  int status = __builtin_amdgcn_readfirstlane(
      __hip_atomic_load(&ctrl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  // the blocks hold tie sets only when the workspace was set up for them
  if (status == ST_OK && !(ctrl->flags & kCoOptimal)) status = ST_EINVAL;
  int end[K];
#pragma unroll
  for (int i = 0; i < K; ++i) end[i] = jd.n[i];
  int H = 0;
  const int F = tr_families<K>(end, H);
  const TrRec rc(sm, F, H);
  if (status == ST_OK) {
    tr_walk_all<K, false, true>(jd, sm, end, rc, F, wave);
    status = sm.status;
  }
  int np = 0;
  if (status == ST_OK) {
    // ---- the first alignment's columns: wave w takes the sums w * per + 1 .. ----
    const CoRec co(rc);
    const int per = (H + kTrThreads - 1) / kTrThreads * 64;
    const int lo = wave * per + 1, hi = min(H, (wave + 1) * per);
    int cnt[K + 1];
#pragma unroll
    for (int i = 0; i <= K; ++i) cnt[i] = 0;
    for (int h0 = lo; h0 <= hi; h0 += 64) {
      const int m = h0 + lane <= hi ? rc.path[h0 + lane] : 0;
      cnt[K] += __builtin_popcountll(__ballot(m != 0));
#pragma unroll
      for (int i = 0; i < K; ++i) cnt[i] += __builtin_popcountll(__ballot((m >> i) & 1));
    }
#pragma unroll
    for (int i = 0; i <= K; ++i) sm.cnt[wave][i] = cnt[i];
    for (int x = tid; x <= H; x += kTrThreads) co.cell[x] = ~0u;
    for (int x = tid; x < H; x += kTrThreads) co.seq[x] = jd.seqs[x];
    __syncthreads();
    int at[K + 1], N = 0;
#pragma unroll
    for (int i = 0; i <= K; ++i) at[i] = 0;
    for (int w = 0; w < kTrWalkers; ++w) {
#pragma unroll
      for (int i = 0; i <= K; ++i) at[i] += w < wave ? sm.cnt[w][i] : 0;
      N += sm.cnt[w][K];
    }
    const uint64_t upto = lane == 63 ? ~0ull : (2ull << lane) - 1;
    for (int h0 = lo; h0 <= hi; h0 += 64) {
      const int h = h0 + lane;
      const int m = h <= hi ? rc.path[h] : 0;
      const uint64_t cols = __ballot(m != 0);
      const int lv = N - (at[K] + __builtin_popcountll(cols & upto));  // from the last column
      at[K] += __builtin_popcountll(cols);
      int64_t t = 0;
      int dl = 0, vv[K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const uint64_t bits = __ballot((m >> i) & 1);
        vv[i] = at[i] + __builtin_popcountll(bits & upto);
        at[i] += __builtin_popcountll(bits);
        const int ci = vv[i] == 0 ? 0 : (vv[i] - 1) / C::T + 1;
        t += (int64_t)ci * jd.tstride[i];
        dl += (vv[i] - (ci == 0 ? 0 : (ci - 1) * C::T + 1)) * C::dstride(i);
      }
      if (m != 0) {
        const int ties = jd.dir[t * C::DBS + dl] & ((1 << C::M) - 1);
        const bool more = (ties & ~((1 << m) - 1)) != 0;  // tied masks above m
        co.cell[h] = (uint32_t)vv[0] | (uint32_t)vv[1] << 16;
        co.level[h] = (uint16_t)lv;
        co.first[lv] = (uint8_t)(m | (more ? kMoreTies : 0));
      }
    }
    __syncthreads();
    // ---- the enumeration (wave 0) ----
    if (wave == 0) {
      for (int x = lane; x < N; x += 64) co.stack[x] = co.first[x];
      int d = N, cur = -1;
      int v[K];
#pragma unroll
      for (int i = 0; i < K; ++i) v[i] = 0;  // the cell after the stack's last column
      for (;;) {
        // v is the origin: stack[0 .. d) is an alignment (stack[d - 1] its first column)
        uint8_t *row = aln_out + (int64_t)np * K * jd.aln_cap;
        for (int x = lane; x < d; x += 64) row[x] = co.stack[d - 1 - x] & C::M;
        if (lane == 0) len_out[np] = d;
        ++np;
        if (np == max_paths || d == 0) break;
        // back up to the deepest column whose cell has tied masks left (lane x
        // reads level e - x), adding the masks of the columns popped to v
        int e = d - 1, found = -1;
        while (e >= 0) {
          const int lvl = e - lane;
          const int ent = lvl >= 0 ? co.stack[lvl] : 0;
          const uint64_t flagged = __ballot((ent & kMoreTies) != 0);
          const int last = flagged ? __builtin_ctzll(flagged) : 63;
          const bool popped = lane <= last && lvl >= 0;
#pragma unroll
          for (int i = 0; i < K; ++i)
            v[i] += __builtin_popcountll(__ballot(popped && ((ent >> i) & 1)));
          if (flagged) {
            found = e - last;
            break;
          }
          e -= 64;
        }
        if (found < 0) break;  // every alignment has been produced
        d = found;
        int tried = co.stack[d] & C::M;
        int h = 0;
#pragma unroll
        for (int i = 0; i < K; ++i) h += v[i];
        // down along the lowest tied masks (the first step: above `tried`) to a
        // cell of the first alignment, whose columns below are this one's too
        bool bad = false;
        for (;;) {
          if (tried == 0 && h > 0) {
            const uint32_t p = (uint32_t)v[0] | (uint32_t)v[1] << 16;
            if ((uint32_t)__builtin_amdgcn_readfirstlane(co.cell[h]) == p) {
              const int lv = __builtin_amdgcn_readfirstlane((int)co.level[h]);
              for (int x = lane; x < N - lv; x += 64) co.stack[d + x] = co.first[lv + x];
              d += N - lv;
              break;
            }
          }
          if (h == 0) break;  // (one-column alignments meet the first one nowhere)
          const int ties = co_ties<K>(jd, sm.dirb[0], cur, v);
          const int rest = ties & ~((1 << tried) - 1);
          if (rest == 0) {  // a flagged column without a tie left, or a cell without one
            bad = true;
            break;
          }
          const int b = __builtin_ctz(rest) + 1;
#pragma unroll
          for (int i = 0; i < K; ++i) {
            bad = bad || (((b >> i) & 1) && v[i] == 0);
            v[i] -= (b >> i) & 1;
          }
          if (bad || d >= H) {
            bad = true;
            break;
          }
          co.stack[d] = (uint8_t)(b | ((rest & ~((1 << b) - 1)) != 0 ? kMoreTies : 0));
          h -= __builtin_popcount(b);
          ++d;
          tried = 0;
        }
        if (bad) {
          status = ST_EDEVICE;
          break;
        }
#pragma unroll
        for (int i = 0; i < K; ++i) v[i] = 0;
      }
      sm.status = status;
      sm.hend = np;
    }
    __threadfence_block();
    __syncthreads();
    status = sm.status;
    np = sm.hend;
    // ---- rows: a wave per alignment; a chunk's masks are read before its
    // columns of the first row are written ----
    if (status == ST_OK) {
      const uint64_t below = (1ull << lane) - 1;
      for (int p = wave; p < np; p += kTrWalkers) {
        uint8_t *blk = aln_out + (int64_t)p * K * jd.aln_cap;
        const int d = (int)len_out[p];
        int pos[K];
#pragma unroll
        for (int i = 0; i < K; ++i) pos[i] = jd.seq_off[i];
        for (int c0 = 0; c0 < d; c0 += 64) {
          const int m = c0 + lane < d ? blk[c0 + lane] : 0;
#pragma unroll
          for (int i = 0; i < K; ++i) {
            const uint64_t bits = __ballot((m >> i) & 1);
            const int x = pos[i] + __builtin_popcountll(bits & below);
            pos[i] += __builtin_popcountll(bits);
            if (m != 0)
              blk[(int64_t)i * jd.aln_cap + c0 + lane] =
                  (m >> i) & 1 ? co.seq[x] : (uint8_t)0xFF;
          }
        }
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    *npaths_out = status == ST_OK ? np : 0;
    *jd.status_out = status;
    if (status != ST_OK) *jd.score_out = 0;
    finish_launch(ctrl);
  }
}

int launch_coopt_trace(const JobDev &jd, Ctrl *ctrl, int32_t max_paths, uint8_t *aln_out,
                       int64_t *len_out, int32_t *npaths_out, hipStream_t s) {
  launch_begin();
  if (jd.k == 2)
    hipLaunchKernelGGL((coopt_trace_kernel<2>), dim3(1), dim3(kTrThreads), 0, s, jd, ctrl,
                       max_paths, aln_out, len_out, npaths_out);
  else
    hipLaunchKernelGGL((coopt_trace_kernel<3>), dim3(1), dim3(kTrThreads), 0, s, jd, ctrl,
                       max_paths, aln_out, len_out, npaths_out);
  return launch_end();
}

// ---------------------------------------------------------------------------
// Near-optimal alignments (near-optimal mode, k <= 6): every global alignment
// whose score is at least opt - delta (Section 6: alignments within a
// threshold of the optimum set by the user).  The fill has also stored every
// cell's score xi, laid out as the direction blocks.  Wave 0 walks depth
// first from the far corner.  At cell v, with s the score of the columns
// taken so far, lane b - 1 tests mask b: v - b lies in the tensor and
// xi(v - b) + SP(col(v, b)) + s >= opt - delta.  xi(v - b) is the score of
// some path from the origin, so every step passing the test leads to at least
// one alignment at or above the threshold (the walk has no dead end), and
// every such alignment is walked.  The masks of a cell are taken in
// ascending order, so the list is sorted by the column masks read from the
// last column to the first, and delta = 0 gives the co-optimal list.  Per
// column the LDS stack keeps the mask taken, the set of masks that passed
// and the score so far (sum n_i <= kNoMaxTotal); after an alignment the walk
// jumps back to the deepest column with a passing mask left, found with one
// wave-wide scan of the stack.  Alignment p goes to aln_out + p * k *
// aln_cap, its score to scores_out[p]; its masks wait in its first row until
// all waves expand the list.
//
// What bounds it: the chain of a step (scores and pair scores of the cell, the
// test, the choice).  A box of the scores at and below the walk's cell and the
// pair scores of its residues sit in LDS, loaded by all waves at once when the
// walk leaves the box.  The list below a cell depends on the cell and on the
// score so far alone, and its first entry is what a walk that comes to both
// again goes on with; so new cells are recorded with that score (k <= 5), and
// a walk that meets such a record copies the columns below it.  A record is found
// by a hash of cell and score.  16 alignments
// of 300 x 257 x 281: 1.54 ms with global loads for everything at every step,
// 1.38 with the box alone, 0.29 now.
// ---------------------------------------------------------------------------
constexpr int kNoThreads = 1024;
constexpr int kNoPool = 3072;    // recorded cells
constexpr int kNoWalks = 512;    // recorded walks
constexpr int kNoHash = 4096;    // chains of records

// Chain of a cell (its packed coordinates) and a score so far: multiplicative
// hashing (Knuth, The Art of Computer Programming, vol. 3, section 6.4) with
// odd multipliers near 2^32 divided by the golden ratio, top 12 bits.
__device__ __forceinline__ int no_hash(uint64_t cell, int32_t score) {
  const uint32_t x = (uint32_t)cell * 0x9E3779B1u + (uint32_t)(cell >> 32) * 0x9E377955u +
                     (uint32_t)score;
  return (int)((x * 0x9E3779B1u) >> 20);
}

template <int K>
struct NoSmem {
  static constexpr int E = K == 2 ? 32 : K == 3 ? 16 : K == 4 ? 8 : K == 5 ? 5 : 4;  // box edge
  static constexpr int N = ipow(E, K);
  static constexpr int NP = K * (K - 1) / 2;
  static constexpr bool Memo = K <= 5;  // a cell fits the record (13 bits a coordinate)
  static constexpr int Pool = Memo ? kNoPool : 1;
  uint64_t cell[Pool];             // recorded cell (v_0 .. v_{k-2} and the sum), by record
  uint64_t pass[kNoMaxTotal + 1];  // masks that passed at a column's cell
  int32_t sofar[kNoMaxTotal + 1];  // score of the columns above it
  int32_t box[N];                  // xi(top - x) at sum x_i * E^(K-1-i)
  // offsets of the box's scores in memory: the parts of dimensions 0 .. H - 1 by
  // x / NL, those of the others by x % NL (negative: below 0 in some dimension)
  static constexpr int H = (K + 1) / 2, NH = ipow(E, H), NL = ipow(E, K - H);
  int64_t part[NH + NL];
  int32_t pair[NP][E * E];         // pair scores of the box's residues, by x_i * E + x_j
  int32_t score[Pool];             // a record's score so far,
  uint32_t set[Pool];              // its cell's passing masks
  uint8_t mask[Pool];              // and the one taken (the lowest)
  uint16_t walk[Pool];             // its walk
  uint16_t link[Pool];             // another record of the same hash
  uint16_t head[Memo ? kNoHash : 1];  // by hash of cell and score (0xFFFF: none)
  uint16_t wend[kNoWalks];         // a walk's records end before this one
  int16_t wnext[kNoWalks];         // and go on with this one (-1: the origin,
  int32_t wlast[kNoWalks];         // with this score)
  uint8_t path[kNoMaxTotal + 1];
  uint8_t seq[kNoMaxTotal + 1];
  int32_t top[K];                  // the box's upper corner
  int32_t more, status, np;
};

template <int K>
__global__ __launch_bounds__(kNoThreads) void nearopt_kernel(JobDev jd, Ctrl *ctrl, int64_t delta,
                                                             int32_t max_paths,
                                                             int64_t *scores_out,
                                                             uint8_t *aln_out, int64_t *len_out,
                                                             int32_t *npaths_out) {
  using C = TrCfg<K>;
  using Sm = NoSmem<K>;
  constexpr int T = C::T;
  constexpr int M = C::M;  // masks 1..M; lane b - 1 tests mask b
  constexpr int E = Sm::E;
  static_assert(M <= 64, "one lane per mask");
  __shared__ Sm sm;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
  int status = __builtin_amdgcn_readfirstlane(
      __hip_atomic_load(&ctrl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  // the cell scores exist only when the workspace was set up for them
  if (status == ST_OK && !(ctrl->flags & kNearOpt)) status = ST_EINVAL;
  const int alpha = ctrl->alpha;
  const int gap = ctrl->gap;
  const int64_t threshold = *jd.score_out - delta;
  const int total = (int)jd.total_len;
  for (int x = tid; x < total; x += kNoThreads) sm.seq[x] = jd.seqs[x];
  if constexpr (Sm::Memo)
    for (int x = tid; x < kNoHash; x += kNoThreads) sm.head[x] = 0xFFFF;
  if (tid == 0) {
    sm.sofar[0] = 0;
    sm.status = status;
    sm.np = 0;
  }
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (tid == i) sm.top[i] = jd.n[i];
  // wave 0's walk
  int v[K];
#pragma unroll
  for (int i = 0; i < K; ++i) v[i] = jd.n[i];
  const int bl = lane + 1;  // this lane's mask
  int lbox = 0;             // its offset in the box
#pragma unroll
  for (int i = 0; i < K; ++i) lbox += ((bl >> i) & 1) * ipow(E, K - 1 - i);
  int d = 0, np = 0;
  int tried = 0;      // masks up to this one were taken at depth d
  bool fresh = true;  // pass[d] not computed yet
  int32_t sf = 0;     // sofar[d]
  int h = total;      // coordinate sum of v
  int nrec = 0, nwalk = 0;  // records, and finished walks, so far
  bool rec = Sm::Memo && total <= kNoPool;  // this walk's cells are recorded
  int64_t steps = 0;
  const int64_t step_limit = (int64_t)max_paths * (2 * jd.total_len + 2) + 2;
  __syncthreads();
  while (status == ST_OK) {
    // ---- all waves: the box of scores below sm.top ----
    {
      // An offset is a sum over the dimensions, so it is put together from two
      // tables (all dimensions for every score: 12 x 4^4 x 12, k = 6, where a walk leaves
      // its box every other column, 1.51 ms against 1.23).
      if (tid < Sm::NH + Sm::NL) {
        const bool high = tid < Sm::NH;
        int rem = high ? tid : tid - Sm::NH;
        int64_t o = 0;
        bool ok = true;
#pragma unroll
        for (int i = K - 1; i >= 0; --i) {
          if (high != (i < Sm::H)) continue;
          const int u = sm.top[i] - rem % E;
          rem /= E;
          ok = ok && u >= 0;
          const int uu = u < 0 ? 0 : u;
          const int ci = uu == 0 ? 0 : (uu - 1) / T + 1;
          o += (int64_t)ci * jd.tstride[i] * C::DBS +
               (uu - (ci == 0 ? 0 : (ci - 1) * T + 1)) * C::dstride(i);
        }
        sm.part[tid] = ok ? o : INT64_MIN / 2;
      }
      __syncthreads();
      constexpr int PER = (Sm::N + kNoThreads - 1) / kNoThreads;
      int32_t got[PER];
#pragma unroll
      for (int y = 0; y < PER; ++y) {
        const int x = min(tid + y * kNoThreads, Sm::N - 1);
        const int64_t o = sm.part[x / Sm::NL] + sm.part[Sm::NH + x % Sm::NL];
        got[y] = jd.scores[o < 0 ? 0 : o];
      }
#pragma unroll
      for (int y = 0; y < PER; ++y)
        if (tid + y * kNoThreads < Sm::N) sm.box[tid + y * kNoThreads] = got[y];
      // and the pair scores of its residues (0 where a coordinate is 0 or below)
      for (int x = tid; x < Sm::NP * E * E; x += kNoThreads) {
        const int p = x / (E * E), r = x % (E * E);
        int i = 0, j = 0, oi = 0, oj = 0;
#pragma unroll
        for (int ii = 0; ii < K; ++ii)
#pragma unroll
          for (int jj = ii + 1; jj < K; ++jj)
            if (p == ii * (2 * K - ii - 1) / 2 + (jj - ii - 1)) {
              i = ii;
              j = jj;
              oi = jd.seq_off[ii];
              oj = jd.seq_off[jj];
            }
        const int a = sm.top[i] - r / E, b = sm.top[j] - r % E;
        (&sm.pair[0][0])[x] = a >= 1 && b >= 1
                                  ? (int32_t)jd.sub[sm.seq[oi + a - 1] * alpha + sm.seq[oj + b - 1]]
                                  : 0;
      }
    }
    __syncthreads();
    if (wave == 0) {
      int top[K];
#pragma unroll
      for (int i = 0; i < K; ++i) top[i] = __builtin_amdgcn_readfirstlane(sm.top[i]);
      int more = 0;  // the walk needs another box
      for (;;) {
        if (h == 0) {
          // path[0..d) (path[d-1] is the first column) is alignment np
          uint8_t *row = aln_out + (int64_t)np * K * jd.aln_cap;
          for (int x = lane; x < d; x += 64) row[x] = sm.path[d - 1 - x];
          if (lane == 0) {
            len_out[np] = d;
            scores_out[np] = sf;
          }
          ++np;
          if (np == max_paths || d == 0) break;
          if constexpr (Sm::Memo) {  // the walk's records end here
            if (rec) {
              sm.wend[nwalk] = (uint16_t)nrec;
              sm.wnext[nwalk] = -1;
              sm.wlast[nwalk] = sf;
              ++nwalk;
            }
          }
          // back up to the deepest column with a passing mask above the one
          // taken: scan the stack 64 entries at a time (lane x reads level
          // e - x), adding the masks of the levels popped to v
          int e = d - 1, found = -1;
          while (e >= 0) {
            const int lvl = e - lane;
            const int ent = lvl >= 0 ? sm.path[lvl] : 0;
            const bool left = lvl >= 0 && (sm.pass[lvl] >> ent) != 0;
            const uint64_t flagged = __ballot(left);
            const int upto = flagged ? __builtin_ctzll(flagged) : 63;
            const bool popped = lane <= upto && lvl >= 0;
#pragma unroll
            for (int i = 0; i < K; ++i)
              v[i] += __builtin_popcountll(__ballot(popped && ((ent >> i) & 1)));
            if (flagged) {
              found = e - upto;
              break;
            }
            e -= 64;
          }
          if (found < 0) break;  // every alignment has been produced
          d = found;
          tried = __builtin_amdgcn_readfirstlane((int)sm.path[d]);
          sf = __builtin_amdgcn_readfirstlane(sm.sofar[d]);
          h = 0;
#pragma unroll
          for (int i = 0; i < K; ++i) h += v[i];
          // (a walk is recorded whole or not at all)
          rec = Sm::Memo && nrec + h <= kNoPool && nwalk < kNoWalks;
          fresh = false;
          continue;
        }
        uint64_t cell = 0;
        if constexpr (Sm::Memo) {
#pragma unroll
          for (int i = 0; i < K - 1; ++i) cell |= (uint64_t)(uint32_t)v[i] << (13 * i);
          cell |= (uint64_t)(uint32_t)h << 52;  // (for the last coordinate; kNoMaxTotal itself, the
                                                // end cell's, is looked up by no walk)
          if (fresh && np > 0) {
            // met a record of this cell and score?  (one lookup per new cell)
            int x = __builtin_amdgcn_readfirstlane((int)sm.head[no_hash(cell, sf)]);
            while (x != 0xFFFF) {
              const bool same = sm.cell[x] == cell && sm.score[x] == sf;
              if (__builtin_amdgcn_readfirstlane((int)same)) break;
              x = __builtin_amdgcn_readfirstlane((int)sm.link[x]);
            }
            if (x != 0xFFFF) {
              if (rec) {  // this walk goes on with that record
                sm.wend[nwalk] = (uint16_t)nrec;
                sm.wnext[nwalk] = (int16_t)x;
                ++nwalk;
                rec = false;
              }
              while (x >= 0) {
                const int w = __builtin_amdgcn_readfirstlane((int)sm.walk[x]);
                const int n = __builtin_amdgcn_readfirstlane((int)sm.wend[w]) - x;
                for (int y = lane; y < n; y += 64) {
                  sm.path[d + y] = sm.mask[x + y];
                  sm.pass[d + y] = sm.set[x + y];
                  sm.sofar[d + y] = sm.score[x + y];
                }
                d += n;
                x = __builtin_amdgcn_readfirstlane((int)sm.wnext[w]);
                sf = __builtin_amdgcn_readfirstlane(sm.wlast[w]);
              }
#pragma unroll
              for (int i = 0; i < K; ++i) v[i] = 0;
              h = 0;  // the path is whole
              continue;
            }
          }
        }
        {  // v and its lower neighbours have to lie in the box
          bool in = true;
#pragma unroll
          for (int i = 0; i < K; ++i) in = in && (unsigned)(top[i] - v[i]) <= (unsigned)(E - 2);
          if (!in) {
            more = 1;
            break;
          }
        }
        if (++steps > step_limit) {  // inconsistent scores: never loop for ever
          status = ST_EDEVICE;
          break;
        }
        // SP(col(v, b)) of this lane's mask: residue pairs, residue-gap pairs
        int32_t sp = 0;
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
          for (int j = i + 1; j < K; ++j) {
            const int32_t ps =
                sm.pair[i * (2 * K - i - 1) / 2 + (j - i - 1)][(top[i] - v[i]) * E + top[j] - v[j]];
            const int bi = (bl >> i) & 1, bj = (bl >> j) & 1;
            sp += (bi && bj) ? ps : (bi ^ bj) ? gap : 0;
          }
        uint64_t set;
        if (fresh) {
          bool ok = lane < M;
          int x = 0;
#pragma unroll
          for (int i = 0; i < K; ++i) {
            ok = ok && v[i] - ((bl >> i) & 1) >= 0;
            x += (top[i] - v[i]) * ipow(E, K - 1 - i);
          }
          const int32_t xi = sm.box[ok ? x + lbox : 0];
          set = __ballot(ok && (int64_t)xi + sp + sf >= threshold);
          if (set == 0) {  // a cell off the origin from which no alignment reaches the threshold
            status = ST_EDEVICE;
            break;
          }
          sm.pass[d] = set;  // every lane stores the same value
        } else {
          const uint64_t p = sm.pass[d];
          set = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)p) |
                (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(p >> 32)) << 32;
        }
        // (masks up to `tried` were taken; a column on the stack keeps at least
        // one more whenever the walk comes back to it)
        const uint64_t rest = tried >= 64 ? 0 : set & ~((1ull << tried) - 1);
        if (rest == 0 || d >= total) {  // or a walk longer than any alignment
          status = ST_EDEVICE;
          break;
        }
        const int b = __builtin_ctzll(rest) + 1;
        const int32_t spb = __builtin_amdgcn_readlane(sp, b - 1);
        // every lane stores the same values; the one wave's LDS accesses stay
        // in program order, so no barrier is needed before they are read back
        sm.path[d] = (uint8_t)b;
        sm.sofar[d] = sf;
        if constexpr (Sm::Memo) {
          if (rec && fresh) {
            sm.cell[nrec] = cell;
            sm.score[nrec] = sf;
            sm.set[nrec] = (uint32_t)set;
            sm.mask[nrec] = (uint8_t)b;
            sm.walk[nrec] = (uint16_t)nwalk;
            const int at = no_hash(cell, sf);
            sm.link[nrec] = sm.head[at];
            sm.head[at] = (uint16_t)nrec;
            ++nrec;
          }
        }
        sf += spb;
#pragma unroll
        for (int i = 0; i < K; ++i) v[i] -= (b >> i) & 1;
        h -= __builtin_popcount(b);
        ++d;
        tried = 0;
        fresh = true;
      }
      sm.more = more;
      sm.status = status;
      sm.np = np;
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (lane == i) sm.top[i] = v[i];
    }
    __syncthreads();
    status = sm.status;
    if (!sm.more) break;
  }
  __threadfence_block();
  __syncthreads();
  np = sm.np;
  // ---- rows: a wave per alignment; a chunk's masks are read before its
  // columns of the first row are written ----
  if (status == ST_OK) {
    const uint64_t below = (1ull << lane) - 1;
    for (int p = wave; p < np; p += kNoThreads / 64) {
      uint8_t *blk = aln_out + (int64_t)p * K * jd.aln_cap;
      const int len = (int)len_out[p];
      int pos[K];
#pragma unroll
      for (int i = 0; i < K; ++i) pos[i] = jd.seq_off[i];
      for (int c0 = 0; c0 < len; c0 += 64) {
        const int m = c0 + lane < len ? blk[c0 + lane] : 0;
#pragma unroll
        for (int i = 0; i < K; ++i) {
          const uint64_t bits = __ballot((m >> i) & 1);
          const int x = pos[i] + __builtin_popcountll(bits & below);
          pos[i] += __builtin_popcountll(bits);
          if (m != 0)
            blk[(int64_t)i * jd.aln_cap + c0 + lane] = (m >> i) & 1 ? sm.seq[x] : (uint8_t)0xFF;
        }
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    *npaths_out = status == ST_OK ? np : 0;
    *jd.status_out = status;
    if (status != ST_OK) *jd.score_out = 0;
    finish_launch(ctrl);
  }
}

template <int K>
static int launch_nearopt_k(const JobDev &jd, Ctrl *ctrl, int64_t delta, int32_t max_paths,
                            int64_t *scores_out, uint8_t *aln_out, int64_t *len_out,
                            int32_t *npaths_out, hipStream_t s) {
  launch_begin();
  hipLaunchKernelGGL((nearopt_kernel<K>), dim3(1), dim3(kNoThreads), 0, s, jd, ctrl, delta,
                     max_paths, scores_out, aln_out, len_out, npaths_out);
  return launch_end();
}

int launch_nearopt(const JobDev &jd, Ctrl *ctrl, int64_t delta, int32_t max_paths,
                   int64_t *scores_out, uint8_t *aln_out, int64_t *len_out, int32_t *npaths_out,
                   hipStream_t s) {
#define MSA_NO_ARGS jd, ctrl, delta, max_paths, scores_out, aln_out, len_out, npaths_out, s
  switch (jd.k) {
    case 2: return launch_nearopt_k<2>(MSA_NO_ARGS);
    case 3: return launch_nearopt_k<3>(MSA_NO_ARGS);
    case 4: return launch_nearopt_k<4>(MSA_NO_ARGS);
    case 5: return launch_nearopt_k<5>(MSA_NO_ARGS);
    case 6: return launch_nearopt_k<6>(MSA_NO_ARGS);
    default: return -1;
  }
#undef MSA_NO_ARGS
}

// Where the walkers take a walk.  They start later than a single wave, share its
// compute unit and take all of it, so they lose
//   - on short walks (single wave and walkers, related sequences, unrelated ones, lengths of
//     one alignment 1 : 0.45: 40^3 11.0 and 13.0, 12.8 and 14.9, 10.6 and 13.2 us; 64^3
//     17.9 and 16.8, 19.5 and 18.8, 15.8 and 17.7; 96^3 23.7 and 14.2, 28.1 and 26.9, 22.4
//     and 22.0; 40^4 19.1 and 14.9, 20.5 and 21.9, 16.3 and 18.5; 64^4 30.3 and 24.6, 31.0
//     and 33.6, 25.6 and 25.4; 96^4 43.1 and 23.5, 47.0 and 54.0, 37.5 and 30.0; 96^2 15.6
//     and 9.6, 17.9 and 13.9), but for k = 5, whose single walk changes its tile every few
//     columns (12^5 11.8 and 9.0, 23 and 12);
//   - for k = 2, whose single walk crosses the fewest tiles, also on longer ones
//     where the lengths are apart, so that three families share the walkers (96 x 48
//     15.6 and 18.3, 128 x 43 19.8 and 21.3, 160 x 80 24.1 and 25.2, 250 x 84 36.2 and
//     36.8, 300 x 60 43.1 and 40.0);
//   - where the jobs at once are more than half the compute units (k = 5: than all
//     of them), since one wave a job runs beside many others (related, unrelated: 64
//     jobs of 100..160 residues, k = 3, 37 and 31, 51 and 52; 256 of them 38 and 40, 53
//     and 66; 1024 74 and 130, 103 and 201; 256 jobs of k = 5, 4..10 residues 17 and
//     13, 28 and 16; 1024 27 and 38, 41 and 50).
bool trace_by_walkers(const int32_t *n, int k, int njobs, int cus) {
  int64_t total = 0;
  int most = 0, least = INT32_MAX;
  for (int i = 0; i < k; ++i) {
    total += n[i];
    most = n[i] > most ? n[i] : most;
    least = n[i] < least ? n[i] : least;
  }
  if (k > kTrMaxK || total > kTrMaxTotal) return false;
  if (k == 5) return njobs == 1 || njobs <= cus;
  const bool apart = 16 * (most - least) > most;  // (as in tr_families)
  if (most < 96 || (k == 2 && apart && most < 256)) return false;
  return njobs == 1 || njobs <= cus / 2;
}

template <int K>
static int launch_trace_k(const JobDev &jd, Ctrl *ctrl, hipStream_t s) {
  launch_begin();
  hipLaunchKernelGGL((trace_kernel<K>), dim3(1), dim3(kTrThreads), 0, s, jd, ctrl);
  return launch_end();
}

int launch_trace(const JobDev &jd, Ctrl *ctrl, hipStream_t s) {
  switch (jd.k) {
    case 2: return launch_trace_k<2>(jd, ctrl, s);
    case 3: return launch_trace_k<3>(jd, ctrl, s);
    case 4: return launch_trace_k<4>(jd, ctrl, s);
    case 5: return launch_trace_k<5>(jd, ctrl, s);
    default: return -1;
  }
}

}  // namespace msa
