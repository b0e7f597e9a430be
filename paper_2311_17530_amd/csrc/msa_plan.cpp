// msa_plan.cpp -- host core of the library (no device calls).
#include "msa_plan.h"

#include <string.h>

#include <algorithm>

#include "../../include/msa_dp.h"

namespace msa {

static int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

static bool mul_ok(int64_t a, int64_t b, int64_t lim) { return a == 0 || b <= lim / a; }

// Whether a streaming fill's exchange regions, which share the face planes'
// memory, are small enough beside them: at most twice as large, or 64 MB; and no
// larger where the workspace is a large part of the card's memory, so that every
// shape that the tile fill's workspace lets on the card still fits it (509 x 1506
// x 1153 x 34: 109 GB, 143 with the exchange regions).
static bool exchange_fits(const Plan &p, int64_t bytes) {
  const int64_t faces = p.face_elems * 4;
  if (bytes <= faces) return true;
  return bytes <= std::max<int64_t>(2 * faces, kS4SmallX) &&
         bytes + p.ntiles * p.dbs <= kStreamWsMax;
}

int make_plan(const int32_t *lens, int32_t k, Plan *p, bool streams) {
  if (!lens || !p || k < 2 || k > kMaxK) return MSA_EINVAL;
  Plan q;
  q.k = k;
  q.T = tile_edge_for_k(k);
  const int64_t lim = (int64_t)1 << 50;
  q.ncell = 1;
  int64_t a = 1;
  for (int i = 0; i < k; ++i) {
    if (lens[i] < 0 || lens[i] > (1 << 24)) return MSA_EINVAL;
    q.n[i] = lens[i];
    q.P[i] = 1 + (lens[i] + q.T - 1) / q.T;
    if (!mul_ok(q.ncell, (int64_t)lens[i] + 1, lim)) return MSA_ENOMEM;
    q.ncell *= (int64_t)lens[i] + 1;
    if (!mul_ok(a, 2 * (int64_t)lens[i] + 1, lim)) return MSA_ENOMEM;
    a *= 2 * (int64_t)lens[i] + 1;
    q.total_len += lens[i];
  }
  q.nu = a - q.ncell;
  q.ntiles = 1;
  for (int i = k - 1; i >= 0; --i) {
    q.tstride[i] = (int32_t)q.ntiles;
    if (!mul_ok(q.ntiles, q.P[i], kMaxTiles)) return MSA_ENOMEM;
    q.ntiles *= q.P[i];
  }
  q.nwaves = 1 - k;
  for (int i = 0; i < k; ++i) q.nwaves += q.P[i];
  // tiles per wave: coefficients of prod_i (1 + x + ... + x^(P_i - 1))
  {
    std::vector<int64_t> cnt(q.nwaves + 1, 0), nxt(q.nwaves + 1, 0);
    cnt[0] = 1;
    int top = 0;
    for (int i = 0; i < k; ++i) {
      std::fill(nxt.begin(), nxt.end(), 0);
      int64_t run = 0;  // sliding window sum of cnt[w - P_i + 1 .. w]
      for (int w = 0; w <= top + q.P[i] - 1; ++w) {
        if (w <= top) run += cnt[w];
        if (w - q.P[i] >= 0) run -= cnt[w - q.P[i]];
        nxt[w] = run;
      }
      top += q.P[i] - 1;
      std::swap(cnt, nxt);
    }
    q.max_wave = *std::max_element(cnt.begin(), cnt.end());
  }
  const int64_t nc = ipow(q.T, k);
  q.dbs = (int32_t)((nc + 15) / 16 * 16);
  // face planes: dimension i keeps P_i - 1 planes over the other dimensions
  q.face_elems = 0;
  for (int i = 0; i < k; ++i) {
    int64_t plane = 1;
    for (int j = k - 1; j >= 0; --j) {
      if (j == i) continue;
      // the kernels form face addresses from 32-bit byte strides (a stride
      // of 2^30 words needs a face plane of at least 2^31 words, 8 GiB)
      if (plane >= ((int64_t)1 << 30)) return MSA_ENOMEM;
      q.fstride[i][j] = plane;
      if (!mul_ok(plane, (int64_t)q.n[j] + 1, lim)) return MSA_ENOMEM;
      plane *= (int64_t)q.n[j] + 1;
    }
    q.fplane[i] = plane;
    q.face_off[i] = q.face_elems;
    if (!mul_ok(plane, (int64_t)q.P[i] - 1, lim)) return MSA_ENOMEM;
    q.face_elems += plane * (q.P[i] - 1);
  }
  if (streams && k == 4 && q.n[3] <= kS4SeqMax) {
    q.s4_nb[0] = (q.n[0] + kS4Rows) / kS4Rows;
    for (int i = 1; i < 3; ++i) q.s4_nb[i] = (q.n[i] + kS4Lanes) / kS4Lanes;
    const int64_t nb0 = q.s4_nb[0], nb1 = q.s4_nb[1], nb2 = q.s4_nb[2];
    // the most steps a block runs, and one more of X0
    q.s4_steps = ((q.n[3] + 3) / 4 * 4 + 1 + 2 * (kS4Lanes - 1) + 7) / 8 * 8 + 1;
    const int64_t S = q.s4_steps;
    // (at most twice as many blocks as tiles, so nothing here overflows)
    q.s4_x0 = (nb0 - 1) * nb1 * nb2 * S * 256;
    q.s4_x1 = nb0 * (nb1 - 1) * nb2 * S * 16 * kS4Rows;
    q.s4_x2 = nb0 * nb1 * (nb2 - 1) * S * 16 * kS4Rows;
    // Shapes whose exchange regions would be far larger than the face planes
    // (short second and third sequences leave most lanes of a block idle) keep
    // the tile fill; the kernel forms a line's offset in the direction blocks
    // of one tile row along dimension 0 in 32 bits.
    q.s4 = exchange_fits(q, sweep4_x_words(q) * 4) &&
           (int64_t)q.tstride[0] * q.dbs < ((int64_t)1 << 32);
  }
  if (streams && k == 5 && q.n[4] <= kS5SeqMax) {
    // the most steps a block runs
    q.s5_steps = ((q.n[4] + 3) / 4 * 4 + 1 + 4 * (q.T - 1) + 7) / 8 * 8;
    q.s5_x = q.ntiles / q.P[4] * q.s5_steps * kS5Step;
    // Shapes whose exchange region would be far larger than the face planes
    // keep the tile fill; the kernel forms offsets in the region in 32 bits.
    const int64_t bytes = sweep5_x_words(q) * 4;
    // Nor do shapes of many tile waves whose blocks are hardly longer than
    // their skew: each wave waits for a block's start (tile and streaming fill, us:
    // 100 x 100 x 3 x 3 x 3, 54 waves, 497 and 547; 4 x 100 x 100 x 4 x 4 524 and 542; 60 x 60 x
    // 8 x 8 x 2, 36 waves, 367 and 363; 40 x 40 x 12 x 12 x 3, 28 waves, 306 and 256; 120 x
    // 60 x 4 x 4 x 8, 50 waves, 525 and 477).
    q.s5 = exchange_fits(q, bytes) && bytes < ((int64_t)1 << 32) &&
           !(q.n[4] <= 4 && q.nwaves > 40);
  }
  // workspace layout
  int64_t o = 0;
  q.off_ctrl = o;   o = align256(o + (int64_t)sizeof(Ctrl));
  q.off_sub = o;    o = align256(o + kSubBytes);
  q.off_order = o;  o = align256(o + q.ntiles * 4);
  q.ncols = q.ntiles / q.P[0];
  q.off_corder = o; o = align256(o + q.ncols * 4);
  q.off_flags = o;  o = align256(o + q.ntiles * 4);
  q.off_path = o;   o = align256(o + std::max<int64_t>(q.total_len, 1));
  q.off_faces = o;
  if (!mul_ok(q.face_elems, 4, lim)) return MSA_ENOMEM;
  // at least one block, so a clamped (unconditional) read at offset 0 is in
  // range; the streaming k = 4 and k = 5 fills' exchange regions share the planes' memory
  // (the words of a tile fill carry no valid tag, and it reads none of theirs)
  o = align256(o + std::max<int64_t>(
                       {q.face_elems * 4, q.s4 ? sweep4_x_words(q) * 4 : 0,
                        q.s5 ? sweep5_x_words(q) * 4 : 0, (int64_t)256}));
  q.off_dir = o;
  if (!mul_ok(q.ntiles, q.dbs, lim)) return MSA_ENOMEM;
  o = align256(o + q.ntiles * q.dbs);
  q.prunable = k >= kPruneMinK && k <= kPruneMaxK;
  for (int i = 0; i < k; ++i) q.prunable = q.prunable && q.n[i] < kPruneMaxLen;
  if (q.prunable) {
    int64_t tab = 0, bm = 0;
    for (int i = 0; i < k; ++i)
      for (int j = i + 1; j < k; ++j) {
        const int p = q.npairs++;
        q.pi[p] = i;
        q.pj[p] = j;
        q.tab_off[p] = tab;
        tab += 2 * ((int64_t)q.n[i] + 1) * ((int64_t)q.n[j] + 1);
        q.bm_off[p] = bm;
        bm += (int64_t)q.P[i] * q.P[j];
      }
    q.nblocks = (int32_t)((q.ntiles + kSelBlock - 1) / kSelBlock);
    q.off_ptab = o;   o = align256(o + tab * 4);
    q.off_pbm = o;    o = align256(o + bm * 4);
    q.off_keep = o;   o = align256(o + q.ntiles);
    q.off_korder = o; o = align256(o + q.ntiles * 4);
    q.off_bcnt = o;   o = align256(o + (int64_t)q.nblocks * 4);
  }
  if (k == 3) {
    q.sw_nb0 = (q.n[0] + 1 + kSwRows - 1) / kSwRows;
    q.sw_nb1 = (q.n[1] + 1 + kSwLanes - 1) / kSwLanes;
    q.x0_plane = ((int64_t)q.n[1] + q.n[2] + 1) * ((int64_t)q.n[1] + 1);
    q.x1_plane = ((int64_t)q.n[0] + 1) * ((int64_t)q.n[2] + kSwNW);  // X1[e = v2 + w][v0]
    q.off_x0 = o;
    o = align256(o + std::max<int64_t>((q.sw_nb0 - 1) * q.x0_plane * 4, 256));
    q.off_x1 = o;
    o = align256(o + std::max<int64_t>((q.sw_nb1 - 1) * q.x1_plane * 4, 256));
    q.x_bytes = o - q.off_x0;
  }
  if (q.s4) {
    q.off_s4order = o;
    o = align256(o + (int64_t)q.s4_nb[0] * q.s4_nb[1] * q.s4_nb[2] * 4);
  }
  if (q.s5) {
    q.off_s4order = o;
    o = align256(o + q.ntiles / q.P[4] * 4);
  }
  q.bytes = o;
  *p = q;
  return MSA_OK;
}

int64_t sweep4_x_words(const Plan &p) {
  return kS4PadFront + p.s4_x0 + p.s4_x1 + p.s4_x2 + kS4PadBack;
}

bool sweep4_eligible(const Plan &p, int alpha, int32_t flags) {
  return p.s4 && flags == 0 && alpha >= 1 && alpha <= kS4SubMax;
}

void fill_sweep4dev(const Plan &p, Sweep4Dev *sd) {
  memset(sd, 0, sizeof(*sd));
  for (int i = 0; i < 4; ++i) sd->n[i] = p.n[i];
  for (int i = 0; i < 3; ++i) {
    sd->nb[i] = p.s4_nb[i];
    sd->ts[i] = p.tstride[i];
  }
  sd->S = p.s4_steps;
}

std::vector<int32_t> sweep4_key_counts(const Plan &p) {
  const int nb0 = p.s4_nb[0], nb1 = p.s4_nb[1], nb2 = p.s4_nb[2];
  // blocks with b1 + b2 = m cover the keys 4 m .. 4 m + nb0 - 1, each as often
  // as there are such (b1, b2)
  std::vector<int32_t> d(sweep4_key(nb0 - 1, nb1 - 1, nb2 - 1) + 2, 0);
  for (int m = 0; m <= nb1 + nb2 - 2; ++m) {
    const int cnt = std::min(m, nb1 - 1) - std::max(0, m - (nb2 - 1)) + 1;
    d[sweep4_key(0, m, 0)] += cnt;
    d[sweep4_key(nb0, m, 0)] -= cnt;
  }
  for (size_t i = 1; i < d.size(); ++i) d[i] += d[i - 1];
  d.pop_back();
  return d;
}

void make_sweep4_order(const Plan &p, std::vector<int32_t> *order) {
  const int nb0 = p.s4_nb[0], nb1 = p.s4_nb[1], nb2 = p.s4_nb[2];
  const auto key = sweep4_key;
  std::vector<int32_t> count(key(nb0, nb1, nb2) + 2, 0);
  for (int b0 = 0; b0 < nb0; ++b0)
    for (int b1 = 0; b1 < nb1; ++b1)
      for (int b2 = 0; b2 < nb2; ++b2) ++count[key(b0, b1, b2) + 1];
  for (size_t i = 1; i < count.size(); ++i) count[i] += count[i - 1];
  order->assign((size_t)nb0 * nb1 * nb2, 0);
  int32_t b = 0;
  for (int b0 = 0; b0 < nb0; ++b0)
    for (int b1 = 0; b1 < nb1; ++b1)
      for (int b2 = 0; b2 < nb2; ++b2) (*order)[count[key(b0, b1, b2)]++] = b++;
}

int64_t sweep5_x_words(const Plan &p) { return kS5PadFront + p.s5_x + kS5PadBack; }

bool sweep5_eligible(const Plan &p, int alpha, int32_t flags) {
  return p.s5 && flags == 0 && alpha >= 1 && alpha <= kS4SubMax;
}

void fill_sweep5dev(const Plan &p, Sweep5Dev *sd) {
  memset(sd, 0, sizeof(*sd));
  for (int i = 0; i < 5; ++i) sd->n[i] = p.n[i];
  for (int i = 0; i < 4; ++i) {
    sd->nb[i] = p.P[i];
    sd->ts[i] = p.tstride[i];
  }
  sd->S = p.s5_steps;
}

std::vector<int32_t> sweep5_key_counts(const Plan &p) {
  std::vector<int32_t> cnt(1, 1);
  for (int i = 0; i < 4; ++i) {
    std::vector<int32_t> nxt(cnt.size() + p.P[i] - 1, 0);
    for (size_t x = 0; x < cnt.size(); ++x)
      for (int c = 0; c < p.P[i]; ++c) nxt[x + c] += cnt[x];
    cnt.swap(nxt);
  }
  return cnt;
}

void make_sweep5_order(const Plan &p, std::vector<int32_t> *order) {
  const std::vector<int32_t> cnt = sweep5_key_counts(p);
  std::vector<int32_t> at(cnt.size(), 0);
  for (size_t x = 1; x < cnt.size(); ++x) at[x] = at[x - 1] + cnt[x - 1];
  order->assign(p.ntiles / p.P[4], 0);
  int32_t b = 0;
  for (int c0 = 0; c0 < p.P[0]; ++c0)
    for (int c1 = 0; c1 < p.P[1]; ++c1)
      for (int c2 = 0; c2 < p.P[2]; ++c2)
        for (int c3 = 0; c3 < p.P[3]; ++c3) (*order)[at[c0 + c1 + c2 + c3]++] = b++;
}

// Where the streaming k = 3 fill is the faster one in the co-optimal and
// near-optimal modes (in the others it always is but for lines far longer than the
// other lengths).  Its time is that of its steps in a row: the third length,
// 66 steps a block along dimension 1 and 14 along dimension 0 later.  The tile
// fill's is that of its waves, and more steps a wave than measured here are
// too many.  Tile and streaming fill, us, by steps a wave:
//   near-optimal, whose stores of scores lengthen every step of a full block:
//     300 x 257 x 281 (13.1) 646 and 534, 157 x 238 x 213 (13.7) 425 and 405, 419 x
//     560 x 464 (13.9) 1226 and 1156; 20 x 200 x 200 (14.2) 284 and 305, 87 x 359 x 173
//     (14.4) 417 and 458, 133 x 400 x 400 (14.8) 633 and 687, 20 x 512 x 512 (15.6) 678
//     and 783; with few rows, 5 x 40 x 300 (14.3) 186 and 143, 1 x 64 x 600 (15.2) 304
//     and 284, 2 x 512 x 512 (15.8) 467 and 501;
//   both, few lines in all, whose tiles are small: co-optimal 2 x 2 x 300 (13.8)
//     138 and 136, 1 x 1 x 600 (14.7) 239 and 264, 3 x 3 x 1000 (15.2) 413 and 432, 4 x 4 x
//     600 (14.8) 274 and 264; near-optimal 1 x 1 x 1000 315 and 374, 4 x 4 x 600 226 and
//     237.
static bool sweep3_pays(const Plan &p, int32_t flags) {
  if (flags != kCoOptimal && flags != kNearOpt) return true;
  const int nb1 = p.n[1] / kSwLanes, nb0 = p.n[0] / kSwRows;  // blocks before the last
  const int64_t steps = (int64_t)p.n[2] + 1 + 66 * (int64_t)nb1 + 14 * (int64_t)nb0 +
                        p.n[1] % kSwLanes + p.n[0] % kSwRows / kSwRPW;
  const int most = std::max(p.n[0], p.n[1]);
  if (most <= (flags == kCoOptimal ? 3 : 7)) return 10 * steps <= 142 * (int64_t)p.nwaves;
  if (flags == kCoOptimal) return true;
  return 10 * steps <= (p.n[0] < 12 ? 155 : 142) * (int64_t)p.nwaves;
}

// The streaming k = 3 fill covers the plain mode and one of the end-gap-free,
// co-optimal and near-optimal ones.
bool sweep3_eligible(const Plan &p, int alpha, int32_t flags) {
  // the loader keeps each exchange element's offset within its window of
  // n2 + 1 steps as 32 bits: n2 steps of n1 + 1 (X0) or n0 + 1 (X1) words
  const int64_t wmax = (int64_t)p.n[2] * ((int64_t)std::max(p.n[0], p.n[1]) + 1);
  const bool mode =
      flags == 0 || flags == kEndGapsFree || flags == kCoOptimal || flags == kNearOpt;
  return p.k == 3 && mode && sweep3_pays(p, flags) && alpha >= 1 && alpha <= kSwSubMax &&
         p.n[2] <= kSwSeqMax && wmax < ((int64_t)1 << 31);
}

void make_tile_order(const Plan &p, std::vector<int32_t> *order) {
  std::vector<int64_t> count(p.nwaves + 1, 0);
  auto wave = [&](int64_t t) {
    int s = 0;
    for (int i = 0; i < p.k; ++i) s += (int)((t / p.tstride[i]) % p.P[i]);
    return s;
  };
  for (int64_t t = 0; t < p.ntiles; ++t) count[wave(t) + 1]++;
  for (int w = 0; w < p.nwaves; ++w) count[w + 1] += count[w];
  order->assign(p.ntiles, 0);
  for (int64_t t = 0; t < p.ntiles; ++t) (*order)[count[wave(t)]++] = (int32_t)t;
}

void make_column_order(const Plan &p, std::vector<int32_t> *order) {
  std::vector<int32_t> all;
  make_tile_order(p, &all);
  order->clear();
  order->reserve(p.ncols);
  for (int32_t t : all)
    if (t / p.tstride[0] == 0) order->push_back(t);  // c_0 = 0: first tile of a column
}

int score_bounds(const int32_t *lens, int32_t k, const int8_t *submat, int32_t alpha,
                 int32_t gap, int64_t *lo, int64_t *hi) {
  if (!lens || !submat || !lo || !hi || k < 2 || k > kMaxK || alpha < 1 || alpha > 255)
    return MSA_EINVAL;
  int64_t sum = 0;
  for (int i = 0; i < k; ++i) {
    if (lens[i] < 0) return MSA_EINVAL;
    sum += lens[i];
  }
  int smax = -128, sabs = 0;
  for (int i = 0; i < alpha * alpha; ++i) {
    smax = std::max<int>(smax, submat[i]);
    sabs = std::max<int>(sabs, submat[i] < 0 ? -submat[i] : submat[i]);
  }
  if (gap <= 0) {
    *lo = (int64_t)gap * (k - 1) * sum;
    int64_t pairs = 0;
    for (int i = 0; i < k; ++i)
      for (int j = i + 1; j < k; ++j) pairs += std::min(lens[i], lens[j]);
    *hi = (int64_t)std::max(0, smax) * pairs;
  } else {
    const int64_t m = std::max<int64_t>(gap, sabs);
    *hi = sum * (int64_t)(k * (k - 1) / 2) * m;
    *lo = -*hi;
  }
  return MSA_OK;
}

int check_scoring(const int32_t *lens, int32_t k, const int8_t *submat, int32_t alpha,
                  int32_t gap) {
  if (!submat || alpha < 1 || alpha > 255) return MSA_EINVAL;
  for (int a = 0; a < alpha; ++a)
    for (int b = a + 1; b < alpha; ++b)
      if (submat[a * alpha + b] != submat[b * alpha + a]) return MSA_EINVAL;
  int64_t lo = 0, hi = 0;
  int rc = score_bounds(lens, k, submat, alpha, gap, &lo, &hi);
  if (rc) return rc;
  // largest |column score|: C(k,2) * max(|gap|, max|sub|)
  int sabs = 0;
  for (int i = 0; i < alpha * alpha; ++i)
    sabs = std::max<int>(sabs, submat[i] < 0 ? -submat[i] : submat[i]);
  const int64_t g = gap < 0 ? -(int64_t)gap : gap;
  const int64_t colmax = (int64_t)(k * (k - 1) / 2) * std::max<int64_t>(g, sabs);
  const int64_t span = (lo < 0 ? -lo : lo) + (hi < 0 ? -hi : hi) + 2 * colmax + 1;
  // keys are score * 2^k; the -infinity key is -2^30 (see kNegKey)
  if (span > (((int64_t)1 << 30) >> k)) return MSA_ERANGE;
  return MSA_OK;
}

int check_scoring_mode(const int32_t *lens, int32_t k, const int8_t *submat, int32_t alpha,
                       int32_t gap, uint32_t flags) {
  int rc = check_scoring(lens, k, submat, alpha, gap);
  if (rc || !(flags & kPrune)) return rc;
  // Pruned mode: a kept tile whose lower neighbours were pruned starts from
  // -infinity halo keys, and such values can travel along a monotone path of
  // up to sum(n_i) cells through kept tiles, each step adding one column score
  // (|column score| <= colmax).  They must stay below every real key (real
  // scores are >= lo) and above the int32 minimum:
  //   -2^30 + 2^k * sum(n) * colmax < 2^k * (lo - 1)
  //   -2^30 - 2^k * sum(n) * colmax >= -2^31.
  int64_t lo = 0, hi = 0;
  rc = score_bounds(lens, k, submat, alpha, gap, &lo, &hi);
  if (rc) return rc;
  int64_t sum = 0;
  for (int i = 0; i < k; ++i) sum += lens[i];
  int sabs = 0;
  for (int i = 0; i < alpha * alpha; ++i)
    sabs = std::max<int>(sabs, submat[i] < 0 ? -submat[i] : submat[i]);
  const int64_t g = gap < 0 ? -(int64_t)gap : gap;
  const int64_t colmax = (int64_t)(k * (k - 1) / 2) * std::max<int64_t>(g, sabs);
  const int64_t chain = sum * colmax;
  const int64_t need = chain + (lo < 0 ? -lo : lo) + 1;
  if (need >= (((int64_t)1 << 30) >> k)) return MSA_ERANGE;
  return MSA_OK;
}

int64_t nearopt_bytes(const Plan &p) { return align256(p.ntiles * (int64_t)p.dbs * 4); }

// Unsigned division of any 32-bit n by an invariant d >= 1 as
// q = (t + ((n - t) >> s1)) >> s2 with t = mulhi(m, n), after Granlund and
// Montgomery, "Division by invariant integers using multiplication" (1994):
// l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1, s1 = min(l, 1),
// s2 = max(l - 1, 0).  The kernels use it for tile coordinates, which then
// take scalar instructions instead of a division on the vector unit.
void udiv_magic(uint32_t d, uint32_t *m, uint32_t *sh) {
  int l = 0;
  while (l < 32 && ((uint64_t)1 << l) < d) ++l;
  *m = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << l) - d)) / d + 1);
  *sh = (uint32_t)std::min(l, 1) | ((uint32_t)std::max(l - 1, 0) << 8);
}

uint32_t udiv_apply(uint32_t n, uint32_t m, uint32_t sh) {
  const uint32_t t = (uint32_t)(((uint64_t)m * n) >> 32);
  return (t + ((n - t) >> (sh & 0xff))) >> (sh >> 8);
}

void fill_jobdev(const Plan &p, char *ws, int alpha, int gap, JobDev *jd) {
  memset(jd, 0, sizeof(*jd));
  jd->k = p.k;
  jd->T = p.T;
  jd->alpha = alpha;
  jd->gap = gap;
  int32_t off = 0;
  for (int i = 0; i < p.k; ++i) {
    jd->n[i] = p.n[i];
    jd->P[i] = p.P[i];
    jd->tstride[i] = p.tstride[i];
    udiv_magic((uint32_t)p.tstride[i], &jd->tdm[i], &jd->tdsh[i]);
    jd->seq_off[i] = off;
    off += p.n[i];
    jd->face_off[i] = p.face_off[i];
    jd->fplane[i] = p.fplane[i];
    for (int j = 0; j < p.k; ++j) jd->fbstride[i][j] = (uint32_t)(4 * p.fstride[i][j]);
  }
  jd->ntiles = (int32_t)p.ntiles;
  jd->nwaves = p.nwaves;
  jd->dbs = p.dbs;
  jd->total_len = p.total_len;
  jd->sub = reinterpret_cast<const int8_t *>(ws + p.off_sub);
  jd->faces = reinterpret_cast<int32_t *>(ws + p.off_faces);
  jd->dir = reinterpret_cast<uint8_t *>(ws + p.off_dir);
  jd->flags = reinterpret_cast<int32_t *>(ws + p.off_flags);
  jd->corder = reinterpret_cast<const int32_t *>(ws + p.off_corder);
  jd->ncols = (int32_t)p.ncols;
  jd->path = reinterpret_cast<uint8_t *>(ws + p.off_path);
  jd->scores = ws ? reinterpret_cast<int32_t *>(ws + p.bytes) : nullptr;
}

}  // namespace msa

namespace msa {

void fill_prunedev(const Plan &p, char *ws, const uint8_t *d_seqs, int64_t *d_score,
                   PruneDev *pd) {
  memset(pd, 0, sizeof(*pd));
  pd->k = p.k;
  pd->npairs = p.npairs;
  pd->T = p.T;
  pd->ntiles = (int32_t)p.ntiles;
  int32_t off = 0;
  for (int i = 0; i < p.k; ++i) {
    pd->n[i] = p.n[i];
    pd->P[i] = p.P[i];
    pd->tstride[i] = p.tstride[i];
    pd->seq_off[i] = off;
    off += p.n[i];
  }
  for (int q = 0; q < p.npairs; ++q) {
    pd->pi[q] = p.pi[q];
    pd->pj[q] = p.pj[q];
    pd->tab_off[q] = p.tab_off[q];
    pd->bm_off[q] = p.bm_off[q];
  }
  pd->nblocks = p.nblocks;
  pd->seqs = d_seqs;
  pd->sub = reinterpret_cast<const int8_t *>(ws + p.off_sub);
  pd->tabs = reinterpret_cast<int32_t *>(ws + p.off_ptab);
  pd->bm = reinterpret_cast<int32_t *>(ws + p.off_pbm);
  pd->keep = reinterpret_cast<uint8_t *>(ws + p.off_keep);
  pd->order = reinterpret_cast<const int32_t *>(ws + p.off_order);
  pd->korder = reinterpret_cast<int32_t *>(ws + p.off_korder);
  pd->bcnt = reinterpret_cast<int32_t *>(ws + p.off_bcnt);
  pd->score = d_score;
}

}  // namespace msa
