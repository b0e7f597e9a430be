// msa_launch.cpp -- staging and running one batched persistent launch.
#include "msa_launch.h"

#include <string.h>

#include <algorithm>
#include <map>

#include "msa_runtime.h"
#include "msa_tune.h"

namespace msa {

static int64_t a256(int64_t x) { return (x + 255) & ~(int64_t)255; }

// The batch descriptor sits right after the control block in every arena, and
// the job descriptors right after it: both addresses are fixed per arena, so
// a captured launch sequence stays valid for every batch the arena holds.
constexpr int64_t kArgsOff = 256;
constexpr int64_t kJobsOff = 512;
static_assert(sizeof(Ctrl) <= kArgsOff, "control block first");
static_assert(kArgsOff + (int64_t)sizeof(BatchArgs) <= kJobsOff, "descriptor before the jobs");

int validate_job(const msa_job &j, int64_t) {
  if (j.k < 2 || j.k > MSA_MAX_K) return MSA_EINVAL;
  if (!j.submat || j.alpha < 1 || j.alpha > 255) return MSA_EINVAL;
  for (int i = 0; i < j.k; ++i) {
    if (j.lens[i] < 0) return MSA_EINVAL;
    if (j.lens[i] > 0 && !j.seqs[i]) return MSA_EINVAL;
    for (int32_t t = 0; t < j.lens[i]; ++t)
      if (j.seqs[i][t] >= j.alpha) return MSA_EINVAL;
  }
  Plan p;
  int rc = make_plan(j.lens, j.k, &p);
  if (rc) return rc;
  return check_scoring(j.lens, j.k, j.submat, j.alpha, j.gap);
}

namespace {
struct JobSizes {
  Plan p;
  int64_t cap = 0;       // alignment row capacity
  int64_t nw = 0;        // waves
  int64_t small = 0;     // host-initialised bytes
  int64_t big = 0;       // device-only bytes (path, faces, dir)
  int64_t out = 0;       // output rows
  bool s4 = false;       // streaming fill (k = 4, 5)
  std::vector<int32_t> keys;  // its blocks per key
  int64_t x = 0;         // its exchange regions (bytes)
  int64_t total(int64_t ntiles) const {
    return small + big + x + out + 12 * ntiles + (int64_t)sizeof(JobDev) + 64 +
           (s4 ? (int64_t)std::max(sizeof(Sweep4Dev), sizeof(Sweep5Dev)) + 8 : 0);
  }
  int64_t blocks() const {  // of a streaming fill
    return p.k == 5 ? p.ntiles / p.P[4] : (int64_t)p.s4_nb[0] * p.s4_nb[1] * p.s4_nb[2];
  }
  int32_t steps() const { return p.k == 5 ? p.s5_steps : p.s4_steps; }
};

// cap: bytes of the arena the job has to fit.  A k = 4 or 5 job takes the streaming
// fill where that is possible; where only the tile fill's smaller layout fits
// the arena, it keeps that.  So do all k = 5 jobs in an arena below kSmallArena: there, fewer
// launches give more than the faster fill, and jobs of both kinds in a launch wait for
// each other (512 jobs of
// 5..12 residues, tile and streaming fill, ms: 32 MB 10.3 and 16.6, 64 MB 9.0 and 11.6,
// 128 MB 8.3 and 9.0, 256 MB 7.9 and 8.0, 512 MB 7.8 and 7.6; 256 of 12..20 64 MB 25.2
// and 32.4, 128 MB 19.4 and 18.6, 256 MB 16.7 and 13.6; k = 4, whose layouts grow by less,
// 512 jobs of 16..40 in 64 MB 15.6 and 13.3).
constexpr int64_t kSmallArena = (int64_t)96 << 20;
int sizes_of(const msa_job &j, int64_t cap, JobSizes *s) {
  int rc = make_plan(j.lens, j.k, &s->p);
  if (rc) return rc;
  const Plan &p = s->p;
  s->cap = std::max<int64_t>(1, p.total_len);
  s->nw = p.nwaves;
  s->small = a256(std::max<int64_t>(p.total_len, 1)) +        // sequences
             a256((int64_t)(j.k + 1) * p.nwaves * 4) +        // wave counts
             a256((int64_t)p.nwaves * 8) +                    // wave queue slots
             256;                                             // job status
  s->big = a256(std::max<int64_t>(p.total_len, 1)) +          // traceback path
           a256(std::max<int64_t>(p.face_elems * 4, 256)) +   // face planes
           a256(p.ntiles * p.dbs);                            // direction blocks
  s->out = a256((int64_t)j.k * s->cap);
  if (sweep4_eligible(p, j.alpha, 0) || sweep5_eligible(p, j.alpha, 0)) {
    JobSizes t = *s;
    t.s4 = true;
    t.keys = p.k == 5 ? sweep5_key_counts(p) : sweep4_key_counts(p);
    t.x = a256((p.k == 5 ? sweep5_x_words(p) : sweep4_x_words(p)) * 4);
    t.small = a256(std::max<int64_t>(p.total_len, 1)) + a256((int64_t)t.keys.size() * 4) + 256;
    t.big = a256(std::max<int64_t>(p.total_len, 1)) + a256(p.ntiles * p.dbs);
    if (t.total(p.ntiles) + Launch::overhead_bytes(1, p.ntiles) <= cap &&
        (p.k == 4 || cap >= kSmallArena))
      *s = t;
  }
  return MSA_OK;
}
}  // namespace

int64_t job_arena_bytes(const msa_job &j, int64_t cap) {
  JobSizes s;
  if (sizes_of(j, cap, &s)) return -1;
  return s.total(s.p.ntiles);
}

bool job_streams(const msa_job &j, int64_t cap) {
  JobSizes s;
  return sizes_of(j, cap, &s) == MSA_OK && s.s4;
}

int64_t Launch::overhead_bytes(int njobs, int64_t ntiles_total) {
  int64_t tables = 0;
  for (int k = 2; k <= kMaxK; ++k) {
    const int T = tile_edge_for_k(k);
    tables += a256((int64_t)ipow(T, k) * 4) + a256((int64_t)(k * (T - 1) + 2) * 4);
  }
  return 768 + tables + a256((int64_t)njobs * sizeof(JobDev)) + a256((int64_t)(njobs + 1) * 8) +
         a256((int64_t)njobs * 24) + 3 * a256(ntiles_total * 4) + 255 * 255 * 4 + 4096;
}

Launch::~Launch() {
  if (busy_) wait();
  drop_graphs();
  if (d_) (void)hipFree(d_);
  if (h_in_) (void)hipHostFree(h_in_);
  if (h_out_) (void)hipHostFree(h_out_);
  if (done_) (void)hipEventDestroy(done_);
  if (start_) (void)hipEventDestroy(start_);
  if (stream_ && own_stream_) (void)hipStreamDestroy(stream_);
}

int Launch::init(int64_t bytes, hipStream_t shared) {
  if (hipGetDevice(&device_) != hipSuccess) return MSA_EDEVICE;
  if (!stream_ && shared) {
    stream_ = shared;
    own_stream_ = false;
  }
  if (!stream_ && hipStreamCreateWithFlags(&stream_, hipStreamNonBlocking) != hipSuccess)
    return MSA_EDEVICE;
  if (!done_ && hipEventCreateWithFlags(&done_, hipEventDefault) != hipSuccess)
    return MSA_EDEVICE;
  if (!start_ && hipEventCreateWithFlags(&start_, hipEventDefault) != hipSuccess)
    return MSA_EDEVICE;
  if (cap_ < bytes) {
    drop_graphs();  // they hold addresses inside the old arena
    if (d_) (void)hipFree(d_);
    d_ = nullptr;
    cap_ = 0;
    if (hipMalloc(&d_, bytes) != hipSuccess) {
      d_ = nullptr;
      return MSA_ENOMEM;
    }
    cap_ = bytes;
    x_clean_ = cap_;  // nothing known of the new arena
  }
  // Pinned staging is made here, once per arena, so that launches allocate none.
  int rc = ensure_host(1 << 20, 1 << 20);
  if (rc) return rc;
  // The stream's first kernel and its first copies each way make the runtime
  // create the hardware queues behind them; doing it here keeps that out of
  // the time when other slots' persistent fills run (the queue list changes
  // then, and running queues are preempted).
  if (hipMemsetAsync(d_, 0, 256, stream_) != hipSuccess ||
      hipMemcpyAsync(d_, h_in_, 256, hipMemcpyHostToDevice, stream_) != hipSuccess ||
      hipMemcpyAsync(h_out_, d_, 256, hipMemcpyDeviceToHost, stream_) != hipSuccess ||
      hipStreamSynchronize(stream_) != hipSuccess)
    return MSA_EDEVICE;
  return MSA_OK;
}

// (Walks past the walkers' bounds, or many k = 5 jobs, are rare: those graphs
// come when they are needed.)
void Launch::ensure_graphs() {
  for (int kc = 0; kc < 4; ++kc) {
    const int grid = batch_grid(kc);
    for (int parts = 0; parts < kBatchParts; ++parts) {
      const bool fills = kc <= 1 ? (parts & (kBatchTiles | kBatchStreams)) != 0
                                 : (parts & (kBatchTiles | kBatchStreams)) == kBatchTiles;
      const int walks = parts & (kBatchWalkers | kBatchSingle);
      if (fills && ((walks == kBatchWalkers && kc <= 1) || (walks == kBatchSingle && kc != 1)))
        (void)ensure_graph(kc, parts, grid);
    }
  }
}

// Persistent workgroups of the batched fill: every one that fits, or the
// tuned count per CU.
int Launch::batch_grid(int kc) const {
  int wpc = batch_occupancy(kc);
  TuneChoice tc;
  if (tune_get(kTuneBatch, kc, 0, &tc) && tc.wpc > 0) wpc = std::min(wpc, (int)tc.wpc);
  const int grid = device_cu_count() * wpc;
  return grid < 1 ? 1 : grid;
}

void Launch::drop_graphs() {
  for (auto &row : graph_)
    for (Graph &gr : row) {
      if (gr.exec) (void)hipGraphExecDestroy(gr.exec);
      gr = Graph();
    }
}

// Captures the launch sequence of k class kc on this arena.  Returns 0 when
// a graph is ready; otherwise the caller launches the kernels directly.
int Launch::ensure_graph(int kc, int parts, int grid) {
  Graph &gr = graph_[kc][parts];
  if (gr.exec && gr.grid != grid) {  // another tuned grid: capture again
    (void)hipGraphExecDestroy(gr.exec);
    gr.exec = nullptr;
  }
  if (gr.exec) return 0;
  if (gr.failed) return -1;
  gr.grid = grid;
  hipGraph_t g = nullptr;
  bool ok = hipStreamBeginCapture(stream_, hipStreamCaptureModeThreadLocal) == hipSuccess;
  if (ok) {
    const int rc = launch_batch(kc, parts, reinterpret_cast<const BatchArgs *>(d_ + kArgsOff),
                                reinterpret_cast<const JobDev *>(d_ + kJobsOff),
                                reinterpret_cast<Ctrl *>(d_), grid, stream_);
    ok = hipStreamEndCapture(stream_, &g) == hipSuccess && rc == 0 && g;
  }
  ok = ok && hipGraphInstantiate(&gr.exec, g, nullptr, nullptr, 0) == hipSuccess;
  if (g) (void)hipGraphDestroy(g);
  if (!ok) {
    gr.exec = nullptr;
    gr.failed = true;
    (void)hipGetLastError();  // clear a capture error; the direct launches follow
    return -1;
  }
  return 0;
}

int Launch::ensure_host(int64_t in_bytes, int64_t out_bytes) {
  if (h_in_cap_ < in_bytes) {
    if (h_in_) (void)hipHostFree(h_in_);
    h_in_ = nullptr;
    h_in_cap_ = 0;
    const int64_t want = std::max<int64_t>(in_bytes, 1 << 20);
    if (hipHostMalloc((void **)&h_in_, want, hipHostMallocDefault) != hipSuccess) return MSA_ENOMEM;
    h_in_cap_ = want;
  }
  if (h_out_cap_ < out_bytes) {
    if (h_out_) (void)hipHostFree(h_out_);
    h_out_ = nullptr;
    h_out_cap_ = 0;
    const int64_t want = std::max<int64_t>(out_bytes, 1 << 20);
    if (hipHostMalloc((void **)&h_out_, want, hipHostMallocDefault) != hipSuccess)
      return MSA_ENOMEM;
    h_out_cap_ = want;
  }
  return MSA_OK;
}

int Launch::start(const std::vector<const msa_job *> &jobs,
                  const std::vector<hipEvent_t> &after) {
  if (busy_ || jobs.empty()) return MSA_EINVAL;
  const int nj = (int)jobs.size();
  const int kc = kclass_of(jobs[0]->k);
  std::vector<JobSizes> sz(nj);
  int64_t tiles = 0, small = 0, big = 0, outb = 0;
  for (int i = 0; i < nj; ++i) {
    if (kclass_of(jobs[i]->k) != kc) return MSA_EINVAL;
    if (sizes_of(*jobs[i], cap_, &sz[i])) return MSA_EINVAL;
    if (!sz[i].s4) tiles += sz[i].p.ntiles;
    small += sz[i].small;
    big += sz[i].big;
    outb += sz[i].out;
  }
  if (tiles >= ((int64_t)1 << 31) - 1) return MSA_ENOMEM;

  // ---- layout: [inputs (one host-to-device copy)][outputs][device only] ----
  int64_t o = 0;
  const int64_t off_ctrl = o;  o += 256;
  const int64_t off_args = o;  o = a256(o + (int64_t)sizeof(BatchArgs));
  const int64_t off_jobs = o;  o = a256(o + (int64_t)nj * sizeof(JobDev));
  if (off_args != kArgsOff || off_jobs != kJobsOff) return MSA_EINVAL;
  const int64_t off_jt = o;    o = a256(o + (int64_t)(nj + 1) * 8);
  const int64_t off_jc = o;    o = a256(o + (int64_t)(nj + 1) * 8);
  int n4 = 0;               // streaming jobs, their blocks and exchange bytes
  int64_t blocks4 = 0, x4 = 0;
  for (int i = 0; i < nj; ++i)
    if (sz[i].s4) {
      ++n4;
      blocks4 += sz[i].blocks();
      x4 += sz[i].x;
    }
  if (blocks4 >= ((int64_t)1 << 30)) return MSA_ENOMEM;
  const int64_t off_s4jobs = o; o = a256(o + (int64_t)n4 * (kc == 1 ? sizeof(Sweep5Dev) : sizeof(Sweep4Dev)));
  const int64_t off_s4pre = o;  o = a256(o + (int64_t)(n4 + 1) * 4);
  // substitution matrices, deduplicated by content
  std::map<std::string, int64_t> subs;
  std::vector<int64_t> sub_off(nj);
  for (int i = 0; i < nj; ++i) {
    const msa_job &j = *jobs[i];
    std::string key((const char *)j.submat, (size_t)j.alpha * j.alpha);
    key.push_back((char)j.alpha);
    auto it = subs.find(key);
    if (it == subs.end()) {
      it = subs.emplace(key, o).first;
      o = a256(o + (int64_t)j.alpha * j.alpha);
    }
    sub_off[i] = it->second;
  }
  std::vector<int64_t> job_small(nj);
  for (int i = 0; i < nj; ++i) {
    job_small[i] = o;
    o += sz[i].small;
  }
  const int64_t in_bytes = o;
  // outputs
  const int64_t off_out = o;
  const int64_t off_score = o;  o = a256(o + (int64_t)nj * 8);
  const int64_t off_len = o;    o = a256(o + (int64_t)nj * 8);
  const int64_t off_stat = o;   o = a256(o + (int64_t)nj * 4);
  const int64_t off_gst = o;    o = a256(o + 72);
  std::vector<int64_t> job_out(nj);
  for (int i = 0; i < nj; ++i) {
    job_out[i] = o;
    o += sz[i].out;
  }
  const int64_t out_bytes = o - off_out;
  // device only
  const int64_t off_qjob = o;  o = a256(o + tiles * 4);
  const int64_t off_qtile = o; o = a256(o + tiles * 4);
  const int64_t off_flags = o; o = a256(o + tiles * 4);
  const int64_t off_s4q = o;   o = a256(o + blocks4 * 8);
  std::vector<int64_t> job_big(nj);
  for (int i = 0; i < nj; ++i) {
    job_big[i] = o;
    o += sz[i].big;
  }
  // The exchange regions of the streaming jobs lie at the arena's end, so that
  // from launch to launch most of them hold words of earlier launches, whose
  // tags are not this launch's.  [x_clean_, cap) holds nothing else; what lies
  // before it, and everything once the tags start again, is cleared.
  const int64_t xlo = (cap_ - x4) / 256 * 256;
  if (o > xlo) return MSA_ENOMEM;
  int rc = ensure_host(in_bytes, out_bytes);
  if (rc) return rc;
  if (x_clean_ < o) x_clean_ = o;
  const int s4tag = sweep_tag(sweeps_, kSweepTags);
  int64_t xzero = 0;
  if (n4 > 0) {
    if (s4tag == 1) x_clean_ = cap_ / 256 * 256;
    xzero = std::max<int64_t>(0, x_clean_ - xlo);
    x_clean_ = std::min(x_clean_, xlo);
    sweeps_ = next_sweep(sweeps_, 1);
  }

  // ---- host image of the input region ----
  char *h = h_in_;
  memset(h, 0, (size_t)in_bytes);
  Ctrl ctrl;
  memset(&ctrl, 0, sizeof(ctrl));
  ctrl.epoch = 1;
  ctrl.wd[0] = -1;  // no job
  // A batched dependency wait is bounded by one job's tile chain (a few ms
  // even for large jobs), so a launch gives up after 250 ms instead of the
  // plain fill's 2 s: a launch that times out is re-run sooner.
  ctrl.wait_limit = wait_limit_ > 0 ? wait_limit_ : kBatchWaitTicks;
  memcpy(h + off_ctrl, &ctrl, sizeof(ctrl));
  for (auto &kv : subs)
    memcpy(h + kv.second, kv.first.data(), kv.first.size() - 1);
  int64_t *jt = reinterpret_cast<int64_t *>(h + off_jt);
  int64_t *jc = reinterpret_cast<int64_t *>(h + off_jc);  // columns before job i
  jt[0] = 0;
  jc[0] = 0;
  meta_.assign(nj, Meta());
  std::vector<const int32_t *> wave_cnt(nj);
  std::vector<int64_t *> wave_base(nj);
  JobDev *jd_all = reinterpret_cast<JobDev *>(h + off_jobs);
  Sweep4Dev *s4_all = reinterpret_cast<Sweep4Dev *>(h + off_s4jobs);
  Sweep5Dev *s5_all = reinterpret_cast<Sweep5Dev *>(h + off_s4jobs);
  int32_t *s4pre = reinterpret_cast<int32_t *>(h + off_s4pre);
  // Walkers take the walks of all jobs, or of none: where there are few jobs each
  // has a compute unit, and a short walk is done before the longest (64 jobs of
  // k = 2 and 100..300 residues 38 us; the shorter half by the single wave's
  // kernel, after the walkers', 78).
  const int cus = device_cu_count();
  bool walkers = false;
  for (int i = 0; i < nj; ++i)
    walkers = walkers || trace_by_walkers(jobs[i]->lens, jobs[i]->k, nj, cus);
  std::vector<int32_t *> s4base;        // queue slots per key, of each streaming job
  std::vector<const JobSizes *> s4size;
  int64_t xo = xlo;
  for (int i = 0; i < nj; ++i) {
    const msa_job &j = *jobs[i];
    const Plan &p = sz[i].p;
    const bool s4 = sz[i].s4;
    jt[i + 1] = jt[i] + (s4 ? 0 : p.ntiles);
    jc[i + 1] = jc[i] + (s4 ? 0 : p.ncols);
    JobDev jd;
    fill_jobdev(p, nullptr, j.alpha, j.gap, &jd);
    // small region of this job
    int64_t so = job_small[i];
    char *hs_base = h + so;
    int64_t pos = 0;
    for (int d = 0; d < j.k; ++d) {
      if (j.lens[d] > 0) memcpy(hs_base + pos, j.seqs[d], (size_t)j.lens[d]);
      pos += j.lens[d];
    }
    const int64_t o_seq = so;
    so += a256(std::max<int64_t>(p.total_len, 1));
    const int64_t o_wcnt = so;
    int64_t o_wst = so;
    const int nw = p.nwaves;
    if (s4) {
      s4base.push_back(reinterpret_cast<int32_t *>(h + so));
      s4size.push_back(&sz[i]);
      so += a256((int64_t)sz[i].keys.size() * 4);
    } else {
      int32_t *wc = reinterpret_cast<int32_t *>(h + so);
      // wc[d][s]: coordinate tuples (c_d..c_{k-1}) with sum s
      for (int s = 0; s < nw; ++s) wc[j.k * nw + s] = (s == 0);
      for (int d = j.k - 1; d >= 0; --d)
        for (int s = 0; s < nw; ++s) {
          int64_t acc = 0;
          for (int c = 0; c < p.P[d] && c <= s; ++c) acc += wc[(d + 1) * nw + (s - c)];
          wc[d * nw + s] = (int32_t)acc;
        }
      so += a256((int64_t)(j.k + 1) * nw * 4);
      o_wst = so;
      wave_cnt[i] = wc + nw;  // row 1: columns by the wave of their first tile
      wave_base[i] = reinterpret_cast<int64_t *>(h + so);
      so += a256((int64_t)nw * 8);
    }
    const int64_t o_jst = so;
    // device pointers
    jd.seqs = reinterpret_cast<const uint8_t *>(d_ + o_seq);
    jd.sub = reinterpret_cast<const int8_t *>(d_ + sub_off[i]);
    jd.wcnt = reinterpret_cast<const int32_t *>(d_ + o_wcnt);
    jd.wbase = reinterpret_cast<const int64_t *>(d_ + o_wst);
    jd.jstatus = reinterpret_cast<int32_t *>(d_ + o_jst);
    jd.qbase = jt[i];
    jd.flags = reinterpret_cast<int32_t *>(d_ + off_flags) + jt[i];
    int64_t bo = job_big[i];
    jd.path = reinterpret_cast<uint8_t *>(d_ + bo);
    bo += a256(std::max<int64_t>(p.total_len, 1));
    jd.faces = s4 ? nullptr : reinterpret_cast<int32_t *>(d_ + bo);
    if (!s4) bo += a256(std::max<int64_t>(p.face_elems * 4, 256));
    jd.dir = reinterpret_cast<uint8_t *>(d_ + bo);
    jd.score_out = reinterpret_cast<int64_t *>(d_ + off_score) + i;
    jd.aln_len_out = reinterpret_cast<int64_t *>(d_ + off_len) + i;
    jd.status_out = reinterpret_cast<int32_t *>(d_ + off_stat) + i;
    jd.aln_out = reinterpret_cast<uint8_t *>(d_ + job_out[i]);
    jd.aln_cap = sz[i].cap;
    jd.walkers = walkers && j.k <= kTrMaxK && p.total_len <= kTrMaxTotal;
    jd.trace = nullptr;
    memcpy(&jd_all[i], &jd, sizeof(JobDev));
    if (s4) {
      const int n = (int)s4base.size() - 1;
      int32_t *const x = reinterpret_cast<int32_t *>(d_ + xo);
      int32_t *const kb = reinterpret_cast<int32_t *>(d_ + o_wcnt);
      xo += sz[i].x;
      auto fill = [&](auto &sd) {
        sd.alpha = j.alpha;
        sd.gap = j.gap;
        sd.seqs = jd.seqs;
        sd.sub = jd.sub;
        sd.dir = jd.dir;
        sd.score_out = jd.score_out;
        sd.status = jd.jstatus;
        sd.kbase = kb;
      };
      if (kc == 1) {
        Sweep5Dev sd;
        fill_sweep5dev(p, &sd);
        fill(sd);
        sd.x = x + kS5PadFront;
        memcpy(&s5_all[n], &sd, sizeof(sd));
      } else {
        Sweep4Dev sd;
        fill_sweep4dev(p, &sd);
        fill(sd);
        sd.x0 = x + kS4PadFront;
        sd.x1 = sd.x0 + p.s4_x0;
        sd.x2 = sd.x1 + p.s4_x1;
        memcpy(&s4_all[n], &sd, sizeof(sd));
      }
      if (n == 0) s4pre[0] = 0;
      s4pre[n + 1] = s4pre[n] + (int32_t)sz[i].blocks();
    }
    meta_[i].k = j.k;
    meta_[i].cap = sz[i].cap;
    meta_[i].aln_off = job_out[i] - off_out;
    meta_[i].qbase = s4 ? -1 - (int64_t)s4base.size() : jt[i];  // (-2 - n of streaming job n)
  }

  // The queue holds tile columns along dimension 0 (a workgroup computes a
  // column bottom up, as in the plain fill) in wave-major order across jobs:
  // every job's columns starting in wave 0, then every job's columns starting
  // in wave 1, ...  The persistent workgroups so work on all jobs' wavefronts
  // at once instead of waiting on one job's dependency chain at a time; a
  // column depends only on columns of its job that start in earlier waves,
  // so the order is topological.
  {
    int wmax = 0;
    for (int i = 0; i < nj; ++i)
      if (!sz[i].s4) wmax = std::max(wmax, sz[i].p.nwaves);
    std::vector<int64_t> slot(wmax, 0);  // next free slot of wave w
    std::vector<int64_t> tot(wmax, 0);
    for (int i = 0; i < nj; ++i)
      for (int w = 0; !sz[i].s4 && w < sz[i].p.nwaves; ++w) tot[w] += wave_cnt[i][w];
    int64_t acc = 0;
    for (int w = 0; w < wmax; ++w) {
      slot[w] = acc;
      acc += tot[w];
    }
    for (int i = 0; i < nj; ++i)
      for (int w = 0; !sz[i].s4 && w < sz[i].p.nwaves; ++w) {
        wave_base[i][w] = slot[w];
        slot[w] += wave_cnt[i][w];
      }
  }

  // The queue of the streaming jobs' blocks: all jobs' blocks in descending
  // order of the steps their job still needs after them (about five per key,
  // and a block's own), so that the longest chains start first and no job is
  // left to run alone at the end; within a job the keys ascend.
  {
    auto bin = [&](int n, int key) {
      return (int)s4size[n]->keys.size() - 1 - key + s4size[n]->steps() / 5;
    };
    int top = -1;
    for (int n = 0; n < n4; ++n) top = std::max(top, bin(n, 0));
    std::vector<int32_t> slot(top + 2, 0);  // next free slot of a bin
    for (int n = 0; n < n4; ++n)
      for (int key = 0; key < (int)s4size[n]->keys.size(); ++key)
        slot[bin(n, key)] += s4size[n]->keys[key];
    int32_t acc = 0;
    for (int b = top; b >= 0; --b) {
      const int32_t c = slot[b];
      slot[b] = acc;
      acc += c;
    }
    for (int n = 0; n < n4; ++n)
      for (int key = 0; key < (int)s4size[n]->keys.size(); ++key) {
        s4base[n][key] = slot[bin(n, key)];
        slot[bin(n, key)] += s4size[n]->keys[key];
      }
  }

  // ---- batch descriptor (read by the launch sequence) ----
  BatchArgs args;
  memset(&args, 0, sizeof(args));
  args.jcols = reinterpret_cast<const int64_t *>(d_ + off_jc);
  args.qjob = reinterpret_cast<int32_t *>(d_ + off_qjob);
  args.qtile = reinterpret_cast<int32_t *>(d_ + off_qtile);
  args.flags = reinterpret_cast<int32_t *>(d_ + off_flags);
  args.gstatus = reinterpret_cast<int32_t *>(d_ + off_gst);
  args.tiles = tiles;
  args.cols = jc[nj];
  args.njobs = nj;
  args.s4n = n4;
  args.s4jobs = reinterpret_cast<const Sweep4Dev *>(d_ + off_s4jobs);
  args.s5jobs = reinterpret_cast<const Sweep5Dev *>(d_ + off_s4jobs);
  args.s4pre = reinterpret_cast<const int32_t *>(d_ + off_s4pre);
  args.s4q = reinterpret_cast<int32_t *>(d_ + off_s4q);
  args.s4total = (int32_t)blocks4;
  args.s4tag = s4tag;
  args.xzero = d_ + xlo;
  args.xzero16 = xzero / 16;
  memcpy(h + off_args, &args, sizeof(args));

  // ---- enqueue: inputs, the launch sequence (a graph replay), outputs ----
  const int grid = batch_grid(kc);
  int parts = (tiles > 0 ? kBatchTiles : 0) | (n4 > 0 ? kBatchStreams : 0);
  for (int i = 0; i < nj; ++i) parts |= jd_all[i].walkers ? kBatchWalkers : kBatchSingle;
  const bool graph = ensure_graph(kc, parts, grid) == 0;
  bool ok = true;
  for (hipEvent_t e : after) ok = ok && hipStreamWaitEvent(stream_, e, 0) == hipSuccess;
  ok = ok && hipEventRecord(start_, stream_) == hipSuccess;
  ok = ok && hipMemcpyAsync(d_, h, (size_t)in_bytes, hipMemcpyHostToDevice, stream_) == hipSuccess;
  if (graph)
    ok = ok && hipGraphLaunch(graph_[kc][parts].exec, stream_) == hipSuccess;
  else
    ok = ok && launch_batch(kc, parts, reinterpret_cast<const BatchArgs *>(d_ + off_args),
                            reinterpret_cast<const JobDev *>(d_ + off_jobs),
                            reinterpret_cast<Ctrl *>(d_ + off_ctrl), grid, stream_) == 0;
  ok = ok && hipMemcpyAsync(h_out_, d_ + off_out, (size_t)out_bytes, hipMemcpyDeviceToHost,
                            stream_) == hipSuccess;
  ok = ok && hipEventRecord(done_, stream_) == hipSuccess;
  out_bytes_ = out_bytes;
  out_off_ = off_out;
  (void)off_score;
  busy_ = true;
  launch_status_ = ok ? MSA_OK : MSA_EDEVICE;
  if (!ok) x_clean_ = cap_;  // the clearing may not have run
  return launch_status_;
}

bool Launch::ready() {
  if (!busy_) return true;
  return hipEventQuery(done_) != hipErrorNotReady;
}

int Launch::wait() {
  if (!busy_) return MSA_OK;
  if (hipEventSynchronize(done_) != hipSuccess) launch_status_ = MSA_EDEVICE;
  return launch_status_;
}

bool Launch::interval_ms(hipEvent_t ref, float *t0, float *t1) const {
  return hipEventElapsedTime(t0, ref, start_) == hipSuccess &&
         hipEventElapsedTime(t1, ref, done_) == hipSuccess;
}

int32_t Launch::device_status() const {
  const int nj = (int)meta_.size();
  const int64_t off_gst = 2 * a256((int64_t)nj * 8) + a256((int64_t)nj * 4);
  return *reinterpret_cast<const int32_t *>(h_out_ + off_gst);
}

int64_t Launch::device_max_pause_us() const {
  const int nj = (int)meta_.size();
  const int64_t off_gst = 2 * a256((int64_t)nj * 8) + a256((int64_t)nj * 4);
  return *reinterpret_cast<const int64_t *>(h_out_ + off_gst + 8) / 100;  // 100 MHz ticks
}

bool Launch::device_timeout(int *job, int64_t *tile, int64_t *missing, int64_t more[4]) const {
  const int nj = (int)meta_.size();
  const int64_t off_gst = 2 * a256((int64_t)nj * 8) + a256((int64_t)nj * 4);
  const int64_t *w = reinterpret_cast<const int64_t *>(h_out_ + off_gst + 16);
  if (device_status() == MSA_OK) return false;
  *job = -1;
  for (int i = 0; i < nj; ++i)
    if (meta_[i].qbase == w[0]) *job = i;
  *tile = w[1];
  *missing = w[2];
  if (more)
    for (int q = 0; q < 4; ++q) more[q] = w[3 + q];
  return true;
}

void Launch::result(int i, LaunchResult *out) const {
  const int nj = (int)meta_.size();
  const int64_t off_len = a256((int64_t)nj * 8);
  const int64_t off_stat = off_len + a256((int64_t)nj * 8);
  const int64_t *scores = reinterpret_cast<const int64_t *>(h_out_);
  const int64_t *lens = reinterpret_cast<const int64_t *>(h_out_ + off_len);
  const int32_t *stats = reinterpret_cast<const int32_t *>(h_out_ + off_stat);
  out->k = meta_[i].k;
  out->cap = meta_[i].cap;
  out->status = launch_status_ != MSA_OK ? launch_status_ : stats[i];
  out->score = out->status == MSA_OK ? scores[i] : 0;
  out->aln_len = out->status == MSA_OK ? lens[i] : 0;
  const uint8_t *rows = reinterpret_cast<const uint8_t *>(h_out_ + meta_[i].aln_off);
  out->aln.assign(rows, rows + (size_t)meta_[i].k * meta_[i].cap);
}

void Launch::fill_result(int i, msa_result *out) const {
  const int nj = (int)meta_.size();
  const int64_t off_len = a256((int64_t)nj * 8);
  const int64_t off_stat = off_len + a256((int64_t)nj * 8);
  const int64_t *scores = reinterpret_cast<const int64_t *>(h_out_);
  const int64_t *lens = reinterpret_cast<const int64_t *>(h_out_ + off_len);
  const int32_t *stats = reinterpret_cast<const int32_t *>(h_out_ + off_stat);
  const int st = launch_status_ != MSA_OK ? launch_status_ : stats[i];
  out->status = st;
  out->score = st == MSA_OK ? scores[i] : 0;
  out->aln_len = st == MSA_OK ? lens[i] : 0;
  if (st == MSA_OK && out->aln && out->aln_len > 0) {
    const uint8_t *rows = reinterpret_cast<const uint8_t *>(h_out_ + meta_[i].aln_off);
    for (int r = 0; r < meta_[i].k; ++r)
      memcpy(out->aln + (int64_t)r * out->aln_cap, rows + (int64_t)r * meta_[i].cap,
             (size_t)out->aln_len);
  }
}

}  // namespace msa
