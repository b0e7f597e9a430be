"""The alignments that a user of this library runs, as a list of cases.

A case is one call path of the Python binding with its sizes:

  plain, egf, coopt, nearopt, prune
      one device-resident alignment of a prepared shape (DeviceAligner), in
      the mode of that name; sequences already on the GPU, outputs left there
  host    one msa.align call: host sequences in, host rows out
  batch   one msa.align_batch call on many independent jobs
  served  jobs handed to a running msa.Server, then waited for

Sizes follow the library's own workloads: three DNA sequences of 40 residues,
three protein sequences of 512, four of 128, five of 40, batches of k = 3, 4
with lengths 16..160 (DNA and protein half and half), and a served mix of
k = 3, 4, 5 (0.6/0.3/0.1) with lengths 16..256, 16..96 and 12..40.

Protein sequences are descendants of one random ancestor (20% substitutions,
5% single-residue indels); DNA sequences are unrelated.  Scores are sums of
pairs, DNA +2/-1 with gap -2, protein a symmetric 20 x 20 matrix (diagonal
4..11, off-diagonal -4..3) with gap -8.
"""
import numpy as np
import torch

import paper_2311_17530_amd as msa

BUDGET = 8 << 30        # device memory for a batch's or the server's jobs
PATHS = 16              # alignments listed in the co-optimal and near-optimal modes
DELTA = 20              # near-optimal margin


def _lens(*n):
    return {"k": len(n), **{"n%d" % i: int(x) for i, x in enumerate(n)}}


def listed():
    return [
        # the smallest call: latency of one short DNA alignment
        {"name": "k3_dna_40", "mode": "plain", "dna": True, **_lens(40, 40, 40)},
        # an ordinary alignment of three protein domains of unequal length
        {"name": "k3_ragged", "mode": "plain", "dna": False, **_lens(157, 93, 201)},
        # the headline workload: three whole proteins
        {"name": "k3_prot_512", "mode": "plain", "dna": False, **_lens(512, 512, 512)},
        # four sequences, the largest single tensor (129^4 cells)
        {"name": "k4_prot_128", "mode": "plain", "dna": False, **_lens(128, 128, 128, 128)},
        # five short sequences, the largest k of the served mix
        {"name": "k5_prot_40", "mode": "plain", "dna": False, **_lens(40, 40, 40, 40, 40)},
        # overlap alignment of three fragments: unaligned ends are free
        {"name": "k3_egf_ragged", "mode": "egf", "dna": False, **_lens(401, 365, 512)},
        # how unique is the optimum: the first 16 co-optimal alignments
        {"name": "k3_coopt_512", "mode": "coopt", "dna": False, **_lens(512, 512, 512)},
        # alternatives close to the optimum: the first 16 within 20 of it
        {"name": "k3_nearopt_ragged", "mode": "nearopt", "dna": False, **_lens(300, 257, 281)},
        # four related sequences with exact pruning of the search space
        {"name": "k4_prune_128", "mode": "prune", "dna": False, **_lens(128, 128, 128, 128)},
        # one call with host buffers, nothing prepared: the simplest entry point
        {"name": "k4_host_ragged", "mode": "host", "dna": False, **_lens(45, 33, 61, 38)},
        # many independent jobs of uneven k and length at once
        {"name": "batch_256", "mode": "batch", "jobs": 256},
        # requests to a running server, every result awaited
        {"name": "served_256", "mode": "served", "jobs": 256},
    ]


def draw(rng):
    def length(lo, hi):  # even over the logarithm of the range
        return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))

    mode = rng.choice(["plain", "plain", "plain", "plain", "egf", "coopt", "nearopt", "prune",
                       "host", "batch", "served"])
    if mode in ("batch", "served"):
        return {"mode": mode, "jobs": length(16, 256)}
    k = {"egf": [3, 4], "coopt": [3], "nearopt": [3], "prune": [3, 4, 5]}.get(mode, [3, 4, 5])
    k = rng.choice(k)
    lo, hi = {3: (16, 512), 4: (16, 128), 5: (12, 40)}[k]
    if mode == "host":
        hi = {3: 256, 4: 96, 5: 32}[k]
    if mode == "nearopt":
        hi = 400
    # pruning pays for related sequences only, the protein recipe
    dna = mode not in ("prune", "nearopt") and rng.random() < 0.4
    top = length(lo, hi)
    return {"mode": mode, "dna": dna,
            **_lens(*[length(max(lo, top // 3), top) for _ in range(k)])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _scoring(dna):
    if dna:
        sub = np.full((4, 4), -1, np.int8)
        np.fill_diagonal(sub, 2)
        return sub, -2
    r = np.random.default_rng(17)
    m = np.triu(r.integers(-4, 4, (20, 20)), 1)
    return (m + m.T + np.diag(r.integers(4, 12, 20))).astype(np.int8), -8


def _descendant(r, anc):
    """20% substitutions, then 5% single-residue indels (half and half)."""
    n = len(anc)
    s = anc.copy()
    at = r.choice(n, int(round(0.2 * n)), replace=False)
    s[at] = (s[at] + r.integers(1, 20, len(at))) % 20
    ev = int(round(0.025 * n))
    if ev:
        s = np.delete(s, r.choice(n, ev, replace=False))
        s = np.insert(s, r.integers(0, len(s) + 1, ev), r.integers(0, 20, ev))
    return s.astype(np.uint8)


def _sequences(r, lens, dna):
    if dna:
        return [r.integers(0, 4, n).astype(np.uint8) for n in lens]
    anc = r.integers(0, 20, max(lens))
    return [np.ascontiguousarray(_descendant(r, anc)[:n]) for n in lens]


def _case_lens(case):
    return [case["n%d" % i] for i in range(case["k"])]


def _jobs(case, seed):
    """Jobs of a batch or of the served mix; their sizes come from the job
    count alone, so that every seed of a case is the same work."""
    shape = np.random.default_rng([4, case["jobs"], case["mode"] == "served"])
    r = np.random.default_rng([seed, case["jobs"]])
    out = []
    for _ in range(case["jobs"]):
        if case["mode"] == "batch":
            k, lo, hi, dna = int(shape.integers(3, 5)), 16, 160, bool(shape.integers(0, 2))
        else:
            k, dna = int(shape.choice([3, 4, 5], p=[0.6, 0.3, 0.1])), False
            lo, hi = {3: (16, 256), 4: (16, 96), 5: (12, 40)}[k]
        lens = [int(x) for x in shape.integers(lo, hi + 1, k)]
        out.append((_sequences(r, lens, dna), *_scoring(dna)))
    return out


_server = None


def _the_server():
    """A program keeps one server for all its requests."""
    global _server
    if _server is None:
        _server = msa.Server(hbm_budget_bytes=BUDGET)
    return _server


def prepare(case, seed):
    mode = case["mode"]
    if mode in ("batch", "served"):
        jobs = _jobs(case, seed)
        return {"mode": mode, "jobs": jobs, "caps": [sum(map(len, j[0])) for j in jobs],
                "server": _the_server() if mode == "served" else None}
    lens = _case_lens(case)
    seqs = _sequences(np.random.default_rng([seed, *lens]), lens, case["dna"])
    sub, gap = _scoring(case["dna"])
    if mode == "host":
        return {"mode": mode, "seqs": seqs, "sub": sub, "gap": gap, "caps": [sum(lens)]}
    dev = msa.DeviceAligner(lens, sub, gap, end_gaps_free=mode == "egf",
                            cooptimal=mode == "coopt", nearopt=mode == "nearopt",
                            prune=mode == "prune")
    dev.set_sequences(seqs)
    return {"mode": mode, "dev": dev}


def _collect(results, caps):
    """(status, score, rows) per job as arrays; the rows of all jobs side by
    side, each job in columns of its own as long as its alignment can be."""
    rows = np.full((max(len(r[2]) for r in results), sum(caps)), 0xFF, np.uint8)
    at = 0
    for (_, _, a), cap in zip(results, caps):
        rows[:len(a), at:at + a.shape[1]] = a
        at += cap
    return {"status": np.array([r[0] for r in results], np.int32),
            "score": np.array([r[1] for r in results], np.int64),
            "len": np.array([r[2].shape[1] for r in results], np.int64), "rows": rows}


def run(state):
    mode = state["mode"]
    if mode == "host":
        score, rows = msa.align(state["seqs"], state["sub"], state["gap"])
        return _collect([(msa.MSA_OK, score, rows)], state["caps"])
    if mode == "batch":
        return _collect(msa.align_batch(state["jobs"], hbm_budget_bytes=BUDGET), state["caps"])
    if mode == "served":
        srv = state["server"]
        tickets = [srv.submit(*job) for job in state["jobs"]]
        return _collect([srv.wait(t) for t in tickets], state["caps"])
    dev = state["dev"]
    if mode == "coopt":
        dev.run_coopt(PATHS)
        return {"status": dev.d_status, "score": dev.d_score, "paths": dev.d_co_np,
                "len": dev.d_co_len, "rows": dev.d_co_aln}
    if mode == "nearopt":
        dev.run_nearopt(DELTA, PATHS)
        return {"status": dev.d_status, "score": dev.d_score, "paths": dev.d_no_np,
                "scores": dev.d_no_sc, "len": dev.d_no_len, "rows": dev.d_no_aln}
    dev.run()
    return {"status": dev.d_status, "score": dev.d_score, "len": dev.d_len, "rows": dev.d_aln}


# ---------------------------------------------------------------------------
# work and exact values
# ---------------------------------------------------------------------------
def _updates(lens):
    """Pairs of a cell and a lower neighbour inside the tensor."""
    a = c = 1
    for n in lens:
        a *= 2 * n + 1
        c *= n + 1
    return a - c


def work(case):
    """Sequences in, rows and scores out; one add and one maximum per
    neighbour update (of every cell, also where a mode may skip some)."""
    if case["mode"] in ("batch", "served"):
        jobs = [[len(s) for s in seqs] for seqs, _, _ in _jobs(case, 0)]
        paths = 1
    else:
        jobs = [_case_lens(case)]
        paths = PATHS if case["mode"] in ("coopt", "nearopt") else 1
    return {"bytes": sum(sum(l) + paths * (len(l) * sum(l) + 16) + 12 for l in jobs),
            "flops": sum(2 * _updates(l) for l in jobs)}


def _columns(seqs, sub, gap, cell):
    """Sum-of-pairs score of each mask's column at a cell (index = mask)."""
    k = len(seqs)
    res = [int(seqs[i][cell[i] - 1]) if cell[i] > 0 else 0 for i in range(k)]
    out = [0] * (1 << k)
    for b in range(1, 1 << k):
        for i in range(k):
            for j in range(i + 1, k):
                bi, bj = b >> i & 1, b >> j & 1
                out[b] += int(sub[res[i], res[j]]) if bi and bj else gap if bi or bj else 0
    return out


def _tensor(seqs, sub, gap, egf):
    """Every cell's score in 64 bits, hyperplane by hyperplane, in an array
    with one layer of minus infinity before each dimension."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    k = len(seqs)
    ext = [len(s) + 2 for s in seqs]
    stride = [int(np.prod(ext[i + 1:], dtype=np.int64)) for i in range(k)]
    low = -(1 << 40)
    S = torch.full((int(np.prod(ext, dtype=np.int64)),), low, dtype=torch.int64, device=dev)
    # cells in order of their coordinate sum
    sums = torch.zeros((1,) * k, dtype=torch.int16, device=dev)
    lin = torch.zeros((1,) * k, dtype=torch.int64, device=dev)
    for i in range(k):
        v = torch.arange(ext[i] - 1, device=dev).view([-1 if d == i else 1 for d in range(k)])
        sums = sums + v.to(torch.int16)
        lin = lin + (v + 1) * stride[i]
    order = torch.argsort(sums.reshape(-1))
    cells = lin.reshape(-1)[order]
    count = torch.bincount(sums.reshape(-1).to(torch.int32)).cpu().tolist()
    del sums, lin, order
    subt = torch.from_numpy(sub.astype(np.int64)).to(dev)
    codes = [torch.cat([torch.zeros(2, dtype=torch.int64),
                        torch.from_numpy(s.astype(np.int64))]).to(dev) for s in seqs]
    at = 0
    for n in count:
        idx = cells[at:at + n]
        at += n
        u = [idx // stride[i] % ext[i] for i in range(k)]  # v + 1
        res = [codes[i][u[i]] for i in range(k)]
        pair = {(i, j): subt[res[i], res[j]] for i in range(k) for j in range(i + 1, k)}
        best = torch.full_like(idx, low)
        for b in range(1, 1 << k):
            bits = [i for i in range(k) if b >> i & 1]
            c = S[idx - sum(stride[i] for i in bits)] + gap * len(bits) * (k - len(bits))
            for p, i in enumerate(bits):
                for j in bits[p + 1:]:
                    c = c + pair[i, j]
            best = torch.maximum(best, c)
        if egf:
            zero = torch.zeros_like(idx, dtype=torch.bool)
            for i in range(k):
                zero |= u[i] == 1
            best = torch.where(zero, 0, best)
        elif at == n:
            best = torch.zeros_like(best)  # the origin
        S[idx] = best
    return S.view(ext).cpu().numpy()


def _rows(seqs, masks, cap):
    """Gapped rows of a path of masks given first column first."""
    out = np.full((len(seqs), cap), 0xFF, np.uint8)
    for i, s in enumerate(seqs):
        cols = [c for c, b in enumerate(masks) if b >> i & 1]
        out[i, cols] = s
    return out


def exact(case, seed):
    if case["mode"] in ("batch", "served"):
        return None
    mode, lens = case["mode"], _case_lens(case)
    seqs = _sequences(np.random.default_rng([seed, *lens]), lens, case["dna"])
    sub, gap = _scoring(case["dna"])
    k, cap = len(lens), sum(lens)
    S = _tensor(seqs, sub, gap, mode == "egf")
    if mode == "egf":
        inner = S[(slice(1, None),) * k]
        far = np.full(inner.shape, np.iinfo(np.int64).min)
        for i in range(k):
            f = (slice(None),) * i + (-1,)
            far[f] = inner[f]
        last = far.size - 1 - int(np.argmax(far.reshape(-1)[::-1]))
        end = [int(x) for x in np.unravel_index(last, far.shape)]
    else:
        end = list(lens)
    score = int(S[tuple(x + 1 for x in end)])
    most = PATHS if mode in ("coopt", "nearopt") else 1
    bound = score - (DELTA if mode == "nearopt" else 0)
    # depth first from the end cell, masks in ascending order
    found, path, so_far, cell, options = [], [], [0], list(end), []

    def choices():
        col = _columns(seqs, sub, gap, cell)
        return [(b, col[b]) for b in range(1, 1 << k)
                if S[tuple(x + 1 - (b >> i & 1) for i, x in enumerate(cell))] + col[b]
                + so_far[-1] >= bound]

    while len(found) < most:
        if not (any(x == 0 for x in cell) if mode == "egf" else not any(cell)):
            options.append(choices())
        else:
            found.append((so_far[-1], path[::-1], list(cell)))
            while options and not options[-1]:
                options.pop()
                b = path.pop()
                so_far.pop()
                cell = [x + (b >> i & 1) for i, x in enumerate(cell)]
            if not options:
                break
            b = path.pop()
            so_far.pop()
            cell = [x + (b >> i & 1) for i, x in enumerate(cell)]
        b, c = options[-1].pop(0)
        path.append(b)
        so_far.append(so_far[-1] + c)
        cell = [x - (b >> i & 1) for i, x in enumerate(cell)]
        # (options[-1] now holds the masks left at the cell before this step)
    full = []
    for sc, masks, start in found:
        if mode == "egf":  # unaligned prefixes and suffixes, sequence 0 first
            masks = ([1 << i for i in range(k) for _ in range(start[i])] + masks +
                     [1 << i for i in range(k) for _ in range(lens[i] - end[i])])
        full.append((sc, masks))
    if mode in ("coopt", "nearopt"):
        pad = [0] * (PATHS - len(full))
        rows = np.full((PATHS, k, cap), 0xFF, np.uint8)
        for p, (_, masks) in enumerate(full):
            rows[p] = _rows(seqs, masks, cap)
        out = {"status": np.zeros(1, np.int32), "score": np.array([score]),
               "paths": np.array([len(full)], np.int32),
               "len": np.array([len(m) for _, m in full] + pad), "rows": rows}
        if mode == "nearopt":
            out["scores"] = np.array([s for s, _ in full] + pad)
        return out
    masks = full[0][1]
    return {"status": np.zeros(1, np.int32), "score": np.array([score]),
            "len": np.array([len(masks)]), "rows": _rows(seqs, masks, cap)}
