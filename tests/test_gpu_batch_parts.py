"""A batched launch runs only the kernels that its jobs need: every combination
of jobs for the tile fill and for the streaming fills, of tracebacks by
several walkers and by a single wave, in batches that follow each other on
one arena (their launch sequences are captured and replayed) and through a
server.  Results equal the oracle's."""
import sys

import numpy as np
import pytest

import paper_2311_17530_amd as msa
from msa_inputs import dna_scoring, protein_scoring
from oracle import oracle_align

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    msa.lib()
    msa.tune_clear()


# tile fill (k = 2, 3), short and long walks, and past the walkers' bound
T_SHORT, T_LONG, T_FAR = [20, 14, 9], [130, 120], [8190, 2]
# streaming fill (k = 4), and tile fill (fourth length past its bound)
S_SHORT, S_LONG, S_FAR = [9, 12, 7, 10], [100, 8, 9, 11], [8189, 1, 1, 1]
F_SHORT = [1, 2, 0, 2049]
# k = 5: streaming, past the walkers' bound, tile fill
S5, S5_FAR, T5 = [6, 5, 7, 4, 9], [8192, 0, 0, 0, 1], [2, 1, 3, 0, 129]
# k = 6 and 7: tile fill and single wave alone
T6, T7 = [3, 4, 2, 5, 3, 2], [2, 1, 2, 2, 1, 2, 1]

BATCHES = [
    [T_SHORT], [T_LONG], [T_FAR], [S_SHORT], [S_LONG], [S_FAR], [S5], [S5_FAR], [T5], [T6], [T7],
    [T_SHORT, T_LONG], [T_SHORT, T_FAR], [S_SHORT, S_LONG, S_FAR], [T_SHORT, S_SHORT],
    [F_SHORT], [F_SHORT, S_SHORT], [T_LONG, S_LONG, T_FAR, S_FAR], [S5, T5], [S5, S5_FAR, T5],
    [T_SHORT, S_SHORT, S5, T6, T7], [T_SHORT] * 3, [S_SHORT] * 3,
]


def jobs_of(shapes, seed):
    out = []
    for i, lens in enumerate(shapes):
        rng = np.random.Generator(np.random.PCG64([seed, i, *lens]))
        sub, gap = dna_scoring() if (i + seed) % 2 else protein_scoring()
        if max(lens) > 1000:
            sub, gap = dna_scoring()
        out.append(([rng.integers(0, sub.shape[0], n).astype(np.uint8) for n in lens], sub, gap))
    return out


def check(jobs, results):
    for (seqs, sub, gap), (st, s1, r1) in zip(jobs, results):
        s0, r0 = oracle_align(seqs, sub, gap)[:2]
        assert st == msa.MSA_OK and s1 == s0 and np.array_equal(r1, r0), [len(s) for s in seqs]


@pytest.mark.parametrize("rnd", range(2))
def test_batches_of_every_composition(rnd):
    for b, shapes in enumerate(BATCHES):
        say("batch", b, shapes)
        jobs = jobs_of(shapes, 10 * rnd + b)
        check(jobs, msa.align_batch(jobs, hbm_budget_bytes=1 << 30))


def test_server_launches_of_every_composition():
    with msa.Server(hbm_budget_bytes=1 << 30, max_inflight=2) as srv:
        for b, shapes in enumerate(BATCHES):
            say("served", b, shapes)
            jobs = jobs_of(shapes, 100 + b)
            tickets = [srv.submit(*j) for j in jobs]
            check(jobs, [srv.wait(t, 30_000_000) for t in tickets])


@pytest.mark.parametrize("k,njobs", [(3, 128), (3, 129), (5, 256), (5, 257)])
def test_traceback_of_few_and_of_many_jobs(k, njobs):
    """Both sides of the number of jobs up to which walkers take the tracebacks
    (half the compute units, k = 5: as many), walks of every length among them."""
    rng = np.random.Generator(np.random.PCG64(70 + njobs))
    sub, gap = protein_scoring()
    shapes = [[int(x) for x in rng.integers(0, 9, k)] for _ in range(njobs)]
    for i in range(0, njobs, 9):
        shapes[i] = [100, 97, 12][:k] + [3] * (k - 3) if k == 3 else [9, 12, 8, 11, 10]
    jobs = [([rng.integers(0, 20, n).astype(np.uint8) for n in lens], sub, gap) for lens in shapes]
    say("batch of", njobs, "jobs, k =", k)
    check(jobs, msa.align_batch(jobs, hbm_budget_bytes=4 << 30))


def test_threads_capture_sequences_beside_each_other():
    """Three threads, each with an arena of its own, meet every composition for
    the first time while the others and a server run theirs."""
    import threading
    errors = []

    def work(n):
        try:
            for b, shapes in enumerate(BATCHES[n:] + BATCHES[:n]):
                jobs = jobs_of(shapes, 200 + 30 * n + b)
                check(jobs, msa.align_batch(jobs, hbm_budget_bytes=256 << 20))
        except BaseException as e:  # noqa: BLE001 - reported by the main thread
            errors.append((n, e))

    say("threads")
    with msa.Server(hbm_budget_bytes=1 << 30, max_inflight=2) as srv:
        threads = [threading.Thread(target=work, args=(n,)) for n in (0, 7, 14)]
        for t in threads:
            t.start()
        for b, shapes in enumerate(BATCHES):
            jobs = jobs_of(shapes, 400 + b)
            tickets = [srv.submit(*j) for j in jobs]
            check(jobs, [srv.wait(t, 30_000_000) for t in tickets])
        for t in threads:
            t.join()
    assert not errors, errors
