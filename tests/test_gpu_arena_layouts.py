"""Layout of k = 4 and 5 jobs in batched arenas: a job keeps the tile fill's
layout where the streaming fill's does not fit the arena, and k = 5 jobs do in
small arenas.  Servers whose slots lie between the two layouts of a job, and
batches in threads of their own (an arena lives as long as its thread's, so
only a fresh one is as small as asked for).  Results equal the oracle's."""
import sys
import threading

import numpy as np
import pytest

import paper_2311_17530_amd as msa
from msa_inputs import dna_scoring, protein_scoring
from oracle import oracle_align

pytestmark = pytest.mark.gpu

MB = 1 << 20


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


def jobs_of(shapes, seed):
    out = []
    for i, lens in enumerate(shapes):
        rng = np.random.Generator(np.random.PCG64([seed, i, *lens]))
        sub, gap = dna_scoring() if i % 2 else protein_scoring()
        out.append(([rng.integers(0, sub.shape[0], n).astype(np.uint8) for n in lens], sub, gap))
    return out


def check(jobs, results):
    for (seqs, sub, gap), (st, s1, r1) in zip(jobs, results):
        s0, r0 = oracle_align(seqs, sub, gap)[:2]
        assert st == msa.MSA_OK and s1 == s0 and np.array_equal(r1, r0), [len(s) for s in seqs]


# a k = 4 job of 7 MB in the tile fill's layout and 14 MB in the streaming one's
# among small ones that stream, and k = 5 jobs on both sides of their rule
@pytest.mark.parametrize("slot_mb", [10, 12, 18, 96])
@pytest.mark.parametrize("shapes", [
    [[140, 2, 34, 33], [9, 12, 7, 10], [2, 72, 71, 1], [12, 9, 17, 20], [5, 5, 5, 5]],
    [[12, 12, 12, 12, 12], [5, 6, 7, 4, 5], [17, 13, 3, 2, 18], [4, 4, 4, 4, 4]]], ids=["k4", "k5"])
def test_server_slots_between_the_layouts(shapes, slot_mb):
    jobs = jobs_of(shapes * 2, slot_mb)
    say("server slots of", slot_mb, "MB")
    with msa.Server(hbm_budget_bytes=2 * slot_mb * MB, max_inflight=2) as srv:
        tickets = [srv.submit(*j) for j in jobs]
        check(jobs, [srv.wait(t, 60_000_000) for t in tickets])


@pytest.mark.parametrize("budget_mb", [12, 24, 95, 96])
def test_batches_in_small_arenas(budget_mb):
    jobs = jobs_of([[140, 2, 34, 33], [9, 12, 7, 10], [2, 72, 71, 1], [20, 14, 9], [30, 40],
                    [12, 12, 12, 12, 12], [5, 6, 7, 4, 5], [13, 12, 11, 10, 9]] * 3, budget_mb)
    out = []

    def work():
        out.append(msa.align_batch(jobs, hbm_budget_bytes=budget_mb * MB))

    say("batch in an arena of", budget_mb, "MB")
    th = threading.Thread(target=work)
    th.start()
    th.join()
    check(jobs, out[0])
