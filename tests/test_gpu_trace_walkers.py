"""Traceback by several walkers where other tests leave it to the single wave:
free end gaps of four sequences, one long sequence beside very short or empty
ones, short alignments of two to four sequences (in a batch whose longest walk
the walkers take, they take all), and both sides of the bound for two
sequences of unequal length.  Rows equal the oracle's."""
import sys

import numpy as np
import pytest

import paper_2311_17530_amd as msa
from msa_inputs import dna_scoring, protein_scoring
from oracle import oracle_align, oracle_align_egf

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


def draw(seed, lens, alpha, related=False):
    rng = np.random.Generator(np.random.PCG64(seed))
    anc = rng.integers(0, alpha, size=max(lens + [1]))
    out = []
    for n in lens:
        s = anc[:n].copy() if related else rng.integers(0, alpha, size=n)
        at = rng.integers(0, max(n, 1), size=n // 6)
        s[at] = rng.integers(0, alpha, size=len(at))
        out.append(s.astype(np.uint8))
    return out


@pytest.mark.parametrize("lens", [[96, 12, 9, 10], [100, 30, 20, 8], [8, 97, 40, 33],
                                  [10, 12, 11, 130], [96, 96, 5, 6], [30, 28, 99, 31]],
                         ids=lambda s: "x".join(map(str, s)))
def test_free_end_gaps_of_four_sequences(lens):
    for seed in range(4):
        sub, gap = dna_scoring() if seed % 2 else protein_scoring()
        dev = msa.DeviceAligner(lens, sub, gap, end_gaps_free=True)
        seqs = draw(600 + seed, lens, sub.shape[0], seed < 2)
        say("walkers egf", lens, "seed", seed)
        dev.set_sequences(seqs)
        dev.run()
        s0, r0 = oracle_align_egf(seqs, sub, gap)[:2]
        s1, r1 = dev.result()
        assert s1 == s0 and np.array_equal(r1, r0)


@pytest.mark.parametrize("lens", [[96, 0], [0, 300], [255, 60], [256, 60], [270, 255], [150, 141],
                                  [96, 0, 0], [1, 200, 2], [0, 3, 500], [96, 0, 1, 2],
                                  [3, 2, 160, 1], [0, 0, 0, 120], [100, 99, 3, 0], [2, 110, 40, 3]],
                         ids=lambda s: "x".join(map(str, s)))
def test_one_long_sequence(lens):
    for seed in range(3):
        sub, gap = dna_scoring() if seed % 2 else protein_scoring()
        dev = msa.DeviceAligner(lens, sub, gap)
        seqs = draw(700 + seed, lens, sub.shape[0], seed == 2)
        say("walkers", lens, "seed", seed)
        dev.set_sequences(seqs)
        dev.run()
        s0, r0 = oracle_align(seqs, sub, gap)[:2]
        s1, r1 = dev.result()
        assert s1 == s0 and np.array_equal(r1, r0)


def test_short_alignments_in_a_batch_with_a_long_one():
    shapes = [[100, 98, 97], [0, 0], [1, 0], [3, 4], [8, 8], [30, 5], [60, 70], [0, 0, 0], [5, 1, 2],
              [4, 4, 4], [16, 16, 16], [17, 40, 9], [0, 0, 0, 0], [2, 3, 1, 2], [9, 9, 8, 9],
              [30, 9, 25, 4], [8, 40, 12, 33], [60, 7, 9, 8], [8, 8, 8, 8], [16, 15, 17, 14]]
    for rnd in range(4):
        jobs = []
        for i, lens in enumerate(shapes):
            sub, gap = dna_scoring() if (i + rnd) % 2 else protein_scoring()
            jobs.append((draw(40 * rnd + i, lens, sub.shape[0], rnd % 2 == 0), sub, gap))
        say("walkers in a batch", rnd)
        for (seqs, sub, gap), (st, s1, r1) in zip(jobs, msa.align_batch(jobs)):
            s0, r0 = oracle_align(seqs, sub, gap)[:2]
            assert st == msa.MSA_OK and s1 == s0 and np.array_equal(r1, r0), [len(s) for s in seqs]
