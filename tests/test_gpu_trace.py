"""GPU parity of the traceback by several walkers: inputs on which the walkers'
paths stay apart for long (unrelated sequences, lengths far from each other,
one dimension much longer), very short ones (one walker, ranges of a few
columns), both sides of the length bound, free end gaps.  Rows equal the
oracle's exactly.
"""
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


def draw(seed, lens, alpha):
    rng = np.random.Generator(np.random.PCG64(seed))
    return [rng.integers(0, alpha, size=n).astype(np.uint8) for n in lens]


SHAPES = [
    [3, 4], [8, 8], [700, 90], [40, 900], [4000, 4191], [4000, 4192],
    [5, 1, 2], [16, 16, 16], [17, 120, 9], [150, 20, 60], [33, 80, 170],
    [2, 3, 1, 2], [30, 9, 25, 4], [8, 40, 12, 33], [60, 7, 9, 8],
    [4, 5, 3, 2, 6], [16, 5, 9, 4, 12], [3, 24, 4, 5, 9],
]


@pytest.mark.parametrize("lens", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dna", [False, True], ids=["protein", "dna"])
def test_rows_match_oracle(lens, dna):
    sub, gap = dna_scoring() if dna else protein_scoring()
    dev = msa.DeviceAligner(lens, sub, gap)
    for seed in range(3):
        seqs = draw(31 * seed + sum(lens), lens, sub.shape[0])
        if seed == 2:  # long runs of one residue: ties almost everywhere
            seqs = [np.where(np.arange(len(s)) % 7 == 3, s, 1).astype(np.uint8) for s in seqs]
        say("trace", lens, "dna" if dna else "protein", "seed", seed)
        dev.set_sequences(seqs)
        dev.run()
        s0, r0 = oracle_align(seqs, sub, gap)[:2]
        s1, r1 = dev.result()
        assert s1 == s0 and np.array_equal(r1, r0)


@pytest.mark.parametrize("lens", [[9, 6], [300, 60], [40, 41, 39], [17, 120, 9], [20, 9, 14, 11]],
                         ids=lambda s: "x".join(map(str, s)))
def test_egf_rows_match_oracle(lens):
    sub, gap = dna_scoring()
    dev = msa.DeviceAligner(lens, sub, gap, end_gaps_free=True)
    for seed in range(4):
        seqs = draw(500 + seed, lens, 4)
        say("trace egf", lens, "seed", seed)
        dev.set_sequences(seqs)
        dev.run()
        s0, r0 = oracle_align_egf(seqs, sub, gap)[:2]
        s1, r1 = dev.result()
        assert s1 == s0 and np.array_equal(r1, r0)


# both sides of the longest length from which the walkers take the walk
@pytest.mark.parametrize("lens", [[95, 10], [96, 10], [95, 20, 41], [12, 96, 30], [95, 12, 9, 10],
                                  [10, 9, 96, 12]], ids=lambda s: "x".join(map(str, s)))
def test_rows_match_oracle_at_the_walkers_bound(lens):
    for sub, gap in (protein_scoring(), dna_scoring()):
        dev = msa.DeviceAligner(lens, sub, gap)
        seqs = draw(900 + sum(lens), lens, sub.shape[0])
        say("trace", lens)
        dev.set_sequences(seqs)
        dev.run()
        s0, r0 = oracle_align(seqs, sub, gap)[:2]
        s1, r1 = dev.result()
        assert s1 == s0 and np.array_equal(r1, r0)
