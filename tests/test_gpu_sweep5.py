"""GPU parity of the streaming five-sequence fill at the sizes where its blocks
can go wrong: lengths at the edges of its blocks of 4 lines a dimension, runs of
the fifth dimension at the edges of its 4-cell direction words, empty and
one-residue sequences, more blocks than fit the chip, both sides of the fifth
length's bound.  Score, rows and the full decision tensor equal the oracle's
exactly (integer arithmetic: no tolerance).
"""
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


def draw(seed, lens, alpha):
    rng = np.random.Generator(np.random.PCG64(seed))
    return [rng.integers(0, alpha, size=n).astype(np.uint8) for n in lens]


SHAPES = [
    [0, 0, 0, 0, 0], [1, 0, 0, 1, 0], [0, 1, 2, 0, 3], [3, 4, 5, 4, 4], [4, 3, 8, 9, 5],
    [7, 8, 4, 5, 8], [8, 5, 7, 1, 9], [9, 6, 3, 12, 12], [5, 2, 9, 4, 31], [2, 13, 6, 7, 15],
    [16, 11, 3, 2, 1], [6, 5, 4, 8, 0], [2, 3, 4, 3, 128], [2, 3, 4, 3, 129],
    # more blocks than fit the chip at once
    [24, 21, 19, 17, 14],
]


@pytest.mark.parametrize("lens", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dna", [False, True], ids=["protein", "dna"])
def test_sweep5_matches_oracle(lens, dna):
    sub, gap = dna_scoring() if dna else protein_scoring()
    dev = msa.DeviceAligner(lens, sub, gap)
    for seed in (1, 2):
        seqs = draw(100 * seed + sum(lens), lens, sub.shape[0])
        say("sweep5", lens, "dna" if dna else "protein", "seed", seed)
        dev.set_sequences(seqs)
        dev.run()
        s0, r0, d0 = oracle_align(seqs, sub, gap, want_dir=True)
        s1, r1 = dev.result()
        assert s1 == s0 and np.array_equal(r1, r0)
        assert np.array_equal(dev.export_dirs(), d0)


def test_sweep5_tags_over_many_launches_and_variants():
    """More launches than there are tags, with the tile fill (which uses the
    exchange region's memory for its faces) now and then in between."""
    lens = [9, 12, 7, 10, 11]
    sub, gap = protein_scoring()
    dev = msa.DeviceAligner(lens, sub, gap)
    try:
        for it in range(36):
            seqs = draw(7000 + it, lens, sub.shape[0])
            msa.tune_set(msa.MSA_TUNE_PLAIN, 5, max(lens), 2 if it % 7 in (3, 4) else 0, 0)
            say("sweep5 launch", it)
            dev.set_sequences(seqs)
            dev.run()
            s0, r0 = oracle_align(seqs, sub, gap)[:2]
            s1, r1 = dev.result()
            assert s1 == s0 and np.array_equal(r1, r0), it
    finally:
        msa.tune_clear()


def test_sweep5_bad_residue_code():
    lens = [9, 10, 9, 8, 9]
    sub, gap = protein_scoring()
    for d in range(5):
        seqs = draw(50 + d, lens, sub.shape[0])
        seqs[d][-1] = 20  # a code outside the alphabet
        dev = msa.DeviceAligner(lens, sub, gap)
        dev.set_sequences(seqs)
        say("sweep5 bad code in sequence", d)
        dev.run()
        assert int(dev.d_status.item()) == msa.MSA_EINVAL


@pytest.mark.parametrize("alpha", [1, 32, 33])  # 33: past the matrix kept in LDS
def test_sweep5_alphabets(alpha):
    rng = np.random.Generator(np.random.PCG64(alpha))
    m = np.triu(rng.integers(-9, 10, (alpha, alpha)))
    sub, gap = (m + np.triu(m, 1).T).astype(np.int8), -3
    lens = [6, 9, 5, 7, 10]
    dev = msa.DeviceAligner(lens, sub, gap)
    seqs = draw(alpha, lens, alpha)
    say("sweep5 alphabet", alpha)
    dev.set_sequences(seqs)
    dev.run()
    s0, r0, d0 = oracle_align(seqs, sub, gap, want_dir=True)
    s1, r1 = dev.result()
    assert s1 == s0 and np.array_equal(r1, r0)
    assert np.array_equal(dev.export_dirs(), d0)


def test_sweep5_batched_jobs_match_oracle():
    """Jobs of uneven lengths in one batch, empty ones and one past the fifth
    length's bound (which takes the tile fill beside the others) among them."""
    shapes = [[5, 6, 7, 8, 9], [0, 0, 0, 0, 0], [12, 3, 9, 4, 16], [2, 3, 4, 3, 129],
              [1, 0, 5, 2, 128], [13, 12, 11, 10, 9], [4, 4, 4, 4, 4]]
    for rnd in range(3):
        jobs = []
        for i, lens in enumerate(shapes):
            sub, gap = dna_scoring() if i % 2 else protein_scoring()
            jobs.append((draw(40 * rnd + i, lens, sub.shape[0]), sub, gap))
        say("sweep5 batch", rnd)
        for (seqs, sub, gap), (st, s1, r1) in zip(jobs, msa.align_batch(jobs)):
            s0, r0 = oracle_align(seqs, sub, gap)[:2]
            assert st == msa.MSA_OK and s1 == s0 and np.array_equal(r1, r0)


# both sides of the rule on short fifth sequences beside many tile waves
@pytest.mark.parametrize("lens", [[64, 64, 3, 3, 4], [68, 72, 3, 4, 4], [68, 72, 3, 4, 5],
                                  [1, 72, 72, 0, 0]], ids=lambda s: "x".join(map(str, s)))
def test_sweep5_many_waves_of_short_blocks(lens):
    sub, gap = protein_scoring()
    dev = msa.DeviceAligner(lens, sub, gap)
    seqs = draw(sum(lens), lens, 20)
    say("sweep5", lens)
    dev.set_sequences(seqs)
    dev.run()
    s0, r0, d0 = oracle_align(seqs, sub, gap, want_dir=True)
    s1, r1 = dev.result()
    assert s1 == s0 and np.array_equal(r1, r0)
    assert np.array_equal(dev.export_dirs(), d0)
    # in a batch, beside a shape of the other kind
    jobs = [(seqs, sub, gap), (draw(1, [5, 6, 7, 8, 9], 20), sub, gap)]
    for (sq, _, _), (st, s1, r1) in zip(jobs, msa.align_batch(jobs)):
        s0, r0 = oracle_align(sq, sub, gap)[:2]
        assert st == msa.MSA_OK and s1 == s0 and np.array_equal(r1, r0)
