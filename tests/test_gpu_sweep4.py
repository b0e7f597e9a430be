"""GPU parity of the streaming four-sequence fill at the sizes where its blocks
can go wrong: lengths at the edges of its 4 x 16 x 16 blocks, runs of the
fourth dimension at the edges of its 4-cell direction words, empty and
one-residue sequences, more blocks than fit the chip.  Score, rows and the full
decision tensor equal the oracle's exactly (integer arithmetic: no tolerance).
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
    [0, 0, 0, 0], [1, 0, 0, 1], [0, 1, 17, 4], [3, 15, 16, 3], [4, 16, 15, 5],
    [7, 17, 31, 8], [8, 31, 32, 9], [9, 32, 14, 12], [25, 33, 33, 1], [2, 47, 48, 31],
    [33, 5, 6, 40], [12, 15, 15, 0],
    # more blocks than fit the chip at once
    [135, 111, 95, 5], [64, 160, 143, 6], [303, 65, 63, 3],
]


@pytest.mark.parametrize("lens", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dna", [False, True], ids=["protein", "dna"])
def test_sweep4_matches_oracle(lens, dna):
    sub, gap = dna_scoring() if dna else protein_scoring()
    dev = msa.DeviceAligner(lens, sub, gap)
    for seed in (1, 2):
        seqs = draw(100 * seed + sum(lens), lens, sub.shape[0])
        say("sweep4", lens, "dna" if dna else "protein", "seed", seed)
        dev.set_sequences(seqs)
        dev.run()
        s0, r0, d0 = oracle_align(seqs, sub, gap, want_dir=True)
        s1, r1 = dev.result()
        assert s1 == s0 and np.array_equal(r1, r0)
        assert np.array_equal(dev.export_dirs(), d0)


def test_sweep4_tags_over_many_launches_and_variants():
    """More launches than there are tags, with the tile fill (which uses the
    exchange regions' memory for its faces) now and then in between."""
    lens = [21, 34, 18, 23]
    sub, gap = protein_scoring()
    dev = msa.DeviceAligner(lens, sub, gap)
    try:
        for it in range(36):
            seqs = draw(7000 + it, lens, sub.shape[0])
            msa.tune_set(msa.MSA_TUNE_PLAIN, 4, max(lens), 2 if it % 7 in (3, 4) else 0, 0)
            say("sweep4 launch", it)
            dev.set_sequences(seqs)
            dev.run()
            s0, r0 = oracle_align(seqs, sub, gap)[:2]
            s1, r1 = dev.result()
            assert s1 == s0 and np.array_equal(r1, r0), it
    finally:
        msa.tune_clear()


def test_sweep4_bad_residue_code():
    lens = [20, 20, 20, 20]
    sub, gap = protein_scoring()
    for d in range(4):
        seqs = draw(50 + d, lens, sub.shape[0])
        seqs[d][19] = 20  # a code outside the alphabet
        dev = msa.DeviceAligner(lens, sub, gap)
        dev.set_sequences(seqs)
        say("sweep4 bad code in sequence", d)
        dev.run()
        assert int(dev.d_status.item()) == msa.MSA_EINVAL
