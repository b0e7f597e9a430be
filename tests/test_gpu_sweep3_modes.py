"""Co-optimal and near-optimal lists of three sequences on both sides of the
rule that chooses between the streaming and the tile fill: long lines beside
few others, few rows, and ordinary shapes.  Lists and tie
sets equal the oracle's."""
import sys

import numpy as np
import pytest

import paper_2311_17530_amd as msa
from msa_inputs import dna_scoring, protein_scoring
from oracle import oracle_coopt, oracle_nearopt

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
    yield
    msa.tune_clear()


SHAPES = [[1, 1, 300], [1, 1, 600], [3, 3, 700], [4, 4, 600], [7, 7, 500], [8, 2, 500], [0, 0, 900],
          [900, 0, 0], [0, 900, 0], [5, 300, 40], [2, 400, 400], [20, 200, 200], [11, 256, 260],
          [12, 256, 260], [60, 70, 50]]


@pytest.mark.parametrize("lens", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_lists_on_both_sides_of_the_rule(lens):
    for sub, gap in (protein_scoring(), dna_scoring()):
        rng = np.random.Generator(np.random.PCG64(sum(lens)))
        seqs = [rng.integers(0, sub.shape[0], size=n).astype(np.uint8) for n in lens]
        dev = msa.DeviceAligner(lens, sub, gap, cooptimal=True)
        dev.set_sequences(seqs)
        say("co-optimal", lens)
        dev.run_coopt(7)
        s1, got = dev.result_coopt()
        s0, want, ties = oracle_coopt(seqs, sub, gap, 7, want_ties=True)[:3]
        assert s1 == s0 and len(got) == len(want)
        assert all(np.array_equal(a, b) for a, b in zip(got, want))
        assert np.array_equal(dev.export_dirs(), ties)
        near = msa.DeviceAligner(lens, sub, gap, nearopt=True)
        near.set_sequences(seqs)
        say("near-optimal", lens)
        near.run_nearopt(5, 7)
        s1, got = near.result_nearopt()
        s0, want = oracle_nearopt(seqs, sub, gap, 5, 7)
        assert s1 == s0 and len(got) == len(want)
        assert all(a[0] == b[0] and np.array_equal(a[1], b[1]) for a, b in zip(got, want))
