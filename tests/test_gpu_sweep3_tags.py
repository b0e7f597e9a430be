"""The streaming three-sequence fill accepts a neighbour's exchange word by the
launch's tag in it, so no word of an earlier fill may carry the tag of the
current one.  Calls that end a launch on the workspace without rewriting the
exchange regions (tile fills, repeated tracebacks) come between streaming
fills here, as many as there are tags.  Every mode; results equal the oracle's.
"""
import sys

import numpy as np
import pytest

import paper_2311_17530_amd as msa
from msa_inputs import protein_scoring
from oracle import oracle_align, oracle_align_egf, oracle_coopt, oracle_nearopt

pytestmark = pytest.mark.gpu

LENS = [60, 130, 40]  # 3 x 3 blocks
PATHS, DELTA = 6, 9


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


def draw(seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return [rng.integers(0, 20, size=n).astype(np.uint8) for n in LENS]


def run_and_check(dev, mode, seqs, sub, gap):
    dev.set_sequences(seqs)
    if mode == "coopt":
        dev.run_coopt(PATHS)
        s1, got = dev.result_coopt()
        s0, want = oracle_coopt(seqs, sub, gap, PATHS)[:2]
        assert s1 == s0 and len(got) == len(want)
        assert all(np.array_equal(a, b) for a, b in zip(got, want))
    elif mode == "nearopt":
        dev.run_nearopt(DELTA, PATHS)
        s1, got = dev.result_nearopt()
        s0, want = oracle_nearopt(seqs, sub, gap, DELTA, PATHS)
        assert s1 == s0 and len(got) == len(want)
        assert all(a[0] == b[0] and np.array_equal(a[1], b[1]) for a, b in zip(got, want))
    else:
        oracle = oracle_align_egf if mode == "egf" else oracle_align
        dev.run()
        s1, r1 = dev.result()
        s0, r0 = oracle(seqs, sub, gap)[:2]
        assert s1 == s0 and np.array_equal(r1, r0)


@pytest.mark.parametrize("mode", ["plain", "egf", "coopt", "nearopt"])
@pytest.mark.parametrize("between", [0, 5, 6, 7])
def test_tile_fills_between_streaming_fills(mode, between):
    sub, gap = protein_scoring()
    dev = msa.DeviceAligner(LENS, sub, gap, end_gaps_free=mode == "egf",
                            cooptimal=mode == "coopt", nearopt=mode == "nearopt")
    seed = 3000
    try:
        for rnd in range(3 if between else 18):
            msa.tune_set(msa.MSA_TUNE_PLAIN, 3, max(LENS), 0, 0)
            say("streaming fill", mode, between, rnd)
            run_and_check(dev, mode, draw(seed), sub, gap)
            seed += 1
            msa.tune_set(msa.MSA_TUNE_PLAIN, 3, max(LENS), 2, 0)
            for _ in range(between):
                run_and_check(dev, mode, draw(seed), sub, gap)
                seed += 1
    finally:
        msa.tune_clear()


def test_repeated_tracebacks_between_streaming_fills():
    sub, gap = protein_scoring()
    dev = msa.DeviceAligner(LENS, sub, gap)
    for rnd in range(4):
        say("streaming fill, then six tracebacks more", rnd)
        run_and_check(dev, "plain", draw(4000 + rnd), sub, gap)
        for _ in range(6):
            dev.run_traceback()


@pytest.mark.parametrize("lens", [[30, 70, 20], [9, 20, 18, 11], [6, 5, 9, 7, 8]],
                         ids=lambda s: "k%d" % len(s))
def test_count_of_streaming_fills_stays_small(lens):
    """The count behind the tags is word 6 of the control block, which a
    workspace starts with.  It starts again after 105 fills and, set to the
    largest integer, goes on with valid tags."""
    import torch
    sub, gap = protein_scoring()
    dev = msa.DeviceAligner(lens, sub, gap)
    off = dev.ws_ptr - dev.ws.data_ptr() + 4 * 6
    count = dev.ws[off: off + 4].view(torch.int32)

    def one(seed):
        rng = np.random.Generator(np.random.PCG64(seed))
        seqs = [rng.integers(0, 20, size=n).astype(np.uint8) for n in lens]
        dev.set_sequences(seqs)
        dev.run()
        s1, r1 = dev.result()
        s0, r0 = oracle_align(seqs, sub, gap)[:2]
        assert s1 == s0 and np.array_equal(r1, r0), seed

    say("count of streaming fills", lens)
    for n in range(110):
        assert int(count.item()) == n % 105
        if n % 10 == 0 or n > 100:
            one(5000 + n)
        else:
            dev.run()
    count.fill_(2 ** 31 - 1)
    for n in range(4):
        one(6000 + n)
        assert 0 <= int(count.item()) < 105


@pytest.mark.parametrize("lens,mode", [(LENS, "plain"), (LENS, "egf"), (LENS, "coopt"),
                                       (LENS, "nearopt"), ([9, 20, 18, 11], "plain"),
                                       ([6, 5, 9, 7, 8], "plain")],
                         ids=lambda x: x if isinstance(x, str) else "k%d" % len(x))
def test_captured_calls_replay_with_new_sequences(lens, mode):
    """The tag is read on the device, so a captured call replays with a tag of
    its own each time, also with eager calls and synchronisations in between."""
    import torch
    sub, gap = protein_scoring()
    dev = msa.DeviceAligner(lens, sub, gap, end_gaps_free=mode == "egf",
                            cooptimal=mode == "coopt", nearopt=mode == "nearopt")

    def sequences(seed):
        rng = np.random.Generator(np.random.PCG64(seed))
        return [rng.integers(0, 20, size=n).astype(np.uint8) for n in lens]

    def call():
        if mode == "coopt":
            dev.run_coopt(PATHS)
        elif mode == "nearopt":
            dev.run_nearopt(DELTA, PATHS)
        else:
            dev.run()

    def result():
        if mode == "coopt":
            return dev.result_coopt()[1]
        return [r for _, r in dev.result_nearopt()[1]] if mode == "nearopt" else [dev.result()[1]]

    say("captured", lens, mode)
    dev.set_sequences(sequences(1))
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for it in range(20):
        seqs = sequences(10 + it)
        if it % 5 == 3:  # an eager call between the replays
            dev.set_sequences(sequences(100 + it))
            call()
        dev.set_sequences(seqs)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        if mode == "coopt":
            want = oracle_coopt(seqs, sub, gap, PATHS)[1]
        elif mode == "nearopt":
            want = [r for _, r in oracle_nearopt(seqs, sub, gap, DELTA, PATHS)[1]]
        else:
            want = [(oracle_align_egf if mode == "egf" else oracle_align)(seqs, sub, gap)[1]]
        got = result()
        assert len(got) == len(want) and all(np.array_equal(a, b) for a, b in zip(got, want)), it
