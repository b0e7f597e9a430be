"""Time-outs of the streaming fills' waits, forced from the host (a wait limit
of one tick; every kernel still exits normally): the server's report names the
job, the block and the block queue, and the jobs are run again."""
import re
import sys

import numpy as np
import pytest

import paper_2311_17530_amd as msa
from msa_inputs import protein_scoring

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


@pytest.mark.parametrize("lens", [[60, 70, 66, 80], [20, 22, 18, 21, 19]], ids=["k4", "k5"])
def test_report_names_job_and_block(lens, capfd):
    sub, gap = protein_scoring()
    rng = np.random.Generator(np.random.PCG64(sum(lens)))
    jobs = [([rng.integers(0, 20, n).astype(np.uint8) for n in lens], sub, gap) for _ in range(6)]
    plain = [msa.align(*j) for j in jobs]
    say("forced time-outs, k =", len(lens))
    with msa.Server(hbm_budget_bytes=2 << 30, max_inflight=1) as srv:
        srv.debug_wait_limit(1, 1)
        tickets = [srv.submit(*j) for j in jobs]
        out = [srv.wait(t, 60_000_000) for t in tickets]
        stats = srv.stats()
    for (st, s1, r1), (s0, r0) in zip(out, plain):
        assert st == msa.MSA_OK and s1 == s0 and np.array_equal(r1, r0)
    err = capfd.readouterr().err
    assert stats["rerun"] > 0 and "timed out" in err, (stats, err)
    m = re.search(r"timed out in a dependency wait: job (-?\d+) \(k = (\d), lengths ([\d ]+)\), "
                  r"block (\d+), queue head (\d+) of (\d+)", err)
    assert m, err
    blocks = int(m[6])
    assert int(m[1]) >= 0 and int(m[2]) == len(lens) and m[3].split() == [str(n) for n in lens]
    assert 0 <= int(m[4]) < blocks and int(m[5]) > 0
