"""The planner's estimate that short whole tiles share a worker: whenever a
plan of one unit size takes more units than workers on the strength of it,
the queue as it is dealt really leaves the busiest worker with no more than
one unit's pages and cost."""
import numpy as np
import pytest

from paper_2609_37626_amd import binding as B

UNIT_X16 = 96   # the planner's fixed cost of a unit, pages * 16


def dealt_loads(units, G):
    """Pages * 16 and unit costs per worker: slot i of pass k goes to worker i,
    or to G - 1 - i on odd passes (which worker a slot is does not matter)."""
    loads = np.zeros(G, np.int64)
    for i, u in enumerate(units):
        k, r = divmod(i, G)
        loads[r if k % 2 == 0 else G - 1 - r] += 16 * int(u[2] - u[1]) + UNIT_X16
    return loads


@pytest.mark.parametrize("q_chunk", [1, 2, 5])
def test_paired_units_fit_the_busiest_worker(q_chunk):
    rng = np.random.default_rng(q_chunk)
    paired = 0
    for trial in range(400):
        G = int(rng.integers(8, 257))
        n = max(1, int(rng.integers(G // 8 + 1, 2 * G)) // q_chunk)
        seq = np.clip(rng.lognormal(8.0, rng.uniform(0.5, 2.0), n), q_chunk, 131072).astype(np.int32)
        d = B.make_desc(n, 128, int(-(-seq.max() // 64)), int((-(-seq // 64)).sum()))
        units, _, stats = B.splash_mla_plan_host(seq, q_chunk, d, G, 0)
        if stats["fold"] or not G < stats["units"] < 2 * G:
            continue
        last = np.array([int(seq[t // q_chunk]) - q_chunk + t % q_chunk + 1 for t in range(n * q_chunk)])
        pages = -(-last // 64)
        size = min(stats["chunk_pages"], int(pages.max()))
        short = int((pages <= (16 * size - UNIT_X16) // 32).sum())
        if 2 * (stats["units"] - G) > short:
            continue
        paired += 1
        assert dealt_loads(units, G).max() <= 16 * size + UNIT_X16
    assert paired >= 10


def test_mixed_batch_takes_shorter_units():
    # 40 histories of 300 pages and 40 of 4: with at most one unit a worker the
    # long ones can be cut six ways (50 pages); cut seven ways, the 40 short
    # units and as many more share workers
    seq = np.array([300 * 64] * 40 + [4 * 64] * 40, np.int32)
    d = B.make_desc(80, 128, 300, int((-(-seq // 64)).sum()))
    units, _, stats = B.splash_mla_plan_host(seq, 1, d, 300, 0)
    assert stats["units"] == 320 and stats["chunk_pages"] == 43
    assert dealt_loads(units, 300).max() <= 16 * 43 + UNIT_X16
