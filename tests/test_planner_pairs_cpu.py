"""The planner's estimate that short whole tiles share a worker (dense plans,
which the host mirror makes; lists and shards: test_gpu_plan_pairs.py).  The
host plan takes the unit size of the plain estimate, and whenever that lets more
units than workers go free, the queue as it is dealt leaves the busiest worker
with no more than one unit's pages and cost."""
import numpy as np
import pytest

from paper_2609_37626_amd import binding as B
from tests import plan_estimate as E


def check_plan(seq, q_chunk, G):
    """1 if more units than workers went free."""
    d = B.make_desc(len(seq), 128, int(-(-seq.max() // 64)), int((-(-seq // 64)).sum()))
    units, _, stats = B.splash_mla_plan_host(seq, q_chunk, d, G, 0)
    if stats["fold"]:
        return 0
    pages = np.array([-(-(int(s) - q_chunk + i + 1) // 64) for s in seq for i in range(q_chunk)])
    size, W, free = E.unit_size(pages, q_chunk, G)
    assert (stats["chunk_pages"], stats["units"]) == (size, W)
    if free:
        assert E.busiest(units, G) <= 16 * min(size, int(pages.max())) + E.UNIT
    return int(free)


@pytest.mark.parametrize("q_chunk", [1, 2, 5, 70])
def test_paired_units_fit_the_busiest_worker(q_chunk):
    rng = np.random.default_rng(q_chunk)
    paired = 0
    for trial in range(400):
        G = int(rng.integers(8, 257))
        n = max(1, int(rng.integers(G // 8 + 1, 2 * G)) // q_chunk)
        paired += check_plan(np.clip(rng.lognormal(8.0, rng.uniform(0.5, 2.0), n), q_chunk, 131072).astype(np.int32),
                             q_chunk, G)
    assert paired >= (10 if q_chunk < 70 else 0)


@pytest.mark.parametrize("q_chunk", [2, 5, 8])
def test_rows_across_a_page_edge(q_chunk):
    # the rows of a short request lie on both sides of a page edge; in the
    # queue they stand where its longest row does
    rng = np.random.default_rng(q_chunk)
    paired = 0
    for trial in range(600):
        long, short = int(rng.integers(1, 5)), int(rng.integers(4, 30))
        G = int(rng.integers(max(8, (long + short) * q_chunk // 2), (long + short) * q_chunk + 40))
        edge = 64 * int(rng.integers(1, 12))
        seq = np.concatenate([rng.integers(3000, 20000, long), np.maximum(edge + rng.integers(0, q_chunk, short), q_chunk)])
        paired += check_plan(seq.astype(np.int32), q_chunk, G)
    assert paired >= 10


def test_mixed_batch_takes_shorter_units():
    # 40 histories of 300 pages and 40 of 4: with at most one unit a worker the
    # long ones can be cut six ways (50 pages); cut seven ways, the 40 short
    # units and as many more share workers
    seq = np.array([300 * 64] * 40 + [4 * 64] * 40, np.int32)
    d = B.make_desc(80, 128, 300, int((-(-seq // 64)).sum()))
    units, _, stats = B.splash_mla_plan_host(seq, 1, d, 300, 0)
    assert stats["units"] == 320 and stats["chunk_pages"] == 43
    assert E.busiest(units, 300) <= 16 * 43 + E.UNIT
