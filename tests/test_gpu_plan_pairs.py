"""The device planner against its host mirror where short whole tiles share
workers (more units than workers), on both sides of that estimate's line."""
import numpy as np
import pytest
import torch

from paper_2609_37626_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q_chunk", [1, 2])
@pytest.mark.parametrize("short", [3, 12, 13, 14, 40])
def test_device_plan_of_mixed_lengths_matches_host(short, q_chunk):
    # few long histories and `short` of 1 .. 20 pages: the short ones that a
    # size lets two of share a worker are counted page by page
    rng = np.random.default_rng(short)
    seq = np.concatenate([rng.integers(200 * 64, 500 * 64, 30), rng.integers(q_chunk, 20 * 64, short)]).astype(np.int32)
    d = B.make_desc(len(seq), 16, int(-(-seq.max() // 64)), int((-(-seq // 64)).sum()))
    ws = torch.zeros(B.workspace_size(len(seq), q_chunk, 16, 0), dtype=torch.uint8, device="cuda")
    B.splash_mla_plan(torch.from_numpy(seq).cuda(), q_chunk, d, ws)
    torch.cuda.synchronize()
    units, _, stats = B.splash_mla_plan_host(seq, q_chunk, d, B.device_workers(), 0)
    offs, _ = B.workspace_offsets(len(seq), q_chunk, 16, 0)
    raw = ws.cpu().numpy()
    hdr = raw[offs[0]:offs[0] + 64].view(np.int32)
    assert (hdr[1], hdr[2], hdr[3]) == (stats["units"], stats["partials"], stats["chunk_pages"])
    dev = raw[offs[1]:offs[1] + 16 * stats["units"]].view(np.int32).reshape(-1, 4)
    canon = lambda u: u[np.lexsort(u.T[::-1])]
    assert np.array_equal(canon(dev), canon(units))
