"""The device planner against its host mirror, and for lists and shards against
the plain estimate and the queue as it is dealt, where short whole tiles share
workers (more units than workers), on both sides of that estimate's line."""
import numpy as np
import pytest
import torch

from paper_2609_37626_amd import binding as B
from tests import plan_estimate as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q_chunk", [1, 2, 5])
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


def shared_pages(seq, q_chunk, heads=16):
    """Inputs whose requests all read one set of pages."""
    n, pages = len(seq) * q_chunk, int(-(-seq.max() // 64))
    kv = torch.randn((pages, 64, 576), device="cuda").bfloat16()
    table = torch.arange(pages, dtype=torch.int32, device="cuda").repeat(len(seq), 1).contiguous()
    q = torch.randn((n, heads, 576), device="cuda").bfloat16()
    return q, kv, table, torch.from_numpy(seq).cuda(), B.make_desc(len(seq), heads, pages, pages)


def device_plan(ws, batch, q_chunk, heads, max_partials):
    torch.cuda.synchronize()
    offs, _ = B.workspace_offsets(batch, q_chunk, heads, max_partials)
    raw = ws.cpu().numpy()
    hdr = raw[offs[0]:offs[0] + 64].view(np.int32)
    return int(hdr[3]), raw[offs[1]:offs[1] + 16 * int(hdr[1])].view(np.int32).reshape(-1, 4)


@pytest.mark.parametrize("long,long_pages,short,short_pages", [(9, 147, 184, 2), (22, 70, 124, 2), (33, 64, 180, 3),
                                                               (34, 49, 187, 5)])
def test_shard_pairs_carry_two_partials(long, long_pages, short, short_pages):
    # a shard's whole tiles write partials too: two of them share a worker
    # only with both partials' cost inside one unit's time
    seq = np.array([long_pages * 64] * long + [short_pages * 64] * short, np.int32)
    n, G, max_partials = len(seq), B.device_workers(), 1024
    q, kv, table, lens, d = shared_pages(seq, 1)
    ws = torch.zeros(B.workspace_size(n, 1, 16, max_partials), dtype=torch.uint8, device="cuda")
    out = torch.empty((n, 1, 16, 512), dtype=torch.float32, device="cuda")
    lse = torch.empty((n, 1, 16), dtype=torch.float32, device="cuda")
    B.splash_mla_attend_shard(q, kv, table, lens, 1, torch.zeros_like(lens), lens, 1, 0, out, lse, d, ws)
    size, units = device_plan(ws, n, 1, 16, max_partials)
    want, W, free = E.unit_size(-(-seq // 64), 1, G, max_partials, shard=True)
    assert (size, len(units)) == (want, W)
    if free:
        assert E.busiest(units, G, shard=True) <= 16 * min(size, long_pages) + E.UNIT + E.SPLIT


@pytest.mark.parametrize("q_chunk,batch,counts", [(2, 137, (2048, 128)), (3, 100, (64, 2048, 2048)), (1, 280, (2048,))])
def test_uneven_lists_of_a_request_do_not_pair(q_chunk, batch, counts):
    # a request's units stand together in the queue, by its longest list: with
    # uneven lists its short end is not short
    seq = np.full(batch, 2048 + q_chunk, np.int32)
    n, G, max_partials = batch * q_chunk, B.device_workers(), 1024
    q, kv, table, lens, d = shared_pages(seq, q_chunk)
    ws = torch.zeros(B.workspace_size(batch, q_chunk, 16, max_partials), dtype=torch.uint8, device="cuda")
    out = torch.empty((n, 16, 512), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((n, 16), dtype=torch.float32, device="cuda")
    count = np.array(list(counts) * batch, np.int32)
    if q_chunk == 1:
        count[100:] = 64   # one row each: the queue is ordered by the lists themselves
    idx = torch.arange(2048, dtype=torch.int32, device="cuda").repeat(n, 1).contiguous()
    B.splash_mla_attend_topk(q, kv, table, lens, q_chunk, idx, torch.from_numpy(count).cuda(), out, lse, d, ws)
    size, units = device_plan(ws, batch, q_chunk, 16, max_partials)
    want, W, free = E.unit_size(-(-count // 64), q_chunk, G, max_partials, 32, listed=True)
    assert (size, len(units)) == (want, W)
    assert free == (q_chunk == 1)
    if free:
        assert E.busiest(units, G) <= 16 * min(size, 32) + E.UNIT


def test_a_queue_in_tile_order_does_not_pair():
    # past 8,192 tiles the queue is not ordered by length: 40 long lists and 240
    # short ones among 8,120 empty ones
    batch, G, max_partials = 8400, B.device_workers(), 1024
    q, kv, table, lens, d = shared_pages(np.full(batch, 2048, np.int32), 1)
    count = np.zeros(batch, np.int32)
    count[::35] = 64
    count[7:8400:210] = 2048
    ws = torch.zeros(B.workspace_size(batch, 1, 16, max_partials), dtype=torch.uint8, device="cuda")
    out = torch.empty((batch, 16, 512), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((batch, 16), dtype=torch.float32, device="cuda")
    idx = torch.arange(2048, dtype=torch.int32, device="cuda").repeat(batch, 1).contiguous()
    B.splash_mla_attend_topk(q, kv, table, lens, 1, idx, torch.from_numpy(count).cuda(), out, lse, d, ws)
    size, units = device_plan(ws, batch, 1, 16, max_partials)
    want, W, free = E.unit_size(-(-count // 64), 1, G, max_partials, 32, listed=True)
    assert (size, len(units), free) == (want, W, False)
