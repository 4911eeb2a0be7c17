"""GPU parity of the attend kernel's head-block variants (8 blocks of 16
heads, 4 for at most 64 heads, 2 for at most 32) on both sides of each line,
for every cache format and at step and page edges, dense and over listed
positions, against the fp64 oracle with the parity bar of the dense tests
(bf16 rounding of the output and of the weights)."""
import dataclasses
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_2609_37626_amd import binding as B
from paper_2609_37626_amd import workloads as W
from paper_2609_37626_amd.device import to_device

pytestmark = pytest.mark.gpu

OUT_TOL = {W.KV_BF16: 1e-2, W.KV_FP8_E4M3: 3e-2, W.KV_FP8_LATENT: 3e-2}
LSE_TOL = 1e-3


def check(batch, out, lse, ref):
    assert np.abs(out.float().cpu().numpy() - ref[0]).max() <= OUT_TOL[batch.kv_dtype]
    assert np.abs(lse.cpu().numpy() - ref[1]).max() <= LSE_TOL


@pytest.mark.parametrize("kv", [W.KV_BF16, W.KV_FP8_E4M3, W.KV_FP8_LATENT])
@pytest.mark.parametrize("heads", [16, 32, 48, 64, 80])
@pytest.mark.parametrize("q", [1, 3])
def test_head_blocks(heads, kv, q):
    # single steps, step and page edges, a run of several pages; split too
    batch = W.make_custom([3, 31, 32, 33, 64, 65, 97, 700], H=heads, q_chunk=q, kv_dtype=kv, seed=heads + q)
    ref = oracle.mla_attention(batch.q, batch.kv, batch.block_table, batch.seq_lens, q, batch.softmax_scale,
                               kv_dtype=kv, kv_scales=batch.kv_scales)
    db = to_device(batch)
    for flags, pages in ((0, 0), (B.FLAG_FORCE_SPLIT, 3)):
        out, lse = db.attend(flags=flags, split_pages=pages)
        check(batch, out, lse, ref)


@pytest.mark.parametrize("kv", [W.KV_BF16, W.KV_FP8_E4M3, W.KV_FP8_LATENT])
@pytest.mark.parametrize("heads", [32, 64])
def test_head_blocks_listed_positions(heads, kv):
    batch = W.make_custom([40, 200, 500], H=heads, kv_dtype=kv, seed=heads)
    rng = np.random.Generator(np.random.PCG64(heads))
    topk, counts = 96, [33, 96, 1]
    idx = np.zeros((3, topk), np.int32)
    for n, (s, c) in enumerate(zip(batch.seq_lens, counts)):
        idx[n, :c] = np.sort(rng.choice(int(s), size=c, replace=False))
    count = np.asarray(counts, np.int32)
    ref = oracle.mla_attention_topk(batch.q, batch.kv, batch.block_table, batch.seq_lens, 1, batch.softmax_scale, idx,
                                    count, kv_dtype=kv, kv_scales=batch.kv_scales)
    db = to_device(batch)
    out, lse = db.alloc_outputs()
    B.splash_mla_attend_topk(db.q, db.kv, db.block_table, db.seq_lens, 1, torch.from_numpy(idx).cuda(),
                             torch.from_numpy(count).cuda(), out, lse, db.desc(), db.workspace())
    torch.cuda.synchronize()
    check(batch, out, lse, ref)


@functools.lru_cache(maxsize=1)
def many_tiles(kv, q):
    # more tiles than workers, of differing lengths: a worker runs several units,
    # longest first (with query chunks a request's side by side)
    rng = np.random.default_rng(q)
    lengths = rng.integers(3, 131, 270) if q == 1 else rng.integers(q, 700, 40)
    batch = W.make_custom(lengths, H=64, q_chunk=q, kv_dtype=kv, seed=q)
    return batch, oracle.mla_attention(batch.q, batch.kv, batch.block_table, batch.seq_lens, q, batch.softmax_scale,
                                       kv_dtype=kv, kv_scales=batch.kv_scales)


@pytest.mark.parametrize("q,kv,heads", [(q, kv, heads) for q in (1, 8)
                                        for kv in (W.KV_BF16, W.KV_FP8_E4M3, W.KV_FP8_LATENT) for heads in (32, 64)])
def test_head_blocks_several_units_a_worker(q, kv, heads):
    batch, ref = many_tiles(kv, q)
    assert len(ref[0]) > B.device_workers()
    few = dataclasses.replace(batch, q=np.ascontiguousarray(batch.q[:, :heads]), H=heads)
    out, lse = to_device(few).attend()
    check(few, out, lse, (ref[0][:, :heads], ref[1][:, :heads]))
