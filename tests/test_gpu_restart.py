"""GPU parity where a unit is redone: a logit more than 64 (base 2) above its
first step's largest makes the workgroup run the unit again from its true
maximum.  Even heads meet keys some 70 to 90 (natural) above the rest, never in
the first step of a unit; odd heads see plain N(0, 1) logits, so that the redone
pass has every key of the unit to get right, and the first pass has left
infinities behind.  The units are those that short parity cases do not reach:
several of a few steps on each worker (the next one's query, pages and first steps
issued before the epilogue), single ones of more than 64 pages (whose page ids are
read again), and lists of 64 steps; every cache format and head-block variant,
the exact QK of the fp8 caches too, and the same units without the outstanding
keys (none redone).  Against the fp64 oracle with the parity bar."""
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

# lengths, query chunk, the forced unit size in pages
SHAPES = {
    # 66 x 5 units of 2 to 4 steps: more units than workers
    "many_units": ([513 + 7 * i % 64 for i in range(66)], 1, 2),
    # units of 79, 65 and 65 pages
    "long_units": ([5000, 8300, 70], 1, 128),
    "chunk": ([900, 330, 2000], 3, 10),
}


def targets(s):
    """Positions of the outstanding keys: never in the first 32 of a page."""
    return np.array([j for j in range(s) if j % 64 >= 32 and j * 2654435761 % 97 == 0 or j == s - 1 and j % 64 >= 32], np.int64)


def outstanding(lengths, q_chunk, kv_dtype, seed, redo):
    batch = W.make_custom(lengths, H=128, q_chunk=q_chunk, kv_dtype=kv_dtype, seed=seed)
    kv, q = batch.kv.copy(), batch.q.copy()
    flat = kv.reshape(-1, kv.shape[-1])
    four = W.f32_to_bf16_bits(np.float32(4.0))
    if kv_dtype == W.KV_FP8_LATENT:
        rope, value = slice(528, 656), np.tile(np.frombuffer(np.uint16(four).tobytes(), np.uint8), 64)
    else:
        rope, value = slice(512, 576), (four if kv_dtype == W.KV_BF16 else np.uint8(0x7E))  # 448 token scales
    flat[:, rope] = 0
    for b, s in enumerate(lengths):
        j = targets(s)
        flat[batch.block_table[b, j // 64].astype(np.int64) * 64 + j % 64, rope] = value
    q[..., 512:] = 0
    if redo:
        q[:, ::2, 512:] = W.f32_to_bf16_bits(np.float32(5.0))
    return dataclasses.replace(batch, kv=kv, q=q)


def check(out, lse, ref, heads, kv_dtype):
    o, l = out.float().cpu().numpy(), lse.cpu().numpy()
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(l))
    # an even head's output is nearly one key's latent, up to 5 in magnitude,
    # and its rounding to bf16 (2^-8 relative) comes on top of the bar, which
    # is for averages of many
    want = ref[0][:, :heads]
    err_o, err_l = (np.abs(o - want) - 2.0 ** -8 * np.abs(want)).max(), np.abs(l - ref[1][:, :heads]).max()
    print(f"out past rounding {err_o:.3e}  lse max-abs {err_l:.3e}", flush=True)
    assert err_o <= OUT_TOL[kv_dtype] and err_l <= LSE_TOL


def first(batch, heads):
    return dataclasses.replace(batch, q=np.ascontiguousarray(batch.q[:, :heads]), H=heads)


@functools.lru_cache(maxsize=1)
def dense_case(shape, kv, redo):
    lengths, q_chunk, _ = SHAPES[shape]
    batch = outstanding(lengths, q_chunk, kv, len(lengths), redo)
    ref = oracle.mla_attention(batch.q, batch.kv, batch.block_table, batch.seq_lens, q_chunk, batch.softmax_scale,
                               kv_dtype=kv, kv_scales=batch.kv_scales)
    return batch, ref


CASES = [(kv, redo, heads) for kv in (W.KV_BF16, W.KV_FP8_E4M3, W.KV_FP8_LATENT)
         for redo, heads in ((True, 16), (True, 32), (True, 64), (True, 128), (False, 32), (False, 64))]


def assert_redone(ref, rows):
    # plain logits stay within 15, the outstanding ones past 15 + 64 ln 2
    assert rows.sum() >= 2 and ref[1][rows, ::2].min() > 15 + 64 * np.log(2) and np.abs(ref[1][:, 1::2]).max() < 15


@pytest.mark.parametrize("shape,kv,redo,heads", [(shape, *case) for shape in SHAPES for case in CASES])
def test_redone_units(shape, kv, redo, heads):
    batch, ref = dense_case(shape, kv, redo)
    if redo:
        assert_redone(ref, np.array([np.any(targets(int(s)) < s - batch.q_chunk + i + 1)
                                     for s in batch.seq_lens for i in range(batch.q_chunk)]))
    db = to_device(first(batch, heads))
    for exact in (0, B.FLAG_EXACT_QK) if kv != W.KV_BF16 else (0,):
        out, lse = db.attend(flags=B.FLAG_FORCE_SPLIT | exact, split_pages=SHAPES[shape][2])
        check(out, lse, ref, heads, kv)


@functools.lru_cache(maxsize=1)
def list_case(kv, redo):
    q_chunk, topk = 2, 2100
    batch = outstanding([2500, 1500], q_chunk, kv, 8, redo)
    rng = np.random.default_rng(8)
    n = batch.B * q_chunk
    idx, count = np.zeros((n, topk), np.int32), np.zeros(n, np.int32)
    for r in range(n):
        s = int(batch.seq_lens[r // q_chunk])
        visible = s - q_chunk + r % q_chunk + 1
        out_of_reach = np.concatenate([targets(s), np.arange(visible, s)])
        plain = rng.permutation(np.setdiff1d(np.arange(visible), out_of_reach))
        mine = targets(s)[targets(s) < visible]
        # in shuffled order, but no target among the first 32 of any 64 entries,
        # so in no unit's first step
        entries = rng.permutation(np.concatenate([plain[:min(topk, visible) - len(mine)], mine]))
        spare = [k for k in range(len(entries)) if k % 64 >= 32 and entries[k] not in set(mine)]
        for k in range(len(entries)):
            if k % 64 < 32 and entries[k] in set(mine):
                p = spare.pop()
                entries[k], entries[p] = entries[p], entries[k]
        idx[r, :len(entries)], count[r] = entries, len(entries)
    ref = oracle.mla_attention_topk(batch.q, batch.kv, batch.block_table, batch.seq_lens, q_chunk, batch.softmax_scale,
                                    idx, count, kv_dtype=kv, kv_scales=batch.kv_scales)
    return batch, idx, count, ref


@pytest.mark.parametrize("kv,redo,heads", CASES)
def test_redone_units_of_listed_positions(kv, redo, heads):
    batch, idx, count, ref = list_case(kv, redo)
    if redo:
        assert_redone(ref, np.ones(len(count), bool))
    db = to_device(first(batch, heads))
    for exact in (0, B.FLAG_EXACT_QK) if kv != W.KV_BF16 else (0,):
        for flags, pages in ((0, 0), (B.FLAG_FORCE_SPLIT, 32)):
            out, lse = db.alloc_outputs()
            B.splash_mla_attend_topk(db.q, db.kv, db.block_table, db.seq_lens, batch.q_chunk,
                                     torch.from_numpy(idx).cuda(), torch.from_numpy(count).cuda(), out, lse,
                                     db.desc(flags | exact, pages), db.workspace())
            torch.cuda.synchronize()
            check(out, lse, ref, heads, kv)
