"""The work that a serving program has this library do, as measurable cases.

Each case is a dict of plain sizes.  `prepare` makes what such a program
holds before the call (the paged cache, the block table, the queries, the
workspace), on the GPU and from a seed; `run` is one pass through the entry
points of `paper_2609_37626_amd.binding`; `exact` is the same result in
float64 from plain torch.

Kinds of work:
  attend  one decode step of one layer (splash_mla_attend): plan, attention,
          merge of the split histories
  layers  one decode step of several layers: one splash_mla_plan and one
          splash_mla_run per layer, each with its own cache and queries
  topk    one sparse step (splash_mla_attend_topk): every row attends the
          positions its indexer listed
  shard   one rank of a position-sharded group: its own partial result
          (splash_mla_attend_shard), then the merge of the group's partials
          (splash_mla_combine)
  dop     one GPU's regroup of query and output rows around the attention
          (the four splash_dop_* calls)

Lengths are drawn from the case's own `lengths_seed` (so a case has one
amount of work) and dealt to the requests in an order made from the seed of
`prepare`, which also makes every value, the page placement and the lists.
"""
import math
import random

import torch

from paper_2609_37626_amd import binding as B

PAGE, DIM_QK, DIM_V = 64, 576, 512
SCALE = 1.0 / math.sqrt(192.0)
KV = {"bf16": B.KV_BF16, "fp8": B.KV_FP8_E4M3, "latent": B.KV_FP8_LATENT}
ROW_BYTES = {"bf16": 2 * DIM_QK, "fp8": DIM_QK + 4, "latent": 656}


def _case(kind, batch, heads, q_chunk, kv, lengths, lo, hi, lengths_seed, **more):
    return dict({"kind": kind, "batch": batch, "heads": heads, "q_chunk": q_chunk, "kv": kv, "lengths": lengths,
                 "lo": lo, "hi": hi, "lengths_seed": lengths_seed}, **more)


def listed():
    return [
        # the smallest call: a few short requests on a rank that holds 16 of
        # the heads; latency and launches
        dict(_case("attend", 4, 16, 1, "bf16", "uniform", 128, 512, 0), name="tiny_h16"),
        # the data-parallel decode regime: a large batch of short requests
        dict(_case("attend", 256, 128, 1, "bf16", "uniform", 1024, 4096, 1), name="many_short"),
        # the long-reasoning tail: a few very long histories, split over the chip
        dict(_case("attend", 4, 128, 1, "bf16", "uniform", 65536, 131072, 2), name="few_long"),
        # a batch in transition from short to long histories
        dict(_case("attend", 64, 128, 1, "bf16", "lognormal", 64, 131072, 3), name="ragged"),
        # eight causal query tokens per request over the per-token fp8 cache
        dict(_case("attend", 16, 128, 8, "fp8", "uniform", 8192, 32768, 4), name="chunk8_fp8"),
        # speculative decoding (two rows per request) over the fp8 latent rows
        dict(_case("attend", 48, 128, 2, "latent", "lognormal", 64, 32768, 5), name="spec2_latent"),
        # a rank that holds 16 of the heads, speculative decoding, fp8 cache
        dict(_case("attend", 96, 16, 2, "fp8", "uniform", 512, 8192, 6), name="heads16_fp8"),
        # one plan for the layers of a step, half the heads
        dict(_case("layers", 32, 64, 1, "bf16", "uniform", 512, 4096, 7, layers=3), name="layers_h64"),
        # sparse attention over the bf16 cache, 2,048 listed positions per row
        dict(_case("topk", 256, 128, 1, "bf16", "uniform", 1024, 4096, 1, topk=2048), name="topk_bf16"),
        # sparse attention over latent rows, speculative decoding
        dict(_case("topk", 64, 128, 2, "latent", "uniform", 2048, 32768, 8, topk=2048), name="topk_latent"),
        # one rank of four that share long histories by position
        dict(_case("shard", 4, 128, 1, "bf16", "uniform", 65536, 131072, 2, shards=4, shard=1), name="shard_few_long"),
        # the regroup around a decode step's attention, 8 ranks
        {"kind": "dop", "rows": 256, "ranks": 8, "heads": 128, "name": "dop_256"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: sizes over their logarithm."""
    kind = rng.choices(["attend", "layers", "topk", "shard", "dop"], [60, 10, 15, 8, 7])[0]
    if kind == "dop":
        ranks = rng.choice([2, 4, 8])
        return {"kind": "dop", "rows": _log_int(rng, 16, 512 * ranks), "ranks": ranks, "heads": 128}
    heads = rng.choices([128, 16, 32, 64, rng.randrange(3, 8) * 16], [45, 20, 10, 15, 10])[0]
    q = rng.choices([1, 2, rng.randrange(3, 9)], [60, 20, 20])[0]
    kv = rng.choice(["bf16", "fp8", "latent"])
    lengths = rng.choice(["uniform", "lognormal"])
    lo = _log_int(rng, 64, 16384)
    hi = max(2 * lo, _log_int(rng, 512, 131072))
    more = {}
    if kind == "layers":
        more["layers"] = rng.randrange(2, 5)
    elif kind == "topk":
        # (a larger list goes past 2,048 entries: split lists)
        more["topk"] = rng.choice([512, 1000, 2048, 2048, 3000])
        hi = min(hi, 32768)
        lo = min(lo, hi // 2)
    elif kind == "shard":
        more["shards"] = rng.choice([2, 4, 8])
        more["shard"] = rng.randrange(more["shards"])
    elif kv != "bf16" and rng.random() < 0.15:
        more["exact_qk"] = True
    batch = _log_int(rng, 1, 256)
    seed = rng.randrange(1 << 30)
    while True:
        case = _case(kind, batch, heads, q, kv, lengths, lo, hi, seed, **more)
        w = work(case)
        pool = sum(-(-s // PAGE) for s in _lengths(case)) * PAGE * ROW_BYTES[kv] * more.get("layers", 1)
        # no larger than the largest listed ones
        if (w["bytes"] <= 8.0e8 and w["flops"] <= 8.0e11 and pool <= 2.0e9 and batch * q <= 2048) or batch == 1:
            if w["flops"] <= 8.0e11 and w["bytes"] <= 8.0e8:
                return case
            hi = max(64 + q, hi // 2)
            lo = min(lo, hi // 2 + q)
        batch = max(1, batch // 2)


# ---------------------------------------------------------------- sizes --

def _lengths(case):
    rng = random.Random(case["lengths_seed"])
    lo, hi = max(case["lo"], case["q_chunk"]), max(case["hi"], case["q_chunk"])
    if case["lengths"] == "uniform":
        return [rng.randint(lo, hi) for _ in range(case["batch"])]
    return [min(max(round(rng.lognormvariate(8.0, 1.5)), lo), hi) for _ in range(case["batch"])]


def _shard_range(case, s):
    pages, n, k = -(-s // PAGE), case["shards"], case["shard"]
    return min(s, pages * k // n * PAGE), min(s, pages * (k + 1) // n * PAGE)


def work(case):
    if case["kind"] == "dop":
        rows = case["rows"] * case["heads"] // case["ranks"]   # one rank's rows, and as an owner as many
        return {"bytes": 2 * 2 * rows * 2 * (DIM_QK + DIM_V), "flops": 0}
    H, q, row = case["heads"], case["q_chunk"], ROW_BYTES[case["kv"]]
    lens = _lengths(case)
    n = len(lens) * q
    keys = visible = 0
    for s in lens:
        lo, hi = 0, s
        if case["kind"] == "shard":
            lo, hi = _shard_range(case, s)
        if case["kind"] == "topk":
            counts = [min(case["topk"], s - q + i + 1) for i in range(q)]
            keys += min(s, sum(counts))
            visible += sum(counts)
        else:
            keys += hi - lo
            visible += sum(max(0, min(hi, s - q + i + 1) - lo) for i in range(q))
    io = n * H * (2 * DIM_QK + 2 * DIM_V + 4)
    if case["kind"] == "shard":
        # the own partial written, the group's partials read, the result written
        io = n * H * (2 * DIM_QK + 4 * (DIM_V + 1) * (1 + case["shards"]) + 2 * DIM_V + 4)
    elif case["kind"] == "topk":
        io += n * case["topk"] * 4
    layers = case.get("layers", 1)
    table = sum(-(-s // PAGE) for s in lens) * 4
    return {"bytes": layers * (keys * row + io + table), "flops": layers * 2 * H * (DIM_QK + DIM_V) * visible}


# --------------------------------------------------------------- inputs --

def _pool(gen, num_pages, kv):
    """N(0, 1) cache rows in the cache's format, and the per-token scales."""
    x = torch.randn((num_pages, PAGE, DIM_QK), generator=gen, device="cuda", dtype=torch.float32)
    if kv == "bf16":
        return x.bfloat16(), None
    if kv == "fp8":
        scale = x.abs().amax(-1) / 448.0
        codes = (x / scale[..., None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
        return codes.view(torch.uint8), scale.contiguous()
    # latent rows: 512 codes, four power-of-two tile scales, 64 bf16 RoPE
    tiles = x[..., :DIM_V].reshape(num_pages, PAGE, 4, 128)
    u = torch.randint(-3, 1, (num_pages, PAGE, 4), generator=gen, device="cuda")
    tiles = tiles * torch.exp2(u.float())[..., None]
    scale = torch.exp2(torch.ceil(torch.log2(tiles.abs().amax(-1) / 448.0)))
    codes = (tiles / scale[..., None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
    out = torch.empty((num_pages, PAGE, 656), dtype=torch.uint8, device="cuda")
    out[..., :512] = codes.view(torch.uint8).reshape(num_pages, PAGE, 512)
    out[..., 512:528] = scale.contiguous().view(torch.uint8)
    out[..., 528:] = x[..., DIM_V:].bfloat16().contiguous().view(torch.uint8)
    return out, None


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).bfloat16()

    if case["kind"] == "dop":
        n, T, H = case["rows"], case["ranks"], case["heads"]
        hl, own = H // T, max(1, n // T)
        return {"kind": "dop", "ranks": T,
                "q_nope": randn(n, hl, DIM_V), "q_rope": randn(n, hl, DIM_QK - DIM_V),
                "order": torch.randperm(n, generator=gen, device="cuda").int(),
                "recv_q": randn(T, own, hl, DIM_QK), "out_owner": randn(own, H, DIM_V), "recv_out": randn(n, hl, DIM_V),
                "send_q": torch.empty((n, hl, DIM_QK), dtype=torch.bfloat16, device="cuda"),
                "q_owner": torch.empty((own, H, DIM_QK), dtype=torch.bfloat16, device="cuda"),
                "send_out": torch.empty((T, own, hl, DIM_V), dtype=torch.bfloat16, device="cuda"),
                "out": torch.empty((n, hl, DIM_V), dtype=torch.bfloat16, device="cuda")}

    lens = _lengths(case)
    random.Random(seed).shuffle(lens)
    b, H, q, kv = len(lens), case["heads"], case["q_chunk"], case["kv"]
    n = b * q
    pages = [-(-s // PAGE) for s in lens]
    num_pages, max_pages = sum(pages), max(pages)
    perm = torch.randperm(num_pages, generator=gen, device="cuda").int().cpu()
    table = torch.full((b, max_pages), -1, dtype=torch.int32)
    off = 0
    for i, p in enumerate(pages):
        table[i, :p] = perm[off:off + p]
        off += p
    st = {"kind": case["kind"], "lens": lens, "q_chunk": q, "heads": H, "kv_format": kv,
          "seq": torch.tensor(lens, dtype=torch.int32).cuda(), "table": table.cuda()}
    st["layers"] = []
    for _ in range(case.get("layers", 1)):
        pool, scales = _pool(gen, num_pages, kv)
        st["layers"].append({
            "kv": pool, "scales": scales, "q": randn(n, H, DIM_QK),
            "out": torch.empty((n, H, DIM_V), dtype=torch.bfloat16, device="cuda"),
            "lse": torch.empty((n, H), dtype=torch.float32, device="cuda"),
            "desc": B.make_desc(b, H, max_pages, num_pages, KV[kv], scales, SCALE,
                                B.FLAG_EXACT_QK if case.get("exact_qk") else 0)})
    # room for the default 1,024 partials, for those that histories past 1,024
    # pages or lists past 2,048 entries force, and for a shard's row each
    partials = max(1024, n * -(-max_pages // 1024) if max_pages > 1024 else 0)
    if case["kind"] == "topk":
        k = case["topk"]
        partials = max(partials, n * -(-k // 2048))
        vis = torch.tensor([s - q + i + 1 for s in lens for i in range(q)], device="cuda")
        idx = torch.zeros((n, k), dtype=torch.int32, device="cuda")
        for r0 in range(0, n, 64):   # distinct positions of the visible prefix, in position order
            v = vis[r0:r0 + 64]
            score = torch.rand((v.numel(), max(max(lens), k)), generator=gen, device="cuda")
            score.masked_fill_(torch.arange(score.shape[1], device="cuda")[None] >= v[:, None], 2.0)
            pos = score.topk(k, dim=1, largest=False).indices
            idx[r0:r0 + 64] = torch.where(pos < v[:, None], pos, 1 << 30).sort(dim=1).values.int()
        st["count"] = vis.clamp(max=k).int()
        st["idx"] = torch.where(torch.arange(k, device="cuda")[None] < st["count"][:, None], idx, 0).int().contiguous()
    elif case["kind"] == "shard":
        ns, me = case["shards"], case["shard"]
        partials = max(partials, n)
        rng_ = [_shard_range(case, s) for s in lens]
        st["begin"] = torch.tensor([r[0] for r in rng_], dtype=torch.int32).cuda()
        st["end"] = torch.tensor([r[1] for r in rng_], dtype=torch.int32).cuda()
        # the other ranks' partials, as they arrive: outputs and LSEs of the
        # size that their keys give
        keys = torch.tensor([max(1, s // ns) for s in lens], device="cuda").float()
        st["part"] = torch.randn((b * ns, q, H, DIM_V), generator=gen, device="cuda") / keys.sqrt().repeat_interleave(ns)[:, None, None, None]
        st["part_lse"] = (torch.randn((b * ns, q, H), generator=gen, device="cuda") * 0.1
                          + (keys.log() + 1.5).repeat_interleave(ns)[:, None, None])
        st["shards"], st["shard"] = ns, me
        st["indptr"] = torch.arange(b + 1, dtype=torch.int32, device="cuda") * ns
    st["ws"] = torch.empty(B.workspace_size(b, q, H, partials), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    if st["kind"] == "dop":
        B.splash_dop_pack_q(st["q_nope"], st["q_rope"], st["order"], st["send_q"])
        B.splash_dop_unpack_q(st["recv_q"], st["ranks"], st["q_owner"])
        B.splash_dop_pack_out(st["out_owner"], st["ranks"], st["send_out"])
        B.splash_dop_unpack_out(st["recv_out"], st["order"], st["out"])
        return {k: st[k] for k in ("send_q", "q_owner", "send_out", "out")}
    L = st["layers"][0]
    if st["kind"] == "attend":
        B.splash_mla_attend(L["q"], L["kv"], st["table"], st["seq"], st["q_chunk"], L["out"], L["lse"], L["desc"], st["ws"])
    elif st["kind"] == "topk":
        B.splash_mla_attend_topk(L["q"], L["kv"], st["table"], st["seq"], st["q_chunk"], st["idx"], st["count"],
                                 L["out"], L["lse"], L["desc"], st["ws"])
    elif st["kind"] == "layers":
        B.splash_mla_plan(st["seq"], st["q_chunk"], L["desc"], st["ws"])
        for l in st["layers"]:
            B.splash_mla_run(l["q"], l["kv"], st["table"], st["seq"], st["q_chunk"], l["out"], l["lse"], l["desc"], st["ws"])
        return [(l["out"], l["lse"]) for l in st["layers"]]
    else:
        ns, me = st["shards"], st["shard"]
        B.splash_mla_attend_shard(L["q"], L["kv"], st["table"], st["seq"], st["q_chunk"], st["begin"], st["end"], ns, me,
                                  st["part"], st["part_lse"], L["desc"], st["ws"])
        B.splash_mla_combine(st["part"], st["part_lse"], st["indptr"], len(st["lens"]), st["q_chunk"], st["heads"],
                             L["out"], L["lse"])
        return st["part"][me::ns], st["part_lse"][me::ns], L["out"], L["lse"]
    return L["out"], L["lse"]


# ------------------------------------------------------------ the result --

def tolerance(case):
    """2-norm of the outputs' error over their norm: about four times what the
    path shows against float64, 1.7e-3 to 2.3e-3 for every cache format (the
    bf16 rounding of the weights and of the output; the LSEs show 1e-7)."""
    if case["kind"] == "dop":
        return "exact"
    return {"rel": 1e-2}


def _rows(st, layer, req):
    """The history of request `req`, float64 [s, 576]."""
    s = st["lens"][req]
    pages = st["table"][req, :-(-s // PAGE)].long()
    rows = layer["kv"][pages].reshape(-1, layer["kv"].shape[-1])[:s]
    if st["kv_format"] == "bf16":
        return rows.double()
    if st["kv_format"] == "fp8":
        return rows.contiguous().view(torch.float8_e4m3fn).double() * layer["scales"][pages].reshape(-1)[:s].double()[:, None]
    lat = rows[:, :512].contiguous().view(torch.float8_e4m3fn).double().reshape(s, 4, 128)
    lat = lat * rows[:, 512:528].contiguous().view(torch.float32).double()[..., None]
    return torch.cat([lat.reshape(s, 512), rows[:, 528:].contiguous().view(torch.bfloat16).double()], dim=1)


def _softmax_values(z, k):
    lse = torch.logsumexp(z, -1)
    w = torch.exp(z - torch.where(torch.isinf(lse), 0.0, lse)[..., None])
    return w @ k[:, :DIM_V], lse


def _attention(st, layer):
    """Attention of every row over its visible (listed, own) keys."""
    q, H = st["q_chunk"], st["heads"]
    scale = float(torch.tensor(SCALE, dtype=torch.float32))
    out = torch.empty(layer["out"].shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(layer["lse"].shape, dtype=torch.float64, device="cuda")
    for r, s in enumerate(st["lens"]):
        k = _rows(st, layer, r)
        for i in range(q):
            n = r * q + i
            query = layer["q"][n].double()
            if st["kind"] == "topk":
                keys = k[st["idx"][n, :int(st["count"][n])].long()]
            else:
                lo, hi = 0, s - q + i + 1
                if st["kind"] == "shard":
                    lo, hi = int(st["begin"][r]), min(hi, int(st["end"][r]))
                keys = k[lo:max(lo, hi)]
            if keys.shape[0] == 0:
                out[n], lse[n] = 0.0, -math.inf
                continue
            out[n], lse[n] = _softmax_values(query @ keys.T * scale, keys)
    return out, lse


def exact(case, seed):
    st = prepare(case, seed)
    if st["kind"] == "dop":
        T, n = st["ranks"], st["recv_q"].shape[1]
        order = st["order"].long()
        out = torch.empty_like(st["out"])
        out[order] = st["recv_out"]
        hl = st["out"].shape[1]
        return {"send_q": torch.cat([st["q_nope"][order], st["q_rope"][order]], dim=2).double(),
                "q_owner": st["recv_q"].permute(1, 0, 2, 3).reshape(n, T * hl, DIM_QK).double(),
                "send_out": st["out_owner"].reshape(n, T, hl, DIM_V).permute(1, 0, 2, 3).double().contiguous(),
                "out": out.double()}
    res = [_attention(st, layer) for layer in st["layers"]]
    if st["kind"] == "layers":
        return res
    if st["kind"] == "shard":
        b, q, H, ns, me = len(st["lens"]), st["q_chunk"], st["heads"], st["shards"], st["shard"]
        own, own_lse = res[0][0].reshape(b, q, H, DIM_V), res[0][1].reshape(b, q, H)
        part = st["part"].double().reshape(b, ns, q, H, DIM_V)
        pl = st["part_lse"].double().reshape(b, ns, q, H)
        part[:, me], pl[:, me] = own, own_lse
        lse = torch.logsumexp(pl, 1)
        out = (torch.exp(pl - lse[:, None])[..., None] * part).sum(1)
        return own, own_lse, out.reshape(b * q, H, DIM_V), lse.reshape(b * q, H)
    return res[0]
