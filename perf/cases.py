"""The work this library is asked to do, as a list of cases that can be timed and compared.

A case is a dict of plain values.  `prepare` builds what a serving program holds before the call (the paged cache, its
metadata, the queries, workspaces and output buffers), `run` is one pass through the public entry points, `work` counts
the bytes and operations the pass cannot do without (`selected`, the share of the blocks the stop rule selects, is measured and
used there only), `tolerance` says how far two correct implementations may be apart.

The caches hold what the path meets in earnest (the recipe of workloads/generator.py, drawn here for all heads at
once): queries of a group share a direction, background keys are N(0, 1), and a few "critical" tokens -- the first 16,
the last 64 and runs of 1 to 16 tokens covering a fraction f of the rest -- are moved along that direction, so that they
carry most of the attention mass.  "flat" caches have no such tokens and small keys: nothing can be skipped.
"""
import math

import torch

import paper_2503_00392_amd as psa

PAGE, DIM, SLICE = 16, 128, 4096       # tokens of a block, channels of a head, bytes of a block's keys of one head
TYPES = {"f16": torch.float16, "bf16": torch.bfloat16}
CHUNK = 1 << 28                        # elements drawn at a time


def _case(name, op, dtype, batch, kv_heads, group, ctx, ctx_min=0, eps=0.95, frac=0.02, frac_hi=0.0, layers=1,
          table="random", scorer="bound", selected=0.3, k=0, m=1, slots=0):
    c = {"op": op, "dtype": dtype, "batch": batch, "kv_heads": kv_heads, "group": group, "ctx": ctx,
         "ctx_min": ctx_min or ctx, "eps": eps, "frac": frac, "frac_hi": frac_hi or frac, "layers": layers, "table": table,
         "scorer": scorer, "selected": selected, "k": k, "m": m, "slots": slots}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one short request: five dependent launches, nothing but latency
        _case("decode_4k_b1", "decode", "f16", 1, 8, 4, 4096, eps=0.90, frac=0.01, table="packed", selected=0.065),
        # an ordinary serving batch of one layer
        _case("decode_32k_b8", "decode", "f16", 8, 8, 4, 32768, frac=0.005, frac_hi=0.10, table="packed", selected=0.24),
        # several layers of a long-context model step, each with its own share of critical tokens
        _case("decode_128k_b4_layers", "decode", "bf16", 4, 8, 4, 131072, frac=0.002, frac_hi=0.20, layers=4, selected=0.30),
        # a large ragged batch, eight query heads to a KV head, a high threshold
        _case("decode_ragged_b64_g8", "decode", "f16", 64, 8, 8, 131072, ctx_min=4096, eps=0.98, frac=0.02, selected=0.59),
        # attention without critical tokens: nearly everything is selected
        _case("decode_flat_64k_b16", "decode", "bf16", 16, 8, 4, 65536, frac=0.0, selected=0.95, table="packed"),
        # as many KV heads as query heads
        _case("decode_mha_32k_b2", "decode", "bf16", 2, 32, 1, 32768, frac=0.005, frac_hi=0.10, selected=0.18),
        # a step of a decode loop: lengths from the scheduler, a token appended to every request, then attention with what
        # the previous step read as the hint
        _case("loop_ragged_16k_b24", "loop", "bf16", 24, 8, 4, 16384, ctx_min=513, frac=0.02, selected=0.19),
        # the fixed budget
        _case("topk128_32k_b8", "topk", "f16", 8, 8, 4, 32768, frac=0.005, frac_hi=0.10, k=128),
        # dense attention over the same layout
        _case("dense_ragged_64k_b6", "dense", "bf16", 6, 8, 4, 65536, ctx_min=9999),
        # metadata of freshly prefilled pages
        _case("metadata_64k_b2", "metadata", "bf16", 2, 8, 4, 65536),
        # mean-key metadata and its scorer, fewer heads, odd lengths, the rule tested every four blocks
        _case("mean_key_ragged_24k_b12", "decode", "bf16", 12, 4, 2, 24001, ctx_min=2005, frac=0.02, scorer="mean", m=4,
              selected=0.21),
        # two tiers: the cache in pinned host memory, a pool of slots on the GPU, four steps with drifting queries
        _case("tier_32k_b2", "tier", "bf16", 2, 8, 4, 32768, frac=0.02, slots=10000, selected=0.25),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode"] * 6 + ["loop"] * 2 + ["topk", "dense", "metadata", "tier"])
    dtype = rng.choice(["f16", "bf16"])
    heads = rng.choice([1, 2, 4, 5, 8, 8, 8, 16, 32])
    group = rng.choice([g for g in (1, 2, 4, 4, 8, 8) if g * heads <= 64])
    ctx = _log(rng, 300, 131072)
    if op == "tier":
        ctx = _log(rng, 2048, 32768)
    # at most 4 GiB of keys and values (256 MiB in host memory)
    most = (1 << 28 if op == "tier" else 1 << 32) // (ctx * heads * 4 * DIM)
    batch = _log(rng, 1, max(1, min(64, most)))
    lo = ctx if rng.random() < 0.3 else max(1, _log(rng, max(1, ctx // 32), ctx))
    eps = rng.choice([0.90, 0.95, 0.95, 0.98])
    flat = op == "decode" and rng.random() < 0.15
    frac = 0.0 if flat else _log(rng, 20, 1000) / 10000.0
    scorer = rng.choice(["bound"] * 4 + ["center", "mean"]) if op in ("decode", "topk") else "bound"
    blocks = batch * ((ctx + PAGE - 1) // PAGE)
    return _case("", op, dtype, batch, heads, group, ctx, ctx_min=lo, eps=eps, frac=frac, scorer=scorer,
                 table=rng.choice(["random", "packed"]), selected=0.95 if flat else 0.3,
                 k=rng.choice([16, 64, 100, 128, 256]) if op == "topk" else 0, m=rng.choice([1, 1, 4]),
                 slots=max(64, blocks * heads // 4) if op == "tier" else 0)


# ---- what a case's numbers mean ---------------------------------------------------------------------------------

def _lengths(case):
    """Context lengths, log-uniform between ctx_min and ctx, the longest among them."""
    lo, hi, n = case["ctx_min"], case["ctx"], case["batch"]
    spread = [hi] + [int(round(lo * (hi / lo) ** ((0.25 + 0.6180339887 * i) % 1.0))) for i in range(1, n)]
    return spread[:n]


def _blocks(tokens):
    return (tokens + PAGE - 1) // PAGE


def _layer_fractions(case):
    """Share of critical tokens per layer, spread evenly over the logarithm of the range (one layer: per head instead)."""
    n, lo, hi = case["layers"], case["frac"], case["frac_hi"]
    return [lo * (hi / lo) ** ((i + 0.5) / n) if lo > 0 else 0.0 for i in range(n)]


def work(case):
    B, H, G, L = case["batch"], case["kv_heads"], case["group"], case["layers"]
    lens = _lengths(case)
    N = sum(_blocks(t) for t in lens)
    once = N * 4 + B * 4 + B * H * G * (DIM * 2 + DIM * 4 + 12)      # table, lengths, queries, outputs
    record = 256 if case["scorer"] == "mean" else 512
    if case["op"] == "metadata":
        return {"bytes": N * H * (SLICE + 512), "flops": N * H * PAGE * DIM * 2}
    if case["op"] == "dense":
        return {"bytes": once + sum(lens) * H * DIM * 4, "flops": sum(lens) * H * G * DIM * 4}
    if case["op"] == "topk":
        read = sum(min(case["k"], _blocks(t)) for t in lens)
    else:
        read = max(B, case["selected"] * N)
    bytes_ = once + N * H * record + read * H * 2 * SLICE
    flops = N * H * G * DIM * (2 if case["scorer"] == "mean" else 4) + read * H * G * PAGE * DIM * 4
    if case["op"] == "tier":
        return {"bytes": 4 * bytes_, "flops": 4 * flops}
    return {"bytes": L * bytes_, "flops": L * flops}


def tolerance(case):
    if case["op"] == "metadata":
        return "exact"
    # Binary32 sums in another order (chunks of another size): up to 4e-6 and, where a head whose P_acc sits on the
    # threshold stops a block earlier or later, 6e-4 on a value; at most 3 stops of 4096 differed.
    return {"rel": 2e-5, "max": 2.5e-3, "differ": 0.005}


# ---- inputs -----------------------------------------------------------------------------------------------------

def _critical(lens, heads, fracs, gen, dev):
    """[B][heads][longest] critical tokens."""
    B, T = len(lens), max(lens)
    mask = torch.zeros((B, heads, T + 1), dtype=torch.int32, device=dev)
    for r, n in enumerate(lens):
        mid = n - 80
        if mid > 0:
            most = max(1, int(round(max(fracs) * mid / 8.5)))
            starts = torch.randint(16, 16 + mid, (heads, most), generator=gen, device=dev)
            ends = (starts + torch.randint(1, 17, (heads, most), generator=gen, device=dev)).clamp_(max=16 + mid)
            runs = torch.tensor([max(1, int(round(f * mid / 8.5))) for f in fracs], device=dev)
            on = (torch.arange(most, device=dev)[None, :] < runs[:, None]).to(torch.int32)
            mask[r].scatter_add_(1, starts, on)
            mask[r].scatter_add_(1, ends, -on)
    mask = torch.cumsum(mask[:, :, :T], 2) > 0
    for r, n in enumerate(lens):
        mask[r, :, :16] = True
        mask[r, :, max(0, n - 64):] = True
        mask[r, :, n:] = False
    return mask


def _normal(shape, dtype, gen, dev, scale=1.0):
    x = torch.empty(shape, dtype=dtype, device=dev)
    flat = x.view(-1)
    for a in range(0, flat.numel(), CHUNK):
        flat[a:a + CHUNK].normal_(0.0, scale, generator=gen)
    return x


class State:
    pass


def _layer(case, layer, gen, room=0):
    """One layer's cache: (KvCache, queries, metadata); `room` more tokens fit every request's row of the table."""
    dev, dt = "cuda", TYPES[case["dtype"]]
    B, H, G = case["batch"], case["kv_heads"], case["group"]
    lens = _lengths(case)
    blocks = [_blocks(t + room) for t in lens]
    total, width = sum(blocks), max(blocks)
    perm = torch.randperm(total, generator=gen, device=dev) if case["table"] == "random" else torch.arange(total, device=dev)
    table = torch.zeros((B, width), dtype=torch.int32, device=dev)
    fill = torch.zeros(total, dtype=torch.int32, device=dev)
    at = 0
    for r, n in enumerate(blocks):
        table[r, :n] = perm[at:at + n].to(torch.int32)
        valid = (lens[r] - PAGE * torch.arange(n, device=dev)).clamp(0, PAGE)
        fill[perm[at:at + n]] = valid.to(torch.int32)
        at += n
    flat = case["frac"] == 0.0 and case["frac_hi"] == 0.0
    k = _normal((total, H, PAGE, DIM), dt, gen, dev, 0.1 if flat else 1.0)
    v = _normal((total, H, PAGE, DIM), dt, gen, dev)
    q = torch.randn((B, H, G, DIM), generator=gen, device=dev)
    if not flat:
        way = torch.randn((B, H, DIM), generator=gen, device=dev)
        way = way / way.norm(dim=2, keepdim=True)
        q += math.sqrt(DIM) * way[:, :, None, :]
        if case["layers"] > 1:
            fracs = [_layer_fractions(case)[layer]] * H
        else:                                             # spread over the heads
            lo, hi = case["frac"], case["frac_hi"]
            fracs = [lo * (hi / lo) ** ((h + 0.5) / H) for h in range(H)]
        mask = _critical(lens, H, fracs, gen, dev)
        for r in range(B):
            h, t = mask[r].nonzero(as_tuple=True)
            page = table[r].long()[t // PAGE]
            for a in range(0, h.numel(), 1 << 21):
                i = (page[a:a + (1 << 21)], h[a:a + (1 << 21)], t[a:a + (1 << 21)] % PAGE)
                k[i] = (k[i].float() + 6.0 * way[r, i[1]]).to(dt)
    kv = psa.KvCache(k, v, table, torch.tensor(lens, dtype=torch.int32, device=dev), H * G)
    if case["scorer"] == "mean":
        meta = psa.build_block_means(kv, page_fill=fill)
    else:
        meta = psa.build_block_metadata(kv, page_fill=fill)
    return kv, q.view(B, H * G, DIM).to(dt).contiguous(), meta, fill


def _outputs(kv, order=False):
    B, Hq, H, MB = kv.block_table.shape[0], kv.num_q_heads, kv.k_pool.shape[1], kv.block_table.shape[1]
    new = lambda shape, dt: torch.zeros(shape, dtype=dt, device="cuda")      # noqa: E731
    return psa.DecodeOutput(new((B, Hq, DIM), torch.float32), new((B, Hq), torch.int32), new((B, Hq), torch.float32),
                            new((B, H), torch.int32), new((B, Hq), torch.float32),
                            new((B, H, MB), torch.int32) if order else None, None, None)


def _space(nbytes):
    return torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 7919 + 17)
    s = State()
    s.case, op = case, case["op"]
    s.scorer = {"bound": psa.SCORE_UPPER_BOUND, "center": psa.SCORE_CUBOID_CENTER, "mean": psa.SCORE_MEAN_KEY}[case["scorer"]]
    s.layers = [_layer(case, i, gen, room=1 if op == "loop" else 0) for i in range(case["layers"])]
    kv, q, meta, fill = s.layers[0]
    if op == "metadata":
        return s
    if op == "dense":
        s.workspace = _space(psa.dense_workspace_bytes(kv))
        s.out, s.lse = _outputs(kv).out, _outputs(kv).lse
        return s
    s.workspace = _space(psa.decode_workspace_bytes(kv))
    s.outs = [_outputs(layer[0], order=op == "tier") for layer in s.layers]
    if op == "loop":
        # the step before: its blocks_read is this step's hint; this step's queries differ a little
        first = psa.decode_attention(kv, q, meta, case["eps"], case["m"], workspace=s.workspace)
        s.tuning = psa.Tuning(depth_hint=first.blocks_read)
        s.queries = (q.float() + 0.15 * torch.randn(q.shape, generator=gen, device="cuda")).to(q.dtype)
        s.lens = kv.ctx_lens.clone()
        new = (case["batch"], case["kv_heads"], DIM)
        s.k_new = torch.randn(new, generator=gen, device="cuda").to(q.dtype)
        s.v_new = torch.randn(new, generator=gen, device="cuda").to(q.dtype)
    if op == "tier":
        pools = [torch.empty(p.shape, dtype=p.dtype, pin_memory=True).copy_(p) for p in (kv.k_pool, kv.v_pool)]
        slices = pools[0].shape[0] * pools[0].shape[1]
        s.tier = psa.Tier(slices, min(case["slots"], slices))
        s.kv = psa.KvCache(pools[0], pools[1], kv.block_table, kv.ctx_lens, kv.num_q_heads, tier=s.tier,
                           staging=psa.Tier.staging_buffer(slices))
        s.layers = [(s.kv, None, meta, fill)]
        s.queries, x = [], q.float()
        for _ in range(4):
            s.queries.append(x.to(q.dtype).contiguous())
            x = x + 0.15 * torch.randn(q.shape, generator=gen, device="cuda")
        s.outs = [_outputs(s.kv, order=True) for _ in range(4)]
        s.stats = [torch.zeros(5, dtype=torch.int32, device="cuda") for _ in range(4)]
        s.scratch = _space(psa.tier_update_workspace_bytes(s.kv))
    return s


# ---- one pass ---------------------------------------------------------------------------------------------------

def _result(o):
    return {"out": o.out, "n_selected": o.n_selected, "mass_est": o.mass_est, "blocks_read": o.blocks_read, "lse": o.lse}


def run(s):
    case, op = s.case, s.case["op"]
    kv, q, meta, fill = s.layers[0]
    if op == "decode":
        for (kv, q, meta, _), o in zip(s.layers, s.outs):
            psa.decode_attention(kv, q, meta, case["eps"], case["m"], workspace=s.workspace, outputs=o, scorer=s.scorer)
        return [_result(o) for o in s.outs]
    if op == "loop":
        kv.ctx_lens.copy_(s.lens)
        psa.append_kv(kv, s.k_new, s.v_new, meta)
        psa.decode_attention(kv, s.queries, meta, case["eps"], case["m"], workspace=s.workspace, outputs=s.outs[0],
                             tuning=s.tuning)
        return [_result(s.outs[0]), meta, kv.k_pool, kv.v_pool, kv.ctx_lens]
    if op == "topk":
        psa.topk_attention(kv, q, meta, case["k"], workspace=s.workspace, outputs=s.outs[0], scorer=s.scorer)
        return _result(s.outs[0])
    if op == "dense":
        return psa.dense_attention(kv, q, workspace=s.workspace, out=s.out, lse=s.lse)
    if op == "metadata":
        return psa.build_block_metadata(kv, meta, page_fill=fill)
    for q, o, st in zip(s.queries, s.outs, s.stats):
        psa.decode_attention(kv, q, meta, case["eps"], case["m"], workspace=s.workspace, outputs=o)
        psa.tier_update(kv, o.order, o.blocks_read, stats=st, workspace=s.scratch)
    return [_result(o) for o in s.outs] + [o.order for o in s.outs] + [st for st in s.stats]
