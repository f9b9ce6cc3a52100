"""Requests that fit one workgroup take one launch instead of four kernels.  Both paths form the same sums in the
same order, so every output has to agree bit for bit; any tuning of the general path selects that path.  Sizes: the
edges of a chunk (32 ranked blocks), of a step of key reads (64) and of the path itself (128 blocks, or up to 256 with
three streams for four blocks)."""
import numpy as np
import pytest
import torch

import gpu_common as gc
from workloads import generate_layer, get_config, step_inputs

pytestmark = pytest.mark.gpu

NAMES = ("out", "n_selected", "mass_est", "blocks_read", "lse", "order", "scores")


@pytest.fixture(scope="module")
def psa():
    import paper_2503_00392_amd as psa
    psa.load_library()
    assert torch.cuda.is_available()
    return psa


def _general(psa):
    return psa.Tuning(spin_limit=1 << 14)            # the default, asked for: the general path


def _layer(G, H, dtype, batch, ctx, ctx_min):
    cfg = get_config(4).scaled(batch=batch, ctx=ctx, ctx_min=ctx_min, num_q_heads=G * H, num_kv_heads=H, dtype=dtype)
    return generate_layer(cfg, device="cuda", poison_tail=True)


def _same(a, b):
    ranked = a.order >= 0                            # scores beyond a request's blocks are not written
    for name in NAMES:
        x, y = getattr(a, name), getattr(b, name)
        if name == "scores":
            x, y = x[torch.sort(ranked, dim=2, descending=True)[0]], y[torch.sort(ranked, dim=2, descending=True)[0]]
        assert torch.equal(x.view(torch.int32), y.view(torch.int32)), name


@pytest.mark.parametrize("G,H,dtype", [(1, 4, "f16"), (2, 8, "bf16"), (4, 2, "f16"), (8, 8, "bf16"), (8, 2, "f16"), (4, 3, "bf16")])
@pytest.mark.parametrize("ctx,ctx_min", [(1, 1), (16 * 31 + 5, 16 * 31 + 5), (512, 17), (513, 513), (1024, 1), (1040, 1025),
                                         (2048, 1500), (2049, 30), (4095, 300), (4096, 1024)])
def test_one_launch_gives_the_general_path_bit_for_bit(psa, G, H, dtype, ctx, ctx_min):
    blocks, batch = (ctx + 15) // 16, 3
    if blocks > 128:                                 # enough streams for the one launch
        H = 16
        batch = (3 * blocks + 4 * H - 1) // (4 * H)
    li = _layer(G, H, dtype, batch, ctx, ctx_min)
    kv = gc.to_kv(li)
    means, boxes = psa.build_block_means(kv, page_fill=li.page_fill), psa.build_block_metadata(kv, page_fill=li.page_fill)
    for eps, m, scorer in [(0.9, 1, 0), (0.95, 4, 2), (0.6, 3, 1), (1.0, 1, 0), (0.0, 50, 2)]:
        meta = means if scorer == 2 else boxes
        args = dict(scorer=scorer, want_order=True, want_scores=True)
        one = psa.decode_attention(kv, li.q, meta, eps, m, **args)
        five = psa.decode_attention(kv, li.q, meta, eps, m, tuning=_general(psa), **args)
        _same(one, five)
    for k in (1, 32, 100):
        one = psa.topk_attention(kv, li.q, boxes, k, want_order=True, want_scores=True)
        five = psa.topk_attention(kv, li.q, boxes, k, want_order=True, want_scores=True, tuning=_general(psa))
        _same(one, five)


@pytest.mark.parametrize("batch,ctx", [(24, 4096), (23, 4096), (1, 2048), (1, 2049)])
def test_the_line_between_the_paths(psa, batch, ctx):
    """8 KV heads: 192 streams of 256 blocks take one launch, 184 the general path; so do 128 and 129 blocks."""
    li = _layer(4, 8, "bf16", batch, ctx, 3)
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    one = psa.decode_attention(kv, li.q, meta, 0.95, 1, want_order=True, want_scores=True, want_traffic=True)
    five = psa.decode_attention(kv, li.q, meta, 0.95, 1, want_order=True, want_scores=True, tuning=_general(psa))
    _same(one, five)
    read = one.traffic.view(-1, 2)
    blocks = ((li.ctx_lens + 15) // 16).repeat_interleave(8).to(read.device)
    assert (read[:, 0] <= blocks).all() and (read[:, 1] <= read[:, 0]).all()


@pytest.mark.parametrize("H,dtype", [(1, "bf16"), (1, "f16"), (3, "f16"), (5, "bf16")])
@pytest.mark.parametrize("ctx,ctx_min", [(1, 1), (250, 3), (513, 513), (1041, 100), (2048, 1500), (2049, 30), (4096, 1024)])
def test_scores_on_the_matrix_cores(psa, H, dtype, ctx, ctx_min):
    """G = 8 and a KV-head count that is 1 or does not divide 16: both paths score on the matrix cores, so a tuning that
    takes the call to the general path moves no bit of a score, and with it no rank and no stop."""
    blocks = (ctx + 15) // 16
    batch = 5 if blocks <= 128 else (3 * blocks + 4 * H - 1) // (4 * H)
    li = _layer(8, H, dtype, batch, ctx, ctx_min)
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    for eps, m, scorer in [(0.9, 1, 0), (0.6, 3, 1), (1.0, 1, 0)]:
        args = dict(scorer=scorer, want_order=True, want_scores=True)
        one = psa.decode_attention(kv, li.q, meta, eps, m, **args)
        five = psa.decode_attention(kv, li.q, meta, eps, m, tuning=_general(psa), **args)
        _same(one, five)
    if batch == 5:
        out = gc.run_gpu_decode(li, 0.95, 1)
        rep = gc.check_decode_against_oracle(gc.to_problem(li), out, 0.95, 1)
        rep.assert_accounted(max_rank_swaps=1)


def test_more_streams_than_one_launch_can_have(psa):
    """4194304 streams would be 2^32 threads and a workgroup more: the general path, whose workgroups are smaller, takes
    them.  All requests share a page and a query, so all results are those of one."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    k, v = (torch.randn((1, 1, 16, 128), generator=gen, device="cuda").half() for _ in range(2))
    q = torch.randn((1, 1, 128), generator=gen, device="cuda").half()

    def call(batch):
        kv = psa.KvCache(k, v, torch.zeros((batch, 1), dtype=torch.int32, device="cuda"),
                         torch.full((batch,), 13, dtype=torch.int32, device="cuda"), 1)
        meta = psa.build_block_metadata(kv, page_fill=torch.tensor([13], dtype=torch.int32, device="cuda"))
        out = psa.decode_attention(kv, q.expand(batch, 1, 128).contiguous(), meta, 0.9, 1)
        torch.cuda.synchronize()
        assert psa.read_device_error(out._workspace) == 0
        return out
    one, many = call(1), call(1 << 22)
    for name in ("out", "n_selected", "mass_est", "blocks_read", "lse"):
        assert (getattr(many, name) == getattr(one, name)).all(), name


def test_bad_tables_and_lengths_are_clamped_and_reported(psa):
    li = _layer(4, 2, "f16", 3, 900, 900)
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    good = psa.decode_attention(kv, li.q, meta, 0.9, 1)
    torch.cuda.synchronize()
    assert psa.read_device_error(good._workspace) == 0
    want = {n: getattr(good, n)[1].clone() for n in ("out", "n_selected", "mass_est", "lse")}
    li.block_table[0, 3] = li.k_pool.shape[0] + 5
    li.ctx_lens[2] = -4
    bad = psa.decode_attention(kv, li.q, meta, 0.9, 1)
    torch.cuda.synchronize()
    assert psa.read_device_error(bad._workspace) == 3
    for n, w in want.items():
        assert torch.equal(getattr(bad, n)[1], w), n
    assert not bad.out[2].any() and not bad.n_selected[2].any()


@pytest.mark.parametrize("batch,H,blocks", [(200, 1, 70), (65, 3, 8), (24, 8, 256)])
def test_every_request_and_column_is_checked(psa, batch, H, blocks):
    """The workgroup that finds the error word takes 64 requests a turn and a lane every 64th column: one bad entry or
    length at a time, at the edges of both, is reported whoever it belongs to, and an entry beyond the request is not."""
    ctx = 16 * blocks - 3
    li = _layer(4, H, "f16", batch, ctx, ctx)
    li.ctx_lens[:] = ctx
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)

    def flags():
        out = psa.decode_attention(kv, li.q, meta, 0.9, 1)
        torch.cuda.synchronize()
        return psa.read_device_error(out._workspace)
    assert flags() == 0
    for r in sorted({0, 3, 4, 63, 64, 67, 127, 128, batch - 2, batch - 1} & set(range(batch))):
        for c in sorted({0, 63, 64, blocks - 1} & set(range(blocks))):
            keep = int(li.block_table[r, c])
            for bad in (-1, li.k_pool.shape[0]):
                li.block_table[r, c] = bad
                assert flags() == 1, (r, c, bad)
            li.block_table[r, c] = keep
        for bad in (-1, 16 * blocks + 1):
            li.ctx_lens[r] = bad
            assert flags() == 2, (r, bad)
        li.ctx_lens[r] = 16 * (blocks - 1)
        keep = int(li.block_table[r, blocks - 1])
        li.block_table[r, blocks - 1] = -1
        assert flags() == 0, r
        li.block_table[r, blocks - 1] = keep
        li.ctx_lens[r] = ctx
    assert flags() == 0


@pytest.mark.parametrize("max_blocks,batch", [(1, 2), (31, 2), (33, 2), (64, 2), (65, 3), (128, 2), (200, 40), (256, 50)])
@pytest.mark.parametrize("pages", [1, 9, 61])
def test_tied_scores_rank_by_block(psa, max_blocks, batch, pages):
    """Blocks that share pages tie: the ranking is the stable sort of the scores, and the general path's."""
    heads = 4
    gen = torch.Generator(device="cuda").manual_seed(max_blocks + pages)
    k = torch.randn((pages, heads, 16, 128), generator=gen, device="cuda").to(torch.bfloat16)
    table = torch.randint(0, pages, (batch, max_blocks), generator=gen, device="cuda", dtype=torch.int32)
    lens = torch.full((batch,), 16 * max_blocks - 3, dtype=torch.int32, device="cuda")
    lens[1] = 16 * (max_blocks // 2) + 1
    kv = psa.KvCache(k, k, table, lens, heads)
    q = torch.randn((batch, heads, 128), generator=gen, device="cuda").to(torch.bfloat16)
    meta = psa.build_block_metadata(kv)
    one = psa.decode_attention(kv, q, meta, 0.7, 1, want_order=True, want_scores=True)
    _same(one, psa.decode_attention(kv, q, meta, 0.7, 1, want_order=True, want_scores=True, tuning=_general(psa)))
    for r in range(batch):
        n = (int(lens[r]) + 15) // 16
        want = torch.sort(one.scores[r, :, :n], dim=1, descending=True, stable=True)[1].to(torch.int32)
        assert torch.equal(one.order[r, :, :n], want), f"request {r}"
        assert (one.order[r, :, n:] == -1).all()


@pytest.mark.parametrize("G,H,batch,ctx", [(4, 2, 3, 1900), (8, 1, 3, 1000), (1, 8, 24, 4000)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -65504.0])
def test_non_finite_keys(psa, G, H, batch, ctx, bad):
    """Keys that are no numbers, infinite or as large as the type allows in one request, metadata included: the ranking stays
    a permutation, the general path agrees wherever numbers come out, the other requests are bit for bit as without them."""
    li = _layer(G, H, "f16", batch, ctx, ctx)
    li.ctx_lens[:] = ctx
    kv = gc.to_kv(li)
    clean = psa.decode_attention(kv, li.q, psa.build_block_metadata(kv, page_fill=li.page_fill), 0.9, 1)
    N = (ctx + 15) // 16
    pages = li.block_table[0, :N].long()
    k = li.k_pool.clone()
    k[pages[5], :, 3, :17] = bad
    k[pages[40], 0, :, 64] = -bad
    k[pages[N - 1], :, 7, :] = bad
    li.k_pool.copy_(k)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    one = psa.decode_attention(kv, li.q, meta, 0.9, 1, want_order=True, want_scores=True)
    five = psa.decode_attention(kv, li.q, meta, 0.9, 1, want_order=True, want_scores=True, tuning=_general(psa))
    torch.cuda.synchronize()
    assert psa.read_device_error(one._workspace) == 0
    for name in NAMES:
        x, y = getattr(one, name), getattr(five, name)
        if name == "scores":
            x, y = x[:, :, :N], y[:, :, :N]
        same = x.view(torch.int32) == y.view(torch.int32)
        if x.dtype == torch.float32:
            same |= x.isnan() & y.isnan()
        assert same.all(), name
    for name in ("out", "n_selected", "mass_est", "blocks_read", "lse"):
        assert torch.equal(getattr(one, name)[1:], getattr(clean, name)[1:]), name
    o = one.order[:, :, :N].sort(dim=-1).values
    assert torch.equal(o, torch.arange(N, device="cuda", dtype=torch.int32).expand_as(o))


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("G,H", [(4, 8), (8, 1)])
def test_a_captured_call_replays(psa, G, H, static):
    """The one launch in a HIP graph: replayed with eager work and synchronisations between the replays and new queries in
    the captured buffer, each replay gives what an eager call gives."""
    li = generate_layer(get_config(3).scaled(batch=2, ctx=2000, layers=1, num_q_heads=G * H, num_kv_heads=H), layer=3, device="cuda")
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    q = li.q.clone()
    first = psa.decode_attention(kv, q, meta, 0.95, 1, want_order=True)
    err = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    psa.decode_attention_static(kv, q, meta, 0.95, 1, first, device_error=err)      # outside the graph: looks the array up
    torch.cuda.synchronize()
    ws, graph, side = first._workspace, torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            if static:
                psa.decode_attention_static(kv, q, meta, 0.95, 1, first, device_error=err, stream=torch.cuda.current_stream())
            else:
                psa.decode_attention(kv, q, meta, 0.95, 1, workspace=ws, outputs=first, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    seen = []
    for step in range(4):
        if step:
            q.copy_(step_inputs(li, step)[0])
        eager = psa.decode_attention(kv, q, meta, 0.95, 1, want_order=True)
        torch.cuda.synchronize()
        first.out.zero_()
        first.n_selected.zero_()
        err.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert (int(err) if static else psa.read_device_error(ws)) == 0
        for name in ("out", "n_selected", "mass_est", "blocks_read", "lse", "order"):
            assert torch.equal(getattr(first, name), getattr(eager, name)), (name, step)
        seen.append(eager.out.clone())
    assert not torch.equal(seen[0], seen[-1])


def test_a_depth_hint_changes_nothing(psa):
    li = _layer(4, 8, "bf16", 3, 1500, 300)
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    want = psa.decode_attention(kv, li.q, meta, 0.95, 1, want_order=True, want_scores=True)
    for hint in (want.blocks_read, torch.zeros_like(want.blocks_read), torch.full_like(want.blocks_read, 1 << 30),
                 torch.full_like(want.blocks_read, -5)):
        got = psa.decode_attention(kv, li.q, meta, 0.95, 1, want_order=True, want_scores=True,
                                   tuning=psa.Tuning(depth_hint=hint))
        _same(got, want)


def test_random_short_shapes_against_the_oracle(psa):
    """Untuned calls only, all of a size that one launch takes."""
    rng = np.random.default_rng(404)
    total = gc.ParityReport()
    for case in range(80):
        G, H = int(rng.choice([1, 2, 4, 8])), int(rng.choice([1, 2, 3, 4, 5, 8]))
        batch, ctx = int(rng.integers(1, 6)), int(np.exp(rng.uniform(0, np.log(2048))))
        if rng.random() < 0.2:                           # up to 256 blocks, with streams enough
            ctx = int(rng.integers(2049, 4097))
            batch = (3 * ((ctx + 15) // 16) + 4 * H - 1) // (4 * H)
        eps, m, scorer = float(rng.choice([0.0, 0.3, 0.8, 0.9, 0.95, 0.99, 1.0])), int(rng.choice([1, 1, 2, 5, 16])), int(rng.choice([0, 0, 1]))
        dtype, lo = str(rng.choice(["f16", "bf16"])), int(rng.integers(1, ctx + 1))
        print(f"case {case}: G {G} H {H} {dtype} batch {batch} ctx {lo}..{ctx} eps {eps} m {m} scorer {scorer}", flush=True)
        li = _layer(G, H, dtype, batch, ctx, lo)
        out = gc.run_gpu_decode(li, eps, m, scorer=scorer)
        some = None if batch <= 8 else sorted(rng.choice(batch, size=5, replace=False).tolist())
        rep = gc.check_decode_against_oracle(gc.to_problem(li), out, eps, m, requests=some, scorer=scorer)
        rep.assert_accounted(max_rank_swaps=1)
        total.add(rep)
    print(f"\n[short shapes] {total}")
    total.assert_accounted(max_stop_flips=max(1, total.heads // 200))
