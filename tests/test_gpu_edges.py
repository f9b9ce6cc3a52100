"""GPU edge cases through the C ABI: empty and one-token requests inside a batch, lengths around a
page boundary, and inputs only the device can see are wrong (a table entry outside the pool, a length
beyond the table row, a negative length) -- the kernels clamp, say so in the sticky error word, and
leave the other requests' results untouched."""
import numpy as np
import pytest
import torch

import gpu_common as gc
from oracle import psa_oracle as po
from workloads import generate_layer, get_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    import paper_2503_00392_amd as psa
    psa.load_library()
    assert torch.cuda.is_available()
    return psa


def _layer(batch, ctx):
    return generate_layer(get_config(1).scaled(batch=batch, ctx=ctx), device="cuda", poison_tail=True)


LENGTHS = [0, 1, 15, 16, 17, 0, 300, 33]


def _cut(li, lengths):
    li.ctx_lens.copy_(torch.tensor(lengths, dtype=torch.int32))
    pb = gc.to_problem(li)
    return pb, torch.from_numpy(pb.page_fill()).cuda()


@pytest.mark.parametrize("eps,m", [(0.9, 1), (0.5, 3), (1.0, 1), (0.0, 2)])
def test_empty_tiny_and_page_boundary_requests(psa, eps, m):
    li = _layer(len(LENGTHS), 320)
    pb, fill = _cut(li, LENGTHS)
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=fill)
    gpu = psa.decode_attention(kv, li.q, meta, eps, m, want_order=True, want_scores=True, want_traffic=True)
    torch.cuda.synchronize()
    assert psa.read_device_error(gpu._workspace) == 0
    rep = gc.check_decode_against_oracle(pb, gpu, eps, m)
    empty = [i for i, n in enumerate(LENGTHS) if n == 0]
    assert rep.empty == len(empty) * pb.q.shape[1]
    rep.assert_accounted()
    for r in empty:
        assert not gpu.out[r].any() and not gpu.n_selected[r].any() and not gpu.mass_est[r].any()
        assert torch.isneginf(gpu.lse[r]).all() and not gpu.blocks_read[r].any()
        assert (gpu.order[r] == -1).all()
    one = LENGTHS.index(1)                       # a single token: attention returns its value, estimate 1
    assert (gpu.n_selected[one] == 1).all() and (gpu.mass_est[one] == 1.0).all()
    page = int(li.block_table[one, 0])
    G = li.cfg.group
    for hq in range(li.cfg.num_q_heads):
        assert torch.equal(gpu.out[one, hq], li.v_pool[page, hq // G, 0].float())


def test_dense_and_topk_on_the_same_batch(psa):
    li = _layer(len(LENGTHS), 320)
    pb, fill = _cut(li, LENGTHS)
    kv = gc.to_kv(li)
    out, lse = psa.dense_attention(kv, li.q)
    torch.cuda.synchronize()
    want, wlse = po.dense_attention(pb)
    live = np.array(LENGTHS) > 0
    assert gc.rel_l2(out.cpu().numpy().astype(np.float64), want).max() <= gc.OUT_RTOL
    np.testing.assert_allclose(lse.cpu().numpy()[live], wlse[live], rtol=0, atol=2e-3)
    assert torch.isneginf(lse[~torch.from_numpy(live).cuda()]).all() and not out[~torch.from_numpy(live).cuda()].any()
    meta = psa.build_block_metadata(kv, page_fill=fill)
    top = psa.topk_attention(kv, li.q, meta, 2, want_order=True)
    torch.cuda.synchronize()
    nb = pb.num_blocks()
    assert np.array_equal(top.n_selected.cpu().numpy(), np.repeat(np.minimum(2, nb)[:, None], li.cfg.num_q_heads, 1))
    own = po.attend_prefix(pb, top.order.cpu().numpy(), top.n_selected.cpu().numpy())
    assert gc.rel_l2(top.out.cpu().numpy().astype(np.float64), own).max() <= gc.OUT_RTOL


def test_inputs_only_the_device_can_see_are_wrong(psa):
    """Request 1 gets a table entry outside the pool, request 2 a length beyond its table row, request
    3 a negative length.  Nothing faults; the error word names both kinds; requests 0 and 4 come out
    exactly as in the clean run."""
    li = _layer(5, 640)
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    clean = psa.decode_attention(kv, li.q, meta, 0.9, 1, want_order=True)
    dclean, _ = psa.dense_attention(kv, li.q)
    torch.cuda.synchronize()
    assert psa.read_device_error(clean._workspace) == 0
    li.block_table[1, 7] = li.k_pool.shape[0] + 12345
    li.ctx_lens[2] = li.block_table.shape[1] * 16 + 999
    li.ctx_lens[3] = -5
    bad = psa.decode_attention(kv, li.q, meta, 0.9, 1, want_order=True)
    torch.cuda.synchronize()
    flags = psa.read_device_error(bad._workspace)
    assert flags == 3, flags
    assert torch.isfinite(bad.out).all()
    for r in (0, 4):
        assert torch.equal(bad.out[r], clean.out[r]) and torch.equal(bad.n_selected[r], clean.n_selected[r])
        assert torch.equal(bad.order[r], clean.order[r])
    assert not bad.out[3].any() and not bad.n_selected[3].any()          # negative length reads as empty
    assert (bad.n_selected[2] <= li.block_table.shape[1]).all()          # clamped to the row
    dbad, _ = psa.dense_attention(kv, li.q)
    torch.cuda.synchronize()
    dflags = psa.read_device_error(dbad._workspace)
    assert dflags & 1 and dflags & 2
    for r in (0, 4):
        assert torch.equal(dbad[r], dclean[r])
    # the next clean call starts from a clean error word
    li.block_table[1, 7] = 0
    li.ctx_lens[2] = 640
    li.ctx_lens[3] = 640
    again = psa.decode_attention(kv, li.q, meta, 0.9, 1, workspace=bad._workspace)
    torch.cuda.synchronize()
    assert psa.read_device_error(again._workspace) == 0


@pytest.mark.parametrize("bad", ["query", "key", "all keys"])
@pytest.mark.parametrize("ctx,G", [(1000, 4), (1800, 8), (5000, 4), (5000, 1)])
def test_a_fixed_budget_holds_for_heads_without_a_number(psa, ctx, G, bad):
    """A NaN query, a NaN in the best block or in every key of one request: P_acc of a head is then no number and passes no
    test, and the head attends its budget all the same.  Other requests, and the other heads of a group whose keys are
    sound, come out as without the NaN.  (1000 and 1800 tokens: one launch; 5000: the general path.)"""
    cfg = get_config(1).scaled(batch=2, ctx=ctx, num_q_heads=2 * G, num_kv_heads=2)
    li = generate_layer(cfg, device="cuda")
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    N = (ctx + 15) // 16
    first = psa.topk_attention(kv, li.q, meta, 1, want_order=True)
    q, nan = li.q.clone(), float("nan")
    if bad == "query":
        q[0, G - 1] = q[0, 0]           # (the group's scores are the maximum over its heads that are numbers)
        sound = q.clone()
        q[0, G - 1, 7] = nan
    elif bad == "key":
        li.k_pool[li.block_table[0, first.order[0, 0, 0]].long(), 0, 3, 9] = nan       # (the metadata stays as it was)
    else:
        li.k_pool[li.block_table[0, :N].long(), 0] = nan
    for k in (1, 5, 32, 33, N - 1, N, N + 7):
        top = psa.topk_attention(kv, q, meta, k, want_order=True, want_traffic=True)
        torch.cuda.synchronize()
        assert psa.read_device_error(top._workspace) == 0
        want = min(k, N)
        assert (top.n_selected == want).all() and (top.blocks_read == want).all()
        assert (top.traffic[:, :, 1] == want).all() and (top.traffic[:, :, 0] >= want).all()
        assert torch.isfinite(top.out[1]).all() and torch.isfinite(top.out[0, G:]).all()
        if bad == "query":
            clean = psa.topk_attention(kv, sound, meta, k)
            for name in ("out", "mass_est", "lse"):
                a, b = getattr(top, name).clone(), getattr(clean, name).clone()
                a[0, G - 1] = b[0, G - 1] = 0
                assert torch.equal(a, b), name


@pytest.mark.parametrize("max_blocks", [20, 300])
def test_a_pool_without_pages_is_never_read(psa, max_blocks):
    """num_pages = 0 leaves the pools and the metadata without an address.  Requests with tokens then have table entries
    that no page can match: they read as empty and the error word says so, whether the table would take the call to the
    one-launch path (20 columns) or to the general one (300), and in the dense control; without tokens there is nothing to
    report."""
    B, H, G = 3, 2, 4
    pool = torch.empty((0, H, 16, 128), dtype=torch.float16, device="cuda")
    assert pool.data_ptr() == 0
    q = torch.randn((B, H * G, 128), device="cuda").half()
    meta = torch.empty((0, H, 2, 128), dtype=torch.float16, device="cuda")
    for lens, want in (([0, 0, 0], 0), ([40, 0, 16 * max_blocks], 1), ([16 * max_blocks + 1, 0, 5], 3), ([0, -1, 0], 2)):
        kv = psa.KvCache(pool, pool, torch.zeros((B, max_blocks), dtype=torch.int32, device="cuda"),
                         torch.tensor(lens, dtype=torch.int32, device="cuda"), H * G)
        for o in (psa.decode_attention(kv, q, meta, 0.9, 1, want_order=True, want_traffic=True),
                  psa.topk_attention(kv, q, meta, 2, want_order=True, want_traffic=True)):
            torch.cuda.synchronize()
            assert psa.read_device_error(o._workspace) == want
            assert not o.out.any() and not o.n_selected.any() and not o.mass_est.any() and not o.blocks_read.any()
            assert torch.isneginf(o.lse).all() and (o.order == -1).all() and not o.traffic.any()
        out, lse = psa.dense_attention(kv, q)
        torch.cuda.synchronize()
        assert psa.read_device_error(out._workspace) == want
        assert not out.any() and torch.isneginf(lse).all()


def _shared_pages(psa, batch, H, G, blocks, seed):
    """Requests over a small pool, every page in many tables; keys too small for anything to stand out."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    k, v = (torch.randn((997, H, 16, 128), generator=gen, device="cuda").mul_(scale).half() for scale in (0.2, 1.0))
    table = torch.randint(0, 997, (batch, blocks), generator=gen, device="cuda", dtype=torch.int32)
    lens = torch.randint(8 * blocks, 16 * blocks + 1, (batch,), generator=gen, device="cuda", dtype=torch.int32)
    q = torch.randn((batch, H * G, 128), generator=gen, device="cuda").half()
    return psa.KvCache(k, v, table, lens, H * G), q


@pytest.mark.parametrize("batch,H,G,blocks", [(1024, 4, 1, 512), (129, 4, 8, 300), (171, 7, 2, 700), (1100, 1, 4, 333)])
def test_more_streams_than_waves_that_fold_them(psa, batch, H, G, blocks):
    """The selection kernel folds 512 streams at a time.  4096, 516, 1197 and 1100 streams: the call completes without giving
    up on any, with threshold 1 it is dense attention, and at any threshold a request's results are bit for bit those it
    has in a call of its own."""
    kv, q = _shared_pages(psa, batch, H, G, blocks, blocks)
    fill = torch.full((997,), 16, dtype=torch.int32, device="cuda")
    meta = psa.build_block_metadata(kv, page_fill=fill)
    dense, lse = psa.dense_attention(kv, q)
    for eps, hint in ((1.0, None), (0.9, None), (0.5, 40)):
        tuning = psa.Tuning(depth_hint=torch.full((batch, H), hint, dtype=torch.int32, device="cuda")) if hint else None
        o = psa.decode_attention(kv, q, meta, eps, 1, want_order=True, tuning=tuning)
        torch.cuda.synchronize()
        assert psa.read_device_error(o._workspace) == 0
        if eps == 1.0:
            assert gc.rel_l2(o.out.cpu().double().numpy(), dense.cpu().double().numpy()).max() <= gc.OUT_RTOL
            assert (o.lse - lse).abs().max() <= gc.LSE_ATOL
        for r in (0, 1, batch // 2, batch - 1):
            alone = psa.KvCache(kv.k_pool, kv.v_pool, kv.block_table[r:r + 1].contiguous(), kv.ctx_lens[r:r + 1].contiguous(), H * G)
            one = psa.decode_attention(alone, q[r:r + 1].contiguous(), meta, eps, 1, want_order=True)
            for name in ("out", "n_selected", "mass_est", "blocks_read", "lse", "order"):
                assert torch.equal(getattr(one, name)[0], getattr(o, name)[r]), (eps, r, name)


@pytest.mark.parametrize("blocks,G", [(8192, 1), (8193, 8), (20011, 4)])
def test_dense_attention_of_one_very_long_stream(psa, blocks, G):
    """One request, one KV head, beyond the 131072 tokens of the sparse call: the dense control takes any length, and cuts
    it into as many splits as its merge has room for."""
    gen = torch.Generator(device="cuda").manual_seed(blocks)
    k, v = (torch.randn((blocks, 1, 16, 128), generator=gen, device="cuda").half() for _ in range(2))
    q = torch.randn((1, G, 128), generator=gen, device="cuda").half()
    table = torch.randperm(blocks, generator=gen, device="cuda").to(torch.int32)[None]
    ctx = 16 * blocks - 5
    kv = psa.KvCache(k, v, table, torch.tensor([ctx], dtype=torch.int32, device="cuda"), G)
    out, lse = psa.dense_attention(kv, q)
    torch.cuda.synchronize()
    assert psa.read_device_error(out._workspace) == 0
    kk, vv = (x[table[0].long(), 0].reshape(-1, 128)[:ctx].cpu().double() for x in (k, v))
    logits = q[0].cpu().double() @ kk.T / 128 ** 0.5
    want = torch.softmax(logits, 1) @ vv
    assert gc.rel_l2(out[0].cpu().double().numpy(), want.numpy()).max() <= gc.OUT_RTOL
    assert (lse[0].cpu().double() - torch.logsumexp(logits, 1)).abs().max() <= gc.LSE_ATOL


def test_bench_read_probe_sizes_and_alignment(psa):
    """The benchmark's measurement aid (bench_probe.hip) reads and keeps nothing: any size runs (empty, below one
    load, ragged, several workgroups' worth), the source is unchanged, a misaligned source is refused on the host."""
    import os
    import sys
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import bench
    probe = bench.load_read_probe()
    buf = torch.arange(1 << 20, dtype=torch.int32, device="cuda")
    before = buf.clone()
    sink = torch.zeros(1, dtype=torch.int64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    for n in (0, 1, 4, 5, 1000, 2048 * 4 + 12, 1 << 20):
        assert probe(buf.data_ptr(), n * 4, sink.data_ptr(), st) == 0
    assert probe(buf.data_ptr(), buf.numel() * 4, None, st) == 0
    torch.cuda.synchronize()
    assert torch.equal(buf, before)
    assert probe(buf.data_ptr() + 4, 4096, sink.data_ptr(), st) == 1        # 4 bytes past a 16-byte boundary


@pytest.mark.parametrize("bad", ["nan", "inf", "huge"])
def test_non_finite_keys_do_not_disturb_other_requests(psa, bad):
    """Keys that are NaN, infinite or as large as the type allows in one request: the call completes (every
    loop of the kernels is bounded whatever the data), the other request's results are bit for bit those
    of a clean run, and the damaged request still reports a block count within its range."""
    cfg = get_config(1).scaled(batch=2, ctx=3000)
    li = generate_layer(cfg, device="cuda")
    clean = gc.run_gpu_decode(li, 0.9, 1)
    val = {"nan": float("nan"), "inf": float("inf"), "huge": 65504.0}[bad]
    pages = li.block_table[0, :188].long()
    k = li.k_pool.clone()
    k[pages[5], :, 3, :17] = val
    k[pages[100], 2, :, 64] = -val if bad != "nan" else val
    k[pages[187], :, 7, :] = val
    li.k_pool.copy_(k)
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    out = psa.decode_attention(kv, li.q, meta, 0.9, 1, want_order=True)
    dense, _ = psa.dense_attention(kv, li.q)
    torch.cuda.synchronize()
    assert psa.read_device_error(out._workspace) == 0
    for name in ("out", "n_selected", "mass_est", "blocks_read", "lse"):
        assert torch.equal(getattr(out, name)[1], getattr(clean, name)[1]), name
    N0 = (int(li.ctx_lens[0]) + 15) // 16
    assert int(out.n_selected[0].min()) >= 0 and int(out.n_selected[0].max()) <= N0
    o = out.order[0, :, :N0].sort(dim=-1).values
    assert torch.equal(o, torch.arange(N0, device="cuda", dtype=torch.int32).expand_as(o)), "ranking must stay a permutation"
    assert torch.isfinite(dense[1]).all()
