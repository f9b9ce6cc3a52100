"""Requests that fit one workgroup take one launch instead of five kernels.  Both paths form the same sums in the
same order, so every output has to agree bit for bit; any tuning of the general path selects that path.  Sizes: the
edges of a chunk (32 ranked blocks), of a step of key reads (64) and of the path itself (128 blocks, or up to 256 with
three streams for four blocks)."""
import pytest
import torch

import gpu_common as gc
from workloads import generate_layer, get_config

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
