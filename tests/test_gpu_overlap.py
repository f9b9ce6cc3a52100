"""Chunk workgroups of the selection kernel go on without chunks that have not been started: a workgroup whose looks run out
reads the missing chunks itself.  Forced by a patience of one look, and met where calls on several streams share the chip.
Both give the bits that the same calls give one after the other with the default patience: whatever a chunk leaves in
memory is the same bits whoever works on it."""
import pytest
import torch

import gpu_common as gc
from workloads import generate_layer, get_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    import paper_2503_00392_amd as psa
    psa.load_library()
    assert torch.cuda.is_available()
    return psa


def _same(a, b):
    for name in ("out", "n_selected", "mass_est", "blocks_read", "lse", "order"):
        x, y = getattr(a, name), getattr(b, name)
        assert torch.equal(x.view(torch.int32), y.view(torch.int32)), name


@pytest.mark.parametrize("G,H,batch,ctx,dtype", [(1, 2, 2, 131072, "f16"), (2, 3, 2, 40000, "bf16"), (4, 8, 3, 32768, "bf16"),
                                                 (8, 8, 2, 30011, "f16"), (4, 2, 300, 3000, "bf16")])
@pytest.mark.parametrize("chunk", [8, 32, 64])
def test_a_patience_of_one_look(psa, G, H, batch, ctx, dtype, chunk):
    """Up to 1024 chunks and 128 groups of chunks to a stream; stops early, late and nowhere; the rule tested at positions that
    are and are not a chunk's last."""
    cfg = get_config(4).scaled(batch=batch, ctx=ctx, ctx_min=ctx // 3, num_q_heads=G * H, num_kv_heads=H, dtype=dtype)
    li = generate_layer(cfg, device="cuda", poison_tail=True)
    kv = gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    hint = torch.full((batch, H), 1 << 29, dtype=torch.int32, device="cuda")
    for eps, m in [(0.9, 1), (0.98, 3), (1.0, 1)]:
        want = psa.decode_attention(kv, li.q, meta, eps, m, want_order=True, tuning=psa.Tuning(chunk_blocks=chunk, spin_limit=1 << 14))
        for tun in (psa.Tuning(chunk_blocks=chunk, spin_limit=1), psa.Tuning(chunk_blocks=chunk, spin_limit=3, depth_hint=hint)):
            got = psa.decode_attention(kv, li.q, meta, eps, m, want_order=True, want_traffic=True, tuning=tun)
            assert psa.read_device_error(got._workspace) == 0
            _same(got, want)
            if eps == 1.0 and chunk == 64 and tun.spin_limit == 1:       # keys were read twice (1.15 to 1.9 times all of them)
                assert int(got.traffic[..., 0].sum()) > int(got.blocks_read.sum())


def test_calls_on_several_streams(psa):
    """Calls of different shapes on three streams, each with its own workspace, over and over: more workgroups than the chip
    holds, of several launches at a time."""
    shapes = [dict(batch=8, ctx=32768, num_q_heads=32, num_kv_heads=8), dict(batch=2, ctx=131072, num_q_heads=16, num_kv_heads=8),
              dict(batch=24, ctx=16384, num_q_heads=64, num_kv_heads=8)]
    calls = []
    for i, kw in enumerate(shapes):
        li = generate_layer(get_config(4).scaled(ctx_min=kw["ctx"] // 8, dtype="bf16", **kw), device="cuda")
        kv = gc.to_kv(li)
        meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
        for eps in (0.9, 0.98, 1.0):
            want = psa.decode_attention(kv, li.q, meta, eps, 1, want_order=True)
            torch.cuda.synchronize()
            calls.append((i, kv, li.q, meta, eps, want))
    streams = [torch.cuda.Stream() for _ in shapes]
    spaces = [torch.empty(max(psa.decode_workspace_bytes(c[1]) for c in calls if c[0] == i), dtype=torch.uint8, device="cuda")
              for i in range(len(shapes))]
    outs = [psa.decode_attention(kv, q, meta, eps, 1, want_order=True) for _, kv, q, meta, eps, _ in calls]
    for turn in range(20):
        for o in outs:
            o.out.zero_()
            o.n_selected.zero_()
        torch.cuda.synchronize()
        for j in range(3):
            for i, st in enumerate(streams):
                _, kv, q, meta, eps, _ = calls[3 * i + (j + turn) % 3]
                psa.decode_attention(kv, q, meta, eps, 1, workspace=spaces[i], outputs=outs[3 * i + (j + turn) % 3], stream=st)
        torch.cuda.synchronize()
        for ws in spaces:
            assert psa.read_device_error(ws) == 0, turn
        for o, c in zip(outs, calls):
            _same(o, c[5])
