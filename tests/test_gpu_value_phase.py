"""The selection kernel's value phase: how many of a chunk's blocks each head uses, at the edges of chunks and of the
request, with one stream and with more than the folds take at a time.  Against the oracle's attention over the GPU's own
ranked prefix (binary32 sums, weights as two 16-bit halves: the bounds of gpu_common)."""
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


def _own_prefix(pb, o):
    n = o.n_selected.cpu().numpy()
    want, lse = po.attend_prefix(pb, o.order.cpu().numpy(), n, want_lse=True)
    got = o.out.cpu().numpy().astype(np.float64)
    assert gc.rel_l2(got, want).max(initial=0.0) <= gc.OUT_RTOL and gc.rel_max(got, want).max(initial=0.0) <= gc.OUT_RTOL
    assert np.abs(o.lse.cpu().numpy() - lse).max(initial=0.0) <= gc.LSE_ATOL
    return n


@pytest.mark.parametrize("G,H,dtype", [(1, 1, "f16"), (2, 3, "bf16"), (4, 2, "bf16"), (8, 1, "f16")])
@pytest.mark.parametrize("chunk", [8, 32, 64])
def test_budgets_at_the_edges_of_chunks(psa, G, H, dtype, chunk):
    """97 blocks, the last with one token: every budget around the edges of the chunks, and none at all."""
    cfg = get_config(4).scaled(batch=2, ctx=16 * 96 + 1, ctx_min=16 * 33 + 7, num_q_heads=G * H, num_kv_heads=H, dtype=dtype)
    li = generate_layer(cfg, device="cuda", poison_tail=True)
    pb, kv = gc.to_problem(li), gc.to_kv(li)
    meta = psa.build_block_metadata(kv, page_fill=li.page_fill)
    tun = psa.Tuning(chunk_blocks=chunk, spin_limit=1 << 14)
    blocks = pb.num_blocks()
    for k in (1, 2, 7, 8, 9, 31, 32, 33, 63, 64, 65, 95, 96, 97, 500):
        o = psa.topk_attention(kv, li.q, meta, k, want_order=True, tuning=tun)
        assert psa.read_device_error(o._workspace) == 0
        assert (_own_prefix(pb, o) == np.minimum(k, blocks)[:, None]).all(), k
    for eps, m in [(0.5, 1), (0.9, 3), (0.98, 1), (0.95, 32), (1.0, 1)]:
        out = gc.run_gpu_decode(li, eps, m, tuning=tun)
        gc.check_decode_against_oracle(pb, out, eps, m).assert_accounted(max_rank_swaps=1)


@pytest.mark.parametrize("batch,H,window", [(1, 1, 1), (130, 5, 0), (513, 2, 3)])
def test_streams_and_windows(psa, batch, H, window):
    """One stream with a window of one chunk; more streams than folding waves (512), in two and three turns."""
    cfg = get_config(4).scaled(batch=batch, ctx=16 * 140, ctx_min=5, num_q_heads=4 * H, num_kv_heads=H, dtype="bf16")
    li = generate_layer(cfg, device="cuda", poison_tail=True)
    some = None if batch == 1 else [0, 1, batch // 2, batch - 2, batch - 1]
    tun = psa.Tuning(window_chunks=window, spin_limit=1 << 14)
    for eps in (0.9, 1.0):
        out = gc.run_gpu_decode(li, eps, 1, tuning=tun)
        gc.check_decode_against_oracle(gc.to_problem(li), out, eps, 1, requests=some).assert_accounted(max_rank_swaps=1)
