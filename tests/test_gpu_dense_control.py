"""The dense control where a wave's blocks pass the 64 whose pages a wave holds at a time, and where it has none, one or two:
one split per request, four waves, blocks every fourth.  Against attention in binary64 (bounds of gpu_common)."""
import numpy as np
import pytest
import torch

import gpu_common as gc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    import paper_2503_00392_amd as psa
    psa.load_library()
    assert torch.cuda.is_available()
    return psa


@pytest.mark.parametrize("G,dtype", [(1, torch.float16), (2, torch.bfloat16), (4, torch.bfloat16), (8, torch.float16)])
@pytest.mark.parametrize("max_blocks", [2, 9, 256, 261, 330, 520])
def test_page_lists_of_a_wave(psa, G, dtype, max_blocks):
    H, batch, pages = 32, 64, 41                         # 2048 streams: one split each
    gen = torch.Generator(device="cuda").manual_seed(max_blocks * 8 + G)
    k, v = (torch.randn((pages, H, 16, 128), generator=gen, device="cuda").to(dtype) for _ in range(2))
    table = torch.randint(0, pages, (batch, max_blocks), generator=gen, device="cuda", dtype=torch.int32)
    lens = torch.randint(1, 16 * max_blocks + 1, (batch,), generator=gen, device="cuda", dtype=torch.int32)
    lens[:6] = torch.tensor([16 * max_blocks, 1, 16, 17, 0, max(1, 16 * max_blocks - 15)], dtype=torch.int32)
    q = torch.randn((batch, H * G, 128), generator=gen, device="cuda").to(dtype)
    kv = psa.KvCache(k, v, table, lens, H * G)
    out, lse = psa.dense_attention(kv, q)
    torch.cuda.synchronize()
    assert psa.read_device_error(out._workspace) == 0
    for r in list(range(6)) + [batch - 1]:
        n = int(lens[r])
        if n == 0:
            assert not out[r].any() and torch.isneginf(lse[r]).all()
            continue
        at = table[r].long()
        for h in (0, 13, H - 1):
            kk, vv = (x[at, h].reshape(-1, 128)[:n].double() for x in (k, v))
            s = q[r, h * G:(h + 1) * G].double() @ kk.T / 128 ** 0.5
            want = (torch.softmax(s, dim=1) @ vv).cpu().numpy()
            got = out[r, h * G:(h + 1) * G].double().cpu().numpy()
            assert np.max(gc.rel_l2(got, want)) <= gc.OUT_RTOL and np.max(gc.rel_max(got, want)) <= gc.OUT_RTOL, (r, h)
            assert (lse[r, h * G:(h + 1) * G].double() - torch.logsumexp(s, dim=1)).abs().max() <= gc.LSE_ATOL, (r, h)
