"""Block scores at the edges of the scoring kernels' units: rounds of 16 blocks, one to four to a wave, KV-head counts that
do and do not divide the workgroup's waves, requests that end inside a unit.  Against the definition in binary64; a score is
a sum of 256 products of numbers below 6 in magnitude, taken in binary32 in any order: 256 * 2^-24 of the sum of the
products' magnitudes, at most 256 * 36 / sqrt(128) * 2^-24 * 256 < 1.3e-2 and, with signs at random, some 1e-5 of a score;
the bound of gpu_common is 2.5e-4."""
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


@pytest.mark.parametrize("G,H,batch,max_blocks", [(8, 1, 3, 129), (8, 3, 2, 145), (8, 8, 2, 160), (8, 16, 2, 513), (8, 5, 130, 211),
                                                  (8, 8, 65, 257), (8, 8, 130, 193), (8, 2, 700, 190), (4, 8, 40, 300), (2, 32, 33, 250),
                                                  (1, 5, 400, 140)])
@pytest.mark.parametrize("scorer,dtype", [(0, torch.float16), (1, torch.bfloat16)])
def test_scores_against_their_definition(psa, G, H, batch, max_blocks, scorer, dtype):
    gen = torch.Generator(device="cuda").manual_seed(G * 1000 + H * 10 + batch)
    pages = 37
    k = torch.randn((pages, H, 16, 128), generator=gen, device="cuda").clamp_(-5, 5).to(dtype)
    table = torch.randint(0, pages, (batch, max_blocks), generator=gen, device="cuda", dtype=torch.int32)
    lens = torch.randint(1, 16 * max_blocks + 1, (batch,), generator=gen, device="cuda", dtype=torch.int32)
    lens[0] = 16 * max_blocks
    lens[-1] = 1
    kv = psa.KvCache(k, k, table, lens, G * H)
    q = torch.randn((batch, G * H, 128), generator=gen, device="cuda").clamp_(-5, 5).to(dtype)
    meta = psa.build_block_metadata(kv)
    out = psa.decode_attention(kv, q, meta, 0.5, 1, want_order=True, want_scores=True, scorer=scorer)
    torch.cuda.synchronize()
    assert psa.read_device_error(out._workspace) == 0
    lo, hi = k.double().amin(dim=2), k.double().amax(dim=2)                     # [pages][H][128]
    qd = q.double().view(batch, H, G, 128)
    for r in sorted({0, 1, batch // 2, batch - 1}):
        n = (int(lens[r]) + 15) // 16
        a, b = lo[table[r, :n].long()], hi[table[r, :n].long()]                 # [n][H][128]
        x = qd[r].permute(0, 2, 1)                                              # [H][128][G]
        if scorer == 0:
            want = torch.matmul(b.permute(1, 0, 2), x.clamp(min=0)) + torch.matmul(a.permute(1, 0, 2), x.clamp(max=0))
        else:
            want = torch.matmul((a + b).permute(1, 0, 2), x) / 2
        want = want.amax(dim=2) / 128 ** 0.5                                    # [H][n]
        assert (out.scores[r, :, :n].double() - want).abs().max() <= gc.SCORE_ERR, r


@pytest.mark.parametrize("G,H", [(8, 1), (8, 2), (8, 3), (8, 8), (8, 16), (4, 8), (2, 5), (1, 32)])
@pytest.mark.parametrize("scorer,dtype", [(0, torch.bfloat16), (1, torch.float16)])
def test_scores_do_not_depend_on_the_other_requests(psa, G, H, scorer, dtype):
    """The width of the block table is that of the batch's longest request.  The same requests in tables of other widths, and
    beside a longer request, get the same bits: scores, ranking, stops and outputs."""
    gen = torch.Generator(device="cuda").manual_seed(G * 100 + H)
    pages, lens = 400, [1, 37, 16 * 61, 16 * 90 + 5]
    k, v = (torch.randn((pages, H, 16, 128), generator=gen, device="cuda").to(dtype) for _ in range(2))
    q = torch.randn((5, G * H, 128), generator=gen, device="cuda").to(dtype)
    rows = torch.randint(0, pages, (5, 1100), generator=gen, device="cuda", dtype=torch.int32)
    want = None
    for longest in (0, 128, 129, 200, 257, 1100):
        n = 5 if longest else 4
        kv = psa.KvCache(k, v, rows[:n, :max(longest, 91)].contiguous(),
                         torch.tensor((lens + [16 * longest])[:n], dtype=torch.int32, device="cuda"), G * H)
        meta = psa.build_block_metadata(kv, page_fill=torch.full((pages,), 16, dtype=torch.int32, device="cuda"))
        out = psa.decode_attention(kv, q[:n].contiguous(), meta, 0.9, 1, want_order=True, want_scores=True, scorer=scorer)
        torch.cuda.synchronize()
        assert psa.read_device_error(out._workspace) == 0
        got = [x[:4] for x in (out.out, out.n_selected, out.mass_est, out.lse)] + [
            x[r, :, :(lens[r] + 15) // 16] for x in (out.scores, out.order) for r in range(4)]
        if want is None:
            want = [x.clone() for x in got]
        for a, b in zip(got, want):
            assert torch.equal(a.contiguous().view(torch.int32), b.contiguous().view(torch.int32)), longest
