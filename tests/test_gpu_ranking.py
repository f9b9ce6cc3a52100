"""The ranking kernel alone matters here: its variants (keys per thread, workgroups per stream, buckets or the sorting
network) at the edges of their sizes, with tied scores, against a stable sort of the scores the same call reports."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    import paper_2503_00392_amd as psa
    psa.load_library()
    assert torch.cuda.is_available()
    return psa


@pytest.mark.parametrize("max_blocks", [257, 511, 512, 513, 2047, 2048, 2049, 4095, 4096, 4098, 8191, 8192])
@pytest.mark.parametrize("batch,heads,pages,bitonic", [(1, 2, 601, 0), (3, 96, 601, 0), (2, 2, 601, 1), (2, 2, 9, 0)])
def test_order_is_the_stable_sort_of_the_scores(psa, max_blocks, batch, heads, pages, bitonic):
    """Pages are shared between blocks, so scores tie (about 14 ways with 601 pages; with 9 pages a bucket holds more than
    the quadratic count takes on).  heads = 96: one workgroup per stream; otherwise up to four."""
    gen = torch.Generator(device="cuda").manual_seed(max_blocks + pages)
    k = torch.randn((pages, heads, 16, 128), generator=gen, device="cuda").to(torch.bfloat16)
    table = torch.randint(0, pages, (batch, max_blocks), generator=gen, device="cuda", dtype=torch.int32)
    lens = torch.tensor([16 * max_blocks - 3, 16 * (max_blocks // 2) + 1, 5][:batch], dtype=torch.int32, device="cuda")
    kv = psa.KvCache(k, k, table, lens, heads)
    q = torch.randn((batch, heads, 128), generator=gen, device="cuda").to(torch.bfloat16)
    meta = psa.build_block_metadata(kv)
    tuning = psa.Tuning(force_bitonic=1) if bitonic else None
    o = psa.topk_attention(kv, q, meta, 1, want_order=True, want_scores=True, tuning=tuning)
    torch.cuda.synchronize()
    assert psa.read_device_error(o._workspace) == 0
    for r in range(batch):
        n = (int(lens[r]) + 15) // 16
        want = torch.sort(o.scores[r, :, :n], dim=1, descending=True, stable=True)[1].to(torch.int32)
        assert torch.equal(o.order[r, :, :n], want), f"request {r}"
        assert (o.order[r, :, n:] == -1).all()
