"""Sequence lengths past the end of the page-table row.  No caller may pass them; attention over
all pages, and selection and attention from given scores, take the row's pages and read nothing
behind the row."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_heads,group,S,pages,k_pages,lens", [
    (4, 1, 16, 40, 7, (1, 37, 9)), (32, 1, 8, 300, 20, (1500, 1, 8)), (2, 4, 16, 130, 16, (3, 4000)),
    (2, 1, 16, 6000, 64, (1, 40000)), (2, 4, 8, 5200, 3000, (9000, 8)), (1, 1, 16, 16390, 600, (1, 100000)),
    (4, 1, 16, 6000, 64, (0, 0, 9000)), (36, 1, 16, 3000, 1, (1, 1)),
])
def test_lengths_past_the_row(kv_heads, group, S, pages, k_pages, lens):
    import torch
    from paper_2406_10774_amd import binding as Q
    dev, N, B = "cuda:0", 50, len(lens)
    gen = torch.Generator(device=dev).manual_seed(pages)
    half = dict(dtype=torch.float16, device=dev, generator=gen)
    k_pool, v_pool = (torch.randn((N, kv_heads, S, 128), **half) for _ in range(2))
    meta = torch.zeros((kv_heads, N, 2, 128), dtype=torch.float16, device=dev)
    table = torch.randint(0, N, (B, pages), dtype=torch.int32, device=dev, generator=gen)
    q = torch.randn((B, kv_heads * group, 128), **half)
    scores = torch.randn((B, kv_heads, pages), device=dev, generator=gen)

    def run(seq):
        cache = Q.Cache(k_pool, v_pool, meta, table, torch.tensor(seq, dtype=torch.int32, device=dev),
                        num_heads=kv_heads * group)
        ws = torch.zeros(Q.quest_workspace_bytes(cache, k_pages), dtype=torch.uint8, device=dev)
        out = torch.full((2, *q.shape), float("nan"), device=dev)
        lse = torch.full((2, *q.shape[:2]), float("nan"), device=dev)
        idx = torch.full((B, kv_heads, k_pages), -7, dtype=torch.int32, device=dev)
        Q.quest_sparse_decode(cache, q, None, 0, 0.1, out[0], lse[0], ws)
        Q.quest_select_decode(cache, q, scores, k_pages, 0.1, idx, out[1], lse=lse[1], workspace=ws)
        torch.cuda.synchronize()
        return out.cpu().numpy(), lse.cpu().numpy(), idx.cpu().numpy()

    full = pages * S
    for got, want in zip(run([full + n for n in lens]), run([full] * B)):
        assert np.array_equal(got, want)
