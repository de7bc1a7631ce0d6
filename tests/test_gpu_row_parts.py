"""Where a kernel's split of a row ends: the part of a thread's pages that is enough for a short sequence in a long row
(quest_topk, and the launch that selects and attends, for which eight waves select and four attend), and the estimate's
blocks in tables of 40961 to 114688 entries."""
import numpy as np
import pytest

from oracle import quest_oracle as O
from test_gpu_estimate_groups import test_scores as check_scores
from test_gpu_long_rows import test_short_sequences_selected_in_the_attention_launch as check_selected

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family", ["spread", "ties"])
@pytest.mark.parametrize("n,part,group", [(5120, 3 * 512, 1), (5121, 5 * 512, 1), (7168, 5 * 512, 1), (7169, 6 * 512, 1),
                                          (5119, 3 * 512, 4), (4098, 3 * 512, 9)])
def test_selected_in_the_attention_launch(n, part, group, family):
    check_selected(n, part, group, family)


@pytest.mark.parametrize("n,part", [(4097, 3 * 512), (6144, 4 * 512), (8192, 6 * 512), (10241, 4 * 1024), (17408, 6 * 1024)])
def test_topk(n, part):
    import torch
    from gpu_util import Layer
    rng = np.random.default_rng(n)
    S, heads = 8, 2
    lens = np.array([S * part, S * (part - 1) + 1, S * part + 1, S * (part + 3) - 5, S * 70, S * n], np.int32)
    pool = np.zeros((1, heads, S, 128), np.float16)
    layer = Layer(pool, pool, np.zeros((len(lens), n), np.int32), lens)
    for scores in (rng.standard_normal((len(lens), heads, n)), rng.integers(0, 9, (len(lens), heads, n))):
        scores = scores.astype(np.float32)
        for k in (1, 65, 800):
            idx, keff = layer.topk(k, scores)
            want, want_keff = O.topk(scores, lens, S, k)
            assert np.array_equal(idx, want) and np.array_equal(keff, want_keff), k


@pytest.mark.parametrize("kv_heads,S,pages,lens", [
    (8, 16, 1000, (1000 * 16, 12 * 16, 12 * 16 + 1, 48 * 16, 47 * 16 + 3, 997 * 16)),
    (8, 8, 2003, (2003 * 8 - 1, 3 * 8, 1, 4 * 8 + 1, 1000 * 8, 48 * 8 + 1)),
    (1, 64, 7001, (7001 * 64, 35 * 64, 36 * 64 + 1, 37 * 64, 7000 * 64 - 63, 12 * 64)),
])
def test_ends_of_blocks(kv_heads, S, pages, lens):
    check_scores(kv_heads, 1, S, pages, lens)


@pytest.mark.parametrize("B,heads,group,n", [
    (32, 16, 1, 4200), (33, 16, 1, 4097), (33, 16, 1, 5120), (33, 16, 1, 5121), (33, 16, 1, 6912), (33, 16, 1, 8704),
    (32, 8, 4, 5120), (33, 8, 4, 4097), (33, 8, 4, 5120), (17, 8, 9, 4600),
])
def test_many_rows_selected_in_the_attention_launch(B, heads, group, n):
    """Eight waves select in up to 512 work-groups (256 of groups), four in more: lists of the separate launches, and as
    four attend either way, their out and lse, bit for bit."""
    import math
    import torch
    from paper_2406_10774_amd import binding as Q
    S, N, gen = 8, 200, torch.Generator(device="cuda").manual_seed(n)
    half = dict(dtype=torch.float16, device="cuda", generator=gen)
    pools = [torch.randn((N, heads, S, 128), **half) for _ in range(2)]
    q = torch.randn((B, heads * group, 128), **half)
    meta = torch.zeros((heads, N, 2, 128), dtype=torch.float16, device="cuda")
    table = torch.randint(0, N, (B, n), dtype=torch.int32, device="cuda", generator=gen)
    lens = torch.randint(1, S * n + 1, (B,), dtype=torch.int32, device="cuda", generator=gen)
    lens[:3] = torch.tensor([S * n, S * n * 3 // 8, 1])
    scores = torch.randn((B, heads, n), device="cuda", generator=gen)
    scores[1::2] = torch.round(4 * scores[1::2])                   # thousands of equal scores
    for k in (16, 300):
        got = []
        for flags in (0, Q.QUEST_FLAG_SEPARATE_LAUNCHES):
            cache = Q.Cache(*pools, meta, table, lens, flags=flags, num_heads=heads * group)
            ws = torch.zeros(max(8, Q.quest_workspace_bytes(cache, k)), dtype=torch.uint8, device="cuda")
            idx = torch.full((B, heads, k), -7, dtype=torch.int32, device="cuda")
            keff = torch.full((B,), -7, dtype=torch.int32, device="cuda")
            out = torch.full(q.shape, float("nan"), device="cuda")
            lse = torch.full(q.shape[:2], float("nan"), device="cuda")
            Q.quest_select_decode(cache, q, scores, k, 1 / math.sqrt(128), idx, out, k_eff=keff, lse=lse, workspace=ws)
            got.append((idx, keff, out, lse))
        for name, a, b in zip(("list", "k_eff", "out", "lse"), *got):
            assert torch.equal(a, b), (name, k)
