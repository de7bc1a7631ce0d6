"""The Top-K selection of one work-group per row where a thread has many pages: rows at the ends of the
longest register tilings, lists from one page to all but one, with few and many equal scores across the
threshold.  Lists are exact."""
import numpy as np
import pytest

from oracle import quest_oracle as O

pytestmark = pytest.mark.gpu
S, H = 16, 5


def rows(rng, n, family):
    """H rows of n scores."""
    x = rng.standard_normal((H, n))
    if family == "spread":
        x[0] = 200 + 30 * x[0]
        x[1] = np.cumsum(x[1])                                 # a walk on both sides of zero
        x[2] = np.arange(n) - n / 2                            # ascending
        x[3] = -x[2]
    else:
        x[0] = np.round(x[0])                                  # thousands of equal scores
        x[1] = 1.5
        x[2] = 10.0 - (np.arange(n) // 64 % 5)                 # runs of 64 equal keys
        x[3] = np.where(np.arange(n) % 3, 0.01 * x[3], np.where(np.arange(n) % 2, np.inf, -np.inf))
        x[4] = np.round(x[4] * 64)                             # a few equal scores at any threshold
    return x.astype(np.float32)


def check_lists(n, lens, family, ks, policy):
    import torch
    from paper_2406_10774_amd import binding as Q
    dev = "cuda:0"
    rng = np.random.default_rng(n + policy)
    lens = np.array(lens, np.int32)
    B = len(lens)
    sc = np.stack([rows(rng, n, family) for _ in lens])
    pool = torch.zeros((1, H, S, 128), dtype=torch.float16, device=dev)
    meta = torch.zeros((H, 1, 2, 128), dtype=torch.float16, device=dev)
    table = torch.zeros((B, n), dtype=torch.int32, device=dev)
    cache = Q.Cache(pool, pool, meta, table, torch.from_numpy(lens).to(dev), flags=policy)
    scores = torch.from_numpy(sc).to(dev)
    for k in ks:
        want, want_keff = O.topk(sc, lens, S, k, keep_first=bool(policy & 4), keep_newest=bool(policy & 8))
        idx = torch.full((B, H, k), -7, dtype=torch.int32, device=dev)
        keff = torch.full((B,), -7, dtype=torch.int32, device=dev)
        Q.quest_topk(cache, scores, k, idx, keff)
        assert np.array_equal(keff.cpu().numpy(), want_keff)
        assert np.array_equal(idx.cpu().numpy(), want), (n, k)


@pytest.mark.parametrize("family", ["spread", "ties"])
@pytest.mark.parametrize("n", [24577, 33792, 33793, 49152, 49153, 65535])
def test_long_rows(n, family):
    check_lists(n, [S * n, S * (n - n // 5) - 3], family, (1, 65, 1000, n // 8, n // 2, n - 1), 12 * (n & 1))


# rows whose tiling has a form for the first pages of each thread alone, and how many pages that is
SHORT = [(10240, 7 * 512), (24576, 9 * 1024), (33792, 12 * 1024), (49152, 18 * 1024), (65535, 24 * 1024)]


@pytest.mark.parametrize("family", ["spread", "ties"])
@pytest.mark.parametrize("n,part", SHORT)
def test_short_sequences_in_long_rows(n, part, family):
    lens = [S * part, S * (part - 1) + 1, S * (part + 1), S * (part + 2), S * 100, S * (part // 2) + 5]
    check_lists(n, lens, family, (1, 2, 64, 257, part // 2, part - 1), 0)
    check_lists(n, lens, family, (1, 2, 257, part - 1), 12)


@pytest.mark.parametrize("family", ["spread", "ties"])
@pytest.mark.parametrize("n,part,group", [(4200, 7 * 256, 1), (6912, 10 * 256, 1), (8704, 12 * 256, 1), (5120, 7 * 256, 4),
                                          (4097, 7 * 256, 9)])
def test_short_sequences_selected_in_the_attention_launch(n, part, group, family):
    """The list, K_b, out and lse are those of the separate launches, bit for bit: four waves either way."""
    import math
    import torch
    from paper_2406_10774_amd import binding as Q
    dev, N = "cuda:0", 300
    rng = np.random.default_rng(n + group)
    lens = np.array([S * part, S * (part - 1) + 1, S * (part + 1), S * (part + 2) - 3, S * 100, S * n], np.int32)
    B = len(lens)
    sc = np.stack([rows(rng, n, family) for _ in lens])
    gen = torch.Generator(device=dev).manual_seed(n)
    half = dict(dtype=torch.float16, device=dev, generator=gen)
    pools = [torch.randn((N, H, S, 128), **half) for _ in range(2)]
    q = torch.randn((B, H * group, 128), **half)
    meta = torch.zeros((H, N, 2, 128), dtype=torch.float16, device=dev)
    table = torch.randint(0, N, (B, n), dtype=torch.int32, device=dev, generator=gen)
    scores, seq = torch.from_numpy(sc).to(dev), torch.from_numpy(lens).to(dev)
    for policy, k in ((0, 1), (0, 64), (12, 129), (4, 700), (8, 2048)):
        want, want_keff = O.topk(sc, lens, S, k, keep_first=bool(policy & 4), keep_newest=bool(policy & 8))
        got = []
        for flags in (0, Q.QUEST_FLAG_SEPARATE_LAUNCHES):
            cache = Q.Cache(*pools, meta, table, seq, flags=policy | flags, num_heads=H * group)
            ws = torch.zeros(max(8, Q.quest_workspace_bytes(cache, k)), dtype=torch.uint8, device=dev)
            idx = torch.full((B, H, k), -7, dtype=torch.int32, device=dev)
            keff = torch.full((B,), -7, dtype=torch.int32, device=dev)
            out = torch.full(q.shape, float("nan"), device=dev)
            lse = torch.full(q.shape[:2], float("nan"), device=dev)
            Q.quest_select_decode(cache, q, scores, k, 1 / math.sqrt(128), idx, out, k_eff=keff, lse=lse, workspace=ws)
            assert np.array_equal(keff.cpu().numpy(), want_keff)
            assert np.array_equal(idx.cpu().numpy(), want), (n, k, flags)
            got.append((out, lse))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), (n, k)
