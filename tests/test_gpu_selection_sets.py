"""The Top-K selection at the borders of its rules: as many pages as a thread's, a lane
group's or a part of a thread's set of pages gives for its lower bound, one more and one less; rows at
the ends of every register tiling; bins that hold 64 or 65 keys, equal keys across the
threshold, and rows with infinite, huge and subnormal scores.  Lists are exact, in launches that attend
as well, whose outputs are those of attention over the list; with groups of query heads too."""
import math

import numpy as np
import pytest

from oracle import quest_oracle as O

pytestmark = pytest.mark.gpu
S, H = 16, 6


def rows(rng, n, family):
    """H rows of n scores."""
    x = rng.standard_normal((H, n))
    if family == "spread":
        x[0] = 3 + x[0]                                        # spans zero, more above
        x[1] = 200 + 30 * x[1]
        x[2] = np.cumsum(x[2])                                 # a walk
        x[3] = np.arange(n) - n / 2                            # ascending
        x[4] = -x[3]
        x[5, rng.integers(0, n, 3)] = 1e6                      # outliers
    elif family == "ties":
        x[0] = np.round(x[0])
        x[1] = 1.5
        x[2] = np.where(np.arange(n) % 7 == 0, 5.0, x[2] * 1e-3)
        x[3] = 10.0 - (np.arange(n) // 64 % 5)                 # runs of 64 equal keys
        x[4] = 10.0 - (np.arange(n) // 65 % 5)
        x[5] = np.where(np.arange(n) % 2, 0.0, -0.0)
    else:
        x[0, ::5] = np.inf
        x[1, ::3] = -np.inf
        x[2, ::4], x[2, 1::4] = np.inf, -np.inf
        x[3] *= 1e-44
        x[4] = np.where(np.arange(n) % 3, 3e38, -3e38) * rng.random(n)
        x[5] = 1.0 + 1e-7 * np.round(x[5])
    return x.astype(np.float32)


# rows at the borders of the tilings of the stand-alone kernel and of the selecting attention launch
ROWS = [1, 65, 512, 513, 1024, 1025, 1537, 2561, 4096, 4097, 5121, 8704, 8705]


@pytest.mark.parametrize("family", ["spread", "ties", "odd"])
@pytest.mark.parametrize("n", ROWS)
def test_lists_at_the_borders(n, family):
    import torch
    from paper_2406_10774_amd import binding as Q
    dev, policy = "cuda:0", 12 * (n & 1)               # odd rows: first and newest page kept
    rng = np.random.default_rng(n + policy)
    # the full row, and sequences that end inside it
    lens = np.array([S * n, max(1, S * n - 5), S * max(1, n // 2) - 3, S * max(1, n - 70)], np.int32)
    B = len(lens)
    sc = np.stack([rows(rng, n, family) for _ in lens])
    N = 64
    gen = torch.Generator(device=dev).manual_seed(n)
    pools = [torch.randn((N, H, S, 128), dtype=torch.float16, device=dev, generator=gen) for _ in range(2)]
    q = torch.randn((B, H, 128), dtype=torch.float16, device=dev, generator=gen)
    meta = torch.zeros((H, N, 2, 128), dtype=torch.float16, device=dev)
    table = torch.randint(0, N, (B, n), dtype=torch.int32, device=dev, generator=gen)
    cache = Q.Cache(*pools, meta, table, torch.from_numpy(lens).to(dev), flags=policy)
    scores = torch.from_numpy(sc).to(dev)
    # 16, 8, 4, 2 lanes a set, one thread, 2, 4, 8 and 16 parts of a thread, all of 256, 512 or 1024 threads
    ks = sorted({k + d for k in (2, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096, 8192) for d in (-1, 0, 1, 2)} |
                {n - 1, n, n + 3, n // 2})
    for k in [k for k in ks if 1 <= k <= n + 3]:
        want, want_keff = O.topk(sc, lens, S, k, keep_first=bool(policy & 4), keep_newest=bool(policy & 8))
        idx = torch.full((B, H, k), -7, dtype=torch.int32, device=dev)
        keff = torch.full((B,), -7, dtype=torch.int32, device=dev)
        Q.quest_topk(cache, scores, k, idx, keff)
        assert np.array_equal(keff.cpu().numpy(), want_keff)
        assert np.array_equal(idx.cpu().numpy(), want), (n, k)
        if k > 300 or k % 3:
            continue
        check_select(cache, q, scores, k, want, want_keff)


def check_select(cache, q, scores, k, want, want_keff):
    """List, K_b, out and lse of the selecting call; out and lse against attention over the list."""
    import torch
    from paper_2406_10774_amd import binding as Q
    dev = scores.device
    ws = torch.zeros(max(8, Q.quest_step_workspace_bytes(cache, k)), dtype=torch.uint8, device=dev)
    idx = torch.full(want.shape, -7, dtype=torch.int32, device=dev)
    keff = torch.full(want_keff.shape, -7, dtype=torch.int32, device=dev)
    out, ref = (torch.full(q.shape, float("nan"), device=dev) for _ in range(2))
    lse, ref_lse = (torch.full(q.shape[:2], float("nan"), device=dev) for _ in range(2))
    scale = 1 / math.sqrt(128)
    Q.quest_select_decode(cache, q, scores, k, scale, idx, out, k_eff=keff, lse=lse, workspace=ws)
    assert np.array_equal(idx.cpu().numpy(), want) and np.array_equal(keff.cpu().numpy(), want_keff), ("select", k)
    Q.quest_sparse_decode(cache, q, idx, k, scale, ref, ref_lse, ws)
    # the same pages in another split of the list, or on more waves: fp32 sums in another order, n 2^-24
    # of sum p |v| each, |v| < 6, and on the matrix cores the logits' sums too (128 products of
    # |q k| < 36 / 4, scaled) and the weights' 23 bits; twice, once for each side
    n = k * cache.k_pool.shape[2]
    logits = 0.0 if q.shape[1] == want.shape[1] else 128 * 2.0 ** -24 * 128 * 9 * scale + 2.0 ** -22
    assert float((out - ref).abs().max()) <= 2 * (n * 2.0 ** -24 + 2 * logits) * 6
    assert float((lse - ref_lse).abs().max()) <= 2 * (n * 2.0 ** -24 + logits) + 1e-6


@pytest.mark.parametrize("family", ["spread", "ties", "odd"])
@pytest.mark.parametrize("n,group,page", [(512, 4, 16), (513, 9, 16), (1024, 2, 8), (1025, 4, 16), (1537, 9, 8), (2560, 8, 16),
                                          (2561, 4, 16), (4096, 9, 16), (4097, 4, 8), (4097, 9, 16), (5120, 4, 16),
                                          (5120, 9, 8), (5121, 4, 16)])
def test_groups_at_the_borders(n, group, page, family):
    """Rows at the ends of the tilings of the launch that selects for a group of query heads."""
    import torch
    from paper_2406_10774_amd import binding as Q
    dev, policy, N = "cuda:0", 12 * (n & 1), 64
    rng = np.random.default_rng(n + group)
    lens = np.array([page * n, max(1, page * n - 5), page * (n // 2) - 3, page * (n - 70), 3], np.int32)
    B = len(lens)
    sc = np.stack([rows(rng, n, family) for _ in lens])
    gen = torch.Generator(device=dev).manual_seed(n)
    pools = [torch.randn((N, H, page, 128), dtype=torch.float16, device=dev, generator=gen) for _ in range(2)]
    pools[0] *= 0.25
    q = torch.randn((B, H * group, 128), dtype=torch.float16, device=dev, generator=gen)
    meta = torch.zeros((H, N, 2, 128), dtype=torch.float16, device=dev)
    table = torch.randint(0, N, (B, n), dtype=torch.int32, device=dev, generator=gen)
    cache = Q.Cache(*pools, meta, table, torch.from_numpy(lens).to(dev), flags=policy, num_heads=H * group)
    scores = torch.from_numpy(sc).to(dev)
    for k in (1, 2, 16, 63, 130, 300, 511, 1025):
        want, want_keff = O.topk(sc, lens, page, k, keep_first=bool(policy & 4), keep_newest=bool(policy & 8))
        check_select(cache, q, scores, k, want, want_keff)
