"""Selection among candidates inside the attention launch (rows of more than 8704 pages, 5120 with
groups of query heads), and of whole rows up to there: the page list, K_b, outputs and lse are those of the separate launches, for rows that end on and
inside chunks, with ties, forced pages, infinite scores, groups of query heads and pages of 8
tokens, with a workspace that has no room for candidates, and on the static entry point."""
import math

import numpy as np
import pytest

from oracle import quest_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_pages,S,group,k_pages,policy", [
    (5120, 16, 1, 64, 0), (5121, 16, 1, 64, 12), (6144, 8, 4, 300, 4), (8193, 16, 1, 256, 12), (8193, 16, 1, 1, 8),
    (8200, 8, 1, 512, 0), (16384, 16, 4, 256, 12), (32769, 16, 1, 256, 0), (32769, 8, 1, 500, 4), (12289, 64, 9, 17, 12),
    (6144, 16, 4, 10, 12), (8193, 8, 9, 16, 0),           # groups whose heads attend one by one
    (8704, 16, 1, 65, 8), (8705, 16, 1, 64, 12), (10001, 8, 1, 512, 0), (12289, 16, 1, 256, 4), (16383, 64, 1, 100, 8),
    (16383, 16, 1, 2048, 12),                             # one query head per KV head, candidates
])
def test_candidates(max_pages, S, group, k_pages, policy):
    import torch
    from paper_2406_10774_amd import binding as Q
    dev, Hkv = "cuda:0", 2
    lens = np.array([S * max_pages, S * 2048 * ((max_pages - 1) // 2048), S * 2048 + 3, S * 4097 - 1, 5], np.int32)
    B, N = len(lens), 600
    rng = np.random.default_rng(max_pages + k_pages)
    sc = (rng.standard_normal((B, Hkv, max_pages)) * 30).astype(np.float32)
    sc[0, 1] = np.round(sc[0, 1] / 20) * 20            # ties across chunks
    sc[1, 0] = 7.0
    sc[2, 1, 2040:2060] += 500                         # winners on both sides of a border
    sc[3, 0, ::1000] = np.inf
    sc[3, 1, 100:] = -np.inf
    gen = torch.Generator(device=dev).manual_seed(max_pages)
    half = dict(dtype=torch.float16, device=dev, generator=gen)
    k_pool, v_pool = (torch.randn((N, Hkv, S, 128), **half) for _ in range(2))
    q = torch.randn((B, Hkv * group, 128), **half)
    meta = torch.zeros((Hkv, N, 2, 128), dtype=torch.float16, device=dev)
    table = torch.randint(0, N, (B, max_pages), dtype=torch.int32, device=dev, generator=gen)
    seq = torch.from_numpy(lens).to(dev)
    scores = torch.from_numpy(sc).to(dev)
    want, want_keff = O.topk(sc, lens, S, k_pages, keep_first=bool(policy & 4), keep_newest=bool(policy & 8))

    def run(flags, size):
        cache = Q.Cache(k_pool, v_pool, meta, table, seq, flags=policy | flags, num_heads=Hkv * group)
        nbytes = Q.quest_workspace_bytes(cache, k_pages)
        idx = torch.full((B, Hkv, k_pages), -7, dtype=torch.int32, device=dev)
        keff = torch.full((B,), -7, dtype=torch.int32, device=dev)
        out = torch.full(q.shape, float("nan"), device=dev)
        lse = torch.full(q.shape[:2], float("nan"), device=dev)
        ws = torch.zeros(max(size(nbytes, cache), 8), dtype=torch.uint8, device=dev)
        for _ in range(2):                             # the second on what the first left in the workspace
            Q.quest_select_decode(cache, q, scores, k_pages, 1 / math.sqrt(128), idx, out, k_eff=keff, lse=lse,
                                  workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(keff.cpu().numpy(), want_keff)
        assert np.array_equal(idx.cpu().numpy(), want)
        return nbytes, out, lse

    plain, ref, ref_lse = run(Q.QUEST_FLAG_SEPARATE_LAUNCHES, lambda n, c: n)
    nbytes, out, lse = run(0, lambda n, c: n)
    whole_rows = 8704 if group == 1 else 5120
    assert (nbytes > plain) == (whole_rows < max_pages < 16384) or max_pages >= 16384
    # the same pages in the same splits, on eight waves instead of four: fp32 sums in another
    # order, n 2^-24 of sum p |v| each, |v| < 6
    n = k_pages * S
    assert float((out - ref).abs().max()) <= 2 * n * 2.0 ** -24 * 6
    assert float((lse - ref_lse).abs().max()) <= 2 * n * 2.0 ** -24 + 1e-6
    if max_pages < 16384:
        _, out, lse = run(0, lambda n, c: plain)       # no room for candidates
        assert torch.equal(out, ref) and torch.equal(lse, ref_lse)
