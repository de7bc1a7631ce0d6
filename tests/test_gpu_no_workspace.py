"""Attention without a workspace, which is refused only where the splits of few heads need one:
many query heads, or few tokens, run in one split each.  Against the oracle, and against the
same call with a workspace."""
import math

import numpy as np
import pytest

from oracle import quest_oracle as O
from paper_2406_10774_amd import synth
from test_gpu_group_attention import bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,kv_heads,group,S,longest", [
    (9, 29, 1, 16, 1500), (9, 8, 4, 16, 1500), (9, 8, 4, 8, 1100), (3, 12, 9, 64, 1900), (2, 4, 1, 16, 60),
    (8, 32, 1, 16, 250),
])
def test_no_workspace(batch, kv_heads, group, S, longest):
    import torch
    from gpu_util import Layer
    from paper_2406_10774_amd import binding as Q
    lens = tuple(1 + (longest - 1) * (i + 1) // batch for i in range(batch))
    w = synth.Workload(780, "no-workspace", batch, kv_heads, lens, token_budget=1024, planted_per_head=1,
                       page_size=S, decode_steps=0)
    table, N = synth.make_page_table(w, permute=True)
    k_pool, v_pool, _ = synth.fill_pools(w, table, N)
    k_pool *= np.float16(0.25)
    H = kv_heads * group
    q = np.random.default_rng(H).standard_normal((batch, H, 128)).astype(np.float16)
    cur = np.array(lens, np.int32)
    scale, K = 1 / math.sqrt(128), w.k_pages
    table = table[:, :max(w.pages_of(b) for b in range(batch))].copy()   # no room behind the longest
    layer = Layer(k_pool, v_pool, table, cur, num_q_heads=H)
    layer.build_meta()
    sc = layer.estimate(q)
    idx, keff, with_ws, _ = layer.select_decode(q, K)
    out = torch.full(q.shape, float("nan"), device=layer.dev)
    lse = torch.full(q.shape[:2], float("nan"), device=layer.dev)
    lists = torch.from_numpy(idx).to(layer.dev)
    mine = torch.full_like(lists, -7)
    for chosen, call in (
            (None, lambda: Q.quest_sparse_decode(layer.cache, layer.half(q), None, 0, scale, out, lse)),
            (idx, lambda: Q.quest_sparse_decode(layer.cache, layer.half(q), lists, K, scale, out, lse)),
            (idx, lambda: Q.quest_select_decode(layer.cache, layer.half(q), layer.scores, K, scale, mine, out, lse=lse)),
            (idx, lambda: Q.quest_decode_step_static(layer.cache, None, None, False, layer.half(q), K, scale,
                                                     layer.scores, mine, out, lse=lse))):
        out.fill_(float("nan"))
        call()
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        limit = bound(k_pool, v_pool, q, table, cur, chosen, scale)
        want, want_lse = O.sparse_decode(k_pool, v_pool, q, table, cur, chosen, scale)
        assert (np.abs(got - want) <= limit).all()
        assert np.abs(lse.cpu().numpy() - want_lse).max() <= 1e-4
        if chosen is not None:
            assert (np.abs(got - with_ws) <= limit).all()
    assert np.array_equal(mine.cpu().numpy(), idx)
