"""The estimate for groups of query heads over large tables (more than 393216 entries: 16 pages per
wave), which nothing else reaches with groups, and over small ones: groups that are no
multiple of the four queries loaded at a time, ragged lengths that end inside and between a
wave's pages, rows that are no multiple of a work-group's pages.  Pages repeat a few physical
ones, so that the pools stay small.  Scores against the oracle; the append against the calls one
by one, bit for bit."""
import numpy as np
import pytest

from oracle import quest_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_heads,group,S,pages,lens", [
    (8, 5, 16, 13013, (13013 * 16, 13000 * 16 + 1, 16 * 64 + 5, 1)),
    (8, 9, 8, 49217, (49217 * 8 - 3,)),
    (4, 4, 64, 33001, (33001 * 64, 40 * 64, 7 * 64 + 63)),
    (2, 2, 16, 24601, (24601 * 16 - 1, 16 * 15, 16 * 16, 16 * 16 + 1, 24577 * 16, 16 * 63, 100, 24601 * 16)),
    (8, 5, 16, 333, (333 * 16, 100, 16 * 17 + 2)), (3, 9, 32, 1027, (1027 * 32 - 5, 32 * 8, 1)),
    (2, 6, 8, 61, (61 * 8, 33)),
])
def test_scores(kv_heads, group, S, pages, lens):
    import torch
    from gpu_util import Layer, score_tolerance
    B, N = len(lens), 40
    rng = np.random.default_rng(pages)
    k_pool = rng.standard_normal((N, kv_heads, S, 128)).astype(np.float16)
    v_pool = np.zeros_like(k_pool)
    q = rng.standard_normal((B, kv_heads * group, 128)).astype(np.float16)
    # the newest token's page is a physical page of its own: the others hold whole pages
    table = rng.integers(B, N, (B, pages)).astype(np.int32)
    cur = np.array(lens, np.int32)
    table[np.arange(B), (cur - 1) // S] = np.arange(B)
    k_new, v_new = (rng.standard_normal((B, kv_heads, 128)).astype(np.float16) for _ in range(2))
    meta = np.stack([k_pool.astype(np.float32).min(2), k_pool.astype(np.float32).max(2)], 2).astype(np.float16)
    meta = np.ascontiguousarray(meta.transpose(1, 0, 2, 3))               # [heads][pages][2][D]

    def layer():
        x = Layer(k_pool, v_pool, table, cur, num_q_heads=kv_heads * group)
        x.meta.copy_(x.half(meta))
        return x

    one = layer()
    one.append(k_new, v_new, write=True)
    got = one.estimate(q)
    after = one.np16(one.meta)
    want = O.estimate(after, q, table, cur, S)
    tol = score_tolerance(after, q, table, cur, S)
    for b in range(B):
        P = -(-int(cur[b]) // S)
        assert (np.abs(got[b, :, :P] - want[b, :, :P]) <= tol[b, :, :P]).all(), b
        assert np.isnan(got[b, :, P:]).all(), b                           # not written
    both = layer()
    fused = both.append_estimate(k_new, v_new, q)
    assert np.array_equal(fused.view(np.uint32), got.view(np.uint32))
    assert np.array_equal(both.np16(both.meta).view(np.uint16), after.view(np.uint16))
    for a, b in ((both.k_pool, one.k_pool), (both.v_pool, one.v_pool)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


# three heads to more than one operand's sixteen, at the border to the vector unit (12288 entries) and
# between 8 and 16 pages per wave (40960), rows that end on a wave's pages, one more and one less
@pytest.mark.parametrize("kv_heads,group,S,pages,lens", [
    (8, 3, 16, 5120, (5120 * 16,)), (8, 3, 16, 5121, (5121 * 16 - 15,)), (1, 16, 8, 41000, (16 * 8 * 200 + 8,)),
    (2, 17, 16, 70, (16 * 16, 16 * 16 + 1, 8 * 16, 8 * 16 + 1, 70 * 16)), (1, 33, 32, 20481, (20481 * 32, 15 * 32)),
    (4, 4, 64, 9, (9 * 64, 1)), (8, 3, 16, 1536, (1536 * 16 - 9,)), (8, 3, 16, 1537, (1537 * 16,)),
    (8, 4, 16, 384, (384 * 16, 5, 100 * 16, 129)), (8, 4, 16, 385, (385 * 16, 5, 100 * 16, 129)),
])
def test_scores_on_the_matrix_cores(kv_heads, group, S, pages, lens):
    test_scores(kv_heads, group, S, pages, lens)


@pytest.mark.parametrize("kv_heads,group,pages", [(2, 4, 61), (8, 8, 5200), (3, 17, 100), (1, 3, 41003), (8, 4, 1600)])
def test_infinite_metadata(kv_heads, group, pages):
    """Infinite entries: the sign of the query picks the row, and the other row's infinity
    meets nothing.  Pages next to them keep the bound of finite ones."""
    import torch
    from paper_2406_10774_amd import binding as Q
    dev, S, N = "cuda:0", 16, 40
    rng = np.random.default_rng(pages)
    meta = np.sort(rng.standard_normal((kv_heads, N, 2, 128)), axis=2).astype(np.float16)
    meta[:, 3, 1, 5] = np.inf                        # only the max row
    meta[:, 4, 0, 77] = -np.inf                      # only the min row
    meta[:, 5, 0, 9], meta[:, 5, 1, 9] = -np.inf, np.inf
    meta[:, 6, :, 100] = np.inf                      # both rows: not a number with a -inf beside it
    meta[:, 6, :, 31] = np.inf
    q = rng.standard_normal((1, kv_heads * group, 128)).astype(np.float16)
    q[q == 0] = 1
    table = rng.integers(0, N, (1, pages)).astype(np.int32)
    t = lambda x: torch.from_numpy(x).to(dev)
    pool = torch.zeros((N, kv_heads, S, 128), dtype=torch.float16, device=dev)
    scores = torch.full((1, kv_heads, pages), -7.0, device=dev)
    cache = Q.Cache(pool, pool, t(meta), t(table), t(np.array([pages * S - 3], np.int32)), num_heads=kv_heads * group)
    Q.quest_estimate(cache, t(q), scores)
    got = scores.cpu().numpy()[0]
    m, x = meta.astype(np.float64), q[0].astype(np.float64).reshape(kv_heads, group, 1, 128)
    with np.errstate(invalid="ignore"):
        term = np.where(x < 0, x * m[:, None, :, 0], x * m[:, None, :, 1])   # [kv heads][group][N][128]
        each = term.sum(-1)
        want = np.fmax.reduce(each, axis=1)
        size = np.where(np.isfinite(each), np.abs(term).sum(-1), 0).max(1)
    want, size = want[:, table[0]], size[:, table[0]]
    odd = ~np.isfinite(want)
    assert np.array_equal(got[odd], want[odd], equal_nan=True) and np.isinf(want).any()
    # 128 exact products summed in fp32, in any order
    assert (np.abs(got[~odd] - want[~odd]) <= 128 * 2.0 ** -24 * size[~odd]).all()
