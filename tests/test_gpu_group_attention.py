"""Attention of query-head groups on the matrix cores (grouped-query attention) at the sizes
where a unit, a wave's share or a split can go wrong: sequences that end inside every part
of a 16-token unit, groups that are not a power of two or need two work-groups, single
pages, page pairs of 8 tokens with one missing, lists with holes, values that are fp16
subnormals, infinite or not numbers; dense, over a given list, and over the list the launch selects itself."""
import math

import numpy as np
import pytest

from oracle import quest_oracle as O
from paper_2406_10774_amd import synth

pytestmark = pytest.mark.gpu


def bound(k_pool, v_pool, q, table, lens, idx, scale):
    """Largest deviation from exact arithmetic, per output value.  A logit is a sum of 128
    exact products in fp32: off by at most 128 * 2^-24 * sum |q_i k_i| (times the scale); a
    weight relative to the sum of weights doubles that.  The weights keep 23 bits (2^-22
    for both), and fp32 sums over n tokens add 2 n 2^-24.  All relative to sum p |v|."""
    spread, _ = O.sparse_decode(k_pool, np.abs(v_pool), q, table, lens, idx, scale)
    logit = float(np.nanmax(np.abs(k_pool.astype(np.float32)).sum(-1))) * float(np.abs(q).max()) * scale
    n = max(int(x) for x in lens)
    return (2 * 128 * 2.0 ** -24 * logit + 2.0 ** -21 + 2 * n * 2.0 ** -24) * spread + 1e-30


@pytest.mark.parametrize("kv_heads,group", [(1, 2), (3, 3), (2, 5), (2, 8), (1, 9), (2, 16)])
@pytest.mark.parametrize("S", [8, 16, 64])
def test_unit_edges(kv_heads, group, S):
    check_edges(kv_heads, group, S, edge_lengths(S), 7, (1, 7, 64))


def edge_lengths(S):
    return (1, 3, 7, 8, 9, 15, 16, 17, 31, 33, 64, 65, S * 37 + 5, S * 40)


@pytest.mark.parametrize("kv_heads,group", [(1, 2), (3, 3), (2, 5), (2, 8), (1, 9), (2, 16)])
@pytest.mark.parametrize("S", [8, 16, 64])
def test_unit_edges_of_longer_lists(kv_heads, group, S):
    """The same for lists that the heads of a group attend over together: short lists of few heads
    are attended over head by head (at most 72k tokens of all heads)."""
    repeat = 1 + 72 * 1024 // (14 * kv_heads * group * 40 * S)
    check_edges(kv_heads, group, S, edge_lengths(S) * repeat, 40, (39, 64))


def check_edges(kv_heads, group, S, lens, pages, select):
    from gpu_util import Layer
    w = synth.Workload(700 + group, f"group-S{S}", len(lens), kv_heads, lens, token_budget=S * pages,
                       planted_per_head=2, page_size=S, decode_steps=0)
    table, N = synth.make_page_table(w, permute=True)
    k_pool, v_pool, _ = synth.fill_pools(w, table, N)          # stale slots hold NaN
    rng = np.random.default_rng([group, S])
    v_pool[..., 3::16] = np.where(np.isnan(v_pool[..., 3::16]), np.nan,
                                  rng.integers(-1023, 1024, v_pool[..., 3::16].shape) * 2.0 ** -24).astype(np.float16)
    k_pool *= np.float16(0.25)
    q = rng.standard_normal((w.batch, kv_heads * group, 128)).astype(np.float16)
    cur = np.array(lens, np.int32)
    layer = Layer(k_pool, v_pool, table, cur, num_q_heads=kv_heads * group)
    layer.build_meta()
    scale = 1 / math.sqrt(128)

    def check(got, lse, idx, what):
        want, want_lse = O.sparse_decode(k_pool, v_pool, q, table, cur, idx, scale)
        off = np.abs(got - want)
        assert (off <= bound(k_pool, v_pool, q, table, cur, idx, scale)).all(), (what, float(off.max()))
        assert np.abs(lse - want_lse).max() <= 1e-4, what

    got, lse = layer.decode(q, None, 0)
    check(got, lse, None, "dense")
    K = w.k_pages
    meta = O.build_meta(k_pool, table, cur)
    sc = O.estimate(meta, q, table, cur, S)
    idx, _ = O.topk(sc, cur, S, K)
    holes = idx.copy()
    for b in range(w.batch):
        if w.pages_of(b) > 3:
            holes[b, :, 1] = -1
            holes[b, :, 2] = w.pages_of(b)
    clean = np.where(holes >= 0, holes, -1)
    for b in range(w.batch):
        clean[b][clean[b] >= w.pages_of(b)] = -1
    got, lse = layer.decode(q, holes, K)
    check(got, lse, clean, "list")
    for k_pages in select:
        idx, keff, got, lse = layer.select_decode(q, k_pages, scores=sc.astype(np.float32))
        check(got, lse, idx, f"select {k_pages}")


@pytest.mark.parametrize("group,S,repeat", [(1, 16, 1), (4, 16, 1), (4, 8, 1), (9, 64, 1), (4, 16, 16), (4, 8, 16), (9, 64, 2)])
def test_infinite_and_nan_values(group, S, repeat):
    """An infinite value is infinite in the output wherever its weight is not zero, a NaN is NaN;
    every other channel and head comes out as without them."""
    from gpu_util import Layer
    lens = (S * 9 + 3, S * 3, 200) * repeat                    # repeated: the heads of a group together
    kv_heads = 2
    w = synth.Workload(760 + group, "non-finite", len(lens), kv_heads, lens, token_budget=S * 64, planted_per_head=0,
                       page_size=S, decode_steps=0)
    table, N = synth.make_page_table(w, permute=True)
    k_pool, v_pool, _ = synth.fill_pools(w, table, N)
    k_pool *= np.float16(0.125)                                # weights of one order of magnitude or two
    plain = v_pool.copy()
    bad = ((0, 0, 4, np.inf), (0, 1, 9, -np.inf), (1, 0, 17, np.nan), (2, 1, 127, np.inf))
    for b, h, ch, x in bad:
        for at in (5, lens[b] - 1):
            v_pool[table[b, at // S], h, at % S, ch] = x
    q = np.random.default_rng(group).standard_normal((w.batch, kv_heads * group, 128)).astype(np.float16)
    cur = np.array(lens, np.int32)
    layer = Layer(k_pool, v_pool, table, cur, num_q_heads=kv_heads * group)
    scale = 1 / math.sqrt(128)
    want, want_lse = O.sparse_decode(k_pool, plain, q, table, cur, None, scale)
    limit = bound(k_pool, plain, q, table, cur, None, scale)
    for b, h, ch, x in bad:
        want[b, h * group:(h + 1) * group, ch] = x
    K = w.k_pages                                              # every page of every sequence
    every = np.where(np.arange(K) < np.array([w.pages_of(b) for b in range(w.batch)])[:, None, None],
                     np.arange(K), -1) + np.zeros((w.batch, kv_heads, K), np.int64)
    sc = np.zeros((w.batch, kv_heads, table.shape[1]), np.float32)
    for got, lse in (layer.decode(q, None, 0), layer.decode(q, every, K), layer.select_decode(q, K, scores=sc)[2:]):
        odd = ~np.isfinite(want)
        assert np.array_equal(got[odd], want[odd], equal_nan=True)
        assert (np.abs(got - want)[~odd] <= limit[~odd]).all()
        assert np.abs(lse - want_lse).max() <= 1e-4


@pytest.mark.parametrize("batch,kv_heads,group,k_pages", [
    (32, 8, 8, 20), (16, 8, 5, 20), (4, 8, 8, 40), (3, 8, 8, 80), (2, 8, 9, 128), (2, 8, 3, 130), (1, 2, 16, 600)])
def test_splits_of_a_list(batch, kv_heads, group, k_pages):
    """1, 2, 8, 10, 8, 15 and 32 splits of a list, whose partial results a wave per query head merges 16
    at a time; given lists and selected ones, fp32 and fp16 outputs."""
    from gpu_util import Layer
    S, N, P = 16, 40, k_pages + 30
    rng = np.random.default_rng([batch, group])
    k_pool, v_pool = (rng.standard_normal((N, kv_heads, S, 128)).astype(np.float16) for _ in range(2))
    k_pool *= np.float16(0.25)
    table = rng.integers(0, N, (batch, P)).astype(np.int32)
    lens = np.array([S * P - 7 * b % (S * 40) for b in range(batch)], np.int32)
    q = rng.standard_normal((batch, kv_heads * group, 128)).astype(np.float16)
    sc = rng.standard_normal((batch, kv_heads, P)).astype(np.float32)
    idx, _ = O.topk(sc, lens, S, k_pages)
    layer = Layer(k_pool, v_pool, table, lens, num_q_heads=kv_heads * group)
    scale = 1 / math.sqrt(128)
    want, want_lse = O.sparse_decode(k_pool, v_pool, q, table, lens, idx, scale)
    limit = bound(k_pool, v_pool, q, table, lens, idx, scale)
    got, lse = layer.decode(q, idx, k_pages)
    assert (np.abs(got - want) <= limit).all() and np.abs(lse - want_lse).max() <= 1e-4
    half, lse16 = layer.decode(q, idx, k_pages, fp16_out=True)
    assert np.array_equal(half, got.astype(np.float16)) and np.array_equal(lse16, lse)
    list_, _, got, lse = layer.select_decode(q, k_pages, scores=sc)
    assert np.array_equal(list_, idx)
    assert (np.abs(got - want) <= limit).all() and np.abs(lse - want_lse).max() <= 1e-4
