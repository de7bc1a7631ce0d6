"""Precision of grouped-query attention on the matrix cores, against 64-bit arithmetic: weights far
below the largest keep their bits, and outputs and lse are as close as those of the same query
heads with KV heads of their own, which the vector unit computes in fp32."""
import math

import numpy as np
import pytest

from oracle import quest_oracle as O
from paper_2406_10774_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,S", [(4, 16), (8, 8), (9, 64)])
def test_small_weights_keep_their_bits(group, S):
    """One token takes nearly all the weight, its values are zero; the others, of weight 2^-e, are
    the output.  Their logits are -e log 2 up to fp16 keys; a logit's two roundings (the product
    with the scale, which is rounded too, and the distance to the largest) cost 3 * 2^-24 |logit|
    of the weight, exp2 and the two parts 2^-22, the sum over n tokens n 2^-24."""
    from gpu_util import Layer
    es = np.arange(2, 29)
    B, n, Hkv = len(es), 3 * S + 5, 2
    pages = -(-n // S)
    table = np.arange(B * pages, dtype=np.int32).reshape(B, pages)
    k_pool = np.zeros((B * pages, Hkv, S, 128), np.float16)
    rng = np.random.default_rng(group)
    v_pool = rng.uniform(0.5, 2.0, k_pool.shape).astype(np.float16)
    for b, e in enumerate(es):
        k_pool[table[b], 0, :, 0] = np.float16(-e * math.log(2) * 1.0371)   # not a power of two
        k_pool[table[b], 1, :, 0] = np.float16(-e * math.log(2) * 0.9817)
        k_pool[table[b, 0], :, 3, 0] = 0
        v_pool[table[b, 0], :, 3] = 0
    q = np.zeros((B, Hkv * group, 128), np.float16)
    q[..., 0] = 1
    lens = np.full(B, n, np.int32)
    layer = Layer(k_pool, v_pool, table, lens, num_q_heads=Hkv * group)
    every = np.broadcast_to(np.arange(pages), (B, Hkv, pages))
    want, want_lse = O.sparse_decode(k_pool, v_pool, q, table, lens, None, 1.0)
    logit = np.abs(k_pool[table[:, 0], :, 0, 0].astype(np.float64)).repeat(group, 1)
    bound = 3 * 2.0 ** -24 * logit + 2.0 ** -22 + n * 2.0 ** -24
    for got, lse in (layer.decode(q, None, 0, sm_scale=1.0), layer.decode(q, every, pages, sm_scale=1.0)):
        off = np.abs(got - want) / want
        assert (off.max(-1) <= bound).all(), (off.max(-1) / bound).max()
        assert np.abs(lse - want_lse).max() <= 2e-6


def test_as_close_as_heads_of_their_own():
    """2-norm of the error over all outputs, and of lse, relative to that of the vector unit on the
    same keys, values and queries.  Few heads with large logits make up a workload's norm, so one
    workload may come out on either side (factors from 0.6 to 1.6 were seen); the geometric mean
    over these workloads is what is asked for, within 1.1."""
    from gpu_util import Layer
    ratios = []
    for kv_heads, group, S, lens in (
            (4, 8, 16, (20000,)), (8, 2, 64, (1053, 700, 900, 300)), (2, 4, 8, (4000, 9000)), (3, 9, 32, (16000, 5)),
            (8, 4, 16, (6000, 2500)), (8, 8, 16, (300,)), (2, 16, 16, (5000,)), (8, 4, 8, (1000, 400, 70)),
            (5, 3, 16, (9000,)), (4, 4, 32, (3000, 2000, 1000))):
        w = synth.Workload(790 + group, "precision", len(lens), kv_heads, lens, token_budget=S * 256, planted_per_head=16,
                           page_size=S, decode_steps=0)
        table, N = synth.make_page_table(w, permute=True)
        k_pool, v_pool, _ = synth.fill_pools(w, table, N)
        H = kv_heads * group
        q = np.random.default_rng(S).standard_normal((len(lens), H, 128)).astype(np.float16)
        cur = np.array(lens, np.int32)
        scale = 1 / math.sqrt(128)
        grouped = Layer(k_pool, v_pool, table, cur, num_q_heads=H)
        own = Layer(k_pool.repeat(group, 1), v_pool.repeat(group, 1), table, cur)
        idx, _ = O.topk(O.estimate(O.build_meta(k_pool, table, cur), q, table, cur, S), cur, S, w.k_pages)
        for one, each in ((None, None), (idx, idx.repeat(group, 1))):
            want = O.sparse_decode(k_pool, v_pool, q, table, cur, one, scale)
            err = [[np.linalg.norm(a.astype(np.float64) - b) for a, b in zip(layer.decode(q, i, w.k_pages), want)]
                   for layer, i in ((grouped, one), (own, each))]
            ratios.append(np.log(np.array(err[0]) / np.array(err[1])))
    mean = np.exp(np.mean(ratios, 0))
    print("out, lse:", mean)
    assert (mean <= 1.1).all(), mean
