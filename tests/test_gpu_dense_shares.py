"""Attention over every page in both of its forms, where the cutting can go wrong.  Splits of the
page-table row (rows of few tokens, or little work): fewer pages than splits, sequences that
end in front of a split, groups that need two work-groups, more sequences than compute units.
Equal shares of the line of all pages (long rows and much work; what counts is the room in the
page table, so the sequences here are short): fewer pages than shares, shares that hold many
whole items, items over many shares, more than 64 sequences (one lane each while the line is
measured), heads by fours and one by one, groups, pages of 8 tokens.  Against the oracle; a
second call on the same workspace gives the same bits."""
import math

import numpy as np
import pytest

from oracle import quest_oracle as O
from paper_2406_10774_amd import synth
from test_gpu_group_attention import bound

pytestmark = pytest.mark.gpu

RAGGED70 = tuple(1 + (i * 37) % 90 for i in range(70))


@pytest.mark.parametrize("kv_heads,group,S,lens", [
    (32, 1, 16, (1,)), (32, 1, 16, (3001,)), (32, 1, 8, (1999, 16)), (36, 1, 64, (700,)),
    (4, 1, 16, RAGGED70), (3, 1, 16, (5003, 1, 17)), (1, 1, 16, (9001,)), (1, 1, 32, RAGGED70 * 2),
    (32, 1, 16, (700, 5)), (8, 1, 32, (903, 1, 32, 738)), (8, 4, 16, (900, 17, 500)),
    (8, 1, 8, (260, 3, 4100, 900)), (2, 9, 16, (2100, 5, 333)), (1, 4, 8, RAGGED70), (2, 4, 64, (6007,)),
    (12, 1, 16, (5999,)), (4, 3, 8, RAGGED70 * 2), (2, 1, 64, (4097, 1)),
])
def test_dense_shares(kv_heads, group, S, lens):
    check(kv_heads, group, S, lens, 0)


def equal_shares(batch, kv_heads, group, S, pages):
    """The rule that decides: rows of more than 3072 tokens with more than 48k units of 16 tokens or more
    than 128 heads (or groups); fewer than 8 of them with long rows."""
    items = batch * kv_heads * -(-group // 8)
    return (pages * S > 3072 and (items * pages * S / 16 > 48 * 1024 or items > 128)) or \
        (items < 8 and pages * S > (16384 if group > 1 else 6400))


@pytest.mark.parametrize("kv_heads,group,S,lens,room", [
    (32, 1, 16, (1,), 2000), (32, 1, 16, (3001,), 2000), (32, 1, 8, (1999, 16), 2000), (36, 1, 64, (700,), 400),
    (4, 1, 16, RAGGED70, 300), (3, 1, 16, (5003, 1, 17), 6000), (1, 1, 16, (9001,), 50000),
    (1, 1, 32, RAGGED70 * 2, 250), (33, 1, 8, (700, 5), 3000), (8, 1, 32, (903, 1, 32, 738), 1000),
    (8, 4, 16, (900, 17, 500), 3000), (8, 1, 8, (260, 3, 4100, 900), 4000), (2, 9, 16, (2100, 5, 333), 6000),
    (1, 4, 8, RAGGED70, 1700), (2, 4, 64, (6007,), 7000), (8, 8, 8, (1, 2000, 9, 700), 4000),
    (12, 2, 32, tuple(1 + i * 13 for i in range(66)), 130), (8, 4, 16, (7000, 9000), 3500),
    (1, 1, 8, (7001, 3), 900), (2, 1, 64, (6500, 64), 110), (1, 5, 16, (17000, 20), 1100),
    (2, 1, 16, RAGGED70, 200), (1, 9, 32, RAGGED70, 100),                    # more than 128 heads or groups
])
def test_equal_shares(kv_heads, group, S, lens, room):
    assert equal_shares(len(lens), kv_heads, group, S, room)
    check(kv_heads, group, S, lens, room)


@pytest.mark.parametrize("kv_heads,group,S,lens,room", [
    # items shorter than, as long as and longer than the 128 KiB that stand in front of each on the line
    (32, 1, 16, (16, 63, 64, 65, 1, 2000, 1), 1000), (1, 1, 16, (255, 256, 257, 1) * 35, 200),
    (8, 4, 16, (255, 256, 257, 3000, 1, 16) * 2, 600), (8, 2, 8, (127, 128, 129, 1) * 4, 1200),
    (32, 1, 64, (64, 65, 1, 900), 400), (2, 1, 16, (1,), 30000), (4, 1, 32, (20000,), 700),
])
def test_borders_between_items(kv_heads, group, S, lens, room):
    assert equal_shares(len(lens), kv_heads, group, S, room)
    check(kv_heads, group, S, lens, room)


def check(kv_heads, group, S, lens, room):
    import torch
    from gpu_util import Layer
    from paper_2406_10774_amd import binding as Q
    w = synth.Workload(740, "dense", len(lens), kv_heads, lens, token_budget=S, planted_per_head=1,
                       page_size=S, decode_steps=0)
    table, N = synth.make_page_table(w, permute=True)
    k_pool, v_pool, _ = synth.fill_pools(w, table, N)
    table = np.pad(table, ((0, 0), (0, max(0, room - table.shape[1]))))
    k_pool *= np.float16(0.25)
    rng = np.random.default_rng(len(lens))
    q = rng.standard_normal((w.batch, kv_heads * group, 128)).astype(np.float16)
    cur = np.array(lens, np.int32)
    scale = 1 / math.sqrt(128)
    want, want_lse = O.sparse_decode(k_pool, v_pool, q, table, cur, None, scale)
    limit = bound(k_pool, v_pool, q, table, cur, None, scale)
    for flags in (0, Q.QUEST_FLAG_DEVICE_FENCES):
        layer = Layer(k_pool, v_pool, table, cur, num_q_heads=kv_heads * group, flags=flags)
        ws = torch.zeros(Q.quest_workspace_bytes(layer.cache, 0), dtype=torch.uint8, device=layer.dev)
        got = []
        for _ in range(2):
            out = torch.full(q.shape, float("nan"), device=layer.dev)
            lse = torch.full(q.shape[:2], float("nan"), device=layer.dev)
            Q.quest_sparse_decode(layer.cache, layer.half(q), None, 0, scale, out, lse, ws)
            torch.cuda.synchronize()
            got.append((out.cpu().numpy(), lse.cpu().numpy()))
        off = np.abs(got[0][0] - want)
        assert (off <= limit).all(), float(off.max())
        assert np.abs(got[0][1] - want_lse).max() <= 1e-4
        assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
