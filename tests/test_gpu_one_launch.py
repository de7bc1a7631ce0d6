"""quest_decode_step as one launch (short rows) against the same call in separate launches: rows that end around a
tile's and a pass's last page, sequences of one page and one token, the newest token first and last in its page,
groups of query heads on both units, few and many rows.  Scores, lists, metadata and pools bit for bit, and nothing
written past a sequence's pages; attention within the rounding of its fp32 sums of float64 attention over the list.
The number of launches is checked too, so that a shape whose route changes does not go untested unnoticed."""
import math

import numpy as np
import pytest

from paper_2406_10774_amd import binding as Q

pytestmark = pytest.mark.gpu

# (sequences, query heads, KV heads, page size, pages of the row, pages of the list), launches that the step is
# expected to be.  Every kernel of a step in one launch is here with pages of 8 tokens and with larger ones.
SHAPES = [
    # one query head per KV head, four waves, up to 128 and 256 pages
    ((3, 2, 2, 16, 1, 1), 1), ((3, 2, 2, 16, 17, 4), 1), ((2, 32, 32, 16, 64, 16), 1), ((3, 3, 3, 8, 65, 300), 1),
    ((2, 1, 1, 32, 127, 40), 1), ((2, 2, 2, 64, 128, 9), 1), ((2, 32, 32, 16, 129, 64), 1), ((3, 1, 1, 8, 255, 2000), 1),
    ((2, 2, 2, 16, 256, 32), 1), ((13, 40, 40, 8, 250, 8), 1), ((130, 8, 8, 8, 65, 3), 1), ((2, 2, 2, 16, 257, 32), 2),
    ((3, 1, 1, 8, 320, 33), 2), ((2, 2, 2, 16, 321, 64), 2), ((1, 32, 32, 16, 257, 32), 2), ((4, 8, 8, 8, 320, 33), 2),
    # eight waves, 512 and 1024 pages
    ((15, 8, 8, 8, 257, 20), 1), ((24, 8, 8, 8, 512, 64), 1), ((6, 32, 32, 64, 314, 16), 1), ((15, 8, 8, 16, 511, 30), 1),
    ((21, 8, 8, 16, 1024, 17), 1), ((25, 8, 8, 8, 1024, 33), 1), ((25, 8, 8, 32, 513, 9), 1), ((25, 8, 8, 8, 1025, 30), 2),
    ((17, 8, 8, 8, 1024, 17), 2), ((16, 8, 8, 8, 513, 40), 2),
    # four waves, 512 pages
    ((49, 8, 8, 8, 511, 16), 1), ((50, 8, 8, 16, 512, 16), 1), ((49, 8, 8, 64, 257, 4), 1), ((33, 8, 8, 8, 511, 16), 2),
    # groups on the vector unit, heads apart and together
    ((2, 4, 2, 16, 31, 4), 1), ((4, 16, 8, 8, 60, 20), 1), ((2, 12, 4, 32, 64, 2), 1), ((3, 32, 8, 16, 127, 63), 1),
    ((3, 32, 8, 8, 120, 60), 1), ((8, 32, 8, 64, 100, 32), 1), ((30, 16, 8, 16, 64, 100), 1), ((2, 12, 4, 8, 128, 500), 2),
    # on the matrix cores, apart and together, in one pass and in two
    ((2, 10, 2, 16, 33, 8), 1), ((3, 40, 5, 8, 17, 6), 1), ((3, 64, 8, 16, 64, 16), 1), ((24, 64, 8, 8, 9, 60), 1),
    ((8, 56, 8, 32, 63, 30), 1), ((16, 32, 8, 16, 100, 40), 1), ((16, 32, 8, 8, 128, 64), 1), ((21, 24, 8, 64, 75, 12), 1),
    ((24, 64, 8, 8, 65, 60), 2),
]


def edge_lengths(n, pages, S, rng):
    """The longest row, and sequences that end just before, at and behind page and pass borders."""
    some = [pages * S, 1, (pages - 1) * S + 1, S, S + 1, 16 * S, 16 * S + 1, 64 * S, 128 * S - 1, 128 * S + 1]
    some += [int(x) for x in rng.integers(1, pages * S + 1, n)]
    return np.array([min(max(x, 1), pages * S) for x in some[:n]], np.int32)


def run(shape, launches, flags, write, with_new, seed):
    import torch
    from gpu_util import check_attention, kernel_launches
    B, H, Hkv, S, pages, K = shape
    rng = np.random.default_rng([seed, *shape])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    half = dict(dtype=torch.float16, device="cuda")
    shared, D = 96, 128                                   # full pages may be anybody's; the newest page is one's own
    N = shared + B
    lens = edge_lengths(B, pages, S, rng)
    table = rng.integers(0, shared, (B, pages)).astype(np.int32)
    for b, n in enumerate(lens):
        table[b, (n - 1) // S] = shared + b
        table[b, (n - 1) // S + 1:] = 2 ** 30             # nobody may look up what lies past the sequence
    k_pool = torch.empty((N, Hkv, S, D), **half).normal_(generator=gen)
    v_pool = torch.empty((N, Hkv, S, D), **half).normal_(generator=gen)
    for b, n in enumerate(lens):                          # stale slots
        k_pool[shared + b, :, (n - 1) % S:] = float("nan")
        v_pool[shared + b, :, (n - 1) % S:] = float("nan")
    new = [torch.empty((B, Hkv, D), **half).normal_(generator=gen) for _ in range(2)]
    q = torch.empty((B, H, D), **half).normal_(generator=gen)
    table = torch.from_numpy(table).cuda()
    lens_t = torch.from_numpy(lens).cuda()
    meta = torch.full((Hkv, N, 2, D), float("nan"), **half)
    safe = torch.arange(N, dtype=torch.int32, device="cuda").view(N, 1)   # metadata of every page by itself
    tokens = torch.full((N,), S, dtype=torch.int32, device="cuda")
    tokens[shared:] = (lens_t - 1) % S
    Q.quest_build_meta(Q.Cache(k_pool, v_pool, meta, safe, tokens))
    if not (with_new and write):                          # the token is in the pools already
        for b, n in enumerate(lens):
            k_pool[shared + b, :, (n - 1) % S] = new[0][b]
            v_pool[shared + b, :, (n - 1) % S] = new[1][b]
    if not with_new:
        tokens[shared:] += 1
        Q.quest_build_meta(Q.Cache(k_pool, v_pool, meta, safe, tokens))
    results = []
    for separate in (False, True):
        kp, vp, mt = k_pool.clone(), v_pool.clone(), meta.clone()
        c = Q.Cache(kp, vp, mt, table, lens_t, num_heads=H, flags=flags | (Q.QUEST_FLAG_SEPARATE_LAUNCHES if separate else 0))
        scores = torch.full((B, Hkv, pages), float("nan"), device="cuda")
        idx = torch.full((B, Hkv, K), -7, dtype=torch.int32, device="cuda")
        keff = torch.full((B,), -7, dtype=torch.int32, device="cuda")
        out = torch.full((B, H, D), float("nan"), device="cuda")
        lse = torch.full((B, H), float("nan"), device="cuda")
        ws = torch.zeros(max(Q.quest_step_workspace_bytes(c, K), 16), dtype=torch.uint8, device="cuda")

        def call():
            Q.quest_decode_step(c, new[0] if with_new else None, new[1] if with_new and write else None, write, q, K,
                                1 / math.sqrt(D), scores, idx, out, ws, k_eff=keff, lse=lse)
        if not separate:
            assert kernel_launches(call) == launches
        call()
        torch.cuda.synchronize()
        assert int(ws[:256 * B * H].max()) == 0 if ws.numel() >= 256 * B * H else True
        results.append((scores, idx, keff, mt, kp, vp, out, lse))
    got, want = results
    for name, g, w in zip(("scores", "list", "k_eff", "metadata", "keys", "values"), got, want):
        bits = torch.int32 if g.element_size() == 4 else torch.int16
        assert torch.equal(g.view(bits), w.view(bits)), name
    for name, (_, idx, _, _, kp, vp, out, lse) in (("one call", got), ("separate", want)):
        check_attention(out, lse, q, kp, vp, table, lens_t, idx, 1 / math.sqrt(D), name)


@pytest.mark.parametrize("shape,launches", SHAPES, ids=str)
def test_equals_separate_launches(shape, launches):
    run(shape, launches, 0, True, True, 1)


@pytest.mark.parametrize("flags,write,with_new", [
    (Q.QUEST_FLAG_KEEP_FIRST_PAGE | Q.QUEST_FLAG_KEEP_NEWEST_PAGE, True, True), (Q.QUEST_FLAG_DEVICE_FENCES, True, True),
    (0, False, True), (0, False, False)])
@pytest.mark.parametrize("shape", [(3, 2, 2, 16, 17, 4), (2, 32, 32, 16, 129, 64), (3, 1, 1, 8, 255, 2000), (25, 8, 8, 8, 1024, 33),
                                   (50, 8, 8, 16, 512, 16), (4, 16, 8, 8, 60, 20), (3, 32, 8, 16, 127, 63), (2, 10, 2, 16, 33, 8),
                                   (3, 64, 8, 16, 64, 16), (16, 32, 8, 8, 128, 64)], ids=str)
def test_options(shape, flags, write, with_new):
    run(shape, 1, flags, write, with_new, 2)


@pytest.mark.parametrize("shape,launches", [
    ((1, 8, 8, 16, 256, 32), 1), ((1, 8, 8, 16, 257, 32), 2),                                # up to 8 rows
    ((1, 9, 9, 16, 192, 96), 1), ((1, 9, 9, 16, 193, 20), 2), ((1, 9, 9, 16, 192, 97), 2),   # up to 112
    ((1, 9, 9, 16, 128, 128), 1), ((1, 9, 9, 16, 129, 128), 2), ((2, 56, 56, 8, 192, 9), 1), ((1, 32, 32, 16, 257, 32), 2),
    ((1, 113, 113, 16, 512, 9), 1), ((4, 40, 40, 16, 512, 9), 1), ((4, 40, 40, 16, 513, 9), 2),
    ((1, 161, 161, 16, 1024, 9), 1), ((8, 32, 32, 8, 1024, 300), 1), ((8, 32, 32, 8, 1025, 300), 2),
    ((1, 150, 150, 16, 256, 192), 1), ((1, 150, 150, 16, 257, 192), 2),                      # three splits
    ((1, 257, 257, 16, 256, 9), 1), ((1, 257, 257, 16, 257, 9), 2), ((12, 32, 32, 8, 257, 30), 2),
    ((1, 385, 385, 8, 512, 30), 1), ((16, 32, 32, 64, 512, 16), 1), ((16, 32, 32, 64, 513, 16), 2),
    ((1, 513, 513, 16, 256, 9), 1), ((1, 513, 513, 16, 257, 9), 2), ((5, 205, 205, 16, 63, 9), 2), ((5, 205, 205, 16, 64, 9), 1),
    ((1, 16, 8, 16, 64, 40), 1), ((1, 16, 8, 16, 65, 40), 2),                                # query heads apart
    ((16, 16, 8, 16, 64, 1), 1), ((17, 16, 8, 16, 64, 1), 2), ((18, 40, 5, 16, 1, 1), 2),
    ((8, 32, 8, 16, 128, 64), 1), ((8, 32, 8, 16, 129, 64), 2), ((8, 32, 8, 16, 128, 65), 2),  # together
    ((32, 32, 8, 16, 64, 64), 1), ((33, 32, 8, 16, 64, 64), 2),
    ((8, 64, 8, 16, 64, 30), 1), ((8, 64, 8, 16, 65, 30), 2), ((2, 72, 8, 16, 30, 20), 2),
], ids=str)
def test_where_one_launch_ends(shape, launches):
    """Only captured: nothing runs, so the buffers hold nothing."""
    import torch
    from gpu_util import kernel_launches
    B, H, Hkv, S, pages, K = shape
    pool = torch.empty((1, Hkv, S, 128), dtype=torch.float16, device="cuda")
    meta = torch.empty((Hkv, 1, 2, 128), dtype=torch.float16, device="cuda")
    table, lens = (torch.zeros(n, dtype=torch.int32, device="cuda") for n in ((B, pages), (B,)))
    c = Q.Cache(pool, pool, meta, table, lens, num_heads=H)
    new, q, out = (torch.empty((B, n, 128), dtype=torch.float16, device="cuda") for n in (Hkv, H, H))
    scores, idx = torch.empty((B, Hkv, pages), device="cuda"), torch.empty((B, Hkv, K), dtype=torch.int32, device="cuda")
    ws = torch.zeros(max(Q.quest_step_workspace_bytes(c, K), 16), dtype=torch.uint8, device="cuda")
    assert kernel_launches(lambda: Q.quest_decode_step(c, new, new, True, q, K, 0.1, scores, idx, out, ws)) == launches
