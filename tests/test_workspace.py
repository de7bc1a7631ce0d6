"""One workspace serves every call on a cache shape, as quest.h says: dense or with any list
length, with and without QUEST_FLAG_SEPARATE_LAUNCHES, whichever call its size was asked for.
The host decides that before anything is launched; on a machine without a GPU an accepted call
then ends with QUEST_ERR_HIP."""
import ctypes
import random

import pytest

from paper_2406_10774_amd import binding

WORKSPACE, HIP = -4, -5


def on_host_only():
    import torch
    if torch.cuda.is_available():
        pytest.skip("the pointers of these calls point nowhere")


def make_cache(batch, kv_heads, group, page_size, pages, flags=0):
    return binding.quest_cache(batch=batch, num_heads=kv_heads * group, head_dim=128, page_size=page_size,
                               max_pages_per_seq=pages, flags=flags, num_phys_pages=64, k_pool=0x1000,
                               v_pool=0x1000, meta=0x1000, page_table=0x1000, seq_lens=0x1000,
                               num_kv_heads=kv_heads if group > 1 else 0)


def size_of(c, k_pages, step=False):
    lib, out = binding.load(), ctypes.c_size_t(0)
    query = lib.quest_step_workspace_bytes if step else lib.quest_workspace_bytes
    assert query(ctypes.byref(c), k_pages, ctypes.byref(out)) == 0
    return out.value


def call(kind, c, k_pages, nbytes):
    lib, r, p = binding.load(), ctypes.byref(c), 0x1000
    ws = p if nbytes else None
    if kind == "dense":
        return lib.quest_sparse_decode(r, p, None, 0, 1.0, p, 0, None, ws, nbytes, None)
    if kind == "list":
        return lib.quest_sparse_decode(r, p, p, k_pages, 1.0, p, 0, None, ws, nbytes, None)
    if kind == "select":
        return lib.quest_select_decode(r, p, p, k_pages, 1.0, p, None, p, 0, None, ws, nbytes, None)
    return lib.quest_decode_step(r, None, None, 0, p, k_pages, 1.0, p, p, None, p, 0, None, ws, nbytes, None)


@pytest.mark.parametrize("pages,asked,used,asked_flags", [
    (16384, 600, 500, 0), (20000, 600, 400, 0), (24000, 400, 330, 0), (16384, 256, 256, 1), (32769, 4000, 3, 0),
    (16384, 0, 300, 0), (2048, 25, 24, 0), (2048, 16, 128, 0), (128, 0, 100, 0), (40000, 5, 1600, 0),
])
@pytest.mark.parametrize("kind", ["dense", "list", "select", "step"])
def test_one_workspace_for_all_list_lengths(kind, pages, asked, used, asked_flags):
    on_host_only()
    for kv_heads, group in ((32, 1), (4, 8), (1, 1)):
        nbytes = size_of(make_cache(1, kv_heads, group, 16, pages, asked_flags), asked)
        if pages < 16384 and asked_flags == 0:
            assert nbytes == size_of(make_cache(1, kv_heads, group, 16, pages), used)
        assert call(kind, make_cache(1, kv_heads, group, 16, pages), used, nbytes) == HIP


def test_one_workspace_on_drawn_shapes():
    on_host_only()
    rng = random.Random(7)
    spread = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    for _ in range(4000):
        shape = (spread(1, 64), rng.choice([1, 2, 8, 12, 29, 32, 40]), rng.choice([1, 1, 2, 4, 5, 8, 9]),
                 rng.choice([8, 16, 32, 64]), spread(1, 70000))
        asked, used = rng.choice([0, spread(1, 4200)]), spread(1, 4200)
        flags = rng.choice([0, 1]), rng.choice([0, 1])
        kind = rng.choice(["dense", "list", "select", "step"])
        nbytes = size_of(make_cache(*shape, flags[0]), asked, step=asked > 0 and rng.random() < 0.5)
        assert call(kind, make_cache(*shape, flags[1]), used, nbytes) == HIP, (shape, asked, used, flags, kind)


@pytest.mark.parametrize("group", [1, 2, 8])
def test_the_benchmark_knows_which_rows_are_selected_whole(group):
    """Where a step is two launches: the library keeps no candidates there."""
    import bench
    for pages in (4096, 4097, 5120, 5121, 8192, 8704, 8705, 12500):
        candidates = size_of(make_cache(1, 32, group, 16, pages), 0) - size_of(make_cache(1, 32, group, 16, pages, 1), 0)
        assert bench.selects_inside(pages, 2048, group > 1) == (candidates == 0)
        assert not bench.selects_inside(pages, 2049, group > 1)


@pytest.mark.parametrize("kind,batch,kv_heads,group,page_size,pages,k_pages,accepted", [
    ("dense", 1, 32, 1, 16, 4, 0, True), ("dense", 1, 32, 1, 16, 5, 0, False), ("dense", 8, 32, 1, 16, 16, 0, True),
    ("dense", 8, 32, 1, 16, 17, 0, False), ("dense", 9, 29, 1, 16, 2048, 0, True), ("dense", 9, 8, 4, 16, 2048, 0, True),
    ("list", 1, 32, 1, 16, 2048, 16, True), ("list", 1, 32, 1, 16, 2048, 17, False),
    ("list", 1, 32, 1, 64, 2048, 1, True), ("list", 4, 32, 1, 16, 2048, 128, False),
    ("list", 129, 1, 1, 16, 2048, 128, True), ("list", 257, 1, 2, 16, 2048, 128, True),
    ("select", 1, 32, 1, 16, 2048, 17, False), ("step", 1, 32, 1, 16, 2048, 16, True),
    ("step", 1, 32, 1, 16, 16384, 16, False), ("step", 9, 32, 1, 16, 16384, 16, False),
    ("step", 9, 32, 1, 16, 16383, 64, True),
])
def test_calls_without_a_workspace(kind, batch, kv_heads, group, page_size, pages, k_pages, accepted):
    """The rule that quest.h states for a workspace of no or too few bytes."""
    on_host_only()
    c = make_cache(batch, kv_heads, group, page_size, pages)
    for nbytes in (0, 64):
        assert call(kind, c, k_pages, nbytes) == (HIP if accepted else WORKSPACE)


@pytest.mark.parametrize("batch,kv_heads,group,page_size,pages,counters,heads,candidates", [
    # (heads: partial results of one query head, of max, denominator and 128 channels each)
    (1, 32, 1, 16, 2048, 32, 192 * 2 * 4, 0),           # equal shares, two slots of four heads each
    (1, 36, 1, 64, 800, 36, 192 * 2 * 4, 0),
    (1, 33, 1, 16, 2048, 33, 192 * 2, 0),               # heads one by one
    (4, 8, 4, 16, 2048, 128, 224 * 2 * 8, 0),           # groups, slots of eight heads
    (2, 4, 12, 16, 6144, 96, 224 * 2 * 8, 2 * 4 * 3072),
    (1, 32, 1, 8, 4096, 32, 256 * 2 * 4, 0),            # pages of 8 tokens
    (1, 32, 1, 16, 100, 32, 32 * 8, 0),                 # little work: eight splits of a row
    (64, 32, 1, 16, 8, 2048, 0, 0),                     # one split
    (3, 32, 1, 8, 150, 96, 96 * 5, 0),                  # pages of 8 tokens: two work-groups per unit
    (1, 1, 1, 16, 16, 1, 0, 0), (1, 8, 4, 16, 500, 32, 32 * 31, 0),
    (1, 32, 1, 16, 16384, 32, 192 * 2 * 4, 32 * 8192),  # very long rows: candidates behind
    (1, 32, 1, 16, 8704, 32, 192 * 2 * 4, 0), (1, 32, 1, 16, 8705, 32, 192 * 2 * 4, 32 * 4096),  # whole rows, candidates
    (1, 8, 4, 16, 5120, 32, 32 * 32, 0), (1, 8, 4, 16, 5121, 32, 32 * 32, 8 * 2560),  # (32 splits of a list)
])
def test_size_is_that_of_the_layout(batch, kv_heads, group, page_size, pages, counters, heads, candidates):
    """Counters, then partial results of dense attention or of the most splits of a list, then
    candidates, as the kernels lay them out."""
    c = make_cache(batch, kv_heads, group, page_size, pages)
    assert size_of(c, 0) == counters * 256 + heads * 130 * 4 + candidates * 8
