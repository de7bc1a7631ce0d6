"""quest_decode_step with results that lie on inputs, as quest.h allows: out, lse, the list and K_b on the new token's key
and value, fp16 outputs on the query.  The results are those of the same call with buffers of their own, and the step is
one launch only where that reads everything before it writes (short rows are one launch)."""
import math

import pytest

from paper_2406_10774_amd import binding as Q

pytestmark = pytest.mark.gpu
S, D = 16, 128


class Step:
    def __init__(self, B, H, Hkv, pages, K):
        import torch
        gen = torch.Generator(device="cuda").manual_seed(B * H + pages)
        half = dict(dtype=torch.float16, device="cuda", generator=gen)
        self.K, N = K, B * pages
        k_pool, v_pool = (torch.randn((N, Hkv, S, D), **half) for _ in range(2))
        meta = torch.zeros((Hkv, N, 2, D), dtype=torch.float16, device="cuda")
        table = torch.randperm(N, device="cuda", generator=gen).to(torch.int32).view(B, pages)
        lens = torch.tensor([pages * S - 3 * b for b in range(B)], dtype=torch.int32, device="cuda")
        self.cache = Q.Cache(k_pool, v_pool, meta, table, lens, num_heads=H)
        Q.quest_build_meta(self.cache)
        self.q = torch.randn((B, H, D), **half)
        self.new = torch.randn((2, B, Hkv, D), **half)
        self.scores = torch.zeros((B, Hkv, pages), device="cuda")
        self.idx = torch.zeros((B, Hkv, K), dtype=torch.int32, device="cuda")
        self.keff = torch.zeros((B,), dtype=torch.int32, device="cuda")
        self.lse = torch.zeros((B, H), device="cuda")
        self.ws = torch.zeros(Q.quest_step_workspace_bytes(self.cache, K), dtype=torch.uint8, device="cuda")

    def run(self, out, q=None, new=None, **on):
        """One step from the same cache; q, new and the results in the given places, out converted to fp32."""
        import torch
        from gpu_util import kernel_launches
        q, new = self.q if q is None else q, self.new if new is None else new
        idx, keff, lse = (on.get(n, getattr(self, n)) for n in ("idx", "keff", "lse"))

        def call():
            Q.quest_decode_step(self.cache, new[0], new[1], True, q, self.K, 1 / math.sqrt(D), self.scores, idx, out,
                                self.ws, k_eff=keff, lse=lse)
        launches = kernel_launches(call)
        call()
        torch.cuda.synchronize()
        return launches, [t.clone() for t in (out, idx, keff, lse, self.scores)]


# (sequences, query heads, KV heads, pages, pages of the list, whether a work-group has one query head of a group)
SHAPES = [(2, 4, 4, 40, 9, False), (1, 32, 32, 100, 64, False), (3, 16, 8, 60, 40, True), (1, 32, 8, 64, 8, True),
          (4, 32, 8, 50, 50, False), (2, 64, 8, 30, 30, False)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(x) for x in s[:5]))
def test_output_on_the_query(shape):
    import torch
    step = Step(*shape[:5])
    launches, want = step.run(torch.empty_like(step.q))
    assert launches == 1
    q = step.q.clone()
    for _ in range(3):
        launches, got = step.run(q, q=q)
        q.copy_(step.q)
        assert launches == (2 if shape[5] else 1)
        close = (got[0].float() - want[0].float()).abs().max() <= 2 ** -10 * want[0].float().abs().max()   # one rounding to fp16
        assert bool(close) and all(torch.equal(g, w) for g, w in zip(got[1:3] + got[4:], want[1:3] + want[4:]))


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[1], SHAPES[3], SHAPES[4]], ids=lambda s: "x".join(str(x) for x in s[:5]))
@pytest.mark.parametrize("which", ["out", "half", "idx", "keff", "lse"])
def test_results_on_the_new_token(shape, which):
    import torch
    B, H, Hkv = shape[:3]
    step = Step(*shape[:5])
    kind = torch.float16 if which == "half" else torch.float32
    launches, want = step.run(torch.empty((B, H, D), dtype=kind, device="cuda"))
    assert launches == 1
    room = torch.zeros((2 * B * Hkv * D + 2 * B * H * D + 64,), dtype=torch.float16, device="cuda")
    new = room[:2 * B * Hkv * D].view(2, B, Hkv, D)
    dtype, size = {"out": (torch.float32, (B, H, D)), "half": (torch.float16, (B, H, D)), "lse": (torch.float32, (B, H)),
                   "idx": (torch.int32, (B, Hkv, shape[4])), "keff": (torch.int32, (B,))}[which]
    # from the last value vector on, or from the first key on
    for start in ((2 * B * Hkv - 1) * D, 0):
        n = math.prod(size) * torch.empty((), dtype=dtype).element_size() // 2
        if start + n > room.numel():
            continue
        place = room[start:start + n].view(dtype).view(size)
        out = place if which in ("out", "half") else torch.empty((B, H, D), device="cuda")
        on = {} if which in ("out", "half") else {which: place}
        new.copy_(step.new)
        launches, got = step.run(out, new=new, **on)
        assert launches == 2
        limit = 2 ** -10 if kind == torch.float16 else 1e-5        # one rounding to fp16; fp32 sums in another order
        assert float((got[0].float() - want[0].float()).abs().max()) <= limit * float(want[0].float().abs().max())
        assert float((got[3] - want[3]).abs().max()) <= 1e-5
        assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2]) and torch.equal(got[4], want[4])


def test_next_to_each_other():
    """Buffers that only touch are no overlap."""
    import torch
    B, H, Hkv = 2, 4, 4
    step = Step(B, H, Hkv, 40, 9)
    n = B * H * D
    room = torch.zeros((4 * n,), dtype=torch.float16, device="cuda")
    q, new, out = room[:n].view(B, H, D), room[n:3 * n].view(2, B, Hkv, D), room[3 * n:].view(B, H, D)
    q.copy_(step.q)
    new.copy_(step.new)
    assert step.run(out, q=q, new=new)[0] == 1
