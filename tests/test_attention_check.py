"""check_attention, the limit of the GPU tests on attention over a list, on the CPU: fp32 attention in another order passes, an
output that left a token out, or attended one twice, does not."""
import math

import pytest
import torch

from gpu_util import check_attention

D = 128


def attention(q, k, v, scale, order, times):
    """fp32 attention of q [H][D] over k, v [Hkv][T][D], tokens in the given order, each taken times[t] times."""
    k, v, w = k[:, order], v[:, order], times[order].float()
    k, v = (x.repeat_interleave(len(q) // len(x), 0) for x in (k, v))
    logits = (k * q[:, None]).sum(-1) * scale
    top = logits.max(-1, keepdim=True).values
    p = (logits - top).exp() * w
    return (p[..., None] * v).sum(1) / p.sum(-1, keepdim=True), top[:, 0] + p.sum(-1).log()


@pytest.mark.parametrize("B,H,Hkv,S,K,last", [(1, 2, 2, 16, 4, 16), (2, 4, 1, 8, 64, 3), (1, 8, 8, 16, 64, 16), (1, 4, 2, 64, 32, 1)])
def test_finds_a_token_too_few_or_too_many(B, H, Hkv, S, K, last):
    gen = torch.Generator().manual_seed(S * K)
    N, scale = B * K, 1 / math.sqrt(D)
    k_pool, v_pool = (torch.randn((N, Hkv, S, D), generator=gen).half() for _ in range(2))
    q = torch.randn((B, H, D), generator=gen).half()
    table = torch.randperm(N, generator=gen).view(B, K)
    n = (K - 1) * S + last
    lens = torch.full((B,), n)
    lists = torch.arange(K).expand(B, Hkv, K)

    def run(times):
        outs = [attention(q[b].float(), *(pool[table[b]].transpose(0, 1).flatten(1, 2)[:, :n].float() for pool in (k_pool, v_pool)),
                          scale, torch.randperm(n, generator=gen), times) for b in range(B)]
        return (torch.stack(x) for x in zip(*outs))

    once = torch.ones(n)
    check_attention(*run(once), q, k_pool, v_pool, table, lens, lists, scale)
    for token in (0, n // 2, n - 1):
        for count in (0, 2):
            times = once.clone()
            times[token] = count
            out, lse = run(times)
            with pytest.raises(AssertionError):
                check_attention(out, lse, q, k_pool, v_pool, table, lens, lists, scale)
