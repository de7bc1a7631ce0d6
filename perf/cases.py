"""Performance cases of the Quest decode path: what a serving program asks of this library.

Such a program keeps a paged KV cache and its min/max metadata per layer.  After a prefill
it builds the metadata of the prompt's pages ("build").  For every token it runs one step
per layer: mostly the one-call step ("step"), also the calls one by one where it needs the
page list in between ("calls"), and attention over all pages in the layers it keeps dense
("dense").  A pass covers `layers` layers with buffers of their own, as the layers of a
model have them, so keys and metadata come from memory rather than from a cache that the
previous pass filled.  With `graph` the program has captured a token's calls in a HIP graph
and replays it; otherwise it makes the calls one after the other.

Fields of a case: kind; layers; batch; heads and kv_heads (query heads and KV heads of
128 channels); page (tokens per page); tokens and shortest (longest and shortest sequence,
the new token of a step counted); budget (tokens attended per head); shuffled (physical
pages in random order, as an allocator leaves them after a while, or one after the other);
half_out (fp16 output instead of fp32); keep (first and newest page always selected);
graph.
"""
import math

import torch

from paper_2406_10774_amd import binding as Q

HEAD_DIM = 128
ROOM = 64                  # tokens of room that a page-table row has behind the longest sequence
PLANTED = 64               # tokens per head that resemble the query
MAX_POOL_BYTES = 10.0e9    # keys + values of all layers of a drawn case
MAX_PASS_BYTES = 1.1e9     # bytes a pass of a drawn case has to move


def _case(name, kind, tokens, **more):
    case = dict(name=name, kind=kind, layers=1, batch=1, heads=32, kv_heads=32, page=16, tokens=tokens,
                shortest=tokens, budget=2048, shuffled=False, half_out=False, keep=False, graph=False)
    case.update(more)
    return case


def listed():
    return [
        # the smallest call: one head, short context, nothing but launches and latency
        _case("step 1 head 4k", "step", 4096, heads=1, kv_heads=1, budget=512),
        # the benchmark's shape (32 heads, 32k context, 2048-token budget) as a serving loop
        # replays it for one user
        _case("step 32k graph", "step", 32769, layers=8, graph=True),
        # the same size of model in a plain loop of calls: a chat of some thousand tokens,
        # pages scattered over the pool, fp16 activations
        _case("step 7k", "step", 6997, layers=8, budget=1024, shuffled=True, half_out=True),
        # long documents: 128k and 512k tokens with a 4096-token budget
        _case("step 128k", "step", 131073, layers=2, budget=4096),
        _case("step 512k", "step", 524289, budget=4096),
        # continuous batching: sixteen ragged sequences of 8k to 64k tokens
        _case("step batch 16", "step", 65519, batch=16, shortest=8209, shuffled=True),
        # grouped-query attention, a small batch of ragged sequences
        _case("step GQA batch 4", "step", 32771, layers=4, batch=4, kv_heads=8, shortest=9001,
              shuffled=True, half_out=True, graph=True),
        # pages of 64 tokens, first and newest page kept, some sequences below the budget
        _case("step page 64 ragged", "step", 20011, layers=4, batch=6, shortest=700, page=64, budget=1024,
              keep=True, shuffled=True),
        # the calls one by one, smallest pages
        _case("calls page 8", "calls", 32769, layers=4, page=8, shuffled=True),
        # after a prefill: metadata of two layers of a 32k prompt
        _case("build 32k", "build", 32749, layers=2),
        # dense layers and the dense fall-back: multi-head, and grouped-query on a ragged batch
        _case("dense 32k", "dense", 32769, layers=2),
        _case("dense GQA batch 4", "dense", 32771, layers=2, batch=4, kv_heads=8, shortest=5003,
              shuffled=True, half_out=True),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "calls", "build", "dense"])
    heads, kv_heads = rng.choice([(32, 32), (32, 32), (40, 40), (8, 8), (32, 8), (64, 8), (16, 8)])
    case = _case("", kind, _spread(rng, 300, 500000), heads=heads, kv_heads=kv_heads,
                 layers=rng.randint(1, 8), batch=_spread(rng, 1, 16), page=rng.choice([16, 16, 16, 8, 32, 64]),
                 budget=_spread(rng, 256, 4096), shuffled=rng.random() < 0.6, half_out=rng.random() < 0.5,
                 keep=rng.random() < 0.3, graph=rng.random() < 0.3)
    ragged = rng.uniform(0.1, 1.0)
    del case["name"]
    while True:
        case["shortest"] = max(2, int(case["tokens"] * ragged)) if case["batch"] > 1 else case["tokens"]
        pools = case["layers"] * sum(_lens(case)) * kv_heads * HEAD_DIM * 4
        if pools <= MAX_POOL_BYTES and work(case)["bytes"] <= MAX_PASS_BYTES:
            return case
        if case["layers"] > 1:
            case["layers"] -= 1
        elif case["batch"] > 1:
            case["batch"] -= 1
        else:
            case["tokens"] = case["tokens"] * 3 // 4


def _lens(case):
    """Tokens of each sequence: evenly spaced from shortest to longest, in mixed order."""
    n = case["batch"]
    order = sorted(range(n), key=lambda i: (i * 0.618034) % 1.0)
    lens = [case["tokens"]] * n
    for rank, b in enumerate(order):
        if rank:
            lens[b] -= (case["tokens"] - case["shortest"]) * rank // (n - 1)
    return lens


def _pages(case):
    return [-(-n // case["page"]) for n in _lens(case)]


def _k_pages(case):
    return max(1, case["budget"] // case["page"])


def work(case):
    H, Hkv, S, K = case["heads"], case["kv_heads"], case["page"], _k_pages(case)
    row = 2 * HEAD_DIM                                        # one fp16 vector
    lens, pages = _lens(case), _pages(case)
    n_out = case["batch"] * H * HEAD_DIM * (2 if case["half_out"] else 4) + case["batch"] * H * 4
    if case["kind"] == "build":
        moved = sum(Hkv * (n * row + p * 2 * row) for n, p in zip(lens, pages))
        return {"bytes": case["layers"] * moved, "flops": case["layers"] * 2 * HEAD_DIM * Hkv * sum(lens)}
    if case["kind"] == "dense":
        moved = sum(Hkv * n * 2 * row for n in lens) + case["batch"] * H * row + n_out
        return {"bytes": case["layers"] * moved, "flops": case["layers"] * 4 * HEAD_DIM * H * sum(lens)}
    moved = n_out + case["batch"] * (H + 4 * Hkv) * row       # query; new key and value, read and stored
    flops = 0
    for n, p in zip(lens, pages):
        chosen = min(K, p)
        attended = min(n, chosen * S)
        moved += Hkv * (p * (2 * row + 4) + attended * 2 * row + K * 4)
        flops += 4 * HEAD_DIM * H * (p + attended)
    return {"bytes": case["layers"] * moved, "flops": case["layers"] * flops}


def tolerance(case):
    """Four times what the path differs by from itself in 64-bit arithmetic: 5.5e-6 with fp32
    outputs (512k tokens; 3e-8 to 7e-8 for scores and lse), 2.1e-4 with fp16 outputs (their
    own rounding; values up to one unit in the last place apart).  Page lists and the cache
    itself came out the same."""
    if case["kind"] == "build":
        return "exact"
    return {"rel": 8e-4, "max": 2e-3} if case["half_out"] else {"rel": 2e-5, "max": 8e-4}


def _tables(case, gen):
    """Page table [batch][pages with room] and the number of physical pages."""
    pages = _pages(case)
    width = -(-(case["tokens"] + ROOM) // case["page"])
    total = sum(pages) + 2
    order = torch.randperm(total, generator=gen, device="cuda") if case["shuffled"] \
        else torch.arange(total, device="cuda")
    table = torch.zeros((case["batch"], width), dtype=torch.int32, device="cuda")
    at = 0
    for b, p in enumerate(pages):
        table[b, :p] = order[at:at + p].int()
        at += p
    return table, total


def _fill_keys(keys, case, table, q, gen):
    """Keys that drift along the context (so pages differ), with a few strong channels per
    head and some tokens that resemble the query."""
    N, H, S, D = keys.shape
    keys.normal_(generator=gen)
    drift = torch.zeros((N, H, D), dtype=torch.float16, device="cuda")
    for b, p in enumerate(_pages(case)):
        walk = torch.randn((p, H, D), generator=gen, device="cuda") * 0.3
        walk[0] = 0
        drift[table[b, :p].long()] = walk.cumsum_(0).half()
    keys += drift.unsqueeze(2)
    strong = torch.rand((H, D), generator=gen, device="cuda").argsort(1)[:, :4]
    scale = torch.ones((H, D), dtype=torch.float16, device="cuda").scatter_(1, strong, 8.0)
    keys *= scale.view(1, H, 1, D)
    head = torch.arange(H, device="cuda").unsqueeze(1)
    for b, n in enumerate(_lens(case)):
        pos = (torch.rand((H, PLANTED), generator=gen, device="cuda") * n).long().clamp_(max=n - 1)
        like = q[b, ::case["heads"] // H].float()
        like = (3 * like / like.norm(dim=1, keepdim=True)).half()
        keys[table[b].long()[pos // S], head, pos % S] = like.unsqueeze(1).expand(H, PLANTED, D)
    return drift, scale


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    L, B, H, Hkv, S, D = case["layers"], case["batch"], case["heads"], case["kv_heads"], case["page"], HEAD_DIM
    K = _k_pages(case)
    half = dict(dtype=torch.float16, device="cuda")
    table, N = _tables(case, gen)
    lens = torch.tensor(_lens(case), dtype=torch.int32, device="cuda")
    flags = (Q.QUEST_FLAG_KEEP_FIRST_PAGE | Q.QUEST_FLAG_KEEP_NEWEST_PAGE) if case["keep"] else 0
    st = dict(case=case, k_pages=K, scale=1 / math.sqrt(D), table=table, lens=lens)
    st["k_pool"] = torch.empty((L, N, Hkv, S, D), **half)
    st["v_pool"] = torch.empty((L, N, Hkv, S, D), **half).normal_(generator=gen)
    st["meta"] = torch.zeros((L, Hkv, N, 2, D), **half)
    st["q"] = torch.empty((L, B, H, D), **half).normal_(generator=gen)
    st["k_new"] = torch.empty((L, B, Hkv, D), **half).normal_(generator=gen)
    st["v_new"] = torch.empty((L, B, Hkv, D), **half).normal_(generator=gen)
    st["scores"] = torch.zeros((L, B, Hkv, table.shape[1]), device="cuda")
    st["list"] = torch.zeros((L, B, Hkv, K), dtype=torch.int32, device="cuda")
    st["k_eff"] = torch.zeros((L, B), dtype=torch.int32, device="cuda")
    st["out"] = torch.zeros((L, B, H, D), dtype=torch.float16 if case["half_out"] else torch.float32, device="cuda")
    st["lse"] = torch.zeros((L, B, H), device="cuda")
    st["caches"], st["steps"] = [], []
    newest = [(b, (n - 1) // S) for b, n in enumerate(_lens(case))]
    for l in range(L):
        drift, scale = _fill_keys(st["k_pool"][l], case, table, st["q"][l], gen)
        for b, p in newest:                                   # the new token goes on where the keys are
            st["k_new"][l, b].add_(drift[table[b, p].long()]).mul_(scale)
        pools = (st["k_pool"][l], st["v_pool"][l], st["meta"][l], table)
        if case["kind"] != "build":                           # everything but the new token is in the metadata
            Q.quest_build_meta(Q.Cache(*pools, lens - 1, num_heads=H))
        st["caches"].append(Q.Cache(*pools, lens, flags=flags, num_heads=H))
        st["steps"].append({k: st[k][l] for k in ("q", "k_new", "v_new", "scores", "list", "k_eff", "out", "lse")})
    c = st["caches"][0]
    dense = case["kind"] == "dense"
    nbytes = Q.quest_workspace_bytes(c, 0 if dense else K) if case["kind"] != "step" \
        else Q.quest_step_workspace_bytes(c, K)
    st["workspace"] = torch.zeros(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    st["topk_workspace"] = None
    if case["kind"] == "calls" and Q.quest_topk_workspace_bytes(c, K):
        st["topk_workspace"] = torch.zeros(Q.quest_topk_workspace_bytes(c, K), dtype=torch.uint8, device="cuda")
    st["graph"] = None
    if case["graph"]:
        _calls(st)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _calls(st)
        st["graph"] = graph
    return st


def _calls(st):
    kind, K, scale, ws = st["case"]["kind"], st["k_pages"], st["scale"], st["workspace"]
    for cache, x in zip(st["caches"], st["steps"]):
        if kind == "step":
            Q.quest_decode_step(cache, x["k_new"], x["v_new"], True, x["q"], K, scale, x["scores"], x["list"],
                                x["out"], ws, k_eff=x["k_eff"], lse=x["lse"])
        elif kind == "calls":
            Q.quest_append_meta(cache, x["k_new"], x["v_new"], True)
            Q.quest_estimate(cache, x["q"], x["scores"])
            Q.quest_topk(cache, x["scores"], K, x["list"], x["k_eff"], st["topk_workspace"])
            Q.quest_sparse_decode(cache, x["q"], x["list"], K, scale, x["out"], x["lse"], ws)
        elif kind == "build":
            Q.quest_build_meta(cache)
        else:
            Q.quest_sparse_decode(cache, x["q"], None, 0, scale, x["out"], x["lse"], ws)


def run(st):
    if st["graph"] is not None:
        st["graph"].replay()
    else:
        _calls(st)
    kind = st["case"]["kind"]
    if kind == "build":
        return {"meta": st["meta"]}
    if kind == "dense":
        return {"out": st["out"], "lse": st["lse"]}
    return {k: st[k] for k in ("out", "lse", "list", "k_eff", "scores", "meta", "k_pool", "v_pool")}
