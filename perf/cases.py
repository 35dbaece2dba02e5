"""Workloads that measure the tree decode-attention library through its Python binding.

Every case is a search forest as a serving program holds it for one transformer layer: queries
(roots) with a prompt, steps below them, pages scattered over the pool as after long serving.
`op` says which call of the program is timed:

  decode    one decode_attention call (masked where `masks`) over the leaves, plan cached, as every
            layer after the first of a decode iteration sees it; q_len queries per leaf
  generate  a step generated token by token: every leaf gets a child, then per token one
            append_tokens and one decode_attention over all branches, then the children are pruned
  write     finished tokens written into the cache (a fresh node each, append_step), read back
            with gather_kv as for moving a query elsewhere, and pruned

Trees are drawn from the case's own `tree_seed`; keys, values and queries from the seed given to
`prepare`.  Keys and values are N(0, 1), queries N(0, 4): scores have a spread of about 2, so a
softmax has a few dominant tokens and a long tail, as in trained models.
"""

import math

import numpy as np
import torch

NO_NODE = -1
_ESZ = {"f32": 4, "bf16": 2, "fp8_e4m3": 1}
_SRC = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8_e4m3": torch.bfloat16}
_DEV = "cuda"


def _case(op, tree, queries, prompt, step, *, heads=(32, 8, 128), kv="bf16", page=16, width=16, depth=5,
          ragged=False, q_len=1, masks=False, iters=0, pieces=1, tree_seed=1, name=None):
    c = dict(op=op, tree=tree, queries=queries, prompt=prompt, step=step, q_heads=heads[0], kv_heads=heads[1],
             head_dim=heads[2], kv=kv, page=page, width=width, depth=depth, ragged=ragged, q_len=q_len, masks=masks,
             iters=iters, pieces=pieces, tree_seed=tree_seed)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a first small search in full precision (correctness work, toy models): launches and latency
        _case("decode", "bfs", 1, 256, 64, heads=(8, 2, 64), kv="f32", width=4, depth=1, name="tiny_fp32"),
        # one user's breadth-first search of width 16: the batch-of-one serving case
        _case("decode", "bfs", 1, 512, 128, name="one_query_bf16"),
        # a batch of such searches, the ordinary serving load
        _case("decode", "bfs", 32, 512, 128, tree_seed=2, name="bfs_bf16"),
        # skewed Monte-Carlo trees with steps of every length and 7 query heads per kv head
        _case("decode", "mcts", 64, 1024, 256, heads=(28, 4, 128), width=64, depth=10, ragged=True, tree_seed=3,
              name="mcts_ragged_bf16"),
        # speculation at scale: long prompts, 8192 branches, 64 query heads, the largest launch
        _case("decode", "chain", 256, 2048, 256, heads=(64, 8, 128), width=32, depth=4, tree_seed=4,
              name="spec_at_scale_bf16"),
        # token trees of drafts verified against an fp8 cache
        _case("decode", "binary", 64, 1024, 128, heads=(40, 8, 128), kv="fp8_e4m3", depth=3, q_len=6, masks=True,
              tree_seed=5, name="drafts_fp8"),
        # a reward model reads every branch's newest step at once (prefill of a step over its prefix)
        _case("decode", "bfs", 32, 512, 128, q_len=128, tree_seed=6, name="step_prefill_bf16"),
        # few branches over very long prompts: little batch, long paths
        _case("decode", "bfs", 4, 16000, 1100, width=4, depth=1, tree_seed=7, name="long_prompt_bf16"),
        # a pool with the page size of another engine (32 tokens), ragged steps
        _case("decode", "bfs", 8, 512, 128, page=32, ragged=True, tree_seed=8, name="page32_bf16"),
        # prompts written into the cache after prefill, and read back
        _case("write", "nodes", 8, 2048, 0, tree_seed=9, name="write_prompts_bf16"),
        # the ragged steps of a frontier of 16 quantised into an fp8 cache, each arriving in two pieces
        _case("write", "nodes", 16, 256, 0, kv="fp8_e4m3", ragged=True, pieces=2, tree_seed=10,
              name="write_steps_fp8"),
        # sixteen tokens of every branch generated one at a time, branches forked before and pruned after
        _case("generate", "bfs", 8, 512, 128, iters=16, tree_seed=11, name="generate_bf16"),
    ]


_HEADS = [(32, 8, 128), (28, 4, 128), (64, 8, 128), (40, 8, 128), (16, 4, 128), (8, 2, 128), (16, 2, 64), (8, 2, 64)]
_OTHER = [((32, 8, 128), 32), ((8, 2, 128), 64), ((6, 3, 40), 16), ((16, 4, 256), 16), ((8, 2, 64), 8),
          ((12, 4, 96), 16)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        op = rng.choices(["decode", "prefill", "generate", "write"], [11, 3, 3, 3])[0]
        seed = rng.randrange(1 << 30)
        if op == "write":
            kv = rng.choice(["bf16", "bf16", "fp8_e4m3", "f32"])
            heads, page = rng.choice([(h, 16) for h in _HEADS] + _OTHER)
            c = _case("write", "nodes", _log(rng, 1, 16), _log(rng, 16, 8192), 0, heads=heads, kv=kv, page=page,
                      ragged=rng.random() < 0.7, pieces=rng.choice([1, 2]), tree_seed=seed)
        else:
            kv = rng.choices(["bf16", "fp8_e4m3", "f32"], [6, 3, 2])[0]
            heads, page = rng.choice(_HEADS), 16
            if rng.random() < 0.2:
                heads, page = rng.choice(_OTHER)
            tree = rng.choice(["bfs", "mcts", "chain", "binary"]) if op == "decode" else "bfs"
            width = {"bfs": rng.choice([4, 8, 16]), "mcts": _log(rng, 2, 64), "chain": _log(rng, 4, 32), "binary": 2}[tree]
            depth = {"bfs": rng.randint(1, 5), "mcts": 10, "chain": rng.randint(1, 4), "binary": rng.randint(1, 4)}[tree]
            q_len = rng.choice([1, 1, 1, rng.randint(2, 16)]) if op == "decode" else 1
            step = _log(rng, 16, 256)
            c = _case("generate" if op == "generate" else "decode", tree, _log(rng, 1, 256), _log(rng, 64, 16000), step,
                      heads=heads, kv=kv, page=page, width=width, depth=depth, ragged=rng.random() < 0.6,
                      q_len=step if op == "prefill" else q_len, masks=op == "decode" and q_len > 1 and rng.random() < 0.5,
                      iters=rng.randint(4, 24) if op == "generate" else 0, tree_seed=seed)
        w = work(c)
        rows = w["flops"] / (4.0 * c["head_dim"])          # pairs of a query row and a visible token
        tiled = c["kv"] != "f32" and c["page"] == 16 and c["head_dim"] in (64, 128)
        if w["bytes"] < 4e9 and w["flops"] < 8e11 and (tiled or rows < 4e7):
            return c


# ---- shapes ------------------------------------------------------------------------------------
def _shape(case):
    """(parent, tokens, leaves): the live forest, parents before children."""
    rng = np.random.default_rng(case["tree_seed"])
    parent, tokens, leaves = [], [], []
    length = (lambda n: int(rng.integers(max(1, n // 8), n + 1))) if case["ragged"] else (lambda n: n)

    def node(par, n):
        parent.append(par)
        tokens.append(n)
        return len(parent) - 1

    step, width, depth = case["step"], case["width"], case["depth"]
    for _ in range(case["queries"]):
        root = node(NO_NODE, length(case["prompt"]))
        if case["tree"] == "nodes":
            leaves.append(root)
        elif case["tree"] == "bfs":            # `width` branches a level; a quarter survives and forks again
            keep = max(1, width // 4)
            kept = [root]
            for d in range(depth):
                level = [(p, length(step)) for p in kept for _ in range(width // len(kept))]
                if d + 1 < depth:
                    level = [level[i] for i in sorted(rng.choice(len(level), keep, replace=False).tolist())]
                kept = [node(p, n) for p, n in level]
            leaves.extend(kept)
        elif case["tree"] == "mcts":           # mostly extends the best path, sometimes forks elsewhere
            target = max(1, min(width, int(2.0 ** rng.uniform(0.0, math.log2(max(width, 2))))))
            deep, kids, tip, ends = {root: 0}, {root: 0}, root, 1
            while ends < target:
                open_nodes = [u for u in deep if deep[u] < depth]
                u = tip if deep[tip] < depth and rng.random() < 0.7 else open_nodes[int(rng.integers(0, len(open_nodes)))]
                new = [node(u, length(step)) for _ in range(int(rng.integers(1, 5)))]
                ends += len(new) - (1 if kids[u] == 0 else 0)
                kids[u] += len(new)
                for c in new:
                    deep[c], kids[c] = deep[u] + 1, 0
                if u == tip:
                    tip = new[0]
            leaves.extend(u for u in deep if kids[u] == 0)
        elif case["tree"] == "chain":          # speculative branches off the nodes of a primary chain
            chain = [root]
            for _d in range(1, depth):
                chain.append(node(chain[-1], length(step)))
            at = np.minimum(rng.geometric(0.5, size=width), depth)
            leaves.extend(node(chain[int(d) - 1], length(step)) for d in at)
        else:                                  # binary: every node of a level has two children
            level = [root]
            for _d in range(depth):
                level = [node(u, length(step)) for u in level for _ in range(2)]
            leaves.extend(level)
    live = sorted({w for u in leaves for w in _path(parent, u)})   # what lost every branch is pruned
    new_id = {u: i for i, u in enumerate(live)}
    parent, tokens = [new_id.get(parent[u], NO_NODE) for u in live], [tokens[u] for u in live]
    leaves = [new_id[u] for u in leaves]
    q_len = case["q_len"]
    if case["masks"]:                          # the drafts are tokens of their own behind the step
        for u in leaves:
            tokens[u] += q_len
    return parent, tokens, leaves


def _path(parent, u):
    p = []
    while u != NO_NODE:
        p.append(u)
        u = parent[u]
    return p[::-1]


def _requests(case):
    """Tree, requested nodes, queries per request and their draft masks."""
    parent, tokens, leaves = _shape(case)
    total = {}
    for u in range(len(parent)):
        total[u] = tokens[u] + (total[parent[u]] if parent[u] != NO_NODE else 0)
    q_lens = [min(case["q_len"], tokens[u]) for u in leaves]
    masks = None
    if case["masks"]:                          # a draft's parent is one of the drafts before it
        rng = np.random.default_rng(case["tree_seed"] + 1)
        masks = []
        for n in q_lens:
            own = [1]
            for j in range(1, n):
                own.append(own[int(rng.integers(0, j))] | (1 << j))
            masks += own
    return parent, tokens, leaves, total, q_lens, masks


def work(case):
    Hq, Hkv, D, esz = case["q_heads"], case["kv_heads"], case["head_dim"], _ESZ[case["kv"]]
    qsz = 4 if case["kv"] == "f32" else 2
    parent, tokens, leaves, total, q_lens, masks = _requests(case)
    per_token = 2.0 * Hkv * D * esz + (8.0 * Hkv / case["page"] if esz == 1 else 0.0)
    n = float(sum(tokens))
    if case["op"] == "write":                  # source read, cache written, cache read, copy written
        return {"bytes": n * (2.0 * Hkv * D * (_SRC[case["kv"]].itemsize + esz) + 2 * per_token), "flops": 0.0}
    row = Hq * (D * (qsz + 4.0) + 4.0)         # query read, output and lse written
    if case["op"] == "decode":
        seen = 0.0
        at = 0
        for u, ql in zip(leaves, q_lens):
            if masks:
                seen += ql * (total[u] - ql) + sum(bin(m).count("1") for m in masks[at:at + ql])
            else:
                seen += ql * (total[u] - ql) + ql * (ql + 1) / 2
            at += ql
        return {"bytes": n * per_token + at * row, "flops": 4.0 * D * Hq * seen}
    T, B = case["iters"], len(leaves)
    seen = sum(T * total[u] for u in leaves) + B * T * (T + 1) / 2.0
    kv = T * n * per_token + B * (T * (T + 1) / 2.0) * per_token
    new = B * T * (2.0 * Hkv * D * _SRC[case["kv"]].itemsize + per_token)
    return {"bytes": kv + new + T * B * row, "flops": 4.0 * D * Hq * seen}


def tolerance(case):
    if case["op"] == "write":
        return "exact"
    # fp32 sums: 7e-7 measured against 64 bits.  Tiled 16-bit and fp8 caches round a softmax weight
    # once to half precision: 2e-4 (bf16) and 3.7e-4 (fp8).
    if case["kv"] == "f32" or case["page"] != 16 or case["head_dim"] not in (64, 128):
        return {"rel": 5e-6}
    return {"rel": 1.5e-3 if case["kv"] == "fp8_e4m3" else 1e-3}


# ---- inputs ------------------------------------------------------------------------------------
def _gen(seed, tag):
    return torch.Generator(device=_DEV).manual_seed((seed * 8 + tag) % (1 << 62))


def _normal(shape, dtype, seed, tag, scale=1.0):
    x = torch.randn(shape, generator=_gen(seed, tag), device=_DEV, dtype=dtype)
    return x if scale == 1.0 else x * scale


def _pages(tokens, page):
    return [-(-n // page) for n in tokens]


def _scales(amax):
    """Page scale of an fp8 cache and its reciprocal, in fp32 on the host."""
    s = (amax.float().cpu() / 448.0).clamp_min(2.0 ** -40)
    return s.to(amax.device), (1.0 / s).to(amax.device)


def _encode(x, tokens, page, pieces=None):
    """e4m3 codes [n, H, D] of all nodes' tokens and the scales [pages, H], a node at a time starting
    a fresh page.  A page's scale covers the tokens of the piece that starts it."""
    n, H, D = x.shape
    pg, lead, base, at = [], [], 0, 0
    for k, t in enumerate(tokens):
        i = np.arange(t)
        pg.append(base + i // page)
        ends = np.asarray(pieces[k] if pieces else [t])
        first = (i // page) * page
        lead.append(i < ends[np.searchsorted(ends, first, side="right")])
        base += -(-t // page)
        at += t
    pg = torch.as_tensor(np.concatenate(pg), device=x.device)
    lead = torch.as_tensor(np.concatenate(lead), device=x.device)
    amax = torch.zeros((base, H), dtype=torch.float32, device=x.device)
    a = x.abs().amax(dim=2).float() * lead[:, None]
    amax.index_reduce_(0, pg, a, "amax")
    s, inv = _scales(amax)
    y = (x.float() * inv[pg][:, :, None]).clamp(-448.0, 448.0)
    return y.to(torch.float8_e4m3fn), s, pg


def _kv(case, seed, tokens):
    """Keys and values of all nodes' tokens in node order: source tensors, and for fp8 scales."""
    n, H, D = sum(tokens), case["kv_heads"], case["head_dim"]
    k = _normal((n, H, D), _SRC[case["kv"]], seed, 1)
    v = _normal((n, H, D), _SRC[case["kv"]], seed, 2)
    return k, v


def _new_tree(case, seed, n_pages):
    import paper_2605_10195_amd as spex
    order = np.random.default_rng([seed % (1 << 32), 77]).permutation(n_pages).astype(np.int32)
    return spex.SpexTree(case["q_heads"], case["kv_heads"], case["head_dim"], case["page"],
                         "f32" if case["kv"] == "f32" else "bf16", case["kv"], num_pages=n_pages, device=_DEV,
                         free_order=order)


def _splits(case, tokens):
    """Ends of the pieces in which every node's tokens arrive."""
    return [[n] if case["pieces"] == 1 or n < 3 else [n - n // 3, n] for n in tokens]


def prepare(case, seed):
    if case["op"] == "write":
        _, tokens, _ = _shape(case)
        k, v = _kv(case, seed, tokens)
        st = dict(case=case, tree=_new_tree(case, seed, sum(_pages(tokens, case["page"]))), pieces=[])
        sk = sv = pg = None
        if case["kv"] == "fp8_e4m3" and case["pieces"] == 1:      # codes and scales made by the program
            k, sk, pg = _encode(k, tokens, case["page"])
            v, sv, _ = _encode(v, tokens, case["page"])
            k, v = k.view(torch.uint8), v.view(torch.uint8)
        at, page = 0, 0
        for n, ends in zip(tokens, _splits(case, tokens)):
            np_ = -(-n // case["page"])
            parts, a = [], 0
            for e in ends:
                parts.append((k[at + a:at + e], v[at + a:at + e],
                              None if sk is None else sk[page:page + np_], None if sv is None else sv[page:page + np_]))
                a = e
            st["pieces"].append((n, parts))
            at += n
            page += np_
        st["quantize"] = case["kv"] == "fp8_e4m3" and case["pieces"] > 1
        return st

    parent, tokens, leaves, _, q_lens, masks = _requests(case)
    T, B = case["iters"], len(leaves)
    pages = _pages(tokens, case["page"])
    tree = _new_tree(case, seed, sum(pages) + B * -(-T // case["page"]))
    k, v = _kv(case, seed, tokens)
    sk = sv = None
    if case["kv"] == "fp8_e4m3":
        k, sk, _ = _encode(k, tokens, case["page"])
        v, sv, _ = _encode(v, tokens, case["page"])
        k, v = k.view(torch.uint8), v.view(torch.uint8)
    at = pg = 0
    for u, (par, n, np_) in enumerate(zip(parent, tokens, pages)):
        assert tree.fork(par, 1) == [u]
        tree.append_step(u, k[at:at + n], v[at:at + n], None if sk is None else sk[pg:pg + np_],
                         None if sv is None else sv[pg:pg + np_])
        at += n
        pg += np_
    qdt = torch.float32 if case["kv"] == "f32" else torch.bfloat16
    Hq, Hkv, D = case["q_heads"], case["kv_heads"], case["head_dim"]
    st = dict(case=case, tree=tree, sm_scale=D ** -0.5, leaves=np.asarray(leaves, np.int32),
              q_lens=None if max(q_lens) == 1 else np.asarray(q_lens, np.int32),
              masks=None if masks is None else np.asarray(masks, np.uint32))
    nq = sum(q_lens)
    if case["op"] == "decode":
        st["q"] = _normal((nq, Hq, D), qdt, seed, 3, 2.0)
        st["out"] = torch.empty((nq, Hq, D), dtype=torch.float32, device=_DEV)
        st["lse"] = torch.empty((nq, Hq), dtype=torch.float32, device=_DEV)
        return st
    st["q"] = _normal((T, B, Hq, D), qdt, seed, 3, 2.0)
    st["k"], st["v"] = _normal((T, B, Hkv, D), _SRC[case["kv"]], seed, 4), _normal((T, B, Hkv, D), _SRC[case["kv"]], seed, 5)
    st["scale"] = None
    if case["kv"] == "fp8_e4m3":               # page scale for tokens still to come: covers 5 sigma
        st["scale"] = torch.full((B, Hkv), 2.0 ** -6, dtype=torch.float32, device=_DEV)
    st["out"] = torch.empty((T, B, Hq, D), dtype=torch.float32, device=_DEV)
    st["lse"] = torch.empty((T, B, Hq), dtype=torch.float32, device=_DEV)
    return st


def run(state):
    case, tree = state["case"], state["tree"]
    if case["op"] == "decode":
        tree.decode_attention(state["leaves"], state["q_lens"], state["q"], state["sm_scale"], state["out"], state["lse"],
                              draft_masks=state["masks"])
        return state["out"], state["lse"]
    if case["op"] == "write":
        nodes = tree.fork(NO_NODE, len(state["pieces"]))
        for u, (_, parts) in zip(nodes, state["pieces"]):
            for k, v, ks, vs in parts:
                tree.append_step(u, k, v, ks, vs, quantize=state["quantize"])
        copies = [tree.gather_kv(u, 0, n) for u, (n, _) in zip(nodes, state["pieces"])]
        for u in nodes:
            tree.prune(u)
        return [t for c in copies for t in c if t is not None]
    nodes = np.asarray([tree.fork(int(u), 1)[0] for u in state["leaves"]], np.int32)
    sc = state["scale"]
    for t in range(case["iters"]):
        tree.append_tokens(nodes, state["k"][t], state["v"][t], sc, sc, quantize=sc is not None)
        tree.decode_attention(nodes, None, state["q"][t], state["sm_scale"], state["out"][t], state["lse"][t])
    for u in nodes:
        tree.prune(int(u))
    return state["out"], state["lse"]


# ---- the same in 64 bits -----------------------------------------------------------------------
def _half_v(case, v):
    """V of a tiled bf16 cache is held in half precision: what lies below 2^-17 keeps multiples of 2^-24."""
    if case["kv"] != "bf16" or case["page"] != 16 or case["head_dim"] not in (64, 128):
        return v
    f = v.double()
    return torch.where(f.abs() < 2.0 ** -17, torch.trunc(f * 2.0 ** 24) * 2.0 ** -24, f).to(v.dtype)


def _attend(q, k, v, sm_scale, visible):
    """q [n, Hq, D], k and v [T, Hkv, D], visible [n, T]; all float64 -> out, lse."""
    n, Hq, D = q.shape
    T, Hkv, _ = k.shape
    G = Hq // Hkv
    qh = q.reshape(n, Hkv, G, D).permute(1, 0, 2, 3).reshape(Hkv, n * G, D).contiguous()
    s = torch.bmm(qh, k.permute(1, 2, 0).contiguous()).reshape(Hkv, n, G, T) * sm_scale
    s = s.masked_fill(~visible[None, :, None, :], -math.inf)
    lse = torch.logsumexp(s, dim=3)
    p = torch.exp(s - lse[..., None]).reshape(Hkv, n * G, T)
    o = torch.bmm(p, v.permute(1, 0, 2).contiguous()).reshape(Hkv, n, G, D)
    return o.permute(1, 0, 2, 3).reshape(n, Hq, D), lse.permute(1, 0, 2).reshape(n, Hq)


def exact(case, seed):
    if case["op"] == "write":
        _, tokens, _ = _shape(case)
        k, v = _kv(case, seed, tokens)
        out = []
        if case["kv"] == "fp8_e4m3":
            ends = _splits(case, tokens)
            k, sk, pg = _encode(k, tokens, case["page"], ends)
            v, sv, _ = _encode(v, tokens, case["page"], ends)
            each = [k.view(torch.uint8), v.view(torch.uint8), sk[pg], sv[pg]]
        else:
            each = [k, _half_v(case, v)]
        for parts in zip(*(t.split(tokens) for t in each)):
            out.extend(parts)
        return out
    parent, tokens, leaves, total, q_lens, masks = _requests(case)
    Hq, Hkv, D, T = case["q_heads"], case["kv_heads"], case["head_dim"], case["iters"]
    start = np.concatenate([[0], np.cumsum(tokens)])
    k, v = _kv(case, seed, tokens)
    if case["kv"] == "fp8_e4m3":
        k, sk, pg = _encode(k, tokens, case["page"])
        v, sv, _ = _encode(v, tokens, case["page"])

    def rows(x, s, u):
        y = [x[start[w]:start[w + 1]].double() for w in _path(parent, u)]
        if case["kv"] == "fp8_e4m3":
            y = [a * s[pg[start[w]:start[w + 1]]].double()[:, :, None] for a, w in zip(y, _path(parent, u))]
        return torch.cat(y)

    if case["kv"] != "fp8_e4m3":
        v, sk, sv = _half_v(case, v), None, None
    qdt = torch.float32 if case["kv"] == "f32" else torch.bfloat16
    scale = D ** -0.5
    if case["op"] == "decode":
        q = _normal((sum(q_lens), Hq, D), qdt, seed, 3, 2.0).double()
        out, lse = torch.empty_like(q), torch.empty(q.shape[:2], dtype=torch.float64, device=_DEV)
        at = 0
        for u, n in zip(leaves, q_lens):
            seen = torch.arange(total[u], device=_DEV)[None, :] <= torch.arange(total[u] - n, total[u], device=_DEV)[:, None]
            if masks:
                m = torch.tensor(masks[at:at + n], device=_DEV)
                seen[:, total[u] - n:] = ((m[:, None] >> torch.arange(n, device=_DEV)[None, :]) & 1).bool()
            out[at:at + n], lse[at:at + n] = _attend(q[at:at + n], rows(k, sk, u), rows(v, sv, u), scale, seen)
            at += n
        return out, lse
    B = len(leaves)
    q = _normal((T, B, Hq, D), qdt, seed, 3, 2.0).double()
    nk, nv = _normal((T, B, Hkv, D), _SRC[case["kv"]], seed, 4), _normal((T, B, Hkv, D), _SRC[case["kv"]], seed, 5)
    if case["kv"] == "fp8_e4m3":
        nk, nv = (((x.float() * 2.0 ** 6).clamp(-448.0, 448.0)).to(torch.float8_e4m3fn).double() * 2.0 ** -6 for x in (nk, nv))
    else:
        nk, nv = nk.double(), _half_v(case, nv).double()
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], dtype=torch.float64, device=_DEV)
    for i, u in enumerate(leaves):             # query t of the branch sees the first t + 1 new tokens
        n = total[u] + T
        seen = torch.arange(n, device=_DEV)[None, :] <= torch.arange(total[u], n, device=_DEV)[:, None]
        out[:, i], lse[:, i] = _attend(q[:, i].contiguous(), torch.cat([rows(k, sk, u), nk[:, i]]),
                                       torch.cat([rows(v, sv, u), nv[:, i]]), scale, seen)
    return out, lse
