"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  Three kinds:

  "step"   one verification step through the four calls: hs_draft_entropy_topk on the expanded draft
           rows, hs_tree_prune on the candidate trees, hs_tree_attention on the kept rows (all decoder
           layers of a single sequence in one call that shares the tree, or one layer of a ragged
           batch), hs_verify_accept on the kept rows' target logits
  "attn"   attention alone, as a model's layer loop calls it: one call per layer (or one call for all
           layers of a shared tree), on dense caches, on caches with spare capacity or on pages; with
           `commit` the accepted rows join the caches afterwards
  "draft"  the drafting half of an adaptive step: per level one scan of the frontier's draft rows and
           one hs_tree_expand, then hs_adaptive_control

Sizes are those of the five workloads in synth/workloads.py and their neighbourhood.  Everything that
sizes a pass (row counts, prefix lengths) follows from the case alone; the seed draws the values.
"""
import math
import random

import numpy as np
import torch

import paper_2505_13254_amd as hs

DEV = "cuda:0"
TYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    step = dict(kind="step", dtype="bf16", B=1, D=128, tree="expand", K=10, F=10, temperature=1.0, mix=0)
    attn = dict(kind="attn", dtype="bf16", B=1, Hq=32, Hkv=8, D=128, fold=False, commit=False, cache="dense", mix=0)
    return [
        # the tiny float32 layer: every call is a few microseconds, so launches and host work count
        dict(step, name="tiny_step", dtype="f32", Hq=8, Hkv=8, D=64, V=1024, L_lo=128, L_hi=128, layers=1, tree="grow",
             logits="gauss", depth=4, nodes_lo=16, nodes_hi=16, accept=0),
        # one step of the 8B shape, 32 layers, greedy: what bench.py times
        dict(step, name="8b_step", Hq=32, Hkv=8, V=128256, L_lo=2048, L_hi=2048, layers=32, logits="zipf", depth=6,
             nodes_lo=60, nodes_hi=60, accept=0),
        # the same step under the sampling rule
        dict(step, name="8b_step_sampling", Hq=32, Hkv=8, V=128256, L_lo=2048, L_hi=2048, layers=32, logits="zipf",
             depth=6, nodes_lo=60, nodes_hi=60, accept=1),
        # the 13B shape: no query grouping, a 128-node tree, 40 layers
        dict(step, name="13b_step", Hq=40, Hkv=40, V=32000, L_lo=4096, L_hi=4096, layers=40, tree="grow", logits="gauss",
             depth=8, nodes_lo=128, nodes_hi=128, accept=0),
        # the 70B shape: eight query heads share a KV head, 80 layers, sampling rule; the largest case
        dict(step, name="70b_step_sampling", Hq=64, Hkv=8, V=128256, L_lo=8192, L_hi=8192, layers=80, tree="grow",
             logits="zipf", depth=10, nodes_lo=96, nodes_hi=96, accept=1),
        # batched serving on the 8B shape: 16 sequences of their own length, depth and node budget, one layer
        dict(step, name="8b_batch_step", B=16, Hq=32, Hkv=8, V=128256, L_lo=512, L_hi=16384, layers=1, logits="gauss",
             depth=10, nodes_lo=8, nodes_hi=128, accept=0),
        # the attention calls of a model's layer loop, one layer at a time
        dict(attn, name="8b_layer_loop", L_lo=2048, L_hi=2048, M_lo=61, M_hi=61, layers=32),
        # a tree that the threshold has cut to a few rows: the attention is a stream of K and V
        dict(attn, name="13b_few_rows", Hq=40, Hkv=40, L_lo=4096, L_hi=4096, M_lo=4, M_hi=4, layers=40, fold=True),
        # serving on paged caches, ragged lengths, one tree beyond 256 rows, accepted rows committed
        dict(attn, name="8b_paged_serving", B=12, L_lo=333, L_hi=12001, M_lo=9, M_hi=300, layers=4, cache="paged",
             commit=True, mix=3),
        # head dimension 64 on caches with spare capacity
        dict(attn, name="hd64_serving", B=4, D=64, L_lo=700, L_hi=6001, M_lo=21, M_hi=97, layers=2, cache="lens",
             commit=True, mix=1),
        # float32 attention of a small ragged batch
        dict(attn, name="f32_batch", dtype="f32", B=3, Hq=8, Hkv=8, D=64, L_lo=100, L_hi=1500, M_lo=17, M_hi=40, layers=1,
             mix=2),
        # the drafting half of the adaptive step on the 8B shape
        dict(kind="draft", name="8b_draft", B=1, V=128256, K=10, F=10, levels=6, logits="zipf", temperature=1.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["small", "step", "step", "deep", "batch", "loop", "stream", "serve", "serve64", "f32", "draft"])
    mix = rng.randrange(1 << 20)
    T = rng.choice([1.0, 1.0, 0.7])
    bf = dict(dtype="bf16", D=128, mix=mix)
    if what == "small":
        return dict(kind="step", dtype="f32", B=1, Hq=8, Hkv=8, D=64, V=_log(rng, 500, 8000), L_lo=(n := _log(rng, 32, 600)),
                    L_hi=n, layers=1, tree="grow", logits="gauss", depth=rng.randint(3, 6), nodes_lo=(m := rng.randint(8, 36)),
                    nodes_hi=m, accept=rng.choice([0, 1]), K=10, F=10, temperature=T, mix=mix)
    if what == "step":
        Hq, Hkv = rng.choice([(32, 8), (32, 8), (64, 8), (40, 40)])
        return dict(bf, kind="step", B=1, Hq=Hq, Hkv=Hkv, V=rng.choice([32000, 50257, 128256]), L_lo=(n := _log(rng, 200, 6000)),
                    L_hi=n, layers=_log(rng, 4, 40), tree="expand", logits=rng.choice(["zipf", "gauss"]),
                    depth=rng.randint(3, 9), nodes_lo=(m := rng.randint(8, 100)), nodes_hi=m, accept=rng.choice([0, 1]), K=10,
                    F=10, temperature=T)
    if what == "deep":
        return dict(bf, kind="step", B=1, Hq=64, Hkv=8, V=128256, L_lo=(n := _log(rng, 1000, 8000)), L_hi=n,
                    layers=rng.randint(16, 80), tree="grow", logits="zipf", depth=rng.randint(5, 10),
                    nodes_lo=(m := rng.randint(40, 96)), nodes_hi=m, accept=1, K=10, F=10, temperature=T)
    if what == "batch":
        return dict(bf, kind="step", B=rng.randint(4, 16), Hq=32, Hkv=8, V=128256, L_lo=_log(rng, 100, 1000),
                    L_hi=_log(rng, 2000, 16384), layers=1, tree="expand", logits=rng.choice(["gauss", "zipf"]),
                    depth=rng.randint(6, 10), nodes_lo=8, nodes_hi=rng.randint(40, 128), accept=rng.choice([0, 0, 1]), K=10,
                    F=10, temperature=T)
    if what == "loop":
        Hq, Hkv = rng.choice([(32, 8), (64, 8), (40, 40)])
        return dict(bf, kind="attn", B=1, Hq=Hq, Hkv=Hkv, L_lo=(n := _log(rng, 100, 9000 if Hkv == 8 else 4000)), L_hi=n,
                    M_lo=(m := rng.randint(9, 129)), M_hi=m, layers=rng.randint(4, 40), fold=False, commit=False, cache="dense")
    if what == "stream":
        Hq, Hkv = rng.choice([(32, 8), (40, 40)])
        return dict(bf, kind="attn", B=1, Hq=Hq, Hkv=Hkv, L_lo=(n := _log(rng, 500, 4096)), L_hi=n,
                    M_lo=(m := rng.randint(1, 12)), M_hi=m, layers=rng.randint(8, 40), fold=True, commit=False, cache="dense")
    if what == "serve":
        return dict(bf, kind="attn", B=rng.randint(2, 20), Hq=32, Hkv=8, L_lo=_log(rng, 60, 600), L_hi=_log(rng, 1000, 12000),
                    M_lo=rng.randint(2, 20), M_hi=rng.choice([61, 97, 129, 300]), layers=rng.randint(1, 4), fold=False,
                    commit=True, cache=rng.choice(["paged", "lens"]))
    if what == "serve64":
        return dict(bf, kind="attn", B=rng.randint(1, 8), Hq=32, Hkv=8, L_lo=_log(rng, 60, 600), L_hi=_log(rng, 1000, 8000),
                    M_lo=rng.randint(2, 20), M_hi=rng.randint(30, 129), layers=rng.randint(1, 3), fold=False, commit=True,
                    cache=rng.choice(["paged", "lens"])) | dict(D=64)
    if what == "f32":
        return dict(kind="attn", dtype="f32", B=rng.randint(1, 4), Hq=8, Hkv=rng.choice([2, 8]), D=rng.choice([64, 128]),
                    L_lo=_log(rng, 20, 200), L_hi=_log(rng, 300, 2000), M_lo=rng.randint(3, 17), M_hi=rng.randint(18, 64),
                    layers=1, fold=False, commit=False, cache="dense", mix=mix)
    return dict(kind="draft", B=_log(rng, 1, 16), V=rng.choice([32000, 50257, 128256]), K=rng.choice([4, 8, 10, 10]), F=10,
                levels=rng.randint(3, 10), logits=rng.choice(["zipf", "gauss"]), temperature=T)


# ------------------------------------------------------------------------------------ sizes
def _lengths(case):
    """Prefix length of each sequence."""
    r = random.Random(1000 + case["mix"])
    lo, hi = case["L_lo"], case["L_hi"]
    return [lo if lo == hi else r.randint(lo, hi) for _ in range(case["B"])]


def _rows(case):
    """Attention cases: tree rows of each sequence; the largest tree is always among them."""
    r = random.Random(2000 + case["mix"])
    lo, hi = case["M_lo"], case["M_hi"]
    usual = min(hi, 129)  # (trees of up to 128 draft nodes; a single one may be larger)
    m = [lo if lo == hi else r.randint(lo, usual) for _ in range(case["B"])]
    m[r.randrange(case["B"])] = hi
    return m


def _budgets(case):
    """Steps: (depth, draft nodes kept) of each sequence.  In a batch low entropy means deeper and fewer."""
    B = case["B"]
    if B == 1:
        return [(case["depth"], case["nodes_lo"])]
    out = []
    for s in range(B):
        b = s * 8 // B
        out.append((max(3, case["depth"] - b), int(round(case["nodes_lo"] + (case["nodes_hi"] - case["nodes_lo"]) * b / 7.0))))
    random.Random(3000 + case["mix"]).shuffle(out)
    return out


def _draft_rows(case):
    """Draft rows that a step quantifies, per sequence."""
    if case["tree"] == "grow":
        return [n + 1 for _, n in _budgets(case)]
    return [1 + case["F"] * (d - 1) for d, _ in _budgets(case)]


def work(case):
    if case["kind"] == "draft":
        rows = case["B"] * (1 + case["F"] * (case["levels"] - 1))
        return {"bytes": 4 * rows * case["V"], "flops": 4 * rows * case["V"]}
    es = 4 if case["dtype"] == "f32" else 2
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
    step = case["kind"] == "step"
    budgets = _budgets(case) if step else None
    M = [n + 1 for _, n in budgets] if step else _rows(case)
    byts = flops = 0
    for L, m in zip(_lengths(case), M):
        byts += (2 * (L + m) * Hkv * D + 2 * m * Hq * D) * es
        flops += 4 * Hq * D * m * (L + 4)
    byts, flops = byts * case["layers"], flops * case["layers"]
    if step:
        # the draft rows, and of the target rows (sampling: and the draft rows) those of one root path: no
        # walk visits more
        rows = sum(_draft_rows(case)) + sum((d + 1) * (2 if case["accept"] else 1) for d, _ in budgets)
        byts += 4 * rows * case["V"]
        flops += 4 * rows * case["V"]
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # about four times the errors against 64-bit arithmetic: bf16 attention rel 3e-3 / max 1.6e-2, float32
    # attention 5e-7 / 4e-6, scan results 1e-7 / 2e-7 (their sums in float32 over up to 128256 terms)
    if case["kind"] == "draft":
        return {"rel": 1e-6, "max": 5e-6}
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1.5e-5}
    return {"rel": 1e-2, "max": 6e-2}


# ------------------------------------------------------------------------------------ inputs
def _logit_base(case, R, gen):
    """What a node's draft and target rows share: the rank of every token, or the correlated normal part."""
    V = case["V"]
    if case["logits"] == "zipf":
        rank = torch.empty((R, V), dtype=torch.float32, device=DEV)
        for r0 in range(0, R, 128):
            n = min(128, R - r0)
            rank[r0:r0 + n] = torch.rand((n, V), generator=gen, device=DEV).argsort(dim=1).float()
        return rank.add_(1.0).log_().mul_(-1.1), None
    tau = torch.exp(torch.empty((R, 1), device=DEV).uniform_(math.log(0.3), math.log(10.0), generator=gen))
    return torch.randn((R, V), generator=gen, device=DEV), tau


def _logit_rows(case, base, gen, pick=None, target=False):
    """Rows of logits on a base: all of it, or the rows `pick` names."""
    z, tau = base
    if pick is not None:
        z, tau = z[pick], None if tau is None else tau[pick]
    if case["logits"] == "zipf":
        return torch.randn(z.shape, generator=gen, device=DEV).mul_(0.5).add_(z)
    if target:
        z = torch.randn(z.shape, generator=gen, device=DEV).mul_(math.sqrt(1 - 0.81)).add_(z, alpha=0.9)
        return z.mul_(tau)
    return z * tau


def _expand(n_rows, depth, K, F, idx, logp):
    """Top-K expansion on the host: parents, tokens, log-confidences, cumulative values and the draft row
    of each expanded node (-1: not expanded).  idx, logp [n_rows, K]: Top-K results of the sequence's rows."""
    parent, token, logc, value, row_of = [-1], [-1], [0.0], [np.float32(0)], [0]
    front, row = [0], 0
    for d in range(depth):
        first = len(parent)
        for f in front:
            row_of[f] = row
            for k in range(K):
                parent.append(f)
                token.append(int(idx[row, k]))
                logc.append(float(logp[row, k]))
                value.append(np.float32(value[f] + min(np.float32(logp[row, k]), np.float32(0))))
                row_of.append(-1)
            row += 1
        new = range(first, len(parent))
        front = sorted(sorted(new, key=lambda i: (-float(value[i]), i))[:F])
    return parent, token, logc, value, row_of


def _grow(n, depth, rng, K):
    """Parents of a random tree of n draft nodes over `depth` levels, in BFS order, at most K children a node."""
    cap = -(-3 * n // (2 * depth))  # rows of a level; more where the levels could not hold the tree otherwise
    while True:
        sizes, left = [], n
        for d in range(depth):
            sizes.append(max(1, min((sizes[-1] if d else 1) * min(K, 3 + d), cap, left - (depth - d - 1))))
            left -= sizes[-1]
        if left <= 0:
            break
        cap += 1
    parent, prev = [-1], [0]
    for size in sizes:
        slots = [p for p in prev for _ in range(K)]
        ps = sorted(rng.sample(slots, min(size, len(slots))))
        cur = list(range(len(parent), len(parent) + len(ps)))
        parent += ps
        prev = cur
    return parent


def _depths(parent):
    d = [0] * len(parent)
    for i in range(1, len(parent)):
        d[i] = d[parent[i]] + 1
    return d


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device=DEV)


def _offsets(counts, dtype=np.int32):
    return np.concatenate([[0], np.cumsum(counts)]).astype(dtype)


def _randn(shape, dtype, gen):
    return torch.randn(shape, generator=gen, device=DEV, dtype=TYPES[dtype])


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rng = random.Random(seed)
    with torch.no_grad():
        return {"step": _prepare_step, "attn": _prepare_attn, "draft": _prepare_draft}[case["kind"]](case, gen, rng)


def _prepare_step(case, gen, rng):
    B, K, V, layers = case["B"], case["K"], case["V"], case["layers"]
    rows = _draft_rows(case)
    R, r_off = sum(rows), _offsets(rows)
    base = _logit_base(case, R, gen)
    draft = _logit_rows(case, base, gen)
    lp, ix = torch.topk(draft, K, dim=1)
    lp = (lp / case["temperature"] - torch.logsumexp(draft / case["temperature"], 1, keepdim=True)).cpu().numpy()
    ix = ix.cpu().numpy()
    cand, kept = [], []
    for s, (depth, nodes) in enumerate(_budgets(case)):
        r0 = int(r_off[s])
        if case["tree"] == "expand":
            par, tok, logc, val, row_of = _expand(rows[s], depth, K, case["F"], ix[r0:], lp[r0:])
            best = sorted(range(1, len(par)), key=lambda i: (-float(val[i]), i))[:nodes]
            keep = [0] + sorted(best)
        else:
            par = _grow(nodes, depth, rng, min(K, 4))
            tok, logc, seen = [-1] * len(par), [0.0] * len(par), {}
            for i in range(1, len(par)):
                k = seen.get(par[i], 0)
                seen[par[i]] = k + 1
                tok[i], logc[i] = int(ix[r0 + par[i], k]), float(lp[r0 + par[i], k])
            row_of, keep = list(range(len(par))), list(range(len(par)))
        cand.append((par, logc))
        new = {c: j for j, c in enumerate(keep)}
        kept.append(([-1] + [new[par[c]] for c in keep[1:]], [tok[c] for c in keep],
                     [r0 + row_of[c] if row_of[c] >= 0 else -1 for c in keep]))
    M = [len(k[0]) for k in kept]
    NN, no = sum(M), _offsets(M)
    max_depth = max(d for d, _ in _budgets(case))
    node_row = np.concatenate([k[2] for k in kept])
    pick = torch.tensor(np.where(node_row >= 0, node_row, np.arange(NN) % R), device=DEV)
    target = torch.cat([_logit_rows(case, base, gen, pick[i:i + 128], target=True) for i in range(0, NN, 128)])
    draft_of = None
    if case["accept"] == 1:
        draft_of = draft[pick] * torch.tensor(node_row >= 0, device=DEV)[:, None]
    co = _offsets([len(c[0]) for c in cand])
    NC = int(co[-1])
    f32 = dict(dtype=torch.float32, device=DEV)
    i32 = dict(dtype=torch.int32, device=DEV)
    st = dict(
        case=case, draft=draft, target=target, draft_of=draft_of, max_depth=max_depth,
        s1=dict(topk_idx=torch.empty((R, K), **i32), topk_logp=torch.empty((R, K), **f32), ent_topk=torch.empty(R, **f32),
                ent_full=torch.empty(R, **f32), lse=torch.empty(R, **f32)),
        ws1=hs.workspace(hs.lib().hs_draft_entropy_topk_workspace(R, V, K), DEV),
        parent=_i32(np.concatenate([c[0] for c in cand])), logc=torch.tensor(np.concatenate([c[1] for c in cand]), **f32),
        cand_offsets=_i32(co), d_max=_i32([d for d, _ in _budgets(case)]), theta=torch.full((B,), -math.inf, **f32),
        max_nodes=_i32([n for _, n in _budgets(case)]),
        s2=dict(depth=torch.empty(NC, **i32), cumlogp=torch.empty(NC, **f32), keep=torch.empty(NC, dtype=torch.uint8, device=DEV),
                out_offsets=torch.empty(B + 1, **i32), out_src=torch.empty(NC, **i32), out_parent=torch.empty(NC, **i32)),
        ws2=hs.workspace(hs.lib().hs_tree_prune_workspace(B, NC), DEV),
        token=_i32(np.concatenate([k[1] for k in kept])), kept_parent=_i32(np.concatenate([k[0] for k in kept])),
        uniforms=torch.rand(NN + B, generator=gen, **f32) if case["accept"] else None,
        s4=dict(accept_len=torch.empty(B, **i32), accept_path=torch.empty((B, max_depth), **i32), bonus_token=torch.empty(B, **i32)),
        ws4=hs.workspace(hs.lib().hs_verify_accept_workspace_mode(B, NN, V, case["accept"]), DEV))
    hs.hs_workspace_prepare(st["ws1"])
    # attention: all layers of a single sequence are one batch that shares the tree
    lens = _lengths(case) * layers
    m_all = M * layers
    ano, apo = _offsets(m_all), _offsets(lens, np.int64)
    dt, Hq, Hkv, D = case["dtype"], case["Hq"], case["Hkv"], case["D"]
    st.update(q=_randn((int(ano[-1]), Hq, D), dt, gen), k_tree=_randn((int(ano[-1]), Hkv, D), dt, gen),
              v_tree=_randn((int(ano[-1]), Hkv, D), dt, gen), k_prefix=_randn((int(apo[-1]), Hkv, D), dt, gen),
              v_prefix=_randn((int(apo[-1]), Hkv, D), dt, gen), no=_i32(ano), po=torch.tensor(apo, device=DEV),
              host_no=torch.from_numpy(ano), host_po=torch.from_numpy(apo), scale=D ** -0.5)
    st["o"] = torch.empty_like(st["q"])
    st["ws3"] = hs.workspace(hs.lib().hs_tree_attention_workspace(B * layers, int(ano[-1]), int(apo[-1]), Hq, Hkv, D,
                                                                 hs.HS_F32 if dt == "f32" else hs.HS_BF16), DEV)
    return st


def _prepare_attn(case, gen, rng):
    B, layers, dt = case["B"], case["layers"], case["dtype"]
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
    M, L = _rows(case), _lengths(case)
    trees = [_grow(m - 1, min(8, m - 1), rng, 10) if m > 1 else [-1] for m in M]
    NN, no = sum(M), _offsets(M)
    st = dict(case=case, scale=D ** -0.5, M=M, parent=_i32(np.concatenate(trees)), no=_i32(no), host_no=torch.from_numpy(no),
              q=_randn((layers, NN, Hq, D), dt, gen), k_tree=_randn((layers, NN, Hkv, D), dt, gen),
              v_tree=_randn((layers, NN, Hkv, D), dt, gen))
    st["o"] = torch.empty_like(st["q"])
    room = 16  # tokens of spare capacity of a sequence
    lens = np.asarray(L, np.int64)
    if case["cache"] == "paged":
        blocks = [-(-(n + room) // 64) for n in L]
        order = list(range(sum(blocks)))
        rng.shuffle(order)
        table = np.zeros((B, max(blocks)), np.int32)
        for s in range(B):
            table[s, :blocks[s]] = [order.pop() for _ in range(blocks[s])]
        shape = (layers, sum(blocks), 64, Hkv, D)
        st["table"] = _i32(table)
    else:
        extra = room if case["cache"] == "lens" else 0
        off = _offsets([n + extra for n in L], np.int64)
        shape = (layers, int(off[-1]), Hkv, D)
        st.update(po=torch.tensor(off, device=DEV), host_po=torch.from_numpy(off))
    st.update(k=_randn(shape, dt, gen), v=_randn(shape, dt, gen), lens=torch.tensor(lens, device=DEV),
              host_lens=torch.from_numpy(lens))
    total = int(lens.sum()) if case["cache"] == "paged" else int(off[-1])
    entries = layers if case["fold"] else 1  # batch entries per sequence of one call
    st["ws"] = hs.workspace(hs.lib().hs_tree_attention_workspace(B * entries, NN * entries, total * entries, Hq, Hkv, D,
                                                                hs.HS_F32 if dt == "f32" else hs.HS_BF16), DEV)
    if case["fold"]:  # all layers in one call: the offsets of `layers` entries of one tree
        fno, fpo = _offsets(M * layers), _offsets(L * layers, np.int64)
        st.update(no=_i32(fno), host_no=torch.from_numpy(fno), po=torch.tensor(fpo, device=DEV), host_po=torch.from_numpy(fpo))
    if case["commit"]:
        # the accepted rows: a walk down each tree
        path = np.full((B, 8), -1, np.int32)
        for s, par in enumerate(trees):
            dep = _depths(par)
            d = min(max(dep), rng.randint(0, 5))
            deep = [i for i in range(len(par)) if dep[i] == d]
            j, p = rng.choice(deep), []
            while j > 0:
                p.append(j)
                j = par[j]
            path[s, :len(p)] = p[::-1]
        st.update(path=_i32(path), accepted=_i32((path >= 0).sum(1)), cache_lens=[torch.tensor(lens, device=DEV) for _ in range(layers)])
    return st


def _prepare_draft(case, gen, rng):
    B, V, K, F, levels = case["B"], case["V"], case["K"], case["F"], case["levels"]
    rows = B * (1 + F * (levels - 1))
    x = _logit_rows(case, _logit_base(case, rows, gen), gen)
    first = np.full(B * F, -1, np.int32)  # the roots' rows; the other slots of the first level are empty
    first[::F] = np.arange(B)
    cap = 1 + K + (levels - 1) * F * K
    f32, i32 = dict(dtype=torch.float32, device=DEV), dict(dtype=torch.int32, device=DEV)
    st = dict(case=case, cap=cap, first=_i32(first), x=[x[:B]] + [x[B + d * B * F:B + (d + 1) * B * F] for d in range(levels - 1)],
              state={k: v.zero_() if k != "node_offsets" else v for k, v in hs.new_tree_state(B, cap, F, DEV).items()},
              s1=dict(topk_idx=torch.zeros((B * F, K), **i32), topk_logp=torch.zeros((B * F, K), **f32),
                      ent_topk=torch.zeros(B * F, **f32)),
              ws=hs.workspace(hs.lib().hs_draft_entropy_topk_workspace(B * F, V, K), DEV),
              edges=[0.5 * levels * e for e in (0.2, 0.4, 0.6, 0.8, 1.0, 1.3, 1.7)],
              control=dict(phi=torch.empty(B, **f32), **{k: torch.empty(B, **i32) for k in ("pstar", "bin", "d_prime", "n_prime")}))
    hs.hs_workspace_prepare(st["ws"])
    return st


# ------------------------------------------------------------------------------------ one pass
def run(st):
    return {"step": _run_step, "attn": _run_attn, "draft": _run_draft}[st["case"]["kind"]](st)


def _run_step(st):
    case = st["case"]
    s1 = hs.hs_draft_entropy_topk(st["draft"], case["K"], case["temperature"], out=st["s1"], ws=st["ws1"], fused=True)
    s2 = hs.hs_tree_prune(st["parent"], st["logc"], st["cand_offsets"], st["d_max"], st["theta"], st["max_nodes"],
                          out=st["s2"], ws=st["ws2"])
    shared = case["layers"] > 1
    # (the layers of a sequence read the tree where the pruning left it; a batch's offsets likewise)
    o, _ = hs.hs_tree_attention(st["q"], st["k_prefix"], st["v_prefix"], st["k_tree"], st["v_tree"], s2["out_parent"],
                                st["no"] if shared else s2["out_offsets"], st["po"], st["host_no"], st["host_po"], st["scale"],
                                out=st["o"], ws=st["ws3"], shared_tree=shared)
    s4 = hs.hs_verify_accept(st["target"], st["draft_of"], st["token"], s2["out_parent"], s2["out_offsets"], case["accept"],
                             case["temperature"], st["uniforms"], st["max_depth"], out=st["s4"], ws=st["ws4"])
    return dict(s1=s1, s2=s2, o=o, s4=s4)


def _run_attn(st):
    case = st["case"]
    layers = case["layers"]
    out = dict(o=st["o"])
    if case["fold"]:
        def flat(t):
            return t.view(-1, t.shape[-2], t.shape[-1])
        hs.hs_tree_attention(flat(st["q"]), flat(st["k"]), flat(st["v"]), flat(st["k_tree"]), flat(st["v_tree"]), st["parent"],
                             st["no"], st["po"], st["host_no"], st["host_po"], st["scale"], out=flat(st["o"]), ws=st["ws"],
                             shared_tree=True)
        return out
    if case["dtype"] == "f32":  # the plain form of the call: outputs and workspace are the call's
        o, lse = hs.hs_tree_attention(st["q"][0], st["k"][0], st["v"][0], st["k_tree"][0], st["v_tree"][0], st["parent"], st["no"],
                                      st["po"], st["host_no"], st["host_po"], st["scale"], want_lse=True)
        return dict(o=o, lse=lse)
    for l in range(layers):
        q, k, v, kt, vt, o = (st[n][l] for n in ("q", "k", "v", "k_tree", "v_tree", "o"))
        if case["cache"] == "paged":
            hs.hs_tree_attention_paged(q, k, v, kt, vt, st["parent"], st["no"], st["host_no"], st["table"], st["lens"],
                                       st["host_lens"], st["scale"], out=o, ws=st["ws"])
        elif case["cache"] == "lens":
            hs.hs_tree_attention(q, k, v, kt, vt, st["parent"], st["no"], st["po"], st["host_no"], st["host_po"], st["scale"], out=o,
                                 ws=st["ws"], prefix_lens=st["lens"], host_prefix_lens=st["host_lens"])
        else:
            hs.hs_tree_attention(q, k, v, kt, vt, st["parent"], st["no"], st["po"], st["host_no"], st["host_po"], st["scale"], out=o,
                                 ws=st["ws"])
    if case["commit"]:
        for l in range(layers):
            k, v, kt, vt, used = st["k"][l], st["v"][l], st["k_tree"][l], st["v_tree"][l], st["cache_lens"][l]
            used.copy_(st["lens"])  # (every pass commits behind the same prefix)
            if case["cache"] == "paged":
                hs.hs_kv_commit_paged(kt, vt, st["no"], st["path"], st["accepted"], k, v, st["table"], used)
            else:
                hs.hs_kv_commit(kt, vt, st["no"], st["path"], st["accepted"], k, v, st["po"], used)
        out.update(k=st["k"], v=st["v"], used=st["cache_lens"])
    return out


def _run_draft(st):
    case = st["case"]
    B, K, F = case["B"], case["K"], case["F"]
    for d, x in enumerate(st["x"]):
        r = hs.hs_draft_entropy_topk(x, K, case["temperature"], out=st["s1"], ws=st["ws"], row_index=st["first"] if d == 0 else None,
                                     fused=True)
        hs.hs_tree_expand(st["state"], r["topk_idx"], r["topk_logp"], r["ent_topk"], None, B, st["cap"], F, K, first=d == 0)
    s = st["state"]
    c = hs.hs_adaptive_control(s["parent"], s["logc"], s["ent"], s["node_offsets"], s["n_nodes"], st["edges"], (0.3, 0.6, 1.0),
                               -(-case["levels"] // 2), case["levels"], 60, out=st["control"])
    return dict(tree=[s[k] for k in ("parent", "token", "depth", "logc", "cumlogp", "ent", "n_nodes", "frontier")], control=c)
