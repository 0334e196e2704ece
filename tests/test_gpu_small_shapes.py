"""Shapes at the edges of the launch rules: short rows of the row scan, attention launches that leave
compute units to spare."""
import numpy as np
import pytest

from synth import workloads as W
from oracle import draft_entropy_topk, pipeline as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("V", [65, 500, 640, 641, 1024, 4096, 8192, 8193, 12000])
@pytest.mark.parametrize("R,K", [(17, 10), (40, 3), (20, 64)])
def test_short_rows(G, R, V, K):
    """Rows that leave waves, or 16-lane groups, of the first tile without a value: the threshold must
    come from groups that hold one.  Tied and masked rows among them."""
    rs = np.random.RandomState(R + V)
    x = (rs.randn(R, V) * np.exp(rs.uniform(np.log(0.3), np.log(8.0), size=(R, 1)))).astype(np.float32)
    x[1] = 1.5
    x[2, 3:] = -np.inf
    x[3] = np.round(x[3])
    want = draft_entropy_topk(x, K, 1.0)
    got = G.run_entropy(x, K, 1.0)
    assert np.array_equal(got["topk_idx"], want["topk_idx"])
    for k in ("ent_topk", "ent_full"):
        assert G.entropy_err(got[k], want[k]) <= 1.0, k


@pytest.mark.parametrize("R,V", [(1, 12288), (3, 12289), (2, 4 * 64 * 4096), (16, 12287), (16, 12288), (16, 16385), (129, 49151), (129, 49152), (129, 49153),
                                 (129, 65536), (129, 65537), (40, 3 * 6 * 16384), (40, 3 * 6 * 16384 + 1), (300, 12288), (300, 12289)])
def test_rows_around_three_tiles_to_a_workgroup(G, R, V):
    """Workgroups of either size with one to three tiles, the last one whole, of one value or one value short, and with four: the
    five best stand in the first and the last tile, with ties and masked logits between them."""
    rs = np.random.RandomState(R + V % 1000)
    x = rs.randn(R, V).astype(np.float32)
    x[:, V // 2:V // 2 + 40] = -np.inf
    x[:, [1, V - 1]] = 7.0
    x[:, [V - 2, 3, V // 3]] = 6.0
    want = draft_entropy_topk(x, 5, 1.0)
    got = G.run_entropy(x, 5, 1.0)
    assert np.array_equal(got["topk_idx"], want["topk_idx"])
    for k in ("ent_topk", "ent_full"):
        assert G.entropy_err(got[k], want[k]) <= 1.0, k


@pytest.mark.parametrize("hq,hkv", [(4, 4), (8, 4), (6, 2)])
@pytest.mark.parametrize("M", [1, 31, 32, 33, 128, 129, 257])
def test_head_dimension_64_row_blocks(G, hq, hkv, M):
    """Head dimension 64: the 32-row blocks of a pair of KV heads are numbered head by head, so a head's
    last block may be short, and a row group may hold rows of one head or of both."""
    from test_gpu_attention import _case, _compare, _random_parents
    w = W.small(W.WORKLOADS[2], Hq=hq, Hkv=hkv, D=64)
    rs = np.random.RandomState(M)
    _compare(G, _case(w, M, [_random_parents(rs, M, back=9), _random_parents(rs, 5)], [333, 64], "unit"), "bf16")


@pytest.mark.parametrize("variant", ["unit", "hot", "cold"])
@pytest.mark.parametrize("D,hq,hkv,M,L", [
    (128, 2, 2, 1, 0), (128, 2, 2, 1, 31), (128, 2, 2, 32, 64), (128, 2, 2, 33, 65), (128, 2, 2, 65, 129), (128, 4, 2, 64, 33),
    (128, 8, 2, 32, 1025), (128, 8, 2, 33, 97), (128, 8, 2, 64, 4000), (128, 8, 2, 75, 448), (128, 2, 1, 300, 200),
    (64, 4, 4, 17, 130), (64, 8, 2, 33, 1000), (64, 4, 2, 129, 63)])
def test_launches_that_leave_compute_units_to_spare(G, D, hq, hkv, M, L, variant):
    """Few work items: two workgroups to an item, two waves to a row block, each on every other 32 keys.
    One to four row blocks in a workgroup, a second workgroup without rows, last tiles with one or two
    32-key blocks, prefixes in one and in several splits, the exact second pass."""
    from test_gpu_attention import _case, _compare, _random_parents
    if variant == "cold" and (L < 64 or M < 2):
        pytest.skip("the planted rows and keys need two rows and 64 keys")
    w = W.small(W.WORKLOADS[2], Hq=hq, Hkv=hkv, D=D)
    rs = np.random.RandomState(M + L)
    _compare(G, _case(w, M, [_random_parents(rs, M, back=9)], [L], variant), "bf16", big_scores=variant != "unit")


@pytest.mark.parametrize("variant", ["unit", "hot"])
@pytest.mark.parametrize("D,hq,hkv,Ms,Ls", [
    (128, 8, 2, [40], [0]), (128, 8, 2, [33], [31]), (128, 8, 2, [56], [64]), (128, 8, 2, [64], [449]), (128, 16, 2, [33], [2048]),
    (128, 8, 2, [65], [130]), (128, 8, 8, [130, 5], [200, 90]), (64, 8, 2, [20], [33]), (64, 8, 2, [33], [300]), (64, 8, 4, [129], [1000]),
    (64, 8, 8, [260], [100]), (64, 8, 4, [1024], [200])])
def test_four_workgroups_to_an_item(G, D, hq, hkv, Ms, Ls, variant):
    """Launches of at most 64 items of more than 128 rows: one or two row blocks to a workgroup, four waves to a block, each on
    every fourth 32 keys.  Fewer keys than waves have turns, odd last blocks and groups, beside a sequence of few rows,
    unsplit and in splits, trees beyond 256 rows, the exact second pass."""
    from test_gpu_attention import _case, _compare, _random_parents
    w = W.small(W.WORKLOADS[2], Hq=hq, Hkv=hkv, D=D)
    rs = np.random.RandomState(sum(Ms) + sum(Ls))
    _compare(G, _case(w, sum(Ms), [_random_parents(rs, m, back=9) for m in Ms], Ls, variant), "bf16", big_scores=variant != "unit")
    import paper_2505_13254_amd as hs
    assert hs.hs_tree_attention_last_form() == 4


@pytest.mark.parametrize("variant", ["unit", "hot"])
@pytest.mark.parametrize("D,hq,hkv,M,L,B,shared", [
    # a block to a wave: at most 256 items, equal single groups up to 1280
    (128, 8, 8, 129, 300, 20, []), (128, 8, 8, 161, 65, 20, []), (128, 32, 4, 65, 130, 17, []), (128, 16, 4, 150, 97, 18, []),
    (128, 8, 8, 129, 1500, 16, []), (128, 8, 8, 257, 100, 16, []), (128, 8, 8, 129, 70, 100, []), (64, 16, 16, 65, 200, 20, []),
    # ragged, more than 256 items: single groups, one tile and many, in splits, trees beyond 256 rows
    (128, 16, 16, 129, 31, 20, [5]), (128, 16, 16, 129, 300, 17, [5]), (128, 16, 16, 192, 640, 17, [6]), (128, 16, 16, 161, 65, 17, [6]),
    (128, 16, 16, 129, 1500, 17, [5]), (128, 16, 16, 257, 100, 17, [5]), (128, 16, 16, 340, 130, 17, [6, 5]), (128, 16, 16, 560, 70, 17, [6, 6, 6]),
    (64, 32, 32, 65, 200, 20, [6]), (64, 32, 32, 81, 65, 20, [6]), (64, 16, 16, 129, 65, 18, [5, 5]), (64, 32, 32, 257, 65, 20, [6, 6, 6]),
    # equal sequences: several groups, in splits too; single groups beyond 1280 items
    (128, 32, 8, 73, 100, 33, [5, 5]), (128, 32, 8, 90, 1000, 33, [6, 6]), (64, 32, 8, 37, 500, 40, [5, 5]),
    (128, 33, 33, 129, 70, 40, [5]), (128, 33, 33, 170, 64, 40, [6]),
    # one grid row to a sequence
    (128, 16, 16, 129, 70, 100, [5]), (128, 16, 16, 170, 70, 100, [6]), (128, 16, 8, 70, 65, 100, [])])
def test_row_blocks_shared_by_waves(G, D, hq, hkv, M, L, B, shared, variant):
    """Row groups of five or six 32-row blocks: in launches of many items the blocks behind the fourth are shared by four
    waves, or by two each, key block by key block (`shared`: the groups that are).  One tile and many, an odd last tile,
    groups of unequal size, splits, one grid row to a sequence, trees beyond 256 rows, the exact second pass."""
    import paper_2505_13254_amd as hs
    from test_gpu_attention import _case, _compare, _random_parents
    w = W.small(W.WORKLOADS[2], Hq=hq, Hkv=hkv, D=D)
    rs = np.random.RandomState(M + L)
    lens = [L] * B if B > 20 else [max(0, L - 16 * i) for i in range(B)]
    _compare(G, _case(w, M, [_random_parents(rs, M, back=9) for _ in range(B)], lens, variant), "bf16", big_scores=variant != "unit")
    _, several, every = G.row_groups(M, hq, hkv, D)
    assert {0: [], 1: several, 2: every}[hs.hs_tree_attention_last_form() >> 4] == shared


@pytest.mark.parametrize("variant", ["unit", "hot", "last"])
@pytest.mark.parametrize("hq,hkv,M,L,B", [
    (32, 8, 65, 100, 33), (32, 8, 68, 64, 40), (64, 8, 33, 0, 33), (8, 8, 65, 31, 40),   # one group: 4, 16, 8 rows; four blocks
    (64, 4, 17, 1000, 66), (64, 4, 16, 200, 70),                             # the last entries in splits; full groups alone
    (64, 8, 65, 130, 32), (64, 8, 66, 65, 32), (64, 8, 67, 65, 32),                  # two
    (64, 8, 97, 129, 20), (64, 8, 98, 1, 32)])                              # three
def test_a_few_rows_behind_full_row_groups(G, hq, hkv, M, L, B, variant):
    """A few rows of a KV head behind what full row groups hold: one tile and many, a partial one, the tree's tiles alone, one node's
    rows and two, splits; scores that leave the fixed reference, of any rows and ("last") of the last row alone."""
    import paper_2505_13254_amd as hs
    from test_gpu_attention import _case, _compare, _random_parents
    w = W.small(W.WORKLOADS[2], Hq=hq, Hkv=hkv, D=128)
    rs = np.random.RandomState(M + L)
    step = _case(w, M, [_random_parents(rs, M, back=9) for _ in range(B)], [L] * B, "unit" if variant == "last" else variant)
    if variant == "last":  # a late key of the prefix, or the tree's last one, along the last row's query of some head
        as_float = lambda bits: (bits.astype(np.uint32) << 16).view(np.float32)
        for s in range(B):
            h, row = s % hq, (s + 1) * M - 1
            q = as_float(step["q"][row, h])
            key = q * np.float32((125.0 + s % 30) * np.sqrt(128.0) / np.dot(q, q))
            keys, at = (step["k_prefix"], (s + 1) * L - 1 - s % min(L, 40)) if L > 0 and s % 3 else (step["k_tree"], row)
            keys[at, h // (hq // hkv)] = torch.from_numpy(key).bfloat16().view(torch.int16).numpy().view(np.uint16)
    _compare(G, step, "bf16", big_scores=variant != "unit")
    assert hs.hs_tree_attention_last_kernel() == 1


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,hq,hkv,M,L,offset", [
    (64, 3, 3, 1, 0, 0), (64, 3, 3, 16, 15, 0), (64, 6, 3, 17, 16, 1), (64, 3, 1, 33, 511, 0), (64, 3, 3, 5, 1040, 3),
    (128, 3, 3, 1, 1, 0), (128, 6, 3, 16, 17, 0), (128, 3, 1, 47, 513, 1), (128, 3, 3, 1024, 40, 0),
    (64, 3, 1, 33, 208, 0), (64, 3, 1, 33, 209, 0), (64, 3, 3, 256, 0, 0), (128, 3, 1, 16, 112, 0), (128, 3, 3, 17, 112, 0)])
def test_attention_of_any_shape_and_address(G, dtype, D, hq, hkv, M, L, offset):
    """The kernel for float32 and for what the bfloat16 matrix kernel refuses (an odd number of KV heads of
    64, arrays off a 16-byte boundary): groups of 16 keys that end short, fewer groups than waves, as many as one trip takes and
    one more, split prefixes, the largest tree, arrays that start `offset` elements off."""
    import paper_2505_13254_amd as hs
    from oracle import pipeline
    from test_gpu_attention import _case, _random_parents
    if dtype == "bf16" and D == 128 and offset == 0:
        offset = 1  # (an aligned array would go to the other kernel)
    w = W.small(W.WORKLOADS[2 if dtype == "bf16" else 1], Hq=hq, Hkv=hkv, D=D)
    rs = np.random.RandomState(M + L)
    step = _case(w, M, [_random_parents(rs, M, back=9), _random_parents(rs, 2)], [L, 64], "unit")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def off(x):
        x = np.ascontiguousarray(x)  # (bfloat16 values come as their bits)
        t = torch.from_numpy(x.view(np.int16)).view(dt) if dtype == "bf16" else torch.from_numpy(x)
        flat = torch.zeros(x.size + offset, dtype=dt, device="cuda:0")
        flat[offset:] = t.flatten().to("cuda:0")
        return flat[offset:].view(x.shape)

    q, kp, vp, kt, vt = (off(step[n]) for n in ("q", "k_prefix", "v_prefix", "k_tree", "v_tree"))
    no, po = torch.from_numpy(step["node_offsets"]), torch.from_numpy(step["prefix_offsets"])
    o, lse = hs.hs_tree_attention(q, kp, vp, kt, vt, torch.from_numpy(step["parent"]).to("cuda:0"), no.to("cuda:0"),
                                  po.to("cuda:0"), no, po, step["scale"], want_lse=True)
    assert hs.hs_tree_attention_last_kernel() == 2
    want_o, want_lse = pipeline.attention_out(step)
    # float32 arithmetic throughout: up to 1088 terms a row, each rounded at 2^-24 of values of order 1 (the
    # bfloat16 result is rounded once more, to 2^-9 of it)
    tol = 2e-6 + (2.0 ** -8 * np.abs(want_o) if dtype == "bf16" else 1e-5 * np.abs(want_o).max())
    assert np.all(np.abs(o.float().cpu().numpy() - want_o) <= tol)
    assert np.abs(lse.cpu().numpy() - want_lse).max() <= 2e-5


@pytest.mark.parametrize("D,hq,hkv,Ms,Ls", [
    (128, 8, 8, [55], [385]), (128, 8, 8, [17, 3, 31], [385, 0, 1000]), (128, 8, 2, [40], [1025]), (128, 3, 3, [1], [1153]),
    (64, 8, 8, [33, 16], [513, 1300]), (64, 8, 2, [5, 1], [2000, 127]), (64, 6, 3, [20], [4100])])
def test_float32_prefixes_in_splits(G, D, hq, hkv, Ms, Ls):
    """The float32 kernel's splits: of 128 tokens and more, last ones of a single key, beside sequences that are not split,
    up to 16 and more of them (the merge takes eight at a time).  A workspace without room for their records gets the
    coarser cut."""
    import paper_2505_13254_amd as hs
    from test_gpu_attention import _case, _random_parents
    w = W.small(W.WORKLOADS[1], Hq=hq, Hkv=hkv, D=D)
    rs = np.random.RandomState(sum(Ls))
    step = _case(w, sum(Ms), [_random_parents(rs, m, back=9) for m in Ms], Ls, "unit")
    want_o, want_lse = P.attention_out(step)
    no, po = torch.from_numpy(step["node_offsets"]), torch.from_numpy(step["prefix_offsets"])
    totals, _ = hs.hs_tree_attention_plan(no, po, hq, hkv, D, hs.HS_F32)
    assert totals[0] == 2 and totals[2] > 1
    args = [G.dev(step[n]) for n in ("q", "k_prefix", "v_prefix", "k_tree", "v_tree", "parent", "node_offsets", "prefix_offsets")]
    for ws in (None, hs.workspace(int(totals[4]) - 256, "cuda:0")):
        o, lse = hs.hs_tree_attention(*args, no, po, step["scale"], want_lse=True, ws=ws)
        # float32 arithmetic: sums of up to 4120 terms, each rounded at 2^-24 of values of order 1
        assert np.abs(G.host(o) - want_o).max() <= 2e-6 + 1e-5 * np.abs(want_o).max()
        assert np.abs(G.host(lse) - want_lse).max() <= 2e-5
    if max(Ls) > 1500:  # (the coarser cut has records as well)
        with pytest.raises(hs.HsError) as e:
            hs.hs_tree_attention(*args, no, po, step["scale"], want_lse=True, ws=hs.workspace(256, "cuda:0"))
        assert e.value.status == hs.binding.HS_ERR_WORKSPACE


@pytest.mark.parametrize("D,hq,hkv,M,L", [(128, 3, 3, 1, 1153), (64, 6, 3, 20, 4100)])
@pytest.mark.parametrize("splits,more", [(1, 0), (8, 0), (8, 37), (9, 1)])
def test_float32_splits_of_masked_keys(G, D, hq, hkv, M, L, splits, more):
    """Keys whose scores are -inf (weight 0) fill whole splits of a float32 call, the first eight that the merge takes
    together among them."""
    import paper_2505_13254_amd as hs
    from test_gpu_attention import _case, _compare, _random_parents
    w = W.small(W.WORKLOADS[1], Hq=hq, Hkv=hkv, D=D)
    rs = np.random.RandomState(D + splits)
    step = _case(w, M, [_random_parents(rs, M, back=9)], [L], "unit")
    totals, _ = hs.hs_tree_attention_plan(torch.from_numpy(step["node_offsets"]), torch.from_numpy(step["prefix_offsets"]), hq, hkv, D, hs.HS_F32)
    assert totals[0] == 2 and totals[2] > splits and totals[2] > 8
    step["q"][:, :, 0] = np.abs(step["q"][:, :, 0]) + 0.1
    step["k_prefix"][:splits * int(totals[3]) + more, :, 0] = -np.inf
    _compare(G, step, "f32")


@pytest.mark.parametrize("k,rem", [(1, 0.6), (8, 0.6), (20, 0.6), (32, 0.5), (64, 0.25), (96, 0.12)])
def test_ratio_rule_around_the_edge_of_a_bucket(G, k, rem):
    """Chains of rejections whose second residual max(p - beta q, 0) has beta at 2^(k/32) and to either side of it, where the
    sort's buckets of the ratio p / q meet, and many tokens with such ratios: the third child's test is put 4e-4 to either
    side of what 64 bits say.  (The kernel's terms carry a few 1e-6 of p each, so its quotient about 1e-4 at most; the tokens
    around the edge, taken for dead or live as a whole bucket, move it by 1e-3 to 1e-2.)"""
    from oracle import verify_accept
    V, NA = 8192, 3000
    steps = [-0.5, -0.02, -0.009, -0.003, 0.0, 0.003, 0.009, 0.02, 0.5]
    rs = np.random.RandomState(k)
    target, draft, u, want_hit, bonus_u = [], [], [], [], []
    for e in steps:
        beta = 2.0 ** ((k + e) / 32)
        near = 2.0 ** ((k + rs.choice([-1.1, -0.9, -0.3, -0.012, -0.008, -0.002, 0.0, 0.002, 0.008, 0.012, 0.3, 0.9, 1.1], size=NA)) / 32)
        pa = rs.uniform(0.5, 1.5, size=NA)
        pa *= (0.1 if k == 1 else 0.4) / pa.sum()
        qa = pa / near
        z1 = (beta - 1.0) * rem                                     # so that 1 + Z / (1 - q(x1)) is beta
        ph = (z1 - (np.maximum(pa - qa, 0)).sum()) / (1 - 1 / (4 * beta))
        p3 = 1e-5                                                   # the third child's token; x1, x2: rejected for certain
        z2 = np.maximum(pa - beta * qa, 0).sum() + ph * 0.75
        eps = 0.5 * z2 / (beta * rem)
        q3 = p3 / (beta * (1 + eps))
        ph -= (p3 - q3) / (1 - 1 / (4 * beta))
        n_h, n_l = 1000, V - NA - 1000 - 3
        h_p = np.full(n_h, ph / n_h)
        q1, q2, p2 = 1 - rem, 1e-5, 1e-7
        low = 1 - q1 - q2 - q3 - qa.sum() - ph / (4 * beta)          # of q, on tokens that p falls short on, x1 among them
        l_q = np.full(n_l, low / n_l)
        l_p = l_q * (1 - min(0.5, 0.5 * z1 / low))
        p1 = 1 - pa.sum() - ph - p2 - p3 - l_p.sum()
        assert ph > 0 and low > 0 and 0 < p1 < 0.995 * q1
        p = np.concatenate([[p1, p2, p3], pa, h_p, l_p])
        q = np.concatenate([[q1, q2, q3], qa, h_p / (4 * beta), l_q])
        order = rs.permutation(V)                                   # the tokens' places in the vocabulary
        place = np.argsort(order)
        t, d = np.log(p[order]).astype(np.float32), np.log(q[order]).astype(np.float32)
        # 64-bit chain on the rounded logits
        P64, Q64 = (np.exp(x.astype(np.float64)) for x in (t, d))
        P64, Q64 = P64 / P64.sum(), Q64 / Q64.sum()
        cp, cq = P64.copy(), Q64.copy()
        for c in (0, 1):
            r = np.maximum(cp - cq, 0)
            cp = r / r.sum()
            cq[place[c]] = 0
            cq /= cq.sum()
        got_beta = 1 + np.maximum(P64 - Q64, 0).sum() / (1 - Q64[place[0]])
        assert abs(32 * np.log2(got_beta) - (k + e)) < 1e-3
        ratio = cp[place[2]] / cq[place[2]]
        assert 0.4 < ratio < 0.6
        rest = np.maximum(cp - cq, 0)
        rest /= rest.sum()
        for sign, last in ((-1, P64), (1, rest)):                   # accepted: the child's own row decides the bonus
            best = int(np.argmax(last))
            target.append(np.repeat(t[None], 4, axis=0))
            draft.append(np.repeat(d[None], 4, axis=0))
            u.append([0.5, 0.999, 0.999, np.float32(ratio * (1 + sign * 4e-4))])
            bonus_u.append(np.float32(last[:best].sum() + 0.5 * last[best]))
            want_hit.append((sign, place[:3]))
    B = len(u)
    target, draft = np.concatenate(target), np.concatenate(draft)
    token = np.concatenate([np.concatenate([[0], pl]) for _, pl in want_hit]).astype(np.int32)
    parent = np.tile(np.asarray([-1, 0, 0, 0], np.int32), B)
    off = (4 * np.arange(B + 1)).astype(np.int32)
    uniforms = np.concatenate([np.asarray(u, np.float32).ravel(), np.asarray(bonus_u, np.float32)])
    want = verify_accept(target, draft, token, parent, off, 1, 1.0, uniforms, 2)
    assert list(want["accept_len"]) == [1 if sign < 0 else 0 for sign, _ in want_hit]
    got = G.run_accept(dict(w=W.WORKLOADS[1], target_logits=target, draft_logits=draft, token=token, parent=parent, node_offsets=off),
                       1, uniforms, 2, temperature=1.0)
    for name in want:
        assert np.array_equal(got[name], want[name]), name


@pytest.mark.parametrize("sizes,spare", [([1], 2), ([5, 3], 3), ([1030], 0), ([1100, 4], 5)])
def test_ratio_rule_on_large_trees_and_spare_rows(G, sizes, spare):
    """Sampling with the draft's ratio rule: trees beyond the 1024 rows that are staged in LDS, and rows
    behind the last sequence (what pruning into arrays with spare capacity leaves), which nobody scans."""
    import paper_2505_13254_amd as hs
    from test_gpu_entropy_prune_accept import _accept_equal, _random_accept_case
    rs = np.random.RandomState(sum(sizes))
    V, D, done = 4100, 5, 0
    for attempt in range(60):
        case = _random_accept_case(rs, sizes, V, 1, 1.0, D)
        if case is None:
            continue
        target, draft, token, parent, offs, u, base = case
        NN = len(token)
        rows = np.full((spare, V), np.nan, np.float32)
        fill = np.full(spare, 0x7fffffff, np.int32)
        out = hs.hs_verify_accept(G.dev(np.concatenate([target, rows])), G.dev(np.concatenate([draft, rows])),
                                  G.dev(np.concatenate([token, fill]), torch.int32), G.dev(np.concatenate([parent, fill]), torch.int32),
                                  G.dev(offs, torch.int32), 1, 1.0,
                                  G.dev(np.concatenate([u[:NN], np.zeros(spare), u[NN:]]), torch.float32), D)
        _accept_equal({k: G.host(v) for k, v in out.items()}, base)
        done += 1
        if done == 4:
            break
    assert done == 4


@pytest.mark.parametrize("D,hq,hkv,M,L,B", [(128, 8, 8, 9, 1500, 33), (128, 8, 4, 40, 833, 70), (64, 8, 8, 5, 2100, 66)])
def test_equal_entries_that_spill_into_another_round(G, D, hq, hkv, M, L, B):
    """A few items more than compute units, all alike: the last entries are cut into splits, the others
    are written directly and the merge starts behind them."""
    import paper_2505_13254_amd as hs
    from test_gpu_attention import _case, _compare, _random_parents
    w = W.small(W.WORKLOADS[2], Hq=hq, Hkv=hkv, D=D)
    rs = np.random.RandomState(B)
    step = _case(w, B, [_random_parents(rs, M, back=9) for _ in range(B)], [L] * B, "unit")
    totals, per = hs.hs_tree_attention_plan(torch.from_numpy(step["node_offsets"]), torch.from_numpy(step["prefix_offsets"]),
                                            hq, hkv, D, hs.HS_BF16)
    assert per[0][0] == 1 and per[B - 1][0] > 1 and totals[2] == per[B - 1][0]
    _compare(G, step, "bf16")


def test_a_workspace_without_room_for_the_finer_last_round(G):
    """The same launch with no room for records runs uncut; a launch that is cut in any plan (one sequence
    of few heads) is refused."""
    import paper_2505_13254_amd as hs
    from test_gpu_attention import P, _case, _random_parents
    for D, hq, hkv, M, L, B in [(128, 8, 8, 9, 1500, 33), (64, 8, 8, 5, 1000, 66), (128, 8, 4, 40, 833, 70), (128, 8, 4, 9, 4000, 1)]:
        w = W.small(W.WORKLOADS[2], Hq=hq, Hkv=hkv, D=D)
        rs = np.random.RandomState(B)
        step = _case(w, B, [_random_parents(rs, M, back=9) for _ in range(B)], [L] * B, "unit")
        no, po = (torch.from_numpy(np.asarray(step[k])) for k in ("node_offsets", "prefix_offsets"))
        args = [G.dev_store(step[k]) for k in ("q", "k_prefix", "v_prefix", "k_tree", "v_tree")]
        args += [G.dev(step["parent"], torch.int32), no.cuda(), po.cuda(), no, po, float(step["scale"])]
        small = torch.empty(256, dtype=torch.uint8, device="cuda")
        if B == 1:
            with pytest.raises(hs.HsError):
                hs.hs_tree_attention(*args, ws=small)
            continue
        got, _ = hs.hs_tree_attention(*args, ws=small)
        # against the checker, within what the kernel's roundings imply element by element, and within 1e-2 of the
        # largest output (what the other bfloat16 comparisons ask; a tile of keys left out moves an output by more)
        want, _ = P.attention_out(step)
        diff = np.abs(G.host(got).astype(np.float64) - want)
        assert (diff / G.attention_error_bound(step, want)).max() <= 1.0
        assert diff.max() <= 1e-2 * np.abs(want).max()


@pytest.mark.parametrize("V", [2050, 4096, 8195])
@pytest.mark.parametrize("n_kids,k", [(1, 0), (1, None), (2, 1), (5, 0), (5, 4), (66, 63), (66, 64), (66, None)])
def test_chains_end_with_their_first_accepted_child(G, V, n_kids, k):
    """The root's k-th child is accepted (None: no child is), and below it a chain of one child, accepted and then
    rejected: one child with the sums alone, chains that end at any place, by the sorted residual and (V = 2050) by passes
    over both rows.  An empty sequence lies between two copies of the tree, the second without room for a second level."""
    import paper_2505_13254_amd as hs
    from oracle import verify_accept
    rs = np.random.RandomState(100 * n_kids + (k or 0))
    at = 1 + (k if k is not None else 0)                   # the child that has the rest of the tree below it
    parent = np.asarray([-1] + [0] * n_kids + [at, n_kids + 1], np.int32)
    n = len(parent)
    draft = (rs.normal(size=(n, V)) * 1.5).astype(np.float32)
    target = (0.8 * draft + rs.normal(size=draft.shape)).astype(np.float32)
    token = np.zeros(n, np.int32)
    token[1:n_kids + 1] = np.argsort(-draft[0], kind="stable")[:n_kids]
    token[n_kids + 1], token[n_kids + 2] = draft[at].argmax(), draft[n_kids + 1].argmax()
    u = np.full(n, 0.9999, np.float32)
    # (a rejected token stands well below its draft probability, an accepted one above it whatever was rejected before)
    target[0, token[1:n_kids + 1]] = draft[0, token[1:n_kids + 1]] - 3.0
    target[n_kids + 1, token[n_kids + 2]] = draft[n_kids + 1, token[n_kids + 2]] - 3.0
    target[at, token[n_kids + 1]] += 9.0
    if k is not None:
        target[0, token[at]] += 12.0
        u[at] = 0.0
    two = [np.concatenate([x, x]) for x in (target, draft, token, parent)]
    offs = np.asarray([0, n, n, 2 * n], np.int32)
    for depth in (3, 1):
        for draw in np.linspace(0.3, 0.7, 50):  # (a draw at the edge of a token's interval may fall to either side)
            uu = np.concatenate([u, u, [draw, 0.5, draw + 0.1]]).astype(np.float32)
            want = verify_accept(two[0], two[1], two[2], two[3], offs, 1, 1.0, uu, depth)
            near = [verify_accept(two[0], two[1], two[2], two[3], offs, 1, 1.0, np.concatenate([uu[:-3], uu[-3:] + e]), depth)
                    for e in (-1e-5, 1e-5)]
            if all(np.array_equal(w["bonus_token"], want["bonus_token"]) for w in near):
                break
        else:
            raise AssertionError("every draw lies at an edge")
        assert want["accept_len"][0] == (0 if k is None else min(depth, 2))
        out = hs.hs_verify_accept(G.dev(two[0]), G.dev(two[1]), G.dev(two[2], torch.int32), G.dev(two[3], torch.int32),
                                  G.dev(offs, torch.int32), 1, 1.0, G.dev(uu, torch.float32), depth)
        for key in want:
            assert np.array_equal(G.host(out[key]), want[key]), (key, depth)


@pytest.mark.parametrize("k", [0, None])
@pytest.mark.parametrize("V", [65535, 65536, 65537])
def test_single_children_around_the_length_from_which_they_are_sorted(G, V, k):
    """One child to a node, accepted or rejected, in rows that its own workgroup passes over and in rows that are sorted."""
    test_chains_end_with_their_first_accepted_child(G, V, 1, k)


@pytest.mark.parametrize("V,n_kids", [(1, 0), (63, 2), (2048, 0), (2049, 2), (4097, 0), (131072, 2), (131073, 2), (524288, 0), (524288, 2)])
def test_bonus_draws_by_the_last_workgroup(G, V, n_kids):
    """Ratio rule: two sequences with an empty one between them and a spare row behind, whose bonus tokens are drawn by the workgroup
    that finishes the row, from fewer rows of 64 tokens than there are workgroups up to as many as LDS holds; from p itself and,
    with all children rejected, from the residual."""
    import paper_2505_13254_amd as hs
    from oracle import verify_accept
    rs = np.random.RandomState(V % 1000)
    n = 1 + n_kids
    parent = np.asarray(([-1] + [0] * n_kids) * 2 + [0], np.int32)
    draft = rs.randn(2 * n + 1, V).astype(np.float32)
    target = (draft + 0.5 * rs.randn(*draft.shape)).astype(np.float32)
    token = np.zeros(2 * n + 1, np.int32)
    for i in range(n_kids):                       # children that stand far below their draft probability
        for g in (0, n):
            token[g + 1 + i] = (i * (V // 2) + g) % V
            draft[g, token[g + 1 + i]], target[g, token[g + 1 + i]] = 5.0, -2.0
    offs = np.asarray([0, n, n, 2 * n], np.int32)
    args = [G.dev(target), G.dev(draft), G.dev(token, torch.int32), G.dev(parent, torch.int32), G.dev(offs, torch.int32), 1, 1.0]
    checked = 0
    for draw in (0.013, 0.3, 0.5, 0.77, 0.98):
        u = lambda e: np.concatenate([np.full(2 * n + 1, 0.9999), [draw + e, 0.5, 0.9 * draw + e]]).astype(np.float32)
        # (the oracle knows no spare row, and no uniform of one)
        want, lo, hi = (verify_accept(target, draft, token, parent, offs, 1, 1.0, np.delete(u(e), 2 * n), 2) for e in (0.0, -1e-6, 1e-6))
        out = hs.hs_verify_accept(*args, G.dev(u(0.0), torch.float32), 2)
        assert G.host(out["accept_len"]).tolist() == want["accept_len"].tolist() == [0, 0, 0]
        assert np.array_equal(G.host(out["accept_path"]), want["accept_path"])
        got = G.host(out["bonus_token"])
        assert got[1] == want["bonus_token"][1] == -1
        for s_ in (0, 2):                         # (float32 probabilities move a token's interval by less than 1e-6 of the mass)
            assert lo["bonus_token"][s_] <= got[s_] <= hi["bonus_token"][s_], (draw, s_)
            checked += lo["bonus_token"][s_] == hi["bonus_token"][s_]
    assert checked > 0 or V > 4097


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("n_kids", [1, 63, 65, 250])
def test_bonus_draws_after_many_rejections(G, mode, n_kids):
    """Bonus draws at the root and at a node below it with up to 250 rejected children, whose corrections are
    made by one to four waves while others may still be trying the children: the checker's tokens, and the
    same ones on every call."""
    import paper_2505_13254_amd as hs
    from oracle import verify_accept
    from test_gpu_entropy_prune_accept import _accept_equal
    rs = np.random.RandomState(n_kids + mode)
    V, done = 8192, 0
    for attempt in range(40):
        # sequence 0: all children of the root are rejected; sequence 1: the root's only child is accepted and
        # all of its children are rejected (the target gives a rejected token a fraction of the draft's share)
        parent = np.concatenate([[-1], [0] * n_kids, [-1, 0], [1] * n_kids]).astype(np.int32)
        offs = np.asarray([0, n_kids + 1, 2 * n_kids + 3], np.int32)
        NN = len(parent)
        draft = (rs.normal(size=(NN, V)) * 2).astype(np.float32)
        target = (0.9 * draft + 0.5 * rs.normal(size=(NN, V))).astype(np.float32)
        token = np.zeros(NN, np.int32)
        for node, first in ((0, 1), (n_kids + 2, n_kids + 3)):
            token[first:first + n_kids] = np.argsort(-draft[node], kind="stable")[:n_kids]
            target[node, token[first:first + n_kids]] -= 3.0
        target[n_kids + 1, token[n_kids + 2]] += 30.0
        u = np.concatenate([0.9 + 0.0999 * rs.rand(NN), rs.rand(2)]).astype(np.float32)
        want = verify_accept(target, draft, token, parent, offs, mode, 1.0, u, 4)
        assert list(want["accept_len"]) == [0, 1]
        near = []
        for sgn in (-1.0, 1.0):  # (a draw at the edge of a token's interval may fall to either side)
            un = u.astype(np.float64)
            un[NN:] = np.clip(un[NN:] + sgn * 1e-5, 0.0, 1.0 - 1e-12)
            near.append(verify_accept(target, draft, token, parent, offs, mode, 1.0, un, 4)["bonus_token"])
        if not all(np.array_equal(b, want["bonus_token"]) for b in near):
            continue
        args = [G.dev(target), G.dev(draft), G.dev(token, torch.int32), G.dev(parent, torch.int32), G.dev(offs, torch.int32), mode,
                1.0, G.dev(u, torch.float32), 4]
        for rep in range(4):
            _accept_equal({k: G.host(v) for k, v in hs.hs_verify_accept(*args).items()}, want)
        done += 1
        if done == 3:
            break
    assert done == 3


@pytest.mark.parametrize("R,V,K", [(1, 262144, 16), (1, 262144, 17), (4, 262144, 20), (1, 262144, 64), (4, 256000, 40), (3, 151936, 30)])
def test_merge_of_many_slices_and_long_lists(G, R, V, K):
    """Few rows of a large vocabulary: up to 64 slices of 4096, more list entries than the merge keeps in
    registers (K = 16: just as many).  A row's K best values lie in its last K slices, one in each, falling
    from slice to slice, so that the merge's threshold is the very last slice's best."""
    import paper_2505_13254_amd as hs
    rs = np.random.RandomState(V + K)
    x = (rs.randn(R, V) * 2 - 100.0).astype(np.float32)
    n_slices = -(-V // 4096)
    for r in range(R):
        for i in range(K):
            sl = n_slices - K + i
            x[r, sl * 4096 + rs.randint(min(4096, V - sl * 4096))] = 40.0 - 0.25 * i
    want, xd = draft_entropy_topk(x, K, 1.0), G.dev(x)
    ws = hs.workspace(hs.lib().hs_draft_entropy_topk_workspace(R, V, K), G.DEV)
    hs.hs_workspace_prepare(ws)
    for fused in (True, False):
        for rep in range(3):
            got = {k: G.host(v) for k, v in hs.hs_draft_entropy_topk(xd, K, 1.0, ws=ws, fused=fused).items()}
            assert np.array_equal(got["topk_idx"], want["topk_idx"]), (fused, rep)
            for k in ("ent_topk", "ent_full"):
                assert G.entropy_err(got[k], want[k]) <= 1.0, k


@pytest.mark.parametrize("K", [1, 5, 16, 17, 33, 64])
@pytest.mark.parametrize("R,V", [(20, 12000), (20, 40000), (3, 12000), (2, 140000)])
def test_lists_of_unequal_length(G, R, V, K):
    """The merges' threshold with more and with fewer lists than K: the row's best all in one wave's lanes, spread
    evenly, tied, rising, and rows with fewer unmasked logits than K."""
    rs = np.random.RandomState(V + K)
    x = (rs.randn(R, V) * 3).astype(np.float32)
    x[0, 256:320] += 50.0
    x[1, :: V // 70] += 50.0
    if R > 2:
        x[2] = np.round(x[2])
    if R > 6:
        x[3] = -np.inf
        x[3, rs.permutation(V)[:K // 2 + 1]] = 1.0
        x[4] = np.sort(x[4])
        x[5, :-K] = -np.inf
        x[6] = 0.5
    want = draft_entropy_topk(x, K, 1.0)
    got = G.run_entropy(x, K, 1.0)
    assert np.array_equal(got["topk_idx"], want["topk_idx"])
    for k in ("ent_topk", "ent_full"):
        assert G.entropy_err(got[k], want[k]) <= 1.0, k


@pytest.mark.parametrize("T", [1.0, 0.7])
@pytest.mark.parametrize("R,V", [(1, 128259), (10, 40000), (51, 50257), (300, 12000)])
def test_masked_logits_at_any_place(G, R, V, T):
    """Rows whose first -inf comes in the first tile, in a later one or at the end, one masked logit, whole
    tiles of them between tiles with values, all but a few: a wave that has met one changes how it sums."""
    rs = np.random.RandomState(R + V)
    x = (rs.randn(R, V) * 2).astype(np.float32)
    for r in range(R):
        kind = r % 6 if R > 1 else 3
        if kind == 0:
            x[r, V // 3] = -np.inf
        elif kind == 1:
            x[r, 4096 * rs.randint(1, 3):] = -np.inf
        elif kind == 2:
            x[r, rs.rand(V) < 0.5] = -np.inf
        elif kind == 3:  # (blocks of the smaller and of the larger tile)
            x[r, np.repeat(rs.rand(-(-V // 4096)) < 0.6, 4096)[:V]] = -np.inf
            x[r, rs.permutation(V)[:20]] = 3.0
        elif kind == 4:
            x[r, rs.permutation(V)[:V - 12]] = -np.inf
        else:
            x[r, V - 1] = -np.inf
    want = draft_entropy_topk(x, 10, T)
    got = G.run_entropy(x, 10, T)
    assert np.array_equal(got["topk_idx"], want["topk_idx"])
    for k in ("ent_topk", "ent_full"):
        assert G.entropy_err(got[k], want[k]) <= 1.0, k


@pytest.mark.parametrize("R,V,K,slices", [(97, 128256, 10, 2), (51, 128256, 10, 4), (200, 50257, 10, 1), (40, 8000, 40, 1), (97, 8000, 10, 1),
                                          (16, 12000, 3, 1), (10, 128256, 10, 16), (600, 8193, 10, 1), (260, 131072, 10, 2),
                                          (260, 61443, 10, 3), (7, 137847, 10, 34), (14, 70001, 24, 18), (16, 70001, 24, 9), (342, 61443, 1, 1)])
def test_a_workspace_for_the_slices_of_the_call(G, R, V, K, slices):
    """A call asks for the slices that its own rows are cut into (a statistics record of 16 bytes and K keys of
    8 each, behind the 65536 counters), not for what smaller calls could need, and is refused without them."""
    import paper_2505_13254_amd as hs
    up = lambda n: -(-n // 256) * 256
    need = 4 * 65536 + up(R * slices * 16) + up(R * slices * K * 8)
    x = (np.random.RandomState(R).randn(R, V) * 2).astype(np.float32)
    want, xd = draft_entropy_topk(x, K, 1.0), G.dev(x)
    guard = torch.full((need + 4096,), 77, dtype=torch.uint8, device=G.DEV)
    ws = guard[:need]
    hs.hs_workspace_prepare(ws)
    for fused in (True, False):
        got = {k: G.host(v) for k, v in hs.hs_draft_entropy_topk(xd, K, 1.0, ws=ws, fused=fused).items()}
        assert np.array_equal(got["topk_idx"], want["topk_idx"])
        for k in ("ent_topk", "ent_full"):
            assert G.entropy_err(got[k], want[k]) <= 1.0, k
    assert bool((guard[need:] == 77).all())
    with pytest.raises(hs.HsError):
        hs.hs_draft_entropy_topk(xd, K, 1.0, ws=ws[:need - 256])


def test_accept_workspaces_hold_every_smaller_call(G):
    """A workspace made for the largest tree serves all smaller ones in every mode, and nothing is written behind it."""
    import paper_2505_13254_amd as hs
    from test_gpu_entropy_prune_accept import _accept_equal
    from oracle import verify_accept
    rs = np.random.RandomState(3)
    V, top = 50257, 140
    for mode in (0, 1, 2):
        need = hs.lib().hs_verify_accept_workspace_mode(1, top, V, mode)
        guard = torch.full((need + 4096,), 77, dtype=torch.uint8, device=G.DEV)
        for NN in (1, 2, 5, 9, 17, 64, 129, top):
            target = (rs.normal(size=(NN, V)) * 3).astype(np.float32)
            draft = (target + rs.normal(size=(NN, V))).astype(np.float32)
            parent = np.asarray([-1] + [(i - 1) // 3 for i in range(1, NN)], np.int32)
            token = np.zeros(NN, np.int32)
            for i in range(1, NN):  # (one of the likely tokens of the parent's row, another for each sibling)
                token[i] = np.argsort(-target[parent[i]], kind="stable")[(i - 1) % 3]
            offs = np.asarray([0, NN], np.int32)
            u = np.concatenate([rs.rand(NN), [0.5]]).astype(np.float32)
            args = [G.dev(target), G.dev(draft), G.dev(token, torch.int32), G.dev(parent, torch.int32), G.dev(offs, torch.int32), mode, 1.0,
                    G.dev(u, torch.float32), 6]
            near = [verify_accept(target, draft, token, parent, offs, mode, 1.0, np.clip(u.astype(np.float64) + d, 0.0, 1.0 - 1e-12), 6)
                    for d in (-1e-5, 0.0, 1e-5)]
            got = {k: G.host(v) for k, v in hs.hs_verify_accept(*args, ws=guard[:need]).items()}
            if all(np.array_equal(n[k], near[1][k]) for n in near for k in near[1] if k in got):
                _accept_equal(got, near[1])
        assert bool((guard[need:] == 77).all())


@pytest.mark.parametrize("R,V,slices", [(2, 11379, 3), (16, 8191, 2), (9, 8192, 1), (257, 8193, 3), (341, 4099, 2), (342, 8193, 1), (260, 12288, 3),
                                        (360, 98304, 2), (361, 98304, 1), (400, 98305, 2)])
def test_argmax_slices_of_a_greedy_walk(G, R, V, slices):
    """Greedy walks over rows cut into up to three slices, aligned or not: every row's largest value stands in two
    places, in the first tile and in the last, and the first one counts.  The workspace holds the slices of the call
    (records of 16 bytes, keys of 8, behind the 65536 counters and the walk's arrays), and no less will do."""
    import paper_2505_13254_amd as hs
    rs = np.random.RandomState(R + V)
    x = torch.randn((R, V), generator=torch.Generator(device=G.DEV).manual_seed(R), device=G.DEV)
    best = rs.randint(0, 4000, size=R)
    rows = torch.arange(R, device=G.DEV)
    x[rows, torch.from_numpy(V - 1 - rs.randint(0, 60, size=R)).to(G.DEV)] = 9.0
    x[rows, torch.from_numpy(best).to(G.DEV)] = 9.0
    # a chain through the first rows, the others hang off it with tokens that no row confirms
    n = min(R, 9)
    parent = np.asarray([-1] + [i - 1 if i < n else rs.randint(0, n) for i in range(1, R)], np.int32)
    token = np.asarray([0] + [best[i - 1] if i < n else 4096 + i for i in range(1, R)], np.int32)
    args = [x, None, G.dev(token, torch.int32), G.dev(parent, torch.int32), G.dev(np.asarray([0, R]), torch.int32), 0, 1.0, None, 12]
    up = lambda n: -(-n // 256) * 256
    query = hs.lib().hs_verify_accept_workspace_mode(1, R, V, 0)
    guard = torch.full((query + 4096,), 77, dtype=torch.uint8, device=G.DEV)
    own = 3 * up(8 * R) + 5 * up(8 * R) + up(2 * R) + 4 * 65536 + up(R * slices * 16) + up(R * slices * 8)
    assert own <= query
    got = hs.hs_verify_accept(*args, ws=guard[:own])
    assert int(got["accept_len"][0]) == n - 1
    assert got["accept_path"][0, :n - 1].tolist() == list(range(1, n))
    assert int(got["bonus_token"][0]) == best[n - 1]
    assert bool((guard[own:] == 77).all())
    with pytest.raises(hs.HsError):
        hs.hs_verify_accept(*args, ws=guard[:own - 256])


@pytest.mark.parametrize("n,depth", [(17, 15), (17, 16), (18, 17), (512, 16), (513, 17), (1024, 16), (1025, 15), (4096, 16), (4097, 16), (8192, 16), (8193, 17)])
def test_trees_around_the_limits_of_a_workgroup(G, n, depth):
    """Trees as deep as a walk in registers and one level deeper, with as many rows as a workgroup has threads or LDS has
    room for, and one more; many equal values.  One tree, and three in a batch."""
    from oracle import adaptive_control, tree_prune
    import paper_2505_13254_amd as hs
    from test_gpu_entropy_prune_accept import _prune_equal
    rs = np.random.RandomState(n + depth)
    def tree(m):
        d, par = [0], [-1]
        for i in range(1, m):                                          # a chain first, then anywhere above the last level
            p = i - 1 if i <= depth else int(rs.randint(0, i))
            while d[p] >= depth:
                p = par[p]
            par.append(p)
            d.append(d[p] + 1)
        lc = np.round(-rs.exponential(0.4, size=m) * 4).astype(np.float32) / 4
        lc[0] = 0
        return np.asarray(par, np.int32), lc
    for sizes in ([n], [n, 5, max(1, n // 3)]):
        ts = [tree(m) for m in sizes]
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        par, lc = np.concatenate([t[0] for t in ts]), np.concatenate([t[1] for t in ts])
        B = len(sizes)
        for budget in (0, max(1, n // 2)):
            pin = dict(parent=par, logc=lc, node_offsets=off, d_max=np.full(B, depth - (budget > 0), np.int32),
                       theta=np.full(B, -6.0, np.float32), max_nodes=np.full(B, budget, np.int32))
            _prune_equal(G.run_prune(pin), tree_prune(par, lc, off, pin["d_max"], pin["theta"], pin["max_nodes"]))
        ent = rs.uniform(0.0, 0.4, size=len(par)).astype(np.float32)
        for mode in (0, 1):
            want = adaptive_control(par, lc, ent, off, [1.0, 2.0, 3.0], [0.5, 0.8], 3, 6, 60, mode)
            got = hs.hs_adaptive_control(G.dev(par), G.dev(lc), G.dev(ent), G.dev(off), None, [1.0, 2.0, 3.0], [0.5, 0.8], 3, 6, 60, mode)
            for k in ("pstar", "bin", "d_prime", "n_prime"):
                assert np.array_equal(G.host(got[k]), want[k]), (k, mode)
            assert np.allclose(G.host(got["phi"]), want["phi"], rtol=1e-5, atol=1e-8)


@pytest.mark.parametrize("K,F", [(10, 10), (1, 7), (13, 10), (16, 40), (4, 1), (3, 300)])
def test_expansion_of_equal_values(G, K, F):
    """Rows of equal value go by their number, across the threads that share a comparison and the ends of their pieces."""
    import paper_2505_13254_amd as hs
    from oracle.tree_expand import new_state, tree_expand
    rs = np.random.RandomState(K * F)
    cap = 1 + 5 * K * F
    state, ref = hs.new_tree_state(1, cap, F, G.DEV), new_state()
    for lvl in range(4):
        lp = np.round(-rs.exponential(0.5, size=(F, K)) * 2).astype(np.float32) / 2
        idx, ent = rs.randint(0, 1000, size=(F, K)).astype(np.int32), rs.uniform(0, 2, size=F).astype(np.float32)
        hs.hs_tree_expand(state, G.dev(idx), G.dev(lp), G.dev(ent), None, 1, cap, F, K, first=lvl == 0)
        tree_expand(ref, idx, lp, ent, F, cap, None)
        n, nf = int(G.host(state["n_nodes"])[0]), int(G.host(state["n_frontier"])[0])
        assert n == len(ref["parent"]) and list(G.host(state["frontier"])[:nf]) == ref["frontier"], lvl
        assert np.array_equal(G.host(state["parent"])[:n], ref["parent"])
        assert np.array_equal(G.host(state["cumlogp"])[:n].view(np.uint32), np.asarray(ref["cum"], np.float32).view(np.uint32))


@pytest.mark.parametrize("sizes,V,pad,depth", [
    ([9000, 9000], 700, 0, 2), ([9000, 9000], 701, 0, 2), ([3, 5000, 0, 4097, 1], 1025, 3, 2), ([60] * 90, 4096, 0, 3),
    ([60] * 90, 4099, 0, 3), ([33] * 30, 65536, 0, 4), ([33] * 20, 65540, 0, 2), ([33] * 40, 65539, 0, 1), ([17] * 40, 131071, 1, 3),
    ([2000, 2000], 4100, 0, 3), ([6000] * 10, 130, 2, 1)])
def test_greedy_walk_by_paths(G, sizes, V, pad, depth):
    """Greedy calls of so many rows that only the paths' rows are read: rows of less than one piece of a workgroup, of whole
    ones and of one more value, aligned or not, trees beyond LDS, empty sequences; equal largest values, masked rows, siblings
    that carry the same token (the deepest confirmed row counts, then the lowest), paths cut off at the depth limit.  Rows
    off the paths are NaN where the outcome may not depend on them."""
    import paper_2505_13254_amd as hs
    rs = np.random.RandomState(V + len(sizes))
    NN = sum(sizes)
    x = torch.full((NN, V + pad), float("nan"), device=G.DEV)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    parent, token, want = [], [], []
    for s, n in enumerate(sizes):
        if n == 0:
            want.append((0, [], -1))
            continue
        par = [-1] + [int(rs.randint(max(0, i - 8), i)) if i < 40 else int(rs.randint(0, i)) for i in range(1, n)]
        tok = rs.randint(0, V, size=n)
        arg = {}
        def row(i):
            if i not in arg:
                r = np.round(rs.randn(V).astype(np.float32) * 4) / 4
                if rs.rand() < 0.3:
                    r[rs.randint(0, V):] = -np.inf
                if rs.rand() < 0.1:
                    r[:] = -np.inf
                x[int(off[s]) + i, :V] = torch.from_numpy(r).to(G.DEV)
                arg[i] = int(np.argmax(r))
            return arg[i]
        level, d = [0], 0
        while True:
            for i in level:
                a = row(i)
                kids = [c for c in range(1, n) if par[c] == i]
                for c in kids:
                    if tok[c] == a:
                        tok[c] = (a + 1) % V
                for c in kids[:: max(1, len(kids) - 1)][:2] if rs.rand() < 0.8 else []:  # (up to two siblings of one token)
                    tok[c] = a
            nxt = [c for c in range(1, n) if par[c] in level and tok[c] == arg[par[c]]] if d < depth else []
            if not nxt:
                break
            level, d = nxt, d + 1
        path, i = [], min(level)
        while i > 0:
            path.append(i)
            i = par[i]
        want.append((d, path[::-1], arg[min(level)]))
        parent += par
        token += list(tok)
    out = hs.hs_verify_accept(x[:, :V], None, G.dev(np.asarray(token, np.int32)), G.dev(np.asarray(parent, np.int32)), G.dev(off), 0, 1.0, None, depth)
    out = {k: G.host(v) for k, v in out.items()}
    for s, (d, path, bonus) in enumerate(want):
        assert int(out["accept_len"][s]) == d and int(out["bonus_token"][s]) == bonus, s
        assert list(out["accept_path"][s]) == path + [-1] * (depth - d), s
    assert max(w[0] for w in want) >= 1
