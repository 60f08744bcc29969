"""GPU parity where the values, not the shapes, are the hard part: softmax weights that must not
lose bits, results near the end of the type's range, values that are not finite.  Attention inputs
here are made by hand: the query is (1, 1, 0, ...), so the score of a key is the sum of its first
two entries, and the columns of V are chosen so that errors of the weights stay when the result
itself is small."""
import numpy as np
import pytest
import torch

from paper_2402_13485_amd import synth
from gpu_util import host_f64, to_host
from test_gpu_dispatch import raw_attention
from test_gpu_parity import dev_tree, pb, run_attention  # noqa: F401

pytestmark = pytest.mark.gpu


def hand_made(dtype, H, d, T, score, second, values):
    """One sequence, a tree of T children of the root whose own keys weigh next to nothing;
    cached keys with scores score[H,L] + second[H,L] and V rows values[H,L,d]."""
    L = score.shape[1]
    w = synth.Workload(91, "case", dtype, 1, H, d, T, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array([L], np.int32), trees=[synth.star_tree(T)])
    k = np.zeros((1, H, L, d), np.float32)
    k[0, :, :, 0], k[0, :, :, 1] = score, second
    q = np.zeros((1, H, T, d), np.float32)
    q[..., 0] = q[..., 1] = 1.0
    kt = np.zeros((1, H, T, d), np.float32)
    kt[..., 0] = -80.0
    x.update(q=synth.from_float(q, dtype), k_cache=synth.from_float(k, dtype), k_tree=synth.from_float(kt, dtype),
             v_cache=synth.from_float(values[None].astype(np.float32), dtype),
             v_tree=synth.from_float(np.zeros((1, H, T, d), np.float32), dtype), scale=1.0)
    return x


def reference(oracle, x):
    return oracle.tree_attention(x["n_nodes"], x["parent"], x["seq_lens"], x["q"], x["k_cache"], x["v_cache"],
                                 x["k_tree"], x["v_tree"], x["scale"])


def bf16(a):
    return synth.as_float(synth.f32_to_bf16_bits(np.asarray(a, np.float32)))


@pytest.mark.parametrize("d", [64, 128])
def test_attention_short_cache_keeps_two_stages_to_a_piece(pb, oracle, d):
    """96 cached rows and a tree are four stages of 32 rows, cut into two pieces of two.  Rows 0
    and 64, one in each piece, hold all the weight; the largest weight of a piece is exactly 1, so bf16
    weights lose nothing, and two values that nearly cancel leave fp32 errors (2e-6 of them) and the
    rounding of the result.  In one piece the smaller weight would be rounded to 8 bits."""
    rng = np.random.default_rng(5)
    H, L = 8, 96
    score = np.full((H, L), -80.0)
    score[:, 0] = 0.0
    score[:, 64] = bf16(rng.uniform(-2.0, -0.1, H))
    v = np.zeros((H, L, d))
    v[:, 0] = bf16(rng.uniform(1.0, 2.0, (H, d)))
    v[:, 64] = -bf16(v[:, 0] / np.exp(score[:, 64:65]))
    x = hand_made("bf16", H, d, 1, score, np.zeros((H, L)), v)
    ref = reference(oracle, x)
    got = host_f64(run_attention(pb, x)[0])
    assert (np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 8e-6).all(), np.abs(got - ref).max()


def test_attention_d64_weights_keep_fp32_precision(pb, oracle):
    """Two keys per column of V with values +1 and -1 and weights w and w (1 + 2^-11): what is left is
    2^-11 w, so an error of the weights of 2^-18 would be one of 2^-7 in the result.  fp32 weights: the
    rounding of the exponents (2^-23 and less), of the exponentials and of the sums, 2e-3 of the
    result together; then the result is rounded to bf16 (2^-9)."""
    rng = np.random.default_rng(6)
    H, d, L, T = 4, 64, 129, 9
    score, second, v = np.full((H, L), 0.0), np.zeros((H, L)), np.zeros((H, L, d))
    s = bf16(rng.uniform(-2.0, -0.05, (H, d)))
    score[:, 1::2], score[:, 2::2] = s, s
    second[:, 2::2] = 2.0 ** -11
    for i in range(d):
        v[:, 1 + 2 * i, i], v[:, 2 + 2 * i, i] = -1.0, 1.0
    x = hand_made("bf16", H, d, T, score, second, v)
    ref = reference(oracle, x)
    got = host_f64(run_attention(pb, x)[0])
    assert (np.abs(got - ref) <= (2.0 ** -9 + 2e-3) * np.abs(ref)).all(), (np.abs(got - ref) / np.abs(ref)).max()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention_d64_values_near_the_largest(pb, oracle, dtype):
    """A maximum that rises after the first rows, and V values within a factor of four of the
    largest float: products of weights above 1 would overflow where the result does not."""
    rng = np.random.default_rng(7)
    H, d, L = 3, 64, 200
    score = rng.uniform(-3.0, -1.0, (H, L))
    score[:, 40], score[:, 130] = 3.0, 4.5
    v = bf16(rng.uniform(-1.0, 1.0, (H, L, d)))
    v[:, 40], v[:, 130] = 1e38, -5e37
    x = hand_made(dtype, H, d, 2, bf16(score), np.zeros((H, L)), v)
    ref = reference(oracle, x)
    got = host_f64(run_attention(pb, x)[0])
    assert np.isfinite(ref).all() and np.isfinite(got).all()
    assert (np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref)).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64)])
def test_attention_with_next_to_no_scale(pb, oracle, dtype, d):
    """A scale of 2^-130 makes all weights equal."""
    rng = np.random.default_rng(9)
    x = hand_made(dtype, 2, d, 3, bf16(rng.uniform(-3.0, 3.0, (2, 100))), np.zeros((2, 100)),
                  bf16(rng.uniform(0.5, 1.0, (2, 100, d))))
    x["scale"] = 2.0 ** -130
    ref = reference(oracle, x)
    got = host_f64(run_attention(pb, x)[0])
    assert (np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref)).all()


def timed(f):
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return sorted(times)[2]


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("where", ["cache", "leaf"])
def test_attention_not_finite_values_cost_no_more(pb, dtype, d, where):
    """One V row per (sequence, head) that holds a NaN: the call takes as long as without (a factor
    of four is allowed; work done query by query for such units takes a hundred times as long)."""
    B, H, T, L = 2, 8, 64, 2048
    gen = torch.Generator(device="cuda").manual_seed(8)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    normal = lambda *s: torch.randn(s, device="cuda", dtype=dt, generator=gen)
    n_nodes, parent, _ = synth.pad_trees([synth.rank_product_tree(T, 4)] * B, T)
    tree = dev_tree(pb, n_nodes, parent)
    q, kt, vt, kc, vc = normal(B, H, T, d), normal(B, H, T, d), normal(B, H, T, d), normal(B, H, L, d), normal(B, H, L, d)
    seq = torch.full((B,), L, dtype=torch.int32, device="cuda")
    call = lambda: pb.propd_tree_attention(tree, q, kc, vc, kt, vt, seq, d ** -0.5)
    clean_out = call()
    clean = timed(call)
    (vc if where == "cache" else vt)[:, :, T - 1, 5] = float("nan")
    out = call()
    seen = torch.zeros_like(out, dtype=torch.bool)
    seen[:, :, (slice(None) if where == "cache" else T - 1), 5] = True  # the last node is a leaf
    assert torch.isnan(out[seen]).all()
    tol = 2.0 ** -8 if dtype == "bf16" else 1e-5
    assert ((out - clean_out)[~seen].abs() <= tol * clean_out.abs().max()).all()
    assert timed(call) <= 4 * clean + 0.05


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_attention_not_finite_keys_stay_where_they_are_seen(pb, dtype, d, value):
    """K entries of a leaf that are not finite reach the leaf's own row and no other."""
    shapes = [synth.rank_product_tree(70, 4)] * 2
    w = synth.Workload(92, "case", dtype, 2, 2, d, 70, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array([600, 33], np.int32), trees=shapes)
    want = host_f64(run_attention(pb, x)[0])
    leaf = 69
    y = dict(x, k_tree=x["k_tree"].copy())
    y["k_tree"][:, :, leaf, 11] = synth.from_float(np.array([value], np.float32), dtype)[0]
    got = host_f64(run_attention(pb, y)[0])
    score = synth.as_float(x["q"])[:, :, leaf, 11] * value  # NaN and +inf: no softmax; -inf: a weight of zero
    assert (np.isnan(got[:, :, leaf]).all(axis=-1) == ~(score < 0)).all()
    rest = [t for t in range(70) if t != leaf]
    tol = 2.0 ** -8 if dtype == "bf16" else 1e-5
    assert (np.abs(got - want)[:, :, rest] <= tol * np.abs(want[:, :, rest]).max(axis=-1, keepdims=True)).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("L", [5, 600])
def test_attention_infinities_of_both_signs(pb, oracle, dtype, d, L):
    """+inf and -inf in V, in one column, in two and in both signs of one column, in cached rows (the
    last one too, which fills its stage) and in tree rows, seen by some nodes and not by others:
    every result is the sum that the node sees."""
    shapes = [synth.rank_product_tree(40, 4)]
    w = synth.Workload(93, "case", dtype, 1, 2, d, 40, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array([L], np.int32), trees=shapes)
    inf = lambda s: synth.from_float(np.array([s * np.inf], np.float32), dtype)[0]
    x["v_cache"][0, :, L - 1, 2] = inf(1)
    x["v_cache"][0, :, 1, 3] = inf(-1)
    x["v_cache"][0, :, 0, 4], x["v_cache"][0, :, L - 1, 4] = inf(1), inf(-1)
    x["v_tree"][0, :, 7, 5], x["v_tree"][0, :, 39, 5], x["v_tree"][0, :, 12, 6] = inf(1), inf(-1), inf(-1)
    with np.errstate(all="ignore"):
        ref = reference(oracle, x)
    got = host_f64(run_attention(pb, x)[0])
    assert not np.isfinite(ref[..., 2:5]).any() and np.isfinite(ref[..., 5]).any() and np.isinf(ref[..., 5]).any()
    same = np.isfinite(ref)
    assert (np.isnan(got) == np.isnan(ref)).all() and (got[~same & ~np.isnan(ref)] == ref[~same & ~np.isnan(ref)]).all()
    tol = 2e-2 if dtype == "bf16" else 1e-5
    assert (np.abs(got[same] - ref[same]) <= tol * max(1.0, np.abs(ref[same]).max())).all()


def same_kind_of_result(x, plain, tiled, sent):
    a, b = host_f64(plain), host_f64(tiled)
    for s in range(x["B"]):
        n = int(x["n_nodes"][s])
        one, other = a[s, :, :n], b[s, :, :n]
        assert np.array_equal(np.isnan(one), np.isnan(other))
        assert np.array_equal(np.isposinf(one), np.isposinf(other))
        assert np.array_equal(np.isneginf(one), np.isneginf(other))
        fin = np.isfinite(one)
        # both round a result that differs by fp32 sums only
        assert (np.abs(one[fin] - other[fin]) <= 2.0 ** -7 * np.maximum(np.abs(one[fin]), 1e-3)).all()
        assert (to_host(tiled)[s, :, n:] == sent[s, :, n:]).all()


@pytest.mark.parametrize("T,L", [(1, 33), (20, 0), (70, 31), (128, 300), (64, 2000)])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_attention_d64_not_finite_like_the_plain_kernel(pb, T, L, value):
    """With and without a workspace (tiled kernel, one wave per query): the same results are NaN, the
    same are infinite, and the finite ones agree, whatever is not finite among V, and for infinities in
    K (a NaN there is a NaN score, whose maximum the plain kernel does not define)."""
    rng = np.random.default_rng(T + L)
    w = synth.Workload(96, "case", "bf16", 2, 2, 64, T, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array([L, L // 2], np.int32), L_max=max(L, 1),
                                    trees=[synth.random_tree(rng, T), synth.random_tree(rng, max(1, T // 2))])
    bad = synth.from_float(np.array([value], np.float32), "bf16")[0]
    for name, n in (("v_tree", 3), ("v_cache", 2), ("k_tree", 0 if np.isnan(value) else 1)):
        rows = x[name].shape[2]
        for _ in range(n):
            x[name][:, rng.integers(0, 2), rng.integers(0, rows), rng.integers(0, 64)] = bad
    st, plain, sent = raw_attention(pb, x, workspace="none")
    assert st == 0
    st, tiled, _ = raw_attention(pb, x, workspace="full")
    assert st == 0
    same_kind_of_result(x, plain, tiled, sent)


@pytest.mark.parametrize("B,H,lens", [(1, 700, [90]), (3, 400, [64, 64, 64]), (5, 80, [300, 0, 1000, 33, 640])])
def test_attention_d64_not_finite_in_the_middle_of_a_workgroup(pb, B, H, lens):
    """Workgroups that do several units and parts of units, some of which are done a second time:
    whole units first and the rest cut, and ranges over ragged units."""
    rng = np.random.default_rng(B * H)
    T = 40
    w = synth.Workload(97, "case", "bf16", B, H, 64, T, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array(lens, np.int32),
                                    trees=[synth.random_tree(rng, T - 7 * (b % 2)) for b in range(B)])
    for value in (np.nan, np.inf, -np.inf):
        bad = synth.from_float(np.array([value], np.float32), "bf16")[0]
        for name in ("v_tree", "v_cache"):
            for _ in range(B * H // 8):
                x[name][rng.integers(0, B), rng.integers(0, H), rng.integers(0, x[name].shape[2]), rng.integers(0, 64)] = bad
    st, plain, sent = raw_attention(pb, x, workspace="none")
    assert st == 0
    st, tiled, _ = raw_attention(pb, x, workspace="full")
    assert st == 0
    same_kind_of_result(x, plain, tiled, sent)


def test_attention_f32_many_units(pb):
    """2^24 units of one node and no cache: more workgroups than one launch dimension takes in
    threads (2^32 of them).  A node that sees itself alone returns its own V row."""
    B, H, d = 1 << 14, 1 << 10, 64
    nn = torch.ones(B, dtype=torch.int32, device="cuda")
    par = torch.full((B, 1), -1, dtype=torch.int32, device="cuda")
    depth, anc = pb.propd_tree_mask(nn, par)
    tree = pb.Tree(n_nodes=nn, parent=par, depth=depth, anc=anc)
    q = torch.empty((B, H, 1, d), device="cuda").normal_()
    v = torch.empty((B, H, 1, d), device="cuda").normal_()
    none = torch.empty((B, H, 0, d), device="cuda")
    out = pb.propd_tree_attention(tree, q, none, none, q, v, torch.zeros(B, dtype=torch.int32, device="cuda"), 0.125)
    assert torch.equal(out, v)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
def test_attention_replayed_with_values_that_come_and_go(pb, dtype, d):
    """A captured call, replayed on inputs that are finite, hold a NaN and are finite again, with the
    caller's own work between the replays: each replay gives the eager bits."""
    B, H, T, L = 2, 4, 48, 700
    gen = torch.Generator(device="cuda").manual_seed(10)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    normal = lambda *s: torch.randn(s, device="cuda", dtype=dt, generator=gen)
    n_nodes, parent, _ = synth.pad_trees([synth.rank_product_tree(T, 4)] * B, T)
    tree = dev_tree(pb, n_nodes, parent)
    q, kt, vt, kc, vc = normal(B, H, T, d), normal(B, H, T, d), normal(B, H, T, d), normal(B, H, L, d), normal(B, H, L, d)
    seq = torch.full((B,), L, dtype=torch.int32, device="cuda")
    ws = torch.empty(pb.workspace_bytes(pb.WS_TREE_ATTENTION, B, T, H, d, L), dtype=torch.uint8, device="cuda")
    out = torch.zeros_like(q)
    call = lambda: pb.propd_tree_attention(tree, q, kc, vc, kt, vt, seq, d ** -0.5, out=out, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    kept = vt[1, 2, 30, 7].clone()
    for value in (None, float("nan"), float("inf"), None):
        vt[1, 2, 30, 7] = kept if value is None else value
        call()
        want = out.clone()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16 if dtype == "bf16" else torch.int32),
                           want.view(torch.int16 if dtype == "bf16" else torch.int32))


@pytest.mark.parametrize("T", [40, 70])  # two waves per 32 queries and one
@pytest.mark.parametrize("B,H,L", [(16, 32, 16640), (4, 32, 65100)])  # 512 workgroups: whole units, units of four pieces
@pytest.mark.parametrize("scores", ["one", "falling"])
def test_attention_high_scores_in_front_of_long_pieces(pb, scores, B, H, L, T):
    """Pieces of 500 stages and more, in which the softmax reference is set anew sixteen times and more, while
    their scores lie up to 2^288 below that of the first key ("one"), or fall with every stage.  Query t has its own distance,
    t * 4 in natural units at most 200, so that the other keys count for some queries and for some they do not."""
    d = 128
    gap = np.minimum(4.0 * np.arange(T), 200.0)
    # a key's score is gap * fall, exact in bf16 and fp32
    fall = np.zeros(L) if scores == "one" else bf16(1.0 - np.arange(L) // 32 * 32 / L)
    fall[0] = 1.0
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    kc = torch.zeros(B, H, L, d, device="cuda", dtype=torch.bfloat16)
    kc[..., 0] = torch.from_numpy(fall).to(torch.bfloat16).cuda()
    vc = torch.empty(B, H, L, d, device="cuda", dtype=torch.bfloat16).normal_(generator=gen)
    kt = torch.zeros(B, H, T, d, device="cuda", dtype=torch.bfloat16)
    vt = torch.empty(B, H, T, d, device="cuda", dtype=torch.bfloat16).normal_(generator=gen)
    q = torch.zeros(B, H, T, d, device="cuda", dtype=torch.bfloat16)
    q[..., 0] = torch.from_numpy(gap).cuda()
    n, parent, _ = synth.pad_trees([synth.chain_tree(T)] * B, T)
    tree = dev_tree(pb, n, parent)
    out = pb.propd_tree_attention(tree, q, kc, vc, kt, vt, torch.full((B,), L, dtype=torch.int32, device="cuda"), 1.0)
    # the weights are the same for all units; node t sees the tree rows 0..t
    w = torch.exp(torch.from_numpy(gap[:, None] * (fall[None] - 1.0)).cuda())
    wt = torch.exp(torch.from_numpy(-gap).cuda())[:, None] * torch.ones(T, T, device="cuda", dtype=torch.float64).tril()
    total = (w.sum(1) + wt.sum(1))[:, None]
    for b, h in ((0, 0), (0, 1), (B // 2, H - 1), (B - 1, H - 1)):
        v, v2 = vc[b, h].double(), vt[b, h].double()
        ref = (w @ v + wt @ v2) / total
        # a weight and the sum of the rounded weights: 2^-9 each, so 2^-8 of the sum of all terms; 2^-9 for the result,
        # and fp32 sums
        bound = (2 ** -8 + 2 ** -14) * (w @ v.abs() + wt @ v2.abs()) / total + 2 ** -9 * ref.abs() + 1e-6
        got = out[b, h].double()
        assert bool(torch.isfinite(got).all()), (b, h)
        assert bool(((got - ref).abs() <= bound).all()), (b, h, ((got - ref).abs() - bound).max().item())
    assert bool(torch.isfinite(out).all())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_prune_empty_slots_cost_next_to_nothing(pb, dtype):
    """128 trees of two nodes in slots of 128 and of 4: the epilogue of the tiles of few rows takes the nodes that exist
    (a walk over all slots took 1.6 to 1.8 times as long, this 1.1)."""
    B, Hd, V = 128, 128, 65536
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    head = torch.randn(V, Hd, device="cuda", dtype=dt)
    took = {}
    for T in (4, 128):
        n, parent, _ = synth.pad_trees([synth.chain_tree(2)] * B, T)
        tree = dev_tree(pb, n, parent, np.full((B, T), 7, np.int32))
        hid = torch.randn(B, T, Hd, device="cuda", dtype=dt)
        ws = torch.empty(pb.workspace_bytes(pb.WS_EARLY_PRUNE, B, T, hidden=Hd, vocab=V), dtype=torch.uint8, device="cuda")
        call = lambda: pb.propd_early_prune(tree, hid, head, V // 2, workspace=ws)
        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):  # the kernels without the host's time
            for _ in range(20):
                call()
        graph.replay()
        took[T] = timed(graph.replay)
    assert took[128] < 1.35 * took[4], took
