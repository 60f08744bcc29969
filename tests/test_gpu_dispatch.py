"""GPU parity at the edges of the kernels' dispatch rules: row counts, lengths, alignments and
types on both sides of every line where a call changes its kernel or tile shape, against the
CPU oracle with the tolerances of test_gpu_parity."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2402_13485_amd import synth
from gpu_util import host_f64, sentinel_like, to_dev, to_host
from test_gpu_parity import (check_attention, check_prob, check_prune, dev_tree, pb,  # noqa: F401
                             prob_reference, run_attention, run_prob, run_prune, threshold_in_a_gap)

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------------ commit of the accepted path


@pytest.mark.parametrize("H,stride", [(64, 8), (65, 8), (4, 128), (5, 128), (1, 1), (31, 16), (21, 16), (22, 16),
                                      (11, 31), (16, 32), (17, 32), (33, 8)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_commit_one_launch_or_two(pb, oracle, dtype, H, stride):
    """Path buffers of up to 5461 pieces of 16 bytes per sequence, of 8192 from 32 nodes on, are committed
    in one launch, larger ones in two: both sides of the lines, paths of every length, caches with and
    without room."""
    rng = np.random.default_rng(H * 1000 + stride)
    B, T, d, L_max = 5, 128, 128 if dtype == "bf16" else 64, 40
    n_nodes = np.array([T, T, 1, 7, T], np.int32)
    token = rng.integers(0, 1000, (B, T)).astype(np.int32)
    alen = np.array([stride, max(1, stride // 2), 1, min(stride, 7), 1], np.int32)
    path = np.full((B, stride), -1, np.int32)
    for b in range(B):
        path[b, :alen[b]] = np.sort(rng.choice(n_nodes[b], alen[b], replace=False))
    nxt = rng.integers(0, 1000, B).astype(np.int32)
    seq = np.array([0, L_max - 3, L_max, 20, L_max - 1], np.int32)
    draw = lambda *s: (rng.integers(0, 1 << 15, s).astype(np.uint16) if dtype == "bf16"
                       else rng.standard_normal(s).astype(np.float32))
    kt, vt, kc, vc = draw(B, H, T, d), draw(B, H, T, d), draw(B, H, L_max, d), draw(B, H, L_max, d)
    kc_r, vc_r, seq_r, out_r = oracle.commit_path(n_nodes, token, alen, path, nxt, kt, vt, kc, vc, seq, out_stride=stride + 1)
    tree = dev_tree(pb, n_nodes, np.maximum(np.arange(T, dtype=np.int32)[None].repeat(B, 0) - 1, -1), token)
    kc_d, vc_d, seq_d = to_dev(kc), to_dev(vc), to_dev(seq)
    out = pb.propd_commit_path(tree, to_dev(alen), to_dev(path), to_dev(nxt), to_dev(kt), to_dev(vt), kc_d, vc_d, seq_d,
                               out_stride=stride + 1)
    assert (to_host(kc_d) == kc_r).all() and (to_host(vc_d) == vc_r).all()
    assert (to_host(seq_d) == seq_r).all() and (to_host(out) == out_r).all()


@pytest.mark.parametrize("B,H,stride,d", [(1 << 22, 1, 1, 8), ((1 << 22) + 3, 1, 1, 8), (9000, 1, 128, 64), (700, 3, 8, 128),
                                          (600, 7, 40, 32), (257, 16, 32, 64), (65, 63, 12, 64)])
def test_commit_many_sequences(pb, B, H, stride, d):
    """More sequences than a launch has room for with 1024 threads each, and batches whose threads
    take several pieces, in one round and in several."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B)
    T, L_max = min(5, max(1, stride - 2)), 2 if B > 10000 else 130
    draw = lambda low, high, *s: torch.randint(low, high, s, device="cuda", generator=gen, dtype=torch.int32)
    rows = lambda n: draw(-30000, 30000, B, H, n, d).to(torch.int16).view(torch.bfloat16)
    n_nodes = torch.full((B,), T, dtype=torch.int32, device="cuda")
    token, nxt, path = draw(0, 1000, B, T), draw(0, 1000, B), draw(0, T, B, stride)
    alen, seq = draw(1, stride + 1, B), draw(0, L_max + 1, B)
    kt, vt, kc, vc = rows(T), rows(T), rows(L_max), rows(L_max)
    old = seq.clone()
    want = []
    j = torch.arange(stride, device="cuda")
    b, at = ((j[None] < alen[:, None]) & (old[:, None] + j[None] < L_max)).nonzero(as_tuple=True)
    for tree_rows, cache in ((kt, kc), (vt, vc)):
        want.append(cache.clone().view(torch.int16))
        want[-1][b, :, old[b].long() + at] = tree_rows.view(torch.int16)[b, :, path[b, at].long()]
    out = pb.propd_commit_path(pb.Tree(n_nodes, draw(0, 1, B, T), token), alen, path, nxt, kt, vt, kc, vc, seq)
    assert torch.equal(kc.view(torch.int16), want[0]) and torch.equal(vc.view(torch.int16), want[1])
    assert torch.equal(seq, torch.minimum(old + alen, torch.full_like(old, L_max)))
    nodes = token.gather(1, torch.cat([path[:, 1:], path[:, :1]], 1).long())
    last = j[None] == alen[:, None] - 1
    assert torch.equal(out, torch.where(j[None] < alen[:, None] - 1, nodes, torch.where(last, nxt[:, None], -1)))


# ------------------------------------------------------------------ fp32 scoring


@pytest.mark.parametrize("shape,Hd,V", [("chain17", 16, 128), ("chain18", 129, 129), ("chain33", 363, 127),
                                        ("chain34", 130, 257), ("chain65", 64, 1003), ("chain66", 47, 513),
                                        ("chain128", 300, 300), ("star128", 33, 1003), ("chain2", 1, 130)])
def test_prune_f32_tile_edges(pb, oracle, shape, Hd, V):
    """One sequence with 1 .. 127 score rows (row tiles of 16, 32 and 64; a chain of T nodes has
    T - 1 rows), a node with more children than a wave has lanes, row lengths that are no
    multiple of four floats, of a chunk (16) or of a block of chunks, ragged column tiles."""
    T = int(shape[5:]) if shape.startswith("chain") else int(shape[4:])
    tree = synth.chain_tree(T) if shape.startswith("chain") else synth.star_tree(T)
    w = synth.Workload(71, "case", "f32", 1, 1, 64, T, Hd, V, 4, 1e-5)
    x = synth.make_prune_inputs(w, trees=[tree])
    x["tau"] = 1e-5
    res, sents = run_prune(pb, x, [x["hidden_states"]])
    check_prune(oracle, x, res, [x["hidden_states"]], sents)
    logm, _, _ = prob_reference(oracle, x, threshold=0.5)
    if T > 2:
        thr = float(np.float32(threshold_in_a_gap(logm, x["n_nodes"], 1e-4)))
        _, _, ref = prob_reference(oracle, x, threshold=thr)
        res, sents = run_prob(pb, x, [x["hidden_states"]], threshold=thr)
        check_prob(pb, oracle, x, res, ref, logm, [x["hidden_states"]], sents)


@pytest.mark.parametrize("Hd,offset", [(64, 4), (61, 0), (61, 12)])
def test_prune_f32_rows_at_any_float(pb, oracle, Hd, offset):
    """fp32 operands need 4-byte alignment only: bases off the 16-byte grid and rows of odd length."""
    w = synth.Workload(72, "case", "f32", 2, 1, 64, 32, Hd, 300, 4, 1e-5)
    x = synth.make_prune_inputs(w, trees=[synth.rank_product_tree(32, 4)] * 2)
    x["tau"] = 1e-5

    def shifted(a):
        t = to_dev(a)
        buf = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")
        view = buf[offset // 4:offset // 4 + t.numel()].view(t.shape)
        view.copy_(t)
        assert view.data_ptr() % 16 == offset
        return view

    tree = dev_tree(pb, x["n_nodes"], x["parent"], x["token"])
    res = pb.propd_early_prune(tree, shifted(x["hidden_states"]), shifted(x["head_weight"]), x["top_k"],
                               want_rank=True)
    check_prune(oracle, x, res)


# ------------------------------------------------------------------ attention, head size 64


def d64_case(seed, T_max, shapes, lens, H=3):
    w = synth.Workload(82, "case", "bf16", len(shapes), H, 64, T_max, 0, 0, 0, 1e-3)
    return synth.make_attention_inputs(w, seq_lens=np.asarray(lens, np.int32), trees=shapes)


def relative_error(oracle, x, out):
    ref = oracle.tree_attention(x["n_nodes"], x["parent"], x["seq_lens"], x["q"], x["k_cache"],
                                x["v_cache"], x["k_tree"], x["v_tree"], x["scale"])
    got, d2, r2 = host_f64(out), 0.0, 0.0
    for b in range(x["B"]):
        T = int(x["n_nodes"][b])
        d2 += ((got[b, :, :T] - ref[b, :, :T]) ** 2).sum()
        r2 += (ref[b, :, :T] ** 2).sum()
    return float(np.sqrt(d2 / r2))


@pytest.mark.parametrize("T_max,lens", [(1, [0, 1, 33]), (8, [31, 32, 2000]), (33, [64, 0, 65]),
                                        (64, [129, 700, 5]), (97, [1, 1000, 31]), (128, [300, 4096, 95])])
def test_attention_d64_matches_oracle(pb, oracle, T_max, lens):
    """The tiled kernel at head size 64: empty and ragged caches, one to four query groups, whole and
    cut units.  Its weights keep fp32 precision, so rounding the result to bf16 (at most 2^-9
    relative) is all the error there is, up to fp32 sums (1e-5)."""
    rng = np.random.default_rng(T_max)
    shapes = [synth.random_tree(rng, T_max), synth.chain_tree(max(1, T_max // 2)), synth.random_tree(rng, max(1, T_max - 1))]
    x = d64_case(T_max, T_max, shapes, lens)
    out, sent = run_attention(pb, x)
    check_attention(oracle, x, out, sent)
    assert relative_error(oracle, x, out) <= 2.0 ** -9 + 1e-5


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("direction", ["rising", "late_spike"])
def test_attention_moving_maximum_other_kernels(pb, oracle, dtype, direction):
    """Scores that grow along the cache move the reference of the online softmax again and again."""
    shapes = [synth.rank_product_tree(40, 4)] * 2
    w = synth.Workload(83, "case", dtype, 2, 2, 64, 40, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array([700, 333], np.int32), trees=shapes, poison=False)
    k = synth.as_float(x["k_cache"]).copy()
    L = k.shape[2]
    ramp = np.linspace(0.1, 6.0, L) if direction == "rising" else np.where(np.arange(L) == 321, 9.0, 0.3)
    x["k_cache"] = synth.from_float((k * ramp[None, None, :, None]).astype(np.float32), dtype)
    out, sent = run_attention(pb, x)
    check_attention(oracle, x, out, sent)


def raw_attention(pb, x, shift=0, workspace="full"):
    """The C entry point itself: tensors `shift` bytes off the 16-byte grid, any workspace."""
    import ctypes
    B, H, T_max, d = x["q"].shape
    es = 2 if x["dtype"] == "bf16" else 4

    def place(a):
        t = to_dev(a)
        buf = torch.empty(t.numel() + 16, dtype=t.dtype, device="cuda")
        v = buf[shift // es:shift // es + t.numel()].view(t.shape)
        v.copy_(t)
        return v

    tree = dev_tree(pb, x["n_nodes"], x["parent"])
    sent = sentinel_like(x["q"])
    q, kc, vc, kt, vt, out = (place(a) for a in (x["q"], x["k_cache"], x["v_cache"], x["k_tree"], x["v_tree"], sent))
    seq = to_dev(x["seq_lens"])
    need = pb.workspace_bytes(pb.WS_TREE_ATTENTION, B, T_max, H, d, kc.shape[2])
    size = {"full": need, "short": need - 1, "none": 0}[workspace]
    ws = torch.empty(max(size, 1), dtype=torch.uint8, device="cuda")
    c_tree = tree._c()
    st = pb.load_library().propd_tree_attention(
        ctypes.byref(c_tree), pb.PROPD_BF16 if x["dtype"] == "bf16" else pb.PROPD_F32, H, d, x["scale"],
        q.data_ptr(), kc.data_ptr(), vc.data_ptr(), kt.data_ptr(), vt.data_ptr(), seq.data_ptr(), kc.shape[2],
        out.data_ptr(), ws.data_ptr() if workspace != "none" else None, size, None)
    torch.cuda.synchronize()
    return st, out, sent


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("shift,workspace", [(0, "none"), (0, "short"), (4, "full"), (0, "full")])
def test_attention_without_workspace_or_alignment(pb, oracle, dtype, d, shift, workspace):
    """fp32 tensors and bf16 tensors with head size 64 are served whatever the workspace is and
    wherever the tensors lie."""
    rng = np.random.default_rng(3)
    shapes = [synth.random_tree(rng, 37), synth.random_tree(rng, 50)]
    w = synth.Workload(84, "case", dtype, 2, 2, d, 50, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array([257, 70], np.int32), trees=shapes)
    st, out, sent = raw_attention(pb, x, shift, workspace)
    assert st == 0
    check_attention(oracle, x, out, sent)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("L", [5, 600])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_attention_not_finite_values_stay_where_they_are_seen(pb, oracle, dtype, d, L, value):
    """V rows of a leaf that hold NaN or an infinity reach the leaf's own result and no other."""
    shapes = [synth.rank_product_tree(70, 4)] * 2
    w = synth.Workload(85, "case", dtype, 2, 2, d, 70, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array([L, L], np.int32), trees=shapes)
    clean, _ = run_attention(pb, x)
    leaf = 69
    assert not (x["parent"][1] == leaf).any()
    y = dict(x, v_tree=x["v_tree"].copy())
    y["v_tree"][1, :, leaf, 3:40:7] = synth.from_float(np.array([value], np.float32), dtype)[0]
    got = host_f64(run_attention(pb, y)[0])
    want = host_f64(clean)
    assert not np.isfinite(got[1, :, leaf, 3:40:7]).any()
    got[1, :, leaf, 3:40:7] = want[1, :, leaf, 3:40:7]
    tol = 2.0 ** -8 if dtype == "bf16" else 1e-5   # one bf16 rounding either way; fp32 sums
    row = np.abs(want[:, :, :70]).max(axis=-1, keepdims=True)
    assert (np.abs(got - want)[:, :, :70] <= tol * row).all()


# ------------------------------------------------------------------ attention, fp32


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T_max,H,lens", [(1, 1, [0, 1]), (16, 2, [128, 17]), (17, 1, [15, 3000]), (33, 2, [700, 0]),
                                          (70, 3, [16, 1025]), (128, 1, [500, 4100])])
def test_attention_f32_matches_oracle(pb, oracle, d, T_max, H, lens):
    """One and two query groups per wave, one to several query groups per unit, keys of a unit in
    one workgroup or split over up to 16, empty and ragged caches, tiles of one row."""
    rng = np.random.default_rng(T_max + d)
    shapes = [synth.random_tree(rng, T_max), synth.random_tree(rng, max(1, T_max - 1))]
    w = synth.Workload(86, "case", "f32", 2, H, d, T_max, 0, 0, 0, 1e-5)
    x = synth.make_attention_inputs(w, seq_lens=np.asarray(lens, np.int32), trees=shapes)
    out, sent = run_attention(pb, x)
    check_attention(oracle, x, out, sent)


# ------------------------------------------------------------------ bf16 scoring, few rows


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,H,T,L,room", [(1, 16, 115, 561, None), (1, 8, 100, 198, None), (1, 1, 16, 128, None), (1, 12, 48, 2129, None),
                                          (2, 16, 48, 1000, None), (5, 8, 43, 458, None), (1, 3, 20, 700, 2), (1, 3, 20, 700, 1), (1, 40, 33, 90, 3)])
def test_attention_f32_splits(pb, oracle, B, H, T, L, room, d):
    """How many workgroups share a unit's keys: one per compute unit and two, fewer and more than the plain rule says, and as many
    as a small workspace has room for."""
    rng = np.random.default_rng([B, H, T])
    lens = rng.integers(0, L + 1, B).astype(np.int32)
    lens[0] = L
    w = synth.Workload(83, "case", "f32", B, H, d, T, 0, 0, 0, 1e-5)
    x = synth.make_attention_inputs(w, seq_lens=lens, trees=[synth.random_tree(rng, T)] * B)
    if room is None:
        out, sent = run_attention(pb, x)
    else:
        dev = {k: to_dev(x[k]) for k in ("q", "k_cache", "v_cache", "k_tree", "v_tree", "seq_lens")}
        sent = sentinel_like(x["q"])
        out = to_dev(sent)
        ws = torch.empty(room * H * ((T + 31) // 32) * 32 * (d + 2) * 4, dtype=torch.uint8, device="cuda")
        tree = dev_tree(pb, x["n_nodes"], x["parent"], np.zeros_like(x["parent"]))
        with pytest.MonkeyPatch.context() as m:  # the call itself takes any workspace
            m.setattr(pb, "_marshal", None)
            m.setattr(pb, "workspace_bytes", lambda *a, **k: 0)
            pb.propd_tree_attention(tree, dev["q"], dev["k_cache"], dev["v_cache"], dev["k_tree"], dev["v_tree"], dev["seq_lens"],
                                    x["scale"], out=out, workspace=ws)
    check_attention(oracle, x, out, sent)


@pytest.mark.parametrize("T", [2, 9, 33, 34, 65, 66, 127, 128])
@pytest.mark.parametrize("Hd,V", [(64, 300), (192, 1003), (640, 257)])
def test_prune_bf16_few_rows_edges(pb, oracle, T, Hd, V):
    """One chain of T nodes has T - 1 score rows: both sides of every ring of the tile for few rows
    (32 and 128 rows), fewer K steps than ring stages and more, ragged column tiles."""
    w = synth.Workload(73, "case", "bf16", 1, 1, 128, T, Hd, V, 4, 1e-3)
    x = synth.make_prune_inputs(w, trees=[synth.chain_tree(T)])
    res, sents = run_prune(pb, x, [x["hidden_states"]])
    check_prune(oracle, x, res, [x["hidden_states"]], sents)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("trees", ["star", "mixed", "small", "rows", "wide"])
def test_prune_children_of_many_sequences(pb, oracle, dtype, trees):
    """The epilogue over whole rows takes the nodes of a tile's rows 512 at a time, from the slots or from the list of
    children: more nodes than that for a few rows (stars), sequences without score rows between others, slots of an odd
    number of nodes or nearly empty ones, and (fp32) rows of one sequence in two row tiles."""
    rng = np.random.default_rng(len(trees))
    shapes = {"star": [synth.star_tree(128)] * 9, "mixed": [synth.star_tree(101), synth.chain_tree(1), synth.chain_tree(30),
              synth.random_tree(rng, 101), synth.chain_tree(1), synth.star_tree(2), synth.chain_tree(40), synth.star_tree(77)],
              "small": [synth.random_tree(rng, int(n)) for n in rng.integers(1, 6, 40)],
              "wide": [synth.random_tree(rng, int(n)) for n in rng.integers(1, 4, 48)] + [synth.rank_product_tree(128, 4)],
              "rows": [synth.chain_tree(51), synth.star_tree(99), synth.chain_tree(61), synth.random_tree(rng, 99)]}[trees]
    T = max(len(t.parent) for t in shapes)
    w = synth.Workload(79, "case", dtype, len(shapes), 1, 128 if dtype == "bf16" else 64, T, 96, 300, 4, 1e-3 if dtype == "bf16" else 1e-5)
    x = synth.make_prune_inputs(w, trees=shapes)
    x["tau"] = 1e-3 if dtype == "bf16" else 1e-5  # the inputs' margin
    res, sents = run_prune(pb, x, [x["hidden_states"]])
    check_prune(oracle, x, res, [x["hidden_states"]], sents)


# ------------------------------------------------------------------ attention: merge of cut units


@pytest.mark.parametrize("B,H,T_max,L", [(1, 1, 40, 4000), (1, 3, 128, 2500), (2, 100, 20, 60), (3, 171, 33, 64),
                                         (9, 57, 16, 100), (1, 600, 33, 90), (2, 130, 100, 700)])
@pytest.mark.parametrize("d", [64, 128])
def test_attention_bf16_merge_of_cut_units(pb, oracle, B, H, T_max, L, d):
    """Units cut into many pieces and into few, records by unit (few units)
    and by workgroup (513 and 600 units: on the chip's 512 workgroups the one or the 88 units left
    after the whole ones are cut into a piece per workgroup), equal lengths and ragged ones."""
    rng = np.random.default_rng(B * 1000 + H)
    shapes = [synth.random_tree(rng, T_max)] + [synth.random_tree(rng, max(1, T_max - 3 * b)) for b in range(1, B)]
    lens = np.full(B, L, np.int32)
    if B == 9:
        lens = rng.integers(0, L + 1, B).astype(np.int32)
    w = synth.Workload(87, "case", "bf16", B, H, d, T_max, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=lens, trees=shapes)
    out, sent = run_attention(pb, x)
    check_attention(oracle, x, out, sent)


@pytest.mark.parametrize("B", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("H,ragged", [(1, True), (9, True), (9, False), (17, False)])
def test_attention_bf16_sequences_of_a_wave(pb, oracle, B, H, ragged):
    """Up to 64 sequences are scheduled from one lane each, more by a loop: ragged lengths with empty
    ones among them, and equal ones, of which the workgroups take one or more units whole."""
    rng = np.random.default_rng(B * 100 + H)
    lens = rng.integers(0, 150, B).astype(np.int32) if ragged else np.full(B, 70, np.int32)
    lens[::7] = 0 if ragged else 70
    trees = [synth.random_tree(rng, int(rng.integers(1, 41)) if ragged else 40) for _ in range(B)]
    w = synth.Workload(86, "case", "bf16", B, H, 64, 40, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=lens, trees=trees)
    out, sent = run_attention(pb, x)
    check_attention(oracle, x, out, sent)


# B, H, T_max, L, ragged lengths: no more units than workgroups (512 on 256 compute units) and more; ranges of one
# unit each (equal lengths, many pieces, one piece, few workgroups) and ranges that cross units; both sides of
# the line between two waves per 32 queries and one (64 queries; at d = 128 as many units as workgroups), and of
# the limits of the longest range by head size and tree size
RANGES = [(1, 1, 64, 3000, False), (1, 8, 59, 2500, False), (2, 16, 64, 700, True), (3, 5, 65, 700, True), (1, 40, 33, 90, False),
          (5, 12, 32, 592, False), (31, 8, 47, 300, True), (8, 64, 20, 60, False), (8, 64, 70, 60, True), (57, 9, 64, 64, True),
          (64, 8, 31, 40, True), (65, 7, 64, 70, True), (20, 30, 64, 100, True), (27, 20, 9, 1024, True), (27, 20, 9, 1023, True),
          (4, 3, 1, 33, True), (16, 1, 127, 136, False), (1, 300, 96, 200, False), (2, 33, 100, 0, False),
          (48, 8, 7, 900, False), (40, 8, 30, 700, True), (19, 8, 65, 980, False)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,H,T_max,L,ragged", RANGES)
def test_attention_bf16_ranges_of_one_unit(pb, oracle, B, H, T_max, L, ragged, d):
    """How a call's stages are cut into ranges, at the edges of the rule, with trees of 1 to T_max nodes."""
    rng = np.random.default_rng([B, H, T_max, L])
    lens = rng.integers(0, L + 1, B).astype(np.int32) if ragged else np.full(B, L, np.int32)
    lens[0] = L
    trees = [synth.rank_product_tree(int(n), 4) for n in (rng.integers(1, T_max + 1, B) if ragged else [T_max] * B)]
    trees[0] = synth.rank_product_tree(T_max, 4)
    w = synth.Workload(3, "ranges", "bf16", B, H, d, T_max, L, 4096, 10, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=lens, trees=trees)
    out, sent = run_attention(pb, x)
    check_attention(oracle, x, out, sent)


@pytest.mark.parametrize("d", [64, 128])
def test_attention_bf16_by_lengths_not_by_slots(pb, d):
    """600 units of up to 200 cached rows in slots of 200 and of 1100: the same kernel and ranges, so the same bits."""
    w = synth.Workload(5, "slots", "bf16", 20, 30, d, 40, 200, 4096, 10, 1e-3)
    lens = np.random.default_rng(d).integers(0, 201, 20).astype(np.int32)
    lens[3] = 200
    x = synth.make_attention_inputs(w, seq_lens=lens, trees=[synth.rank_product_tree(40, 4)] * 20)
    outs = [run_attention(pb, x)[0]]
    for name in ("k_cache", "v_cache"):
        x[name] = np.concatenate([x[name], np.zeros((20, 30, 1100 - x[name].shape[2], d), x[name].dtype)], 2)
    outs.append(run_attention(pb, x)[0])
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


@pytest.mark.parametrize("H", [127, 128, 129, 160])
@pytest.mark.parametrize("d,T_max,L", [(64, 40, 500), (128, 33, 480)])
def test_attention_bf16_merge_at_four_pieces(pb, oracle, H, d, T_max, L):
    """18 and 17 stages per unit: at most 128 units are merged by unit on the chip's 512 workgroups, more by
    workgroup."""
    w = synth.Workload(88, "case", "bf16", 1, H, d, T_max, 0, 0, 0, 1e-3)
    x = synth.make_attention_inputs(w, seq_lens=np.array([L], np.int32), trees=[synth.rank_product_tree(T_max, 4)])
    out, sent = run_attention(pb, x)
    check_attention(oracle, x, out, sent)


# ------------------------------------------------------------------ bf16 scoring, many rows


@pytest.mark.parametrize("Hd", [32, 96, 160, 288])
def test_prob_prune_several_tiles_per_workgroup(pb, oracle, Hd):
    """The criterion whose epilogue passes nothing through LDS, with K loops of one step to five: 396 score
    rows are 2 x 125 tiles, one for each workgroup."""
    B, T_max, V = 9, 128, 32000
    w = synth.Workload(74, "case", "bf16", B, 1, 128, T_max, Hd, V, 8, 1e-3)
    x = synth.make_prune_inputs(w, trees=[synth.rank_product_tree(128, 5)] * B)
    logm, _, _ = prob_reference(oracle, x, threshold=0.5)
    thr = float(np.float32(threshold_in_a_gap(logm, x["n_nodes"], 1e-3, 0.6)))
    _, _, ref = prob_reference(oracle, x, threshold=thr)
    res, sents = run_prob(pb, x, [x["hidden_states"]], threshold=thr)
    check_prob(pb, oracle, x, res, ref, logm, [x["hidden_states"]], sents)


def whole_number_scores(pb, parent, token, Hd, V, seed):
    """Hidden states, head weight and what every rank and log-probability must be: operands of -1, 0 and 1
    (weights in eighths), whose sums fp32 holds exactly in any order, scored by a plain product."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    draw = lambda *s: torch.randint(-1, 2, s, device="cuda", generator=gen, dtype=torch.int8).to(torch.bfloat16)
    B, T = parent.shape
    hid, head = draw(B, T, Hd), draw(V, Hd) / 8
    rows, which = np.unique((np.arange(B)[:, None] * T + parent)[:, 1:].reshape(-1), return_inverse=True)
    flat, tok = hid.view(-1, Hd)[torch.from_numpy(rows).cuda()].float(), torch.from_numpy(token[:, 1:].reshape(-1).astype(np.int64)).cuda()
    which = torch.from_numpy(which.reshape(-1)).cuda()
    chunks = [(v, flat @ head[v:v + 8192].float().T) for v in range(0, V, 8192)]
    z = torch.cat([c for _, c in chunks], 1)
    own = z[which, tok]
    rank = torch.zeros_like(tok)
    for v, c in chunks:
        c, ids = c[which], torch.arange(v, v + c.shape[1], device="cuda")
        rank += ((c > own[:, None]) | ((c == own[:, None]) & (ids[None] < tok[:, None]))).sum(1)
    logq = own.double() - torch.logsumexp(z.double(), 1)[which]
    shape = (B, T - 1)
    return hid, head, to_host(rank).reshape(shape), to_host(logq).reshape(shape)


@pytest.mark.parametrize("Hd", [32, 352, 384])
@pytest.mark.parametrize("B", [1, 3, 4, 5, 11, 6, 14, 8])
def test_prune_bf16_several_tiles_per_workgroup(pb, B, Hd):
    """More column tiles than workgroups, for the tile of few rows and for every shape of many (32 * MI rows
    with MI = 5, 6, 7, 8, 9, 10, 11 on 256 compute units), both criteria: a workgroup's next tile starts in
    memory that its last one has used.  One step, and enough of them that every ring wraps, with a half
    step at the end and without."""
    groups = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    T, V = 128, 256 * (groups + 70) + 3
    assert (V + 255) // 256 > (groups + 7) // 8 * 8
    shape = synth.rank_product_tree(T, 5)  # 44 of its nodes have children
    n, parent, _ = synth.pad_trees([shape] * B, T)
    token = np.random.default_rng(B).integers(0, V, (B, T)).astype(np.int32)
    hid, head, rank, logq = whole_number_scores(pb, parent, token, Hd, V, 100 * B + Hd)
    tree = dev_tree(pb, n, parent, token)
    got = to_host(pb.propd_early_prune(tree, hid, head, 8, want_rank=True).rank)
    assert (got[:, 1:] == rank).all()
    # a row's log-sum-exp is merged from at most V / 128 partials, one fp32 rounding each at worst, and a path
    # has at most five nodes
    lm = to_host(pb.propd_early_prune_prob(tree, hid, head, threshold=1e-30, want_log_marginal=True).log_marginal)
    want = np.zeros((B, T))
    for i in range(1, T):
        want[:, i] = want[np.arange(B), parent[:, i]] + logq[:, i - 1]
    assert np.abs(lm - want).max() <= 5 * (V / 128) * 2.0 ** -24 + 5 * 2.0 ** -24 * np.abs(want).max()


@pytest.mark.parametrize("B,T,V", [(1, 128, 32000), (2, 66, 32000), (2, 128, 4001), (3, 87, 32000), (3, 128, 32000),
                                   (4, 112, 32000), (4, 128, 32000), (5, 116, 32000), (5, 128, 32000), (6, 118, 32000),
                                   (7, 120, 32001), (7, 120, 700)])
def test_prune_bf16_every_tile_shape(pb, oracle, B, T, V):
    """B chains of T nodes have B * (T - 1) score rows.  Against 32000 entries on 256 compute units the
    counts 127, 130, 254, 261, 381, 444, 508, 575, 635, 702 and 833 take every tile there is, with
    its last rows missing; both criteria, rows of an odd number of 32s."""
    w = synth.Workload(76, "case", "bf16", B, 1, 128, T, 96, V, 6, 1e-3)
    x = synth.make_prune_inputs(w, trees=[synth.chain_tree(T)] * B, p_pass=0.8)
    res, sents = run_prune(pb, x, [x["hidden_states"]])
    check_prune(oracle, x, res, [x["hidden_states"]], sents)
    logm, _, _ = prob_reference(oracle, x, threshold=0.5)
    thr = float(np.float32(threshold_in_a_gap(logm, x["n_nodes"], 1e-3, 0.95)))
    _, _, ref = prob_reference(oracle, x, threshold=thr)
    res, sents = run_prob(pb, x, [x["hidden_states"]], threshold=thr)
    check_prob(pb, oracle, x, res, ref, logm, [x["hidden_states"]], sents)


@pytest.mark.parametrize("Hd", [32, 64, 160, 192])
@pytest.mark.parametrize("B,T", [(3, 87), (6, 118)])
def test_prune_bf16_tall_tiles_short_rows(pb, oracle, Hd, B, T):
    """One half step, one step, a half step behind two, three steps, on a tile that addresses rows by
    pointers (258 score rows) and on one that does by offsets (702); the last column tile not full."""
    w = synth.Workload(78, "case", "bf16", B, 1, 128, T, Hd, 31990, 6, 1e-3)
    x = synth.make_prune_inputs(w, trees=[synth.chain_tree(T)] * B, p_pass=0.8)
    res, sents = run_prune(pb, x, [x["hidden_states"]])
    check_prune(oracle, x, res, [x["hidden_states"]], sents)


@pytest.mark.parametrize("B,T,Hd,V", [(2, 65, 96, 1000), (2, 66, 1152, 1000), (2, 66, 1120, 1000), (2, 66, 1184, 32768),
                                      (2, 66, 1184, 32769), (2, 81, 3072, 1000), (2, 81, 3104, 1000), (2, 81, 3040, 1000),
                                      (2, 97, 5120, 1000), (2, 97, 5152, 300), (2, 97, 5088, 1000), (2, 98, 5280, 1000)])
def test_prune_bf16_few_rows_rule(pb, oracle, B, T, Hd, V):
    """128 score rows, and 130, 160 and 192 of at least 1152, 3072 and 5120, take the tile of few rows in one
    round (32768 entries on 256 compute units); shorter rows, 194 of them or 32769 entries take another. Both
    criteria, rows of an even and of an odd number of 32s."""
    w = synth.Workload(79, "case", "bf16", B, 1, 128, T, Hd, V, 6, 1e-3)
    x = synth.make_prune_inputs(w, trees=[synth.chain_tree(T)] * B, p_pass=0.8)
    res, sents = run_prune(pb, x, [x["hidden_states"]])
    check_prune(oracle, x, res, [x["hidden_states"]], sents)
    logm, _, _ = prob_reference(oracle, x, threshold=0.5)
    thr = float(np.float32(threshold_in_a_gap(logm, x["n_nodes"], 1e-3, 0.95)))
    _, _, ref = prob_reference(oracle, x, threshold=thr)
    res, sents = run_prob(pb, x, [x["hidden_states"]], threshold=thr)
    check_prob(pb, oracle, x, res, ref, logm, [x["hidden_states"]], sents)


@pytest.mark.parametrize("B,T,V", [(2, 66, 8192), (2, 66, 16001), (2, 128, 8192), (2, 128, 33001), (2, 89, 40000), (2, 65, 70000)])
def test_prune_bf16_few_rows_or_tiles(pb, oracle, B, T, V):
    """More score rows than the tile of few rows takes, in little and in much vocabulary: 130, 254, 176
    and 128 rows, both criteria."""
    w = synth.Workload(77, "case", "bf16", B, 1, 128, T, 64, V, 6, 1e-3)
    x = synth.make_prune_inputs(w, trees=[synth.chain_tree(T)] * B, p_pass=0.8)
    res, sents = run_prune(pb, x, [x["hidden_states"]])
    check_prune(oracle, x, res, [x["hidden_states"]], sents)
    logm, _, _ = prob_reference(oracle, x, threshold=0.5)
    thr = float(np.float32(threshold_in_a_gap(logm, x["n_nodes"], 1e-3, 0.95)))
    _, _, ref = prob_reference(oracle, x, threshold=thr)
    res, sents = run_prob(pb, x, [x["hidden_states"]], threshold=thr)
    check_prob(pb, oracle, x, res, ref, logm, [x["hidden_states"]], sents)


PLAN_CHILD = """
import sys
sys.path[:0] = {path!r}
from oracle import oracle
from paper_2402_13485_amd import binding, synth
from test_gpu_parity import check_prune, run_prune
binding.load_library()
w = synth.Workload(95, "case", "bf16", 3, 1, 128, 128, 64, 700, 6, 1e-3)
x = synth.make_prune_inputs(w, trees=[synth.chain_tree(128)] * 3)
res, sents = run_prune(binding, x, [x["hidden_states"]])
check_prune(oracle, x, res, [x["hidden_states"]], sents)
print("same as the oracle")
"""


@pytest.mark.parametrize("value", ["1", "2", "7"])
def test_prune_with_the_tile_shape_given(pb, oracle, value):
    """PROPD_HEAD_PLAN takes the choice of the tile shape away: 381 score rows are scored
    whatever it holds.  (It is read once per process, hence the child.)"""
    child = PLAN_CHILD.format(path=[os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                                    os.path.dirname(os.path.abspath(__file__))])
    done = subprocess.run([sys.executable, "-c", child], env=dict(os.environ, PROPD_HEAD_PLAN=value), timeout=100,
                          capture_output=True, text=True)
    assert done.returncode == 0 and "same as the oracle" in done.stdout, done.stderr[-2000:]


@pytest.mark.parametrize("C", [8, 24, 264, 2048, 2056, 5])
@pytest.mark.parametrize("T,outer", [(1, 1), (33, 3), (128, 2)])
def test_prune_payload_row_sizes(pb, C, T, outer):
    """Payload rows of 1, 3, 33, 256 and 257 pieces of 16 bytes, and of 10 bytes: survivors in their
    order, everything behind them as it was."""
    B = 3
    w = synth.Workload(93, "case", "f32", B, 1, 64, T, 32, 2000, 4, 1e-5)
    x = synth.make_prune_inputs(w, trees=[synth.chain_tree(T), synth.star_tree(T), synth.chain_tree(max(1, T // 2))])
    tree = dev_tree(pb, x["n_nodes"], x["parent"], x["token"])
    src = torch.randint(0, 30000, (B, outer, T, C), device="cuda").to(torch.int16)
    res = pb.propd_early_prune(tree, to_dev(x["hidden_states"]), to_dev(x["head_weight"]), 40, payloads=[src],
                               payload_out=[torch.full_like(src, -5)])
    origin, got, want = to_host(res.orig_index), to_host(res.payloads[0]), np.full(src.shape, -5, np.int16)
    for b, o in enumerate(origin):
        o = o[o >= 0]
        want[b, :, :len(o)] = to_host(src)[b][:, o]
    assert (got == want).all()


FAR_ROWS_CHILD = """
import sys
sys.path[:0] = {path!r}
import numpy as np
import torch
from paper_2402_13485_amd import binding as pb
from paper_2402_13485_amd import synth
B, T, Hd, V = 128, 128, 1 << 17, 300
gen = torch.Generator(device="cuda")
gen.manual_seed(5)
small = lambda *shape: torch.randint(-1, 2, shape, device="cuda", generator=gen, dtype=torch.int8).to(torch.bfloat16)
n, parent, _ = synth.pad_trees([synth.chain_tree(T if b in (0, 64, 125, 127) else 1) for b in range(B)], T)
token = np.random.default_rng(5).integers(0, V, (B, T)).astype(np.int32)
token[np.arange(T)[None] >= n[:, None]] = -1
hid = torch.zeros(B, T, Hd, device="cuda", dtype=torch.bfloat16)
head = small(V, Hd)
nn, par, tok = (torch.from_numpy(x.astype(np.int32)).cuda() for x in (n, parent, token))
depth, anc = pb.propd_tree_mask(nn, par)
for b in (0, 64, 125, 127):
    hid[b] = small(T, Hd)
rank = pb.propd_early_prune(pb.Tree(nn, par, tok, depth, anc), hid, head, 5, want_rank=True).rank.cpu().numpy()
for b in (0, 64, 125, 127):
    z = (hid[b].float().cpu() @ head.float().cpu().T).numpy()  # whole numbers: exact in any order
    for i in range(1, T):
        row, t = z[i - 1], token[b, i]
        assert rank[b, i] == (row > row[t]).sum() + (row[:t] == row[t]).sum(), (b, i)
print("ranks as counted")
"""


@pytest.mark.parametrize("B,T", [(1, 5), (2, 128), (3, 17), (64, 9), (65, 1), (66, 2), (131, 3), (255, 6), (256, 6), (257, 6), (513, 4),
                                 (1100, 3)])
@pytest.mark.parametrize("crit", ["topk", "prob"])
def test_prune_sequences_of_a_batch(pb, oracle, B, T, crit):
    """One workgroup per sequence and many: decisions, payload rows and the prefix sum of the survivor counts, which the
    last sequence to be decided writes (sequences arrive on one line up to 64, then on as many as there is room for);
    twice with one workspace, whose counters the second call finds used."""
    rng = np.random.default_rng([B, T])
    trees = [synth.random_tree(rng, int(n)) for n in rng.integers(1, T + 1, B)]
    trees[0] = synth.random_tree(rng, T)
    n_nodes, parent, _ = synth.pad_trees(trees, T)
    token = rng.integers(0, 300, (B, T)).astype(np.int32)
    tree = dev_tree(pb, n_nodes, parent, token)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B)
    hid = torch.randn(B, T, 32, device="cuda", generator=gen).to(torch.bfloat16)
    w = torch.randn(300, 32, device="cuda", generator=gen).to(torch.bfloat16)
    pay = [hid, torch.randn(B, 3, T, 24, device="cuda", generator=gen), torch.randint(0, 255, (B, T, 7), device="cuda", generator=gen).to(torch.uint8)]
    ws = torch.empty(pb.workspace_bytes(pb.WS_EARLY_PRUNE, B, T, hidden=32, vocab=300), dtype=torch.uint8, device="cuda")
    ws.fill_(0xa5)
    for again in range(2):
        dst = [torch.full_like(x, 3) for x in pay]
        if crit == "topk":
            r = pb.propd_early_prune(tree, hid, w, 150, payloads=pay, payload_out=dst, want_rank=True, workspace=ws)
            fail_rank = to_host(r.rank)
        else:
            r = pb.propd_early_prune_prob(tree, hid, w, keep_count=max(1, T // 2), payloads=pay, payload_out=dst,
                                          want_log_marginal=True, workspace=ws)
            lm = to_host(r.log_marginal)
            fail_rank = np.zeros((B, T), np.int32)
            for b in range(B):  # the kernel's own marginals, ranked: equal ones by node index
                n = int(n_nodes[b])
                for i in range(1, n):
                    fail_rank[b, i] = 500 if sum(lm[b, j] > lm[b, i] or (lm[b, j] == lm[b, i] and j < i) for j in range(n)) >= max(1, T // 2) else 0
        ref = oracle.prune_compact(n_nodes, parent, token, fail_rank, 150)
        for name in ("new_index", "orig_index", "n_kept", "cu_nodes"):
            assert (to_host(getattr(r, name)) == ref[name]).all(), (name, again)
        for name in ("parent", "token", "depth"):
            assert (to_host(getattr(r.tree, name)) == ref[name]).all(), (name, again)
        assert (to_host(r.tree.anc).view(np.uint64) == ref["anc"]).all()
        orig = torch.from_numpy(ref["orig_index"]).cuda().long()
        bs, js = (orig >= 0).nonzero(as_tuple=True)
        for x, y in zip(pay, dst):
            want = torch.full_like(x, 3)
            if x.dim() == 3:
                want[bs, js] = x[bs, orig[bs, js]]
            else:
                want[bs, :, js] = x[bs, :, orig[bs, js]]
            assert torch.equal(want, y)


def test_prune_payload_of_more_than_2_31_pieces(pb):
    """Rows of an odd number of bytes, one byte per piece, with nothing pruned (top_k covers the vocabulary)."""
    T, C = 128, (1 << 24) + 1
    n_nodes, parent, _ = synth.pad_trees([synth.chain_tree(T)], T)
    tree = dev_tree(pb, n_nodes, parent, np.zeros((1, T), np.int32))
    src = torch.arange(T * C, device="cuda", dtype=torch.int64).mul_(2654435761).bitwise_right_shift_(13).to(torch.uint8).view(1, T, C)
    dst = torch.zeros_like(src)
    hid, w = torch.zeros(1, T, 32, device="cuda"), torch.zeros(4, 32, device="cuda")
    r = pb.propd_early_prune(tree, hid, w, 4, payloads=[src], payload_out=[dst])
    assert to_host(r.n_kept).tolist() == [T] and to_host(r.cu_nodes).tolist() == [0, T]
    assert torch.equal(src, dst)


def test_prune_rows_further_apart_than_32_bits(pb):
    """Hidden states of 4 GiB: the tallest tiles, which address rows by 32-bit offsets, are asked for
    and give way to the tallest that does not; 508 score rows, the last ones beyond 4 GB."""
    child = FAR_ROWS_CHILD.format(path=[os.path.dirname(os.path.dirname(os.path.abspath(__file__)))])
    done = subprocess.run([sys.executable, "-c", child], env=dict(os.environ, PROPD_HEAD_PLAN="2"), timeout=100,
                          capture_output=True, text=True)
    assert done.returncode == 0 and "ranks as counted" in done.stdout, done.stderr[-2000:]


@pytest.mark.parametrize("B,T,Hd,V", [(3, 87, 8192, 262208), (4, 89, 16384, 151936), (1, 128, 8192, 262208)])
def test_prune_head_weight_beyond_32_bits(pb, B, T, Hd, V):
    """Head weights of 4 to 5 GiB: 258, 352 and 127 score rows take tiles of 288 and 352 rows, which address
    rows by 32-bit offsets, and the tile of few rows.  In the tile whose distance to the end of the
    weights lies just above 4 GiB (entries 0 to 255 of 262208, 20736 to 20991 of 151936) as in any other
    every entry counts with its own score; the entries there are the only ones above zero."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    hid = torch.randint(0, 3, (B, T, Hd), device="cuda", generator=gen, dtype=torch.int8).to(torch.bfloat16)
    head = torch.empty(V, Hd, device="cuda", dtype=torch.bfloat16)
    for v in range(0, V, 16384):  # -1 and 0: scores of at most 0, whole numbers that fp32 sums hold exactly
        head[v:v + 16384] = torch.randint(-1, 1, (min(V - v, 16384), Hd), device="cuda", generator=gen, dtype=torch.int8)
    first = V - 1 - ((1 << 32) // (2 * Hd))  # a distance of 4 GiB ends here
    for v in range(max(0, first - 256), first + 1):
        head[v] = -head[v]
    n, parent, _ = synth.pad_trees([synth.chain_tree(T)] * B, T)
    token = np.random.default_rng(V).integers(0, V, (B, T)).astype(np.int32)
    token[:, 1::2] = np.random.default_rng(T).integers(max(0, first - 256), first + 1, token[:, 1::2].shape)
    tree = dev_tree(pb, n, parent, token)
    rank = to_host(pb.propd_early_prune(tree, hid, head, 5, want_rank=True).rank)
    rows = hid[:, :-1].reshape(-1, Hd).double().cpu()  # node i - 1 is the parent of node i
    child = torch.from_numpy(token[:, 1:].reshape(-1).astype(np.int64))
    own = (rows * head[child.cuda()].double().cpu()).sum(1, keepdim=True).cuda()
    ahead = torch.zeros(len(child), dtype=torch.int64, device="cuda")
    for v in range(0, V, 16384):
        z = rows.float().cuda() @ head[v:v + 16384].float().T
        before = torch.arange(v, v + z.shape[1], device="cuda")[None] < child.cuda()[:, None]
        ahead += ((z.double() > own) | ((z.double() == own) & before)).sum(1)
    assert (rank[:, 1:].reshape(-1) == to_host(ahead)).all()


def test_prune_outputs_are_aligned(pb):
    """Every output is a tensor that any call takes: bases on 16 bytes, also for one sequence and
    for an odd number of nodes."""
    for B, T in ((1, 33), (3, 5), (1, 1), (2, 64), (5, 7)):
        shapes = [synth.chain_tree(T)] * B
        w = synth.Workload(94, "case", "f32", B, 1, 64, T, 32, 100, 4, 1e-5)
        x = synth.make_prune_inputs(w, trees=shapes)
        tree = dev_tree(pb, x["n_nodes"], x["parent"], x["token"])
        res = pb.propd_early_prune(tree, to_dev(x["hidden_states"]), to_dev(x["head_weight"]), 4, want_rank=True)
        outs = [res.keep_bits, res.new_index, res.orig_index, res.n_kept, res.cu_nodes, res.rank, res.tree.n_nodes,
                res.tree.parent, res.tree.token, res.tree.depth, res.tree.anc]
        assert all(t.is_contiguous() and t.data_ptr() % 16 == 0 for t in outs), (B, T)
        assert all(tuple(t.shape) == (B, T) for t in (res.new_index, res.rank, res.tree.parent))
        assert (to_host(res.n_kept) == to_host(res.tree.n_nodes)).all()
