"""The calls a decoding loop makes of this library, as cases that can be timed and compared.

One case is one call (or one whole verification step) at one set of sizes.  Sizes come from
the benchmark workloads in ``synth.WORKLOADS`` (7B/13B-class decoders, batch 1..32, trees of
16..128 nodes, up to 8192 cached tokens) and from the types and head sizes the C boundary
takes besides them (fp32, head size 64).

The kinds:
  attention   propd_tree_attention, one layer of one step
  prune       propd_early_prune with the rows that go on past the pruning point as payloads
  prune_prob  propd_early_prune_prob, threshold criterion
  accept      propd_accept_path
  step        mask, attention on the whole tree, pruning, attention on the compacted tree,
              acceptance and commit: what one iteration of the loop asks of the library
Inputs are N(0,1) (head weights N(0, 0.02^2)); about half of the children pass the top-k test,
and every decision keeps a margin to its boundary that rounding cannot bridge.
"""
import math
import types

import numpy as np
import torch

from paper_2402_13485_amd import binding as pb
from paper_2402_13485_amd import synth

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
PATH_STRIDE = 8        # deepest tree here: 6 nodes on a path
KEEP_SHARE = 0.3       # prune_prob: share of the nodes that the threshold keeps


def listed():
    return [
        # the smallest step there is: fp32, one head, 128 cached tokens; launches and host latency
        dict(name="step_f32_tiny", kind="step", dtype="f32", B=1, H=1, d=64, T=16, L=128, ragged=False,
             hidden=64, vocab=256, top_k=4),
        # one layer of a single-user chat: latency
        dict(name="attn_b1", kind="attention", dtype="bf16", B=1, H=32, d=128, T=64, L=1024, ragged=False),
        # a whole iteration of a small server: mixed lengths, pruning, commit
        dict(name="step_b4", kind="step", dtype="bf16", B=4, H=32, d=128, T=64, L=2048, ragged=True,
             hidden=4096, vocab=32000, top_k=10),
        # one layer of a large batch of long sequences: the K/V stream
        dict(name="attn_b16", kind="attention", dtype="bf16", B=16, H=40, d=128, T=128, L=4096, ragged=False),
        # one layer of continuous batching: lengths 512..8192, trees 16..128
        dict(name="attn_ragged_b32", kind="attention", dtype="bf16", B=32, H=32, d=128, T=128, L=8192, ragged=True),
        # the smaller head size
        dict(name="attn_d64", kind="attention", dtype="bf16", B=8, H=16, d=64, T=64, L=2048, ragged=False),
        # fp32 tensors: a model kept in full precision, or a check of a 16-bit one
        dict(name="attn_f32", kind="attention", dtype="f32", B=2, H=16, d=128, T=48, L=1024, ragged=True),
        # pruning for one user: a stream of the head weight, few rows
        dict(name="prune_b1", kind="prune", dtype="bf16", B=1, H=32, d=128, T=64, L=0, ragged=False,
             hidden=4096, vocab=32000, top_k=10),
        # pruning of a large batch: a large contraction, and payload rows of every kind
        dict(name="prune_b16", kind="prune", dtype="bf16", B=16, H=40, d=128, T=128, L=0, ragged=False,
             hidden=5120, vocab=32000, top_k=8),
        # the probability criterion on trees of mixed sizes
        dict(name="prune_prob_b32", kind="prune_prob", dtype="bf16", B=32, H=32, d=128, T=128, L=0, ragged=True,
             hidden=4096, vocab=32000, top_k=10),
        # pruning with fp32 tensors, a small model
        dict(name="prune_f32", kind="prune", dtype="f32", B=2, H=16, d=64, T=32, L=0, ragged=False,
             hidden=1024, vocab=32000, top_k=8),
        # acceptance for a large batch: the final logits read once
        dict(name="accept_b16", kind="accept", dtype="bf16", B=16, H=1, d=128, T=128, L=0, ragged=False,
             vocab=32000),
    ]


def draw(rng):
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.choice(["attention", "attention", "attention", "prune", "prune", "prune_prob", "accept", "step"])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    c = dict(kind=kind, dtype=dtype, B=log(1, 32), H=rng.choice([8, 12, 16, 32, 40]),
             d=64 if rng.random() < 0.25 else 128, T=rng.randint(8, 128), L=0, ragged=rng.random() < 0.5)
    if kind in ("attention", "step"):
        c["L"] = log(100, 8192)
        # no more K/V than the largest listed case; where no matrix cores are used, no more work
        # than the listed cases of those kinds
        if dtype == "bf16" and c["d"] == 128:
            room = 16 * 40 * 4096
        elif dtype == "bf16":
            room = 8 * 16 * 2048 * 64 // c["T"]
        else:
            room = 2 * 16 * 1024 * 48 // c["T"]
        while c["B"] * c["H"] * c["L"] > room:
            key = "B" if c["B"] > 1 else ("L" if c["L"] > 300 else "H")
            c[key] = max(1, c[key] // 2)
    if kind != "attention":
        c["vocab"] = rng.choice([8192, 16001, 32000, 32001]) if dtype == "bf16" else log(250, 32000)
    if kind in ("prune", "prune_prob", "step"):
        c["top_k"] = rng.randint(4, 16)
        if dtype == "bf16":
            c["hidden"] = 32 * rng.randint(32, 160)
        else:
            c["hidden"], c["B"], c["T"] = log(60, 1024), min(c["B"], 2), min(c["T"], 32)
    return c


# ---------------------------------------------------------------------------------------------
# sizes of a case that do not depend on the seed
# ---------------------------------------------------------------------------------------------


def _shape(c):
    """Sequence lengths, tree sizes and parents of a case (fixed by its sizes)."""
    rng = np.random.default_rng([c["B"], c["T"], c["L"], 7])
    if c["ragged"]:
        lens = np.rint(np.exp(rng.uniform(math.log(max(1, c["L"] / 16)), math.log(max(1, c["L"])), c["B"])))
        nodes = rng.choice(sorted({max(2, c["T"] * s // 8) for s in (1, 2, 4, 6, 8)}), c["B"])
        lens[0], nodes[0] = c["L"], c["T"]  # the longest one sets the slot sizes
    else:
        lens, nodes = np.full(c["B"], c["L"]), np.full(c["B"], c["T"])
    depth = 3 if c["T"] <= 16 else 4 if c["T"] <= 64 else 5
    cache = {int(n): synth.rank_product_tree(int(n), depth) for n in set(nodes.tolist())}
    trees = [cache[int(n)] for n in nodes]
    n_nodes, parent, dep = synth.pad_trees(trees, c["T"])
    return lens.astype(np.int32), n_nodes, parent, dep


def _children(parent_row, n):
    kids = {}
    for i in range(1, n):
        kids.setdefault(int(parent_row[i]), []).append(i)
    return kids


def work(c):
    lens, n_nodes, parent, dep = _shape(c)
    es = 2 if c["dtype"] == "bf16" else 4
    row = c["H"] * c["d"] * es
    by = fl = 0.0

    def attention(nodes):
        kv = float((lens.astype(np.float64) * row * 2).sum())
        side = float(nodes.sum()) * row * 4
        fl = float((nodes * (lens + nodes)).sum()) * c["H"] * c["d"] * 4.0
        return kv + side, fl

    # expected survivors: every node of a path passes with probability one half
    valid = np.arange(c["T"])[None] < n_nodes[:, None]
    kept = (0.5 ** dep * valid).sum(1)
    if c["kind"] == "prune_prob":
        kept = np.maximum(1, KEEP_SHARE * n_nodes)
    if c["kind"] in ("attention", "step"):
        b, f = attention(n_nodes.astype(np.float64))
        by, fl = by + b, fl + f
    if c["kind"] in ("prune", "prune_prob", "step"):
        rows = sum(len(_children(parent[b], int(n))) for b, n in enumerate(n_nodes))
        payload_rows = c["hidden"] * es + (0 if c["kind"] == "prune_prob" else 3 * row)
        by += (rows + c["vocab"]) * c["hidden"] * es + float(kept.sum()) * 2 * payload_rows
        fl += 2.0 * rows * c["hidden"] * c["vocab"]
    if c["kind"] == "step":
        b, f = attention(kept)
        by, fl = by + b, fl + f
    if c["kind"] in ("accept", "step"):
        rows = float(kept.sum() if c["kind"] == "step" else n_nodes.sum())
        by, fl = by + rows * c["vocab"] * es, fl + rows * c["vocab"]
    return {"bytes": by, "flops": fl}


def tolerance(c):
    if c["kind"] in ("accept", "prune"):
        return "exact"  # whole numbers and copied rows
    if c["dtype"] == "f32" or c["kind"] == "prune_prob":
        return {"rel": 1e-5, "max": 1e-4}  # fp32 sums (prune_prob: of up to five fp32 logarithms)
    # bf16 weights inside and a bf16 result: 2.3e-3 away from 64 bits, so two may differ by that and more
    return {"rel": 1e-2, "max": 4e-2}


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------


def _compact(n_nodes, parent, token, fail):
    """Survivors (old indices), and the parents and tokens of the compacted trees, per sequence."""
    out = []
    for b, n in enumerate(n_nodes):
        keep, new = [], {}
        for i in range(int(n)):
            if i == 0 or (int(parent[b, i]) in new and not fail[b, i]):
                new[i] = len(keep)
                keep.append(i)
        out.append((keep, [-1] + [new[int(parent[b, i])] for i in keep[1:]], [int(token[b, i]) for i in keep]))
    return out


def _place_tokens(rng, c, z, rows, n_nodes, parent):
    """A token id for every node: about half of the children inside the top_k of their parent's
    scores z[row], the others below, all at least tau away from the boundary."""
    tau = 1e-3 if c["dtype"] == "bf16" else 1e-4
    k = c["top_k"]
    vals, ids = (t.cpu().numpy() for t in z.topk(min(c["vocab"], 64 * k), dim=1))
    token = rng.integers(0, c["vocab"], (len(n_nodes), c["T"])).astype(np.int32)
    fail = np.zeros(token.shape, bool)
    for r, (b, p, kids) in enumerate(rows):
        ok = rng.permutation(np.flatnonzero(vals[r, :k] - vals[r, k] >= tau)).tolist()
        bad = rng.permutation(np.flatnonzero(vals[r, k - 1] - vals[r] >= tau)).tolist()
        for i in kids:
            good = bool(rng.random() < 0.5) and len(ok) > 0
            token[b, i] = ids[r, (ok if good else bad).pop()]
            fail[b, i] = not good
    token[np.arange(c["T"])[None] >= n_nodes[:, None]] = -1
    return token, fail


def _plant_chain(rng, logits, trees):
    """Raises logits so that a chain of geometric length is accepted in every sequence;
    ``trees`` holds (parents, tokens) of the tree that the logits belong to."""
    bs, ns, vs = [], [], []
    for b, (par, tok) in enumerate(trees):
        kids = _children(par, len(par))
        node, steps = 0, int(rng.geometric(0.45)) - 1
        while steps > 0 and kids.get(node):
            nxt = int(rng.choice(kids[node]))
            bs, ns, vs = bs + [b], ns + [node], vs + [tok[nxt]]
            node, steps = nxt, steps - 1
        taken = {tok[i] for i in kids.get(node, [])}
        free = next(v for v in rng.integers(0, logits.shape[2], 1000).tolist() if v not in taken)
        bs, ns, vs = bs + [b], ns + [node], vs + [free]
    bs, ns, vs = (torch.tensor(x, device="cuda") for x in (bs, ns, vs))
    logits[bs, ns, vs] = logits[bs, ns].amax(-1) + 1


def _log_marginals(z, rows, token, shape):
    """log of the product of the tokens' probabilities along every root path (scores z)."""
    logq = z.log_softmax(1)
    r = torch.tensor([i for i, (_, _, kids) in enumerate(rows) for _ in kids], device="cuda")
    t = torch.tensor([int(token[b, i]) for b, _, kids in rows for i in kids], device="cuda")
    q = iter(logq[r, t].cpu().numpy().tolist())
    lm = np.zeros(shape)
    for b, p, kids in rows:  # parents come before their children
        for i in kids:
            lm[b, i] = lm[b, p] + next(q)
    return lm


def _score_rows(c, n_nodes, parent):
    return [(b, p, kids) for b, n in enumerate(n_nodes) for p, kids in sorted(_children(parent[b], int(n)).items())]


def _scores(s, dtype):
    at = torch.tensor([b * s.c["T"] + p for b, p, _ in s.rows], device="cuda")
    return s.hid.reshape(-1, s.c["hidden"])[at].to(dtype) @ s.head.to(dtype).T.contiguous()


def prepare(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    dt = DTYPES[c["dtype"]]
    normal = lambda *shape: torch.randn(shape, device="cuda", dtype=dt, generator=gen)
    lens, n_nodes, parent, _ = _shape(c)
    B, H, T, d = c["B"], c["H"], c["T"], c["d"]
    s = types.SimpleNamespace(c=c, kind=c["kind"], lens=lens, n_nodes=n_nodes, parent=parent, scale=1.0 / math.sqrt(d))
    s.nn, s.par = torch.from_numpy(n_nodes).cuda(), torch.from_numpy(parent).cuda()
    s.depth, s.anc = pb.propd_tree_mask(s.nn, s.par)
    token = None
    attends, prunes = c["kind"] in ("attention", "step"), c["kind"] in ("prune", "prune_prob", "step")
    if c["kind"] in ("attention", "step", "prune"):
        s.q, s.kt, s.vt = normal(B, H, T, d), normal(B, H, T, d), normal(B, H, T, d)
    if attends:
        # a step also appends to the cache, so it has room for that
        s.L_max = c["L"] + (PATH_STRIDE if c["kind"] == "step" else 0)
        s.kc, s.vc = normal(B, H, s.L_max, d), normal(B, H, s.L_max, d)
        s.seq = torch.from_numpy(lens).cuda()
        s.out = torch.zeros_like(s.q)
        s.ws_att = torch.empty(max(256, pb.workspace_bytes(pb.WS_TREE_ATTENTION, B, T, H, d, s.L_max)),
                               dtype=torch.uint8, device="cuda")
    if prunes:
        s.hid, s.head = normal(B, T, c["hidden"]), normal(c["vocab"], c["hidden"]) * 0.02
        s.rows = _score_rows(c, n_nodes, parent)
        z = _scores(s, torch.float32)
        token, fail = _place_tokens(rng, c, z, s.rows, n_nodes, parent)
        if c["kind"] == "prune_prob":
            lm = _log_marginals(z.double(), s.rows, token, token.shape)
            # the threshold lies in the widest gap around the wanted share of the nodes
            flat = np.sort(lm[np.arange(T)[None] < n_nodes[:, None]])
            at = min(len(flat) - 2, int((1 - KEEP_SHARE) * len(flat)))
            lo, hi = max(0, at - 20), min(len(flat) - 1, at + 20)
            g = lo + int(np.argmax(np.diff(flat[lo:hi + 1])))
            s.threshold = float(math.exp((flat[g] + flat[g + 1]) / 2))
        del z
        s.payloads = [s.hid] if c["kind"] == "prune_prob" else [s.hid, s.q, s.kt, s.vt]
        s.payload_out = [torch.zeros_like(x) for x in s.payloads]
        s.ws_prune = torch.empty(pb.workspace_bytes(pb.WS_EARLY_PRUNE, B, T, hidden=c["hidden"], vocab=c["vocab"]),
                                 dtype=torch.uint8, device="cuda")
    if c["kind"] in ("accept", "step"):
        if token is None:
            token = synth.draw_tokens(rng, n_nodes, parent, c["vocab"])
            fail = np.zeros(token.shape, bool)
        # a step's logits are those of the surviving nodes
        s.logits = normal(B, T, c["vocab"])
        _plant_chain(rng, s.logits, [(p, t) for _, p, t in _compact(n_nodes, parent, token, fail)])
        s.ws_acc = torch.empty(pb.workspace_bytes(pb.WS_ACCEPT_PATH, B, T, vocab=c["vocab"]),
                               dtype=torch.uint8, device="cuda")
    if c["kind"] == "step":
        s.out2 = torch.zeros_like(s.q)
    s.token = token
    s.tok = torch.from_numpy(token).cuda() if token is not None else None
    s.tree = pb.Tree(n_nodes=s.nn, parent=s.par, token=s.tok, depth=s.depth, anc=s.anc)
    return s


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------


def _prune_outputs(r):
    return {"keep_bits": r.keep_bits, "new_index": r.new_index, "orig_index": r.orig_index, "n_kept": r.n_kept,
            "cu_nodes": r.cu_nodes, "n_nodes": r.tree.n_nodes, "parent": r.tree.parent, "token": r.tree.token,
            "depth": r.tree.depth, "anc": r.tree.anc, "payloads": r.payloads}


def run(s):
    c = s.c
    if s.kind == "attention":
        return pb.propd_tree_attention(s.tree, s.q, s.kc, s.vc, s.kt, s.vt, s.seq, s.scale, out=s.out,
                                       workspace=s.ws_att)
    if s.kind == "prune":
        return _prune_outputs(pb.propd_early_prune(s.tree, s.hid, s.head, c["top_k"], payloads=s.payloads,
                                                   payload_out=s.payload_out, workspace=s.ws_prune))
    if s.kind == "prune_prob":
        r = pb.propd_early_prune_prob(s.tree, s.hid, s.head, threshold=s.threshold, payloads=s.payloads,
                                      payload_out=s.payload_out, want_log_marginal=True, workspace=s.ws_prune)
        return dict(_prune_outputs(r), log_marginal=r.log_marginal)
    if s.kind == "accept":
        return pb.propd_accept_path(s.tree, s.logits, path_stride=PATH_STRIDE, workspace=s.ws_acc)
    depth, anc = pb.propd_tree_mask(s.nn, s.par)
    tree = pb.Tree(n_nodes=s.nn, parent=s.par, token=s.tok, depth=depth, anc=anc)
    pb.propd_tree_attention(tree, s.q, s.kc, s.vc, s.kt, s.vt, s.seq, s.scale, out=s.out, workspace=s.ws_att)
    r = pb.propd_early_prune(tree, s.hid, s.head, c["top_k"], payloads=s.payloads, payload_out=s.payload_out,
                             workspace=s.ws_prune)
    _, q2, kt2, vt2 = r.payloads
    pb.propd_tree_attention(r.tree, q2, s.kc, s.vc, kt2, vt2, s.seq, s.scale, out=s.out2, workspace=s.ws_att)
    alen, path, nxt = pb.propd_accept_path(r.tree, s.logits, path_stride=PATH_STRIDE, workspace=s.ws_acc)
    seq = s.seq.clone()  # the lengths advance in place, and the next pass starts from the same ones
    toks = pb.propd_commit_path(r.tree, alen, path, nxt, kt2, vt2, s.kc, s.vc, seq, out_stride=PATH_STRIDE)
    return {"out": s.out, "prune": _prune_outputs(r), "out2": s.out2, "accept_len": alen, "path": path,
            "next": nxt, "tokens": toks, "seq_lens": seq, "k_cache": s.kc, "v_cache": s.vc}


# ---------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------


def _attention64(s, nodes, parents, q, kt, vt):
    """Attention of ``nodes[b]`` tree nodes with the given parents; other rows are zero."""
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    for b, n in enumerate(nodes):
        L, n = int(s.lens[b]), int(n)
        seen = np.zeros((n, L + n), bool)
        seen[:, :L] = True
        for i in range(n):
            if i:
                seen[i, L:] = seen[int(parents[b][i]), L:]
            seen[i, L + i] = True
        hide = torch.from_numpy(~seen).cuda()
        for h in range(q.shape[1]):
            k = torch.cat([s.kc[b, h, :L], kt[b, h, :n]]).double()
            v = torch.cat([s.vc[b, h, :L], vt[b, h, :n]]).double()
            w = (q[b, h, :n].double() @ k.T.contiguous() * s.scale).masked_fill(hide, -math.inf)
            out[b, h, :n] = w.softmax(1) @ v
    return out


def exact(c, seed):
    if c["kind"] == "accept":
        return None
    s = prepare(c, seed)
    if c["kind"] == "attention":
        return _attention64(s, s.n_nodes, s.parent, s.q, s.kt, s.vt)
    z = _scores(s, torch.float64)
    fail = np.zeros(s.token.shape, bool)
    if c["kind"] == "prune_prob":
        lm = _log_marginals(z, s.rows, s.token, s.token.shape)
        fail = lm < math.log(s.threshold)
    else:
        for r, (b, _, kids) in enumerate(s.rows):
            t = torch.tensor([int(s.token[b, i]) for i in kids], device="cuda")
            fail[b, kids] = ((z[r][None] > z[r][t][:, None]).sum(1) >= c["top_k"]).cpu().numpy()
    kept = _compact(s.n_nodes, s.parent, s.token, fail)
    payloads = []
    for x in s.payloads:
        y = torch.zeros(x.shape, dtype=torch.float64, device="cuda")
        for b, (keep, _, _) in enumerate(kept):
            y[b][..., :len(keep), :] = x[b][..., keep, :].double()
        payloads.append(y)
    whole = dict.fromkeys(("keep_bits", "new_index", "orig_index", "n_kept", "cu_nodes", "n_nodes", "parent",
                           "token", "depth", "anc"))
    if c["kind"] == "prune_prob":
        return dict(whole, payloads=payloads, log_marginal=torch.from_numpy(lm))
    if c["kind"] == "prune":
        return dict(whole, payloads=payloads)
    return {"out": _attention64(s, s.n_nodes, s.parent, s.q, s.kt, s.vt), "prune": dict(whole, payloads=payloads),
            "out2": _attention64(s, [len(k) for k, _, _ in kept], [p for _, p, _ in kept], *payloads[1:]),
            "accept_len": None, "path": None, "next": None, "tokens": None, "seq_lens": None,
            "k_cache": None, "v_cache": None}
