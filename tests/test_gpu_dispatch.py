"""GPU parity at the edges of the kernels' dispatch rules: row counts, lengths, alignments and
types on both sides of every line where a call changes its kernel or tile shape, against the
CPU oracle with the tolerances of test_gpu_parity."""
import numpy as np
import pytest
import torch

from paper_2402_13485_amd import synth
from gpu_util import host_f64, sentinel_like, to_dev, to_host
from test_gpu_parity import (check_attention, check_prob, check_prune, dev_tree, pb,  # noqa: F401
                             prob_reference, run_attention, run_prob, run_prune, threshold_in_a_gap)

pytestmark = pytest.mark.gpu


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
