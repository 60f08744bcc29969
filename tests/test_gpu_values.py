"""GPU parity where the values, not the shapes, are the hard part: softmax weights that must not
lose bits, results near the end of the type's range, values that are not finite.  Attention inputs
here are made by hand: the query is (1, 1, 0, ...), so the score of a key is the sum of its first
two entries, and the columns of V are chosen so that errors of the weights stay when the result
itself is small."""
import numpy as np
import pytest

from paper_2402_13485_amd import synth
from gpu_util import host_f64
from test_gpu_parity import pb, run_attention  # noqa: F401

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
