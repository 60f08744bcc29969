"""The native argument marshalling against the Python code of the binding: the same outputs, and the same
errors for what is refused."""
import ctypes
import threading
import time

import numpy as np
import pytest
import torch

from paper_2402_13485_amd import synth
from test_gpu_parity import dev_tree, pb  # noqa: F401

pytestmark = pytest.mark.gpu

B, H, T, L, HD, V = 2, 3, 9, 40, 64, 96


class Sub(torch.Tensor):
    pass


def flat(x):
    if torch.is_tensor(x):
        return [x]
    if isinstance(x, (list, tuple)):
        return [z for y in x for z in flat(y)]
    return flat([v for v in vars(x).values() if v is not None]) if hasattr(x, "__dataclass_fields__") else []


def both(pb, monkeypatch, call):
    """(outputs or error) of the native marshalling and of the Python code."""
    assert pb._native() is not None, "the native marshalling is not built"
    out = []
    for native in (True, False):
        with monkeypatch.context() as m:
            if not native:
                m.setattr(pb, "_marshal", None)
            try:
                out.append(call())
            except Exception as e:  # compared below
                out.append(e)
    torch.cuda.synchronize()
    return out


@pytest.fixture(params=["bf16", "f32"])
def x(request, pb):
    dt = torch.bfloat16 if request.param == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    r = lambda *s: torch.randn(s, device="cuda", generator=gen).to(dt)
    n, par, _ = synth.pad_trees([synth.rank_product_tree(T, 3), synth.rank_product_tree(T - 2, 3)], T)
    tok = np.random.default_rng(0).integers(0, V, (B, T)).astype(np.int32)
    d = dict(tree=dev_tree(pb, n, par, tok), q=r(B, H, T, 64), kt=r(B, H, T, 64), vt=r(B, H, T, 64), kc=r(B, H, L, 64),
             vc=r(B, H, L, 64), seq=torch.tensor([30, 7], dtype=torch.int32, device="cuda"), hid=r(B, T, HD), head=r(V, HD),
             logits=r(B, T, V))
    d["acc"] = pb.propd_accept_path(d["tree"], d["logits"])
    return d


def calls(pb, x):
    t, a = x["tree"], x["acc"]
    att = lambda **k: pb.propd_tree_attention(t, x["q"], x["kc"], x["vc"], x["kt"], x["vt"], x["seq"], 0.125, **k)
    ws = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")

    def commit(**k):
        kc, vc, seq = x["kc"].clone(), x["vc"].clone(), x["seq"].clone()
        return [pb.propd_commit_path(t, *a, x["kt"], x["vt"], kc, vc, seq, **k), kc, vc, seq]

    # rows past a tree are left as they were by attention, and unspecified past the survivors in payloads made here
    zero = lambda *ts: [torch.zeros_like(y) for y in ts]
    return {
        "mask": lambda: pb.propd_tree_mask(t.n_nodes, t.parent),
        "attention": lambda: att(out=torch.zeros_like(x["q"])),
        "attention_ws": lambda: att(out=torch.zeros_like(x["q"]), workspace=ws),
        "prune": lambda: pb.propd_early_prune(t, x["hid"], x["head"], 20),
        "prune_rank": lambda: pb.propd_early_prune(t, x["hid"], x["head"], 20, want_rank=True, workspace=ws),
        "prune_payloads": lambda: pb.propd_early_prune(t, x["hid"], x["head"], 20, payloads=(x["hid"], x["q"]),
                                                       payload_out=zero(x["hid"], x["q"])),
        "prob": lambda: pb.propd_early_prune_prob(t, x["hid"], x["head"], threshold=1e-3),
        "prob_rank": lambda: pb.propd_early_prune_prob(t, x["hid"], x["head"], keep_count=3, want_log_marginal=True,
                                                       payloads=[x["q"]], payload_out=zero(x["q"])),
        "accept": lambda: pb.propd_accept_path(t, x["logits"]),
        "accept_stride": lambda: pb.propd_accept_path(t, x["logits"], path_stride=4, workspace=ws),
        "commit": commit,
        "commit_stride": lambda: commit(out_stride=5),
    }


def test_same_outputs(pb, monkeypatch, x):
    for name, call in calls(pb, x).items():
        native, python = both(pb, monkeypatch, call)
        assert type(native) is type(python), (name, native, python)
        native, python = flat(native), flat(python)
        assert len(native) == len(python) > 0, name
        for a, b in zip(native, python):
            assert a.shape == b.shape and a.dtype == b.dtype and a.stride() == b.stride() and a.data_ptr() % 16 == 0, name
            assert torch.equal(a, b), name


def test_payloads_made_by_the_call(pb, monkeypatch, x):
    for r in both(pb, monkeypatch, lambda: pb.propd_early_prune(x["tree"], x["hid"], x["head"], V, payloads=[x["q"], x["hid"]])):
        assert r.log_marginal is None and r.rank is None and len(r.payloads) == 2
        for src, dst in zip((x["q"], x["hid"]), r.payloads):
            for b, n in enumerate(x["tree"].n_nodes.tolist()):
                assert torch.equal(src[b][..., :n, :], dst[b][..., :n, :])


def test_same_errors(pb, monkeypatch, x):
    t, q, kc, vc, kt, vt, seq = (x[k] for k in ("tree", "q", "kc", "vc", "kt", "vt", "seq"))
    att = lambda *a, **k: lambda: pb.propd_tree_attention(*a, **k)
    half = torch.empty(8, dtype=torch.uint8, device="cuda")
    small = pb.Tree(t.n_nodes[:1], t.parent[:1], t.token[:1], t.depth[:1], t.anc[:1])
    strange = torch.zeros(B, H, T, 48, dtype=q.dtype, device="cuda")
    bad = [
        att(t, q.cpu(), kc, vc, kt, vt, seq, 0.125),
        att(t, q.half(), kc, vc, kt, vt, seq, 0.125),
        att(t, q, kc.transpose(2, 3), vc, kt, vt, seq, 0.125),
        att(t, q, kc[:, :, :30].contiguous(), vc, kt, vt, seq, 0.125),
        att(t, q, kc, vc, kt, vt[:1], seq, 0.125),
        att(t, q, kc, vc, kt, vt, seq.long(), 0.125),
        att(t, q, kc, vc, kt, vt, seq, -1.0),
        att(t, q, kc, vc, kt, vt, seq, "1"),
        att(t, q, kc, vc, kt, vt, seq, 0.125, workspace=half),
        att(small, q, kc, vc, kt, vt, seq, 0.125),
        att(t, strange, torch.zeros(B, H, L, 48, dtype=q.dtype, device="cuda"), torch.zeros(B, H, L, 48, dtype=q.dtype, device="cuda"),
            strange, strange, seq, 0.125),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], 0),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], np.int64(5)),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], 1 << 40),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"][:, :-1], 5),
        lambda: pb.propd_early_prune(t, x["hid"][:1], x["head"], 5),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], 5, payloads=[q.transpose(1, 2)]),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], 5, payloads=[q], payload_out=[kc]),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], 5, payloads=[q], payload_out=[q]),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], 5, payloads=[q] * 9),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], 5, workspace=half),
        lambda: pb.propd_early_prune(t, x["hid"], x["head"], 5, want_rank=np.zeros(2)),
        lambda: pb.propd_early_prune_prob(t, x["hid"], x["head"], threshold=2.0),
        lambda: pb.propd_early_prune_prob(t, x["hid"], x["head"], keep_count=0),
        lambda: pb.propd_accept_path(t, x["logits"].half()),
        lambda: pb.propd_accept_path(t, x["logits"], path_stride=0),
        lambda: pb.propd_accept_path(small, x["logits"]),
        lambda: pb.propd_accept_path(pb.Tree(t.n_nodes, t.parent), x["logits"]),
        lambda: pb.propd_commit_path(t, *x["acc"], kt, vt, kc, vc[:, :, :5].contiguous(), seq),
        lambda: pb.propd_commit_path(t, x["acc"][0].long(), *x["acc"][1:], kt, vt, kc, vc, seq),
        lambda: pb.propd_tree_mask(t.n_nodes.cpu(), t.parent),
        lambda: pb.propd_tree_mask(t.n_nodes, t.parent[:, ::2]),
    ]
    for n, call in enumerate(bad):
        native, python = both(pb, monkeypatch, call)
        assert type(native) is type(python), (n, native, python)
        if isinstance(python, Exception):
            assert str(native) == str(python), (n, native, python)
        else:  # an integer of another class, which the Python code takes
            assert n == 12 and all(torch.equal(a, b) for a, b in zip(flat(native), flat(python))), (n, python)


def test_other_tensor_classes_and_streams(pb, monkeypatch, x):
    """A subclass of Tensor is left to the Python code, a Parameter is not; the current stream is the one used."""
    call = lambda k: lambda: pb.propd_tree_attention(x["tree"], k(x["q"]), x["kc"], x["vc"], x["kt"], x["vt"], x["seq"], 0.125,
                                                     out=torch.zeros_like(x["q"]))
    want = call(lambda q: q)()
    for k in (lambda q: q.as_subclass(Sub), lambda q: torch.nn.Parameter(q, requires_grad=False)):
        for got in both(pb, monkeypatch, call(k)):
            assert torch.equal(got.as_subclass(torch.Tensor), want)
    stream = torch.cuda.Stream()
    seen = []
    real = ctypes.c_void_p(stream.cuda_stream).value
    monkeypatch.setattr(pb, "_stream", lambda inner=pb._stream: seen.append(inner()) or seen[-1])
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        got = both(pb, monkeypatch, call(lambda q: q))
    assert seen == [real, real] and all(torch.equal(g, want) for g in got)


def test_out_of_host_memory_leaves_no_call_behind(pb, x):
    """Wherever host memory ends, a call that did not return its results was not made: the Python code makes it
    then, and a commit made twice would append its rows twice."""
    testcapi = pytest.importorskip("_testcapi")
    t, kc, vc, seq = x["tree"], x["kc"].clone(), x["vc"].clone(), x["seq"].clone()
    commit = pb._native().commit_path
    args = (t.n_nodes, t.parent, t.token, t.depth, t.anc, *x["acc"], x["kt"], x["vt"], kc, vc, seq, None, pb._stream)
    made = []
    for n in range(40):  # the n-th request for memory fails
        result = None
        testcapi.set_nomemory(n, n + 1)
        try:
            result = commit(*args)
        except (MemoryError, RuntimeError):
            pass
        finally:
            testcapi.remove_mem_hooks()
        torch.cuda.synchronize()
        made.append(result is not None)
        assert (seq.tolist() != x["seq"].tolist()) == made[-1], n
        seq.copy_(x["seq"])
    assert made[-1] and not all(made)


def test_other_threads_run_during_a_call(pb, x):
    """The C call (here one that sleeps in place of a launch that waits) and the allocations leave the interpreter to
    other threads, as calls through ctypes do."""
    native, lib = pb._native(), pb.load_library()
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    sleep = address(ctypes.CDLL(None).sleep)  # of the seconds that its first argument says: B
    n, parent = torch.ones(1, dtype=torch.int32, device="cuda"), -torch.ones(1, 1, dtype=torch.int32, device="cuda")
    ticks, stop = [], threading.Event()

    def tick():
        while not stop.wait(0.01):
            ticks.append(time.perf_counter())

    thread = threading.Thread(target=tick)
    try:
        native.init(sleep, *[address(lib.propd_tree_attention)] * 6)
        thread.start()
        start = time.perf_counter()
        native.tree_mask(n, parent, pb._stream)
        end = time.perf_counter()
    finally:
        stop.set()
        thread.join()
        pb._init_marshal(lib)
    assert end - start > 0.9
    assert sum(start + 0.1 < at < end - 0.1 for at in ticks) > 10
