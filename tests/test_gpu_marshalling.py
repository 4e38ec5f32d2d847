"""The native marshalling of the binding against its ctypes calls: the same results for everything that both take, and what
either refuses is refused with the same message by a Layer that has both."""
import numpy as np
import pytest
import torch

import paper_2603_05353_amd.binding as B

DEV = "cuda:0"


def layer(native, **kw):
    args = dict(dtype="bf16", n_q_heads=8, n_kv_heads=2, head_dim=64, rope_theta=5e5, max_ctx=600, max_prompt=8)
    L = B.Layer(**{**args, **kw})
    if not native:
        L._native = None
    return L


def tensors(seed, dev=DEV):
    g = torch.Generator().manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=g).to(torch.bfloat16).to(dev)

    lens = [100, 0, 37, 260]
    return dict(k=[normal(n, 2, 64) for n in lens], v=[normal(n, 2, 64) for n in lens], q_prompt=normal(8, 8, 64), k_prompt=normal(9, 2, 64),
                q=normal(40, 8, 64), kn=normal(40, 2, 64), vn=normal(41, 2, 64),
                pos=torch.sort(torch.randperm(397, generator=g)[:40])[0].to(torch.int32).to(dev), order=[2, 0, 3, 1])


def run_all(L, x, as_tuple=False, accumulate=False, with_v=True):
    """Every call that both ways serve; all tensors that come back or are written."""
    seq = tuple if as_tuple else list
    K, V, scores = L.empty_cache(400), L.empty_cache(400), torch.ones(405, device=DEV)
    K.zero_(), V.zero_()
    out = []
    r = L.reposition_keys(seq(x["k"]), seq(x["v"]) if with_v else None, chunk_order=seq(x["order"]), cached_pos0=[0, 5, 0, 3], k_out=K, v_out=V)
    out += [r[0].clone(), r[1].clone(), r[2], r[3]]
    r = L.reposition_score(seq(x["k"]), seq(x["v"]), x["q_prompt"], chunk_order=seq(x["order"]), delta_override=[1, 2, 3, 4], k_out=K, v_out=V,
                           k_prompt=x["k_prompt"], scores=scores, accumulate=accumulate)
    out += [r[0].clone(), r[1].clone(), r[2], r[3], r[4].clone()]
    out.append(L.score_tokens(K, x["q_prompt"], scores=scores, accumulate=accumulate).clone())
    out.append(L.select_topk(scores, ratio=0.1, idx_out=torch.zeros(50, dtype=torch.int32, device=DEV)).clone())
    out.append(L.select_topk(scores, k=7, idx_out=torch.zeros(7, dtype=torch.int32, device=DEV)).clone())
    q, kn = x["q"].clone(), x["kn"].clone()
    out += [L.rope_rows(q, x["pos"]).clone(), L.rope_rows(kn, x["pos"]).clone()]
    L.splice_kv(kn, x["vn"], x["pos"], K, V)
    L.splice_kv(kn, None, x["pos"], K, None)
    out += [K.clone(), V.clone(), L.recompute_attention(q, x["pos"], K, V).clone()]
    out += [t.clone() for t in L.recompute_attention(q, x["pos"], K, V, out=torch.empty_like(q), return_lse=True)]
    return out


class Served:
    """The native calls, with what each of them returned."""

    def __init__(self, native):
        self.native, self.returned = native, []

    def __getattr__(self, name):
        def call(*args):
            r = getattr(self.native, name)(*args)
            self.returned.append((name, r))
            return r
        return call


@pytest.mark.gpu
@pytest.mark.parametrize("strides", [(0, 0), (2 * 64 + 8, 64), (64, 600 * 64)], ids=["packed", "padded", "head-major"])
@pytest.mark.parametrize("as_tuple,accumulate,with_v", [(False, False, True), (True, True, False)])
def test_native_and_ctypes_calls_agree(strides, as_tuple, accumulate, with_v):
    if strides[1] == 600 * 64:
        kw = dict(token_stride=64, head_stride=600 * 64)
    else:
        kw = dict(token_stride=strides[0], head_stride=strides[1] if strides[0] else 0)
    results = []
    for native in (True, False):
        L = layer(native, **kw)
        if native:
            L._native = served = Served(L._native)
        results.append(run_all(L, tensors(3), as_tuple, accumulate, with_v))
        torch.cuda.synchronize()
        if native:  # none of them went on to ctypes
            assert all(r is not None for _, r in served.returned), [name for name, r in served.returned if r is None]
            assert [name for name, _ in served.returned] == ["reposition_keys", "reposition_score", "score_tokens", "select_topk", "select_topk",
                                                             "rope_rows", "rope_rows", "splice_kv", "splice_kv", "recompute_attention",
                                                             "recompute_attention"]
        L.close()
    assert len(results[0]) == len(results[1])
    for a, b in zip(*results):
        assert torch.equal(a, b) if isinstance(a, torch.Tensor) else a == b


def mistakes(x, K, V, dev):
    """(stage, positional arguments, keywords) of calls that must not reach the library or that it refuses."""
    idx = torch.zeros(50, dtype=torch.int32, device=dev)
    scores = torch.zeros(405, device=dev)
    q = x["q"]
    att = lambda **kw: ("recompute_attention", (), {**dict(q_sel=q, row_pos=x["pos"], k_cache=K, v_cache=V, out=torch.empty_like(q)), **kw})
    spl = lambda **kw: ("splice_kv", (), {**dict(k_new=x["kn"], v_new=x["vn"], idx=x["pos"], k_cache=K, v_cache=V), **kw})
    rep = lambda **kw: ("reposition_keys", (), {**dict(k_chunks=x["k"], v_chunks=x["v"], chunk_order=x["order"], k_out=K, v_out=V), **kw})
    return [
        att(q_sel=q.float()), att(q_sel=q[:, :4]), att(q_sel=q.transpose(0, 1)), att(row_pos=x["pos"].long()), att(row_pos=x["pos"][:-1]),
        att(k_cache=K[:, :1]), att(k_cache=K.float()), att(out=torch.empty_like(q)[:-1]), att(k_cache=K[::2]), att(v_cache=None), att(row_pos=None),
        spl(v_new=None), spl(k_new=x["kn"][:-1]), spl(idx=x["pos"].long()), spl(v_cache=V[:, :1]),
        rep(chunk_order=[0, 0, 1, 2]), rep(chunk_order=[0, 1, 2, 7]), rep(v_chunks=x["v"][:3]), rep(k_chunks=[t.float() for t in x["k"]]),
        rep(k_out=K[:300]), rep(v_chunks=[x["v"][0], x["v"][1], x["v"][3], x["v"][2]]),
        ("score_tokens", (K, x["q_prompt"][:, :3]), dict(scores=scores)), ("score_tokens", (K, x["q_prompt"]), dict(scores=scores[:100])),
        ("score_tokens", (K, x["q_prompt"], x["k_prompt"][:5]), dict(scores=scores)), ("score_tokens", (K, torch.cat([x["q_prompt"]] * 2)), dict(scores=scores)),
        ("select_topk", (scores,), dict(ratio=1.5, idx_out=idx)), ("select_topk", (scores.double(),), dict(ratio=0.1, idx_out=idx)),
        ("select_topk", (scores[::2],), dict(ratio=0.1, idx_out=idx)), ("select_topk", (scores,), dict(ratio=0.1, idx_out=idx.long())),
        ("rope_rows", (q[:, :, :32], x["pos"]), {}), ("rope_rows", (q.float(), x["pos"]), {}), ("rope_rows", (q, x["pos"][:-1]), {}), ("rope_rows", (q[0], x["pos"]), {}),
    ]


def outcome(L, stage, args, kw):
    try:
        getattr(L, stage)(*args, **kw)
    except Exception as e:  # noqa: BLE001 -- the kind and the message are what is compared
        return type(e).__name__, str(e)
    return None


@pytest.mark.gpu
def test_mistakes_are_refused_with_the_same_message():
    x = tensors(4)
    both, only = layer(True), layer(False)
    K, V = both.empty_cache(400), both.empty_cache(400)
    for stage, args, kw in mistakes(x, K, V, DEV):
        a, b = outcome(both, stage, args, kw), outcome(only, stage, args, kw)
        assert a is not None and a == b, (stage, a, b)
    both.close(), only.close()
    assert outcome(both, "recompute_attention", (x["q"], x["pos"], K, V), {}) == outcome(only, "recompute_attention", (x["q"], x["pos"], K, V), {})


def test_tensors_that_are_not_on_the_gpu_do_not_reach_the_library():
    """(host only) The native calls return None, the layer says what is wrong."""
    x = tensors(5, "cpu")
    both, only = layer(True, stream=0), layer(False, stream=0)
    K, V = torch.zeros(400, 2, 64, dtype=torch.bfloat16), torch.zeros(400, 2, 64, dtype=torch.bfloat16)
    n = both._native
    scores, idx = torch.zeros(400), torch.zeros(50, dtype=torch.int32)
    assert n.reposition_keys(x["k"], x["v"], x["order"], None, None, K, V) is None
    assert n.reposition_score(x["k"], x["v"], x["order"], None, None, K, V, x["q_prompt"], None, scores, False) is None
    assert n.score_tokens(K, x["q_prompt"], None, scores, False) is None
    assert n.select_topk(scores, 0.1, -1, idx) is None
    assert n.recompute_attention(x["q"], x["pos"], K, V, x["q"], None) is None
    assert n.splice_kv(x["kn"], x["vn"], x["pos"], K, V) is None
    assert n.rope_rows(x["q"], x["pos"]) is None
    for bad in (None, 3, "x", np.zeros((4, 2, 64), np.float32), [], torch.tensor(1.0)):  # nor do things that are no tensors
        assert n.recompute_attention(bad, bad, bad, bad, bad, bad) is None and n.rope_rows(bad, bad) is None
        assert n.splice_kv(bad, bad, bad, bad, bad) is None and n.select_topk(bad, bad, bad, bad) is None
        assert n.reposition_keys(bad, bad, bad, bad, bad, bad, bad) is None
    for stage, args, kw in mistakes(x, K, V, "cpu"):
        a, b = outcome(both, stage, args, kw), outcome(only, stage, args, kw)
        assert a is not None and a == b, (stage, a, b)
    both.close(), only.close()
    assert both._native is None


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False], ids=["native", "ctypes"])
@pytest.mark.parametrize("call", ["select_topk", "select_topk_noalloc"])
@pytest.mark.parametrize("n,kw", [(405, dict(k=20)), (405, dict(ratio=0.05)), (20000, dict(ratio=0.001))], ids=str)
def test_a_buffer_of_too_few_indices_is_refused_before_anything_is_written(call, native, n, kw):
    L = layer(native, max_ctx=20000)
    scores, room = torch.rand(n, device=DEV), torch.full((64,), -7, dtype=torch.int32, device=DEV)
    need = L.budget_of(n, **kw)
    assert need == 20
    with pytest.raises(ValueError, match="fewer entries than k"):
        getattr(L, call)(scores, idx_out=room[:need - 1], **kw)
    torch.cuda.synchronize()
    assert (room == -7).all()
    got = getattr(L, call)(scores, idx_out=room[:need], **kw)
    torch.cuda.synchronize()
    assert got.tolist() == sorted(torch.topk(scores, need).indices.tolist()) and (room[need:] == -7).all()
    L.close()


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False], ids=["native", "ctypes"])
def test_a_value_cache_of_fewer_rows_than_the_key_cache_is_refused(native):
    """The library takes one number of rows for both; a longer value cache is as good as one of the same length."""
    x, L = tensors(7), layer(native)
    K, V = L.empty_cache(400), L.empty_cache(400)
    K.normal_(), V.normal_()
    want, before = L.recompute_attention(x["q"], x["pos"], K, V).clone(), V.clone()
    with pytest.raises(ValueError, match="v_cache: 396 rows, the other cache has 400"):
        L.recompute_attention(x["q"], x["pos"], K, V[:396])
    idx = x["pos"].clone()
    idx[-1] = 399
    with pytest.raises(ValueError, match="v_cache: 396 rows, the other cache has 400"):
        L.splice_kv(x["kn"], x["vn"], idx, K, V[:396])
    torch.cuda.synchronize()
    assert torch.equal(V, before)
    assert torch.equal(L.recompute_attention(x["q"], x["pos"], K[:397], V), want)
    L.splice_kv(x["kn"], x["vn"], x["pos"], K[:397], V)
    assert torch.equal(V[x["pos"].long()], x["vn"][:40])
    L.close()


class Taken(B.Layer):
    """A Layer whose native calls are there when a stage asks, and gone when it asks again, as where another thread's bind() comes
    between."""

    class Stub:
        def __getattr__(self, name):
            return lambda *args: (0, [0], 5) if name.startswith("repo") else (0, 3) if name == "select_topk" else 0

    reads = 0

    @property
    def _native(self):
        self.reads += 1
        return self.Stub() if self.reads % 2 == 1 else None

    @_native.setter
    def _native(self, value):
        self.reads = 0


@pytest.mark.parametrize("stage", ["reposition_keys", "reposition_score", "score_tokens", "select_topk", "recompute_attention", "splice_kv", "rope_rows"])
def test_a_stage_asks_for_the_native_calls_once(stage):
    """(host only)"""
    x = tensors(6, "cpu")
    K, V, scores = torch.zeros(400, 2, 64, dtype=torch.bfloat16), torch.zeros(400, 2, 64, dtype=torch.bfloat16), torch.zeros(400)
    calls = dict(reposition_keys=((x["k"],), dict(k_out=K)), reposition_score=((x["k"], None, x["q_prompt"]), dict(k_out=K, scores=scores)),
                 score_tokens=((K, x["q_prompt"]), dict(scores=scores)), select_topk=((scores,), dict(k=3, idx_out=torch.zeros(3, dtype=torch.int32))),
                 recompute_attention=((x["q"], x["pos"], K, V), dict(out=x["q"])), splice_kv=((x["kn"], x["vn"], x["pos"], K, V), {}),
                 rope_rows=((x["q"], x["pos"]), {}))
    L = Taken("bf16", 8, 2, 64, 5e5, max_ctx=600, max_prompt=8, stream=0)
    args, kw = calls[stage]
    getattr(L, stage)(*args, **kw)
    assert L.reads == 1
    L.close()


@pytest.mark.parametrize("state", ["absent", "no module", "another torch"])
def test_a_tree_with_the_library_alone_serves_through_ctypes(monkeypatch, tmp_path, state):
    """(host only) Without the native module, silently; with one that cannot be used, with a warning."""
    path = tmp_path / "_ifkv_marshal.so"
    if state == "no module":
        path.write_bytes(b"not a library")
    monkeypatch.setattr(B, "_marshal", None)
    if state == "another torch":
        monkeypatch.setattr(torch, "__version__", "1.0.0+cpu")
    else:
        monkeypatch.setattr(B, "MARSHAL_PATH", str(path))
    if state == "absent":
        assert B.load_marshal() is None
    else:
        with pytest.warns(RuntimeWarning, match="not used"):
            assert B.load_marshal() is None
    L = layer(True, stream=0)
    assert L._native is None and L.budget_of(100, 0.25) == 25
    with pytest.raises(ValueError, match="on the GPU"):
        L.rope_rows(torch.zeros(3, 2, 64, dtype=torch.bfloat16), torch.zeros(3, dtype=torch.int32))
    L.close()
