"""Rows that are not finite: what a row does not see must not show in its result, and what it sees must."""
import numpy as np
import pytest
import torch

from oracle import infoflow_oracle as O
from paper_2603_05353_amd import Layer
from tests.helpers import DEV, assert_attention_close, score_tol, to_dev, to_host_f64
from workloads import to_f64, to_storage

pytestmark = pytest.mark.gpu

# every stage-4 kernel on the matrix units, not cut and cut into parts of one and of three kv tiles, first and second sweep
KERNELS = {"f32-64": ("f32", 64, {}), "f32-128": ("f32", 128, {}), "bf16-64": ("bf16", 64, {}),
           "bf16-128-narrow": ("bf16", 128, {"attn_wide": 2}), "bf16-128-wide": ("bf16", 128, {"attn_wide": 1})}
CUTS = {"whole": {"attn_split_parts": 1}, "parts-of-1": {"attn_part_tiles": 1}, "parts-of-3": {"attn_part_tiles": 3},
        "second-sweep": {"attn_split_parts": 1, "attn_exact_sweep": 1}}
N, TAIL, HQ, HKV = 700, 37, 8, 2  # the last TAIL cache rows are never seen


def inputs(dtype, d, rows):
    g = np.random.Generator(np.random.Philox(key=[d + rows, 61]))
    K, V = (to_storage(g.standard_normal((N, HKV, d)), dtype) for _ in range(2))
    q = to_storage(g.standard_normal((rows, HQ, d)), dtype)
    pos = np.sort(g.choice(N - TAIL, size=rows, replace=False)).astype(np.int64)
    pos[0], pos[-1] = 0, N - TAIL - 1
    return K, V, q, pos


def cache(x, dtype, padding=0):
    """On the GPU, rows `padding` elements apart beyond their length, with NaN in between."""
    x = to_dev(x, dtype)
    if padding == 0:
        return x
    n, heads, d = x.shape
    base = torch.full((n, heads * d + padding), float("nan"), dtype=x.dtype, device=DEV)
    c = torch.as_strided(base, (n, heads, d), (heads * d + padding, d, 1))
    c.copy_(x)
    return c


def attend(dtype, d, knobs, q, pos, kd, vd):
    L = Layer(dtype, HQ, HKV, d, 5e5, max_ctx=N, max_prompt=1, token_stride=kd.stride(0), head_stride=kd.stride(1))
    for key, value in knobs.items():
        L.set_tuning(key, value)
    out, lse = L.recompute_attention(to_dev(q, dtype), torch.from_numpy(pos.astype(np.int32)).to(DEV), kd, vd, return_lse=True)
    torch.cuda.synchronize()
    L.close()
    return to_host_f64(out, dtype), lse.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("rows", [300, 9], ids=["dense", "sparse-padded-cache"])
@pytest.mark.parametrize("cut", CUTS)
@pytest.mark.parametrize("kernel", KERNELS)
def test_value_rows_reach_only_the_rows_that_see_them(kernel, cut, rows):
    """An unwritten tail of the cache (NaN in keys and values) and single elements of V that are NaN or infinite: every
    element of the result is what the rows up to its own position make it."""
    dtype, d, knobs = KERNELS[kernel]
    K, V, q, pos = inputs(dtype, d, rows)
    ref, lse_ref = O.recompute_attention(to_f64(q, dtype), pos, to_f64(K, dtype), to_f64(V, dtype), d ** -0.5)
    ref_abs, _ = O.recompute_attention(to_f64(q, dtype), pos, to_f64(K, dtype), np.abs(to_f64(V, dtype)), d ** -0.5)
    kd, vd = (cache(x, dtype, 16 if rows < 20 else 0) for x in (K, V))
    kd[N - TAIL:] = float("nan")
    vd[N - TAIL:] = float("nan")
    G = HQ // HKV
    spoilt = [(90, 0, 5, float("nan")), (333, 1, 40, float("inf")), (334, 1, 41, float("-inf")), (335, 1, d - 1, float("nan"))]
    for j, g, c, x in spoilt:
        vd[j, g, c] = x
    out, lse = attend(dtype, d, {**knobs, **CUTS[cut]}, q, pos, kd, vd)
    for j, g, c, x in spoilt:
        seen = out[pos >= j, g * G:(g + 1) * G, c]
        assert np.array_equal(seen, np.full(seen.shape, x), equal_nan=True), (j, c)
        out[pos >= j, g * G:(g + 1) * G, c] = ref[pos >= j, g * G:(g + 1) * G, c]
    assert np.isfinite(out).all()
    assert_attention_close(out, ref, ref_abs, dtype, lse, lse_ref)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("cut", CUTS)
@pytest.mark.parametrize("kernel", KERNELS)
def test_a_logit_that_is_not_a_number_shows(kernel, cut, bad):
    """A key with a NaN or with a logit of +infinity: no softmax exists for the rows that see it, however the launch is cut."""
    dtype, d, knobs = KERNELS[kernel]
    K, V, q, pos = inputs(dtype, d, 120)
    q[:, HQ // HKV:, 3] = to_storage(np.abs(to_f64(q[:, HQ // HKV:, 3], dtype)) + 0.5, dtype)
    ref, lse_ref = O.recompute_attention(to_f64(q, dtype), pos, to_f64(K, dtype), to_f64(V, dtype), d ** -0.5)
    ref_abs, _ = O.recompute_attention(to_f64(q, dtype), pos, to_f64(K, dtype), np.abs(to_f64(V, dtype)), d ** -0.5)
    kd, vd = to_dev(K, dtype), to_dev(V, dtype)
    j = 270
    kd[j, 1, 3] = bad
    out, lse = attend(dtype, d, {**knobs, **CUTS[cut]}, q, pos, kd, vd)
    heads = slice(HQ // HKV, HQ)
    assert np.isnan(out[pos >= j, heads]).all() and np.isnan(lse[pos >= j, heads]).all()
    out[pos >= j, heads], lse[pos >= j, heads] = ref[pos >= j, heads], lse_ref[pos >= j, heads]
    assert_attention_close(out, ref, ref_abs, dtype, lse, lse_ref)


@pytest.mark.parametrize("m", [6, 24, 40, 130, 200])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)], ids=["bf16-128", "bf16-64", "f32-64", "f32-128"])
def test_a_prompt_key_that_is_not_a_number_takes_its_rows_out(dtype, d, m):
    """The prompt rows from it on have no normaliser: they add nothing to the scores, as in the ALU kernels."""
    g = np.random.Generator(np.random.Philox(key=[m, 62]))
    K, q, kp = (to_storage(g.standard_normal(s), dtype) for s in ((900, HKV, d), (m, HQ, d), (m, HKV, d)))
    K64, q64, kp64 = to_f64(K, dtype), to_f64(q, dtype), to_f64(kp, dtype)
    G, t = HQ // HKV, m // 3
    ref = (O.score_tokens(K64[:, :1], q64[:, :G], d ** -0.5, k_prompt=kp64[:, :1])
           + O.score_tokens(K64[:, 1:], q64[:t, G:], d ** -0.5, k_prompt=kp64[:t, 1:])) / HKV
    kpd = to_dev(kp, dtype)
    kpd[t, 1, 7] = float("nan")
    for flags in (0, 1):
        L = Layer(dtype, HQ, HKV, d, 5e5, max_ctx=900, max_prompt=m, flags=flags)
        s = L.score_tokens(to_dev(K, dtype), to_dev(q, dtype), k_prompt=kpd)
        torch.cuda.synchronize()
        assert (np.abs(s.cpu().numpy() - ref) <= score_tol(ref, m, 1.2e-4)).all(), flags
        L.close()


# parts whose keys all lie 2^290 and more below the others': the first or the last, a whole round of eight, all parts of one wavefront
VANISHING = {9: [[0], [8], list(range(8))], 12: [[3, 7, 11], [8, 9, 10, 11]], 17: [[0], [16], [0, 4, 8, 12, 16], [3, 7, 11, 15]]}


@pytest.mark.parametrize("rows", [40, 300])
@pytest.mark.parametrize("parts,low", [(p, low) for p, lows in VANISHING.items() for low in lows], ids=str)
@pytest.mark.parametrize("kernel", ["f32-64", "f32-128", "bf16-64", "bf16-128-narrow"])
def test_an_infinite_value_in_a_part_of_no_weight_adds_nothing(kernel, parts, low, rows):
    """Whichever part holds it, and however the merge goes through the parts (eight at a time, or dealt out to four wavefronts)."""
    dtype, d, knobs = KERNELS[kernel]
    n, tiles = 512 * parts, 8
    g = np.random.Generator(np.random.Philox(key=[parts + rows, 63]))
    K, V = (to_storage(g.standard_normal((n, HKV, d)), dtype) for _ in range(2))
    q = g.standard_normal((rows, HQ, d))
    q[:, :, 5] = 1.0
    q = to_storage(q, dtype)
    in_low = np.isin(np.arange(n) // 512, low)
    K[:, :, 5] = to_storage(np.where(in_low, -230.0 * d ** 0.5, 0.0)[:, None] * np.ones((1, HKV)), dtype)
    pos = np.arange(n - rows, n, dtype=np.int64)
    ref, lse_ref = O.recompute_attention(to_f64(q, dtype), pos, to_f64(K, dtype), to_f64(V, dtype), d ** -0.5)
    ref_abs, _ = O.recompute_attention(to_f64(q, dtype), pos, to_f64(K, dtype), np.abs(to_f64(V, dtype)), d ** -0.5)
    kd, vd = to_dev(K, dtype), to_dev(V, dtype)
    for p in low:
        vd[512 * p + 7, :, 3] = float("inf")
    L = Layer(dtype, HQ, HKV, d, 5e5, max_ctx=n, max_prompt=1)
    for key, value in {**knobs, "attn_part_tiles": tiles}.items():
        L.set_tuning(key, value)
    assert L.attention_plan(rows, n)["parts"] == parts
    out, lse = L.recompute_attention(to_dev(q, dtype), torch.from_numpy(pos.astype(np.int32)).to(DEV), kd, vd, return_lse=True)
    torch.cuda.synchronize()
    L.close()
    assert_attention_close(to_host_f64(out, dtype), ref, ref_abs, dtype, lse.cpu().numpy().astype(np.float64), lse_ref)
