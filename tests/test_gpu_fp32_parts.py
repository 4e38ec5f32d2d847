"""fp32 attention whose products run on sums of three bf16 numbers: sizes around a kv tile, and numbers whose parts are not
enough (infinities, the ends of the exponent range), where the sweep is repeated with fp32 operands."""
import numpy as np
import pytest
import torch

from oracle import infoflow_oracle as O
from paper_2603_05353_amd import Layer
from tests.helpers import DEV, attention_error_bound

pytestmark = pytest.mark.gpu


def attend(q, pos, K, V, knobs):
    (n, hkv, d), hq = K.shape, q.shape[1]
    L = Layer("f32", hq, hkv, d, 5e5, max_ctx=n, max_prompt=1)
    for key, value in knobs.items():
        L.set_tuning(key, value)
    out, lse = L.recompute_attention(*(torch.from_numpy(x).to(DEV) for x in (q, pos.astype(np.int32), K, V)), return_lse=True)
    torch.cuda.synchronize()
    L.close()
    return out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)


def case(n, d, hq=8, hkv=2, rows=40):
    g = np.random.Generator(np.random.Philox(key=[n, d]))
    K, V = (g.standard_normal((n, hkv, d)).astype(np.float32) for _ in range(2))
    rows = min(rows, n)
    pos = np.sort(g.choice(n, size=rows, replace=False)).astype(np.int64)
    pos[-1] = n - 1
    return K, V, g.standard_normal((rows, hq, d)).astype(np.float32), pos


def reference(q, pos, K, V, d):
    q, K, V = (x.astype(np.float64) for x in (q, K, V))
    ref, lse = O.recompute_attention(q, pos, K, V, d ** -0.5)
    return ref, lse, O.recompute_attention(q, pos, K, np.abs(V), d ** -0.5)[0]


@pytest.mark.parametrize("knobs", [{}, {"attn_part_tiles": 1}, {"attn_split_parts": 1}, {"attn_split_parts": 1, "attn_exact_sweep": 1}],
                         ids=["plain", "parts-of-1", "whole", "fp32-operands"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 700])
@pytest.mark.parametrize("d", [64, 128])
def test_error_is_that_of_fp32(d, n, knobs):
    """Per element: the logit's error, d terms of 2^-24 each at most, moves a weight by d 2^-24 sum|q k| / sqrt(d) <= 6e-5 in the
    worst case and by its root-mean-square, some 2^-24 |q||k| / sqrt(d) = 2^-24 sqrt(d), as a rule; 32 of these is 2.2e-5 at
    most.  Over all elements together the errors are independent: 2^-24 sqrt(d) < 6.8e-7 of the result's norm."""
    K, V, q, pos = case(n, d)
    ref, lse_ref, ref_abs = reference(q, pos, K, V, d)
    out, lse = attend(q, pos, K, V, knobs)
    err = np.abs(out - ref)
    assert (err <= attention_error_bound(ref, ref_abs, "f32")).all()
    assert np.linalg.norm(err) <= 2.0 ** -24 * np.sqrt(d) * np.linalg.norm(ref_abs)
    assert np.abs(lse - lse_ref).max() <= 1e-5


# 2.0 ** x on K, q and V: parts lost below 2^-126 (also of V alone), parts that overflow the rounding to bf16
SCALES = {"small-v": (0, 0, -118), "smaller-v": (0, 0, -122), "small-k": (-120, 120, 0), "small-q": (100, -100, 0), "large-v": (0, 0, 124)}


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("d", [64, 128])
def test_the_ends_of_the_range(d, scale):
    """Powers of two on both sides of a product change nothing.  (V at 2^-122: a value down to 2^-130 has 19 bits left, an error of
    2^-149 each on values of 2^-122.)"""
    K, V, q, pos = case(300, d)
    ref, lse_ref, ref_abs = reference(q, pos, K, V, d)
    k, x, v = SCALES[scale]
    out, lse = attend(np.ldexp(q, x), pos, np.ldexp(K, k), np.ldexp(V, v), {})
    assert (np.abs(np.ldexp(out, -v) - ref) <= attention_error_bound(ref, ref_abs, "f32") + 2.0 ** -26).all()
    assert np.abs(lse - lse_ref).max() <= 1e-5


@pytest.mark.parametrize("knobs", [{}, {"attn_part_tiles": 1}], ids=["plain", "parts-of-1"])
@pytest.mark.parametrize("d", [64, 128])
def test_keys_with_a_logit_of_minus_infinity_take_no_part(d, knobs):
    """An infinite element of a key against queries of the other sign, and the type's lowest value, whose rounding to bf16 is
    infinite: a weight of 0, as in fp32, for them and no change for the others."""
    K, V, q, pos = case(300, d)
    q[:, :, 5] = np.abs(q[:, :, 5]) + 0.5
    gone = [17, 130, 131, 299]
    K[gone, :, 5] = [[-np.inf], [-np.inf], [np.finfo(np.float32).min], [-np.inf]]
    pos[0] = 16  # a row before them all
    pos.sort()
    K64 = K.astype(np.float64)
    K64[gone, :, 5] = -1e30
    ref, lse_ref, ref_abs = reference(q, pos, K64, V, d)
    out, lse = attend(q, pos, K, V, knobs)
    assert (np.abs(out - ref) <= attention_error_bound(ref, ref_abs, "f32")).all()
    assert np.abs(lse - lse_ref).max() <= 1e-5
