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


def scaled(K, V, q, pos, name):
    """Inputs in which single elements lie far from the rest, so that parts of them are lost below 2^-126 while the largest
    query element and the result look ordinary."""
    n, hkv, d = K.shape
    if name in ("channel-of-small-q", "channel-of-large-q"):  # logits of order one, to which that channel adds like the others
        x = 124 if name == "channel-of-small-q" else -70
        K[:, :, 5], q[:, :, 5] = np.ldexp(K[:, :, 5], x), np.ldexp(q[:, :, 5], -x)
    elif name in ("small-weights", "smaller-weights"):  # weights of about 2^-118 (2^-122) and values as large
        x = 118 if name == "small-weights" else 122
        keys = [3, 70, 71, n // 2]
        q *= 0.25
        q[:, :, 5] = 1.0
        K[keys] = 0.0
        K[keys, :, 5] = -x * np.log(2.0) * d ** 0.5
        V[keys] = np.ldexp(V[keys], x + 2)
    elif name == "values-below-a-large-sum":  # all keys but the first tile's 2^7.9 above the reference, values of 2^-118
        K[:], q[:, :, 5] = 0.0, 1.0
        K[64:, :, 5] = 7.9 * np.log(2.0) * d ** 0.5
        V[:] = np.ldexp(1.0 + np.abs(V), -118)
    elif name == "denormal-values":
        V[:] = np.ldexp(V, -137)
    elif name == "one-denormal-column":
        V[:, :, 7] = np.ldexp(V[:, :, 7], -140)
    elif name == "one-small-and-one-large-column":
        V[:, :, 7], V[:, :, 8] = np.ldexp(V[:, :, 7], -60), np.ldexp(V[:, :, 8], 60)
    elif name == "columns-of-zeros":
        V[:, :, 40:] = 0.0
        V[0] = 0.0
    return K, V, q, pos


@pytest.mark.parametrize("knobs", [{}, {"attn_part_tiles": 1}, {"attn_split_parts": 1}], ids=["plain", "parts-of-1", "whole"])
@pytest.mark.parametrize("name", ["channel-of-small-q", "channel-of-large-q", "small-weights", "smaller-weights", "values-below-a-large-sum",
                                  "denormal-values", "one-denormal-column", "one-small-and-one-large-column", "columns-of-zeros"])
@pytest.mark.parametrize("d", [64, 128])
def test_elements_far_from_the_rest(d, name, knobs):
    """The bound of fp32 arithmetic, element by element; a denormal result has an ulp of 2^-149, of which the n roundings of the
    products and the last one take 2^-145 at most after the division by the sum."""
    K, V, q, pos = scaled(*case(2048 if name == "values-below-a-large-sum" else 300, d), name)
    ref, lse_ref, ref_abs = reference(q, pos, K, V, d)
    out, lse = attend(q, pos, K, V, knobs)
    err, bound = np.abs(out - ref), attention_error_bound(ref, ref_abs, "f32") - 1e-30 + 2.0 ** -145
    worst = (err / bound).max()
    assert worst <= 1.0, worst
    assert np.abs(lse - lse_ref).max() <= 1e-5
    if name == "columns-of-zeros":
        assert not out[:, :, 40:].any()


@pytest.mark.parametrize("column", [0, 3, 4, 13, 31, 32, 46, 63, 64, 95, 101, 127])
def test_a_denormal_column_among_zeros(column):
    """Results of exactly 0 are right for the other columns, and found not to be for this one, whichever it is."""
    for d in (64, 128):
        if column >= d:
            continue
        K, V, q, pos = case(300, d)
        keep = np.ldexp(V[:, 1, column], -141)
        V[:] = 0.0
        V[:, 1, column] = keep
        ref = reference(q, pos, K, V, d)[0]
        out = attend(q, pos, K, V, {})[0]
        assert np.abs(out - ref).max() <= 2.0 ** -145
        assert ref.any() and out[:, 4:, column].any()


@pytest.mark.parametrize("last", [0, 7, 62])
@pytest.mark.parametrize("d", [64, 128])
def test_large_values_that_nobody_sees_change_nothing(d, last):
    """Rows behind the last position share a tile with it: whatever they hold, the result is the same bit for bit (a repeated sweep would
    round otherwise); one that is seen is found."""
    n = 320
    K, V, q, pos = case(n, d)
    pos[:] = np.arange(256 + last + 1 - len(pos), 256 + last + 1)
    want = attend(q, pos, K, V, {})
    V[256 + last + 1:] = np.float32(3e30)
    got = attend(q, pos, K, V, {})
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    V[256 + last] = np.float32(3e30)
    ref, _, ref_abs = reference(q, pos, K, V, d)
    assert (np.abs(attend(q, pos, K, V, {})[0] - ref) <= attention_error_bound(ref, ref_abs, "f32")).all()
