"""GPU parity of the matrix kernels at the edges of their tiles and dispatch rules, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import infoflow_oracle as O
from tests.helpers import DEV, score_tol, to_dev, to_host_f64
from workloads import to_f64, to_storage

pytestmark = pytest.mark.gpu


def gauss(seed, stream, shape, dtype):
    g = np.random.Generator(np.random.Philox(key=[seed, stream]))
    return to_storage(g.standard_normal(shape), dtype)


# ---------------------------------------------------------------------------
# stage 2.  Query rows per kv head (m * H_q / H_kv) choose the block: at most 32 rows, 128, 256 or 512; contexts end
# inside and at the end of a tile of 64 (128 for the smallest block) keys; the last case gives a block more than the
# 2048 keys whose sums it keeps at a time.
# ---------------------------------------------------------------------------
SCORE_EDGES = [  # n_ctx, m, H_q, H_kv, with the prompt's own keys
    (1, 1, 8, 8, True), (127, 5, 8, 2, True), (128, 8, 16, 4, False), (129, 31, 4, 4, True), (700, 33, 4, 4, False),
    (64, 31, 8, 2, True), (65, 32, 8, 2, False), (191, 33, 14, 2, True), (192, 64, 8, 2, True), (63, 65, 8, 2, False),
    (1000, 80, 8, 2, True), (320, 96, 28, 4, True), (449, 127, 16, 4, False), (2100, 128, 16, 4, True),
    (333, 257, 8, 2, True), (4300, 512, 32, 8, False), (4300, 2048, 32, 32, False),
]


@pytest.mark.parametrize("n,m,hq,hkv,own", SCORE_EDGES, ids=[f"N{c[0]}-M{c[1]}-{c[2]}q{c[3]}kv{'-own' if c[4] else ''}" for c in SCORE_EDGES])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)], ids=["bf16-128", "bf16-64", "f32-64", "f32-128"])
def test_score_matrix_kernels_at_their_edges(dtype, d, n, m, hq, hkv, own):
    """Logits have a standard deviation of one.  Products are exact in fp32, so a logit's error is at most that of a
    d-term fp32 sum, d 2^-24 sum|q k| / sqrt(d) < 6e-5 for d = 128, and enters a score twice (its own term, the
    normaliser)."""
    from paper_2603_05353_amd import Layer
    K, q = gauss(n + m, 1, (n, hkv, d), dtype), gauss(n + m, 2, (m, hq, d), dtype)
    kp = gauss(n + m, 3, (m, hkv, d), dtype) if own else None
    ref = O.score_tokens(to_f64(K, dtype), to_f64(q, dtype), d ** -0.5, k_prompt=None if kp is None else to_f64(kp, dtype))
    L = Layer(dtype, hq, hkv, d, 5e5, max_ctx=n, max_prompt=m)
    kd, qd, kpd = to_dev(K, dtype), to_dev(q, dtype), None if kp is None else to_dev(kp, dtype)
    s = L.score_tokens(kd, qd, k_prompt=kpd)
    again = L.score_tokens(kd, qd, k_prompt=kpd)
    s2 = L.score_tokens(kd, qd, k_prompt=kpd, scores=torch.ones(n, device=DEV), accumulate=True)
    torch.cuda.synchronize()
    got = s.cpu().numpy().astype(np.float64)
    assert (np.abs(got - ref) <= score_tol(ref, m, 1.2e-4)).all()
    assert torch.equal(s, again)  # no order of the blocks shows
    assert torch.equal(s2, s + 1.0)
    L.close()


@pytest.mark.parametrize("dtype,hq,hkv,d,n,m", [("bf16", 16, 16, 128, 20000, 4), ("bf16", 16, 16, 128, 20000, 30), ("bf16", 16, 16, 128, 32768, 64),
                                               ("bf16", 32, 8, 128, 32768, 4), ("f32", 16, 16, 128, 9000, 20), ("bf16", 16, 16, 64, 20000, 100)])
def test_scores_of_few_query_rows_do_not_depend_on_timing(dtype, hq, hkv, d, n, m):
    """Few query rows: a tile's products take less time than its keys need to arrive, so the wavefronts of a block drift apart.  A wavefront
    that ends a key range must not overwrite column sums that another one has yet to collect."""
    from paper_2603_05353_amd import Layer
    K, q = gauss(n + m, 4, (n, hkv, d), dtype), gauss(n + m, 5, (m, hq, d), dtype)
    ref = O.score_tokens(to_f64(K, dtype), to_f64(q, dtype), d ** -0.5)
    L = Layer(dtype, hq, hkv, d, 5e5, max_ctx=n, max_prompt=m)
    kd, qd = to_dev(K, dtype), to_dev(q, dtype)
    runs = torch.stack([L.score_tokens(kd, qd) for _ in range(20)])
    torch.cuda.synchronize()
    assert (np.abs(runs[0].cpu().numpy().astype(np.float64) - ref) <= score_tol(ref, m, 1.2e-4)).all()
    assert (runs == runs[0]).all()
    L.close()


# ---------------------------------------------------------------------------
# stage 4 with 32-bit sums: heads of 64 in bf16 (a probability is the sum of two bf16 numbers, 16 bits), fp32.  Caches end inside and at the end of a 64-row tile, rows
# fill one and several blocks of 128 query columns; the knobs cut the kv axis and the rows.
# ---------------------------------------------------------------------------
ATTENTION_EDGES = [  # n_kv, rows, H_q, H_kv, knobs
    (1, 1, 8, 8, {}), (63, 63, 8, 2, {}), (64, 20, 14, 2, {}), (65, 65, 4, 4, {}), (130, 129, 4, 4, {"attn_part_tiles": 1}),
    (513, 40, 32, 1, {}), (1000, 150, 8, 8, {}), (1000, 150, 8, 8, {"attn_split_parts": 1}),
    (1500, 300, 16, 4, {"attn_max_row_blocks": 3, "attn_part_tiles": 5}), (2300, 7, 28, 4, {}),
]


@pytest.mark.parametrize("n,rows,hq,hkv,knobs", ATTENTION_EDGES, ids=[f"N{c[0]}-R{c[1]}-{c[2]}q{c[3]}kv-{len(c[4])}knobs" for c in ATTENTION_EDGES])
@pytest.mark.parametrize("gain", [1.0, 6.0, 30.0], ids=["flat", "peaked", "second-sweep"])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)], ids=["bf16-64", "f32-64", "f32-128"])
def test_attention_with_split_and_fp32_probabilities(dtype, d, gain, n, rows, hq, hkv, knobs):
    """fp32 logits of up to L = 8 gain: their error, d 2^-24 sum|q k| / sqrt(d) <= 128 x 2^-24 x 7.3 x gain = 5.6e-5 gain,
    enters a weight once and the normaliser once.  bf16 (8 significant bits, so rounding moves a value by at most 2^-8 of
    it) adds the split of a probability p into two bf16 numbers -- the remainder of the first is at most 2^-8 p, rounding
    it moves it by at most 2^-17 p -- and one rounding of the result, 2^-8 of it; not the 2^-8 of every probability that
    bf16 weights would cost."""
    from paper_2603_05353_amd import Layer
    K, V = gauss(n + rows, 4, (n, hkv, d), dtype), gauss(n + rows, 5, (n, hkv, d), dtype)
    g = np.random.Generator(np.random.Philox(key=[n + rows, 6]))
    q = to_storage(gain * g.standard_normal((rows, hq, d)), dtype)
    pos = np.sort(g.choice(n, size=rows, replace=False)).astype(np.int64)
    pos[-1] = n - 1
    K64, V64, q64 = to_f64(K, dtype), to_f64(V, dtype), to_f64(q, dtype)
    ref, lse_ref = O.recompute_attention(q64, pos, K64, V64, d ** -0.5)
    ref_abs, _ = O.recompute_attention(q64, pos, K64, np.abs(V64), d ** -0.5)
    L = Layer(dtype, hq, hkv, d, 5e5, max_ctx=n, max_prompt=1)
    for key, value in knobs.items():
        L.set_tuning(key, value)
    out, lse = L.recompute_attention(to_dev(q, dtype), torch.from_numpy(pos.astype(np.int32)).to(DEV), to_dev(K, dtype),
                                     to_dev(V, dtype), return_lse=True)
    torch.cuda.synchronize()
    rel = 2 * 5.6e-5 * gain
    bound = rel * ref_abs + ((2.0 ** -17 + rel * 2.0 ** -8) * ref_abs + 2.0 ** -8 * np.abs(ref) if dtype == "bf16" else 0.0)
    assert (np.abs(to_host_f64(out, dtype) - ref) <= bound).all()
    assert (np.abs(lse.cpu().numpy() - lse_ref) <= 5.6e-5 * gain + 1e-6 * np.abs(lse_ref) + 1e-6).all()
    L.close()


@pytest.mark.parametrize("n,rows,hq,hkv", [(200, 40, 16, 4), (1600, 100, 32, 8), (8000, 120, 14, 2)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)], ids=["f32-64", "f32-128", "bf16-64"])
def test_attention_is_as_exact_as_the_alu_kernel(dtype, d, n, rows, hq, hkv):
    """The layer types that have an ALU kernel with 32-bit sums: the matrix kernel's error against 64 bits is no larger (the
    result of a bf16 layer, whose rounding outweighs the split of the probabilities by a factor of 1000: not by one part in
    10000)."""
    from paper_2603_05353_amd import Layer
    K, V, q = gauss(n, 7, (n, hkv, d), dtype), gauss(n, 8, (n, hkv, d), dtype), gauss(n, 9, (rows, hq, d), dtype)
    g = np.random.Generator(np.random.Philox(key=[n, 10]))
    pos = np.sort(g.choice(n, size=rows, replace=False)).astype(np.int64)
    ref, lse_ref = O.recompute_attention(to_f64(q, dtype), pos, to_f64(K, dtype), to_f64(V, dtype), d ** -0.5)
    err = []
    for flags in (0, 1):
        L = Layer(dtype, hq, hkv, d, 5e5, max_ctx=n, max_prompt=1, flags=flags)
        out, lse = L.recompute_attention(to_dev(q, dtype), torch.from_numpy(pos.astype(np.int32)).to(DEV), to_dev(K, dtype),
                                         to_dev(V, dtype), return_lse=True)
        torch.cuda.synchronize()
        L.close()
        err.append([np.linalg.norm(a - b) for a, b in ((lse.cpu().numpy(), lse_ref), (to_host_f64(out, dtype), ref))])
    assert err[0][0] <= err[1][0] and err[0][1] <= err[1][1] * (1.0001 if dtype == "bf16" else 1.0), err
