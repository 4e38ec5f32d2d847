"""GPU parity of the matrix kernels at the edges of their tiles and dispatch rules, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import infoflow_oracle as O
from tests.helpers import DEV, score_tol, to_dev
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
