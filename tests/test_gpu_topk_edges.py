"""Top-k at the edges of its kernels, their chunks (2048 and 4096 keys) and budgets, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import infoflow_oracle as O
from paper_2603_05353_amd import Layer
from tests.helpers import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32769, 34816, 36863, 36864, 36865, 131072, 133119, 133120, 133121, 135167, 135168, 135169, 200003])  # 131073: other kernels
@pytest.mark.parametrize("kind", ["one-bin", "two-values", "infinities", "wide"])
def test_topk_over_many_workgroups(n, kind):
    g = np.random.Generator(np.random.Philox(key=[n, 3]))
    s = {"one-bin": lambda: np.float32(0.5) + g.integers(0, 900, n).astype(np.float32) * np.float32(2.0 ** -24),  # the last digit only
         "two-values": lambda: np.where(g.random(n) < 0.5, -1.0, 2.0),
         "infinities": lambda: np.where(g.random(n) < 0.01, np.inf, np.where(g.random(n) < 0.01, -np.inf, g.standard_normal(n))),
         "wide": lambda: np.exp(12.0 * g.standard_normal(n)) * np.where(g.random(n) < 0.3, -1.0, 1.0)}[kind]().astype(np.float32)
    L = Layer("bf16", 32, 8, 128, 5e5, max_ctx=n, max_prompt=1)
    for shift in (0, 1):  # the second one starts 4 bytes into an allocation: no 16-byte loads
        buf = torch.empty(n + 1, dtype=torch.float32, device=DEV)
        d = buf[shift:shift + n]
        d.copy_(torch.from_numpy(s))
        for k in (1, 777, n // 7, n - 1, n):
            idx = L.select_topk(d, k=k)
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy().astype(np.int64), O.select_topk(s, k)), (k, shift)
    L.close()


@pytest.mark.parametrize("n", [1, 31, 33, 8191, 8192, 8193, 20001, 32768])
@pytest.mark.parametrize("bits", [1, 14, 15, 16, 17, 18, 20, 24, 28, 30, 31])
def test_topk_in_one_workgroup_stops_when_every_key_left_is_taken(n, bits):
    """The descent ends once the k-th key differs from the next one in the bits seen so far: keys that agree in all but
    the highest `bits` bits below the sign, so that it ends before, at and after each look, or at the last bit; with ties,
    with both signs and with fewer keys than the padding of the last word."""
    g = np.random.Generator(np.random.Philox(key=[n, bits]))
    u = g.integers(0, 2 ** bits, n, dtype=np.int64) << (31 - bits)
    u = np.where(u >= 0x7F800000, u - 0x40000000 if bits > 1 else 0, u) | (g.integers(0, 2, n, dtype=np.int64) << 31)
    s = np.where(np.isfinite(x := u.astype(np.uint32).view(np.float32)), x, np.float32(1.0))
    L = Layer("bf16", 32, 8, 128, 5e5, max_ctx=n, max_prompt=1)
    d = torch.from_numpy(s).to(DEV)
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    for k in sorted({1, max(1, n // 7), max(1, n - 1), n}):
        # above 8192 scores the one workgroup serves the entry point that allocates nothing, the other one takes two launches
        for idx in (L.select_topk(d, k=k), L.select_topk_noalloc(d, out, k=k)):
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy().astype(np.int64), O.select_topk(s, k)), k
    L.close()


def sampled(n):
    """The places of the 4096 scores that the bracket of the two-launch select is taken from."""
    return np.array([((x << 32 | x * 2654435769 % 2 ** 32) * n // 4096) >> 32 for x in range(4096)])


def spread(n, kind):
    g = np.random.Generator(np.random.Philox(key=[n, 5]))
    if kind.startswith("sample"):  # the sample holds only keys below / above the threshold: it lies outside the bracket
        s = g.random(n)
        s[sampled(n)] += {"sample-low": -2.0, "sample-high": 2.0}[kind]
        return s
    return {"near-uniform": lambda: 1.0 + 1e-4 * g.standard_normal(n), "all-equal": lambda: np.full(n, -3.0),
            "few-values": lambda: g.integers(0, 40, n), "ascending": lambda: np.sort(g.standard_normal(n)),
            "mostly-zeros": lambda: np.where(g.random(n) < 0.95, 0.0, g.random(n)), "far-outliers": lambda: np.where(np.arange(n) % 9973 == 5, 1e30 * g.standard_normal(n), 1e-6 * (1 + 1e-3 * g.random(n))),
            "highest-keys": lambda: np.where(g.random(n) < 0.2, np.inf, 3e38 * g.random(n)),
            "lowest-keys": lambda: np.where(g.random(n) < 0.9, -np.inf, -3e38 * g.random(n))}[kind]()


@pytest.mark.parametrize("n", [8193, 12288, 12289, 32768, 131071, 131072, 131073])
@pytest.mark.parametrize("kind", ["near-uniform", "all-equal", "few-values", "ascending", "mostly-zeros", "far-outliers", "highest-keys", "lowest-keys",
                                  "sample-low", "sample-high"])
def test_topk_in_two_launches(n, kind):
    """One to 32 chunks of 4096 scores and one score more on either side, keys that leave the bracket empty, full or beside
    the threshold, and all of them through the entry point whose work memory is shared, too."""
    s = spread(n, kind).astype(np.float32)
    L = Layer("bf16", 32, 8, 128, 5e5, max_ctx=n, max_prompt=1)
    buf = torch.empty(n + 1, dtype=torch.float32, device=DEV)
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    for shift in (0, 1):  # the second one starts 4 bytes into an allocation: no 16-byte loads
        d = buf[shift:shift + n]
        d.copy_(torch.from_numpy(s))
        for k in (1, 64, n // 9, n // 2, n - 4096, n - 1, n):
            ref = O.select_topk(s, k)
            for idx in (L.select_topk(d, k=k), L.select_topk_noalloc(d, out, k=k)):
                torch.cuda.synchronize()
                assert np.array_equal(idx.cpu().numpy().astype(np.int64), ref), (k, shift)
    L.close()


@pytest.mark.parametrize("n", [700, 8192, 8193, 20001, 32768])
@pytest.mark.parametrize("shift", [0, 1, -5], ids=["same-start", "one-on", "five-before"])
def test_topk_into_the_memory_of_the_scores(n, shift):
    """Up to 32768 scores all of them are read before an index is written."""
    g = np.random.Generator(np.random.Philox(key=[n, 6]))
    s = (1.0 + 0.01 * g.standard_normal(n)).astype(np.float32)
    L = Layer("bf16", 32, 8, 128, 5e5, max_ctx=n, max_prompt=1)
    buf = torch.empty(n + 16, dtype=torch.float32, device=DEV)
    for k in (n // 7, n - 6):
        ref = O.select_topk(s, k)
        for call in (L.select_topk, L.select_topk_noalloc):
            d = buf[8:8 + n]
            d.copy_(torch.from_numpy(s))
            out = buf.view(torch.int32)[8 + shift:8 + shift + k]
            call(d, idx_out=out, k=k)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().astype(np.int64), ref), k
    L.close()
