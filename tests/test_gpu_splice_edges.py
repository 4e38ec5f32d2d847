"""Stage 5 where rows and blocks of its kernel do not match: bit for bit against indexing."""
import pytest
import torch

from paper_2603_05353_amd import Layer
from tests.helpers import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("values", [True, False], ids=["kv", "k-only"])
@pytest.mark.parametrize("rows", [1, 3, 4, 5, 64, 65, 333])
@pytest.mark.parametrize("dtype,hkv,d,strides", [
    ("bf16", 1, 64, None), ("bf16", 3, 128, None), ("f32", 5, 64, (5 * 64 + 8, 64)), ("bf16", 8, 128, (128, 700 * 128)),
    ("f32", 16, 128, None), ("f32", 40, 128, None)])  # 8 to 1280 vectors a row: many rows a block, one, and a row of several batches
def test_splice_of_every_row_size(dtype, hkv, d, strides, rows, values):
    n, dt = 700, {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator(device=DEV).manual_seed(rows + hkv)
    kw = {} if strides is None else dict(token_stride=strides[0], head_stride=strides[1])
    ts, hs = strides or (hkv * d, d)

    def cache():
        base = torch.randn((n - 1) * ts + (hkv - 1) * hs + d + 8, generator=g, device=DEV).to(dt)
        return base, torch.as_strided(base, (n, hkv, d), (ts, hs, 1))

    (kb, k), (vb, v) = cache(), cache()
    k_new, v_new = (torch.randn(rows, hkv, d, generator=g, device=DEV).to(dt) for _ in range(2))
    idx = torch.sort(torch.randperm(n, generator=g, device=DEV)[:rows])[0].to(torch.int32)
    keep = torch.arange(rows, device=DEV) % 7 != 3
    idx[~keep] = torch.where(torch.arange(rows, device=DEV)[~keep] % 2 == 0, -1, n).to(torch.int32)  # outside: skipped
    want = []
    for base, new in ((kb, k_new), (vb, v_new)):
        w = base.clone()
        torch.as_strided(w, (n, hkv, d), (ts, hs, 1))[idx[keep].long()] = new[keep]
        want.append(w)
    L = Layer(dtype, hkv, hkv, d, 5e5, max_ctx=n, max_prompt=1, **kw)
    L.splice_kv(k_new, v_new if values else None, idx, k, v if values else None)
    torch.cuda.synchronize()
    assert torch.equal(kb, want[0])
    if values:
        assert torch.equal(vb, want[1])
    L.close()


def test_splice_of_more_rows_than_a_grid_has_blocks():
    """2^24 + 5 rows of 264 vectors, one row a block, would be 2^32 threads and more.  Nearly all of them lie outside the cache."""
    rows, hkv, d, n = 2 ** 24 + 5, 33, 64, 1000
    if torch.cuda.mem_get_info()[0] < rows * hkv * d * 2 + (2 << 30):
        pytest.skip("needs 73 GB of device memory")
    k_new = torch.empty(rows, hkv, d, device=DEV, dtype=torch.bfloat16)
    k = torch.zeros(n, hkv, d, device=DEV, dtype=torch.bfloat16)
    idx = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
    at = torch.tensor([0, 1, 2, 3, 4095, 2 ** 23 - 1, 2 ** 23, 2 ** 24 - 1, 2 ** 24, rows - 2, rows - 1], device=DEV)
    idx[at] = 7 + 50 * torch.arange(len(at), device=DEV, dtype=torch.int32)
    k_new[at] = torch.randn(len(at), hkv, d, device=DEV).bfloat16()
    want = k.clone()
    want[idx[at].long()] = k_new[at]
    L = Layer("bf16", hkv, hkv, d, 5e5, max_ctx=n, max_prompt=1)
    L.splice_kv(k_new, None, idx, k, None)
    torch.cuda.synchronize()
    assert torch.equal(k, want)
    L.close()
    del k_new, idx
    torch.cuda.empty_cache()
