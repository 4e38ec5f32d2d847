"""Stage 4: the kernel with 256 query columns per workgroup (bf16, heads of 128) at the edges of its tiles against the fp64
oracle, the rules that choose it and cut launches, and the wait states around its hand-placed matrix instructions."""
import os
import re
import subprocess

import numpy as np
import pytest
import torch

import paper_2603_05353_amd.binding as B
from oracle import infoflow_oracle as O
from paper_2603_05353_amd import build
from tests.helpers import DEV, assert_attention_close, to_dev, to_host_f64
from workloads import to_f64, to_storage

D = 128

# Caches end inside and at the end of a 64-row tile (tiles at the end are staged from 64 rows before the end), with one to
# many tiles, which covers every position in the ring of four LDS stages and both halves of the unrolled loop; rows fill
# parts of one block of 256 query columns, one whole and several; cuts leave whole parts, remainders and empty parts.
EDGES = [  # n_kv, rows, H_q, H_kv, knobs, (token stride, head stride) or None
    (64, 1, 8, 8, {}, None), (65, 64, 8, 2, {}, None), (127, 37, 28, 4, {}, (4 * 128 + 8, 128)), (128, 128, 1, 1, {}, None),
    (129, 129, 4, 2, {"attn_part_tiles": 1}, None), (193, 8, 32, 1, {}, None), (256, 256, 1, 1, {"attn_part_tiles": 2}, None),
    (257, 257, 1, 1, {"attn_part_tiles": 2}, (256, 128)), (320, 65, 16, 4, {"attn_part_tiles": 3}, None),
    (447, 9, 32, 1, {"attn_part_tiles": 3}, None), (512, 100, 6, 2, {"attn_split_parts": 4}, (128, 513 * 128)),
    (1000, 300, 8, 2, {}, None), (1000, 300, 8, 2, {"attn_max_row_blocks": 3, "attn_part_tiles": 5}, None),
    (1087, 40, 40, 8, {"attn_part_tiles": 4}, None), (1088, 520, 2, 2, {"attn_exact_sweep": 1}, None),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,rows,hq,hkv,knobs,layout", EDGES, ids=[f"N{c[0]}-R{c[1]}-{c[2]}q{c[3]}kv-{len(c[4])}knobs" for c in EDGES])
@pytest.mark.parametrize("gain", [1.0, 6.0, 30.0], ids=["flat", "peaked", "second-sweep"])
def test_wide_kernel_at_its_edges(gain, n, rows, hq, hkv, knobs, layout):
    """The bounds are those of every bf16 attention test (tests/helpers.py): one rounding of each probability, one of the
    result.  A row position outside the cache gives zeros and leaves the other rows alone."""
    g = np.random.Generator(np.random.Philox(key=[n + rows, 8]))
    K, V = (to_storage(g.standard_normal((n, hkv, D)) * s, "bf16") for s in (0.5, 0.5))
    q = to_storage(gain * 0.5 * g.standard_normal((rows, hq, D)), "bf16")
    pos = np.sort(g.choice(n, size=rows, replace=False)).astype(np.int64)
    pos[-1] = n - 1
    K64, V64, q64 = to_f64(K, "bf16"), to_f64(V, "bf16"), to_f64(q, "bf16")
    ref, lse_ref = O.recompute_attention(q64, pos, K64, V64, D ** -0.5)
    ref_abs, _ = O.recompute_attention(q64, pos, K64, np.abs(V64), D ** -0.5)
    kw = {} if layout is None else dict(token_stride=layout[0], head_stride=layout[1])
    L = B.Layer("bf16", hq, hkv, D, 5e5, max_ctx=n, max_prompt=1, **kw)
    for key, value in {**knobs, "attn_wide": 1}.items():
        L.set_tuning(key, value)

    def cache(x):
        if layout is None:
            return to_dev(x, "bf16")
        base = torch.full(((n - 1) * layout[0] + (hkv - 1) * layout[1] + D,), float("nan"), dtype=torch.bfloat16, device=DEV)
        c = torch.as_strided(base, (n, hkv, D), (*layout, 1))
        c.copy_(to_dev(x, "bf16"))
        return c

    kd, vd, qd, pd = cache(K), cache(V), to_dev(q, "bf16"), torch.from_numpy(pos.astype(np.int32)).to(DEV)
    out, lse = L.recompute_attention(qd, pd, kd, vd, return_lse=True)
    torch.cuda.synchronize()
    assert_attention_close(to_host_f64(out, "bf16"), ref, ref_abs, "bf16", lse.cpu().numpy(), lse_ref)
    if rows > 1:
        bad = pd.clone()
        bad[rows // 2] = n
        out2 = L.recompute_attention(qd, bad, kd, vd)
        torch.cuda.synchronize()
        assert not out2[rows // 2].any()
        keep = [r for r in range(rows) if r != rows // 2]
        assert_attention_close(to_host_f64(out2, "bf16")[keep], ref[keep], ref_abs[keep], "bf16")
    L.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n,rows", [(8200, 1700), (16500, 2500)], ids=["cut", "cut-longer"])
def test_wide_kernel_where_the_rule_chooses_it(n, rows):
    """The library's own choice (the wide kernel, cut) and the same rows on the narrow kernel, against the oracle and each
    other."""
    g = np.random.Generator(np.random.Philox(key=[n + rows, 9]))
    K, V = (to_storage(g.standard_normal((n, 8, D)) * 0.5, "bf16") for _ in range(2))
    q = to_storage(g.standard_normal((rows, 32, D)), "bf16")
    pos = np.sort(g.choice(n, size=rows, replace=False)).astype(np.int64)
    L = B.Layer("bf16", 32, 8, D, 5e5, max_ctx=n, max_prompt=1)
    args = (to_dev(q, "bf16"), torch.from_numpy(pos.astype(np.int32)).to(DEV), to_dev(K, "bf16"), to_dev(V, "bf16"))
    assert L.attention_plan(rows, n)["parts"] > 1
    pick = np.unique(np.concatenate([[0, 1, rows - 1], g.choice(rows, 24, replace=False)]))
    q64, K64, V64 = to_f64(q, "bf16")[pick], to_f64(K, "bf16"), to_f64(V, "bf16")
    ref, lse_ref = O.recompute_attention(q64, pos[pick], K64, V64, D ** -0.5)
    ref_abs, _ = O.recompute_attention(q64, pos[pick], K64, np.abs(V64), D ** -0.5)
    for wide in (0, 2):
        L.set_tuning("attn_wide", wide)
        out, lse = L.recompute_attention(*args, return_lse=True)
        torch.cuda.synchronize()
        assert_attention_close(to_host_f64(out, "bf16")[pick], ref, ref_abs, "bf16", lse.cpu().numpy()[pick], lse_ref)
    L.close()


@pytest.mark.gpu
def test_a_cut_of_the_wide_kernel_does_not_round_other_probabilities():
    """Every part takes its reference exponent from key 0, so the probabilities are rounded as without a cut and only the
    order of 32-bit sums differs: a relative 1e-6 of a result, which moves it to another bf16 number (a relative 2^-8
    apart at least) for one element in 2000 at most.  (References of their own: one in six.)"""
    n, rows = 8200, 1700
    g = np.random.Generator(np.random.Philox(key=[n + rows, 11]))
    q, K, V = (to_dev(to_storage(g.standard_normal(s) * a, "bf16"), "bf16") for s, a in (((rows, 32, D), 1.0), ((n, 8, D), 0.5), ((n, 8, D), 1.0)))
    pos = torch.from_numpy(np.sort(g.choice(n, size=rows, replace=False)).astype(np.int32)).to(DEV)
    outs = []
    for knobs in ({"attn_split_parts": 1}, {}, {"attn_part_tiles": 40}):
        L = B.Layer("bf16", 32, 8, D, 5e5, max_ctx=n, max_prompt=1)
        for key, value in {"attn_wide": 1, **knobs}.items():
            L.set_tuning(key, value)
        assert (L.attention_plan(rows, n)["parts"] > 1) == (knobs != {"attn_split_parts": 1})
        outs.append(L.recompute_attention(q, pos, K, V))
        torch.cuda.synchronize()
        L.close()
    for out in outs[1:]:
        assert (out != outs[0]).double().mean().item() <= 5e-4


@pytest.mark.gpu
def test_blocks_that_are_all_long_are_not_cut():
    """The rows of a long prompt at the end of the cache, one block or less per CU: bit for bit the launch without a cut,
    while as many rows spread over the cache are cut."""
    n, rows = 8200, 1700
    g = np.random.Generator(np.random.Philox(key=[n + rows, 13]))
    q64, K64, V64 = (g.standard_normal(s) for s in ((rows, 32, D), (n, 8, D), (n, 8, D)))
    q, K, V = (to_storage(x, "bf16") for x in (q64, K64, V64))
    end, spread = np.arange(n - rows, n), np.sort(g.choice(n, size=rows, replace=False))
    args = to_dev(q, "bf16"), to_dev(K, "bf16"), to_dev(V, "bf16")
    outs = {}
    for split in (0, 1):
        L = B.Layer("bf16", 32, 8, D, 5e5, max_ctx=n, max_prompt=1)
        L.set_tuning("attn_wide", 1)
        L.set_tuning("attn_split_parts", split)
        assert (L.attention_plan(rows, n)["parts"] > 1) == (split == 0)
        for name, pos in (("end", end), ("spread", spread)):
            out, lse = L.recompute_attention(args[0], torch.from_numpy(pos.astype(np.int32)).to(DEV), *args[1:], return_lse=True)
            torch.cuda.synchronize()
            outs[name, split] = out, lse
        L.close()
    assert torch.equal(outs["end", 0][0], outs["end", 1][0]) and torch.equal(outs["end", 0][1], outs["end", 1][1])
    assert not torch.equal(outs["spread", 0][0], outs["spread", 1][0])
    pick = np.sort(g.choice(rows, 16, replace=False))
    ref, lse_ref = O.recompute_attention(to_f64(q, "bf16")[pick], end[pick], to_f64(K, "bf16"), to_f64(V, "bf16"), D ** -0.5)
    ref_abs, _ = O.recompute_attention(to_f64(q, "bf16")[pick], end[pick], to_f64(K, "bf16"), np.abs(to_f64(V, "bf16")), D ** -0.5)
    out, lse = outs["end", 0]
    assert_attention_close(to_host_f64(out, "bf16")[pick], ref, ref_abs, "bf16", lse.cpu().numpy()[pick], lse_ref)


@pytest.mark.gpu
@pytest.mark.parametrize("parts", [2, 3, 4, 5, 8])
def test_blocks_that_are_all_long_are_not_cut_into_any_number_of_parts(parts):
    """256 workgroups on rows at the end of the cache, for which the kernel drops the cut that the knob asks for: the workgroups of
    every part but one have nothing to do, whatever their number."""
    n, rows, heads = 4096, 1024, 64
    g = torch.Generator(device=DEV).manual_seed(parts)
    K, V = (torch.randn(n, heads, D, device=DEV, generator=g).to(torch.bfloat16) for _ in range(2))
    q = torch.randn(rows, heads, D, device=DEV, generator=g).to(torch.bfloat16)
    pos = torch.arange(n - rows, n, dtype=torch.int32, device=DEV)
    results = []
    for p in (1, parts):
        L = B.Layer("bf16", heads, heads, D, 5e5, max_ctx=n, max_prompt=1)
        L.set_tuning("attn_wide", 1)
        L.set_tuning("attn_split_parts", p)
        assert L.attention_plan(rows, n)["parts"] == p
        out = torch.full_like(q, float("nan"))
        _, lse = L.recompute_attention(q, pos, K, V, out=out, return_lse=True)
        torch.cuda.synchronize()
        L.close()
        results.append((out, lse))
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])
    assert torch.isfinite(results[0][0]).all()


@pytest.mark.gpu
@pytest.mark.parametrize("part_tiles", [36, 24, 18, 14, 9, 8, 2, 1])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)], ids=["bf16-128", "bf16-64", "f32-64"])
def test_merge_of_two_to_71_parts(dtype, d, part_tiles):
    """Every branch of the merge: 2, 3, 4, 6, 8, 9, 36 and 71 parts, of which the rows at the front see only the first
    ones, with peaked logits whose largest lies in any part."""
    n, rows, hq, hkv = 4500, 13, 8, 4
    g = np.random.Generator(np.random.Philox(key=[part_tiles, 10]))
    K, V = (to_storage(g.standard_normal((n, hkv, d)) * 0.5, dtype) for _ in range(2))
    q = to_storage(6.0 * g.standard_normal((rows, hq, d)), dtype)
    pos = np.sort(g.choice(n, size=rows, replace=False)).astype(np.int64)
    pos[0], pos[1], pos[-1] = 0, 70, n - 1
    q64, K64, V64 = to_f64(q, dtype), to_f64(K, dtype), to_f64(V, dtype)
    ref, lse_ref = O.recompute_attention(q64, pos, K64, V64, d ** -0.5)
    ref_abs, _ = O.recompute_attention(q64, pos, K64, np.abs(V64), d ** -0.5)
    L = B.Layer(dtype, hq, hkv, d, 5e5, max_ctx=n, max_prompt=1)
    L.set_tuning("attn_part_tiles", part_tiles)
    assert L.attention_plan(rows, n)["parts"] == -(-71 // part_tiles)
    out, lse = L.recompute_attention(to_dev(q, dtype), torch.from_numpy(pos.astype(np.int32)).to(DEV), to_dev(K, dtype),
                                     to_dev(V, dtype), return_lse=True)
    torch.cuda.synchronize()
    assert_attention_close(to_host_f64(out, dtype), ref, ref_abs, dtype, lse.cpu().numpy(), lse_ref)
    L.close()


@pytest.mark.gpu
@pytest.mark.parametrize("part_tiles", [18, 12, 9], ids=["2-parts", "3-parts", "4-parts"])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)], ids=["bf16-128", "bf16-64", "f32-64", "f32-128"])
def test_merge_of_many_rows(dtype, d, part_tiles):
    """16800 (row, head) pairs in two to four parts take the merge with 16 lanes a pair, four consecutive pairs a wavefront: 14
    heads, so that they straddle rows, and rows at the front and outside the cache, which need no merge or get zeros."""
    n, rows, hq, hkv = 2300, 1200, 14, 2
    g = np.random.Generator(np.random.Philox(key=[part_tiles, 12]))
    K, V = (to_storage(g.standard_normal((n, hkv, d)) * 0.5, dtype) for _ in range(2))
    q = to_storage(6.0 * g.standard_normal((rows, hq, d)), dtype)
    pos = np.sort(g.choice(n, size=rows, replace=False)).astype(np.int64)
    pos[-1] = n - 1
    asked = pos.copy()
    asked[700] = -1
    L = B.Layer(dtype, hq, hkv, d, 5e5, max_ctx=n, max_prompt=1)
    L.set_tuning("attn_part_tiles", part_tiles)
    assert L.attention_plan(rows, n)["parts"] == 36 // part_tiles
    out, lse = L.recompute_attention(to_dev(q, dtype), torch.from_numpy(asked.astype(np.int32)).to(DEV), to_dev(K, dtype),
                                     to_dev(V, dtype), return_lse=True)
    torch.cuda.synchronize()
    L.close()
    out, lse = to_host_f64(out, dtype), lse.cpu().numpy()
    assert not out[700].any() and not lse[700].any()
    pick = np.unique(np.concatenate([[0, 1, 699, 701, rows - 2, rows - 1], np.delete(g.choice(rows, 60, replace=False), 0)]))
    pick = pick[pick != 700]
    q64, K64, V64 = to_f64(q, dtype)[pick], to_f64(K, dtype), to_f64(V, dtype)
    ref, lse_ref = O.recompute_attention(q64, pos[pick], K64, V64, d ** -0.5)
    ref_abs, _ = O.recompute_attention(q64, pos[pick], K64, np.abs(V64), d ** -0.5)
    assert_attention_close(out[pick], ref, ref_abs, dtype, lse[pick], lse_ref)


@pytest.mark.gpu
@pytest.mark.parametrize("part_tiles,parts", [(8, 9), (5, 15), (5, 14), (4, 17)], ids=["9-parts", "15-parts", "14-parts-odd-rows", "17-parts"])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128)], ids=["bf16-128", "bf16-64", "f32-128"])
def test_merge_of_nine_and_more_parts_of_many_columns(dtype, d, part_tiles, parts):
    """More than 2048 (row, head) pairs: up to 16 parts go through one wavefront in rounds of eight, more through four; 7 query heads per
    kv head leave two of a block's 128 columns empty, and the last block of rows holds a few."""
    n, rows, hq, hkv = 64 * part_tiles * parts - 70, 149, 14, 2
    g = np.random.Generator(np.random.Philox(key=[parts, 18]))
    K, V = (to_storage(g.standard_normal((n, hkv, d)) * 0.5, dtype) for _ in range(2))
    q = to_storage(6.0 * g.standard_normal((rows, hq, d)), dtype)
    pos = np.sort(g.choice(n, size=rows, replace=False)).astype(np.int64)
    pos[0], pos[-1] = 0, n - 1
    L = B.Layer(dtype, hq, hkv, d, 5e5, max_ctx=n, max_prompt=1)
    L.set_tuning("attn_part_tiles", part_tiles)
    L.set_tuning("attn_wide", 2)
    assert L.attention_plan(rows, n)["parts"] == parts
    out, lse = L.recompute_attention(to_dev(q, dtype), torch.from_numpy(pos.astype(np.int32)).to(DEV), to_dev(K, dtype),
                                     to_dev(V, dtype), return_lse=True)
    torch.cuda.synchronize()
    L.close()
    pick = np.unique(np.concatenate([[0, 1, 17, 18, rows - 6, rows - 1], g.choice(rows, 30, replace=False)]))
    q64, K64, V64 = to_f64(q, dtype)[pick], to_f64(K, dtype), to_f64(V, dtype)
    ref, lse_ref = O.recompute_attention(q64, pos[pick], K64, V64, d ** -0.5)
    ref_abs, _ = O.recompute_attention(q64, pos[pick], K64, np.abs(V64), d ** -0.5)
    assert_attention_close(to_host_f64(out, dtype)[pick], ref, ref_abs, dtype, lse.cpu().numpy()[pick], lse_ref)


def test_wide_rule():
    """Parts of 1.25 times the even share of 256 slots where the rule chooses the wide kernel, what the narrow one had elsewhere;
    partial results always fit the scratch."""
    def plan(hq, hkv, rows, n, **knobs):
        L = B.Layer("bf16", hq, hkv, D, 5e5, max_ctx=n, max_prompt=1, stream=0)
        for key, value in knobs.items():
            L.set_tuning(key, value)
        p = L.attention_plan(rows, n)
        assert p["partial_bytes"] <= p["scratch_bytes"]
        L.close()
        return p

    assert plan(32, 8, 1638, 32768)["part_tiles"] == 260            # 208 jobs of 512 tiles
    assert plan(28, 4, 3072, 20480)["part_tiles"] == 269            # 86 blocks of 36 rows, 344 jobs of 320 tiles
    assert plan(32, 8, 3072, 32768)["part_tiles"] == 480            # 384 and 400 jobs
    assert plan(16, 16, 6200, 40000)["part_tiles"] == 610
    assert plan(32, 8, 4915, 32768)["parts"] == 1                   # 616 jobs: the even share is the longest block
    for rows, n in [(1228, 8192), (128, 32896), (2749, 8192), (2048, 4096)]:
        assert plan(32, 8, rows, n) == plan(32, 8, rows, n, attn_wide=2)
    for hq, hkv in [(32, 8), (28, 4), (40, 8), (16, 16), (16, 2), (64, 8), (32, 1), (8, 8)]:
        for n in (8192, 10001, 32768, 131072):
            for rows in (*range(200, 5000, 173), n):
                if rows <= n:
                    plan(hq, hkv, rows, n)


@pytest.mark.parametrize("hq,hkv,rows,n,parts,part_tiles", [
    (32, 8, 128, 32768, 16, 32), (32, 8, 256, 40000, 8, 79), (64, 8, 64, 32768, 16, 32), (16, 16, 256, 65536, 16, 64),
    (32, 1, 8, 2 ** 20, 64, 256), (16, 2, 32, 2 ** 18, 64, 64), (32, 8, 110, 32768, 16, 32), (32, 8, 320, 65536, 8, 128)])
def test_few_rows_stay_on_the_narrow_kernel(hq, hkv, rows, n, parts, part_tiles):
    """Up to 40 wide jobs, one to three among them: the plan is the one that the narrow kernel gets when it is asked for."""
    L = B.Layer("bf16", hq, hkv, D, 5e5, max_ctx=n, max_prompt=1, stream=0)
    p = L.attention_plan(rows, n)
    L.set_tuning("attn_wide", 2)
    assert p == L.attention_plan(rows, n)
    assert (p["parts"], p["part_tiles"]) == (parts, part_tiles) and p["partial_bytes"] <= p["scratch_bytes"], p
    L.close()


@pytest.mark.gpu
@pytest.mark.parametrize("where", ["end", "spread", "clusters"])
def test_few_rows_against_a_long_cache(where):
    """The prompt's rows over 33000 keys, and rows whose wavefronts hold columns that see none, some and all keys of a tile, on the
    kernel of the rule and on either one; a key that is not a number shows only in the rows behind it.  Against the oracle."""
    n, rows = 33000, 128
    g = np.random.Generator(np.random.Philox(key=[n, 15]))
    K, V = (to_storage(g.standard_normal((n, 8, D)) * 0.5, "bf16") for _ in range(2))
    q = to_storage(g.standard_normal((rows, 32, D)), "bf16")
    pos = {"end": lambda: np.arange(n - rows, n), "spread": lambda: np.sort(g.choice(n, size=rows, replace=False)),
           "clusters": lambda: np.concatenate([np.arange(32) + b for b in (0, 12800 - 16, 20000, n - 32)])}[where]()
    pick = np.arange(0, rows, 5)
    q64, K64, V64 = to_f64(q, "bf16")[pick], to_f64(K, "bf16"), to_f64(V, "bf16")
    ref, lse_ref = O.recompute_attention(q64, pos[pick], K64, V64, D ** -0.5)
    ref_abs, _ = O.recompute_attention(q64, pos[pick], K64, np.abs(V64), D ** -0.5)
    kd, qd, pd, vd = to_dev(K, "bf16"), to_dev(q, "bf16"), torch.from_numpy(pos.astype(np.int32)).to(DEV), to_dev(V, "bf16")
    for wide in (0, 1, 2):
        L = B.Layer("bf16", 32, 8, D, 5e5, max_ctx=n, max_prompt=1)
        L.set_tuning("attn_wide", wide)
        out, lse = L.recompute_attention(qd, pd, kd, vd, return_lse=True)
        torch.cuda.synchronize()
        assert_attention_close(to_host_f64(out, "bf16")[pick], ref, ref_abs, "bf16", lse.cpu().numpy()[pick], lse_ref)
        j = int(pos[rows // 2]) + 1
        bad = kd.clone()
        bad[j, 3] = float("nan")
        out2, lse2 = L.recompute_attention(qd, pd, bad, vd, return_lse=True)
        torch.cuda.synchronize()
        behind = torch.from_numpy(pos >= j).to(DEV)
        assert torch.isnan(out2[behind][:, 12:16]).all() and torch.isnan(lse2[behind][:, 12:16]).all()
        got = to_host_f64(out2, "bf16")[pick]
        got[pos[pick] >= j, 12:16] = ref[pos[pick] >= j, 12:16]
        assert_attention_close(got, ref, ref_abs, "bf16")
        L.close()


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,rows", [(32, 8, 4350), (32, 8, 5800), (28, 4, 5600)], ids=["2.1-rounds", "2.8-rounds", "2.4-rounds"])
@pytest.mark.parametrize("where", ["spread", "end", "denser-towards-the-end", "start"])
def test_the_shortest_blocks_of_a_whole_launch_go_second(hq, hkv, rows, where):
    """Launches of two to three rounds of blocks have a dispatch order of their own if their rows are spread evenly: every row
    of them against the narrow kernel, by the norm of its difference (both round each probability and the result to bf16), and
    some against the oracle."""
    n = 8200
    g = np.random.Generator(np.random.Philox(key=[n + rows, 17]))
    K, V = (to_storage(g.standard_normal((n, hkv, D)) * 0.5, "bf16") for _ in range(2))
    q = to_storage(g.standard_normal((rows, hq, D)), "bf16")
    weight = np.arange(1, n + 1) / (n * (n + 1) / 2)
    pos = {"spread": lambda: np.sort(g.choice(n, size=rows, replace=False)), "end": lambda: np.arange(n - rows, n), "start": lambda: np.arange(rows),
           "denser-towards-the-end": lambda: np.sort(g.choice(n, size=rows, replace=False, p=weight))}[where]().astype(np.int64)
    args = (to_dev(q, "bf16"), torch.from_numpy(pos.astype(np.int32)).to(DEV), to_dev(K, "bf16"), to_dev(V, "bf16"))
    outs = []
    for wide in (0, 2):
        L = B.Layer("bf16", hq, hkv, D, 5e5, max_ctx=n, max_prompt=1)
        L.set_tuning("attn_wide", wide)
        assert L.attention_plan(rows, n)["parts"] == 1
        outs.append(L.recompute_attention(*args).double())
        torch.cuda.synchronize()
        L.close()
    a, b = outs
    assert ((a - b).norm(dim=2) <= 0.02 * torch.maximum(a.norm(dim=2), b.norm(dim=2))).all()
    pick = np.unique(np.concatenate([[0, 1, rows - 1], g.choice(rows, 12, replace=False)]))
    q64, K64, V64 = to_f64(q, "bf16")[pick], to_f64(K, "bf16"), to_f64(V, "bf16")
    ref, _ = O.recompute_attention(q64, pos[pick], K64, V64, D ** -0.5)
    ref_abs, _ = O.recompute_attention(q64, pos[pick], K64, np.abs(V64), D ** -0.5)
    assert_attention_close(a.cpu().numpy()[pick], ref, ref_abs, "bf16")


@pytest.mark.gpu
@pytest.mark.parametrize("part_tiles", [12, 13, 15, 17, 19, 20, 21, 23])
def test_every_row_block_of_a_launch_cut_in_two(part_tiles):
    """Remainders and uncut blocks share the last z of a launch: 10 row blocks, of which none to five are cut if the rows are spread
    evenly, and rows that are not."""
    n, rows, hq, hkv = 1500, 600, 8, 2
    g = np.random.Generator(np.random.Philox(key=[part_tiles, 16]))
    K, V = (to_storage(g.standard_normal((n, hkv, D)) * 0.5, "bf16") for _ in range(2))
    q = to_storage(g.standard_normal((rows, hq, D)), "bf16")
    q64, K64, V64 = to_f64(q, "bf16"), to_f64(K, "bf16"), to_f64(V, "bf16")
    L = B.Layer("bf16", hq, hkv, D, 5e5, max_ctx=n, max_prompt=1)
    L.set_tuning("attn_wide", 1)
    L.set_tuning("attn_part_tiles", part_tiles)
    assert L.attention_plan(rows, n)["parts"] == 2
    for pos in (np.sort(g.choice(n, size=rows, replace=False)), np.arange(n - rows, n), np.concatenate([np.arange(rows - 40), n - 40 + np.arange(40)])):
        out, lse = L.recompute_attention(to_dev(q, "bf16"), torch.from_numpy(pos.astype(np.int32)).to(DEV), to_dev(K, "bf16"),
                                         to_dev(V, "bf16"), return_lse=True)
        torch.cuda.synchronize()
        ref, lse_ref = O.recompute_attention(q64, pos, K64, V64, D ** -0.5)
        ref_abs, _ = O.recompute_attention(q64, pos, K64, np.abs(V64), D ** -0.5)
        assert_attention_close(to_host_f64(out, "bf16"), ref, ref_abs, "bf16", lse.cpu().numpy(), lse_ref)
    L.close()


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,rows,n,power", [(32, 8, 2560, 20000, 0.2), (32, 8, 2429, 32768, 0.4), (28, 4, 2400, 32768, 0.1)])
def test_rows_denser_towards_the_front_do_not_leave_a_long_block_for_the_end(hq, hkv, rows, n, power):
    """The wide kernel cuts these launches by the length of the cache, and fewer blocks than evenly spread rows would have are longer
    than a part.  One block of almost a part's length that starts last makes a launch 1.4 to 1.55 times as long; the narrow
    kernel, within a tenth of the wide one here, is the yardstick."""
    u = (np.arange(rows) + 0.5) / rows
    pos = np.unique((n * (1 - (1 - u) ** (1 / (1 + power)))).astype(np.int64))
    g = torch.Generator(device=DEV).manual_seed(rows)
    q = torch.randn(len(pos), hq, D, generator=g, device=DEV).bfloat16()
    K, V = (torch.randn(n, hkv, D, generator=g, device=DEV).bfloat16() for _ in range(2))
    pd, times, layers = torch.from_numpy(pos.astype(np.int32)).to(DEV), {0: [], 2: []}, {}
    for wide in times:
        layers[wide] = B.Layer("bf16", hq, hkv, D, 5e5, max_ctx=n, max_prompt=1)
        layers[wide].set_tuning("attn_wide", wide)
    for _ in range(8):
        for wide, L in layers.items():
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            a.record()
            for _ in range(3):
                L.recompute_attention(q, pd, K, V)
            b.record()
            b.synchronize()
            times[wide].append(a.elapsed_time(b) / 3)
    for L in layers.values():
        L.close()
    print({wide: round(1000 * min(t)) for wide, t in times.items()})
    assert min(times[0]) <= 1.25 * min(times[2])


@pytest.mark.parametrize("dtype,hq,hkv,d,rows,n,part_tiles", [
    ("bf16", 32, 8, 128, 16, 4000, 4),       # 8 jobs: parts of 8 would fill an eighth of the slots
    ("bf16", 32, 8, 128, 128, 4000, 8), ("bf16", 14, 2, 64, 60, 8000, 4), ("bf16", 14, 2, 64, 400, 4000, 8),
    ("bf16", 32, 8, 128, 1228, 8192, 49),    # 312 jobs, an even share of 39
    ("bf16", 64, 8, 128, 700, 3000, 32),     # 352 jobs: no shorter than 32
    ("f32", 8, 8, 64, 153, 1024, 1),
    ("bf16", 32, 8, 128, 16, 65536, 32), ("bf16", 16, 16, 128, 100, 32768, 32), ("bf16", 32, 8, 128, 1, 20480, 10),  # one row block
])
def test_narrow_parts(dtype, hq, hkv, d, rows, n, part_tiles):
    L = B.Layer(dtype, hq, hkv, d, 5e5, max_ctx=n, max_prompt=1, stream=0)
    p = L.attention_plan(rows, n)
    assert p["part_tiles"] == part_tiles and p["partial_bytes"] <= p["scratch_bytes"], p
    L.close()


@pytest.mark.parametrize("hq,hkv,d,rows,n,jobs", [(32, 8, 128, 64, 4000, 16), (14, 2, 64, 100, 8161, 12), (8, 8, 128, 100, 8161, 8)])
def test_fp32_launches_of_few_jobs_have_a_piece_per_cu(hq, hkv, d, rows, n, jobs):
    L = B.Layer("f32", hq, hkv, d, 5e5, max_ctx=n, max_prompt=1, stream=0)
    p = L.attention_plan(rows, n)
    assert p["parts"] * jobs <= 256 and p["part_tiles"] == -(-(-(-n // 64)) // (256 // jobs)), p
    L.close()


def test_parts_that_do_not_fit_are_merged_until_they_do():
    """fp32, 819 rows of a 32/8-head layer over 8192 keys: at most 64 MiB of partial results, 13.4 MB a part."""
    L = B.Layer("f32", 32, 8, D, 5e5, max_ctx=8192, max_prompt=1, stream=0)
    p = L.attention_plan(819, 8192)
    assert 2 <= p["parts"] <= 4 and p["partial_bytes"] <= p["scratch_bytes"] <= 64 << 20, p
    L.set_tuning("attn_part_tiles", 2)  # a forced cut is made as asked for or not at all
    assert L.attention_plan(819, 8192)["parts"] == 1
    L.close()


@pytest.mark.parametrize("hq,hkv,rows,units", [(32, 32, 128, 4), (32, 32, 5, 1), (64, 32, 64, 4)])
def test_one_row_block_of_a_type_without_a_wide_kernel_is_cut_as_far_as_its_results_fit(hq, hkv, rows, units):
    """fp32, 32 jobs: 16 parts fill the 512 slots, with up to 34 MB of partial results (32 x 16 pieces of one to four 16640-byte slots)."""
    L = B.Layer("f32", hq, hkv, D, 5e5, max_ctx=8192, max_prompt=1, stream=0)
    p = L.attention_plan(rows, 8192)
    assert p["parts"] == 16 and p["partial_bytes"] - 32 * 16 * units * 16640 in range(769), p
    L.close()


def test_the_last_row_block_takes_room_for_the_rows_it_holds():
    """fp32, 32/8 heads of 128: with 1000 rows four parts fit 64 MiB (31 blocks of 32 rows and one slot of 8), up to 1008 rows (a
    fourth part 525 -> 492 us over 8192 keys); 1009 rows would need three slots in the last block."""
    L = B.Layer("f32", 32, 8, D, 5e5, max_ctx=8192, max_prompt=1, stream=0)
    assert [L.attention_plan(rows, 8192)["parts"] for rows in (992, 993, 1000, 1008, 1009)] == [4, 4, 4, 4, 3]
    p = L.attention_plan(1000, 8192)
    assert p["partial_bytes"] - (31 * 4 + 1) * 8 * 4 * 16640 in range(1000 * 4, 1000 * 4 + 513), p
    L.close()


# ---------------------------------------------------------------------------
# The first product's MFMAs are written as inline assembly, so the compiler neither counts the wait states before an
# instruction that touches their result nor those after a vector instruction that writes one of their operands.  The
# source keeps these distances by construction; this test reads the assembly that the compiler made of it and follows
# every path.  Architecture: two wait states from a vector write to an MFMA that reads it, 19 from a 16-pass MFMA to
# anything but an MFMA that touches its result.
# ---------------------------------------------------------------------------
def registers(operand):
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", operand) or re.fullmatch(r"([va])(\d+)()", operand)
    return {(m[1], i) for i in range(int(m[2]), int(m[3] or m[2]) + 1)} if m else set()


def kernel_instructions(text, name):
    """[(opcode, operands, written by hand)] and, for each, the indices of the instructions that may follow."""
    body = re.search(rf"^\S*{name}\S*:.*?^\.Lfunc_end", text, re.S | re.M)[0]
    ins, labels, by_hand = [], {}, False
    for line in body.splitlines()[1:]:
        if "#ASMSTART" in line or "#ASMEND" in line:
            by_hand = "#ASMSTART" in line
            continue
        line = line.split(";")[0].strip()
        if m := re.fullmatch(r"(\.L\w+):", line):
            labels[m[1]] = len(ins)
        elif line and not line.startswith("."):
            op, _, rest = line.partition(" ")
            ins.append((op, [a.strip() for a in rest.split(",")], by_hand))
    after = []
    for i, (op, args, _) in enumerate(ins):
        nxt = [] if op in ("s_branch", "s_endpgm") else [i + 1]
        if "branch" in op:
            nxt.append(labels[args[0]])
        after.append([j for j in nxt if j < len(ins)])
    return ins, after


def wait_states(ins, i):
    op, args, _ = ins[i]
    return int(args[0], 0) + 1 if op == "s_nop" else 8 if op.startswith("v_mfma") else 1


def reachable(ins, edges, start, limit):
    """Instructions fewer than `limit` wait states away from `start` along `edges` (start excluded)."""
    best, todo = {}, [(j, 0) for j in edges[start]]
    while todo:
        j, ws = todo.pop()
        if ws >= limit or best.get(j, limit) <= ws:
            continue
        best[j] = ws
        todo += [(k, ws + wait_states(ins, j)) for k in edges[j]]
    return best


def hazards(text):
    ins, after = kernel_instructions(text, "attn_wide_kernel")
    before = [[] for _ in ins]
    for i, nxt in enumerate(after):
        for j in nxt:
            before[j].append(i)
    found, checked = [], 0
    for i, (op, args, by_hand) in enumerate(ins):
        if not (by_hand and op.startswith("v_mfma")):
            continue
        checked += 1
        read, written = set().union(*map(registers, args[1:4])), registers(args[0])
        for j in reachable(ins, before, i, 2):
            o, a, _ = ins[j]
            if o.startswith("v_") and not o.startswith("v_mfma") and registers(a[0]) & read:
                found.append((ins[j], ins[i]))
        for j in reachable(ins, after, i, 19):
            o, a, _ = ins[j]
            if not o.startswith(("v_mfma", "s_")) and any(registers(x) & written for x in a):
                found.append((ins[i], ins[j]))
    return found, checked


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc in this environment")
def test_wait_states_around_the_hand_placed_matrix_instructions(tmp_path):
    out = tmp_path / "attention.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "attention_mfma.hip"), "-o", str(out)],
                   check=True, capture_output=True, timeout=300)
    text = out.read_text()
    found, checked = hazards(text)
    assert checked >= 96 and not found, found[:4]
    # the scan sees a result that is read too early and an operand that is written too late
    ins = re.findall(r"^\tv_mfma_f32_32x32x16_bf16 (v\[(\d+):\d+\]), (v\[(\d+):\d+\]), a", text, re.M)[0]
    line = f"\tv_mfma_f32_32x32x16_bf16 {ins[0]}, {ins[2]}, a"
    assert hazards(text.replace(line, f"\tv_mov_b32 v{ins[3]}, 0\n{line}", 1))[0]
