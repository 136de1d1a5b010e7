"""GPU parity of calls with few units against the oracle: the index split with a
workgroup per row, decode attention over many splits of one unit, and the score
of units with at most 32 window rows or with many key chunks."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import assert_scores_close, cu, f32, say
from tests.test_gpu_ops import test_split_bit_exact as split_bit_exact

pytestmark = pytest.mark.gpu


# rows x longest row: around one sweep (4,096 entries), several sweeps, short rows
# beside a long one (some empty), and either side of the rule (256 entries per
# row on average; the row count rule takes 512 rows and more to the other form)
@pytest.mark.parametrize("rows,maxn", [(1, 4096), (1, 4097), (3, 4095), (2, 20000), (70, 2293), (64, 600), (511, 700),
                                       (512, 700), (5, 400)])
@pytest.mark.parametrize("reorder", [0, 1])
def test_split_few_rows_bit_exact(gpu_lib, reorder, rows, maxn):
    split_bit_exact(gpu_lib, reorder, rows, maxn, 5000)


def test_split_few_rows_bad_offsets(gpu_lib):
    """Rows whose offsets do not ascend are empty; their neighbours are split."""
    say("split bad offsets")
    n, total = 700, 2100
    row_off = np.array([0, 700, 400, 2100], np.int32)         # row 1 descends
    g = np.random.default_rng(3)
    ix = g.integers(0, 900, total).astype(np.int32)
    mask = g.integers(0, 3, 3 * 900).astype(np.int8)
    i32 = dict(dtype=torch.int32, device="cuda")
    loc, rem, nl, nr = (torch.full((k,), -9, **i32) for k in (total, total, 3, 3))
    gpu_lib.sg_split(cu(row_off), cu(ix), cu(mask, dtype=torch.int8), cu(np.arange(3) * 900, dtype=torch.int64),
                     cu(np.full(3, 900)), 0, loc, rem, nl, nr)
    torch.cuda.synchronize()
    assert nl[1].item() == 0 and nr[1].item() == 0
    m = mask[2 * 900 + ix[400:2100]]
    assert nl[2].item() == (m == 1).sum() and nr[2].item() == (m == 2).sum()
    assert nl[0].item() == (mask[ix[:n]] == 1).sum()


@pytest.mark.parametrize("dtype,G,d", [("bf16", 4, 128), ("f32", 1, 64), ("bf16", 16, 64)])
@pytest.mark.parametrize("rows", [0, 1, 127, 129, 1024, 1025, 3000, 4096])
def test_decode_many_splits(gpu_lib, dtype, G, d, rows):
    """One unit over up to 32 splits, most of them past its rows; the workspace
    starts as NaN patterns.  Tolerance: a result is a weighted mean of O(1)
    values, its fp32 rounding a few 2^-24 per merged state and per step of a
    wavefront's sums (at most 64), so under 64 x 2^-24 x |v| (5 at most) = 2e-5."""
    say("decode splits", dtype, G, d, rows)
    P, pages = 16, 256
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(rows + d)
    q = torch.randn((1, G, d), generator=g).to(td)
    k, v = (torch.randn((pages * P, d), generator=g).to(td) for _ in range(2))
    pt = (torch.randperm(pages, generator=g) * P).to(torch.int32).view(1, 1, pages)
    nr = torch.full((1, 1), rows, dtype=torch.int32)
    ws = torch.full((gpu_lib.decode_workspace_size(1, G, 1, d, pages, P),), 0xFF, dtype=torch.uint8, device="cuda")
    out = torch.empty((1, G, d), device="cuda")
    gpu_lib.sg_decode_attn(q.cuda(), k.cuda(), v.cuda(), pt.cuda(), nr.cuda(), P, out, ws=ws)
    torch.cuda.synchronize()
    ref = oracle.decode_attn(f32(q), f32(k), f32(v), pt.numpy(), nr.numpy(), P)
    np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=0, atol=2e-5)


@pytest.mark.parametrize("dtype,G,W,d,lens", [
    ("f32", 1, 32, 64, (2048,)), ("f32", 1, 32, 128, (1000, 33)), ("bf16", 1, 31, 128, (5000,)),
    ("bf16", 2, 16, 64, (700, 16, 3000)), ("bf16", 2, 17, 128, (5000,)), ("f32", 1, 33, 64, (2049,)),
    ("bf16", 4, 64, 128, (20000,))])
def test_score_few_units(gpu_lib, dtype, G, W, d, lens):
    """At most 32 rows per unit (half of a wavefront's), and one unit in more
    chunks than one batch of statistics holds."""
    say("score few units", dtype, G, W, d, lens)
    T, Hkv = sum(lens), 1
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(T + W)
    q = torch.randn((len(lens), 1, Hkv * G, W, d), generator=g).to(td)
    k = torch.randn((1, Hkv, T, d), generator=g).to(td)
    cus = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ws = torch.full((gpu_lib.score_workspace_size(len(lens), 1, Hkv * G, Hkv, d, W, max(lens)),), 0xFF,
                    dtype=torch.uint8, device="cuda")
    out = torch.empty((1, Hkv, T), device="cuda")
    gpu_lib.sg_score(q.cuda(), k.cuda(), cu(cus), T, max(lens), Hkv, out, ws=ws)
    torch.cuda.synchronize()
    assert_scores_close(out.cpu().numpy(), oracle.score(f32(q), f32(k), cus, Hkv), rtol=1e-4)
    alpha = 3.0
    cnt = torch.empty_like(out)
    gpu_lib.sg_score_count(q.cuda(), k.cuda(), cu(cus), T, max(lens), Hkv, cnt, alpha, ws)
    torch.cuda.synchronize()
    ref = np.asarray(oracle.score_count(f32(q), f32(k), cus, Hkv, alpha))
    # an fp32 logit within a rounding of its threshold may fall on either side
    assert np.abs(cnt.cpu().numpy() - ref).sum() <= 2 + 1e-3 * ref.sum()
