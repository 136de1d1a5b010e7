"""GPU parity of sg_score_topshare where its passes hand a row on: each sample
size, intervals misjudged or widened by far outliers, bins of ties (one value,
several side by side), lists that run over, ranks at both ends, logits that are
not finite, short requests beside long ones, more units than a launch holds.
Inputs are integers, so every logit is exact in fp32 and fp64 and the counts
must equal the oracle's.  The calls' workspace shows which rows a path left to
the radix select."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import say
from tests.test_gpu_selectors import _ints, _topshare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,G,W,d,lens,bp,kind", [
    ("bf16", 4, 64, 64, (12288,), 2000, "plain"),        # 512 sampled keys
    ("bf16", 4, 64, 64, (12289, 700), 2000, "plain"),    # 1024
    ("bf16", 1, 33, 128, (24577, 40, 3000), 4000, "plain"),   # 2048, requests far shorter, N just above W
    ("f32", 2, 16, 64, (24577,), 1000, "plain"),
    ("bf16", 4, 64, 64, (9000,), 2000, "outliers"),      # the sample's range is mostly empty
    ("bf16", 4, 64, 64, (9000,), 1, "outliers"),         # the maxima
    ("bf16", 4, 40, 64, (8191,), 9999, "plain"),         # nearly every key
    ("bf16", 2, 64, 64, (5000, 513), 2000, "ties"),      # a few distinct logits
    ("f32", 4, 16, 64, (3000,), 5000, "ties"),
    ("bf16", 4, 64, 64, (4096,), 2000, "zeros"),         # one logit
    ("bf16", 4, 64, 64, (9001,), 3000, "half"),          # half the keys tied at zero
    ("bf16", 8, 64, 128, (4097,), 2000, "plain"),        # 512 rows
])
def test_topshare_paths_exact(gpu_lib, dtype, G, W, d, lens, bp, kind):
    say("topshare paths", dtype, G, W, d, lens, bp, kind)
    L, Hkv, T = 1, 2, sum(lens)
    span = 1 if kind == "ties" else 0 if kind == "zeros" else 40
    q = _ints((len(lens), L, Hkv * G, W, d), -max(span, 1), max(span, 1), T + W, dtype)
    k = _ints((L, Hkv, T, d), -span, span, T + d, dtype)
    if kind == "outliers":                               # still exact: below 2^24
        k[:, :, ::1500] *= 32
    if kind == "half":
        k[:, :, ::2] = 0
    got, cus = _topshare(gpu_lib, q, k, lens, Hkv, bp)
    ref = oracle.score_topshare(q.float().numpy(), k.float().numpy(), cus, Hkv, bp)
    np.testing.assert_array_equal(got, ref.astype(np.float32))


def _workspace(gpu_lib, q, lens, Hkv):
    B, L, Hq, W, d = q.shape
    return torch.full((gpu_lib.score_topshare_workspace_size(B, L, Hq, Hkv, d, W, max(lens)),), 0xA5,
                      dtype=torch.uint8, device="cuda")


def _radix_groups(ws, q, lens, Hkv):
    """Groups of 32 rows of each unit that took the radix select: the bits of the
    workspace's words after 98 words per row, one word per unit."""
    B, L, Hq, W, _ = q.shape
    units = B * L * Hkv
    at = units * (Hq // Hkv) * W * 98
    return [bin(x & 0xffffffff).count("1") for x in ws.view(torch.int32)[at:at + units].tolist()]


def _again_units(ws, q, lens, Hkv):
    """Units that took the histogram again: the workspace's words after those."""
    B, L, Hq, W, _ = q.shape
    units = B * L * Hkv
    at = units * (Hq // Hkv) * W * 98 + units
    return sum(x != 0 for x in ws.view(torch.int32)[at:at + units].tolist())


@pytest.mark.parametrize("n,kind", [(900, "rising"), (1500, "rising"), (2040, "rising"), (8192, "rising"),
                                    (8192, "period 16"), (8192, "period 64"), (16384, "period 16")])
def test_topshare_sample_is_fair(gpu_lib, n, kind):
    """Logits that rise with the position, or whose level repeats: the sampled
    interval holds every row's threshold, so no row needs the radix select."""
    say("topshare sample", n, kind)
    G, W, d, Hkv = 4, 64, 64, 2
    q = _ints((1, 1, Hkv * G, W, d), 10, 50, n, "bf16")
    k = _ints((1, Hkv, n, d), -40, 40, n + 1, "bf16")
    if kind == "rising":
        level = np.arange(n) * 60 // n
    else:
        p = int(kind.split()[1])
        level = np.random.default_rng(p).integers(-60, 61, p)[np.arange(n) % p]
    k += torch.from_numpy(level.astype(np.float32)).to(torch.bfloat16)[None, None, :, None]     # whole, below 2^8
    ws = _workspace(gpu_lib, q, (n,), Hkv)
    got, cus = _topshare(gpu_lib, q, k, (n,), Hkv, 2000, ws=ws)
    ref = oracle.score_topshare(q.float().numpy(), k.float().numpy(), cus, Hkv, 2000)
    np.testing.assert_array_equal(got, ref.astype(np.float32))
    assert _radix_groups(ws, q, (n,), Hkv) == [0] * Hkv


@pytest.mark.parametrize("W,n", [(64, 130), (64, 200), (64, 300), (64, 513), (33, 90), (512, 700), (512, 513)])
def test_topshare_window_keys_on_top(gpu_lib, W, n):
    """Short prompts of rising logits: the window's own keys, which only some
    rows see, are the largest, and the first histogram holds every row's
    threshold."""
    say("topshare window keys on top", W, n)
    G, d, Hkv = 4 if W < 128 else 1, 64, 2
    q = _ints((1, 1, Hkv * G, W, d), 10, 50, n, "bf16")
    k = _ints((1, Hkv, n, d), -40, 40, n + 1, "bf16")
    k += torch.from_numpy((np.arange(n) * 200 // n).astype(np.float32)).to(torch.bfloat16)[None, None, :, None]
    ws = _workspace(gpu_lib, q, (n,), Hkv)
    got, cus = _topshare(gpu_lib, q, k, (n,), Hkv, 2000, ws=ws)
    ref = oracle.score_topshare(q.float().numpy(), k.float().numpy(), cus, Hkv, 2000)
    np.testing.assert_array_equal(got, ref.astype(np.float32))
    assert _again_units(ws, q, (n,), Hkv) == 0 and _radix_groups(ws, q, (n,), Hkv) == [0] * Hkv


@pytest.mark.parametrize("dtype,G,d,n,B", [("bf16", 4, 64, 2048, 64), ("f32", 2, 64, 2048, 64), ("bf16", 8, 128, 4096, 16)])
def test_topshare_bins_in_one_chunk(gpu_lib, dtype, G, d, n, B):
    """Logits that follow the position: all the keys of a row's bin lie in a few
    neighbouring tiles of one 2,048-key chunk, and are gathered all the same
    (half of the key's step in noise, so that no two logits tie)."""
    say("topshare bins in one chunk", dtype, G, d, n, B)
    W, Hkv, L = 16, 8, 2
    q = _ints((B, L, Hkv * G, W, d), 30, 50, n, dtype)
    k = _ints((L, Hkv, B * n, d), -1, 1, n + 1, dtype)
    k += torch.from_numpy(np.tile(np.arange(n) * 250 // n, B).astype(np.float32)).to(k.dtype)[None, None, :, None]
    ws = _workspace(gpu_lib, q, [n] * B, Hkv)
    got, cus = _topshare(gpu_lib, q, k, [n] * B, Hkv, 2000, ws=ws)
    assert sum(_radix_groups(ws, q, [n] * B, Hkv)) == 0
    for b in (0, B - 1):
        ref = oracle.score_topshare(q[b:b + 1].float().numpy(), k[:, :, b * n:(b + 1) * n].float().numpy(), [0, n], Hkv,
                                    2000)
        np.testing.assert_array_equal(got[:, :, b * n:(b + 1) * n], ref.astype(np.float32))


@pytest.mark.parametrize("bp", [1, 10, 100, 9990, 9999])
@pytest.mark.parametrize("dtype,n,kind", [("bf16", 12000, "plain"), ("bf16", 16384, "plain"), ("bf16", 9000, "outliers"),
                                          ("f32", 5000, "plain"), ("bf16", 700, "plain")])
def test_topshare_ranks_at_the_ends(gpu_lib, dtype, n, kind, bp):
    """The largest keys, or all but the smallest: those beyond the sample's
    extremes are gathered, so no row needs the radix select."""
    say("topshare ranks at the ends", dtype, n, kind, bp)
    G, W, d, Hkv = 4, 16, 64, 2
    q = _ints((1, 1, Hkv * G, W, d), -40, 40, n, dtype)
    k = _ints((1, Hkv, n, d), -40, 40, n + 1, dtype)
    if kind == "outliers":                               # still exact: below 2^24
        k[:, :, 100::1500] *= 32
    ws = _workspace(gpu_lib, q, (n,), Hkv)
    got, cus = _topshare(gpu_lib, q, k, (n,), Hkv, bp, ws=ws)
    ref = oracle.score_topshare(q.float().numpy(), k.float().numpy(), cus, Hkv, bp)
    np.testing.assert_array_equal(got, ref.astype(np.float32))
    assert _radix_groups(ws, q, (n,), Hkv) == [0] * Hkv


@pytest.mark.parametrize("dtype,G,W,d,n,kind", [
    ("bf16", 4, 64, 64, 8192, "zeros"), ("bf16", 4, 64, 128, 5000, "few"), ("f32", 4, 16, 64, 3000, "few"),
    ("bf16", 8, 64, 64, 4096, "few"), ("bf16", 4, 64, 64, 30000, "few"), ("f32", 2, 64, 64, 15000, "few"), ("bf16", 4, 64, 64, 5000, "large"),
    ("f32", 4, 32, 128, 14000, "large"), ("bf16", 2, 64, 128, 30000, "large"), ("bf16", 2, 64, 64, 8192, "period 16"), ("bf16", 4, 32, 128, 8191, "period 64"),
    ("f32", 2, 33, 128, 4000, "period 16"), ("bf16", 1, 40, 64, 30000, "period 64"), ("bf16", 4, 64, 64, 9001, "half")])
def test_topshare_ties_settle(gpu_lib, dtype, G, W, d, n, kind):
    """More equal logits at a row's threshold than it may gather (one value, a
    few, repeated keys): found equal, not handed to the radix select."""
    say("topshare ties", dtype, G, W, d, n, kind)
    Hkv = 2
    q = _ints((1, 1, Hkv * G, W, d), -1 if kind == "few" else -40, 1 if kind == "few" else 40, n, dtype)
    k = _ints((1, Hkv, n, d), -1 if kind == "few" else -40, 1 if kind == "few" else 40, n + 1, dtype)
    if kind == "zeros":
        k *= -0.0
    elif kind == "half":
        k[:, :, ::2] = 0
    elif kind == "large":         # two values, their step far below their size
        g = np.random.default_rng(n)
        q[..., 1:], k[..., 1:] = 0, 0
        q[..., 0], k[..., 0], q[..., 1] = q[..., 0].abs() + 200, 255, 1
        k[..., 1] = torch.from_numpy((g.random((1, Hkv, n)) < 0.3).astype(np.float32))
    elif kind != "few":
        k = k[:, :, torch.arange(n) % int(kind.split()[1])].contiguous()
    for bp in (700, 5000):
        ws = _workspace(gpu_lib, q, (n,), Hkv)
        got, cus = _topshare(gpu_lib, q, k, (n,), Hkv, bp, ws=ws)
        ref = oracle.score_topshare(q.float().numpy(), k.float().numpy(), cus, Hkv, bp)
        np.testing.assert_array_equal(got, ref.astype(np.float32))
        assert sum(_radix_groups(ws, q, (n,), Hkv)) <= 1, bp      # (of up to 32 groups of rows)


def test_topshare_tied_value_at_an_interval_end(gpu_lib):
    """8,192 rows over 64K keys with logits of a few values: a row here and there
    has its tied threshold at an end of its interval, and none loses it."""
    say("topshare tied interval end")
    L, Hkv, G, W, d, n, bp = 4, 8, 4, 64, 128, 65536, 2000
    gen = torch.Generator(device="cuda").manual_seed(1)
    for shape in ((1, L, Hkv * G, W, d), (L, Hkv, n, d)):       # (draws of this seed with such a row)
        torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)
    q, k = (torch.randint(-1, 2, shape, generator=gen, device="cuda").to(torch.bfloat16)
            for shape in ((1, L, Hkv * G, W, d), (L, Hkv, n, d)))
    ws = _workspace(gpu_lib, q, (n,), Hkv)
    got, _ = _topshare(gpu_lib, q, k, (n,), Hkv, bp, ws=ws)
    assert sum(_radix_groups(ws, q, (n,), Hkv)) == 0
    pos = n - W + torch.arange(G * W, device="cuda") % W
    for l, h in ((0, 0), (3, 6), (3, 7)):
        z = q[0, l, h * G:(h + 1) * G].reshape(G * W, d).float() @ k[l, h].float().t().contiguous()
        z.masked_fill_(torch.arange(n, device="cuda")[None] > pos[:, None], -1e9)
        kth = (pos + 1) * bp // 10000
        thr = z.sort(dim=1, descending=True).values.gather(1, (kth - 1)[:, None])
        np.testing.assert_array_equal(got[l, h], (z >= thr).sum(0).float().cpu().numpy())


@pytest.mark.parametrize("dtype,G,W,d,n", [("bf16", 4, 64, 64, 8192), ("f32", 4, 16, 128, 3000), ("bf16", 8, 64, 128, 2500),
                                           ("f32", 1, 33, 64, 14000)])
def test_topshare_ties_side_by_side(gpu_lib, dtype, G, W, d, n):
    """Three neighbouring logits with a twentieth of the keys each around the
    threshold, the other keys far apart: where no bin tells them apart, the
    radix select does."""
    say("topshare ties side by side", dtype, G, W, d, n)
    Hkv = 2
    g = np.random.default_rng(n)
    q = torch.zeros((1, 1, Hkv * G, W, d))
    q[..., 0] = torch.from_numpy(g.integers(128, 257, q.shape[:-1]).astype(np.float32))
    q[..., 1] = 1
    k = torch.zeros((1, Hkv, n, d))
    k[..., 0] = torch.from_numpy(g.integers(-250, 251, (1, Hkv, n)).astype(np.float32))
    tied = torch.from_numpy(g.random((1, Hkv, n)) < 0.15)
    k[..., 0] = torch.where(tied, 7.0, k[..., 0])
    k[..., 1] = torch.from_numpy(g.integers(-1, 2, (1, Hkv, n)).astype(np.float32))
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k = q.to(td), k.to(td)
    left = 0
    for bp in (4400, 4900, 5400):          # (41% of the keys lie above the ties)
        ws = _workspace(gpu_lib, q, (n,), Hkv)
        got, cus = _topshare(gpu_lib, q, k, (n,), Hkv, bp, ws=ws)
        ref = oracle.score_topshare(q.float().numpy(), k.float().numpy(), cus, Hkv, bp)
        np.testing.assert_array_equal(got, ref.astype(np.float32))
        left += sum(_radix_groups(ws, q, (n,), Hkv))
    assert left > 0


@pytest.mark.parametrize("dtype,G,W,d,n,bp", [("bf16", 4, 16, 64, 3000, 2000), ("f32", 2, 33, 64, 1500, 300),
                                              ("bf16", 8, 64, 128, 5000, 9000), ("bf16", 1, 16, 64, 500, 100)])
@pytest.mark.parametrize("kind", ["inf", "nan", "many nan", "all"])
def test_topshare_not_finite(gpu_lib, dtype, G, W, d, n, bp, kind):
    """Infinite and NaN logits, in the documented order of their bit patterns: a
    NaN takes a rank, above +inf or with its sign bit set below -inf, and is
    never picked itself.  (The matrix instructions of fp32 keep the key's NaN,
    those of bf16 make one with the sign bit.)"""
    low = dtype == "bf16"
    say("topshare not finite", dtype, G, W, d, n, bp, kind)
    Hkv = 2
    q = _ints((1, 1, Hkv * G, W, d), -20, 20, n, dtype)
    q[..., 0] = torch.where(q[..., 0] >= 0, 3.0, -3.0).to(q.dtype)      # an infinite key channel: +-inf, no NaN
    k = _ints((1, Hkv, n, d), -40, 40, n + 1, dtype)
    g = np.random.default_rng(n)
    if kind in ("inf", "all"):
        k[0, :, g.choice(n, max(1, n // 40), replace=False), 0] = float("inf")
        k[0, :, g.choice(n, max(1, n // 40), replace=False), 0] = float("-inf")
    if kind in ("nan", "many nan", "all"):
        k[0, :, g.choice(n, n // 3 if kind == "many nan" else max(1, n // 90), replace=False)] = float("nan")
    got, cus = _topshare(gpu_lib, q, k, (n,), Hkv, bp)
    with np.errstate(invalid="ignore"):
        z = np.einsum("hgwd,hnd->hgwn", q.double().numpy()[0, 0].reshape(Hkv, G, W, d), k.double().numpy()[0])
    ref = np.zeros((1, Hkv, n), np.float32)
    for w in range(W):
        seen = n - W + w + 1
        kk = min(seen, max(1, seen * bp // 10000))
        x = z[:, :, w, :seen]
        order = np.sort(np.where(np.isnan(x), -np.inf if low else np.inf, x), axis=-1)[..., ::-1]
        nan = np.isnan(x).sum(-1)
        thr = order[..., kk - 1] if low else np.where(nan >= kk, np.nan, order[..., kk - 1])
        if kk == seen:
            thr = np.full_like(thr, -np.inf)
        with np.errstate(invalid="ignore"):
            ref[0, :, :seen] += (x >= thr[..., None]).sum(1)
    np.testing.assert_array_equal(got, ref)


def test_topshare_many_units(gpu_lib):
    """8,388,672 units of one row and two keys: more threads than one launch of
    some passes may hold.  Integer logits, so the larger one (both, if they tie)
    is picked exactly."""
    B, L, d, N = 131073, 64, 64, 2
    say("topshare many units", B, L)
    T = B * N
    g = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randint(-3, 4, (B, L, 1, 1, d), generator=g, device="cuda", dtype=torch.int8).to(torch.bfloat16)
    k = torch.randint(-3, 4, (L, 1, T, d), generator=g, device="cuda", dtype=torch.int8).to(torch.bfloat16)
    cus = torch.arange(0, T + 1, N, dtype=torch.int32, device="cuda")
    ws = torch.full((gpu_lib.score_topshare_workspace_size(B, L, 1, 1, d, 1, N),), 0xA5, dtype=torch.uint8,
                    device="cuda")
    out = torch.full((L, 1, T), -1.0, device="cuda")
    gpu_lib.sg_score_topshare(q, k, cus, T, N, 1, out, 5000, ws)
    for l in range(L):
        z = (q[:, l, 0].float() * k[l, 0].view(B, N, d).float()).sum(-1)
        assert torch.equal(out[l, 0].view(B, N), (z >= z.amax(1, keepdim=True)).float()), l
