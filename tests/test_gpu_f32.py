"""The float32 matrix-core kernels against the oracle: products at the edges of
every tile form and of the rule that chooses it, attention at the edges of its
32-key tiles and four-wave key split, a block whose gated-residual products run
on the 64 x 64 tiles (GPU)."""
import numpy as np
import pytest

import synth
from oracle import dit
from tests.gpu_util import TOL_F32, context, rel_l2, row_rel_l2, small_cfg, torch_cuda

pytestmark = pytest.mark.gpu


# 16 x 16 tiles (one row and column, remainders of both), 32 x 32 (tiles of 32
# cover 256 compute units, tiles of 64 do not), 64 x 64 (last rows and columns
# partial), 128 x 64 (fewer dispatch rounds), K of 1, 2 and 3 stages, and the
# shapes only the plain kernel takes (K not a multiple of 32, odd row strides)
@pytest.mark.parametrize("m,n,k,pad", [
    (1, 1, 32, 0), (17, 33, 96, 4), (40, 130, 1056, 0), (250, 1000, 160, 0), (705, 1000, 64, 8), (705, 1001, 32, 0),
    (1921, 1024, 96, 0), (1920, 1030, 32, 4), (65, 64, 33, 0), (65, 64, 64, 1)])
def test_linear_f32_tiles_match_oracle(m, n, k, pad):
    torch = torch_cuda()
    cfg = synth.get_config("tiny")
    ctx = context(cfg, weights=False)
    rng = np.random.default_rng(m + n + k)
    a = rng.standard_normal((m, k + pad)).astype(np.float32)
    w, b = rng.standard_normal((n, k)).astype(np.float32), rng.standard_normal(n).astype(np.float32)
    out = torch.full((m, n + pad), 7.0, device="cuda")
    ctx.linear(ctx.to_device(a), ctx.to_device(w), ctx.to_device(b), out, m, n, k, lda=k + pad, ldc=n + pad)
    got = out.cpu().numpy()
    ref = dit.linear({"l.w": w, "l.b": b}, "l", a[:, :k].astype(np.float64))
    # k rounded additions per output, each at most 2^-24 of the partial sum
    tol = max(4, np.sqrt(k)) * 4 * 2.0 ** -24
    err, rerr = rel_l2(got[:, :n], ref), row_rel_l2(got[:, :n], ref)
    print(f"{m}x{n}x{k}: rel_l2 {err:.2e}, worst row {rerr:.2e}, bound {tol:.2e}")
    assert err <= tol and rerr <= 4 * tol
    assert (got[:, n:] == 7.0).all()


@pytest.mark.parametrize("head_dim,heads,n,spread", [
    (64, 4, 1, 1), (64, 4, 31, 1), (64, 8, 33, 1), (64, 4, 128, 1), (64, 16, 161, 12), (64, 12, 449, 1),
    (128, 2, 32, 1), (128, 8, 97, 12), (128, 2, 300, 1)])
def test_attention_f32_matches_oracle(head_dim, heads, n, spread):
    """spread 12 grows the scores along the keys, so the running max moves in
    every wave and the waves' parts carry very different weights."""
    torch = torch_cuda()
    ctx = context(small_cfg("f32", head_dim=head_dim, hidden=heads * head_dim, heads=heads), weights=False)
    rng = np.random.default_rng(n)
    q, k, v = (rng.standard_normal((heads, n, head_dim)).astype(np.float32) for _ in range(3))
    k *= np.linspace(1, spread, n, dtype=np.float32)[None, :, None]
    npad, ldo = ctx.attn_pad(n), heads * head_dim + 3
    dev = []
    for x in (q, k, v):
        p = np.zeros((heads, npad, head_dim), np.float32)
        p[:, :n] = x
        dev.append(ctx.to_device(p))
    out = torch.full((n, ldo), 7.0, device="cuda")
    ctx.attention(*dev, n, out, ldo)
    got = out.cpu().numpy()
    ref = dit.attention(*(x.astype(np.float64) for x in (q, k, v))).transpose(1, 0, 2).reshape(n, -1)
    err = rel_l2(got[:, :heads * head_dim], ref)
    print(f"hd {head_dim} heads {heads} n {n}: rel_l2 {err:.2e}")
    # scores up to about 40 carry a few 2^-24 of their size into the exponential
    assert err <= (1e-5 if spread > 1 else 2e-6)
    assert (got[:, heads * head_dim:] == 7.0).all()


@pytest.mark.parametrize("head_dim,heads,n", [(64, 4, 100), (64, 8, 449), (128, 2, 160)])
def test_attention_f32_infinite_and_nan_scores(head_dim, heads, n):
    """Keys 32..95, whole tiles of two waves, score -inf for every query: weight 0. A NaN
    query row stays NaN by itself; a +inf score makes its row NaN."""
    torch = torch_cuda()
    ctx = context(small_cfg("f32", head_dim=head_dim, hidden=heads * head_dim, heads=heads), weights=False)
    rng = np.random.default_rng(n)
    q, k, v = (rng.standard_normal((heads, n, head_dim)).astype(np.float32) for _ in range(3))
    q[:, :, 0] = np.abs(q[:, :, 0]) + 0.1
    k[:, 32:96, 0] = -np.inf
    q[:, 7, 3] = np.nan
    k[:, n - 1, 5], q[:, :, 5] = np.inf, -np.abs(q[:, :, 5]) - 0.1
    q[:, 40, 5] = 0.5                          # +inf against the last key
    npad, ldo = ctx.attn_pad(n), heads * head_dim
    dev = []
    for x in (q, k, v):
        p = np.zeros((heads, npad, head_dim), np.float32)
        p[:, :n] = x
        dev.append(ctx.to_device(p))
    out = torch.full((n, ldo), 7.0, device="cuda")
    ctx.attention(*dev, n, out, ldo)
    got = out.cpu().numpy()
    assert np.isnan(got[[7, 40]]).all()
    rows = [r for r in range(n) if r not in (7, 40)]
    keys = [j for j in range(n - 1) if not 32 <= j < 96]
    ref = dit.attention(q[:, rows].astype(np.float64), *(x[:, keys].astype(np.float64) for x in (k, v)))
    err = rel_l2(got[rows], ref.transpose(1, 0, 2).reshape(len(rows), -1))
    print(f"hd {head_dim} n {n}: rel_l2 {err:.2e}")
    assert err <= 2e-6


@pytest.mark.parametrize("m,n,k", [(17, 33, 96), (250, 1000, 160), (705, 1000, 64), (1921, 1024, 96)])
def test_linear_f32_infinities_and_nan_stay_in_their_rows_and_columns(m, n, k):
    """Every tile form: a NaN in the last row of A and an infinity in the last row of W touch only
    that output row and column."""
    torch = torch_cuda()
    ctx = context(synth.get_config("tiny"), weights=False)
    rng = np.random.default_rng(m)
    a, w, b = (rng.standard_normal(s).astype(np.float32) for s in ((m, k), (n, k), (n,)))
    a[:, 1] = np.abs(a[:, 1]) + 0.1
    a[m - 1, 2], w[n - 1, 1] = np.nan, np.inf
    out = torch.zeros((m, n), device="cuda")
    ctx.linear(ctx.to_device(a), ctx.to_device(w), ctx.to_device(b), out, m, n, k)
    got = out.cpu().numpy()
    assert np.isnan(got[m - 1]).all() and np.isposinf(got[:m - 1, n - 1]).all()
    ref = dit.linear({"l.w": w[:n - 1], "l.b": b[:n - 1]}, "l", a[:m - 1].astype(np.float64))
    assert rel_l2(got[:m - 1, :n - 1], ref) <= max(4, np.sqrt(k)) * 4 * 2.0 ** -24


def test_block_f32_gated_residual_on_tiles():
    """728 tokens, D = 1,024: every product of the block runs on the 64 x 64 or 128 x 64 tiles."""
    torch = torch_cuda()
    cfg = small_cfg("f32", head_dim=64, hidden=1024, heads=16, latent=(16, 4, 28, 26), text_tokens=0, n_dual=0)
    ctx = context(cfg)
    W, x, c = synth.gen_weights(cfg), synth.gen_block_input(cfg), synth.gen_cemb(cfg)
    for b in range(cfg.n_blocks):
        xd = torch.from_numpy(x).cuda()
        ctx.block_forward(b, xd, torch.from_numpy(c).cuda())
        err = rel_l2(xd.cpu().numpy(), dit.block_forward(W, cfg, b, x, c))
        print("block", b, "rel_l2", err)
        assert err <= TOL_F32 / 20     # the float32 bar is 1e-4; sums of 4,096 rounded terms stay near 1e-6
