"""The q/k/v projection with per-head RMSNorm, RoPE and the attention layouts
fused into the GEMM epilogue, against the plain GEMM followed by the separate
preparation kernels (GPU). Both round the projection to bf16 once and then
apply the same float32 arithmetic, so the blocks must agree bit for bit; the
oracle comparison of the fused path is in the block, forward and full-size
tests."""
import os

import numpy as np
import pytest

import synth
from oracle import dit
from tests.gpu_util import TOL_BF16_BLOCK, rel_l2, small_cfg, torch_cuda

pytestmark = pytest.mark.gpu


def _pair(cfg, max_batch=1):
    """(fused, separate) contexts sharing one weight blob. These products are
    too small to fill a dispatch round of 256 x 256 tiles, which would send
    them to smaller tiles: the fused context keeps the tile size the shape
    selects (WDC_FILL_TILES=0)."""
    import paper_2608_01845_amd as wdc
    os.environ["WDC_FILL_TILES"] = "0"
    try:
        fused = wdc.Context(cfg, max_batch=max_batch)
    finally:
        del os.environ["WDC_FILL_TILES"]
    fused.load_weights(synth.gen_weights(cfg))
    os.environ["WDC_FUSE_QKV"] = "0"
    try:
        sep = wdc.Context(cfg, max_batch=max_batch, allocate_weights=False)
    finally:
        del os.environ["WDC_FUSE_QKV"]
    sep.bind_weights(fused.weights)
    return fused, sep


@pytest.mark.parametrize("head_dim,rope", [(64, True), (128, True), (64, False), (128, False)])
def test_fused_qkv_blocks_equal_separate_preparation(head_dim, rope):
    """560 video + 21 text tokens: the sequential and single blocks and the
    dual block's video stream take the fused epilogue (the 21 text rows of the
    dual block stay on the separate kernels); the last 256-row tile is partial
    and its last group of 16 tokens incomplete. Without rotary dimensions the
    epilogue takes its form without rotation-table reads."""
    torch = torch_cuda()
    cfg = small_cfg("bf16", head_dim=head_dim, latent=(16, 4, 20, 28), **({} if rope else {"rope": (0, 0, 0)}))
    fused, sep = _pair(cfg)
    x = synth.gen_block_input(cfg)
    c = torch.from_numpy(synth.gen_cemb(cfg)).cuda()
    W = synth.gen_weights(cfg)
    for b in range(cfg.n_blocks):
        xf = torch.from_numpy(x).cuda()
        xs = xf.clone()
        fused.block_forward(b, xf, c)
        sep.block_forward(b, xs, c)
        diff = float((xf - xs).abs().max())
        print(f"hd {head_dim} block {b}: fused vs separate max |diff| {diff:.3e}")
        assert torch.equal(xf, xs), (b, diff)
        err = rel_l2(xf.cpu().numpy(), dit.block_forward(W, cfg, b, x, synth.gen_cemb(cfg)))
        print(f"hd {head_dim} block {b} ({dit.block_kind(cfg, b)}): fused == separate, oracle rel_l2 {err:.2e}")
        assert err <= TOL_BF16_BLOCK


def test_fused_qkv_batched_forward_equals_separate_preparation():
    """Two samples in one product: 581-token samples, so a 256-row tile holds
    rows of both samples and the first token of most tiles is not 16-aligned
    (the element-wise V^T path)."""
    torch = torch_cuda()
    cfg = small_cfg("bf16", head_dim=64, latent=(16, 4, 20, 28))
    fused, sep = _pair(cfg, max_batch=2)
    zs = [torch.from_numpy(synth.gen_tensor(s, "z", cfg.latent)).cuda() for s in (1, 2)]
    inp = synth.gen_inputs(cfg)
    conds = [fused.to_device(inp["cond"])] * 2
    texts = [fused.to_device(inp["text"])] * 2
    cams = [fused.to_device(inp["cam"])] * 2
    vf = fused.forward_batch(zs, 0.4, conds, texts, cams)
    vs = sep.forward_batch(zs, 0.4, conds, texts, cams)
    for a, b in zip(vf, vs):
        print("batched forward: fused vs separate max |diff|", float((a - b).abs().max()))
        assert torch.isfinite(a).all() and torch.equal(a, b)


def test_fill_tiles_mid_forward_bitwise_equal():
    """The mid-size forward (2,688 tokens, D = 1,024) with its products, the fused
    q/k/v projection among them, on smaller tiles (the default: no product fills
    a dispatch round of 256 x 256 tiles) against the 256 x 256 tiles: both sum
    every output over K in the same order and apply the same float32 arithmetic
    afterwards, so the velocities agree bit for bit."""
    torch = torch_cuda()
    import paper_2608_01845_amd as wdc
    cfg = synth.get_config("mid")
    fill = wdc.Context(cfg)
    fill.init_random_weights(seed=5, std=0.02)
    os.environ["WDC_FILL_TILES"] = "0"
    try:
        shape = wdc.Context(cfg, allocate_weights=False)
    finally:
        del os.environ["WDC_FILL_TILES"]
    shape.bind_weights(fill.weights)
    inp = synth.gen_inputs(cfg)
    z = torch.from_numpy(inp["z_T"]).cuda()
    cond = fill.to_device(inp["cond"])
    a = fill.forward(z, 0.7, cond)
    b = shape.forward(z, 0.7, cond)
    print("mid forward: smaller tiles vs 256 x 256 max |diff|", float((a - b).abs().max()))
    assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("hidden,head_dim,latent,batch", [
    (256, 64, (16, 7, 28, 30), 1),      # 1,470 + 21 tokens: 96 x 128 tiles
    (256, 128, (16, 7, 28, 30), 1),
    (256, 128, (16, 12, 38, 40), 1),    # 4,560 + 21 tokens: 128 x 128 tiles, one per compute unit
    (768, 64, (16, 7, 38, 42), 1),      # 2,793 + 21 tokens: 256 x 128 tiles
    (256, 64, (16, 4, 20, 38), 2),      # two samples of 781 tokens share tiles: element-wise V^T
    (512, 128, (16, 7, 38, 42), 1),     # 192 x 128 tiles
    (512, 64, (16, 4, 38, 38), 2)])
def test_fused_qkv_on_small_tiles_equals_separate_preparation(hidden, head_dim, latent, batch):
    """Projections that do not fill a dispatch round of 256 x 256 tiles, fused on
    the tiles they take instead, against the separate kernels bit for bit."""
    torch = torch_cuda()
    import paper_2608_01845_amd as wdc
    cfg = small_cfg("bf16", head_dim=head_dim, hidden=hidden, heads=hidden // head_dim, latent=latent)
    fused = wdc.Context(cfg, max_batch=batch)
    fused.load_weights(synth.gen_weights(cfg))
    os.environ["WDC_FUSE_QKV"] = "0"
    try:
        sep = wdc.Context(cfg, max_batch=batch, allocate_weights=False)
    finally:
        del os.environ["WDC_FUSE_QKV"]
    sep.bind_weights(fused.weights)
    zs = [torch.from_numpy(synth.gen_tensor(s, "z", cfg.latent)).cuda() for s in range(batch)]
    inp = {k: [fused.to_device(v)] * batch for k, v in synth.gen_inputs(cfg).items()}
    vf = fused.forward_batch(zs, 0.4, inp["cond"], inp["text"], inp["cam"])
    vs = sep.forward_batch(zs, 0.4, inp["cond"], inp["text"], inp["cam"])
    for a, b in zip(vf, vs):
        assert torch.isfinite(a).all() and torch.equal(a, b)


# tokens per sample are no multiple of 16, so a part of a product starts inside a sample. 4 x
# 4,125 rows: the last 116 run apart, on 128 x 128 tiles (q/k/v) and 64 x 64 ones; 4 x 4,421
# rows: 1,300 apart; 10 x 4,421: the last two chunks of the rectangle order apart, columns too.
# The gated products run as a batch of one per sample, with rows of each sample apart.
@pytest.mark.parametrize("latent,batch,head_dim", [
    ((16, 6, 36, 76), 4, 64), ((16, 11, 40, 40), 4, 128), ((16, 11, 40, 40), 10, 64)])
def test_split_last_rounds_of_a_batch_bitwise_equal(latent, batch, head_dim):
    """A batched forward whose large products run their last rows as a second launch: with the
    fused q/k/v epilogue against the separate kernels, and each sample against its forward
    alone (attention without key ranges, whose plan follows the number of heads)."""
    torch = torch_cuda()
    import paper_2608_01845_amd as wdc
    cfg = small_cfg("bf16", head_dim=head_dim, hidden=1024, heads=1024 // head_dim, latent=latent)
    os.environ["WDC_ATTN_SPLITS"] = "1"
    try:
        fused = wdc.Context(cfg, max_batch=batch)
        os.environ["WDC_FUSE_QKV"] = "0"
        sep = wdc.Context(cfg, max_batch=batch, allocate_weights=False)
    finally:
        del os.environ["WDC_ATTN_SPLITS"]
        os.environ.pop("WDC_FUSE_QKV", None)
    fused.init_random_weights(seed=5, std=0.02)
    sep.bind_weights(fused.weights)
    g = torch.Generator(device="cuda")
    g.manual_seed(batch)
    zs = [torch.randn(latent, generator=g, device="cuda") for _ in range(batch)]
    one = {k: fused.to_device(v) for k, v in synth.gen_inputs(cfg).items() if k != "z_T"}
    many = [[one[k]] * batch for k in ("cond", "text", "cam")]
    vf, vs = fused.forward_batch(zs, 0.4, *many), sep.forward_batch(zs, 0.4, *many)
    for b in range(batch):
        assert torch.isfinite(vf[b]).all() and torch.equal(vf[b], vs[b]), b
        assert torch.equal(vf[b], fused.forward(zs[b], 0.4, one["cond"], one["text"], one["cam"])), b
