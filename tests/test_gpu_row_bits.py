"""A product's rows do not depend on their company: the same row of A gives the same
bits whatever the number of rows of the call, on every tile form (GPU)."""
import pytest

import synth
from tests.gpu_util import context, small_cfg, torch_cuda

pytestmark = pytest.mark.gpu


def _linear(ctx, a, w, b, m):
    torch = torch_cuda()
    out = torch.full((m, w.shape[0]), 7.0, dtype=a.dtype, device="cuda")
    ctx.linear(a, w, b, out, m, w.shape[0], w.shape[1])
    return out


def _operands(dtype, m, n, k, seed):
    torch = torch_cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    ctx = context(synth.get_config("mid" if dtype == "bf16" else "tiny"), weights=False)
    a, w, b = (torch.randn(s, generator=g, device="cuda") * f for s, f in (((m, k), 1.0), ((n, k), 0.05), ((n,), 0.1)))
    return ctx, a.to(ctx.tdtype), w.to(ctx.tdtype), b.to(ctx.tdtype)


# lone 64 x 64 blocks, 96 x 128, 128 x 128, 192 x 128, 256 x 128 and 256 x 256 with a split last round
@pytest.mark.parametrize("n,k", [(3072, 4096), (1024, 1088), (64, 640)])
def test_linear_bf16_rows_keep_their_bits(n, k):
    torch = torch_cuda()
    ctx, a, w, b = _operands("bf16", 6000, n, k, n + k)
    whole = _linear(ctx, a, w, b, 6000)
    for m in (1, 63, 64, 226, 400, 700, 1400, 2688, 3500, 5000):
        assert torch.equal(_linear(ctx, a, w, b, m), whole[:m]), m


def test_linear_bf16_split_rows_keep_their_bits():
    """The last 100 rows of this product run as a launch of their own: the same rows
    as the first 100 there, and alone."""
    torch = torch_cuda()
    ctx, a, w, b = _operands("bf16", 2148, 8192, 8192, 5)
    a[2048:] = a[:100]
    out = _linear(ctx, a, w, b, 2148)
    assert torch.equal(out[2048:], out[:100])
    assert torch.equal(_linear(ctx, a, w, b, 100), out[:100])


# 16 x 16, 32 x 32, 64 x 64 and 128 x 64 tiles; K of one stage, and of parts that start inside a stage
@pytest.mark.parametrize("n,k", [(1024, 1024), (1000, 32), (256, 544), (72, 96)])
def test_linear_f32_rows_keep_their_bits(n, k):
    torch = torch_cuda()
    ctx, a, w, b = _operands("f32", 6000, n, k, n + k)
    whole = _linear(ctx, a, w, b, 6000)
    for m in (1, 17, 64, 226, 300, 700, 1400, 1921, 2688, 5000):
        assert torch.equal(_linear(ctx, a, w, b, m), whole[:m]), m


def test_forward_f32_sample_keeps_its_bits_in_a_batch():
    """Five samples of a float32 model against each alone: the batched products run on larger tiles."""
    torch = torch_cuda()
    import paper_2608_01845_amd as wdc
    cfg = small_cfg("f32", latent=(16, 5, 14, 18))
    ctx = wdc.Context(cfg, max_batch=5)
    ctx.load_weights(synth.gen_weights(cfg))
    inp = synth.gen_inputs(cfg)
    zs = [torch.from_numpy(synth.gen_tensor(b, "z", cfg.latent)).cuda() for b in range(5)]
    one = {key: ctx.to_device(v) for key, v in inp.items() if key != "z_T"}
    outs = ctx.forward_batch(zs, 0.4, *([one[key]] * 5 for key in ("cond", "text", "cam")))
    for b in range(5):
        assert torch.equal(outs[b], ctx.forward(zs[b], 0.4, one["cond"], one["text"], one["cam"])), b
