"""Statistics kernels of the surrogate at the edges of their slice plan, and
the rollout's use of the caller's latent, against the oracle (GPU)."""
import numpy as np
import pytest

import synth
from oracle import params as P
from oracle import rollout as ro
from tests.gpu_util import context, rel_l2, torch_cuda, wdc_params
from tests.test_gpu_variants import compare, run_variant

pytestmark = pytest.mark.gpu


def _cfg(t):
    """A latent of 16 channels x t positions (no blocks: surrogate-only use)."""
    return synth.ModelConfig(name=f"t{t}", dtype="f32", hidden=256, heads=4, head_dim=64, latent=(16, 1, 1, t),
                             patch=(1, 1, t), rope=(0, 0, 0), steps=10, seed=17)


# segments (t / 8 positions) of one element and remainders, one slice, the last
# length of four 256-thread slices and the first of 1,024-thread ones, several of those
@pytest.mark.parametrize("t,overrides", [
    (9, {}), (8 * 61 + 3, {"bank_capacity": 8}), (8 * 4096 + 1, {"bank_capacity": 1}),
    (8 * 16384, {"observation": "linear", "bank_capacity": 3}), (8 * 16384 + 5, {"bank_capacity": 5}),
    (8 * 40000 + 7, {"surrogate": "secant"})])
def test_replay_rollout_at_slice_edges(t, overrides):
    run_variant(_cfg(t), 10, {"period": 3, **overrides}, "periodic")


def test_wave_sums_of_a_long_slice_are_added_without_loss():
    """One 1,024-thread slice per segment: the first wave's sum of |z| is 2^24, where adding
    the 1 of each of the other 15 waves would be lost in float32."""
    torch = torch_cuda()
    cfg = _cfg(8 * 16384 + 8)
    z_T, vel = np.zeros(cfg.latent, np.float32), np.zeros((2,) + cfg.latent, np.float32)
    z_T[0, 0, 0, 256 * np.arange(16)] = 1.0
    z_T[0, 0, 0, 0] = 2.0 ** 24
    vel[0, 0, 0, 0, 100] = 2.0 ** 20
    p = P.with_(P.DEFAULTS, theta_q=1.0, theta_sim=-1.0)
    ctx = context(cfg, weights=False, params=wdc_params(p))
    logs = ctx.rollout(ctx.new_state(), torch.from_numpy(z_T).cuda(), 2, mode=1, forced=[0, 0],
                       replay_v=torch.from_numpy(vel).cuda())[1]
    want = 0.5 * 2.0 ** 20 / (2.0 ** 24 + 15 + p.eps)     # mean |z_1 - z_0| over mean |z_0| (Eq. (6))
    assert abs(logs[1]["d_z"] - want) <= 1e-9 * want, (logs[1]["d_z"], want)


@pytest.mark.parametrize("steps,forced", [
    (1, [0]), (2, [0, 0]), (2, [0, 1]), (3, [0, 1, 1]), (5, [0, 0, 1, 1, 0]), (6, [0, 1, 0, 1, 0, 1])])
def test_rollout_writes_the_callers_latent_only_at_the_end(steps, forced):
    """Every way the last step can end (exact or surrogate, from the caller's
    latent or the library's), twice on one state: the second rollout starts
    from the first one's result."""
    torch = torch_cuda()
    cfg = _cfg(8 * 50 + 2)
    p = P.with_(P.DEFAULTS, theta_q=1.0, theta_sim=-1.0)
    vel = synth.gen_replay_velocities(cfg, steps)
    ctx = context(cfg, weights=False, params=wdc_params(p))
    st, z, ref_z = ctx.new_state(), None, synth.gen_inputs(cfg)["z_T"]
    z = torch.from_numpy(ref_z).cuda()
    for _ in range(2):
        ref = ro.rollout(ro.replay_denoiser(vel), ref_z, steps, p, mode="forced", forced=forced)
        sched, logs = ctx.rollout(st, z, steps, mode=1, forced=forced, replay_v=torch.from_numpy(vel).cuda())
        assert sched == ref.schedule == forced
        compare(logs, ref.log)
        assert rel_l2(z.cpu().numpy(), ref.z) <= 1e-5
        ref_z = z.cpu().numpy()


@pytest.mark.parametrize("forced", [[0, 1, 0], [0, 1, 1, 0]])
def test_rollout_leaves_the_callers_latent_alone_until_the_end(forced):
    """The velocity of the last step lies in the latent's own memory: nothing may be
    written there while the rollout can still read it, or fail."""
    torch = torch_cuda()
    cfg, steps = _cfg(8 * 50 + 2), len(forced)
    p = P.with_(P.DEFAULTS, theta_q=1.0, theta_sim=-1.0)
    vel = synth.gen_replay_velocities(cfg, steps)
    z_T = vel[-1].copy()
    ctx = context(cfg, weights=False, params=wdc_params(p))
    vd = torch.from_numpy(vel).cuda()
    ref = ro.rollout(ro.replay_denoiser(vel), z_T, steps, p, mode="forced", forced=forced)
    sched, logs = ctx.rollout(ctx.new_state(), vd[-1], steps, mode=1, forced=forced, replay_v=vd)
    assert sched == ref.schedule == forced
    compare(logs, ref.log)
    err = rel_l2(vd[-1].cpu().numpy(), ref.z)
    print(forced, err)
    assert err <= 1e-5


def test_rollout_of_an_unaligned_latent_has_the_same_bits():
    torch = torch_cuda()
    cfg, steps, forced = _cfg(8 * 4096 + 3), 4, [0, 1, 0, 1]
    ctx = context(cfg, weights=False, params=wdc_params(P.with_(P.DEFAULTS, theta_q=1.0, theta_sim=-1.0)))
    vd = torch.from_numpy(synth.gen_replay_velocities(cfg, steps)).cuda()
    z_T = torch.from_numpy(synth.gen_inputs(cfg)["z_T"]).cuda()
    buf = torch.empty(z_T.numel() + 3, device="cuda")
    out = []
    for shift in (0, 1, 3):
        z = buf[shift:shift + z_T.numel()].view_as(z_T)
        z.copy_(z_T)
        logs = ctx.rollout(ctx.new_state(), z, steps, mode=1, forced=forced, replay_v=vd)[1]
        out.append((z.clone(), [{k: v for k, v in lg.items() if v == v} for lg in logs]))   # (d_cf is NaN at first)
    for z, logs in out[1:]:
        assert torch.equal(z, out[0][0]) and logs == out[0][1]


def test_rollout_batch_from_another_states_bank_slot():
    """A latent that lies in the bank slot another sample's first exact step fills."""
    torch = torch_cuda()
    import paper_2608_01845_amd as wdc
    cfg, steps, B = _cfg(8 * 50 + 2), 3, 2
    p = P.with_(P.DEFAULTS, theta_q=1.0, theta_sim=-1.0)
    vels = [(b + 1) * synth.gen_replay_velocities(cfg, steps) for b in range(B)]
    z_T = [(b + 1) * synth.gen_inputs(cfg)["z_T"] for b in range(B)]
    ctx = wdc.Context(cfg, params=wdc_params(p), allocate_weights=False, max_batch=B)
    states = [ctx.new_state() for _ in range(B)]
    off = states[0].bank_slot(0)[0] - states[0].mem.data_ptr()
    slot = states[0].mem[off:off + 4 * z_T[1].size].view(torch.float32).view(cfg.latent)
    slot.copy_(torch.from_numpy(z_T[1]))
    zs = [torch.from_numpy(z_T[0]).cuda(), slot]
    forced = [[0, 0, 0]] * B
    scheds, logs = ctx.rollout_batch(states, zs, steps, mode=1, forced=forced,
                                     replay_vs=[torch.from_numpy(v).cuda() for v in vels])
    for b in range(B):
        ref = ro.rollout(ro.replay_denoiser(vels[b]), z_T[b], steps, p, mode="forced", forced=forced[b])
        compare(logs[b], ref.log)
        assert rel_l2(zs[b].cpu().numpy(), ref.z) <= 1e-5, b
