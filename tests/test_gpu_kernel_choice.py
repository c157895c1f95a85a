"""Where a call takes one kernel or another, by its size: the results on both
sides of each line, and against references that do not depend on it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2106_13281_amd import braxmi, synth
from test_gpu_split import PAIR_TOL, SYSTEMS, check_vjp, equal, head, inputs, star, text

pytestmark = pytest.mark.gpu


def n_cu():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("E", [50, 9000])  # two wavefronts per work item, one
def test_control_cost_rounding(E):
    """A three-axis joint's squared actions are added by fused multiply-adds in axis
    order and the bodies' in body order, on every kernel: exact (tolerance zero)."""
    name = "biped"
    o = oracle.Oracle(synth.system_text(name)).system
    s = braxmi.System(synth.system_text(name), E, device=0)
    x, acts = inputs(s, 4, 1)
    a = acts[0].contiguous()
    s.env_configure([dict(forward_weight=0.0, healthy_reward=0.0, ctrl_cost=1.0)])
    _, _, reward, _ = s.env_step(x, a, s.default_qp())
    a = a.cpu().numpy()
    ctrl = np.zeros(E, np.float32)
    for b in range(o.nb):
        sq = np.zeros(E, np.float32)
        for k, act in enumerate(o.actions):
            if o.joints[act[0]]["child"] == b:
                r = a[k].astype(np.longdouble)
                sq = (r * r + sq).astype(np.float32)
        ctrl += sq
    assert np.array_equal(reward.cpu().numpy(), -ctrl)


@pytest.mark.parametrize("name,per_wave", SYSTEMS)
def test_few_steps_around_the_line(name, per_wave):
    """Steps, environment steps and short rollouts take two wavefronts up to four work
    items per compute unit (three with body-body contacts), rollouts of four steps up
    to five: the last batch on two against the first environments of the next, and
    between the lines a short rollout against the first steps of a longer one (zero
    tolerance)."""
    E = (3 if name == "grasp" else 4) * n_cu() * per_wave
    big = braxmi.System(synth.system_text(name), E + 1, device=0)
    small = braxmi.System(synth.system_text(name), E, device=0)
    s, acts = inputs(big, 6, 4)
    x, a = head(s, E), acts[..., :E].contiguous()
    for T in (1, 3):
        out, _ = big.rollout(s, acts[:T].contiguous(), flags=braxmi.BRAX_NONFINITE_FLAGS)
        so, _ = small.rollout(x, a[:T].contiguous(), flags=braxmi.BRAX_NONFINITE_FLAGS)
        assert equal(so.fields(), head(out, E).fields()) and torch.equal(small.nonfinite(), big.nonfinite()[:E])
    _, traj = big.rollout(s, acts, save_every=1)        # four steps: two wavefronts
    assert equal(out.fields(), [f[2] for f in traj.fields()])
    for y in (big, small):
        y.env_configure([dict(z_min=0.15, z_max=0.6)])
    reset = big.default_qp()
    eo, obs, rew, done = big.env_step(s, acts[0].contiguous(), reset)
    so, o, r, d = small.env_step(x, a[0].contiguous(), head(reset, E))
    assert equal(so.fields(), head(eo, E).fields()) and torch.equal(d, done[:E])
    assert torch.equal(o, obs[:, :E]) and torch.equal(r, rew[:E])
    _, tape1 = big.rollout_tape(s, acts[:1].contiguous())   # taped: one wavefront for one step, two for more
    _, tape2 = big.rollout_tape(s, acts[:2].contiguous())
    g = head(s, E + 1)
    for f, h in zip(big.step_vjp_tape(tape1[0], acts[0].contiguous(), g)[0].fields(),
                    big.step_vjp_tape(tape2[0], acts[0].contiguous(), g)[0].fields()):
        assert torch.equal(f, h)


@pytest.mark.parametrize("name", [n for n, _ in SYSTEMS])
def test_vjp_around_the_line(name):
    """The largest batch whose single-step adjoint has room on the compute units with three
    wavefronts per work item (two items each; one with body-body contacts) against the first
    environments of the next, on one, and a partly filled work item, normwise as two FP32
    evaluations of one adjoint along the same forward values."""
    nb = {"chain": 3, "quadruped": 9, "biped": 11}.get(name, 7)
    E = (1 if name == "grasp" else 2) * n_cu() * (64 // nb)
    big = braxmi.System(synth.system_text(name), E + 1, device=0)
    s, acts = inputs(big, 9, 20)
    s, _ = big.rollout(s, acts)
    a = acts[0].contiguous()
    g = braxmi.State(*(torch.randn(f.shape, generator=torch.Generator().manual_seed(i)).cuda()
                       for i, f in enumerate(s.fields())))
    bi, ba = big.step_vjp(s, a, g)
    ref = torch.cat([f.flatten(0, 1) for f in bi.fields()] + [ba])
    for n in (E, 64 // nb + 1):
        small = braxmi.System(synth.system_text(name), n, device=0)
        si, sa = small.step_vjp(head(s, n), a[:, :n].contiguous(), head(g, n))
        r = ref[:, :n]
        d = torch.cat([f.flatten(0, 1) for f in si.fields()] + [sa]) - r
        assert (d.norm(dim=0) < PAIR_TOL * r.norm(dim=0)).float().mean() > 0.99 and d.norm() < PAIR_TOL * r.norm()


@pytest.mark.parametrize("substeps", [32, 33, 36, 37])
@pytest.mark.parametrize("name", ["star", "biped"])
def test_vjp_lds_limits_match_oracle(name, substeps):
    """The recomputing adjoint's LDS at 160 KiB: 32 substeps are the last on three wavefronts,
    33 and 36 the first and last on one, 37 the first per phase."""
    check_vjp(star(2, substeps) if name == "star" else text(name, substeps), 6, substeps)


def test_autotune_picks_no_block_shape_by_noise():
    """On two wavefronts per work item the block shape plays no part: the tuner's first stays."""
    s = braxmi.System(synth.system_text("quadruped"), 700, device=0)
    for _ in range(3):
        assert s.autotune()[1] == 1


@pytest.mark.parametrize("E", [40, 12000])  # two wavefronts per work item, one
@pytest.mark.parametrize("flags", [braxmi.BRAX_FUSED, braxmi.BRAX_PLAIN])
def test_trajectory_pads_with_zeros(E, flags):
    """A trajectory's body slots beyond a system's bodies are written as zeros, as every state's."""
    names = list(synth.MIXED_TYPES)
    s = braxmi.System([synth.system_text(n) for n in names], E, env_desc=(torch.arange(E) % len(names)).tolist(), device=0)
    x, acts = s.default_qp(), (torch.rand(3, s.a_max, E, generator=torch.Generator().manual_seed(8)) * 2 - 1).cuda()
    traj = s.new_state(lead=(3,))
    for f in traj.fields():
        f.fill_(float("nan"))
    s.rollout(x, acts, save_every=1, traj=traj, flags=flags)
    for t, n in enumerate(names):
        nb = oracle.Oracle(synth.system_text(n)).system.nb
        for f in traj.fields():
            assert torch.isfinite(f[:, :, :nb, t::len(names)]).all() and (f[:, :, nb:, t::len(names)] == 0).all()
