"""The step on two wavefronts per work item against the one-wavefront kernels,
and the adjoint on three against the oracle.

Both advance an environment by the same formulas in the same order, so every
output is equal bit for bit (tolerance zero). A batch that fills the GPU runs
one wavefront per work item; its first environments alone are a small batch
that runs two. The sizes cover a single environment, a partly filled last
wavefront, and the largest batch that takes two wavefronts with the smallest
that does not; substep counts 1, odd and even cover the alternation of the
exchange rows.
"""
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2106_13281_amd import braxmi, synth

pytestmark = pytest.mark.gpu

# (system, environments per full wavefront)
SYSTEMS = [("chain", 21), ("quadruped", 7), ("biped", 5), ("manipulator", 6), ("cheetah", 9), ("grasp", 6)]


def text(name, substeps):
    """The system's text with another substep count and the same substep length."""
    t = synth.system_text(name)
    n = int(re.search(r"^substeps: (\d+)", t, re.M).group(1))
    dt = float(re.search(r"^dt: ([\d.]+)", t, re.M).group(1))
    t = re.sub(r"^substeps: \d+", f"substeps: {substeps}", t, flags=re.M)
    return re.sub(r"^dt: [\d.]+", f"dt: {dt * substeps / n}", t, flags=re.M)


def inputs(system, seed, T):
    g = torch.Generator().manual_seed(seed)
    E, dev = system.n_envs, system.device

    def uni(*shape):
        return (torch.rand(*shape, generator=g) * 2 - 1).to(dev)

    s = system.default_qp(uni(system.d_max, E) * 0.1 + system.default_angles(0)[:, None].to(dev), uni(3, E) * 0.05)
    s.vel.add_(0.5 * uni(*s.vel.shape))
    s.ang.add_(0.5 * uni(*s.ang.shape))
    return s, uni(T, system.a_max, E)


def head(s, n):
    return braxmi.State(*(f[..., :n].contiguous() for f in s.fields()))


def equal(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("substeps", [1, 3, 4])
@pytest.mark.parametrize("name,per_wave", SYSTEMS)
def test_split_equals_one_wavefront(name, per_wave, substeps):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    limit = (3 if name == "grasp" else 5) * n_cu * per_wave   # the largest batch on two wavefronts
    T = 4
    big = braxmi.System(text(name, substeps), limit + 1, device=0)
    s, acts = inputs(big, 3, T)
    out, traj = big.rollout(s, acts, save_every=2, flags=braxmi.BRAX_NONFINITE_FLAGS)
    flags = big.nonfinite()
    env = [dict(z_min=0.15, z_max=0.6)]
    big.env_configure(env)
    reset = big.default_qp()
    eo, obs, rew, done = big.env_step(s, acts[0].contiguous(), reset)
    for E in (1, per_wave + 1, limit):
        small = braxmi.System(text(name, substeps), E, device=0)
        so, st = small.rollout(head(s, E), acts[..., :E].contiguous(), save_every=2, flags=braxmi.BRAX_NONFINITE_FLAGS)
        assert equal(so.fields(), head(out, E).fields())
        assert equal(st.fields(), head(traj, E).fields())
        assert torch.equal(small.nonfinite(), flags[:E])
        small.env_configure(env)
        x, o, r, d = small.env_step(head(s, E), acts[0, :, :E].contiguous(), head(reset, E))
        assert equal(x.fields(), head(eo, E).fields()) and torch.equal(d, done[:E])
        assert torch.equal(o, obs[:, :E]) and torch.allclose(r, rew[:E], rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("name,per_wave", SYSTEMS)
def test_split_tape(name, per_wave):
    """The taped step (one lane per body) and its state; the tape's rows of live lanes are equal."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    nb = {"chain": 3, "quadruped": 9, "biped": 11}.get(name, 7)
    per_wave = 64 // nb
    limit = (3 if name == "grasp" else 5) * n_cu * per_wave
    T = 2
    big = braxmi.System(text(name, 3), limit + 1, device=0)
    s, acts = inputs(big, 5, T)
    out, tape = big.rollout_tape(s, acts)
    E = limit
    small = braxmi.System(text(name, 3), E, device=0)
    so, st = small.rollout_tape(head(s, E), acts[..., :E].contiguous())
    assert equal(so.fields(), head(out, E).fields())
    def records(x):  # the live lanes' state and torque [..][4][lane][4], and contact counts [..][lane]
        r = x.view(T, 3, -1, 17 * 64)[:, :, :E // per_wave]
        return r[..., :1024].reshape(*r.shape[:3], 4, 64, 4)[..., :per_wave * nb, :], r[..., 1024:][..., :per_wave * nb]

    assert equal(records(st), records(tape))


def test_split_in_place_and_mixed():
    """out aliasing in, and a batch of several types around the limit."""
    names = list(synth.MIXED_TYPES)
    texts = [synth.system_text(n) for n in names]
    E = 20000
    types = torch.arange(E) % 4
    big = braxmi.System(texts, E, env_desc=types.tolist(), device=0)
    s = big.default_qp()
    acts = (torch.rand(3, big.a_max, E, generator=torch.Generator().manual_seed(1)) * 2 - 1).cuda()
    out, _ = big.rollout(s, acts)
    n = 4000
    small = braxmi.System(texts, n, env_desc=types[:n].tolist(), device=0)
    x = head(s, n)
    small.rollout(x, acts[..., :n].contiguous(), out=x)
    assert equal(x.fields(), head(out, n).fields())


# ------------------------------------------------------------------ adjoint
GRAD_TOL = 1e-3   # normwise per environment against the oracle, as in the adjoint's other parity tests
PAIR_TOL = 1e-4   # two FP32 evaluations of one adjoint, as tape against recompute there


def star(n, substeps):
    """A sphere with n links on hinges about it: more children than are gathered at once."""
    t = f"substeps: {substeps}\ndt: {0.001 * substeps}\ngravity {{ z: -9.81 }}\nfriction: 0.8\n"
    t += 'bodies { name: "hub" mass: 4 colliders { sphere { radius: 0.12 } } }\n'
    for i in range(n):
        t += (f'bodies {{ name: "l{i}" mass: 0.5 inertia {{ x: 0.004 y: 0.004 z: 0.004 }} '
              f"colliders {{ capsule {{ radius: 0.03 length: 0.2 }} }} }}\n")
    for i in range(n):
        a = 2 * np.pi * i / n
        x, y = np.cos(a), np.sin(a)
        t += (f'joints {{ name: "j{i}" parent: "hub" child: "l{i}" parent_offset {{ x: {0.12 * x:.6f} y: {0.12 * y:.6f} }} '
              f"child_offset {{ x: {-0.1 * x:.6f} y: {-0.1 * y:.6f} }} rotation {{ z: {np.degrees(a) + 90:.4f} }} "
              f"stiffness: 4000 damping: 6 angular_stiffness: 200 angular_damping: 0.2 limit_stiffness: 200 "
              f"angle_limit {{ min: -40 max: 40 }} }}\n")
    for i in range(n):
        t += f'actuators {{ name: "a{i}" joint: "j{i}" strength: 4 }}\n'
    return t


def check_vjp(text_, E, seed):
    o = oracle.Oracle(text_)
    nb, na = o.nb, o.na
    rng = np.random.default_rng(seed)
    X = np.stack([o.default_qp(o.system.default_angles() + rng.uniform(-0.1, 0.1, o.system.ndof)) for _ in range(E)])
    X[:, :, 2] -= 0.012                       # the lowest points in the ground
    X[:, :, 7:13] += rng.uniform(-0.5, 0.5, (E, nb, 6)) * np.concatenate([o.system.bodies[0]["free_pos"],
                                                                         o.system.bodies[0]["free_rot"]])
    X = X.astype(np.float32).astype(np.float64)
    act = rng.uniform(-1, 1, (E, na)).astype(np.float32)
    g = rng.normal(size=X.shape).astype(np.float32).astype(np.float64)
    ref_s, ref_a = o.step_vjp(X, act.astype(np.float64), g)
    _, mg = o.step(X, act.astype(np.float64), margins=True)
    clear = mg.min(1) >= 1e-6                 # away from jumps and kinks
    assert clear.sum() >= E // 2
    sysg = braxmi.System(text_, E, device=0)
    dev = lambda Y: braxmi.State(*(torch.from_numpy(a).cuda() for a in synth.to_soa(Y)))
    A = torch.from_numpy(np.ascontiguousarray(act.T)).cuda()
    ref = np.concatenate([ref_s.reshape(E, -1), ref_a], 1)
    _, tape = sysg.rollout_tape(dev(X), A[None].contiguous())
    for gi, ga in (sysg.step_vjp(dev(X), A, dev(g)), sysg.step_vjp_tape(tape[0], A, dev(g))):
        torch.cuda.synchronize()
        got = np.concatenate([synth.from_soa(*(f.cpu().numpy() for f in gi.fields()), n_body=nb).reshape(E, -1),
                              ga.cpu().numpy().T], 1)
        err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert (err[clear] < GRAD_TOL).all(), err[clear].max()


@pytest.mark.parametrize("children", [1, 3, 5, 7])
def test_star_vjp_matches_oracle(children):
    check_vjp(star(children, 3), 12, children)


@pytest.mark.parametrize("substeps", [1, 2, 31, 32])
def test_vjp_substep_counts_match_oracle(substeps):
    """One substep, an even and an odd count, and the counts around the LDS limit of the recomputing adjoint."""
    check_vjp(star(2, substeps), 6, substeps)


@pytest.mark.parametrize("children", [3, 6])
def test_star_split_equals_one_wavefront(children):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    limit = 5 * n_cu * (64 // (children + 1))
    big = braxmi.System(star(children, 5), limit + 1, device=0)
    s, acts = inputs(big, 7, 2)
    out, _ = big.rollout(s, acts)
    small = braxmi.System(star(children, 5), 50, device=0)
    so, _ = small.rollout(head(s, 50), acts[..., :50].contiguous())
    assert equal(so.fields(), head(out, 50).fields())


def test_pair_vjp_around_the_limit():
    """Body-body contacts: the largest batch on three wavefronts against the first environments of the next."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    E = 9 * n_cu
    big = braxmi.System(synth.system_text("grasp"), E + 1, device=0)
    s, acts = inputs(big, 9, 20)
    s, _ = big.rollout(s, acts)
    g = braxmi.State(*(torch.randn(f.shape, generator=torch.Generator().manual_seed(i)).cuda()
                       for i, f in enumerate(s.fields())))
    _, tape = big.rollout_tape(s, acts[:2].contiguous())
    bi, ba = big.rollout_vjp_tape(tape, acts[:2].contiguous(), g)
    ri, ra = big.step_vjp(s, acts[0].contiguous(), g)
    small = braxmi.System(synth.system_text("grasp"), E, device=0)
    A = acts[:2, :, :E].contiguous()
    _, tape = small.rollout_tape(head(s, E), A)
    si, sa = small.rollout_vjp_tape(tape, A, head(g, E))
    qi, qa = small.step_vjp(head(s, E), A[0].contiguous(), head(g, E))
    for x, y in ((si, head(bi, E)), (qi, head(ri, E))):
        for f, h in zip(x.fields(), y.fields()):
            d = (f - h).flatten(0, 1).norm(dim=0) / h.flatten(0, 1).norm(dim=0).clamp_min(1e-30)
            assert (d < PAIR_TOL).float().mean() > 0.99 and (f - h).norm() / h.norm() < PAIR_TOL
    assert (sa - ba[..., :E]).norm() / ba.norm() < PAIR_TOL and (qa - ra[:, :E]).norm() / ra.norm() < PAIR_TOL
