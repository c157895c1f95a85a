"""The step on two wavefronts per work item against the one-wavefront kernels.

Both advance an environment by the same formulas in the same order, so every
output is equal bit for bit (tolerance zero). A batch that fills the GPU runs
one wavefront per work item; its first environments alone are a small batch
that runs two. The sizes cover a single environment, a partly filled last
wavefront, and the largest batch that takes two wavefronts with the smallest
that does not; substep counts 1, odd and even cover the alternation of the
exchange rows.
"""
import re

import pytest
import torch

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
    rows = tape.view(T, 3, -1, 17, 64)[:, :, :E // per_wave, :, :per_wave * nb]
    assert torch.equal(st.view(T, 3, -1, 17, 64)[..., :per_wave * nb], rows)


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
