"""A NaN or an infinity in one lateral velocity of a body that touches the ground.

A candidate whose slip is NaN takes its normal impulse and no friction, so the
NaN stays in that velocity and the position it moves: on the plain path, on one
and on two wavefronts per work item, with and without a tape, in the
environment layer's done flag alike. The expected pattern is the plain path's;
its finite values are compared within FP32 rounding of one step (1e-5 of a state
of order one; cotangents 1e-4, the repository's bound for two FP32 evaluations
of one adjoint).
"""
import numpy as np
import pytest
import torch

from paper_2106_13281_amd import braxmi

pytestmark = pytest.mark.gpu

HEAD = "substeps: 4\ndt: 0.004\ngravity { z: -9.81 }\nfriction: 0.8\n"
BODY = 'bodies {{ name: "{}" mass: 2 inertia {{ x: 0.02 y: 0.03 z: 0.04 }} colliders {{ {} }} }}\n'
SHAPES = {"sphere": "sphere { radius: 0.1 }", "capsule": "capsule { radius: 0.1 length: 0.5 }",
          "box": "box { halfsize { x: 0.2 y: 0.15 z: 0.1 } }"}
SYSTEMS = {k: HEAD + BODY.format("a", v) for k, v in SHAPES.items()}
SYSTEMS["pair"] = (HEAD + BODY.format("a", SHAPES["sphere"]) + BODY.format("b", SHAPES["capsule"]) +
                   'body_contacts { first: "a" second: "b" }\n')
PER_WAVE = {"sphere": 64, "capsule": 64, "box": 16, "pair": 32}


def scene(name, bad, E):
    s = braxmi.System(SYSTEMS[name], E, device=0)
    x = s.default_qp()
    low = 0.01 + 0.002                          # the clearance, then the lowest point in the ground
    x.pos[2] -= low
    if name == "pair":
        x.pos[0, 1] += 5.0                      # beyond each other's reach
    for b in range(x.pos.shape[1]):
        x.vel[0, b], x.vel[1, b], x.vel[2, b] = bad, 0.3, -0.5
    return s, x, torch.zeros(3, s.a_max, E, device=x.pos.device)


def same(got, want, tol, n):
    for f, r in zip(got.fields(), want.fields()):
        f, r = f[..., :n].cpu().numpy(), r[..., :n].cpu().numpy()
        assert np.array_equal(np.isnan(f), np.isnan(r)) and np.array_equal(np.isinf(f), np.isinf(r))
        ok = np.isfinite(r)
        np.testing.assert_allclose(f[ok], r[ok], rtol=tol, atol=tol)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", list(SYSTEMS))
def test_nonfinite_slip(name, bad):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 3
    s, x, acts = scene(name, bad, n)
    a0 = acts[0].contiguous()
    ref = s.step(x, a0, flags=braxmi.BRAX_PLAIN)
    want, _ = s.rollout(x, acts, flags=braxmi.BRAX_PLAIN)
    if np.isnan(bad):                           # the pattern: x alone
        assert torch.isnan(ref.vel[0]).all() and torch.isfinite(ref.vel[1:]).all() and torch.isfinite(ref.rot).all()
    same(s.step(x, a0), ref, 1e-5, n)
    same(s.rollout(x, acts)[0], want, 1e-5, n)
    same(s.rollout_tape(x, acts)[0], want, 1e-5, n)
    env = [dict(z_min=float(ref.pos[2].min()) - 1e-3, z_max=1.0)]
    s.env_configure(env)
    reset = s.default_qp()
    out, _, _, done = s.env_step(x, a0, reset)
    assert not done.any()
    same(out, ref, 1e-5, n)
    # one wavefront per work item: more items than the two-wavefront kernels take
    big, bx, bacts = scene(name, bad, (5 * n_cu + 1) * PER_WAVE[name])
    same(big.step(bx, bacts[0].contiguous()), ref, 1e-5, n)
    same(big.rollout_tape(bx, bacts)[0], want, 1e-5, n)
    big.env_configure(env)
    out, _, _, done = big.env_step(bx, bacts[0].contiguous(), big.default_qp())
    assert not done.any()
    same(out, ref, 1e-5, n)
    # the adjoint on three wavefronts: NaN nowhere that the one-wavefront
    # recomputing adjoint (with parameter cotangents) is finite, and there its values
    g = braxmi.State(*(torch.ones_like(f) for f in x.fields()))
    par = s.step_vjp_params(x, a0, g)[0]
    for f, r in zip(s.step_vjp(x, a0, g)[0].fields(), par.fields()):
        ok = torch.isfinite(r)
        assert torch.isfinite(f[ok]).all()
        torch.testing.assert_close(f[ok], r[ok], rtol=1e-4, atol=1e-4)
