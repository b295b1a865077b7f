"""Rollouts of articulated models with a block of spheres on either side of the
slot-by-slot pair test, at every workgroup size, against the chain of steps."""
import numpy as np
import pytest

from paper_2603_12185_amd import scenes

from parity import tdev

pytestmark = pytest.mark.gpu


def _scene(n, nw=8):
    rng = np.random.default_rng(n)
    b = scenes._Builder(nw)
    b.geom(scenes.PLANE, -1, friction=(0.6, 0.003, 0.0003))
    parent = -1
    for k in range(2):  # a two-link pendulum above the spheres
        parent = b.body(scenes.JNT_HINGE, parent, pos=(0, 0, 0.5) if k == 0 else (0.15, 0, 0), axis=(0, 1, 0),
                        ipos=(0.075, 0, 0), mass=0.2, inertia=(1e-4, 5e-4, 5e-4))
        b.geom(scenes.CAPSULE, parent, size=(0.015, 0.05, 0), pos=(0.075, 0, 0),
               quat=scenes._quat_z_to((1.0, 0.0, 0.0)), friction=(0.6, 0.003, 0.0003))
    b.geom(scenes.SPHERE, parent, size=(0.03, 0, 0), pos=(0.15, 0, 0), friction=(0.6, 0.003, 0.0003))
    for i in range(n):
        r = rng.uniform(0.02, 0.04, nw)
        m = 1000 * 4 / 3 * np.pi * r ** 3
        f = b.body(scenes.JNT_FREE, mass=m, inertia=(0.4 * m * r * r)[:, None] * np.ones(3))
        b.geom(scenes.SPHERE, f, size=np.stack([r, 0 * r, 0 * r], 1), friction=(0.5, 0.003, 0.0003))
    s = b.build(condim=3, ncon_max=512)
    side = int(np.ceil(n ** 0.5))
    at = np.array([[i % side, i // side, 0] for i in range(n)], float)
    q = s["q0"][:, 2:].reshape(nw, n, 7)
    q[:, :, 0:3] = 0.055 * at + rng.uniform(-0.003, 0.003, (nw, n, 3)) + [0, 0, 0.03]
    q[:, :, 3:7] = [1, 0, 0, 0]
    s["q0"][:, 2:] = q.reshape(nw, -1)
    s["q0"][:, :2] = rng.uniform(-0.2, 0.2, (nw, 2))
    s["v0"][:] = rng.normal(0, 0.05, s["v0"].shape)
    return s


@pytest.mark.parametrize("n", [2, 40, 41, 64, 65])
@pytest.mark.parametrize("block", [64, 128, 256])
def test_rollout_equals_steps(n, block):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    print(f"case: pendulum and {n} spheres, {block} threads", flush=True)
    s = _scene(n)
    m = cfsim.Model(s)
    m.set_launch(64, 64, block)
    T, q0, v0 = 5, tdev(s["q0"]), tdev(s["v0"])
    ncon = torch.zeros((T, m.nworld), dtype=torch.int32, device="cuda")
    q, v = m.rollout(T, q0, v0, ncon_traj=ncon)
    con = m.alloc_contacts()
    touching = 0
    for t in range(T):  # each step from the rollout's own state: one step's rounding apart
        q1, v1 = m.step(q[t], v[t], contacts=con)
        assert torch.equal(ncon[t], con["ncon"])
        touching += int(ncon[t].sum())
        # velocities of order one, the summation order of the workgroup size
        assert float((v[t + 1] - v1).abs().max()) <= 1e-5 * max(1.0, float(v1.abs().max()))
        assert float((q[t + 1] - q1).abs().max()) <= 1e-6
    assert touching > 0
