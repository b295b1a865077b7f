"""The one-kernel step of worlds of 65 to 128 free bodies (two waves) against the
two kernels it replaces: the same contacts, and every float32 result equal to
rounding (the compiler may fuse a multiply and an add differently in the two
compilations: a few 2^-24 of the largest value, 1e-6 allowed)."""
import numpy as np
import pytest

from paper_2603_12185_amd import scenes

from parity import tdev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,condim", [(65, 3), (80, 1), (96, 4), (128, 6), (128, 3)])
@pytest.mark.parametrize("impedance", [0, 1])
def test_two_wave_step_equals_two_kernels(n, condim, impedance):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    print(f"case: two-wave step {n} bodies condim {condim} impedance {impedance}", flush=True)
    rng = np.random.default_rng(n)
    b = scenes._Builder(5)
    b.geom(scenes.PLANE, -1)
    b.geom(scenes.PLANE, -1, pos=(-0.02, 0, 0), quat=scenes._quat_z_to((1, 0, 0.1)), friction=(0.3, 0.001, 0.0001))
    at = np.array([[i % 5, i // 5 % 5, i // 25] for i in range(n)], float) * 0.06 + 0.03
    for i in range(n):
        r = rng.uniform(0.02, 0.045, 5)
        m = 1000 * 4 / 3 * np.pi * r ** 3
        body = b.body(scenes.JNT_FREE, mass=m, inertia=(0.4 * m * r * r)[:, None] * np.array([1.0, 1.1, 0.9]))
        b.geom(scenes.SPHERE, body, size=np.stack([r, 0 * r, 0 * r], 1), friction=(0.6, 0.003, 0.0003))
    s = b.build(condim=condim, ncon_max=1024)
    q = s["q0"].reshape(5, n, 7)
    q[:, :, 0:3] = at + rng.uniform(-0.01, 0.01, (5, n, 3))
    q[:, :, 3:7] = rng.normal(size=(5, n, 4))
    s["v0"][:] = rng.normal(0, 0.2, s["v0"].shape)
    m = cfsim.Model(dict(s, impedance=impedance))
    assert m.step_kernels() == 1
    q0, v0 = tdev(s["q0"]), tdev(s["v0"])
    tau = tdev(rng.normal(0, 0.01, s["v0"].shape).astype(np.float32))
    c1, c2 = m.alloc_contacts(), m.alloc_contacts()
    q1, v1 = m.step(q0, v0, tau=tau, contacts=c1)
    m.set_launch(128, 256)
    assert m.step_kernels() == 2
    q2, v2 = m.step(q0, v0, tau=tau, contacts=c2)
    assert int(c1["ncon"].sum()) > 0
    for k in ("ncon", "overflow", "geom", "sub"):
        assert torch.equal(c1[k], c2[k]), k
    for x, y in [(q1, q2), (v1, v2)] + [(c1[k], c2[k]) for k in ("dist", "pos", "frame", "impulse")]:
        assert float((x - y).abs().max()) <= 1e-6 * max(1.0, float(x.abs().max()))
    # in place, as a program steps
    m.set_launch(128, 128)
    m.step(q0, v0, tau=tau, q_out=q0, v_out=v0)
    assert torch.equal(q0, q1) and torch.equal(v0, v1)
