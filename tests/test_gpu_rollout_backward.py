"""cf_rollout_backward against the chain of cf_step_backward calls and adds that
it stands for: worlds of free bodies (one persistent kernel; contact records in
LDS up to 128 slots, else in the workspace; contacts dropped beyond ncon_max;
sphere blocks on both sides of the slot-by-slot pair test), diagonal impedance,
learned gains and articulated models (step calls).

Both sides differentiate the same float32 states, so only float32 rounding
differs: a step's gradient to a few 2^-24, which the chain multiplies by the
growth of the adjoint over its steps (at most about a hundredfold here): 1e-4 of
each gradient's norm.
"""
import numpy as np
import pytest

from paper_2603_12185_amd import scenes

pytestmark = pytest.mark.gpu


def _pile(n, worlds, seed, condim=3, **kw):
    s = scenes.dense_pile(worlds, 16 * ((n + 15) // 16), seed=seed, condim=condim, **kw)
    if s["nbody"] != n:
        s = _first(s, n)
    q = s["q0"].reshape(worlds, n, 7)
    q[:, :, 0:3] *= 0.62  # overlapping: contacts from the first step
    return s


def _first(s, n):
    out = dict(s, nbody=n, ngeom=s["ngeom"] - s["nbody"] + n)
    for k in ("body_parent", "body_jnt", "body_pos", "body_quat", "body_ipos", "jnt_axis"):
        out[k] = s[k][:n]
    for k in ("geom_type", "geom_body"):
        out[k] = s[k][:out["ngeom"]]
    for k in ("body_mass", "body_inertia"):
        out[k] = s[k][:, :n]
    for k in ("geom_size", "geom_pos", "geom_quat", "geom_friction"):
        out[k] = s[k][:, :out["ngeom"]]
    out["q0"], out["v0"] = s["q0"][:, :7 * n].copy(), s["v0"][:, :6 * n].copy()
    return out


CASES = {
    "pusher_c6": lambda: scenes.pusher_ball(nworld=8, seed=2),
    "pusher_capped": lambda: scenes.pusher_ball(nworld=8, seed=2, ncon_max=3),
    "one_sphere": lambda: scenes.sphere_on_plane(nworld=4, z0=0.0495),
    "mixed_c4": lambda: scenes.mixed_shapes(nworld=8, seed=3, condim=4),
    "pile16_c1": lambda: _pile(16, 4, 1, condim=1),
    "pile33": lambda: _pile(33, 4, 2),
    "pile40_c6": lambda: _pile(40, 4, 3, condim=6),
    "pile41": lambda: _pile(41, 4, 4),
    "pile64": lambda: _pile(64, 4, 5),
    "pile64_capped": lambda: _pile(64, 4, 5, ncon_max=70),
    "pile24_diag": lambda: dict(_pile(24, 4, 6, condim=4), impedance=1),
    "hand_c6": lambda: scenes.hand_cube(nworld=4, seed=4),
    "pile16_learned": lambda: _pile(16, 4, 7),
}


@pytest.mark.parametrize("name", list(CASES))
def test_rollout_backward_is_the_chain(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim, learned
    print(f"case: rollout backward {name}", flush=True)
    s = CASES[name]()
    m = cfsim.Model(s)
    rng = np.random.default_rng(len(name))
    if name.endswith("learned"):
        f = rng.normal(0, 0.02, (512, 8)).astype(np.float32)
        m.set_learned_impedance(cfsim.ImpedanceNet(learned.init_params(torch.from_numpy(f))), margin=1e-4)
    T = 4
    q0, v0 = torch.from_numpy(s["q0"]).cuda(), torch.from_numpy(s["v0"]).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    tau = 0.02 * torch.randn((T, m.nworld, m.nv), generator=g, device="cuda") if "pile" not in name else None
    q, v = m.rollout(T, q0, v0, tau)
    gq_t = torch.randn(q.shape, generator=g, device="cuda")
    gv_t = torch.randn(v.shape, generator=g, device="cuda")
    for gqt, gvt in ((gq_t, gv_t), (None, gv_t), (gq_t, None)):
        gtau = torch.full((T, m.nworld, m.nv), float("nan"), device="cuda")
        gq, gv = m.rollout_backward(T, q, v, tau, gqt, gvt, gtau)
        z = torch.zeros_like
        rq, rv = (gqt[T] if gqt is not None else z(q0)).clone(), (gvt[T] if gvt is not None else z(v0)).clone()
        rtau = torch.empty_like(gtau)
        for t in range(T - 1, -1, -1):
            a, b, c = m.step_backward(q[t], v[t], None if tau is None else tau[t], rq, rv)
            rtau[t] = c
            rq = a + (gqt[t] if gqt is not None else 0)
            rv = b + (gvt[t] if gvt is not None else 0)
        for x, y in ((gq, rq), (gv, rv), (gtau, rtau)):
            rel = float((x.double() - y.double()).norm() / y.double().norm())
            print(f"{name}: rel {rel:.2e}")
            assert rel <= 1e-4
        again = m.rollout_backward(T, q, v, tau, gqt, gvt)
        assert torch.equal(again[0], gq) and torch.equal(again[1], gv)  # same run to run


def test_rollout_backward_arguments():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    m = cfsim.Model(scenes.sphere_on_plane(nworld=3))  # rows of 84 bytes: not 16-byte aligned
    q, v = (torch.zeros((3, 3, k), device="cuda") for k in (7, 6))
    q[..., 3] = 1.0
    with pytest.raises(cfsim.CFError):
        m.rollout_backward(2, q, v, None, q, v)
    with pytest.raises(cfsim.CFError):
        m.rollout_backward(0, q[:1], v[:1], None, None, None)
    with pytest.raises(ValueError):
        m.rollout_backward(2, q[:2], v, None, None, None)
    gq, gv = m.rollout_backward(1, q[:2], v[:2], None, None, torch.ones((2, 3, 6), device="cuda"))
    assert torch.isfinite(gq).all() and torch.isfinite(gv).all()
