"""Rollouts of small batches of free bodies (state, constants and contacts held
on the chip) against repeated steps from each of their states: the same contact
counts, positions and velocities to float32 rounding (a step's result may differ
by a few 2^-24 where two compilations fuse a multiply and an add differently:
1e-6 of the largest value), with applied forces, overflowing contact capacity,
more than one chunk of contacts and batches of one and two worlds per SIMD.
And the trajectory's row 0 wherever the initial state lies."""
import numpy as np
import pytest

from paper_2603_12185_amd import scenes

from parity import tdev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scene,nw,cm", [("pusher", 1, 32), ("pusher", 7, 3), ("pusher", 1025, 32), ("mixed", 5, 64),
                                         ("pile", 6, 384), ("pile", 3, 70), ("pile64x6", 2, 384)])
def test_held_rollout_equals_steps(scene, nw, cm):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    print(f"case: held rollout {scene} worlds {nw} contacts {cm}", flush=True)
    if scene == "pusher":
        s = scenes.pusher_ball(nworld=nw, ncon_max=cm)
    elif scene == "mixed":
        s = scenes.mixed_shapes(nworld=nw, seed=3, condim=4)
    else:
        s = scenes.dense_pile(nworld=nw, nsphere=64, seed=4, ncon_max=cm)
        s["q0"].reshape(nw, 64, 7)[:, :, 2] *= 0.8  # pressed together: contacts from the first step
        if scene == "pile64x6":
            s = scenes.with_params(s, condim=6)
    m = cfsim.Model(s)
    assert m.get_launch()[3]
    T, rng = 6, np.random.default_rng(nw)
    q0, v0 = tdev(s["q0"]), tdev(s["v0"])
    tau = tdev(rng.normal(0, 0.01, (T, *s["v0"].shape)).astype(np.float32))
    n1 = torch.full((T, nw), -1, dtype=torch.int32, device="cuda")
    o1 = torch.full((T, nw), -1, dtype=torch.int32, device="cuda")
    qt, vt = m.rollout(T, q0, v0, tau_seq=tau, ncon_traj=n1, overflow_traj=o1)
    assert torch.equal(qt[0], q0) and torch.equal(vt[0], v0)
    for t in range(T):
        c = m.alloc_contacts()
        q, v = m.step(qt[t].clone(), vt[t].clone(), tau=tau[t].clone(), contacts=c)
        assert torch.equal(c["ncon"], n1[t]) and torch.equal(c["overflow"], o1[t]), t
        for x, y in ((q, qt[t + 1]), (v, vt[t + 1])):
            assert float((x - y).abs().max()) <= 1e-6 * max(1.0, float(y.abs().max())), t
    assert int(n1.sum()) > 0


@pytest.mark.parametrize("scene", ["pusher", "hand"])
def test_row0_wherever_the_state_lies(scene):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    s = scenes.pusher_ball(nworld=8) if scene == "pusher" else scenes.hand_cube(nworld=8)
    m = cfsim.Model(s)
    T = 3
    q0, v0 = tdev(s["q0"]), tdev(s["v0"])
    qr, vr = m.rollout(T, q0, v0)
    assert torch.equal(qr[0], q0) and torch.equal(vr[0], v0)
    nq, nv = q0.numel(), v0.numel()
    for at in (0, 1, T):  # the state in a row of the trajectory that is written
        qt = torch.zeros_like(qr)
        vt = torch.zeros_like(vr)
        qt[at], vt[at] = q0, v0
        m.rollout(T, qt[at], vt[at], q_traj=qt, v_traj=vt)
        assert torch.equal(qt, qr) and torch.equal(vt, vr), at
    # in no whole row of it (a row and four values in)
    qt = torch.zeros_like(qr)
    vt = torch.zeros_like(vr)
    qv, vv = qt.view(-1)[nq + 4:2 * nq + 4], vt.view(-1)[nv + 4:2 * nv + 4]
    qv.copy_(q0.view(-1))
    vv.copy_(v0.view(-1))
    m.rollout(T, qv.view_as(q0), vv.view_as(v0), q_traj=qt, v_traj=vt)
    assert torch.equal(qt, qr) and torch.equal(vt, vr)
