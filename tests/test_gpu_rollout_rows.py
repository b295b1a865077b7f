"""autograd.rollout at sizes and with gradients whose rows do not begin on 16 bytes."""
import pytest

from paper_2603_12185_amd import scenes

from parity import tdev

pytestmark = pytest.mark.gpu


def _model(name):
    from paper_2603_12185_amd import cfsim
    kind, nw = name.split()[0], int(name.split()[-1])
    if kind == "hand":
        s = scenes.hand_cube(nworld=nw, seed=2)
    elif kind == "pushers":
        s = scenes.pusher_ball(nworld=nw, seed=2)
    else:  # a cluster of spheres per world
        s = scenes.select_worlds(scenes.sphere_cluster(nsphere=int(name.split()[1]), seed=2), [0] * nw)
    return s, cfsim.Model(s)


# rows of nworld*nq and nworld*nv floats off 16 bytes; models on either side of the persistent adjoint kernel
@pytest.mark.parametrize("name", ["hand 1", "hand 3", "spheres 41 3", "spheres 5 1025", "pushers 3"])
def test_one_step_of_odd_rows(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import autograd
    print(f"case: one step, {name}", flush=True)
    s, m = _model(name)
    assert m.nworld * m.nq % 4 or m.nworld * m.nv % 4
    q0, v0 = tdev(s["q0"]).requires_grad_(True), tdev(s["v0"]).requires_grad_(True)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    q, v = autograd.rollout(m, 1, q0, v0)
    gq_t = torch.randn(q.shape, generator=g, device="cuda")
    gv_t = torch.randn(v.shape, generator=g, device="cuda")
    gq, gv = torch.autograd.grad([q, v], [q0, v0], [gq_t, gv_t])
    a, b, _ = m.step_backward(q0.detach(), v0.detach(), None, gq_t[1].clone(), gv_t[1].clone())
    for x, y in ((gq, a + gq_t[0]), (gv, b + gv_t[0])):  # the same sums, but for one fused rounding
        assert float((x.double() - y.double()).norm() / y.double().norm()) <= 1e-6


# gradients that begin one to three floats into a buffer
@pytest.mark.parametrize("T", [1, 3])
@pytest.mark.parametrize("name", ["pushers 4", "hand 4", "spheres 41 4"])
def test_gradient_off_16_bytes(name, T):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import autograd
    print(f"case: gradient off 16 bytes, {name}, T {T}", flush=True)
    s, m = _model(name)
    q0, v0 = tdev(s["q0"]).requires_grad_(True), tdev(s["v0"]).requires_grad_(True)
    q, v = autograd.rollout(m, T, q0, v0)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    buf = torch.randn(3 + max(q.numel(), v.numel()), generator=g, device="cuda")
    ref = None
    for clone in (True, False):
        for k in (1, 2, 3):
            gq, gv = buf[k:k + q.numel()].view(q.shape), buf[4 - k:4 - k + v.numel()].view(v.shape)
            assert gq.data_ptr() % 16 and gv.data_ptr() % 16
            if clone:
                gq, gv = gq.clone(), gv.clone()
            out = torch.autograd.grad([q, v], [q0, v0], [gq, gv], retain_graph=True)
            if clone:
                ref = (ref or []) + [out]
            else:
                assert torch.equal(out[0], ref[k - 1][0]) and torch.equal(out[1], ref[k - 1][1])
    # the slice that a concatenation's gradient is
    cost = torch.cat((q.sum().view(1), q.flatten()))
    gq, = torch.autograd.grad(cost, [q0], torch.ones_like(cost))
    assert torch.isfinite(gq).all()
