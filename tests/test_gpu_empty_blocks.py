"""Sphere blocks without a pair (spheres that share a body or are all static), with
no slot at all and with slots before the block: every kernel that tests the
block slot by slot, against the oracle (a step), the chain of steps (a rollout)
and the chain of step adjoints (its adjoint)."""
import numpy as np
import pytest

from oracle.cfo import Oracle
from paper_2603_12185_amd import scenes

from parity import compare_step, tdev, to_np

pytestmark = pytest.mark.gpu


def _scene(kind, nw):
    rng = np.random.default_rng(7)
    b = scenes._Builder(nw)
    body = dict(mass=0.5, inertia=(2e-4, 3e-4, 4e-4))
    if kind == "plane, one body":
        b.geom(scenes.PLANE, -1, friction=(0.6, 0.003, 0.0003))
    if kind in ("one body", "plane, one body"):
        f = b.body(scenes.JNT_FREE, pos=(0, 0, 0.045), **body)
        for r in (0.05, 0.03):
            b.geom(scenes.SPHERE, f, size=(r, 0, 0), friction=(0.6, 0.003, 0.0003))
    else:
        if kind == "box, static":  # slots: box-capsule twice, box-sphere per static sphere
            b.geom(scenes.BOX, b.body(scenes.JNT_FREE, pos=(0, 0, 0.06), **body), size=(0.05, 0.05, 0.02))
        jnt, at = (scenes.JNT_HINGE, 0.3) if kind == "hinge, static" else (scenes.JNT_FREE, 0.1)
        f = b.body(jnt, pos=(0, 0, at), axis=(0, 1, 0), ipos=(0.02 if jnt == scenes.JNT_HINGE else 0, 0, 0), **body)
        b.geom(scenes.CAPSULE, f, size=(0.02, 0.04, 0))
        for x in (-0.02, 0.02):
            b.geom(scenes.SPHERE, -1, size=(0.05, 0, 0), pos=(x, 0, 0), friction=(0.6, 0.003, 0.0003))
    s = b.build(condim=3, ncon_max=16)
    s["v0"][:] = rng.normal(0, 0.1, s["v0"].shape)
    return s


KINDS = ["one body", "plane, one body", "static", "box, static", "hinge, static"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("nw", [4, 2200, 3300])  # rollouts of one and three waves per SIMD, and beyond
def test_block_without_pairs(kind, nw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    print(f"case: block without pairs: {kind}, {nw} worlds", flush=True)
    s = _scene(kind, nw)
    m = cfsim.Model(s)
    q0, v0 = tdev(s["q0"]), tdev(s["v0"])
    oracle = Oracle(s)
    shown = range(4)
    found = 0
    for block in (64, 128, 256):
        m.set_launch(block, block, block)
        con = m.alloc_contacts()
        q1, v1 = m.step(q0, v0, contacts=con)
        st = compare_step(s, oracle, s["q0"], s["v0"], None, q1.cpu().numpy(), v1.cpu().numpy(), to_np(con),
                          worlds=shown)
        assert st["checked"] == len(shown)
        found = st["contacts"]
        T = 4
        q, v = m.rollout(T, q0, v0)
        a, b = q0, v0
        for t in range(T):
            a, b = m.step(a, b)
            # a few float32 roundings a step of coordinates and speeds of order one
            assert float((q[t + 1] - a).abs().max()) <= 4e-6 and float((v[t + 1] - b).abs().max()) <= 4e-6
        gq, gv = m.rollout_backward(T, q, v, None, torch.ones_like(q), torch.ones_like(v))
        x, y = torch.ones_like(q0), torch.ones_like(v0)
        for t in range(T - 1, -1, -1):
            x, y, _ = m.step_backward(q[t], v[t], None, x, y)
            x, y = x + 1, y + 1
        for got, ref in ((gq, x), (gv, y)):
            assert float((got.double() - ref.double()).norm() / ref.double().norm()) <= 1e-4
    assert (found > 0) == (kind in ("plane, one body", "box, static"))
