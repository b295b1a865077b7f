"""cf_step_backward on small articulated subtrees (one to four hinge or slide
bodies, computed by a quad of lanes and one lane per body and joint direction):
every subtree size, both joint types in either order, branching trees, position
actuators, and more subtrees than one pass of a workgroup's lanes covers, against
FP64 central differences of the oracle.  The tolerance is the other adjoint
tests': relative error of a world's whole gradient at most 1e-3 (float32 gradient,
differences of 1e-6 in float64).
"""
import numpy as np
import pytest

from oracle.cfo import Oracle  # noqa: F401  (the oracle is built by the session fixture)
from paper_2603_12185_amd import scenes

from adjoint_fd import step_grad_fd
from parity import tdev

pytestmark = pytest.mark.gpu
REL = 1e-3

H, S = scenes.JNT_HINGE, scenes.JNT_SLIDE
TREES = {  # per subtree: (joint type, parent within the subtree) of each body
    "h": [[(H, -1)]],
    "s": [[(S, -1)]],
    "hs": [[(H, -1), (S, 0)]],
    "sh": [[(S, -1), (H, 0)]],
    "hsh": [[(H, -1), (S, 0), (H, 1)]],
    "shhs": [[(S, -1), (H, 0), (H, 1), (S, 2)]],
    "branch": [[(H, -1), (H, 0), (S, 0), (H, 2)]],
    "fork": [[(S, -1), (H, 0), (H, 0), (H, 0)]],
    "mixed_sizes": [[(H, -1)], [(S, -1), (H, 0), (H, 1), (H, 2)], [(H, -1), (S, 0)]],
    "many": [[(H, -1), (H, 0), (S, 1), (H, 2)] if i % 2 else [(S, -1), (H, 0), (H, 0)] for i in range(12)],
}


def small_trees(trees, nworld, seed, actuated, condim):
    rng = np.random.default_rng(seed)
    b = scenes._Builder(nworld)
    b.geom(scenes.PLANE, -1, quat=scenes._quat_z_to((0.1, -0.05, 1.0)), friction=(0.6, 0.004, 0.0004))
    for i, tree in enumerate(trees):
        base = None
        for k, (jnt, parent) in enumerate(tree):
            ax = rng.normal(size=3)
            m = rng.uniform(0.1, 0.4, nworld)
            inertia = m[:, None] * rng.uniform(5e-4, 2e-3, 3)
            at = (0.6 * i, 0.0, 0.09) if parent < 0 else rng.uniform(0.03, 0.08, 3) * (1, 1, -0.3)
            body = b.body(jnt, -1 if parent < 0 else base + parent, pos=at, quat=scenes._random_quat(rng),
                          ipos=rng.uniform(-0.02, 0.02, 3), axis=ax / np.linalg.norm(ax), mass=m, inertia=inertia)
            base = body if base is None else base
            b.geom(scenes.SPHERE, body, size=(rng.uniform(0.08, 0.12), 0, 0), pos=rng.uniform(-0.02, 0.02, 3),
                   friction=(rng.uniform(0.4, 0.9), 0.003, 0.0003))
    s = b.build(condim=condim, ncon_max=64, name="small_trees")
    nq = scenes.dims(s)[0]
    s["q0"] = rng.uniform(-0.3, 0.3, (nworld, nq)).astype(np.float32) * np.where(
        np.array([s["body_jnt"][k] for k in range(s["nbody"])]) == H, 1.0, 0.05).astype(np.float32)
    s["v0"] = rng.normal(0, 0.4, (nworld, nq)).astype(np.float32)
    if actuated:
        s["dof_kp"] = scenes.f32(np.where(rng.random(nq) < 0.6, rng.uniform(0.5, 2.0, nq), 0.0))
        s["dof_kd"] = scenes.f32(np.where(rng.random(nq) < 0.6, rng.uniform(0.005, 0.02, nq), 0.0))
    return s


@pytest.mark.parametrize("name", list(TREES))
@pytest.mark.parametrize("actuated", [False, True])
def test_small_subtree_adjoint(name, actuated):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    print(f"case: small subtree adjoint {name} actuated {actuated}", flush=True)
    nw = 2
    s = small_trees(TREES[name], nw, sum(map(ord, name)), actuated, 6 if actuated else 3)
    rng = np.random.default_rng(len(name) + actuated)
    q, v = s["q0"], s["v0"]
    nv = v.shape[1]
    tau = rng.normal(0, 0.3, (nw, nv)).astype(np.float32)
    gq_out = rng.normal(size=q.shape).astype(np.float32)
    gv_out = rng.normal(size=v.shape).astype(np.float32)
    model = cfsim.Model(s)
    got = model.step_backward(tdev(q), tdev(v), tdev(tau), tdev(gq_out), tdev(gv_out))
    got = np.concatenate([g.cpu().numpy() for g in got], 1)
    ncon = 0
    for w in range(nw):
        g_fd, ok, out = step_grad_fd(s, w, q, v, tau, gq_out, gv_out)
        ncon += int(out["ncon"][0])
        rel = np.linalg.norm((got[w] - g_fd)[ok]) / np.linalg.norm(g_fd[ok])
        print(f"{name} world {w}: contacts {int(out['ncon'][0])}, kinked {int((~ok).sum())}, rel {rel:.2e}")
        assert ok.mean() > 0.5
        assert rel <= REL
    assert ncon > 0
