"""Plane rows (static planes with their poses kept in the model) against the same
worlds with one more geom, a static box far from everything, which sends the
planes through the general slot path.  Planes tilted and placed differently in
every world.  The same contacts; distances, points and frames of coordinates of
order one to a few float32 roundings (1e-6 allowed)."""
import numpy as np
import pytest

from paper_2603_12185_amd import scenes

from parity import tdev

pytestmark = pytest.mark.gpu


def _worlds(nw, n, npl, per_world, box):
    rng = np.random.default_rng(100 * n + npl)
    b = scenes._Builder(nw)
    if box:
        b.geom(scenes.BOX, -1, pos=(50.0, 50.0, 50.0), size=(0.1, 0.1, 0.1))
    for k in range(npl):
        pos = rng.uniform(-0.02, 0.02, (nw if per_world else 1, 3))
        quat = rng.normal(0, 0.2, (nw if per_world else 1, 4)) + np.array([1.0, 0, 0, 0])
        quat /= np.linalg.norm(quat, axis=1, keepdims=True)
        b.geom(scenes.PLANE, -1, pos=np.broadcast_to(pos, (nw, 3)), quat=np.broadcast_to(quat, (nw, 4)))
    for i in range(n):
        r = rng.uniform(0.02, 0.04, nw)
        m = 1000 * 4 / 3 * np.pi * r ** 3
        body = b.body(scenes.JNT_FREE, mass=m, inertia=(0.4 * m * r * r)[:, None] * np.ones(3))
        b.geom(scenes.SPHERE, body, size=np.stack([r, 0 * r, 0 * r], 1))
    s = b.build(condim=3, ncon_max=2048)
    q = s["q0"].reshape(nw, n, 7)
    q[:, :, 0:3] = rng.uniform([-0.3, -0.3, 0.0], [0.3, 0.3, 0.06], (nw, n, 3))
    q[:, :, 3:7] = [1, 0, 0, 0]
    return s


@pytest.mark.parametrize("n,npl", [(2, 1), (41, 2), (64, 3), (65, 1), (128, 2), (200, 1)])
@pytest.mark.parametrize("per_world", [False, True])
def test_plane_rows_equal_plane_slots(n, npl, per_world):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    print(f"case: plane rows {n} spheres {npl} planes per world {per_world}", flush=True)
    out = []
    for box in (0, 1):
        s = _worlds(5, n, npl, per_world, box)
        m = cfsim.Model(s)
        c = m.alloc_contacts()
        m.step(tdev(s["q0"]), tdev(s["v0"]), contacts=c)
        out.append((s, c))
    (s, a), (_, b) = out
    assert int(a["overflow"].sum()) == 0 and torch.equal(a["ncon"], b["ncon"])
    planes = 0
    for w in range(5):
        k = int(a["ncon"][w])
        assert torch.equal(a["geom"][w, :k] + 1, b["geom"][w, :k])
        planes += int((a["geom"][w, :k] < npl).any(-1).sum())
        for key in ("dist", "pos", "frame"):
            assert float((a[key][w, :k] - b[key][w, :k]).abs().max() if k else 0.0) <= 1e-6, key
    assert planes > 0
