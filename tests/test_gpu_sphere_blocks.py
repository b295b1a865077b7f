"""The ways a block of spheres finds its pairs (slot by slot for few spheres, Gram
matrix on the matrix cores for up to 64 in one wave and 128 in two, lane by lane
otherwise) give the same contacts, bit for bit: every size around their limits,
spheres that touch exactly (pairs within the matrix's band), one sphere that is
not finite, more contacts than kept.  The workgroup of 256 threads tests lane by
lane above the slot-by-slot sizes and serves as the reference; a small
block is checked against the oracle.
"""
import numpy as np
import pytest

from oracle.cfo import Oracle
from paper_2603_12185_amd import scenes

pytestmark = pytest.mark.gpu


def spheres(n, worlds, seed, touching=False, ncon_max=1024):
    rng = np.random.default_rng(seed)
    b = scenes._Builder(worlds)
    b.geom(scenes.PLANE, -1)
    side = int(np.ceil(n ** (1 / 3)))
    at = np.array([[i, j, k] for k in range(side) for j in range(side) for i in range(side)], float)[:n]
    for i in range(n):
        r = np.full(worlds, 0.03125) if touching else rng.uniform(0.02, 0.05, worlds)
        m = 1000 * 4 / 3 * np.pi * r ** 3
        body = b.body(scenes.JNT_FREE, mass=m, inertia=np.repeat((0.4 * m * r * r)[:, None], 3, 1))
        b.geom(scenes.SPHERE, body, size=np.stack([r, 0 * r, 0 * r], 1), friction=(0.5, 0.003, 0.0003))
    s = b.build(ncon_max=ncon_max, name=f"spheres_{n}")
    q = s["q0"].reshape(worlds, n, 7)
    q[:, :, 0:3] = at * 0.0625 + 0.03125 if touching else at * 0.06 + rng.uniform(-0.01, 0.01, (worlds, n, 3)) + 0.03
    if touching:  # half the worlds a hair closer or wider than touching
        q[worlds // 2:, :, 0:3] *= 1 + 2.0 ** -22 * rng.integers(-3, 4, (worlds - worlds // 2, 1, 1))
    q[:, :, 3] = 1.0
    return s


def contacts(s, block, q=None):
    import torch
    from paper_2603_12185_amd import cfsim
    m = cfsim.Model(s)
    m.set_launch(block, 256, 256)
    q = torch.from_numpy(s["q0"] if q is None else q).cuda()
    con = m.alloc_contacts()
    m.step(q, torch.from_numpy(s["v0"]).cuda(), contacts=con)
    return {k: v.cpu().numpy() for k, v in con.items()}


def same(a, b):
    assert (a["ncon"] == b["ncon"]).all() and (a["overflow"] == b["overflow"]).all()
    keep = np.arange(a["geom"].shape[1])[None] < a["ncon"][:, None]
    for k in ("geom", "sub", "dist", "pos", "frame"):
        x, y = a[k][keep], b[k][keep]
        assert np.array_equal(x.view(np.int32), y.view(np.int32)), k


@pytest.mark.parametrize("n", [2, 3, 12, 13, 39, 40, 41, 47, 48, 49, 63, 64, 65, 79, 80, 81, 96, 127, 128, 129])
@pytest.mark.parametrize("touching", [False, True])
def test_same_contacts(n, touching):
    pytest.importorskip("torch")
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case: sphere block {n} touching {touching}", flush=True)
    s = spheres(n, 6, n, touching)
    ref = contacts(s, 256)
    assert touching or n < 4 or ref["ncon"].sum() > 0  # touching spheres may all stay apart
    for block in (64, 128):
        same(contacts(s, block), ref)
    if n == 41 and not touching:  # more contacts than kept: the same first ones
        s["ncon_max"] = 9
        ref = contacts(s, 256)
        assert (ref["overflow"] > 0).any()
        for block in (64, 128):
            same(contacts(s, block), ref)


@pytest.mark.parametrize("n", [20, 64, 100])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_one_sphere_not_finite(n, bad):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case: sphere block {n} with a coordinate {bad}", flush=True)
    s = spheres(n, 4, n)
    q = s["q0"].copy()
    q.reshape(4, n, 7)[1, n // 2, 1] = bad
    ref = contacts(s, 256, q)
    for block in (64, 128):
        got = contacts(s, block, q)
        same(got, ref)
        pairs = got["geom"][1, :got["ncon"][1]]
        assert got["ncon"][1] > 0 and not ((pairs == 1 + n // 2) & (pairs[:, :1] > 0)).any()


@pytest.mark.parametrize("n", [5, 40])
def test_small_blocks_match_the_oracle(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s = spheres(n, 4, 100 + n)
    got = contacts(s, 64)
    _, _, out = Oracle(s).step(s["q0"], s["v0"])
    assert (got["ncon"] == out["ncon"]).all() and got["ncon"].sum() > 0
    for w in range(4):
        k = got["ncon"][w]
        assert (got["geom"][w, :k] == out["geom"][w, :k]).all()
        # float32 centres and radii below 1 m: a few ulp of the coordinates
        assert np.abs(got["dist"][w, :k] - out["dist"][w, :k]).max() <= 4e-7
