"""Learned gains of a batch of more than twelve worlds per CU (eight worlds per
workgroup) against the same worlds in small batches (four per workgroup).  A
network of output biases alone has exact outputs: the same contacts, results to
float32 rounding (1e-6 of the largest value).  A network with weights: bf16
operands may round the other way where a feature's last bit differs, 2^-8 of each
of three layers' sums, |y| <= 0.5: gains, and the velocity change they cause,
within 0.6%."""
import numpy as np
import pytest

from oracle import mlp
from paper_2603_12185_amd import scenes

from parity import tdev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,condim", [(16, 3), (48, 6), (64, 1), (64, 4)])
@pytest.mark.parametrize("weights", [False, True])
def test_large_batch_equals_small(n, condim, weights):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    nw = 12 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    print(f"case: learned batch {nw} worlds of {n} condim {condim} weights {weights}", flush=True)
    rng = np.random.default_rng(n)
    s = scenes.dense_pile(nworld=nw, nsphere=n, seed=n, condim=condim)
    s["q0"].reshape(nw, n, 7)[:, :, 2] *= 0.8  # pressed together
    p = np.zeros(mlp.NPARAM, np.float32)
    if weights:
        p[:] = rng.uniform(-0.05, 0.05, mlp.NPARAM)
    p[mlp.OFF_STD:mlp.OFF_W1] = 1.0
    p[mlp.OFF_B3:] = rng.uniform(-0.3, 0.3, mlp.NPARAM - mlp.OFF_B3)

    def run(sc):
        m = cfsim.Model(sc)
        net = cfsim.ImpedanceNet(p)
        m.set_learned_impedance(net, margin=1e9)
        c = m.alloc_contacts()
        q, v = m.step(tdev(sc["q0"]), tdev(sc["v0"]), contacts=c)
        return q.view(sc["nworld"], -1), v.view(sc["nworld"], -1), c

    q1, v1, c1 = run(s)
    for idx in (np.arange(6), np.arange(nw - 9, nw)):
        q2, v2, c2 = run(scenes.select_worlds(s, idx))
        i = torch.as_tensor(idx, device="cuda")
        assert int(c2["ncon"].sum()) > 0
        for k in ("ncon", "geom"):
            assert torch.equal(c1[k][i], c2[k]), k
        if weights:
            dv = float((v2 - tdev(s["v0"][idx]).view_as(v2)).abs().max())
            assert float((v1[i] - v2).abs().max()) <= 0.006 * dv
        else:
            for x, y in ((q1[i], q2), (v1[i], v2), (c1["impulse"][i], c2["impulse"])):
                assert float((x - y).abs().max()) <= 1e-6 * max(1.0, float(y.abs().max()))
