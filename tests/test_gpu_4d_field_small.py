"""The 4D field on either side of the size up to which one workgroup forms all
of it: the force of a given density and the density of a run, against the
oracle.  The force is the same sums in the same order, bit for bit; the
density's sites agree in assignment and differ by roundings of the
interpolation only (1e-12, the parity bar of the 4D tests)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nv", [(8, 4), (12, 36), (16, 12), (24, 12)])
def test_field(orc, ns, nv):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle.vp4 as o4
    import paper_1705_03750_amd.vp4 as v4
    p = dict(ns=ns, nv=nv, L=5.0, vmax=2.0, ss=4, sv=4, G=-0.5, dt=0.05)
    print(f"[4d small field] ns={ns} nv={nv}", flush=True)
    o, g = o4.Oracle4(**p), v4.VlasovRun4(device="cuda:0", **p)
    rho = 1.0 + 0.3 * np.random.default_rng(ns).uniform(-1, 1, (ns, ns))
    for a, b in zip(g.field(rho), o.field(rho)):
        assert np.array_equal(a.cpu().numpy(), b)
    f0 = np.random.default_rng(nv).uniform(0.5, 1.0, o.shape)
    o.init_conditions(f0)
    g.init_conditions(f0)
    o.step(2)
    g.step(2)
    ref = o.density()
    assert np.abs(g.density().cpu().numpy() - ref).max() <= 1e-12 * ref.max()
    ref = o.reconstruct_f(0)
    assert np.abs(g.reconstruct_f(0).cpu().numpy() - ref).max() <= 1e-12
    g.sync()
