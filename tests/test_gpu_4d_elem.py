"""The 4D element pass with 1, 4 and 16 elements per workgroup, the last workgroup
full and partial: two steps from the initial condition and two of sheared
elements follow the oracle, the assignment of one state bit for bit.  A pass of
few sheared elements does not queue its claims in a few workgroups."""
import numpy as np
import pytest

from parity import MAP_TOL, map_gap4

pytestmark = pytest.mark.gpu

L, VMAX = 6.0, 2.0


def pair(ns, nv, ss, sv):
    import oracle.vp4 as o4
    import torch

    import paper_1705_03750_amd.vp4 as v4
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[4d elem] ns={ns} nv={nv} ss={ss} sv={sv}", flush=True)
    p = dict(ns=ns, nv=nv, L=L, vmax=VMAX, ss=ss, sv=sv, G=-0.5, dt=0.05)
    o, g = o4.Oracle4(**p), v4.VlasovRun4(device="cuda:0", **p)
    f = np.random.default_rng(ns * 100 + nv).uniform(0.5, 1.0, o.shape)
    o.init_conditions(f)
    g.init_conditions(f)
    D = np.array([L / ns * ss] * 2 + [2.0 * VMAX / nv * sv] * 2)
    return o, g, D


@pytest.mark.parametrize("ns,nv,ss,sv", [
    (12, 20, 4, 4),     # 225 elements: one per workgroup
    (16, 8, 2, 2),      # 1024, the most of these
    (20, 28, 4, 4),     # 1225, four per workgroup: the last takes one
    (20, 44, 2, 4),     # 12100, sixteen: the last takes four
])
def test_element_pass(orc, ns, nv, ss, sv):
    o, g, D = pair(ns, nv, ss, sv)
    rng = np.random.default_rng(ns + nv)
    for shear in (0.0, 0.4):
        if shear > 0.0:
            el = o.get_elements().copy()
            for a in range(2):
                el[4 + 4 * a + a + 2] += shear * rng.uniform(
                    0.5, 1.0, o.E) * D[a] / D[a + 2]
            o.set_elements(el)
            g.set_elements(el)
        o.step(2)
        g.step(2)
        gap = map_gap4(g.get_elements().cpu().numpy(), o.get_elements(), D)
        assert gap <= MAP_TOL, gap
        ref = o.reconstruct_f()
        assert np.abs(g.reconstruct_f().cpu().numpy() -
                      ref).max() <= 1e-12 * np.abs(ref).max()
    g.set_elements(o.get_elements())
    assert np.array_equal(g.assignment().cpu().numpy(), o.assignment())
    g.sync()


def test_claims_of_few_sheared_elements(orc):
    """25 elements after 30 steps of a plasma on a ring of 20 sites: the element
    pass takes at most the time of the reconstruction that reads its lists (98
    us against 36 when two workgroups made all the claims)."""
    import math

    import torch

    import paper_1705_03750_amd.vp4 as v4
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ns, nv = 20, 20
    print(f"[4d elem] claims of ns={ns} nv={nv}", flush=True)
    g = v4.VlasovRun4(device="cuda:0", ns=ns, nv=nv, L=4.0 * math.pi, vmax=4.0,
                      ss=4, sv=20, G=-0.5, dt=0.02)
    x = np.arange(ns) / ns * 2.0 * math.pi
    e = np.exp(-4.0 * np.linspace(-1.0, 1.0, nv) ** 2)
    f = np.einsum("w,u,y,x->wuyx", e, e, 1.0 + 0.1 * np.cos(x),
                  1.0 + 0.1 * np.cos(x))
    g.init_conditions(f / f.mean())
    g.step(30)
    g.reconstruct_f()
    ms = []  # the least of five: a launch may be held up by something else
    for _ in range(5):
        g.prof_begin(64)
        for _ in range(8):
            g.reconstruct_f()
        r = g.prof_end()
        ms.append((r["predict"][0], r["recon"][0]))
    predict, recon = (min(t) for t in zip(*ms))
    assert predict <= recon, ms
