"""4D grids of so few elements that no lists are kept, and those next to them:
the assignment is the oracle's bit for bit, and f by both schemes and the
density follow it; the element pass of such a grid does not grow with its
sites (it made all the claims in one workgroup)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L, VMAX = 6.0, 2.0


def pair(ns, nv, ss, sv, **kw):
    import oracle.vp4 as o4
    import torch

    import paper_1705_03750_amd.vp4 as v4
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[4d few] ns={ns} nv={nv} ss={ss} sv={sv} {kw}", flush=True)
    p = dict(ns=ns, nv=nv, L=L, vmax=VMAX, ss=ss, sv=sv, G=-0.5, dt=0.1)
    o, g = o4.Oracle4(**p), v4.VlasovRun4(device="cuda:0", **p, **kw)
    f0 = np.random.default_rng(ns * 100 + nv).uniform(0.5, 1.0, o.shape)
    o.init_conditions(f0)
    g.init_conditions(f0)
    return o, g


def compare(o, g):
    assert np.array_equal(g.assignment().cpu().numpy(), o.assignment())
    for scheme in (0, 1):
        ref = o.reconstruct_f(scheme)
        d = np.abs(g.reconstruct_f(scheme).cpu().numpy() - ref).max()
        assert d <= 1e-12 * np.abs(ref).max(), (scheme, d)
    rho = o.density()
    assert np.abs(g.density().cpu().numpy() - rho).max() <= 1e-12 * rho.max()
    g.sync()


@pytest.mark.parametrize("ns,nv,ss,sv", [
    (8, 4, 8, 4), (8, 8, 4, 4), (16, 16, 8, 8), (16, 16, 16, 4),
    (16, 16, 8, 4),              # 64 elements: the most without lists
    (12, 12, 4, 4),              # 81, three per ring: lists
    (8, 20, 4, 4),               # 100, two per ring: lists
])
def test_few_elements(orc, ns, nv, ss, sv):
    o, g = pair(ns, nv, ss, sv)
    compare(o, g)
    el = o.get_elements()
    o.step(4)
    g.step(4)
    got = g.get_elements().cpu().numpy()
    ref = o.get_elements()
    assert np.abs(got - ref).max() <= 1e-11 * np.abs(ref).max()
    assert not np.array_equal(ref, el)
    g.set_elements(ref)
    compare(o, g)


def test_element_pass_without_lists(orc):
    """16 elements of 32^4 sites: the element pass of the reconstruction takes
    at most three times that of 16 elements of 8^4 (both are one workgroup of
    the same arithmetic; with lists the larger made 65536 claims, 242 us
    against 13)."""
    ms = {}
    for ns, s in ((8, 4), (32, 16)):
        _, g = pair(ns, ns, s, s)
        g.reconstruct_f()
        t = []  # the least of five: a launch may be held up by something else
        for _ in range(5):
            g.prof_begin(64)
            for _ in range(8):
                g.reconstruct_f()
            t.append(g.prof_end()["predict"][0])
        ms[ns] = min(t)
    assert ms[32] <= 3.0 * ms[8], ms
