"""The 4D queries where windows are too wide for lists and every element is
scanned: the resampling first tests the elements 64 at a time against each
sub-block (element counts on both sides of one and of several 64).  The
assignment is the oracle's bit for bit, and f by both schemes and the density
follow it."""
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
    print(f"[4d scan] ns={ns} nv={nv} ss={ss} sv={sv} {kw}", flush=True)
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
    (12, 12, 4, 4),              # 81 elements
    (16, 16, 4, 8),              # 64
    (20, 16, 4, 4),              # 400
    (32, 8, 4, 4),               # 256
    (36, 8, 4, 4),               # 324
])
@pytest.mark.parametrize("off", [0.0, 2.5])
def test_scan_of_every_element(orc, ns, nv, ss, sv, off):
    o, g = pair(ns, nv, ss, sv)
    rng = np.random.default_rng(ns + nv)
    el = o.get_elements().copy()
    E = el.shape[1]
    D = np.array([L / ns * ss] * 2 + [2.0 * VMAX / nv * sv] * 2)
    el[:4] += rng.uniform(-0.2, 0.2, (4, E)) * D[:, None]
    el[:2] %= L
    # sheared far beyond the ring: too wide for lists
    for a in range(2):
        el[4 + 4 * a + a + 2] += (8.0 * rng.uniform(0.5, 1.0, E) * D[a] /
                                  D[a + 2])
    if off > 0.0:
        # half of the elements off the square; the oracle's own search takes
        # them on it, so only the exhaustive assignment is compared
        el[:2, ::2] += rng.uniform(-off, off, (2, (E + 1) // 2)) * L
    o.set_elements(el)
    g.set_elements(el)
    if off > 0.0:
        assert np.array_equal(g.assignment().cpu().numpy(),
                              o.assignment(brute=True))
        g.sync()
        return
    compare(o, g)
