"""The 4D field and spline fit at the edges of their launches: rows shorter
and longer than a workgroup, the largest grid, lines that do not fill the
fit's LDS tile.  The force of a given density equals the oracle's bit for bit
(the same sums in the same order) where the two sides' tables do; the spline
of f0 reproduces the oracle's resampling value to 1e-12, the parity bar of the
4D tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def v4():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_03750_amd.vp4 as v4
    v4.lib()
    return v4


@pytest.mark.parametrize("ns", [8, 12, 60, 256, 260, 512])
def test_force(orc, v4, ns):
    import oracle.vp4 as o4
    L, G = 5.0, -0.5
    p = dict(ns=ns, nv=4, L=L, vmax=2.0, ss=4, sv=4, G=G, dt=0.1)
    rho = 1.0 + 0.3 * np.random.default_rng(ns).uniform(-1, 1, (ns, ns))
    print(f"[4d field] ns={ns}", flush=True)
    o, g = o4.Oracle4(**p), v4.VlasovRun4(device="cuda:0", **p)
    ref = o.field(rho)
    got = [a.cpu().numpy() for a in g.field(rho)]
    g.sync()
    if ns in (8, 12, 256, 512):
        for a, b in zip(got, ref):
            assert np.array_equal(a, b)
        return
    # at 60 and 260 a few entries of the two cosine and sine tables differ in
    # the last bit (the oracle's compiler merges the calls into sincos).  An
    # ulp u = 2^-52 in the tables moves rho^ by at most 2 u sum rho, which
    # |a^| = 2 |G| |rho^| / |k| and the inverse's 1 / n^2 carry into a, and
    # the two inverse transforms by 2 u of the spectrum's sum each.
    u = 2.0 ** -52
    k = 2 * np.pi * np.fft.fftfreq(ns, 1.0 / ns) / L
    k2 = np.hypot(*np.meshgrid(k, k))
    k2[0, 0] = np.inf
    fwd = 2 * u * rho.mean() * (2 * abs(G) / k2).sum()
    for a, b in zip(got, ref):
        spec = np.abs(np.fft.fft2(b)).sum() / ns ** 2
        assert np.abs(a - b).max() <= 2 * fwd + 4 * u * spec


@pytest.mark.parametrize("ns,nv", [(8, 4), (100, 4), (20, 12), (132, 4)])
def test_fit_lines(orc, v4, ns, nv):
    import oracle.vp4 as o4
    p = dict(ns=ns, nv=nv, L=5.0, vmax=2.0, ss=4, sv=4, G=-0.5, dt=0.1)
    o, g = o4.Oracle4(**p), v4.VlasovRun4(device="cuda:0", **p)
    f0 = np.random.default_rng(ns).uniform(0.5, 1.0, o.shape)
    print(f"[4d fit] ns={ns} nv={nv}", flush=True)
    o.init_conditions(f0)
    g.init_conditions(f0)
    o.step(1)  # off the nodes
    g.step(1)
    ref = o.reconstruct_f(1)
    got = g.reconstruct_f(1).cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
    g.sync()
