"""Periodic x: elements that lie more than a period off the box (set by the
caller, or moved there by a drift longer than the period, which re-enters by
one period only).  A site sees an element through at most one period, as in
the oracle's inverse map, so such an element serves the sites that this image
reaches and no others: the assignment equals the oracle's exhaustive one bit
for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nv,s", [(64, 32, 8), (96, 24, 4), (128, 64, 8)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_assignment_through_one_period(orc, nx, nv, s, precision):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L = 8.0
    p = dict(nx=nx, nv=nv, x_min=0.0, x_max=L, v_min=-2.0, v_max=2.0, sx=s,
             sv=s, G=-0.5, dt=0.05, n_s=0, bc=1)
    print(f"[far images] {nx}x{nv} s={s} {precision}", flush=True)
    rng = np.random.default_rng(nx + nv)
    f0 = rng.uniform(0.5, 1.0, (nv, nx))
    o = orc.Oracle(**p)
    g = vp.VlasovRun(device="cuda:0", precision=precision, **p)
    o.init_conditions(f0)
    g.init_conditions(f0)
    el = o.get_elements().copy()
    el[0] += rng.uniform(-0.2, 0.2, o.E) * L / nx * s
    # a third each: on the ring, off it by up to 1.5 periods, by 1.5 to 3
    off = rng.uniform(0.0, 1.5, o.E) * rng.choice((-1.0, 1.0), o.E)
    far = rng.uniform(1.5, 3.0, o.E) * rng.choice((-1.0, 1.0), o.E)
    kind = rng.integers(0, 3, o.E)
    el[0] += np.where(kind == 1, off, np.where(kind == 2, far, 0.0)) * L
    o.set_elements(el)
    g.set_elements(el)
    got, ref = g.assignment().cpu().numpy(), o.assignment(brute=True)
    assert (ref < 0).any() and (ref >= 0).any()
    assert np.array_equal(got, ref), int((got != ref).sum())


def test_drift_longer_than_the_period(orc):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # free streaming (G = 0), |v| dt up to 4 periods: after one step the
    # fastest elements lie almost two periods off the box; the windows, 8 + 64
    # columns to each side, stay narrow enough for lists
    p = dict(nx=256, nv=256, x_min=0.0, x_max=1.0, v_min=-4.0, v_max=4.0,
             sx=8, sv=8, G=0.0, dt=1.0, n_s=0, bc=1)
    print("[far images] one step of four periods", flush=True)
    f0 = np.random.default_rng(7).uniform(0.5, 1.0, (256, 256))
    o, g = orc.Oracle(**p), vp.VlasovRun(device="cuda:0", **p)
    for e in (o, g):
        e.init_conditions(f0)
        e.step(1)
    el = g.get_elements().cpu().numpy()
    assert np.array_equal(el, o.get_elements())
    assert np.abs(el[0] - 0.5).max() > 2.0
    assert np.array_equal(g.assignment().cpu().numpy(), o.assignment(True))
    assert np.abs(g.reconstruct_f().cpu().numpy() -
                  o.reconstruct_f()).max() <= 1e-12
