"""4D: elements off the periodic square by more than half a period (set by
the caller, or moved there by a drift longer than the period) whose windows
are wider than half of it.  A site sees an element through at most one period
per axis, as in the oracle's inverse map, so the image may lie further than
half a period away: the assignment equals the oracle's exhaustive one bit for
bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nv,ss,sv,shear", [
    (8, 8, 4, 4, 0.0), (8, 8, 4, 4, 1.0), (12, 8, 4, 4, 2.0),
    (16, 8, 4, 4, 3.0), (16, 8, 8, 4, 1.5), (32, 8, 8, 4, 3.0),
    (32, 8, 4, 4, 0.3)])
@pytest.mark.parametrize("reach", [1.0, 3.0])
def test_assignment_through_one_period(orc, ns, nv, ss, sv, shear, reach):
    import oracle.vp4 as o4
    import torch

    import paper_1705_03750_amd.vp4 as v4
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L, vmax = 6.0, 2.0
    p = dict(ns=ns, nv=nv, L=L, vmax=vmax, ss=ss, sv=sv, G=-0.5, dt=0.1)
    print(f"[4d far] ns={ns} nv={nv} ss={ss} sv={sv} shear={shear} "
          f"reach={reach}", flush=True)
    o, g = o4.Oracle4(**p), v4.VlasovRun4(device="cuda:0", **p)
    rng = np.random.default_rng(ns * 100 + nv + int(10 * shear))
    f0 = rng.uniform(0.5, 1.0, o.shape)
    o.init_conditions(f0)
    g.init_conditions(f0)
    el = o.get_elements().copy()
    E = el.shape[1]
    D = np.array([L / ns * ss] * 2 + [2.0 * vmax / nv * sv] * 2)
    el[:4] += rng.uniform(-0.2, 0.2, (4, E)) * D[:, None]
    el[:2] += rng.uniform(-reach, reach, (2, E)) * L
    for a in range(4):
        for b in range(4):
            d = rng.uniform(-0.05, 0.05, E)
            if b == a + 2:
                d = d + shear * rng.uniform(0.5, 1.0, E)
            el[4 + 4 * a + b] += d * D[a] / D[b]
    o.set_elements(el)
    g.set_elements(el)
    got, ref = g.assignment().cpu().numpy(), o.assignment(brute=True)
    assert np.array_equal(got, ref), int((got != ref).sum())
    g.sync()
