"""The two-launch diagnostics at the edges of their grids (fewer workgroups
than shares, ragged element counts, more elements than threads), each force,
against the oracle to the 1e-10 of the parity tests; flags raised on the
device come back with the diagnostics."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nv,sx,sv,kw", [
    (8, 8, 4, 4, {}),
    (12, 131, 4, 1, dict(dt=2e-4)),
    (264, 60, 8, 4, dict(force_mode=1, ext=(0.1, -0.5, 0.2))),
    (512, 512, 1, 1, dict(dt=2e-4)),
    (1020, 1004, 4, 4, {}),
    (200, 72, 8, 8, dict(bc=1, G=-0.5)),
])
def test_against_oracle(orc, nx, nv, sx, sv, kw):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = dict(nx=nx, nv=nv, sx=sx, sv=sv, dt=kw.pop("dt", 1e-3), G=1.0)
    p.update(kw)
    print(f"[diag] {p}", flush=True)
    f0 = np.random.default_rng(nx + nv).uniform(0.5, 1.0, (nv, nx))
    o, g = orc.Oracle(**p), vp.VlasovRun(device="cuda:0", **p)
    o.init_conditions(f0)
    g.init_conditions(f0)
    o.step(2)
    g.step(2)
    ref, got = o.diagnostics(), g.diagnostics()
    for k in ("mass", "e_kin", "e_pot", "energy", "entropy", "l1", "l2"):
        assert abs(got[k] - ref[k]) <= 1e-10 * max(abs(ref[k]), abs(ref["e_kin"])), k
    assert abs(got["max_det_dev"] - ref["max_det_dev"]) <= 1e-13
    assert abs(got["emap"] - o.emap()) <= 1e-10
    assert got["step"] == 2 and got["overflow_blocks"] == 0
    g.close()


def test_flag_comes_back():
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = vp.VlasovRun(device="cuda:0", nx=64, sx=8, dt=1e-3)
    g.init_conditions(np.ones((64, 64)))
    el = g.get_elements().cpu().numpy()
    el[2, 3] = -1.0  # det T < 0
    g.set_elements(el)
    with pytest.raises(vp.VPError) as err:
        g.diagnostics()
    assert err.value.code == vp.ENUMERIC
    g.close()
