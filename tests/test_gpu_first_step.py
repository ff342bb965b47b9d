"""The first variable step from the column sums of the initial condition, at
the edges of their launches (row groups cut by the element lattice's offset,
fewer rows than a group, columns that do not fill a workgroup): dt = C_dyn /
sqrt(max rho), rho summed by numpy.  Two orders of n positive terms differ by
at most 2 n eps relative, dt by half of that and the rounding of the root."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nv,sx,sv", [
    (8, 8, 4, 4), (264, 60, 4, 4), (64, 68, 8, 4), (1020, 1004, 4, 4),
    (256, 128, 1, 1), (272, 272, 16, 16), (12, 131, 4, 1),
])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_first_step(nx, nv, sx, sv, precision):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[first step] {nx}x{nv} s={sx},{sv} {precision}", flush=True)
    f0 = np.random.default_rng(nx + nv).uniform(0.5, 1.0, (nv, nx))
    c = 0.1
    g = vp.VlasovRun(device="cuda:0", nx=nx, nv=nv, sx=sx, sv=sv, dt=1.0,
                     c_dyn=c, precision=precision)
    g.init_conditions(f0)
    got = g.diagnostics()["dt"]
    f = f0.copy()
    f[0] = f[-1] = 0.0
    f[:, 0] = f[:, -1] = 0.0
    if precision == "mixed":
        f = f.astype(np.float32).astype(np.float64)
    ref = c / np.sqrt((2.0 / nv) * f.sum(0).max())
    assert abs(got - ref) <= (nv + 4) * 2.0 ** -52 * ref
    g.close()
