"""The spline fit with each number of tiles per segment: grids just inside and
outside a tile, ragged last segments, and lines whose extension tile is the
short end of the line.  At t = 0 the origin scheme evaluates the spline at the
sites themselves, where it must return f0 (the outermost ring zeroed)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# FP64 tiles per segment (x, v) 1/1, 1/1, 2/2, 4/4, 4/8, 8/8; the widths leave
# ends of 4, 28 and 0 positions in a tile of 32, and of 4 to 60 in one of 64
SIZES = [(8, 8), (68, 36), (996, 1020), (1028, 1980), (2052, 1284),
         (2048, 2084)]


@pytest.mark.parametrize("nx,nv", SIZES)
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_fit_returns_the_data(nx, nv, bc, precision):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if bc:
        nx = (nx + 7) // 8 * 8
    print(f"[fit] {nx}x{nv} bc={bc} {precision}", flush=True)
    g = vp.VlasovRun(nx=nx, nv=nv, x_min=-1.0, x_max=1.0, v_min=-1.0,
                     v_max=1.0, sx=4, sv=4, dt=1e-4, n_s=0, bc=bc,
                     precision=precision)
    f = np.random.default_rng(nx + nv).uniform(0.5, 1.0, (nv, nx))
    g.init_conditions(f)
    f[0] = f[-1] = 0.0
    if not bc:
        f[:, 0] = f[:, -1] = 0.0
    got = g.reconstruct_f(1).cpu().numpy().astype(np.float64)
    # |c| <= 9 max f (each inverse has row sums of at most 3); 32 roundings
    # of the fit and the 16-point sum, and sites known to 4 n u grid steps
    # (in double at either precision), where the slope is at most 2 max |c|
    u = 2.0 ** -24 if precision == "mixed" else 2.0 ** -53
    tol = 9 * (32 * u + 8 * max(nx, nv) * 2.0 ** -53)
    assert np.abs(got - f).max() <= tol
