"""The spline fit in segments of 1, 2, 4 and 8 tiles, in each precision and each
pass, with the same and with different lengths along x and v.  At t = 0 the
origin scheme evaluates the spline at the sites themselves, where it must
return f0 (the outermost ring zeroed)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = {"fp64": [(996, 1020), (1284, 1284), (1380, 1068), (1284, 1508),
                  (2052, 1284), (260, 1284)],
         "mixed": [(996, 1020), (1284, 1980), (2052, 2084), (2436, 1604),
                   (2884, 3012), (2692, 2884)]}


def tiles_per_segment(n, lines, precision):
    """The fewest of 1, 2, 4 and 8 tiles (32 positions of doubles, 64 of
    floats) that keep a pass over lines of n positions, 64 to a workgroup, at 8
    workgroups per position of a tile."""
    width = 64 if precision == "mixed" else 32
    chunks, tiles, t = -(-lines // 64), -(-n // width), 1
    while t < 8 and chunks * -(-tiles // t) > 8 * width:
        t *= 2
    return t


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_sizes_cover_every_length(precision):
    x = {tiles_per_segment(nx, nv, precision) for nx, nv in SIZES[precision]}
    v = {tiles_per_segment(nv, nx, precision) for nx, nv in SIZES[precision]}
    assert x == v == {1, 2, 4, 8}, (x, v)


@pytest.mark.parametrize("precision,nx,nv", [
    (p, nx, nv) for p in SIZES for nx, nv in SIZES[p]])
@pytest.mark.parametrize("bc", [0, 1])
def test_fit_returns_the_data(precision, nx, nv, bc):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if bc:
        nx = (nx + 7) // 8 * 8
    print(f"[fit segments] {nx}x{nv} bc={bc} {precision}", flush=True)
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
