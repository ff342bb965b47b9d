"""The periodic spline fit gives the same coefficients every time: the rows'
ends, which every wavefront of a row's workgroup reads, are not replaced while
one of them is still to read them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nv", [(2048, 2084), (1024, 260)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_fit_repeats(nx, nv, precision):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[fit repeats] {nx}x{nv} {precision}", flush=True)
    g = vp.VlasovRun(nx=nx, nv=nv, x_min=-1.0, x_max=1.0, v_min=-1.0,
                     v_max=1.0, sx=4, sv=4, dt=1e-4, n_s=0, bc=1,
                     precision=precision)
    f = torch.as_tensor(np.random.default_rng(nx).uniform(0.5, 1.0, (nv, nx)),
                        device="cuda:0")
    ref = None
    for _ in range(300):
        g.init_conditions(f)
        got = g.reconstruct_f(1)
        if ref is None:
            ref = got
        assert torch.equal(got, ref)
