"""Every query outside the stepping loop leaves the block lists empty: the
same query twice over, and every other one in between, gives the same arrays
bit for bit (a list that kept its entries would hold every element twice and
overflow), also on grids whose last block row or row group is partial."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nv,sx,sv", [(8, 8, 4, 4), (68, 132, 4, 4),
                                         (264, 60, 8, 4), (48, 80, 16, 16)])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_queries_repeat(nx, nv, sx, sv, bc, precision):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nx = (nx + 7) // 8 * 8 if bc else nx
    print(f"[query clears] {nx}x{nv} bc={bc} {precision}", flush=True)
    g = vp.VlasovRun(nx=nx, nv=nv, sx=sx, sv=sv, x_min=-1.0, x_max=1.0,
                     v_min=-1.0, v_max=1.0, dt=1e-2, n_s=0, bc=bc,
                     precision=precision)
    f0 = np.random.default_rng(nx + nv).uniform(0.5, 1.0, (nv, nx))
    g.init_conditions(f0)
    g.step(2)
    queries = [g.density, g.assignment, g.reconstruct_f,
               lambda: g.reconstruct_f(vp.SCHEME_REMAP),
               lambda: torch.tensor(g.diagnostics()["emap"])]
    ref = [q() for q in queries]
    for _ in range(3):
        for k in (0, 1, 2, 3, 4, 3, 2, 1, 0):
            assert torch.equal(queries[k](), ref[k]), k
    assert g.diagnostics()["overflow_blocks"] == 0
    # and the run goes on as one that was never asked
    h = vp.VlasovRun(nx=nx, nv=nv, sx=sx, sv=sv, x_min=-1.0, x_max=1.0,
                     v_min=-1.0, v_max=1.0, dt=1e-2, n_s=0, bc=bc,
                     precision=precision)
    h.init_conditions(f0)
    h.step(5)
    g.step(3)
    assert torch.equal(g.reconstruct_f(), h.reconstruct_f())
