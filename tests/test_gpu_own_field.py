"""The element pass that forms the field itself (small grids) and the one that
takes it from a launch of its own, on either side of the rule's limits and
with ragged columns and row groups, isolated and periodic x, fixed and
variable step, against the oracle (parity.py's bars: f and rho 1e-12, elements
by their maps)."""
import numpy as np
import pytest

from parity import RTOL, assert_elements_close, rel_linf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nv,s,bc,c_dyn", [
    (8, 8, 4, 0, 0.0), (8, 16, 4, 1, 0.0), (68, 72, 4, 0, 5e-3),
    (120, 264, 8, 1, 5e-3), (1024, 512, 8, 0, 0.0), (1024, 512, 8, 1, 0.0),
    (1032, 64, 8, 0, 0.0), (1032, 64, 8, 1, 0.0), (640, 1032, 8, 0, 5e-3),
    (648, 1032, 8, 1, 0.0),
])
def test_steps(orc, nx, nv, s, bc, c_dyn):
    import torch

    import paper_1705_03750_amd as vp
    import workloads as W
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    box = (0.0, 10.0 * np.pi, -8.0, 8.0) if bc else (-1.0, 1.0, -1.0, 1.0)
    p = dict(nx=nx, nv=nv, sx=s, sv=s, dt=0.03 if bc else 2e-3, n_s=4,
             G=-0.5 if bc else 1.0, x_min=box[0], x_max=box[1], v_min=box[2],
             v_max=box[3], bc=bc, c_dyn=c_dyn)
    print(f"[own field] {nx}x{nv} s={s} bc={bc} c_dyn={c_dyn}", flush=True)
    if bc:
        f0 = W.two_stream(nx, nv, box, 0.2, 2.4, 0.05)
    else:
        f0 = W.finish(W.halo_sum(nx, nv, box, np.random.default_rng(nx), 3), box)
    o, g = orc.Oracle(**p), vp.VlasovRun(device="cuda:0", **p)
    o.init_conditions(f0)
    g.init_conditions(f0)
    o.step(7)
    g.step(7)
    assert_elements_close(g.get_elements().cpu().numpy(), o)
    assert rel_linf(g.reconstruct_f().cpu().numpy(), o.reconstruct_f()) <= RTOL
    assert rel_linf(g.density().cpu().numpy(), o.density()) <= RTOL
    g.sync()
    g.close()
