"""A served batch across the widths at which the field and the kick change
their form (chunks of 64 columns finished in the kick up to 2048, the force
table above), with ragged last chunks, strides above and below those of the
workgroup's slot table, an external force, and runs that start, resample and
finish in different steps: each run bit for bit the one by itself."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GRIDS = [dict(nx=8, nv=8, sx=4, sv=4), dict(nx=68, nv=60, sx=4, sv=4),
         dict(nx=1984, nv=24, sx=8, sv=8), dict(nx=2048, nv=40, sx=16, sv=8),
         dict(nx=2052, nv=24, sx=4, sv=4), dict(nx=2064, nv=32, sx=16, sv=16),
         dict(nx=72, nv=72, sx=8, sv=8, force_mode=1, ext=(0.1, -0.2, 0.3))]


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_served_equals_alone(precision):
    import torch

    import paper_1705_03750_amd as vp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fdt = torch.float32 if precision == "mixed" else torch.float64
    reqs = []
    for k, g in enumerate(GRIDS):
        rng = np.random.default_rng(k)
        f0 = torch.as_tensor(rng.uniform(0.5, 1.0, (g["nv"], g["nx"])),
                             device="cuda:0")
        reqs.append(dict(
            params=dict(g, dt=2e-4, n_s=(0, 3, 5)[k % 3], precision=precision),
            f0=f0, out=torch.full((g["nv"], g["nx"]), float("nan"), dtype=fdt,
                                  device="cuda:0"),
            nsteps=6 + k, tag=k, arrival_s=0.0))
    print(f"[serve grids] {precision}", flush=True)
    srv = vp.Server(precision=precision, max_active=8, pool_bytes=1 << 28)
    res, _ = srv.run(reqs)
    torch.cuda.synchronize()
    for r, x in zip(reqs, res):
        assert x["status"] == 0
        run = vp.VlasovRun(device="cuda:0", **r["params"])
        run.init_conditions(r["f0"])
        run.step(r["nsteps"])
        assert torch.equal(r["out"], run.reconstruct_f()), r["params"]
    srv.close()
