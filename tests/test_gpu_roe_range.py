"""The double solver where rho is far from 1 or below 0.

Scaling: (rho, m, E) -> (s^2 rho, s m, E) with dt / s leaves the equations as they
are, and with s a power of two every product, quotient and root of the step scales
exactly, so that the scaled step equals the step scaled bitwise, as far as the
exponents reach (s^2 = 2^-800 .. 2^800: no product of two densities is formed).

Negative density: no root of it exists, so every flux of such a cell is NaN, also
between two such cells, and the cell's new state is NaN and counted."""
import numpy as np
import pytest
import torch

from paper_1007_3818_amd import hydro
from paper_1007_3818_amd import workloads as W

pytestmark = pytest.mark.gpu
G53 = 5.0 / 3.0


def _step(solve, pad, dt, dh, dev, **kw):
    one = [torch.tensor([x], dtype=torch.float64, device=dev) for x in (dt, dh)]
    fl = torch.empty((pad.shape[0], 3, 3, 5, 16, 16), dtype=torch.float64, device=dev)
    st = torch.empty((pad.shape[0], 8), dtype=torch.float64, device=dev)
    step = hydro.hydro_solve_batched if solve == "muscl" else hydro.ctu_solve_batched
    return step(pad, None, *one, G53, fluxes_out=fl, group_stats=st, **kw), fl, st


@pytest.mark.parametrize("solve", ["muscl", "ctu"])
@pytest.mark.parametrize("half", [-400, -300, 300, 400])
def test_scaled_flow(gpu, half, solve):
    st, dh = W.cosmo_like(n=64)  # contrasts: entropy fixes and both fallbacks act
    dt = hydro.cfl_dt(st.to(gpu), dh, G53, 0.5)
    pad = hydro.pack_periodic(st.to(gpu), 4, 4, 4)
    s = 2.0 ** half
    scale = torch.tensor([s, 1.0, 1.0, 1.0, 1.0 / s], dtype=torch.float64, device=gpu)[:, None, None, None] * s
    out, fl, stats = _step(solve, pad, dt, dh, gpu)
    out2, fl2, stats2 = _step(solve, pad * scale, dt * s, dh, gpu)
    assert torch.isfinite(out).all() and float(stats[:, 7].sum()) > 0
    assert torch.equal(out2, out * scale)
    # flux: the state's scale times the velocity's, 1 / s
    assert torch.equal(fl2, fl * (scale / s).reshape(5, 1, 1))
    assert torch.equal(stats2[:, 6:], stats[:, 6:])


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("solve", ["muscl", "ctu"])
def test_negative_density_gives_nan(gpu, solve, dtype):
    pad = torch.empty((1, 5, 20, 20, 20), dtype=torch.float64)
    for v, x in enumerate((1.0, 0.1, -0.2, 0.05, 2.5)):
        pad[:, v] = x
    # 3^3 cells of negative density and pressure: the inner one meets only such cells
    block = (slice(8, 11),) * 3
    for v, x in enumerate((-1.0, 0.0, 0.0, 0.0, -2.5)):
        pad[(0, v) + block] = x
    pad = pad.to(gpu, dtype)
    bad = torch.zeros(2, dtype=torch.int64, device=gpu)
    one = [torch.tensor([x], dtype=torch.float64, device=gpu) for x in (1e-3, 0.1)]
    step = hydro.hydro_solve_batched if solve == "muscl" else hydro.ctu_solve_batched
    out = step(pad, None, *one, G53, bad_count=bad)
    nan = torch.isnan(out).any(1)[0].cpu().numpy()  # (z, y, x)
    assert nan[6:9, 6:9, 6:9].all()
    # the cells with a face to one of them too; cells further off stay as they were
    for a in range(3):
        for at in (5, 9):
            cells = [slice(6, 9)] * 3
            cells[a] = at
            assert nan[tuple(cells)].all()
    far = np.ones_like(nan)
    far[3:12, 3:12, 3:12] = False
    assert not nan[far].any()
    assert int(bad[0]) == int(nan.sum())
