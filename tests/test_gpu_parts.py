"""Small batches are advanced in z parts of a group, one work-group per part: the
new state, flux planes, stats (fallback counts included) and bad-cell counts are
bitwise those of whole-group sweeps (an explicit grid or zseg), at both sides of
every batch size where the number of parts changes (float: 48, 96, 192 and 384
groups; double: 32, 64, 128 and 256)."""
import pytest
import torch

from paper_1007_3818_amd import hydro
from paper_1007_3818_amd import workloads as W

pytestmark = pytest.mark.gpu
G53 = 5.0 / 3.0


@pytest.fixture(scope="module")
def flow(gpu):
    st, dh = W.cosmo_like(n=128)  # 512 groups; both fallbacks act
    return st.to(gpu), dh


def _same(a, b, what):
    for x, y, name in zip(a, b, ("state", "fluxes", "stats", "bad")):
        # whole bytes: NaN groups (a level out of range) compare too
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), (what, name)


def _outputs(n, dtype, dev):
    return dict(out=torch.full((n, 5, 16, 16, 16), 7.0, dtype=dtype, device=dev),
                fluxes_out=torch.full((n, 3, 3, 5, 16, 16), 7.0, dtype=dtype, device=dev),
                group_stats=torch.full((n, 8), 7.0, dtype=torch.float64, device=dev),
                bad_count=torch.zeros(2, dtype=torch.int64, device=dev))


@pytest.mark.parametrize("limiting", ["primitive", "characteristic"])
@pytest.mark.parametrize("dtype,compute,sizes", [
    (torch.float32, None, (1, 48, 49, 96, 97, 192, 193, 384, 385)),
    (torch.float64, None, (1, 32, 33, 64, 65, 128, 129, 256, 257)),
    (torch.float64, torch.float32, (1, 49, 384)),
])
def test_batched_parts_equal_whole_groups(gpu, flow, dtype, compute, sizes, limiting):
    st, dh = flow
    pad = hydro.pack_periodic(st.to(dtype), 8, 8, 8)
    dt_dev = torch.tensor([1e-4, 5e-5, 2e-5], dtype=torch.float64, device=gpu)
    dh_dev = torch.tensor([dh, dh / 2, dh / 4], dtype=torch.float64, device=gpu)
    fallbacks = 0
    for n in sizes:
        level = (torch.arange(n, device=gpu) % 3).to(torch.int8)
        level[n // 2] = 3  # out of range: NaN output, counted once
        got = []
        for grid in (None, n):
            o = _outputs(n, dtype, gpu)
            hydro.hydro_solve_batched(pad[:n], level, dt_dev, dh_dev, G53, limiting=limiting, compute=compute,
                                      grid=grid, **o)
            got.append([o[k] for k in ("out", "fluxes_out", "group_stats", "bad_count")])
        torch.cuda.synchronize()
        _same(*got, (n, dtype, compute))
        assert got[0][3][1].item() == 1
        # without stats the step is the same
        out = hydro.hydro_solve_batched(pad[:n], level, dt_dev, dh_dev, G53, limiting=limiting, compute=compute)
        assert torch.equal(out.view(torch.uint8), got[0][0].view(torch.uint8)), n
        fallbacks += int(got[0][2][:, 6:].sum())
    assert fallbacks > 0


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 3, 1), (1, 2, 5), (3, 4, 8), (7, 7, 7)])
def test_periodic_parts_equal_whole_groups(gpu, flow, dtype, shape):
    st, dh = flow
    gx, gy, gz = shape
    n = gx * gy * gz
    st = st[:n].to(dtype).contiguous()
    dt_dev = torch.tensor([1e-4], dtype=torch.float64, device=gpu)
    dh_dev = torch.tensor([dh], dtype=torch.float64, device=gpu)
    got = []
    for zseg in (None, 1, gz):
        o = _outputs(n, dtype, gpu)
        hydro.hydro_solve_periodic(st, gx, gy, gz, dt_dev, dh_dev, G53, zseg=zseg, **o)
        got.append([o[k] for k in ("out", "fluxes_out", "group_stats", "bad_count")])
    torch.cuda.synchronize()
    _same(got[0], got[1], (shape, "zseg 1"))
    _same(got[0], got[2], (shape, "zseg gz"))
