"""The relaxing-TVD step takes different launches by input and size: whole-grid
sweeps or padded blocks, x and y in one launch or two, segments of two to 128
cells, runs of cells along x of different widths.  They evaluate the same
functions of the same values with a rounding fixed by the source, so all of them
must agree bitwise."""
import pytest
import torch

from paper_1007_3818_amd import hydro
from paper_1007_3818_amd import workloads as W

pytestmark = pytest.mark.gpu
G53 = 5.0 / 3.0


def _pad3(state, gx, gy, gz):
    u = state.reshape(gz, gy, gx, 5, 16, 16, 16).permute(3, 0, 4, 1, 5, 2, 6).reshape(5, gz * 16, gy * 16, gx * 16)
    for axis, n in ((1, gz * 16), (2, gy * 16), (3, gx * 16)):
        u = u.index_select(axis, torch.arange(-3, n + 3, device=u.device) % n)
    u = u.unfold(1, 22, 16).unfold(2, 22, 16).unfold(3, 22, 16)
    return u.permute(1, 2, 3, 0, 4, 5, 6).reshape(gx * gy * gz, 5, 22, 22, 22).contiguous()


def _state(n, dtype, dev):
    """n different groups: copies of a smooth 512-group flow, each scaled a little."""
    st, _ = W.smooth_modes(n=128)
    st = st.to(dev)
    scale = 1.0 + 0.01 * torch.sin(torch.arange(n, dtype=torch.float64, device=dev))
    return (st.repeat(-(-n // 512), 1, 1, 1, 1)[:n] * scale[:, None, None, None, None]).to(dtype).contiguous()


# one group; runs of 32, 56 and 54/54/52 cells along x with segments of 2, 4 and 8
# cells; the fused launch with segments of 32 and of 64 + 16 cells along y, and with
# long segments along z
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", [(1, 1, 1), (4, 2, 1), (7, 1, 3), (10, 3, 2), (10, 4, 43), (10, 5, 43), (3, 90, 12)])
def test_periodic_equals_padded(gpu, dtype, shape):
    gx, gy, gz = shape
    st = _state(gx * gy * gz, dtype, gpu)
    dt_dev = torch.tensor([2e-3], dtype=torch.float64, device=gpu)
    dh_dev = torch.tensor([1.0 / 64], dtype=torch.float64, device=gpu)
    pad = _pad3(st, gx, gy, gz)
    for order in (0, 1):
        per = hydro.rtvd_solve_periodic(st, gx, gy, gz, dt_dev, dh_dev, G53, order)
        ref = hydro.rtvd_solve_batched(pad, None, dt_dev, dh_dev, G53, order)
        assert torch.isfinite(ref).all()
        assert torch.equal(per, ref), (shape, order)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("order", [0, 1])
def test_padded_batch_sizes_agree(gpu, dtype, order):
    """Batches from 1,024 groups (float, x first) or 128 groups (y before x) on take
    the x and y sweeps in one launch; each group's result is that of a smaller
    batch, its level's dt and dh included."""
    n = 1030
    pad = _pad3(_state(n, dtype, gpu), 10, 103, 1)
    level = (torch.arange(n, device=gpu) % 2).to(torch.int8)
    dt_dev = torch.tensor([2e-3, 1e-3], dtype=torch.float64, device=gpu)
    dh_dev = torch.tensor([1.0 / 64, 1.0 / 128], dtype=torch.float64, device=gpu)
    whole = hydro.rtvd_solve_batched(pad, level, dt_dev, dh_dev, G53, order)
    for a, b in ((0, 1023), (1023, 1030), (0, 127), (127, 255)):
        part = hydro.rtvd_solve_batched(pad[a:b].contiguous(), level[a:b].contiguous(), dt_dev, dh_dev, G53, order)
        assert torch.equal(part, whole[a:b]), (a, b)
