"""The one-level reduction adds no more roundings in a row than a thread per group."""
import pytest
import torch

from paper_1007_3818_amd import hydro

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [512, 1024, 2048, 3000, 65536, 262144])
def test_depth(gpu, n):
    """Large terms, and small ones each of which vanishes when added to one of them
    alone.  A thread per group (1,024 of them) rounds a sum ceil(n / 1024) - 1 times,
    its wave 6 times and the 16 waves 15; the totals' weight adds one.  Each rounding
    is within 2^-53 of the partial sum."""
    host = torch.ones(n, 8, dtype=torch.float64)
    host[:256, :] = 2.0 ** 53  # the first group of every thread, where four share a group
    dh = torch.tensor([0.5], dtype=torch.float64, device=gpu)
    dt = torch.zeros(1, dtype=torch.float64, device=gpu)
    tot = torch.zeros(7, dtype=torch.float64, device=gpu)
    hydro.step_reduce(host.to(gpu), None, dh, 0.4, dt_out=dt, totals_out=tot)
    depth = -(-n // 1024) - 1 + 6 + 15 + 1
    for q, x in enumerate(tot.tolist()):
        want = (256 * 2 ** 53 + (n - 256)) * (0.125 if q < 5 else 1.0)
        assert abs(x - want) <= depth * 2.0 ** -53 * want, (n, q, (x - want) / want * 2 ** 53, depth)
    assert dt.item() == 0.4 * 0.5 / 2.0 ** 53
