"""A group's step does not depend on how many groups share the call.  Batches of up
to 384 groups (float arithmetic) or 256 (double) run the kernel that can split a
group in z, larger ones the one that cannot: the same groups on either side of that
size give the same bits, state, flux planes, stats and fallback counts, for padded
and for periodic input; and the two inputs give the same bits as each other."""
import pytest
import torch

from paper_1007_3818_amd import hydro
from paper_1007_3818_amd import workloads as W

pytestmark = pytest.mark.gpu
G53 = 5.0 / 3.0
KINDS = [(torch.float32, None, 384), (torch.float64, torch.float32, 384), (torch.float64, None, 256)]


@pytest.fixture(scope="module")
def flow(gpu):
    st, dh = W.cosmo_like(n=128)  # 512 groups; both fallbacks act
    return st.to(gpu), dh


def _one(x, dev):
    return torch.tensor([x], dtype=torch.float64, device=dev)


def _outputs(n, dtype, dev):
    return dict(out=torch.empty((n, 5, 16, 16, 16), dtype=dtype, device=dev),
                fluxes_out=torch.empty((n, 3, 3, 5, 16, 16), dtype=dtype, device=dev),
                group_stats=torch.empty((n, 8), dtype=torch.float64, device=dev))


def _same(a, b, what):
    for k in a:
        assert torch.isfinite(a[k]).all(), (what, k)
        assert torch.equal(a[k], b[k]), (what, k)


@pytest.mark.parametrize("limiting", ["primitive", "characteristic"])
@pytest.mark.parametrize("dtype,compute,most", KINDS)
def test_padded(gpu, flow, dtype, compute, most, limiting):
    st, dh = flow
    pad = hydro.pack_periodic(st.to(dtype), 8, 8, 8)
    dt = hydro.cfl_dt(st, dh, G53, 0.5)
    got = []
    for n in (most, most + 1, 512):
        o = _outputs(n, dtype, gpu)
        hydro.hydro_solve_batched(pad[:n], None, _one(dt, gpu), _one(dh, gpu), G53, limiting=limiting,
                                  compute=compute, **o)
        got.append({k: v[:most] for k, v in o.items()})
    assert float(got[0]["group_stats"][:, 6:].sum()) > 0
    _same(got[0], got[1], most + 1)
    _same(got[0], got[2], 512)


@pytest.mark.parametrize("limiting", ["primitive", "characteristic"])
@pytest.mark.parametrize("dtype,compute,most", KINDS)
def test_periodic(gpu, flow, dtype, compute, most, limiting):
    """A grid and the grid of twice as many groups that repeats it along x."""
    st, dh = flow
    gy, gz = 8, 8
    gx = most // (gy * gz)
    one = st.to(dtype).reshape(gz, gy, 8, 5, 16, 16, 16)[:, :, :gx]
    two = torch.cat([one, one], dim=2)
    dt = 0.5 * hydro.cfl_dt(st, dh, G53, 0.5)
    got = []
    for g, x in ((one, gx), (two, 2 * gx)):
        n = x * gy * gz
        o = _outputs(n, dtype, gpu)
        hydro.hydro_solve_periodic(g.reshape(n, 5, 16, 16, 16).contiguous(), x, gy, gz, _one(dt, gpu), _one(dh, gpu),
                                   G53, limiting=limiting, compute=compute, **o)
        got.append({k: v.reshape(gz, gy, x, *v.shape[1:])[:, :, :gx] for k, v in o.items()})
    _same(got[0], got[1], "periodic")


@pytest.mark.parametrize("limiting", ["primitive", "characteristic"])
@pytest.mark.parametrize("dtype,compute,most", KINDS)
def test_padded_equals_periodic(gpu, flow, dtype, compute, most, limiting):
    """The default variant on either input, in a batch that is split and in one that is not."""
    st, dh = flow
    for gx, gy, gz in ((4, 4, 4), (8, 8, 8)):
        n = gx * gy * gz
        s = st[:n].to(dtype).contiguous()
        dt = 0.1 * hydro.cfl_dt(st, dh, G53, 0.5)  # the cut-out grid has jumps at its ends
        kw = dict(limiting=limiting, compute=compute)
        a, b = _outputs(n, dtype, gpu), _outputs(n, dtype, gpu)
        hydro.hydro_solve_periodic(s, gx, gy, gz, _one(dt, gpu), _one(dh, gpu), G53, **kw, **a)
        hydro.hydro_solve_batched(hydro.pack_periodic(s, gx, gy, gz), None, _one(dt, gpu), _one(dh, gpu), G53, **kw, **b)
        _same(a, b, (n, limiting))
