"""step_reduce at the edges of its passes: one level (four threads per group, 256
groups per pass of a work-group, 8 passes in flight), several levels (a thread per
group, 4 in flight) and more levels than one pass takes (4), against sums and maxima
in plain float64 on the CPU."""
import math

import pytest
import torch

from paper_1007_3818_amd import _native, hydro

pytestmark = pytest.mark.gpu


def _reduce(stats, level, dh_dev, dt, totals):
    """The library's call itself, which takes either output or both."""
    hydro._stream()
    _native.check(_native.lib().gamer_step_reduce(hydro._ptr(stats), stats.shape[0], hydro._ptr(level),
                                                  hydro._ptr(dh_dev), dh_dev.numel(), 0.4, hydro._ptr(dt),
                                                  hydro._ptr(totals)))


def _check(stats, level, dh, cfl, dt, totals):
    n, nl = stats.shape[0], len(dh)
    lev = torch.zeros(n, dtype=torch.int64) if level is None else level.long()
    inside = (lev >= 0) & (lev < nl)
    for L in range(nl):
        s = stats[lev == L, 5]
        top = float(s.max()) if len(s) else 0.0
        want = cfl * dh[L] / top if top > 0 else (math.nan if math.isnan(top) else math.inf)
        # one product and one quotient, either of which may be rounded once more
        assert (math.isnan(want) and math.isnan(dt[L])) or dt[L] == want or abs(dt[L] - want) <= 4e-16 * want, (n, L)
    w = torch.where(inside, torch.tensor(dh, dtype=torch.float64)[lev.clamp(0, nl - 1)] ** 3, 0.0)
    cols = [w * stats[:, q] for q in range(5)] + [stats[:, 6], stats[:, 7]]
    for q, c in enumerate(cols):
        want = math.fsum(c.tolist())
        if q < 5 and not bool(inside.all()):  # a group of no level
            assert math.isnan(totals[q])
            continue
        # sums of n positive terms in any order, each product within 3 roundings
        assert abs(totals[q] - want) <= (n + 4) * 2.3e-16 * abs(want), (n, q)


@pytest.mark.parametrize("n_levels", [1, 3, 4, 5, 7])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 255, 256, 257, 1793, 2047, 2048, 2049, 4095, 4097, 9001])
def test_reduce_edges(gpu, n, n_levels):
    g = torch.Generator().manual_seed(n)
    # an odd offset: rows 8-byte but not 16-byte aligned
    store = torch.rand(n * 8 + 1, generator=g, dtype=torch.float64) + 0.5
    dh = [0.5 ** L for L in range(n_levels)]
    dh_dev = torch.tensor(dh, dtype=torch.float64, device=gpu)
    level = None if n_levels == 1 else (torch.arange(n) % n_levels).to(torch.int8)
    dlevel = None if level is None else level.to(gpu)
    for what in ("plain", "nan"):
        dev = store.to(gpu)
        stats = dev[1:].view(n, 8)
        host = store[1:].view(n, 8).clone()
        if what == "nan":  # the last group's speed: its level's step alone
            stats[n - 1, 5] = math.nan
            host[n - 1, 5] = math.nan
        outs = []
        for use_dt, use_tot in ((True, True), (True, False), (False, True)):
            dt = torch.zeros(n_levels, dtype=torch.float64, device=gpu) if use_dt else None
            tot = torch.zeros(7, dtype=torch.float64, device=gpu) if use_tot else None
            _reduce(stats, dlevel, dh_dev, dt, tot)
            outs.append((dt, tot))
        torch.cuda.synchronize()
        _check(host, level, dh, 0.4, outs[0][0].tolist(), outs[0][1].tolist())
        assert torch.equal(outs[0][0].view(torch.int64), outs[1][0].view(torch.int64))
        assert torch.equal(outs[0][1], outs[2][1])


def test_reduce_level_out_of_range(gpu):
    """Groups of no level: in no time step, conserved totals NaN, fallbacks counted."""
    n = 2050
    g = torch.Generator().manual_seed(3)
    host = torch.rand(n, 8, generator=g, dtype=torch.float64) + 0.5
    level = (torch.arange(n) % 3).to(torch.int8)
    level[7], level[2049] = 3, -1
    host[7, 5], host[2049, 5] = 1e9, math.nan
    dh = [1.0, 0.5, 0.25]
    dt = torch.zeros(3, dtype=torch.float64, device=gpu)
    tot = torch.zeros(7, dtype=torch.float64, device=gpu)
    hydro.step_reduce(host.to(gpu), level.to(gpu), torch.tensor(dh, dtype=torch.float64, device=gpu), 0.4,
                      dt_out=dt, totals_out=tot)
    _check(host, level, dh, 0.4, dt.tolist(), tot.tolist())
