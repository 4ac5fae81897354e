"""Roe's entropy fix on every kind of face: neither acoustic wave fixed, wave 1,
wave 5, both, and HLLE, along each direction, against the oracle.

Each group alternates two states along one direction (every cell an extremum, so
that all slopes vanish and the faces see the two states themselves), the pairs
drawn so that each kind is there.  The flux planes lie between the first and the
second state of a pair; the update also takes the faces the other way round.
FP64 within 1e-12 per value and per cell, the bar of the other parity tests; the
fallback counts equal."""
import numpy as np
import pytest
import torch

import oracle
from paper_1007_3818_amd import hydro
from parity import flux_close, state_close

pytestmark = pytest.mark.gpu
PER_KIND = 12


def _pairs(gamma, rng, n=400_000):
    """(kind, (rho, u, p) left, right) for PER_KIND faces of each kind."""
    def pos():
        return np.exp(0.5 * rng.standard_normal(n))
    rl, rr, pl, pr = pos(), pos(), pos(), pos()
    ul, du = 2 * rng.standard_normal(n), 3 * rng.standard_normal(n)
    ur = ul + du
    cl, cr = np.sqrt(gamma * pl / rl), np.sqrt(gamma * pr / rr)
    el, er = pl / (gamma - 1) + 0.5 * rl * ul ** 2, pr / (gamma - 1) + 0.5 * rr * ur ** 2
    sl, sr = np.sqrt(rl), np.sqrt(rr)
    u = (sl * ul + sr * ur) / (sl + sr)
    h = ((el + pl) / sl + (er + pr) / sr) / (sl + sr)
    a2 = (gamma - 1) * (h - 0.5 * u * u)
    a = np.sqrt(a2)
    al1 = ((pr - pl) - sl * sr * a * du) / (2 * a2)
    al5 = ((pr - pl) + sl * sr * a * du) / (2 * a2)
    l1, l5 = u - a, u + a
    r1, m1, e1 = rl + al1, rl * ul + al1 * l1, el + al1 * (h - u * a)
    r5, m5, e5 = rr - al5, rr * ur - al5 * l5, er - al5 * (h + u * a)
    q1, q5 = 2 * r1 * e1 - m1 * m1, 2 * r5 * e5 - m5 * m5
    gq = 0.5 * gamma * (gamma - 1)
    with np.errstate(invalid="ignore", divide="ignore"):
        c1, c5 = np.sqrt(gq * q1) / r1, np.sqrt(gq * q5) / r5
        gaps = [l1 - (ul - cl) - abs(l1), (m1 / r1 - c1) - l1 - abs(l1),
                (ur + cr) - l5 - abs(l5), l5 - (m5 / r5 + c5) - abs(l5)]
    low = np.minimum(np.minimum(r1, r5), np.minimum(q1, q5))
    ok, hlle = low > 1e-3, low < -1e-3  # clear of the fallback's threshold
    f1, f5 = np.maximum(gaps[0], gaps[1]), np.maximum(gaps[2], gaps[3])
    kinds = {"none": ok & (f1 < 0) & (f5 < 0), "one": ok & (f1 > 0) & (f5 < 0), "five": ok & (f1 < 0) & (f5 > 0),
             "both": ok & (f1 > 0) & (f5 > 0), "hlle": hlle}
    out = []
    for k, m in kinds.items():
        i = np.flatnonzero(m)[:PER_KIND]
        assert len(i) == PER_KIND, (k, len(i))
        out += [(k, (rl[q], ul[q], pl[q]), (rr[q], ur[q], pr[q])) for q in i]
    return out


@pytest.mark.parametrize("gamma", [1.4, 5.0 / 3.0])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_fix_kinds(gpu, axis, gamma):
    pairs = _pairs(gamma, np.random.default_rng(5))
    n = len(pairs)
    pad = np.empty((n, 5, 20, 20, 20))
    for g, (_, left, right) in enumerate(pairs):
        for odd, (r, u, p) in ((1, left), (0, right)):
            mom = [0.1 * r, -0.2 * r, 0.3 * r]
            mom[axis] = r * u
            e = p / (gamma - 1) + 0.5 * sum(m * m for m in mom) / r
            cells = [slice(None)] * 3
            cells[2 - axis] = slice(odd, None, 2)
            for v, x in enumerate([r, *mom, e]):
                pad[g, v][tuple(cells)] = x
    dt, dh = 1e-3, 0.1
    ref, ofl, cnt = oracle.hydro_solve(pad, dt, dh, gamma, want_fluxes=True)
    assert cnt[1] > 0
    fl = torch.empty((n, 3, 3, 5, 16, 16), dtype=torch.float64, device=gpu)
    stats = torch.empty((n, 8), dtype=torch.float64, device=gpu)
    one = [torch.tensor([x], dtype=torch.float64, device=gpu) for x in (dt, dh)]
    out = hydro.hydro_solve_batched(torch.from_numpy(pad).to(gpu), None, *one, gamma, fluxes_out=fl, group_stats=stats)
    state_close(out.cpu().numpy(), ref, 1e-12, f"axis {axis} state", gamma=gamma)
    flux_close(fl.cpu().numpy().transpose(0, 3, 1, 2, 4, 5), ofl.transpose(0, 3, 1, 2, 4, 5), 1e-12, "fluxes")
    s = stats.cpu().numpy()
    assert (int(s[:, 6].sum()), int(s[:, 7].sum())) == tuple(cnt)
