"""GPU tests of wavefronts with few orbits at work, whose other lanes mirror
one of them: results are those of a wavefront that is full throughout."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import dev, from_soa, orbit_states, rel_err_rows, to_soa

pytestmark = pytest.mark.gpu

FLI = dict(r_merge=9.5, r_esc=36.0)      # ends at the start, in the middle and at t_end
KEYS = ("fli", "label", "status", "steps", "renorms", "newton_max", "dH", "dJ", "y_final", "trace")


@pytest.fixture(scope="module")
def pn():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_1802_00147_amd import pn as P
    P.lib()
    return P


def bits(t):
    return t.contiguous().view(torch.int64) if t.dtype == torch.float64 else t


def orbit(out, key, i):
    return bits(out[key][..., i].contiguous())


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("method,mode", [("rk4", "six"), ("rk5", "dual"), ("rk4", "spin"), ("rk5", "none")])
def test_scans_of_few_orbits(pn, shared, method, mode):
    """Orbit by orbit, the bits of a scan of 32 copies (a full wavefront whose
    orbits all end at once), for the counts around the lanes that full speed
    needs, ends that differ, and a parameter set that is refused."""
    n = 35
    rng = np.random.default_rng(311)
    ys, betas = orbit_states(O, rng, n, beta=0.5 if shared else None)
    chi = np.full(n, 0.8)
    if not shared:
        chi[[3, 16]] = 2.0
    t = rng.integers(15, 120, n).astype(float)
    t[rng.integers(0, n, 8)] = 120.0
    kw = dict(integrator=dict(method=method), correction=dict(mode=mode), fli=FLI, trace_every=15)

    def par(idx):
        return (0.5, 0.8, 0.6) if shared else (dev(betas[idx]), dev(chi[idx]), dev(np.full(len(idx), 0.6)))

    full = [pn.fli_scan(to_soa(ys[[i] * 32]), dev(t[[i] * 32]), *par([i] * 32), **kw) for i in range(n)]
    same = [pn.fli_scan(to_soa(ys[[i] * 32]), 120.0, *par([i] * 32), **kw) for i in range(n)]
    for m in (1, 2, 15, 16, 17, 18, 31, 33, 35):
        idx = list(range(m))
        y0 = to_soa(ys[:m])
        for out, ref in ((pn.fli_scan(y0, dev(t[:m]), *par(idx), **kw), full),
                         (pn.batch_scan(y0, dev(t[:m]), *par(idx), **kw), full),
                         (pn.fli_scan_balanced(y0, 120.0, *par(idx), slots=(m + 1) // 2, **kw), same)):
            for i in range(m):
                for key in KEYS:
                    a, b = orbit(out, key, i), orbit(ref[i], key, 0)
                    if key == "trace":       # rows past an orbit's end stay NaN
                        assert bool(out[key][len(b):, i].isnan().all()), (m, i)
                        a = a[:len(b)]
                        b = b[:len(a)]
                    assert torch.equal(a, b), (m, i, key)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65])
@pytest.mark.parametrize("rr", [0, 1])
def test_trajectories_of_few_orbits(pn, n, rr):
    """States and rows of the first n orbits, and nothing behind them: the
    bits of a run of 128, two full wavefronts."""
    ys, _ = orbit_states(O, np.random.default_rng(312), 128, beta=0.5)
    kw = dict(model=dict(rad_reaction=rr))
    y_all = to_soa(ys)
    rows_all = pn.trajectory(y_all, 0.5, 0.8, 0.6, 40, 7, **kw)
    y = to_soa(ys)
    rows = pn.trajectory(y, 0.5, 0.8, 0.6, 40, 7, n=n, **kw)
    assert torch.equal(bits(y[:, :n]), bits(y_all[:, :n]))
    assert torch.equal(bits(y[:, n:]), bits(to_soa(ys)[:, n:]))
    assert torch.equal(bits(rows[:, :, :n]), bits(rows_all[:, :, :n]))


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("rr", [0, 1])
@pytest.mark.parametrize("method", ["rk4", "rk5"])
@pytest.mark.parametrize("mode", ["none", "spin", "six", "dual"])
def test_trajectories_match_the_oracle(pn, shared, rr, method, mode):
    """Every step kernel, with one parameter table and with arrays: the oracle's
    state after 30 steps, within the 1e-10 that holds up to 1,000."""
    n = 66
    ys, betas = orbit_states(O, np.random.default_rng(313), n, beta=0.5 if shared else None)
    par = (0.5, 0.8, 0.6) if shared else (dev(betas), dev(np.full(n, 0.8)), dev(np.full(n, 0.6)))
    kw = dict(model=dict(rad_reaction=rr), integrator=dict(method=method),
              correction=None if mode == "none" else dict(mode=mode))
    exp = O.step(ys, betas, 0.8, 0.6, 30, **kw)
    y = to_soa(ys)
    kw["correction"] = dict(mode=mode)
    rows = pn.trajectory(y, *par, 30, 10, **kw)
    assert np.all(rel_err_rows(from_soa(y), exp) <= 1e-10)
    assert torch.equal(bits(rows[-1]), bits(y))
