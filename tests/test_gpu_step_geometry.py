"""GPU tests of what a corrected step hands to the next one and of the
momentum scaling's first Newton iteration."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import dev, from_soa, orbit_states, rel_err_rows, to_soa

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pn():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_1802_00147_amd import pn as P
    P.lib()
    return P


@pytest.mark.parametrize("n", [1, 65])
@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("method", ["rk4", "rk5"])
@pytest.mark.parametrize("mode", ["none", "spin", "six", "dual"])
def test_steps_of_one_call_equal_single_steps(pn, n, shared, method, mode):
    """A call of 9 steps takes each step's geometry from the correction before
    it, nine calls form it from the state: the same bits."""
    ys, betas = orbit_states(O, np.random.default_rng(211), n, beta=0.5 if shared else None)
    par = (0.5, 0.8, 0.6) if shared else (dev(betas), dev(np.full(n, 0.8)), dev(np.full(n, 0.6)))
    kw = dict(integrator=dict(method=method), correction=dict(mode=mode))
    H, J = O.invariants(ys, betas, 0.8, 0.6)
    ref = dev(np.concatenate([H[None], J.T]))
    once, single = to_soa(ys), to_soa(ys)
    pn.step(once, *par, 9, ref=ref, **kw)
    for _ in range(9):
        pn.step(single, *par, 1, ref=ref, **kw)
    assert torch.equal(once.view(torch.int64), single.view(torch.int64))


@pytest.mark.parametrize("max_iter", [1, 2, 20])
@pytest.mark.parametrize("off", [1e-9, 1e-5, 1e-3])
def test_momentum_scaling_iterations(pn, off, max_iter):
    """States far enough from their references for one, two and more Newton
    iterations, and stopped early: iteration counts as the oracle's (a count
    may differ where an update lands on the limit), states to 1e-12: rounding
    of 1e-15 in the projection's multiplier, times a displacement of up to
    1e-3, times the damping's bound 1 / (2 mu) = 5e4."""
    rng = np.random.default_rng(212)
    ys, betas = orbit_states(O, rng, 100)
    H, J = O.invariants(ys, betas, 0.8, 0.6)
    ref = np.concatenate([H[:, None], J], axis=1)
    pert = ys * (1 + off * rng.normal(size=ys.shape))
    corr = dict(mode="six", max_iter=max_iter)
    exp, it_exp = O.manifold_correct(pert, ref, betas, 0.8, 0.6, correction=corr)
    yg = to_soa(pert)
    it = pn.manifold_correct(yg, dev(ref.T), dev(betas), dev(np.full(100, 0.8)), dev(np.full(100, 0.6)), correction=corr)
    assert np.all(rel_err_rows(from_soa(yg), exp) <= 1e-12)
    assert np.mean(it.cpu().numpy() == it_exp) >= 0.95


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("method", ["rk4", "rk5"])
@pytest.mark.parametrize("mode", ["none", "spin", "six", "dual"])
def test_last_trace_row_is_the_fli(pn, shared, method, mode):
    """The separation inside the step loop and the one after it are the same
    function of the same states, with one value for both lanes of a pair: a
    trace row at the last step equals the FLI bit for bit, on the plain,
    balanced and batch kernels alike."""
    n, steps = 65, 60
    ys, betas = orbit_states(O, np.random.default_rng(213), n, beta=0.5 if shared else None)
    par = (0.5, 0.8, 0.6) if shared else (dev(betas), dev(np.full(n, 0.8)), dev(np.full(n, 0.6)))
    kw = dict(integrator=dict(method=method), correction=dict(mode=mode), trace_every=20)
    y0 = to_soa(ys)
    t_end = torch.full((n,), float(steps), dtype=torch.float64, device=y0.device)
    for out in (pn.fli_scan(y0, float(steps), *par, **kw), pn.fli_scan_balanced(y0, float(steps), *par, slots=7, **kw),
                pn.batch_scan(y0, t_end, *par, **kw)):
        ok = (out["status"] & 0xFF) == 0
        assert bool(ok.any())
        assert torch.equal(out["trace"][-1][ok].view(torch.int64), out["fli"][ok].view(torch.int64))
