"""Exact Riemann solver in FP32 over pressure units: p -> s p, v -> sqrt(s) v at the same
densities only changes the unit of velocity, so the results are those of s = 1 times powers of
sqrt(s) (a power of two), to rounding, also where the square of a pressure leaves the FP32 range.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
G14 = 1.4


def _jumps(n, unit):
    """Piecewise constant cells with strong jumps; velocities in multiples of `unit`."""
    rng = np.random.default_rng(17)
    U = np.zeros((12, n[0] * n[1]))
    rho, p = rng.uniform(0.5, 2.0, U.shape[1]), np.exp(rng.uniform(-1.5, 1.5, U.shape[1]))
    vx, vy = rng.uniform(-0.5, 0.5, (2, U.shape[1]))
    U[0], U[3], U[6] = rho, rho * vx * unit, rho * vy * unit
    U[9] = (p / (G14 - 1.0) + 0.5 * rho * (vx ** 2 + vy ** 2)) * unit ** 2
    return U.reshape(-1)


@pytest.mark.parametrize("power", [33, -38])
def test_exact_flux_does_not_depend_on_the_pressure_unit(power):
    """Bound: 64 units of FP32 rounding of the largest value of each field (the starting guess of
    the iteration takes logarithms of p, whose rounding differs; the iteration ends within half a
    unit of p* from either)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_5536_amd.solver import Solver, cartesian
    n, unit = (70, 33), 2.0 ** power
    s = Solver(cartesian(n, (0.0, 0.0), (1.0, 1.0)), precision="fp32", limiter=False, gamma=G14,
               flux="exact")
    dt = 2.0 ** -10
    field = np.repeat([1.0, unit, unit, unit ** 2], 3)[:, None]
    for call, rate in ((lambda u, k: s.rhs(u), unit), (lambda u, k: s.step_mh(u, dt / k), 1.0)):
        ref, got = (call(s.to_device(_jumps(n, k)), k).cpu().numpy().astype(float).reshape(12, -1)
                    for k in (1.0, unit))
        s.check()
        got = got / (field * rate)
        for v in range(4):
            scale = np.abs(ref[3 * v:3 * v + 3]).max()
            err = np.abs(got[3 * v:3 * v + 3] - ref[3 * v:3 * v + 3]).max()
            assert err <= 64 * 2.0 ** -23 * scale, (v, err / scale)
