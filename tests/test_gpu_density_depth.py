"""Density-matrix tiles past the last whole round: in quarters from 121 (complex128)
and 17 (complex64) realisations on, whole below, against A A^H / R in FP64 of the
states that the plan holds, on both sides of that rule.

Bound: an entry is a sum of 2 R products, one rounding each, then one
division: (2 R + 4) u sum_r |a_r,i| |a_r,j| / R with u the type's unit
roundoff (two roundings to spare), plus 2 R of the type's smallest normal
number for products that underflow."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,N,R", [("c64", 65, 16), ("c64", 65, 17), ("c128", 46, 120), ("c128", 46, 121)])
def test_tiles_past_a_round(dtype, N, R):
    g = np.random.default_rng(R)
    reals = [(N, 1 + 0.1 * g.standard_normal(N - 1), g.uniform(-0.3, 0.3, N), 1.0) for _ in range(R)]
    plan = gpu_plan(m=2, statistics="distinguishable", boundary="open", interaction="onsite", dtype=dtype,
                    reals=reals, dt=0.3, order=8, tol=0.0, sites=[N // 2, N // 2 + 1])
    plan.propagate(10)
    A = plan.state_numpy().reshape(R, N * N).astype(np.complex128)
    say(f"case: density tiles {dtype}, D={N * N}, R={R}")
    rho = plan.density_matrix(0).cpu().numpy()
    ref = A.T @ A.conj() / R
    u = 2.0 ** -24 if dtype == "c64" else 2.0 ** -53
    tiny = float(np.finfo(np.float32 if dtype == "c64" else np.float64).tiny)
    bound = (2 * R + 4) * u * (np.abs(A).T @ np.abs(A)) / R + 2 * R * tiny
    err = np.maximum(np.abs(rho.real - ref.real), np.abs(rho.imag - ref.imag))
    say(f"  worst error / bound {np.max(err / bound):.2f}")
    assert np.all(err <= bound)
