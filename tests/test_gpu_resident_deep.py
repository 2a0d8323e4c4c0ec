"""The truncation estimate of steps held on chip, for large dt ||H||: the last
term enters it before its 1/n!, and its squares leave FP32's range (two bosons,
32 nodes, J = 1, dt = 1.5: 27 terms, a squared norm of 1e40) while the amplitudes
do not.  Against the general passes, which sum it in FP64.

With x = dt ||H|| = 6 and one step from the same state, either path forms each
level with ten roundings of at most x times the vector before it: the last
term is off by at most 10 n 6e-8 x^n = 1.6e-5 x^n.  Its norm is about x^n / 10
(1e20 against 6^27), so its square is within 2 x 1.6e-4 each way: 1e-3.  The
state is off by at most the terms' errors, 10 x e^x 6e-8 = 1.5e-3, and its
square within twice that each way: 6e-3.
"""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stat", ["boson", "fermion"])
@pytest.mark.parametrize("N,dt", [(32, 1.5), (17, 1.5), (70, 1.4)])
def test_deep_series_keep_a_finite_truncation_estimate(stat, N, dt):
    reals = [(N, np.ones(N - 1), np.zeros(N), 0.0)] * 2
    got = []
    for launch in ({}, {"chunked": 1}):
        plan = gpu_plan(m=2, statistics=stat, boundary="open", interaction="onsite", dtype="c64", reals=reals, dt=dt,
                        tol=1e-7, launch=launch, sites=[N // 2 - 1, N // 2])
        plan.propagate(1)   # raises on a non-finite estimate
        got.append((plan.orders()[0], *plan.realization_norms(), plan.stats().flags))
    (n, n2, t2, flags), (_, rn2, rt2, rflags) = got
    say(f"case: deep series {stat} N={N} order {n}: last term {t2[0]:.3e} / {rt2[0]:.3e}, flags {flags} / {rflags}")
    assert n >= 24 and flags == rflags
    assert np.all(np.isfinite(t2)) and np.allclose(t2, rt2, rtol=1e-3, atol=0)
    assert np.allclose(n2, rn2, rtol=6e-3, atol=0)
