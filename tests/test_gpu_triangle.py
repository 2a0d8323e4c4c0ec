"""complex64 triangle steps at one column per lane form a row's couplings
once (doubled on the diagonal, zero below it); two columns per lane select
them at every level.  Both evaluate the same polynomial.

Bound: the sums of a level round at most ten times per amplitude, and with
dt ||H|| < 0.4 the terms of a step sum to less than 1.5 |psi|: below 15 steps x
10 x 1.5 x 6e-8 = 1.4e-5 for amplitudes of at most 1, each way."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stat,interaction", [("boson", "onsite"), ("boson", "nearest"), ("fermion", "nearest")])
@pytest.mark.parametrize("order", [1, 4, 7, 9])
@pytest.mark.parametrize("acc", ["kahan", "plain"])
def test_row_couplings_match_selected_ones(stat, interaction, order, acc):
    g = np.random.default_rng(order)
    # above 128 columns every step is a band sweep; the small ones ride along
    reals = [(N, 1 + 0.1 * g.standard_normal(N - 1), g.uniform(-0.3, 0.3, N), 1.1) for N in (140, 2, 65, 257)]
    out = []
    for P in (1, 2):
        plan = gpu_plan(m=2, statistics=stat, boundary="open", interaction=interaction, dtype="c64", accumulation=acc,
                        reals=reals, dt=0.05, order=order, tol=0.0, sites=[0, 1], launch={"cols_per_lane": P})
        plan.propagate(15)
        out.append(plan.state_numpy())
    d = float(np.max(np.abs(out[0] - out[1])))
    say(f"case: triangle {stat} {interaction} order {order} {acc}: max difference {d:.1e}")
    assert np.all(np.isfinite(out[0])) and d <= 2.8e-5
