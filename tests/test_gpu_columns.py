"""Two columns per lane above their compiled depth: the steps run in one pass
at one column per lane, bit for bit the steps of that request; at a depth
that neither has, in chunked passes as before."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,order", [("c64", 10), ("c64", 12), ("c64", 13), ("c128", 9), ("c128", 12), ("c128", 17)])
@pytest.mark.parametrize("m,stat", [(1, "distinguishable"), (2, "distinguishable"), (2, "boson")])
def test_deep_orders_do_not_depend_on_the_columns(m, stat, dtype, order):
    g = np.random.default_rng(order)
    reals = [(N, 1 + 0.1 * g.standard_normal(N - 1), g.uniform(-0.3, 0.3, N), 1.1) for N in (140, 171)]
    out = []
    for P in (1, 2):
        plan = gpu_plan(m=m, statistics=stat, boundary="open", interaction="onsite", dtype=dtype, reals=reals, dt=0.1,
                        order=order, tol=0.0, sites=list(range(70, 70 + m)), launch={"cols_per_lane": P})
        plan.propagate(9)
        out.append((plan.state_numpy(), *plan.realization_norms()))
    say(f"case: columns m={m} {stat} {dtype} order {order}: norm {out[1][1][0]:.12f}")
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    assert abs(out[0][1][0] - 1) < 1e-4
