"""Split sweeps of small batches: a long chain's rows in more than 16
segments, and three walkers' planes in segments."""

import numpy as np
import pytest

from oracle import propagate as P
from oracle import basis as B

from _helpers import gpu_plan, gpu_to_oracle, oracle_H, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("boundary", ["open", "periodic"])
@pytest.mark.parametrize("N", [300, 601])
def test_many_row_segments_give_the_unsplit_bits(N, boundary):
    """complex64 full grid: one fixed sequence of FMAs per amplitude, so the
    default split (over 16 segments here) gives the bits of the whole sweep."""
    g = np.random.default_rng(N)
    nb = N if boundary == "periodic" else N - 1
    reals = [(N, 1 + 0.1 * g.standard_normal(nb), g.uniform(-0.5, 0.5, N), 2.0)]
    out = []
    for seg in (0, 1):
        plan = gpu_plan(m=2, statistics="distinguishable", boundary=boundary, interaction="onsite", dtype="c64", reals=reals,
                        dt=0.05, order=7, launch={"cols_per_lane": 2, "row_segments": seg}, sites=[0, N - 1])
        items = plan.work_items()[0]
        say(f"case: N={N} {boundary} row_segments={seg}: {items} items")
        plan.propagate(9)
        out.append((items, plan.state_numpy(), plan.realization_norms()[0]))
    assert out[0][0] > 16 * out[1][0]
    assert np.array_equal(out[0][1], out[1][1])
    assert np.allclose(out[0][2], out[1][2], rtol=1e-12, atol=0)


@pytest.mark.parametrize("boundary,N,order,form", [("open", 21, 5, 0), ("periodic", 19, 6, 0), ("open", 23, 7, 1),
                                                   ("periodic", 16, 4, 1)])
def test_three_walkers_in_plane_segments(boundary, N, order, form):
    """One realisation (a few tiles, so split planes) against the oracle's
    Taylor map of the same order: FP64 roundings of 3 steps, 1e-12."""
    say(f"case: three walkers N={N} {boundary} order {order} form {form}")
    g = np.random.default_rng(order)
    J, eps = 1 + 0.2 * g.standard_normal(N if boundary == "periodic" else N - 1), g.uniform(-1, 1, N)
    sites = [0, N // 2, N - 1]
    plan = gpu_plan(m=3, statistics="distinguishable", boundary=boundary, interaction="nearest", dtype="c128",
                    reals=[(N, J, eps, 1.5)], dt=0.05, order=order, launch={"three_form": form}, sites=sites)
    plan.propagate(3)
    H = oracle_H(N, 3, B.DISTINGUISHABLE, boundary, "nearest", J, eps, 1.5)
    ref, _, _ = P.evolve_taylor(H, B.product_state(N, sites), 0.05, 3, order=order)
    assert np.max(np.abs(gpu_to_oracle(plan.state_numpy(), N, 3, B.DISTINGUISHABLE) - ref)) <= 1e-12
