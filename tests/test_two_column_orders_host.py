"""Two columns per lane asked for at an order that only one column per lane is
compiled for: one pass over wide bands, or passes of a few terms over bands
with little halo (56 output columns of 64 in complex128, 48 in complex64),
whichever the batch's sizes make the faster.  The number of bands and the
workspace tell."""

import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(ROOT, "paper_1612_00746_amd", "libctqw.so")),
                                reason="libctqw.so not built")


def bands(m, N, R, order, dtype, stat="distinguishable", boundary="periodic", J=1.0, **launch):
    """order 0: a-priori orders."""
    from paper_1612_00746_amd import Plan, make_problem
    pr, keep = make_problem(m, R, N, 0.05, dtype=dtype, statistics=stat, boundary=boundary, taylor_order=order,
                            taylor_tol=0.0 if order else 1e-12, observables=1)
    plan = Plan(pr)
    plan._keep.append(keep)
    plan.set_launch(cols_per_lane=2, row_segments=1, **launch)
    bonds = N - (boundary == "open")
    plan.set_params(np.repeat(np.broadcast_to(J, R), bonds), np.zeros(R * N), np.ones(R))
    return (plan.work_items()[0] / R, plan.sizes()[1]), plan.orders()


@pytest.mark.parametrize("m,N,R,order,dtype,stat,passes", [
    (1, 300, 1, 12, "c128", "distinguishable", False), (1, 300, 100, 9, "c128", "distinguishable", False),
    (1, 300, 1600, 9, "c128", "distinguishable", True), (1, 4000, 400, 12, "c128", "distinguishable", True),
    (1, 300, 1600, 11, "c64", "distinguishable", False), (1, 300, 1600, 12, "c64", "distinguishable", True),
    (1, 300, 16, 12, "c64", "distinguishable", False),
    (2, 300, 400, 12, "c128", "distinguishable", False), (2, 300, 1000, 11, "c64", "distinguishable", False),
    (2, 300, 400, 9, "c128", "boson", False), (2, 128, 1000, 12, "c128", "boson", True),
])
def test_passes_where_they_are_faster(m, N, R, order, dtype, stat, passes):
    open_ = "open" if stat != "distinguishable" else "periodic"
    got, _ = bands(m, N, R, order, dtype, stat, open_)
    whole, _ = bands(m, N, R, order, dtype, stat, open_, chunked=1)
    assert (got == whole) == passes, (got, whole)


@pytest.mark.parametrize("m,N,J,passes", [
    (1, 300, 1.4, False), (1, 300, np.array([1.4, 1.4, 1.0, 1.4]), True),
    (2, 30, 1.0, False), (2, 30, np.array([1.0, 0.6, 1.0, 1.0]), True), (2, 60, np.array([1.0, 0.6, 1.0, 1.0]), False), (2, 40, np.array([1.0, 0.6, 1.0, 1.0]), True),
])
def test_two_orders(m, N, J, passes):
    """Two a-priori orders are two launches of one pass each, so a small batch
    of short sweeps runs them in passes."""
    got, orders = bands(m, N, 4, 0, "c128", J=J)
    whole, _ = bands(m, N, 4, 0, "c128", J=J, chunked=1)
    assert orders.max() >= 8 and (orders.min() < orders.max()) == (np.ndim(J) > 0)
    assert (got == whole) == passes, (got, whole, orders)
