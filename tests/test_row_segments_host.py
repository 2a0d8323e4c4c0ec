"""How many row segments a batch of few bands is split into: none of its full
grids' items may fall into a second round of the device's 1024 SIMDs where the
kernel holds one wave on each (complex64 with 12 terms, complex128 from 8), nor a
few of them where it holds two."""

import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(ROOT, "paper_1612_00746_amd", "libctqw.so")),
                                reason="libctqw.so not built")


def items(N, R, order, dtype, boundary="open", **launch):
    from paper_1612_00746_amd import Plan, make_problem
    pr, keep = make_problem(2, R, N, 0.05, dtype=dtype, boundary=boundary, taylor_order=order, observables=1)
    plan = Plan(pr)
    plan._keep.append(keep)
    plan.set_launch(**launch)
    plan.set_params(np.ones(R * (N - (boundary == "open"))), np.zeros(R * N), np.ones(R))
    return plan.work_items()[0]


@pytest.mark.parametrize("N,R,order,dtype,boundary", [
    (2000, 1, 12, "c64", "open"), (2000, 1, 12, "c64", "periodic"), (1121, 2, 12, "c64", "open"),
    (143, 123, 12, "c64", "open"),                       # one wave per SIMD
    (1212, 5, 10, "c128", "open"), (545, 5, 9, "c128", "periodic"),
    (1024, 3, 7, "c64", "open"), (1024, 3, 7, "c64", "periodic"), (964, 2, 3, "c64", "open"),   # a few past the target
    (1104, 1, 7, "c64", "open"),
])
def test_no_few_items_in_a_second_round(N, R, order, dtype, boundary):
    assert 700 <= items(N, R, order, dtype, boundary) <= 1024


@pytest.mark.parametrize("N,R,order,dtype", [(839, 33, 3, "c64"), (286, 50, 5, "c64"), (486, 38, 3, "c128")])
def test_many_more_items_fill_the_second_wave(N, R, order, dtype):
    assert items(N, R, order, dtype) > 1024
