"""A workspace sized at one column per lane also holds two: their bands are
fewer, and so are the norm partials, whether or not several steps' are held."""

import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(ROOT, "paper_1612_00746_amd", "libctqw.so")),
                                reason="libctqw.so not built")


@pytest.mark.parametrize("Ns", [[1024] * 4096, [256] * 16384, [64 + (k * 137) % 961 for k in range(7000)],
                                [64 + (k * 137) % 961 for k in range(8192)], [300] * 1700, [1024] * 3277],
                         ids=["1024x4096", "256x16384", "uneven-7000", "uneven-8192", "300x1700", "1024x3277"])
def test_two_columns_per_lane_need_no_more_workspace(Ns):
    from paper_1612_00746_amd import Plan, make_problem
    pr, keep = make_problem(2, len(Ns), Ns[0] if len(set(Ns)) == 1 else Ns, 0.05, dtype="c64", taylor_order=7,
                            observables=1)
    plan = Plan(pr)
    plan._keep.append(keep)
    plan.set_params(np.ones(sum(Ns) - len(Ns)), np.zeros(sum(Ns)), np.ones(len(Ns)))
    sizes = []
    for P in (1, 2):
        plan.set_launch(cols_per_lane=P)
        sizes.append((plan.work_items()[0], plan.sizes()[1]))
    assert sizes[1][0] < sizes[0][0] and sizes[1][1] <= sizes[0][1], sizes
