"""Row segments of the adjoint passes: a small batch splits a band's rows
into eight segments, a large one into four.  A batch of equal realisations has
the gradient of one of them: the amplitudes of a row do not depend on the
split and 512 is a power of two (the loss weights carry 1 / R in the state's
precision), so the two differ only in the order of FP64 sums.  Orders 2, 5 and 9
reach every depth of pass; chains of one band, of several, and shorter than
a pass's halo.  One of the two is checked against finite differences
elsewhere.

Tolerance: at most 512 x 45 x 16900 FP64 terms whose magnitudes sum to at
most (bound of the loss) x (number of operators); 1e-11 is over 1e4 times the
rounding of such a sum in random order."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("stat,boundary", [("boson", "open"), ("distinguishable", "open"),
                                           ("distinguishable", "periodic")])
@pytest.mark.parametrize("N,order,interaction", [(3, 5, "onsite"), (17, 9, "nearest"), (130, 2, "onsite"),
                                                 (130, 9, "nearest")])
def test_many_equal_realisations_have_the_gradient_of_one(stat, boundary, dtype, N, order, interaction):
    g = np.random.default_rng(N + order)
    nb = N if boundary == "periodic" else N - 1
    real = (N, 1 + 0.1 * g.standard_normal(nb), g.uniform(-0.3, 0.3, N), 1.2)
    sw = np.linspace(-1, 1, N)
    out = []
    for R in (1, 512):
        plan = gpu_plan(m=2, statistics=stat, boundary=boundary, interaction=interaction, dtype=dtype,
                        reals=[real] * R, dt=0.05, order=order, tol=0.0, sites=[N // 2 - 1, N // 2 + 1])
        out.append(plan.gradient(5, 2, sw, "one_body"))
    (l1, j1, e1), (lr, jr, er) = out
    d = max(np.max(np.abs(j1 - jr)), np.max(np.abs(e1 - er)))
    say(f"case: segments {stat} {boundary} {dtype} N={N} order {order}: max difference {d:.1e}, |gE| {np.max(np.abs(e1)):.1e}")
    assert np.max(np.abs(e1)) > 1e-6
    assert abs(l1 - lr) <= 1e-11 and d <= 1e-11
