"""Launch shapes set after a plan is bound at the default one run in the
workspace that it was bound with, also where their bands, segments or tiles are
a few more: the layout then holds the partials of one step and splits less.

Against a plan of its own workspace for the same shape, 2-norm relative: the
splits change which lanes sum what, not an amplitude's neighbours; held to the
rounding of 5 steps, complex64 5 (n + 1) 6e-8 <= 3e-6 each way at n = 9, complex128
1e-13."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,stat,N,R,order,dtype,launch", [
    (3, "distinguishable", 20, 16, 5, "c64", {"terms_per_pass": 1}),
    (3, "distinguishable", 35, 131, 9, "c64", {"terms_per_pass": 2}),
    (3, "distinguishable", 50, 1, 9, "c128", {"terms_per_pass": 3}),
    (2, "distinguishable", 264, 23, 5, "c128", {"cols_per_lane": 2}),
    (2, "distinguishable", 347, 31, 10, "c128", {"row_segments": 8}),
    (2, "boson", 1237, 1, 9, "c64", {"band_align": 0}),
    (2, "boson", 281, 3, 10, "c64", {"band_mode": 1}),
])
def test_shapes_run_in_the_workspace_of_the_default(m, stat, N, R, order, dtype, launch):
    g = np.random.default_rng(N)
    reals = [(N, 1 + 0.1 * g.standard_normal(N - 1), g.uniform(-0.3, 0.3, N), 1.0) for _ in range(R)]
    kw = dict(m=m, statistics=stat, boundary="open", interaction="onsite", dtype=dtype, reals=reals, dt=0.05, order=order,
              sites=list(range(3, 3 + m)))
    bound, own = gpu_plan(**kw), gpu_plan(**kw, launch=launch)
    room, need = bound.sizes()[1], own.sizes()[1]
    bound.set_launch(**launch)
    say(f"case: shape after binding m={m} {stat} N={N} R={R} {dtype} {launch}: bound {room}, its own {need}, "
        f"used {bound.sizes()[1]}")
    assert bound.sizes()[1] <= room
    for p in (bound, own):
        p.propagate(5)
    a, b = bound.state_numpy().astype(np.complex128), own.state_numpy().astype(np.complex128)
    assert np.linalg.norm(a - b) <= (6e-6 if dtype == "c64" else 2e-13) * np.linalg.norm(b)
    n, k = bound.realization_norms()[0], own.realization_norms()[0]
    assert np.allclose(n, k, rtol=1.2e-5 if dtype == "c64" else 4e-13, atol=0)
