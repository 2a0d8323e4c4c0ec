"""Two columns per lane asked for at an order that only one column per lane is
compiled for, in one pass or in passes: the same steps as one column per lane,
with a workspace of the plan's own and with that of the default shape, which has
no room for the passes' buffers.

Tolerance, 2-norm relative after 5 steps: each way rounds the state and its sum
of terms once per pass, complex64 5 (1 + 12 x 0.3) 6e-8 each way <= 3e-6; complex128
1e-13."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,stat,bc,N,R,order,dtype", [
    (1, "distinguishable", "open", 300, 150, 12, "c128"), (1, "distinguishable", "periodic", 70, 700, 9, "c128"),
    (1, "distinguishable", "open", 90, 1100, 12, "c64"), (1, "distinguishable", "open", 300, 3, 8, "c128"),
    (1, "distinguishable", "periodic", 300, 400, 10, "c64"), (2, "boson", "open", 150, 400, 12, "c128"),
    (2, "fermion", "open", 140, 3, 12, "c128"), (2, "distinguishable", "open", 140, 300, 12, "c64"),
])
def test_two_columns_asked_for(m, stat, bc, N, R, order, dtype):
    g = np.random.default_rng(N + R)
    bonds = N - (bc == "open")
    reals = [(N, 1 + 0.1 * g.standard_normal(bonds), g.uniform(-0.3, 0.3, N), 1.0) for _ in range(R)]
    kw = dict(m=m, statistics=stat, boundary=bc, interaction="onsite", dtype=dtype, reals=reals, dt=0.05, order=order,
              sites=list(range(3, 3 + m)))
    one, two, late = gpu_plan(**kw), gpu_plan(**kw, launch={"cols_per_lane": 2}), gpu_plan(**kw)
    room = late.sizes()[1]
    late.set_launch(cols_per_lane=2)
    say(f"case: m={m} {stat} {bc} N={N} R={R} order {order} {dtype}: workspace {room}, {two.sizes()[1]}, "
        f"{late.sizes()[1]}")
    assert late.sizes()[1] <= room
    bar = 3e-6 if dtype == "c64" else 1e-13
    for p in (one, two, late):
        p.propagate(5)
    a = one.state_numpy().astype(np.complex128)
    n = one.realization_norms()[0]
    for p in (two, late):
        err = np.linalg.norm(p.state_numpy().astype(np.complex128) - a) / np.linalg.norm(a)
        say(f"  {err:.1e}")
        assert err <= bar
        assert np.allclose(p.realization_norms()[0], n, rtol=2 * bar, atol=0)
