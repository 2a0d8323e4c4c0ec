"""Calls of one plan that take different paths: steps on chip and band sweeps.

On states beyond the caches a call of one step goes over bands and one of many on
chip.  complex64 grids evaluate the same FMAs in the same order on both, so a run
does not depend on its portions, bit for bit; triangles agree to rounding, the
compensated sum's 8 (n + 1) 6e-8 <= 4e-6 (2-norm, relative) each way.  And
the widest complex128 shapes, which batches of few realisations leave to the
bands, against the chunked passes: 6 (n + 1) 1.1e-16 <= 1e-14 each way."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


def batch(N, R, bc, seed=2, distinct=16):
    g = np.random.default_rng(seed)
    some = [(N, 1 + 0.1 * g.standard_normal(N if bc == "periodic" else N - 1), g.uniform(-0.3, 0.3, N),
             float(g.uniform(0.5, 2))) for _ in range(distinct)]
    return [some[r % distinct] for r in range(R)]


@pytest.mark.parametrize("bc,N,R", [("open", 64, 9000), ("open", 128, 2400), ("periodic", 64, 9000)])
@pytest.mark.parametrize("acc", ["kahan", "plain"])
def test_grids_do_not_depend_on_the_portions(bc, N, R, acc):
    say(f"case: portions, complex64 grid {bc} N={N} R={R} {acc}")
    got = []
    for calls in ([16], [1] * 16):
        p = gpu_plan(m=2, statistics="distinguishable", boundary=bc, interaction="onsite", dtype="c64", accumulation=acc,
                     reals=batch(N, R, bc), dt=0.05, order=6, sites=[N // 2, N // 2 + 1])
        for n in calls:
            p.propagate(n)
        got.append((p.state_numpy(), *p.realization_norms()))
    assert np.array_equal(got[0][0], got[1][0])
    assert np.allclose(got[0][1], got[1][1], rtol=1e-12, atol=0) and np.allclose(got[0][2], got[1][2], rtol=1e-4, atol=0)


@pytest.mark.parametrize("stat", ["boson", "fermion"])
def test_triangles_agree_to_rounding(stat):
    say(f"case: portions, complex64 {stat} N=128 R=8000")
    got = []
    for calls in ([8], [1] * 8):
        p = gpu_plan(m=2, statistics=stat, boundary="open", interaction="onsite", dtype="c64", reals=batch(128, 8000, "open"),
                     dt=0.05, order=6, sites=[60, 63])
        for n in calls:
            p.propagate(n)
        got.append(p.state_numpy())
    a, b = got
    assert np.linalg.norm(a - b) <= 8e-6 * np.linalg.norm(b)


@pytest.mark.parametrize("bc,Ns", [("periodic", [81, 96, 84, 90]), ("open", [81, 96, 84, 90]), ("periodic", [65, 80])])
def test_widest_complex128_shapes(bc, Ns):
    say(f"case: wide complex128 grids {bc} {Ns} x 8")
    g = np.random.default_rng(5)
    reals = [(N, 1 + 0.2 * g.standard_normal(N if bc == "periodic" else N - 1), g.uniform(-0.5, 0.5, N), 1.3)
             for N in Ns * 8]
    got = []
    for launch in ({}, {"chunked": 1}):
        p = gpu_plan(m=2, statistics="distinguishable", boundary=bc, interaction="nearest", dtype="c128", reals=reals,
                     dt=0.05, order=9, launch=launch, sites=[0, 64])
        p.propagate(6)
        got.append((p.state_numpy(), *p.realization_norms()))
    a, b = got
    assert np.linalg.norm(a[0] - b[0]) <= 2e-14 * np.linalg.norm(b[0])
    assert np.allclose(a[1], b[1], rtol=4e-14, atol=0) and np.allclose(a[2], b[2], rtol=1e-4, atol=1e-300)
