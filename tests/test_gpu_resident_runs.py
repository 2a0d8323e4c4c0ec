"""Runs held on chip are cut into launches of at most 256 steps: the state,
norms, estimates and alarm counts of 600 steps (256 + 256 + 88) equal those of
the same steps taken in other portions, bit for bit, and a gradient does not
depend on where its segments are cut."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


def plan_of(stat, dtype, **kw):
    g = np.random.default_rng(4)
    reals = [(N, 1 + 0.1 * g.standard_normal(N - 1), g.uniform(-0.3, 0.3, N), 1.0) for N in kw.pop("Ns", (24, 9, 33))]
    return gpu_plan(m=2, statistics=stat, boundary="open", interaction="onsite", dtype=dtype, reals=reals, dt=0.05, order=5,
                    sites=[3, 4], **kw)


@pytest.mark.parametrize("stat", ["distinguishable", "boson"])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("renorm", [False, True])
def test_runs_do_not_depend_on_their_cuts(stat, dtype, renorm):
    got = []
    for calls in ((600,), (255, 2, 343), (1, 599)):
        p = plan_of(stat, dtype, renormalize=renorm)
        for n in calls:
            p.propagate(n)
        st = p.stats()
        got.append((p.state_numpy(), *p.realization_norms(), (st.flags, st.alarms, st.steps_done)))
    say(f"case: cut runs {stat} {dtype} renormalize={renorm}: {got[0][3]}")
    for other in got[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(got[0][:3], other[:3])) and got[0][3] == other[3]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_gradients_do_not_depend_on_their_cuts(dtype):
    """600 steps with segments of 600 (stored by launches of 256, 256 and 87
    steps) and of 40: the same states, so the same sums."""
    w = np.linspace(-1, 1, 24)
    out = [plan_of("boson", dtype, Ns=(24, 24)).gradient(600, every, w, "one_body") for every in (600, 40)]
    say(f"case: cut gradients {dtype}: loss {out[0][0]:.6f}")
    for a, b in zip(*out):
        assert np.array_equal(np.asarray(a), np.asarray(b))
