"""Norm partials of several steps are reduced together: norms, truncation
estimates and alarm counts of a loop of steps equal those of the same steps
enqueued one by one, bit for bit (7 steps: one partly filled set; 8: a full
one; 19: two and a remainder), eager and as a captured loop, for one, two and
three walkers, and where every step renormalises (no holding there)."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [7, 8, 19])
@pytest.mark.parametrize("m,N,graph,renorm", [(1, 70, 0, False), (2, 140, 0, False), (2, 140, 1, False),
                                              (2, 140, 1, True), (3, 9, 0, False)])
def test_held_norms_equal_single_steps(m, N, graph, renorm, steps):
    from paper_1612_00746_amd import CtqwError
    g = np.random.default_rng(N)
    reals = [(N, 1 + 0.1 * g.standard_normal(N - 1), g.uniform(-0.3, 0.3, N), 1.0) for _ in range(2)]
    got = []
    for runs in ([steps], [1] * steps):
        plan = gpu_plan(m=m, statistics="distinguishable", boundary="open", interaction="onsite", dtype="c128",
                        reals=reals, dt=0.05, order=6, tol=0.0, norm_alarm=0.0 if renorm else 0.5, renormalize=renorm,
                        launch={"use_graph": graph}, sites=list(range(2, 2 + m)))
        psi = plan.state_numpy()
        psi[len(psi) // 2:] *= 2.0   # the second realisation raises an alarm every step
        plan.set_state_numpy(psi)
        for n in runs:
            if renorm:
                plan.propagate(n)
            else:
                with pytest.raises(CtqwError):
                    plan.propagate(n)
        st = plan.stats()
        got.append((plan.state_numpy(), *plan.realization_norms(), st.flags, st.steps_done, st.alarms))
    a, b = got
    say(f"case: held norms m={m} graph={graph} renorm={renorm} steps={steps}: alarms {a[5]} / {b[5]}")
    assert all(np.array_equal(x, y) for x, y in zip(a[:3], b[:3]))
    assert a[3:5] == b[3:5]
    if not renorm:
        assert a[5] == steps   # of the whole run
