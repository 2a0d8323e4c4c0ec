"""Steps of small lattices held on chip, against the general passes (forced
with chunked=1: the same polynomial through other kernels) and the FP64
oracle, at the edges of the kernel's shapes: lattice sizes around a wave's
rows and columns, both parities (the triangle's rotated row differs), one
and two columns per lane, few and many realisations, uneven batches, orders
from 1 to above the bands' depth.

Tolerances, 2-norm relative, over at most 6 steps: complex64 rounds the
state once per term it adds (plain) or once plus the sum of the terms
(compensated), at most 6 (n + 1) 6e-8 <= 3e-6 at n = 7 (later terms are below
the rounding); complex128 6 (n + 1) 1.1e-16 <= 2e-14 at n = 24, held to
1e-13.  Squared norms: twice that.  The last term's squared norm only scales
a bound and is summed in the state's precision: 1e-4."""

import numpy as np
import pytest

from oracle import basis as B
from oracle import propagate as P

from _helpers import gpu_plan, gpu_to_oracle, oracle_H, oracle_to_gpu, say

pytestmark = pytest.mark.gpu

BAR = {"c64": 3e-6, "c128": 1e-13}


def draw(Ns, bc, seed):
    g = np.random.default_rng(seed)
    return [(N, 1 + 0.2 * g.standard_normal(N if bc == "periodic" else N - 1), g.uniform(-0.5, 0.5, N),
             float(g.uniform(0.5, 3.0))) for N in Ns]


def spread_state(Ns, stat, seed):
    g = np.random.default_rng(seed)
    out = []
    for N in Ns:
        D = {"distinguishable": N * N, "boson": N * (N + 1) // 2, "fermion": N * (N - 1) // 2}[stat]
        c = g.standard_normal(D) + 1j * g.standard_normal(D)
        out.append(oracle_to_gpu(c / np.linalg.norm(c), N, 2, stat))
    return np.concatenate(out)


def final(plan, psi, calls):
    plan.set_state_numpy(psi)
    for n in calls:
        plan.propagate(n)
    return plan.state_numpy().astype(np.complex128), plan.realization_norms(), plan.stats()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("stat,bc,Ns,order,extra", [
    ("distinguishable", "open", [2, 3, 16, 17], 1, {}),
    ("distinguishable", "open", [31, 32, 33, 64, 5], 7, {"interaction": "nearest"}),
    ("distinguishable", "open", [65, 80, 2], 6, {"accumulation": "plain"}),
    ("distinguishable", "open", [81, 95, 96], 9, {"renormalize": True}),
    ("distinguishable", "open", [97, 127, 128, 64], 7, {}),
    ("distinguishable", "periodic", [3, 4, 16, 33], 2, {"interaction": "nearest"}),
    ("distinguishable", "periodic", [63, 64, 17], 20, {}),
    ("distinguishable", "periodic", [65, 66, 96], 7, {"renormalize": True}),
    ("boson", "open", [2, 3, 4, 5, 17], 1, {}),
    ("boson", "open", [31, 32, 33, 63, 64], 7, {"interaction": "nearest"}),
    ("boson", "open", [65, 66, 127, 128, 2], 12, {}),
    ("boson", "open", [90, 14, 91], 24, {"renormalize": True}),
    ("fermion", "open", [2, 3, 18, 64, 61], 7, {"interaction": "nearest"}),
    ("fermion", "open", [65, 100, 128, 33], 8, {"accumulation": "plain"}),
])
def test_small_lattices_match_the_general_passes(stat, bc, Ns, order, extra, dtype):
    say(f"case: on-chip steps {stat} {bc} {Ns} order {order} {extra} {dtype}")
    reals, psi = draw(Ns, bc, 3), spread_state(Ns, stat, 4)
    kw = dict(m=2, statistics=stat, boundary=bc, dtype=dtype, reals=reals, dt=0.05 if order < 20 else 0.3, order=order,
              observables=1, **{"interaction": "onsite", **extra})
    got, (n2, t2), st = final(gpu_plan(**kw), psi, (1, 3, 2))
    ref, (rn2, rt2), rst = final(gpu_plan(**kw, launch={"chunked": 1}), psi, (6,))
    d = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    say(f"  {d:.1e}; norms {np.max(np.abs(n2 / rn2 - 1)):.1e}, last term {np.max(np.abs(t2 / rt2 - 1)):.1e}")
    assert d <= BAR[dtype]
    assert np.allclose(n2, rn2, rtol=2 * BAR[dtype], atol=0) and np.allclose(t2, rt2, rtol=1e-4, atol=1e-300)
    assert (st.steps_done, st.flags, st.alarms) == (rst.steps_done, rst.flags, rst.alarms)


@pytest.mark.parametrize("R", [255, 300])
@pytest.mark.parametrize("N", [16, 33, 64])
def test_few_and_many_realisations_agree_with_the_oracle(N, R):
    """Up to 256 realisations run with few rows per wave, more with many;
    the first and last realisation against the oracle's map."""
    for stat, bc in (("boson", "open"), ("distinguishable", "periodic")):
        say(f"case: {R} realisations, {stat} {bc} N={N}")
        reals = draw([N] * R, bc, 8)
        plan = gpu_plan(m=2, statistics=stat, boundary=bc, interaction="onsite", dtype="c128", reals=reals, dt=0.05,
                        order=9, sites=[3, 5])
        plan.propagate(5)
        psi, off = plan.state_numpy(), plan.layout()
        sb = B.BOSON if stat == "boson" else B.DISTINGUISHABLE
        for r in (0, R - 1):
            _, J, eps, U = reals[r]
            ref, _, _ = P.evolve_taylor(oracle_H(N, 2, sb, bc, "onsite", J, eps, U), B.product_state(N, [3, 5], sb),
                                        0.05, 5, order=9)
            assert np.max(np.abs(gpu_to_oracle(psi[off[r]:off[r + 1]], N, 2, sb) - ref)) <= 1e-13


def test_alarms_count_every_step_and_realisation():
    """A batch whose second realisation starts at norm 2 raises one alarm per
    step, as the general passes count them."""
    reals = draw([20, 20], "open", 5)
    psi = spread_state([20, 20], "boson", 6)
    psi[len(psi) // 2:] *= 2.0
    from paper_1612_00746_amd import CtqwError
    for launch in ({}, {"chunked": 1}):
        plan = gpu_plan(m=2, statistics="boson", boundary="open", interaction="onsite", dtype="c128", reals=reals, dt=0.05,
                        order=9, norm_alarm=0.5, launch=launch)
        plan.set_state_numpy(psi)
        with pytest.raises(CtqwError):
            plan.propagate(7)
        st = plan.stats()
        say(f"case: alarms {launch}: {st.alarms}, flags {st.flags}")
        assert (st.alarms, st.flags, st.steps_done) == (7, 2, 7)
