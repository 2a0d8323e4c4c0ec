"""Band sweeps on batches with small lattices.  Batches of two walkers on at most
128 nodes run on chip; one realisation of 140 nodes more in each batch here keeps
all of it on the bands: captured step loops and their timing, the persistent
grid, two columns per lane, forced passes, the compensated sum, the triangle
kernel, and the gradient's kept segment.

Bars.  complex128 against the oracle's Taylor map of the same order: 1e-12 (60
steps of a few rounding errors).  complex64, 200 steps: the compensated sum rounds
an amplitude once per step (6e-8), in a random walk over amplitudes below 0.25
sqrt(200) x 0.25 x 6e-8 = 2.1e-7; the FP32 tables shift the phases by t ||dH|| = 10 x
4 x 6e-8, times 0.25: 6e-7; together below 1e-6.  A plain sum rounds once per term:
seven times that."""

import numpy as np
import pytest

from oracle import basis as B
from oracle import propagate as P

from _helpers import gpu_plan, gpu_to_oracle, oracle_H, say

pytestmark = pytest.mark.gpu


def draw(Ns, seed, bc="open"):
    g = np.random.default_rng(seed)
    return [(N, 1 + 0.2 * g.standard_normal(N if bc == "periodic" else N - 1), g.uniform(-0.5, 0.5, N),
             float(g.uniform(0, 2))) for N in Ns]


def worst_error(plan, reals, stat, bc, interaction, sites, dt, steps, order):
    psi, off = plan.state_numpy(), plan.layout()
    worst = 0.0
    for r, (N, J, eps, U) in enumerate(reals):
        H = oracle_H(N, 2, stat, bc, interaction, J, eps, U)
        ref, _, _ = P.evolve_taylor(H, B.product_state(N, sites, stat), dt, steps, order=order)
        worst = max(worst, float(np.max(np.abs(gpu_to_oracle(psi[off[r]:off[r + 1]], N, 2, stat) - ref))))
    return worst


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_captured_loops_match_eager_launches(dtype):
    """Replays of a captured loop (persistent grid, its claim lists), with eager
    work and synchronisation between, from either starting buffer."""
    say(f"case: captured loops on bands, {dtype}")
    reals = draw([100, 33, 140, 64], 14)
    kw = dict(m=2, statistics="distinguishable", boundary="open", interaction="onsite", dtype=dtype, reals=reals, dt=0.05,
              tol=1e-7, sites=[20, 21])
    eager, graph = gpu_plan(**kw, launch={"persistent": 1}), gpu_plan(**kw, launch={"persistent": 1, "use_graph": 1})
    for n in (6, 6, 7, 7, 6, 7):
        eager.propagate(n)
        graph.propagate(n)
        assert np.array_equal(graph.observe(1), eager.observe(1))
        assert np.array_equal(graph.state_numpy(), eager.state_numpy())
        assert all(np.array_equal(a, b) for a, b in zip(graph.realization_norms(), eager.realization_norms()))
    assert graph.stats().steps_done == eager.stats().steps_done == 39


def test_timed_captured_loops_count_every_step():
    say("case: timed captured loops on bands, 2 x 300 steps")
    kw = dict(m=2, statistics="distinguishable", boundary="open", interaction="onsite", dtype="c64",
              reals=draw([100, 33, 140], 16), dt=0.05, tol=1e-7, launch={"persistent": 1, "use_graph": 1}, sites=[20, 21])
    plain, timed = gpu_plan(**kw), gpu_plan(**kw)
    timed.set_timing(True)
    for rep in (1, 2):
        plain.propagate(300)
        timed.propagate(300)
        ms, launches = timed.get_timing()
        assert launches == 300 * rep and ms > 0
        assert np.array_equal(plain.state_numpy(), timed.state_numpy())


@pytest.mark.parametrize("stat,bc,interaction", [("fermion", "open", "nearest"), ("boson", "open", "onsite"),
                                                 ("distinguishable", "periodic", "nearest")])
@pytest.mark.parametrize("launch", [{}, {"cols_per_lane": 2}, {"chunked": 1}, {"persistent": 1, "waves_per_block": 2}])
def test_complex128_against_the_oracle(stat, bc, interaction, launch):
    reals = draw([71, 140, 9, 64], 3, bc)
    plan = gpu_plan(m=2, statistics=stat, boundary=bc, interaction=interaction, dtype="c128", reals=reals, dt=0.05, order=7,
                    tol=0.0, launch=launch, sites=[3, 7])
    plan.propagate(60)
    err = worst_error(plan, reals, stat, bc, interaction, [3, 7], 0.05, 60, 7)
    say(f"case: bands c128 {stat} {bc} {interaction} {launch}: {err:.1e}")
    assert err <= 1e-12


@pytest.mark.parametrize("acc", ["kahan", "plain"])
@pytest.mark.parametrize("stat", ["distinguishable", "boson", "fermion"])
@pytest.mark.parametrize("launch", [{}, {"cols_per_lane": 2}, {"chunked": 1}])
def test_complex64_against_the_oracle(stat, acc, launch):
    reals = draw([64, 140, 100], 10)
    plan = gpu_plan(m=2, statistics=stat, boundary="open", interaction="onsite", dtype="c64", accumulation=acc,
                    reals=reals, dt=0.05, order=7, tol=0.0, launch=launch, sites=[30, 33])
    plan.propagate(200)
    err = worst_error(plan, reals, stat, "open", "onsite", [30, 33], 0.05, 200, 7)
    n2, _ = plan.realization_norms()
    say(f"case: bands c64 {stat} {acc} {launch}: {err:.1e}, |norm - 1| {np.max(np.abs(np.sqrt(n2) - 1)):.1e}")
    assert err <= (1e-6 if acc == "kahan" else 7e-6)


def test_compensated_sum_against_plain():
    """400 steps at a fixed order against the FP64 map of the same order: the
    compensated sum drifts less than half as much in norm, and is closer."""
    reals, steps = draw([140, 48], 21), 400
    res = {}
    for acc in ("kahan", "plain"):
        plan = gpu_plan(m=2, statistics="distinguishable", boundary="open", interaction="onsite", dtype="c64",
                        accumulation=acc, reals=reals, dt=0.05, order=7, tol=0.0, sites=[23, 24])
        plan.propagate(steps)
        err = worst_error(plan, reals, "distinguishable", "open", "onsite", [23, 24], 0.05, steps, 7)
        n2, _ = plan.realization_norms()
        res[acc] = (err, float(np.max(np.abs(n2 - 1))))
        say(f"case: sums on bands, {acc}: {err:.2e}, norm drift {res[acc][1]:.2e}")
    assert res["kahan"][0] < res["plain"][0] and res["kahan"][1] < 0.5 * res["plain"][1]


@pytest.mark.parametrize("dtype,bar", [("c128", 1e-12), ("c64", 6e-7)])
def test_forced_passes_match_the_fused_kernel(dtype, bar):
    """60 steps; complex64: a rounding of 6e-8 per step on either side in a
    random walk, sqrt(60) 6e-8 = 4.6e-7, times sqrt 2."""
    reals = draw([100, 140, 33], 4)
    kw = dict(m=2, statistics="distinguishable", boundary="open", interaction="onsite", dtype=dtype, reals=reals, dt=0.05,
              order=7, tol=0.0, sites=[16, 17])
    fused, passes = gpu_plan(**kw), gpu_plan(**kw, launch={"chunked": 1})
    for p in (fused, passes):
        p.propagate(60)
    d = float(np.max(np.abs(fused.state_numpy().astype(np.complex128) - passes.state_numpy())))
    say(f"case: passes and fused steps on bands, {dtype}: {d:.1e}")
    assert d <= bar


@pytest.mark.parametrize("stat,bc", [("boson", "open"), ("distinguishable", "periodic")])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_checkpoint_spacing_with_a_kept_segment(stat, bc, dtype):
    """The forward run keeps the newest segment's states where the backward pass
    would recompute them: one to 12 of them, or none (spacing 1).  The same bits
    for every spacing, and through the two-call form with the loss between."""
    N = 140
    g = np.random.default_rng(8)
    reals = [(N, 1 + 0.1 * g.standard_normal(N if bc == "periodic" else N - 1), g.uniform(-0.3, 0.3, N), 1.0) for _ in range(2)]
    sw = np.linspace(-1, 1, N)
    plan = gpu_plan(m=2, statistics=stat, boundary=bc, interaction="onsite", dtype=dtype, reals=reals, dt=0.05, order=6,
                    tol=0.0, sites=[60, 63])
    out = []
    for every in (1, 2, 5, 7, 12, 13, 40):
        plan.init_product_state([60, 63])
        loss, gJ, gE = plan.gradient(13, every, sw, "product")
        out.append(np.concatenate([[loss], gJ, gE]))
    plan.init_product_state([60, 63])
    plan.forward_ckpt(13, 5)
    between = plan.loss(sw, "product")
    loss, gJ, gE = plan.backward(sw, "product")
    out.append(np.concatenate([[loss], gJ, gE]))
    say(f"case: kept segment {stat} {bc} {dtype}: loss {out[0][0]:.6e} / {between:.6e}")
    assert np.all(np.isfinite(out[0])) and np.linalg.norm(out[0][1:]) > 0 and between == loss
    for o in out[1:]:
        assert np.array_equal(o, out[0])


@pytest.mark.parametrize("dtype,bar", [("c128", 1e-12), ("c64", 2e-6)])
def test_bosons_of_128_nodes_on_bands_and_on_chip(dtype, bar):
    """The two-boson batch's size, 100 steps, once with a realisation of 140
    nodes beside it.  complex64: the plain random walk of 100 roundings on either
    side, 2 x sqrt(100) 6e-8 = 1.2e-6."""
    reals = draw([128] * 60, 5)
    kw = dict(m=2, statistics="boson", boundary="open", interaction="onsite", dtype=dtype, dt=0.05, order=12, tol=0.0,
              sites=[63, 64])
    chip, bands = gpu_plan(**kw, reals=reals), gpu_plan(**kw, reals=reals + draw([140], 6))
    for p in (chip, bands):
        p.propagate(100)
    n = int(chip.layout()[-1])
    d = float(np.max(np.abs(chip.state_numpy().astype(np.complex128) - bands.state_numpy()[:n])))
    say(f"case: 60 x two bosons, N = 128, {dtype}: on chip and on bands {d:.1e}")
    assert d <= bar
