"""Observables of a given state at the edges of their tiles (16 x 128 pairs,
32 x 128 for three particles), for one and many segments of realisations and
uneven groups, against the definition evaluated by numpy in FP64 on the same
state.  Both add the same FP64 products in other orders: sums of at most 2e6
positive terms, relative 1e-12 of the largest entry."""

import numpy as np
import pytest

from _helpers import say

pytestmark = pytest.mark.gpu


def make(m, stat, Ns, dtype, seed):
    from paper_1612_00746_amd import Plan, make_problem
    g = np.random.default_rng(seed)
    uniform = len(set(Ns)) == 1
    pr, keep = make_problem(m, len(Ns), Ns[0] if uniform else Ns, 0.05, statistics=stat, dtype=dtype, taylor_order=3,
                            observables=1 if m == 1 else 3)
    plan = Plan(pr)
    plan._keep.append(keep)
    plan.set_params(np.ones(sum(N - 1 for N in Ns)), np.zeros(sum(Ns)), np.ones(len(Ns)))
    plan.bind()
    n = int(plan.layout()[-1])
    psi = (g.standard_normal(n) + 1j * g.standard_normal(n)).astype(np.complex64 if dtype == "c64" else np.complex128)
    plan.set_state_numpy(psi)
    return plan, psi


def expected(m, stat, Ns, off, psi):
    out = []
    for N in sorted(set(Ns)):
        rs = [r for r in range(len(Ns)) if Ns[r] == N]
        occ, pair = np.zeros(N), np.zeros((N, N))
        for r in rs:
            p = np.abs(psi[off[r]:off[r + 1]].astype(np.complex128)) ** 2
            if m == 2 and stat != "distinguishable":
                full = np.zeros((N, N))
                full[np.triu_indices(N)] = p
                p = np.where(np.eye(N, dtype=bool), full, full + full.T)
            p = p.reshape([N] * m)
            for a in range(m):
                occ += p.sum(tuple(x for x in range(m) if x != a))
                for b in range(a + 1, m):
                    q = p.sum(tuple(x for x in range(m) if x not in (a, b)))
                    pair += q + q.T
        out += [occ / len(rs)] if m == 1 else [occ / len(rs), (pair / len(rs)).ravel()]
    return np.concatenate(out)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("m,stat,Ns", [
    (1, "distinguishable", [2, 128, 129, 127, 300, 128] + [33] * 70),
    (1, "distinguishable", [700]),
    (2, "distinguishable", [2, 15, 16, 17] + [33] * 40),
    (2, "distinguishable", [129]),
    (2, "distinguishable", [127, 128, 129, 160, 128]),
    (2, "boson", [2, 15, 16, 17, 130] + [48] * 30),
    (2, "fermion", [64] * 5),
    (3, "distinguishable", [31]),
    (3, "distinguishable", [33] * 5),
    (3, "distinguishable", [130]),
])
def test_observables_against_their_definition(m, stat, Ns, dtype):
    say(f"case: observables m={m} {stat} N={sorted(set(Ns))} R={len(Ns)} {dtype}")
    plan, psi = make(m, stat, Ns, dtype, 11)
    want = expected(m, stat, Ns, plan.layout(), psi)
    got = plan.observe(1 if m == 1 else 3)
    assert np.max(np.abs(got - want)) <= 1e-12 * np.max(np.abs(want))


def test_snapshots_of_a_long_run_match_single_observations():
    """More outputs than the device holds at a time (64): each equals the
    observation made at its step of an identical run."""
    say("case: 150 snapshots")
    runs = [make(2, "boson", [9, 14, 9], "c128", 5)[0] for _ in range(2)]
    out = runs[0].propagate(149, 1, 3)
    for k in range(150):
        if k:
            runs[1].propagate(1)
        assert np.array_equal(out[k], runs[1].observe(3)), k


def test_state_copies_on_the_device():
    """ctqw_set_state / ctqw_get_state with device pointers, 16-byte aligned
    and not (an odd element offset of complex64)."""
    import ctypes as C

    import torch
    plan, psi = make(2, "distinguishable", [17, 5], "c64", 3)
    n = len(psi)
    for shift in (0, 1):
        buf = torch.zeros(n + 2, dtype=torch.complex64, device="cuda")
        view = buf[shift:shift + n]
        assert plan.lib.ctqw_get_state(plan.h, C.c_void_p(view.data_ptr()), 1) == 0
        assert np.array_equal(view.cpu().numpy(), psi) and float(buf[n + 1].abs()) == 0.0
        twice = (2 * view).clone() if shift == 0 else torch.cat([buf[:1], 2 * view])[1:]
        torch.cuda.synchronize()
        assert plan.lib.ctqw_set_state(plan.h, C.c_void_p(twice.data_ptr()), 1) == 0
        assert np.array_equal(plan.state_numpy(), 2 * psi)
        plan.set_state_numpy(psi)
