"""Gradients of one particle: its adjoint passes are stencils of a single row.
Chains and rings of one band, of several, at a band's edges and shorter than a
pass's halo, at orders that reach every depth of pass, against the derivative
of the truncated map in FP64 (numpy, the recursion written out densely).

Tolerance: in 6 steps the state and the adjoint vector each collect 6 (1 + 0.3 n)
roundings, 6e-8 each in complex64, 1.7e-6 at n = 12; a gradient is
2 dt sum_steps Im <u|dH|v> with |u||v| <= e^0.2, so its error is below
2 x 0.05 x 6 x 2 x 1.7e-6 x 1.3 = 2.7e-6: 4e-6, and 1e-13 in complex128."""

import math

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


def reference(reals, sites, boundary, dt, order, steps, w):
    N, R = reals[0][0], len(reals)
    loss, gJ, gE = 0.0, 0.0, 0.0
    a = np.arange(N if boundary == "periodic" else N - 1)
    b = (a + 1) % N
    for _, J, eps, _ in reals:
        H = np.diag(eps).astype(complex)
        H[a, b] += J
        H[b, a] += J
        A = -1j * dt * H
        psi = [np.zeros(N, complex)]
        psi[0][sites[0]] = 1
        for _ in range(steps):
            t = out = psi[-1]
            for j in range(1, order + 1):
                t = A @ t / j
                out = out + t
            psi.append(out)
        lam = w * psi[-1]
        loss += np.vdot(psi[-1], lam).real
        for k in range(steps - 1, -1, -1):
            v = [psi[k]]
            for _ in range(order - 1):
                v.append(A @ v[-1])
            u = lam / math.factorial(order)
            for i in range(order - 1, -1, -1):
                gE = gE + 2 * dt * np.imag(np.conj(u) * v[i])
                gJ = gJ + 2 * dt * np.imag(np.conj(u[a]) * v[i][b] + np.conj(u[b]) * v[i][a])
                u = lam / math.factorial(i) + A.conj().T @ u
            lam = u
    return loss / R, gJ / R, gE / R


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("N,R,boundary,order", [
    (2, 3, "open", 1), (3, 2, "periodic", 4), (5, 9, "open", 12), (51, 2, "periodic", 11), (56, 3, "open", 9),
    (57, 1, "open", 8), (60, 4, "periodic", 2), (61, 2, "open", 3), (63, 2, "open", 5), (64, 8, "periodic", 6),
    (65, 2, "open", 7), (113, 3, "periodic", 10), (130, 17, "open", 12), (300, 2, "periodic", 8),
])
def test_one_particle(N, R, boundary, order, dtype):
    dt, steps = 0.05, 6
    g = np.random.default_rng(N + order)
    bonds = N if boundary == "periodic" else N - 1
    reals = [(N, 1 + 0.1 * g.standard_normal(bonds), g.uniform(-0.3, 0.3, N), 1.0) for _ in range(R)]
    sites, w = [N // 2], np.linspace(-1, 1, N)
    plan = gpu_plan(m=1, statistics="distinguishable", boundary=boundary, interaction="onsite", dtype=dtype, reals=reals,
                    dt=dt, order=order, tol=0.0, sites=sites)
    loss, gJ, gE = plan.gradient(steps, 4, w, "one_body")
    l0, j0, e0 = reference(reals, sites, boundary, dt, order, steps, w)
    bar = 4e-6 if dtype == "c64" else 1e-13
    dJ, dE = np.linalg.norm(gJ - j0), np.linalg.norm(gE - e0)
    say(f"case: one-particle gradient N={N} R={R} {boundary} order {order} {dtype}: loss {abs(loss - l0):.1e}, J {dJ:.1e}, "
        f"eps {dE:.1e}, |gE| {np.linalg.norm(e0):.1e}")
    assert abs(loss - l0) <= 10 * bar and dJ <= bar and dE <= bar
