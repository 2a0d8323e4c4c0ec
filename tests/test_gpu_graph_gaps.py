"""Graph terms over tables with gaps: slots that are empty at some nodes, at all
nodes of a wave (64) and at all nodes, in every position of a group of four, with
one to nine realisations (complex64 takes four per thread, or one where there are
fewer).  Against the series in numpy (FP64) on the same tables, with dt ||H|| <=
0.6: complex128 2 steps x 6 terms x 16 products x 1.1e-16 = 2e-14; complex64 the
same count at 6e-8, 1.2e-5.  Norms: FP64 sums of the stored state, 1e-13."""

import numpy as np
import pytest

from _helpers import say

pytestmark = pytest.mark.gpu


def table(width, pattern, n, g):
    nbr = np.full((width, n), -1, np.int32)
    for k in range(width):
        used = np.zeros(n, bool)
        if pattern == "ends":            # the first and the last slot only
            used[:] = k in (0, width - 1)
        elif pattern == "waves":         # slot k at the waves k, k + 3, ... of 64 nodes
            used[:] = (np.arange(n) // 64 + k) % 3 == 0
        elif pattern == "few":           # one node per slot
            used[(37 * k) % n] = True
        else:                            # "some": at random
            used[:] = g.random(n) < 0.4
        nbr[k, used] = g.integers(0, n, int(used.sum()))
    if pattern == "some":
        nbr[0, ::7] = n                  # past the end: empty as well
    return nbr


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("pattern", ["ends", "waves", "few", "some"])
@pytest.mark.parametrize("width,n,R", [(1, 70, 1), (4, 300, 2), (5, 300, 3), (12, 700, 1), (13, 129, 4), (16, 64, 5),
                                       (31, 257, 9)])
def test_gaps(width, n, R, pattern, dtype):
    import torch

    from paper_1612_00746_amd import graph_evolve
    say(f"case: gaps {pattern} width={width} n={n} R={R} {dtype}")
    g = np.random.default_rng(width * n + R)
    nbr = table(width, pattern, n, g)
    hop, on = g.uniform(-1, 1, (R, width, n)), g.uniform(-1, 1, (R, n))
    hop /= max(1, width)
    psi = g.standard_normal((R, n)) + 1j * g.standard_normal((R, n))
    psi /= np.linalg.norm(psi, axis=1, keepdims=True)
    real, cplx = (np.float32, np.complex64) if dtype == "c64" else (np.float64, np.complex128)
    hop, on, psi = hop.astype(real), on.astype(real), psi.astype(cplx)
    order, steps, dt = 6, 2, 0.3
    ref = psi.astype(np.complex128)
    valid = (nbr >= 0) & (nbr < n)
    safe = np.where(valid, nbr, 0)
    for _ in range(steps):
        term, total = ref, ref.copy()
        for j in range(1, order + 1):
            h = on.astype(np.float64) * term
            for k in range(width):
                h = h + np.where(valid[k], hop[:, k].astype(np.float64) * term[:, safe[k]], 0.0)
            term = (-1j * dt / j) * h
            total = total + term
        ref = total
    d = {t: torch.from_numpy(np.ascontiguousarray(x)).cuda() for t, x in
         (("nbr", nbr), ("hop", hop), ("on", on), ("psi", psi))}
    norms = torch.empty((steps, R), dtype=torch.float64, device="cuda")
    graph_evolve(d["nbr"], d["hop"], d["on"], d["psi"], dt, order, steps, norms=norms)
    got = d["psi"].cpu().numpy().astype(np.complex128)
    err = np.max(np.abs(got - ref))
    say(f"  max error {err:.1e}")
    assert err <= (1.2e-5 if dtype == "c64" else 2e-14)
    assert np.allclose(norms[-1].cpu().numpy(), np.sum(np.abs(got) ** 2, axis=1), rtol=1e-13, atol=0)
