"""Block mapping of the general-graph terms: groups of realisations go to one
XCD each where they fill the device evenly (8, 14 or 33 groups here) and are
dealt in turn otherwise (1, 5, 9).  A realisation's arithmetic does not depend
on its batch, so its state and its norms are bit for bit those of a batch of
one.  500 nodes (two blocks, the second partly empty), a node without
neighbours, slots of width 1 to 6, orders whose last term does and does not
add the term before it."""

import numpy as np
import pytest

from _helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("width,order,R", [(1, 1, 5), (2, 2, 8), (4, 3, 9), (5, 6, 14), (6, 7, 33), (4, 5, 132)])
def test_a_realisation_does_not_depend_on_its_batch(dtype, width, order, R):
    import torch
    from paper_1612_00746_amd import graph_evolve
    n, steps = 500, 3
    g = np.random.default_rng(R)
    nbr = g.integers(-1, n, (width, n)).astype(np.int32)   # any gather table: symmetry is not required
    nbr[:, 7] = -1
    nbr[0, 8] = n                                          # past the end: empty as well
    cplx, real = (np.complex128, np.float64) if dtype == "c128" else (np.complex64, np.float32)
    hop = g.uniform(0.5, 1.0, (R, width, n)).astype(real)
    on = g.uniform(-0.5, 0.5, (R, n)).astype(real)
    psi0 = (g.standard_normal((R, n)) + 1j * g.standard_normal((R, n))).astype(cplx)

    def run(rs):
        psi = torch.from_numpy(psi0[rs].copy()).cuda()
        norms = torch.zeros(steps, len(rs), dtype=torch.float64, device="cuda")
        graph_evolve(torch.from_numpy(nbr).cuda(), torch.from_numpy(hop[rs].copy()).cuda(),
                     torch.from_numpy(on[rs].copy()).cuda(), psi, 0.1, order, steps, norms=norms)
        return psi.cpu().numpy(), norms.cpu().numpy()

    psi, norms = run(list(range(R)))
    say(f"case: graph blocks {dtype} width {width} order {order} R={R}: first norm {norms[0, 0]:.6f}")
    for r in sorted({0, R // 2, R - 1}):
        one, n1 = run([r])
        assert np.array_equal(one[0], psi[r]) and np.array_equal(n1[:, 0], norms[:, r]), r
    assert np.allclose(norms[-1], np.sum(np.abs(psi.astype(np.complex128)) ** 2, axis=1), rtol=1e-12)
