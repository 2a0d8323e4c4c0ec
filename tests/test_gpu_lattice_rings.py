"""The lattice kernel's two rings: orders 4 to 9 sweep in blocks of either
length, whichever covers the sweep in fewer rows, against the same Taylor
polynomial in FP64.

Tolerances, 2-norm relative after 2 steps at dt = 0.05 (dt ||H|| < 0.3): a step
rounds the state once and its terms' sum n times at less than 0.3 of it,
2 (1 + 0.3 n) 6e-8 <= 5e-7 at n = 9 in complex64, 1e-6; complex128 1e-15, held
to 1e-13; squared norms to twice that."""

import numpy as np
import pytest

from _helpers import say
from test_gpu_lattice_tiles import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("order", [4, 5, 6, 7, 8, 9])
def test_sweeps_over_either_ring(order, dtype):
    """Rows such that the sweep's length falls on every remainder of both
    rings' blocks, open and closed in y, in one and two bands; the longest also
    in segments."""
    import torch

    from paper_1612_00746_amd import lattice_evolve
    real, cplx = (np.float32, np.complex64) if dtype == "c64" else (np.float64, np.complex128)
    bar = 1e-6 if dtype == "c64" else 1e-13
    g = np.random.default_rng(order)
    for Lx, R, py, Ly in [(Lx, R, py, Ly) for Lx, R in ((5, 3), (70, 2), (40, 1100)) for py in (0, 1)
                          for Ly in (range(3, 17) if R < 1000 else (3, 8, 13)) if py == 0 or Ly >= 3] + [(9, 2, 0, 61)]:
        say(f"case: lattice {Lx}x{Ly} R={R} ring in y {py} order {order} {dtype}")
        shape = (R, Ly, Lx)
        Jx, Jy = ((1 + 0.1 * g.standard_normal(shape)).astype(real) for _ in range(2))
        eps = g.uniform(-0.5, 0.5, shape).astype(real)
        psi = (g.standard_normal(shape) + 1j * g.standard_normal(shape)).astype(cplx)
        psi /= np.sqrt(np.sum(np.abs(psi) ** 2, axis=(1, 2), keepdims=True))
        ref, norms = reference(Jx, Jy, eps, psi, 0, py, 0.05, order, 2)
        dev = [torch.from_numpy(x).cuda() for x in (Jx, Jy, eps, psi.copy())]
        out = torch.empty((2, R), dtype=torch.float64, device="cuda")
        lattice_evolve(*dev, 0.05, order, 2, periodic=(False, bool(py)), norms=out)
        got = dev[3].cpu().numpy()
        err = np.linalg.norm((got - ref).reshape(R, -1), axis=1).max()
        say(f"  error {err:.1e}, norms {np.abs(out.cpu().numpy() - norms).max():.1e}")
        assert err <= bar and np.abs(out.cpu().numpy() - norms).max() <= 2 * bar
