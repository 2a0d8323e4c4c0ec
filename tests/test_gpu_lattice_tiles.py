"""The lattice kernel at the edges of its shapes: widths around the bands of
64 and 128 columns, odd and even (paired access), rows whole and in segments,
every ring combination, orders 1 to 12, and arrays that are not 16-byte
aligned, against the same Taylor polynomial in FP64 (numpy, term by term).

Tolerances, 2-norm relative after 3 steps at dt = 0.05 (dt ||H|| < 0.3): each
step rounds the state once and the sum of its terms n times at less than 0.3
of it, 3 (1 + 0.3 n) 6e-8 <= 9e-7 at n = 12 in complex64, 1e-6; complex128
2e-15, held to 1e-13."""

import math

import numpy as np
import pytest

from _helpers import say

pytestmark = pytest.mark.gpu


def reference(Jx, Jy, eps, psi, px, py, dt, order, steps):
    Jx, Jy = Jx.astype(np.float64).copy(), Jy.astype(np.float64).copy()
    if not px:
        Jx[:, :, -1] = 0
    if not py:
        Jy[:, -1, :] = 0
    eps = eps.astype(np.float64)
    jl, ju = np.roll(Jx, 1, 2), np.roll(Jy, 1, 1)
    x, norms = psi.astype(np.complex128), []
    for _ in range(steps):
        t, out = x, x
        for k in range(1, order + 1):
            h = (eps * t + Jx * np.roll(t, -1, 2) + jl * np.roll(t, 1, 2) + Jy * np.roll(t, -1, 1) + ju * np.roll(t, 1, 1))
            t = -1j * dt / k * h
            out = out + t
        x = out
        norms.append(np.sum(np.abs(x) ** 2, axis=(1, 2)))
    return x, np.array(norms)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("Lx,Ly,R,px,py,order,shift", [
    (1, 1, 3, 0, 0, 3, 0), (3, 2, 2, 1, 0, 2, 0), (2, 7, 5, 0, 1, 1, 0),
    (44, 20, 2, 0, 0, 10, 0), (63, 9, 3, 1, 1, 9, 0), (64, 31, 2, 0, 0, 10, 0), (65, 64, 1, 0, 0, 6, 0),
    (64, 12, 1500, 0, 1, 4, 0), (108, 11, 1100, 0, 0, 10, 0), (109, 5, 1100, 1, 0, 9, 0),
    (118, 14, 1050, 0, 0, 10, 0), (127, 6, 1050, 0, 0, 7, 0), (128, 8, 1050, 0, 1, 10, 0), (128, 6, 1100, 0, 0, 9, 1),
    (129, 10, 700, 1, 1, 5, 0), (246, 7, 700, 0, 0, 10, 0), (300, 90, 1, 1, 1, 8, 0), (250, 40, 2, 0, 0, 10, 1),
    (70, 25, 3, 0, 0, 12, 0), (200, 33, 2, 0, 1, 11, 0),
])
def test_lattice_shapes(Lx, Ly, R, px, py, order, shift, dtype):
    import torch

    from paper_1612_00746_amd import lattice_evolve
    if dtype == "c128" and order > 10:
        order = 10
    say(f"case: lattice {Lx}x{Ly} R={R} rings {px}{py} order {order} shift {shift} {dtype}")
    g = np.random.default_rng(Lx * 1000 + Ly)
    real, cplx = (np.float32, np.complex64) if dtype == "c64" else (np.float64, np.complex128)
    shape = (R, Ly, Lx)
    Jx, Jy = ((1 + 0.1 * g.standard_normal(shape)).astype(real) for _ in range(2))
    eps = g.uniform(-0.5, 0.5, shape).astype(real)
    psi = ((g.standard_normal(shape) + 1j * g.standard_normal(shape)) / math.sqrt(2 * Lx * Ly)).astype(cplx)
    want, wn = reference(Jx, Jy, eps, psi, px, py, 0.05, order, 3)
    # an open axis's last bonds are ignored, whatever they hold
    if not px:
        Jx[:, :, -1] = np.nan
    if not py:
        Jy[:, -1, :] = np.inf

    def place(a):       # `shift` elements into a buffer: not 16-byte aligned
        buf = torch.zeros(a.size + 1, dtype=torch.from_numpy(a).dtype, device="cuda")
        v = buf[shift:shift + a.size].view(shape)
        v.copy_(torch.from_numpy(a))
        return v

    d = place(psi)
    norms = torch.zeros((3, R), dtype=torch.float64, device="cuda")
    lattice_evolve(place(Jx), place(Jy), place(eps), d, 0.05, order, 3, periodic=(px, py), norms=norms)
    got = d.cpu().numpy().astype(np.complex128)
    bar = 1e-6 if dtype == "c64" else 1e-13
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    say(f"  {err:.1e}, norms {np.max(np.abs(norms.cpu().numpy() / wn - 1)):.1e}")
    assert err <= bar
    assert np.allclose(norms.cpu().numpy(), wn, rtol=2 * bar, atol=0)


def test_norms_of_more_steps_than_one_reduction_takes():
    """20 steps (the partials of 8 wait for one reduction): the same norms as
    20 calls of one step, which leave the state in the other buffer."""
    import torch

    from paper_1612_00746_amd import lattice_evolve
    say("case: norms over 20 steps")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    J = 1 + 0.1 * torch.randn((3, 21, 34), generator=gen, device="cuda", dtype=torch.float64)
    psi = torch.randn((3, 21, 34), generator=gen, device="cuda", dtype=torch.complex128)
    a, b = psi.clone(), psi.clone()
    n20 = torch.zeros((20, 3), dtype=torch.float64, device="cuda")
    lattice_evolve(J, J, J, a, 0.05, 5, 20, norms=n20)
    for k in range(20):
        n1 = torch.zeros((1, 3), dtype=torch.float64, device="cuda")
        lattice_evolve(J, J, J, b, 0.05, 5, 1, norms=n1)
        assert torch.equal(n1[0], n20[k]), k
    assert torch.equal(a, b)
