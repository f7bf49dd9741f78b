"""Run-time-length FFTs (gp_rfft.hpp, gp_rx.hpp): the dipolar potential of a random density
against numpy's FFTs, with x, y and z lengths that take every radix, every tile width and
Bluestein's algorithm.

An FFT's error grows with the stages: the potential is held to 16 units in the last place
times log2 of the points, relative to its largest value."""
import numpy as np
import pytest

import oracle as O
from tests.gpu_util import banner, oparams

pytestmark = pytest.mark.gpu

# (nx, ny, nz); at least one length keeps the grid off the specialised passes
GRIDS = [
    (18, 22, 26), (18, 28, 33), (18, 34, 36), (18, 37, 39), (18, 42, 45), (18, 49, 50),
    (18, 54, 63), (18, 66, 70), (18, 74, 77), (18, 81, 91), (18, 100, 121), (18, 126, 143),
    (18, 135, 169), (18, 144, 196), (18, 210, 225), (18, 97, 101),
    (18, 14, 600), (18, 9, 1100), (18, 14, 397),       # narrower strided tiles, Bluestein
    (18, 601, 14), (22, 1024, 1), (22, 2000, 1), (22, 1999, 1), (22, 1331, 1), (22, 1093, 1),
    (26, 15, 18), (37, 18, 20), (63, 17, 18), (77, 34, 15), (100, 9, 18), (121, 18, 7), (169, 18, 9),
    (225, 33, 8), (397, 18, 10), (600, 21, 9), (1024, 18, 1), (1331, 21, 1), (2000, 19, 1),
    (1999, 18, 1), (144, 130, 70),
    # grids of a range that takes radices up to 8
    (36, 32, 30), (60, 50, 40), (63, 45, 20), (100, 81, 18), (225, 210, 1), (540, 600, 1),
    (700, 720, 1),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", GRIDS, ids=lambda n: "x".join(map(str, n)))
def test_potential(n, prec):
    from paper_1601_04640_amd.binding import Solver
    banner(n, prec)
    geom = "3d" if n[2] > 1 else "2dxy"
    w = dict(geom=geom, nx=n[0], ny=n[1], nz=n[2], dx=0.3, dy=0.25, dz=0.35, dt=0.001, gamma=1.0,
             nu=1.0, lam=2.0, g=10.0, gdd=5.0, R=2.0)
    p = oparams(w)
    rng = np.random.default_rng(n[1] * 4096 + n[2])
    psi = rng.uniform(0.5, 1.0, p.shape()) * np.exp(1j * rng.uniform(-1, 1, p.shape()))
    psi = O.zero_boundary(psi)
    if prec == "fp32":
        psi = psi.astype(np.complex64).astype(np.complex128)
    s = Solver(w, prec=prec)
    s.set_psi(psi)
    got = s.dipolar_potential()
    s.close()
    ref = O.dipolar_potential(np.abs(psi) ** 2, p)
    eps = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24}[prec]
    tol = 16 * eps * np.log2(psi.size)
    assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref))
