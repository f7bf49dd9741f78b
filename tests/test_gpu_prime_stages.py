"""Lengths with prime factors 17 to 31 run those factors as stages of their own: every such
radix alone, with a small one behind it, twice, and two of them; along x, y and z, planar (the y
convolution turns at the line's last radix) and 3D."""
import numpy as np
import pytest
import scipy.fft

import oracle as O
from tests.gpu_util import banner, oparams

pytestmark = pytest.mark.gpu

GRIDS = [
    (17, 19, 23), (29, 31, 17), (19, 34, 31), (38, 29, 46), (62, 58, 68), (51, 93, 85),
    (289, 323, 1), (31, 527, 1), (961, 34, 1), (34, 961, 1), (667, 17, 1), (1190, 186, 1),
    (203, 18, 119), (18, 14, 437), (18, 14, 380), (340, 310, 1), (187, 247, 1), (242, 713, 1),
    (1054, 40, 1), (290, 70, 46),
]


def _case(n, prec):
    geom = "3d" if n[2] > 1 else "2dxy"
    w = dict(geom=geom, nx=n[0], ny=n[1], nz=n[2], dx=0.3, dy=0.25, dz=0.35, dt=0.001, gamma=1.0,
             nu=1.0, lam=2.0, g=10.0, gdd=5.0, R=2.0)
    p = oparams(w)
    rng = np.random.default_rng(n[0] * 65536 + n[1] * 4096 + n[2])
    psi = rng.uniform(0.5, 1.0, p.shape()) * np.exp(1j * rng.uniform(-1, 1, p.shape()))
    psi = O.zero_boundary(psi)
    if prec == "fp32":
        psi = psi.astype(np.complex64).astype(np.complex128)
    return w, p, psi


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", GRIDS, ids=lambda n: "x".join(map(str, n)))
def test_potential(n, prec):
    """Phi of a random density, to 16 units in the last place times log2 of the points of its
    largest value (as the other line transforms)."""
    from paper_1601_04640_amd.binding import Solver
    banner("prime stages", n, prec)
    w, p, psi = _case(n, prec)
    s = Solver(w, prec=prec)
    s.set_psi(psi)
    got = s.dipolar_potential()
    s.close()
    ref = O.dipolar_potential(np.abs(psi) ** 2, p)
    eps = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24}[prec]
    assert np.max(np.abs(got - ref)) <= 16 * eps * np.log2(psi.size) * np.max(np.abs(ref))


@pytest.mark.parametrize("n", [(340, 54, 1), (54, 1190, 1), (18, 14, 380), (18, 14, 310)],
                         ids=lambda n: "x".join(map(str, n)))
def test_no_further_off_than_lengths_of_small_factors(n):
    """FP64 Phi against transforms in long double.  Lengths of 2, 3 and 5 are off by 0.17 (planar)
    and 0.36 (3D) units in the last place per log2 of the points in the root mean square; stages
    of a prime factor round no more often.  Twice that is half of what the detour over a
    convolution of twice the length gives."""
    from paper_1601_04640_amd.binding import Solver
    banner("prime stages, error", n)
    w, p, psi = _case(n, "fp64")
    s = Solver(w, prec="fp64")
    s.set_psi(psi)
    got = s.dipolar_potential()
    s.close()
    dens = psi.real.astype(np.longdouble) ** 2 + psi.imag.astype(np.longdouble) ** 2
    ref = scipy.fft.irfftn(scipy.fft.rfftn(dens) * O.dipolar_kernel(p).astype(np.longdouble), s=dens.shape)
    err = np.linalg.norm((got - ref).astype(np.float64)) / np.linalg.norm(ref.astype(np.float64))
    per_level = 2 * (0.36 if n[2] > 1 else 0.17)
    assert err <= per_level * 2.0 ** -53 * np.log2(psi.size)
