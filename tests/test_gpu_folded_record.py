"""Per-step records where a step's finalisation rides in the next step's passes, against
the same steps with a finalisation of their own (per-pass timing on)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# run-time-length grids with x blocks of one wave, two, four and more; the last sums its
# partials in two stages (the second in the y lines)
GRIDS = [(90, 70, 1), (600, 540, 1), (1001, 777, 1), (1500, 1300, 1), (33, 45, 50),
         (101, 75, 63), (200, 150, 130)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", GRIDS, ids=lambda n: "x".join(map(str, n)))
def test_folded_records_are_the_same(n, prec):
    from paper_1601_04640_amd.binding import Solver
    w = dict(geom="3d" if n[2] > 1 else "2dxz", nx=n[0], ny=n[1], nz=n[2], dx=0.3, dy=0.25,
             dz=0.35, dt=0.001, gamma=1.0, nu=1.0, lam=2.0, g=10.0, gdd=5.0, R=0.0)
    if n[2] == 1:
        w.update(ny=1, nz=n[1], nu=4.0)
    print(n, prec, flush=True)
    got = []
    for timed in (False, True):
        s = Solver(w, prec=prec)
        if timed:
            s.timing_enable(("finalize",))
        z = np.random.default_rng(n[0]).standard_normal(s.shape + (2,)) @ np.array([1.0, 1j])
        s.set_psi(z / np.sqrt((np.abs(z) ** 2).sum()))
        s.step_imag(3)
        s.step_real(2)
        s.step_imag(10)
        got.append((s.history(15), s.get_psi(), s.energy()))
        s.close()
    assert len(got[0][0]) == 15
    assert str(got[0][0]) == str(got[1][0])  # the same sums in the same order, bit for bit
    assert np.array_equal(got[0][1], got[1][1]) and got[0][2] == got[1][2]
