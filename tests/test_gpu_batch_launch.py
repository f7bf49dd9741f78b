"""Launch forms of the batched ensemble: both size classes in one launch, a launch per
class, and persistent blocks run the same tile bodies on the same tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# instances of one class only, of both, and of classes that differ between the axes; 17
# tiles leave a remainder beside the runs of 16 items
SETS = {
    "short": [(32, 48), (96, 64), (256, 192)],
    "long": [(384, 512)],
    "both": [(512, 32), (32, 384), (96, 128), (192, 512), (48, 48)],
}


def _params(n0, n1, i):
    p = dict(nx=n0, dx=0.1, dy=0.1, dz=0.1, dt=1e-3, g=5.0 + i, gdd=2.0, gamma=1.0)
    if i % 2:
        return dict(p, geom="2dxz", ny=1, nz=n1, nu=4.0, lam=1.0 + 0.1 * i)
    return dict(p, geom="2dxy", ny=n1, nz=1, nu=1.0 + 0.1 * i, lam=4.0)


def _run(prec, sizes, imag, change):
    from paper_1601_04640_amd.binding import Batch
    b = Batch([_params(n0, n1, i) for i, (n0, n1) in enumerate(sizes)], prec=prec)
    change(b)
    rng = np.random.default_rng(7)
    for i in range(b.count):
        z = rng.standard_normal(b.shapes[i] + (2,)) @ np.array([1.0, 1j])
        b.set_psi(i, z / np.sqrt((np.abs(z) ** 2).sum() * 0.01))
    (b.step_imag if imag else b.step_real)(3)
    out = [b.get_psi(i) for i in range(b.count)]
    hist = [b.history(i, 3) for i in range(b.count)]
    b.close()
    return out, hist


def _persistent(b):
    for (p, k), (items, _) in b.plan().items():
        if items > 1:
            b.set_blocks(p, k, min(items - 1, 16))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("sizes", list(SETS))
@pytest.mark.parametrize("imag", [True, False])
def test_launch_forms_agree_bitwise(prec, sizes, imag):
    ref, href = _run(prec, SETS[sizes], imag, lambda b: None)
    for change in (lambda b: b.use_streams(True), _persistent):
        got, hgot = _run(prec, SETS[sizes], imag, change)
        for x, y in zip(ref, got):
            assert np.all(np.isfinite(x)) and np.array_equal(x, y)
        assert str(href) == str(hgot)


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-6)])
def test_energies_of_all_instances(prec, tol):
    """The records of one batch call against each instance's own (same terms and sums;
    multiply-adds may be contracted differently), after steps and with a changed coupling;
    an instance without a state, or with a state that is not finite, is an error."""
    from paper_1601_04640_amd.binding import Batch, GPError, gp_energy, gp_set_couplings
    sizes = SETS["both"]
    b = Batch([_params(n0, n1, i) for i, (n0, n1) in enumerate(sizes)], prec=prec)
    rng = np.random.default_rng(11)
    psi = [rng.standard_normal(s + (2,)) @ np.array([1.0, 1j]) for s in b.shapes]
    for i, z in enumerate(psi[:-1]):
        b.set_psi(i, z / np.sqrt((np.abs(z) ** 2).sum() * 0.01))
    with pytest.raises(GPError):
        b.energy()
    b.set_psi(b.count - 1, psi[-1])
    b.step_real(2)
    gp_set_couplings(b.ctxs[1], 3.0, 1.0)
    for got, ctx in zip(b.energy(), b.ctxs):
        ref = gp_energy(ctx)
        for key in ref:
            assert np.allclose(got[key], ref[key], rtol=tol, atol=tol * abs(ref["energy"])), key
    bad = psi[2].copy()
    bad[3, 5] = np.nan
    b.set_psi(2, bad)
    with pytest.raises(GPError):
        b.energy()
    b.close()
