"""3D y and z lines past the register sweeps' 2048 rows: with at least 32768 lines one thread per
line and the forward values in a scratch grid (kg_cn_cols), with fewer several waves per line
over strided tiles (kg_cn_tile).  Free product states as in test_gpu_sweep, at its tolerance;
tests/host/shapes_main.hip checks that these lengths take these forms."""
import pytest

from tests.test_gpu_sweep import test_free_product_state as check_product_state

pytestmark = pytest.mark.gpu

SHAPES = [
    ("3d", (182, 2100, 181), "fp32"),    # 32942 lines of 2100
    ("3d", (182, 181, 2100), "fp32"),
    ("3d", (182, 2100, 181), "fp64"),
    ("3d", (182, 181, 2052), "fp64"),
    ("3d", (18, 2100, 22), "fp32"),      # 396 lines
    ("3d", (18, 22, 2052), "fp32"),
    ("3d", (18, 2052, 22), "fp64"),
    ("3d", (18, 22, 2100), "fp64"),
]


@pytest.mark.parametrize("imag", [True, False], ids=["imag", "real"])
@pytest.mark.parametrize("geom,n,prec", SHAPES, ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_lines_past_the_register_sweeps(geom, n, prec, imag):
    check_product_state(geom, n, prec, imag)
