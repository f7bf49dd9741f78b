"""The x sweep where its factors take the twiddles' LDS and its gains come from L2: tiles of one
and two pairs with lines of one wave to sixteen, in both precisions, and the longest lines (the
free product states of test_gpu_sweep, at its tolerance)."""
import pytest

from tests.test_gpu_sweep import test_free_product_state as check_product_state

pytestmark = pytest.mark.gpu

SHAPES = [
    ("2dxy", (34, 1030, 1), "fp64"),     # a chunk and two rows
    ("2dxy", (640, 1030, 1), "fp64"),    # two pairs
    ("3d", (760, 18, 70), "fp64"),
    ("2dxy", (1200, 22, 1), "fp64"),     # one pair
    ("2dxy", (1210, 601, 1), "fp64"),    # radix 11
    ("2dxy", (1728, 21, 1), "fp64"),
    ("2dxy", (2000, 23, 1), "fp64"),
    ("2dxy", (1922, 20, 1), "fp64"),     # radix 31, the last two lengths to 2048
    ("2dxy", (2048, 21, 1), "fp64"),
    ("2dxy", (1600, 1090, 1), "fp32"),   # two pairs of 8-row chunks
    ("2dxy", (2000, 530, 1), "fp32"),    # one pair
    ("3d", (500, 180, 100), "fp32"),     # 16-row chunks
    ("2dxy", (2048, 2050, 1), "fp32"),
    ("2dxy", (3978, 22, 1), "fp32"),     # 16-row chunks past 2048 points
    ("2dxy", (4056, 23, 1), "fp32"),
]


@pytest.mark.parametrize("imag", [True, False], ids=["imag", "real"])
@pytest.mark.parametrize("geom,n,prec", SHAPES, ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_x_sweep(geom, n, prec, imag):
    check_product_state(geom, n, prec, imag)
