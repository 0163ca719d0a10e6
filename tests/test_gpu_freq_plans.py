"""The frequency significance at the edges of the transforms' plans: lone and
small radices, the longest sides, odd heights (a row without a partner), and
row and column groups that the image does not fill.  Tolerance as for the
other sizes."""
import pytest

from test_gpu_freq import _check_X

pytestmark = pytest.mark.gpu

SMOOTH = [n for n in range(1, 65) if all(n % p for p in range(8, n + 1) if all(p % q for q in range(2, p)))]


@pytest.mark.parametrize("sizes", [
    [(n, SMOOTH[-1 - i]) for i, n in enumerate(SMOOTH)],
    [(2560, 5), (3, 2560), (2401, 4), (6, 2401), (2187, 3), (9, 2187), (2048, 2), (1, 2048), (2500, 7), (10, 2520)],
    [(375, 81), (640, 75), (1600, 9), (1620, 7), (1680, 3), (810, 125), (405, 245)],
    [(1600, 63), (960, 135), (240, 1029), (125, 1372)],
])
def test_significance_at_the_plans_edges(sizes):
    _check_X(sizes, 90 + len(sizes))
