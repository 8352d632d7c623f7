"""RAS sweep and factorisation with long wells.

A row's entries past the eighth lie apart and are worked on in rounds of pairs
of columns, whose two block layouts alternate.  Wells of 37 to 625
perforations: odd and even numbers of pairs, the second well's pairs behind an
odd and an even number of the first one's, and last rounds of every length.
Checked as in the layout test.
"""
import pytest

from test_gpu_ras_layout import test_factors_and_application as check_layout

pytestmark = pytest.mark.gpu

# nx, ny, nz (the perforations of a well), px, py, overlap, order, spread
CASES = [(3, 3, nz, 1, 1, 0, 1, 5.0) for nz in (37, 38, 40, 41, 43, 45, 46, 48, 50)] + [
    (3, 3, 200, 1, 1, 0, 1, 50.0), (2, 2, 333, 1, 1, 0, 1, 50.0), (4, 2, 625, 2, 1, 1, 1, 50.0),
    (3, 2, 120, 1, 1, 0, 0, 0.0)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_long_wells(case, precision):
    check_layout(case, precision)
