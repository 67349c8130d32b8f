"""Sums over the gradient rows of rows that a batch addresses very often: units of 256 gradient rows, with remainders, for every
alignment of a row and every number of lanes that share one.  Bars and inputs as in the parity tests."""

import pytest

from tests.test_gpu_nonfinite import DOT, DST, LOGISTIC
from tests.test_gpu_parity import BOTH, COMPLEX, DISTMULT, SOFTMAX, _case, _check_every_batch

pytestmark = pytest.mark.gpu

# Two batches each, the second a partial one, of more than 4096 gradient rows on few table rows; 16, 8 and 4 bytes' alignment, rows
# narrower and wider than the columns of a pass.  12 nodes: several units a row; 110: one unit, most of it empty.
_LONG = [
    _case("d1_v12", DOT, LOGISTIC, DST, 12, 0, 1, 1, 0, 0, 500, 50, 500, 0, 700, 0.5),
    _case("d30_v40", DISTMULT, SOFTMAX, BOTH, 40, 2, 30, 1, 0, 0, 300, 50, 500, 0, 520, 0.3),
    _case("d33_v12", DOT, SOFTMAX, DST, 12, 0, 33, 1, 0, 0, 500, 50, 500, 0, 777, 0.3),
    _case("d50_v110", COMPLEX, SOFTMAX, BOTH, 110, 3, 50, 1, 0, 0, 400, 100, 600, 0, 611, 0.3),
    _case("d100_v40", DOT, SOFTMAX, DST, 40, 0, 100, 1, 0, 0, 600, 50, 513, 0, 900, 0.3),
    _case("d130_v12", DISTMULT, LOGISTIC, BOTH, 12, 1, 130, 1, 0, 0, 200, 50, 600, 0, 333, 0.2),
    _case("d257_v110", DOT, LOGISTIC, DST, 110, 0, 257, 1, 0, 0, 500, 100, 900, 0, 800, 0.15),
    _case("d400_v40", DISTMULT, SOFTMAX, BOTH, 40, 2, 400, 1, 0, 0, 200, 100, 700, 0, 300, 0.15),
]


@pytest.mark.parametrize("c", _LONG, ids=[c["name"] for c in _LONG])
def test_rows_of_many_gradients(c):
    _check_every_batch(c)
