"""The one-column pass on both sides of the lines of its rule (GPU tier): the smallest problems of a
few columns that it takes and the largest left to the row tile, odd columns with and without row
padding in float64. Bars and references as in test_gpu_one_column.py."""
import pytest

import test_gpu_one_column as one_column

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("link", ["logit", "poisson", "probit"])
@pytest.mark.parametrize("f64,n,p,pad", [
    (False, 65535, 3, 0), (False, 65536, 3, 0), (False, 65536, 1, 2), (False, 16383, 15, 1), (False, 16384, 15, 1),
    (False, 16385, 4, 0), (False, 8191, 16, 0), (False, 8192, 16, 3), (True, 700001, 3, 1), (True, 33000, 64, 0),
    (True, 16513, 127, 0), (True, 16513, 127, 1), (True, 16257, 129, 0)])
def test_lines(lib, f64, n, p, pad, link):
    one_column.test_edges(lib, f64, n, p, pad, link)
