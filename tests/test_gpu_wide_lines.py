"""Wide-p gradient between 256 and 320 workgroups of the wider spans (GPU tier), where short or many
row slices take 16 columns per wave, and just outside. Bars and references as in
test_gpu_wide_columns.py."""
import pytest

import test_gpu_wide_columns as wide

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f64,n,p,K,pad", [
    (False, 324, 12637, 32, 1), (False, 1402, 2908, 32, 0), (False, 5767, 532, 20, 0), (False, 646, 11334, 17, 0),
    (False, 1090, 15666, 20, 0), (False, 250, 20481, 20, 0), (True, 65, 32969, 17, 0), (True, 1159, 1687, 24, 1),
    (True, 13996, 411, 20, 0), (True, 8574, 688, 64, 0), (True, 427, 12026, 32, 0)])
def test_lines(lib, f64, n, p, K, pad):
    wide.test_span_edges(lib, n, p, K, pad, 0, f64)
