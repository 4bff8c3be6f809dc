"""The checks of the element-layout test at further sizes around the bricks of 16 x 4 x 2 elements: odd numbers of
element layers against two, and one element fewer and more than four rows (same oracle, same tolerances)."""
import pytest

import test_gpu_element_layout as layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [2, 3, 5, 17])
def test_brick_edges(n, prec):
    layout.test_element_layout_edges(n, prec)
