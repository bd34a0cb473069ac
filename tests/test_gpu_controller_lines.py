"""The controller on both sides of the lines between its two layouts, which lie by elements,
steps, type and direction, against float64 (as test_gpu_controller_split has it)."""
import pytest

import test_gpu_controller_split as split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,T", [(16384, 1), (16385, 7), (16385, 8), (16385, 12), (16385, 15), (16385, 16), (16385, 32),
                                 (32769, 24), (32769, 31), (32769, 64), (49152, 16), (49153, 24), (49153, 47),
                                 (49153, 48), (49153, 96), (65537, 64)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_lines(n, T, dtype):
    split.test_layouts(n, 3, T, 2, dtype)
