"""The depthwise convolution's streaming path with its frames cut into segments (few bricks, at
least 8 frames), in both dtypes, against the fp64 oracle; the tolerances of test_gpu_dwconv."""
import pytest

from tests.test_gpu_dwconv import _gpu, conv, run_case  # noqa: F401 (the module's GPU check)

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = [
    # two segments of 4 frames, three of a ragged split, a time extent of 1, two batch items
    conv("bf16_T8", 1, 8, 5, 9, 130, (3, 3, 3), "bf16", 60),
    conv("f32_T8", 1, 8, 5, 9, 130, (3, 3, 3), "f32", 61),
    conv("bf16_T13", 1, 13, 4, 8, 64, (3, 3, 1), "bf16", 62),
    conv("f32_T13_B2", 2, 13, 3, 10, 64, (3, 1, 3), "f32", 63),
    conv("f32_T17_1x3x3", 1, 17, 6, 7, 32, (1, 3, 3), "f32", 64),
    # fp32 bricks whose last rows, columns and channels lie outside the grid
    conv("f32_ragged", 1, 3, 9, 17, 258, (3, 3, 3), "f32", 65),
    conv("f32_1x1x1", 1, 2, 3, 5, 6, (1, 1, 1), "f32", 66),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_parity(w):
    run_case(w)
