"""The depthwise convolution's streaming path with its frames cut into segments (few bricks, at
least 8 frames), in both dtypes, against the fp64 oracle; the tolerances of test_gpu_dwconv."""
import numpy as np
import pytest

import testgen
from tests.util import to_device, to_host
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


# W is a multiple of 8: the columns past a strip's end are zeros that meet the filter in every path
INF_CASES = [conv("f32_inf", 1, 8, 6, 16, 4, (3, 3, 3), "f32", 70),
             conv("f32_inf_one_segment", 1, 5, 6, 16, 4, (3, 3, 3), "f32", 71),
             conv("bf16_inf", 1, 8, 8, 16, 4, (3, 3, 3), "bf16", 72)]


@pytest.mark.parametrize("w", INF_CASES, ids=lambda w: w.name)
def test_an_infinite_input_reaches_its_own_taps_only(w):
    """dw of a tap is infinite exactly where dy has a token that meets the infinite x through that
    tap: x at the first and the last frame and row (fp32), and beside a cut of the frames, where the
    next segment reads it as its halo."""
    import paper_2607_22696_amd as dsa
    bf = w.dtype == "bf16"
    x, dy, wt, _ = testgen.gen_conv_inputs(w)
    dyd, wd = to_device(dy, bf), to_device(wt, False)
    base = to_host(dsa.dwconv3d_backward(to_device(x, bf), wd, dyd)[1])
    edges = [(3, 2, 5), (4, 3, 9)]
    if not bf:
        edges += [(0, 2, 5), (w.T - 1, 3, 6), (2, 0, 9), (2, w.H - 1, 10), (0, 0, 4)]
    for t, i, j in edges:
        xd = to_device(x, bf)
        xd[0, t, i, j, 1] = float("inf")
        dw = to_host(dsa.dwconv3d_backward(xd, wd, dyd)[1])
        hit = np.zeros(dw.shape, bool)
        for a in range(3):
            for e in range(3):  # the token that meets (t, i, j) through tap (a, e, f)
                hit[1, a, e] = 0 <= t - a + 1 < w.T and 0 <= i - e + 1 < w.H
        assert np.isinf(dw[hit]).all(), (t, i, j)
        assert np.array_equal(dw[~hit], base[~hit]), (t, i, j)


def test_an_infinite_weight_does_not_meet_the_padding():
    """fp32: rows and frames outside the grid are skipped, not multiplied by zero."""
    import paper_2607_22696_amd as dsa
    w = conv("f32_inf_weight", 1, 9, 6, 16, 4, (3, 3, 1), "f32", 73)
    x, _, wt, bias = testgen.gen_conv_inputs(w)
    xd, bd = to_device(x, False), to_device(bias, False)
    for a, e in ((0, 1), (2, 1), (1, 0), (1, 2), (0, 0)):
        wi = wt.copy()
        wi[1, a, e, 0] = np.inf
        y = to_host(dsa.dwconv3d_forward(xd, to_device(wi, False), bd))
        t, i = np.meshgrid(np.arange(w.T) + a - 1, np.arange(w.H) + e - 1, indexing="ij")
        inside = (t >= 0) & (t < w.T) & (i >= 0) & (i < w.H)
        assert np.isfinite(y[0][..., [0, 2, 3]]).all()
        assert np.array_equal(np.isinf(y[0, ..., 1]), np.repeat(inside[..., None], w.W, 2)), (a, e)
        assert np.isfinite(y[0, ..., 1][~inside]).all()
