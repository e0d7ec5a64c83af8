"""Distinct-voxel slots (csrc/dsa3d_slots.h) against the fp64 oracle, at the sizes where they can
go wrong: the rounds of 16 points and the chunks of 32 and 80 that are numbered together, rows of
four tokens cut by the grid's edge, boxes that overflow inside a tile judged by one token, corners
outside the buffer window, and rows of V that hold infinities.

Tolerances are those of test_gpu_parity: fp32 max-abs 1e-5, bf16 the relative metric 2e-2.
"""
import numpy as np
import pytest

import oracle
import testgen
from tests.util import max_abs, rel_err, say, shape9, to_device, to_host

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_22696_amd as dsa
    dsa.load()
    yield


def check(name, got, ref, bf16):
    e = rel_err(got, ref) if bf16 else max_abs(got, ref)
    say(f"  {name}: {e:.3e}")
    assert e <= (2e-2 if bf16 else 1e-5), (name, e)


def case(name, **kw):
    return testgen.WORKLOADS["tiny_f32"].with_grid(name=name, **kw)


def run(w, host):
    import paper_2607_22696_amd as dsa
    q, k, v, off, dout = host
    bf = w.dtype == "bf16"
    qd, kd, vd, gd = (to_device(a, bf) for a in (q, k, v, dout))
    od = to_device(off, False)
    kern = (w.kt, w.kh, w.kw)
    out, lse = dsa.forward(qd, kd, vd, od, kernel=kern)
    grads = dsa.backward(qd, kd, vd, od, lse, gd, kernel=kern)
    torch.cuda.synchronize()
    return (out, lse) + tuple(grads)


def compare(w, host):
    bf = w.dtype == "bf16"
    q, k, v, off, dout = host
    got = [to_host(t) for t in run(w, host)]
    ref = oracle.forward(shape9(w), w.dtype, q, k, v, off)
    check("out", got[0].reshape(ref[0].shape), ref[0], bf)
    check("lse", got[1].reshape(-1), ref[1], bf)
    for name, g, r in zip(("dq", "dk", "dv", "doff"), got[2:],
                          oracle.backward(shape9(w), w.dtype, q, k, v, off, dout)):
        check(name, g, r, bf)


N05 = testgen.Dist(testgen.NORMAL, 0.0, 0.5)
CASES = [
    # points per query: one under, at and over a round (16), two rounds (32) and five (80)
    case("k335_f32_d32", T=3, H=5, W=9, heads=2, head_dim=32, kt=3, kh=3, kw=5, seed=70),
    case("k1115_f32_d64", T=2, H=3, W=21, heads=1, head_dim=64, kt=1, kh=1, kw=15, seed=71),
    case("k1117_bf16_d64", T=2, H=3, W=21, heads=2, head_dim=64, kt=1, kh=1, kw=17, dtype="bf16",
         seed=72),
    case("k1311_bf16_d128", T=2, H=5, W=18, heads=1, head_dim=128, kt=1, kh=3, kw=11,
         dtype="bf16", seed=73),
    case("k1127_bf16_d128", T=1, H=2, W=30, heads=2, head_dim=128, kt=1, kh=1, kw=27,
         dtype="bf16", seed=74),
    case("k399_bf16_d64", T=3, H=9, W=10, heads=1, head_dim=64, kt=1, kh=9, kw=9, dtype="bf16",
         seed=75, offsets=N05),
    case("k399_f32_d64", T=2, H=8, W=7, heads=1, head_dim=64, kt=1, kh=9, kw=9, seed=76),
    # the last four-token cell of a row holds 1, 2 and 3 tokens; two batch items
    case("w5_bf16_d128", B=2, T=2, H=3, W=5, heads=1, head_dim=128, dtype="bf16", seed=77),
    case("w6_bf16_d64", T=2, H=13, W=6, heads=3, head_dim=64, dtype="bf16", seed=78),
    case("w7_f32_d32", T=2, H=3, W=7, heads=2, head_dim=32, seed=79),
    # a grid beyond one tile per pencil frame, so that tiles keep their full size
    case("tiles_bf16_d64", T=8, H=16, W=24, heads=8, head_dim=64, dtype="bf16", seed=80),
    # 65 heads x 256-byte rows: no buffer window, every row by a global load
    case("no_window_bf16_d128", T=2, H=3, W=5, heads=65, head_dim=128, dtype="bf16", seed=81),
    case("no_window_f32_d64", T=2, H=3, W=5, heads=65, head_dim=64, seed=82),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_parity(w):
    host = list(testgen.gen_inputs(w))
    if host[4] is None:
        host[4] = testgen.gen_tensor(w, testgen.TID_DOUT, w.qkv_shape(), w.dout, True)
    compare(w, host)


@pytest.mark.parametrize("dtype,dim,kernel", [("bf16", 128, (3, 3, 3)), ("bf16", 64, (3, 5, 5)),
                                              ("f32", 64, (3, 3, 3)), ("f32", 32, (3, 7, 7))])
def test_points_that_leave_the_box(dtype, dim, kernel):
    """A tile is judged by its first token; here other tokens of compact tiles reach across the
    whole grid (rounds without shared slots) and a few points lie far outside it."""
    w = case("box", T=20, H=20, W=36, heads=1, head_dim=dim, kt=kernel[0], kh=kernel[1],
             kw=kernel[2], dtype=dtype, seed=83)
    host = list(testgen.gen_inputs(w))
    host[4] = testgen.gen_tensor(w, testgen.TID_DOUT, w.qkv_shape(), w.dout, True)
    off = host[3]
    off[:, :, :, 2::5] = np.sign(off[:, :, :, 2::5]) * (np.abs(off[:, :, :, 2::5]) * 40)
    off[:, :, 1::7, 1::6, :, 3] = 1e4
    compare(w, host)


@pytest.mark.parametrize("dim", [64, 128])
def test_infinite_values_stay_where_they_are(dim):
    """An infinite channel of a V row makes that channel of the queries that sample it infinite
    (or NaN where signs meet), as a plain sum does, and touches no other channel or query."""
    import paper_2607_22696_amd as dsa
    w = case("inf", T=3, H=6, W=10, heads=1, head_dim=dim, dtype="bf16", seed=84)
    q, k, v, off, _ = testgen.gen_inputs(w)
    off = np.full_like(off, 0.25)
    qd, kd, vd = (to_device(a, True) for a in (q, k, v))
    od = to_device(off, False)
    clean = to_host(dsa.forward(qd, kd, vd, od)[0])
    vd[0, 1, 2, 3, 0, 5] = float("inf")
    got = to_host(dsa.forward(qd, kd, vd, od)[0])
    hit = np.zeros(clean.shape, bool)
    # the queries whose 3x3x3 points at +0.25 have voxel (1, 2, 3) among their corners
    hit[0, 0:3, 0:4, 1:5, 0, 5] = True
    assert np.array_equal(got[~hit], clean[~hit])
    assert np.all(np.isposinf(got[hit]))
