"""Distinct-voxel slots (csrc/dsa3d_slots.h) against the fp64 oracle, at the sizes where they can
go wrong: the rounds of 16 points and the chunks of 32 and 80 that are numbered together, rows of
four tokens cut by the grid's edge, queries whose points leave a wave's box or need more slots than
there are, calm and wide tokens side by side, corners outside the buffer window, rows that hold
infinities, and coefficients and values of very different size.

Tolerances are those of test_gpu_parity: fp32 max-abs 1e-5, bf16 the relative metric 2e-2.
"""
import numpy as np
import pytest

import oracle
import testgen
from tests.util import max_abs, rel_err, reorder_bound, say, shape9, to_device, to_host

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

# (case, rounds that the forward and the backward number together, 0: every tile gathers).  The
# rounds are asserted without a GPU by test_slot_rules.py, so that a change of the dispatch cannot
# turn these into tests of the gathering code.
CASES = [
    # points per query: under, at and over a round (16), two rounds (32) and five (80)
    (case("k335_f32_d32", T=3, H=5, W=9, heads=2, head_dim=32, kt=3, kh=3, kw=5, seed=70), 5, 5),
    (case("k1115_f32_d64", T=2, H=3, W=21, heads=1, head_dim=64, kt=1, kh=1, kw=15, seed=71), 0, 0),
    (case("k1117_bf16_d64", T=2, H=21, W=21, heads=20, head_dim=64, kt=1, kh=1, kw=17,
          dtype="bf16", seed=72), 2, 0),
    (case("k1311_bf16_d128", T=2, H=5, W=18, heads=1, head_dim=128, kt=1, kh=3, kw=11,
          dtype="bf16", seed=73), 5, 5),
    (case("k1127_bf16_d128", T=2, H=21, W=30, heads=14, head_dim=128, kt=1, kh=1, kw=27,
          dtype="bf16", seed=74), 2, 2),
    (case("k399_bf16_d64", T=3, H=9, W=10, heads=61, head_dim=64, kt=1, kh=9, kw=9, dtype="bf16",
          seed=75, offsets=N05), 5, 0),
    (case("k399_f32_d64", T=3, H=8, W=7, heads=98, head_dim=64, kt=1, kh=9, kw=9, seed=76), 5, 5),
    (case("k377_bf16_d128", T=3, H=8, W=11, heads=2, head_dim=128, kt=3, kh=7, kw=7, dtype="bf16",
          seed=85), 5, 5),
    (case("k377_f32_d32", T=3, H=8, W=11, heads=2, head_dim=32, kt=3, kh=7, kw=7, seed=86), 5, 5),
    # four chunks that start at any point
    (case("k579_bf16_d128", T=5, H=7, W=9, heads=2, head_dim=128, kt=5, kh=7, kw=9, dtype="bf16",
          seed=96, offsets=N05), 5, 5),
    # an ordinary training step's kernel
    (case("k333_bf16_d128", T=8, H=12, W=24, heads=8, head_dim=128, dtype="bf16", seed=87), 2, 2),
    (case("k355_f32_d64", T=6, H=12, W=24, heads=10, head_dim=64, kt=3, kh=5, kw=5, seed=88), 5, 5),
    (case("k333_f32_d64", T=8, H=12, W=24, heads=8, head_dim=64, seed=89), 2, 0),
    # the last four-token cell of a row holds 1, 2 and 3 tokens; two batch items
    (case("w5_bf16_d128", B=2, T=10, H=9, W=5, heads=20, head_dim=128, dtype="bf16", seed=77), 2, 2),
    (case("w6_bf16_d64", T=7, H=13, W=6, heads=31, head_dim=64, dtype="bf16", seed=78), 2, 0),
    (case("w7_f32_d32", T=2, H=3, W=7, heads=2, head_dim=32, seed=79), 2, 0),
    # a grid beyond one tile per pencil frame, so that tiles keep their full size
    (case("tiles_bf16_d64", T=8, H=16, W=24, heads=8, head_dim=64, dtype="bf16", seed=80), 2, 0),
    # 65 heads x 256-byte rows: no buffer window, every row by a global load
    (case("no_window_bf16_d128", T=4, H=9, W=8, heads=65, head_dim=128, dtype="bf16", seed=81), 2, 2),
    (case("no_window_f32_d64", T=4, H=9, W=8, heads=65, head_dim=64, kt=3, kh=3, kw=5, seed=82),
     5, 5),
]


@pytest.mark.parametrize("w", [c[0] for c in CASES], ids=lambda w: w.name)
def test_parity(w):
    host = list(testgen.gen_inputs(w))
    if host[4] is None:
        host[4] = testgen.gen_tensor(w, testgen.TID_DOUT, w.qkv_shape(), w.dout, True)
    compare(w, host)


def pw_case(name, **kw):
    return testgen.PW_WORKLOADS["pw_64x34x60"].with_grid(name=name, offsets=N05, **kw)


# (case of the predicted-weights variant, its forward's rounds)
PW_CASES = [
    (pw_case("pw_k333_bf16_d128", T=8, H=12, W=24, heads=8, head_dim=128, seed=90), 2),
    (pw_case("pw_k377_bf16_d128", T=3, H=8, W=11, heads=2, head_dim=128, kh=7, kw=7, seed=91), 5),
    (pw_case("pw_k355_bf16_d64", T=6, H=12, W=24, heads=10, kh=5, kw=5, seed=92), 5),
    (pw_case("pw_k333_f32_d32", T=3, H=7, W=10, heads=2, head_dim=32, dtype="f32", seed=93), 2),
    (pw_case("pw_k335_f32_d64", T=6, H=12, W=24, heads=10, kw=5, dtype="f32", seed=94), 5),
]


@pytest.mark.parametrize("w", [c[0] for c in PW_CASES], ids=lambda w: w.name)
def test_predicted_weights_parity(w):
    """Some logits are -inf (weight 0), up to a row's first 20 points."""
    import paper_2607_22696_amd as dsa
    bf = w.dtype == "bf16"
    logits, v, off, dout = testgen.gen_pw_inputs(w)
    lead = np.arange(logits[..., 0].size).reshape(logits.shape[:-1]) % 21
    for p in range(20):
        logits[..., p][lead > p] = -np.inf
    ld, od = to_device(logits, False), to_device(off, False)
    vd, gd = to_device(v, bf), to_device(dout, bf)
    kern = (w.kt, w.kh, w.kw)
    out, lse = dsa.pw_forward(ld, vd, od, kernel=kern)
    grads = dsa.pw_backward(ld, vd, od, lse, gd, kernel=kern)
    torch.cuda.synchronize()
    ref = oracle.pw_forward(shape9(w), w.dtype, logits, v, off)
    check("out", to_host(out).reshape(ref[0].shape), ref[0], bf)
    check("lse", to_host(lse).reshape(-1), ref[1], bf)
    rdl, rdv, rdo = oracle.pw_backward(shape9(w), w.dtype, logits, v, off, dout)
    for name, g, r in zip(("dlogits", "dv", "doff"), grads, (rdl, rdv, rdo)):
        check(name, to_host(g), r, bf)


def box_case(dtype, dim, kernel):
    return case("box", T=20, H=20, W=36, heads=2, head_dim=dim, kt=kernel[0], kh=kernel[1],
                kw=kernel[2], dtype=dtype, seed=83)


BOX_CASES = [(box_case("bf16", 128, (3, 3, 3)), 2, 2), (box_case("bf16", 64, (3, 5, 5)), 5, 0),
             (box_case("f32", 64, (3, 3, 3)), 2, 0), (box_case("f32", 64, (3, 5, 5)), 5, 5),
             (box_case("f32", 32, (3, 7, 7)), 5, 5)]


@pytest.mark.parametrize("w", [c[0] for c in BOX_CASES],
                         ids=lambda w: f"{w.dtype}-{w.head_dim}-{w.kt}x{w.kh}x{w.kw}")
def test_points_that_leave_the_box(w):
    """Queries whose points lie close together each, but apart from their neighbours': further than
    a wave's box reaches (rounds without shared slots), and within it but with more voxels than
    there are slots (fewer rounds at a time).  A few points lie far outside the grid."""
    host = list(testgen.gen_inputs(w))
    host[4] = testgen.gen_tensor(w, testgen.TID_DOUT, w.qkv_shape(), w.dout, True)
    off = host[3]
    off[:, :, :10, 2::5, :, :, 0] += np.where(np.arange(2, w.W, 5) < 18, 25.0, -25.0)[:, None, None]
    off[:, :, 10:, 1::2, :, :, 1] -= 8.0
    off[:, :, 1::7, 1::6, :, 3] = 1e4
    compare(w, host)


MIXED_CASES = [(case("mixed", T=6, H=11, W=20, heads=14, head_dim=d, kt=k[0], kh=k[1], kw=k[2],
                     dtype=t, seed=95), f, b)
               for t, d, k, f, b in (("bf16", 128, (3, 3, 3), 2, 2), ("bf16", 64, (3, 5, 5), 5, 0),
                                     ("f32", 64, (3, 5, 5), 5, 5), ("f32", 32, (3, 7, 7), 5, 5),
                                     ("bf16", 128, (3, 7, 7), 5, 5))]


@pytest.mark.parametrize("w", [c[0] for c in MIXED_CASES],
                         ids=lambda w: f"{w.dtype}-{w.head_dim}-{w.kt}x{w.kh}x{w.kw}")
def test_calm_and_wide_tokens_side_by_side(w):
    """Waves of one workgroup that go different ways: runs of calm and of wide tokens of every
    length, and single points of calm tokens that lie far away (seen or not by the samples)."""
    host = list(testgen.gen_inputs(w))
    host[4] = testgen.gen_tensor(w, testgen.TID_DOUT, w.qkv_shape(), w.dout, True)
    off = host[3]
    rng = np.random.default_rng(w.seed)
    token = np.cumsum(rng.random(off.shape[:4]) < 0.3, axis=3) % 2  # runs along x
    off[...] = np.where(token[..., None, None, None] == 0, off, off * 16)
    far = rng.random(off.shape[:6]) < 0.002
    off[far] += 11.0
    compare(w, host)


def test_window_of_one_frame():
    """Frames of 2.5 GB: the buffer window holds one of the two frames, and every row of the other
    one is a global load.  The same heads on their own (a window of both frames) take the same sums
    in the same order."""
    import paper_2607_22696_amd as dsa
    T, H, W, heads, few, D, kernel = 2, 400, 400, 60, 2, 128, (3, 1, 7)
    gen = torch.Generator(device="cuda").manual_seed(7)

    def randn(*shape, dtype=torch.bfloat16):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)

    q, k, v, dout = (randn(1, T, H, W, heads, D) for _ in range(4))
    off = randn(1, T, H, W, heads, 21, 3, dtype=torch.float32).mul_(0.5)
    out, lse = dsa.forward(q, k, v, off, kernel=kernel)
    dq, dk, dv, doff = dsa.backward(q, k, v, off, lse, dout, kernel=kernel)
    part = [x[:, :, :, :, :few].contiguous() for x in (q, k, v, off, dout)]
    out2, lse2 = dsa.forward(*part[:4], kernel=kernel)
    dq2, dk2, dv2, doff2 = dsa.backward(*part[:4], lse2, part[4], kernel=kernel)
    for name, a, b in (("out", out, out2), ("lse", lse, lse2), ("dq", dq, dq2),
                       ("doff", doff, doff2)):
        assert torch.equal(a[:, :, :, :, :few], b), name
    for name, a, b in (("dk", dk, dk2), ("dv", dv, dv2)):  # the order of a voxel's entries differs
        d = (a[:, :, :, :, :few] - b).abs().max().item()
        say(f"  {name}: {d:.3e}")
        assert d <= reorder_bound(21, b.abs().max().item()), name


# Rows with an infinity: a bf16 grid of 16,384 rows (FINITE_CASES, asserted to take the slots), every
# offset +0.25, so that voxel (t, i, j) is a corner of the points of the queries (t-2 .. t+1, ...).
def finite_case(dim, kernel, dtype="bf16"):
    return case("finite", T=4, H=16, W=32, heads=8, head_dim=dim, kt=kernel[0], kh=kernel[1],
                kw=kernel[2], dtype=dtype, seed=84)


FINITE_CASES = [(finite_case(128, (3, 3, 3)), 2, 2), (finite_case(128, (3, 5, 5)), 5, 5),
                (finite_case(64, (3, 3, 3)), 2, 0), (finite_case(64, (3, 5, 5)), 5, 0),
                (finite_case(32, (3, 5, 5), "f32"), 5, 5)]
VOXEL = (1, 8, 13)


def finite_id(w):
    return f"{w.dtype}-{w.head_dim}-{w.kt}x{w.kh}x{w.kw}"


def finite_inputs(w, offset=0.25):
    bf = w.dtype == "bf16"
    q, k, v, off, _ = testgen.gen_inputs(w)
    dout = testgen.gen_tensor(w, testgen.TID_DOUT, w.qkv_shape(), w.dout, True)
    off = np.full_like(off, offset)
    return tuple(to_device(a, bf) for a in (q, k, v)) + (to_device(off, False), to_device(dout, bf))


def samplers(w):
    """Queries (head 0) that have VOXEL among the corners of their points at +0.25."""
    hit = np.zeros((w.B, w.T, w.H, w.W, w.heads), bool)
    at = [slice(max(c - r - 1, 0), c + r + 1) for c, r in
          zip(VOXEL, ((w.kt - 1) // 2, (w.kh - 1) // 2, (w.kw - 1) // 2))]
    hit[0, at[0], at[1], at[2], 0] = True
    return hit


def close(w, got, want):
    """Sums taken again in another order: the tolerances of the file."""
    check("elsewhere", got, want, w.dtype == "bf16")


@pytest.mark.parametrize("w", [c[0] for c in FINITE_CASES], ids=finite_id)
def test_an_infinite_key_reaches_its_own_queries_only(w):
    import paper_2607_22696_amd as dsa
    q, k, v, off, dout = finite_inputs(w)
    kern = (w.kt, w.kh, w.kw)
    hit = samplers(w)
    out0, lse0 = (to_host(x) for x in dsa.forward(q, k, v, off, kernel=kern))
    good = dsa.forward(q, k, v, off, kernel=kern)[1]
    dq0, _, _, do0 = dsa.backward(q, k, v, off, good, dout, kernel=kern)
    k[(0,) + VOXEL + (0, 5)] = float("inf")
    out, lse = dsa.forward(q, k, v, off, kernel=kern)
    dq, _, _, do = dsa.backward(q, k, v, off, lse, dout, kernel=kern)
    out, lse = to_host(out), to_host(lse)
    for name, got, want in (("out", out, out0), ("lse", lse, lse0), ("dq", to_host(dq), to_host(dq0)),
                            ("doff", to_host(do), to_host(do0))):
        assert np.isfinite(got[~hit]).all(), name
        close(w, got[~hit], want[~hit])


@pytest.mark.parametrize("w", [c[0] for c in FINITE_CASES], ids=finite_id)
@pytest.mark.parametrize("value,offset", [(float("inf"), 0.25), (float("nan"), 0.25),
                                          (float("inf"), 2.0 ** -12), (float("inf"), 0.0)])
def test_an_infinite_value_reaches_its_own_queries_only(w, value, offset):
    """An infinite channel of a V row makes that channel of the queries that sample it infinite, as
    a plain sum does, however small its weight is (NaN where the weight is 0), and touches no other
    channel or query; in the backward every gradient of those queries is lost, and no other."""
    import paper_2607_22696_amd as dsa
    q, k, v, off, dout = finite_inputs(w, offset)
    kern = (w.kt, w.kh, w.kw)
    hit = samplers(w)
    out0, lse = dsa.forward(q, k, v, off, kernel=kern)
    dq0, _, _, do0 = dsa.backward(q, k, v, off, lse, dout, kernel=kern)
    v[(0,) + VOXEL + (0, 5)] = value
    out = to_host(dsa.forward(q, k, v, off, kernel=kern)[0])
    dq, _, _, do = (to_host(x) for x in dsa.backward(q, k, v, off, lse, dout, kernel=kern))
    channel = np.zeros(out.shape, bool)
    channel[..., 5] = hit
    if offset == 0.0:
        # NaN from corners of weight 0 (and inf - inf never: the weights are not negative)
        assert not np.isfinite(out[channel]).any() and np.isnan(out[channel]).any()
    else:
        assert np.array_equal(out[channel], np.full(channel.sum(), value, np.float32),
                              equal_nan=True)
    assert np.isfinite(out[~channel]).all()
    close(w, out[~channel], to_host(out0)[~channel])
    assert not np.isfinite(dq[hit]).any()
    for name, got, want in (("dq", dq, to_host(dq0)), ("doff", do, to_host(do0))):
        assert np.isfinite(got[~hit]).all(), name
        close(w, got[~hit], want[~hit])


@pytest.mark.parametrize("w", [c[0] for c in FINITE_CASES], ids=finite_id)
def test_a_weight_of_zero_on_the_largest_value_adds_nothing(w):
    """Offsets of 0: the queries that have a voxel as an upper corner only, with weight 0, do not see
    a value of 3e38 there."""
    import paper_2607_22696_amd as dsa
    q, k, v, off, dout = finite_inputs(w, 0.0)
    kern = (w.kt, w.kh, w.kw)
    out0, lse = dsa.forward(q, k, v, off, kernel=kern)
    v[(0,) + VOXEL + (0, 5)] = 3e38
    out = to_host(dsa.forward(q, k, v, off, kernel=kern)[0])
    sampled = np.zeros(samplers(w).shape, bool)
    at = [slice(max(c - r, 0), c + r + 1) for c, r in
          zip(VOXEL, ((w.kt - 1) // 2, (w.kh - 1) // 2, (w.kw - 1) // 2))]
    sampled[0, at[0], at[1], at[2], 0] = True
    assert (samplers(w) & ~sampled).any()
    assert np.array_equal(out[~sampled], to_host(out0)[~sampled])
    assert (np.abs(out[sampled][:, 5]) > 1e30).all()


@pytest.mark.parametrize("w", [c[0] for c in FINITE_CASES], ids=finite_id)
def test_powers_of_two_pass_through(w):
    """Values near 1e30 and gradients near 1e-21: every sum is linear in V, K and dout, and scaling
    by a power of two changes no bit of it while nothing overflows."""
    import paper_2607_22696_amd as dsa
    q, k, v, off, dout = finite_inputs(w)
    kern, scale = (w.kt, w.kh, w.kw), 2.0 ** -3
    up, down = 2.0 ** 100, 2.0 ** -70

    def both(k, v, dout, scale):
        out, lse = dsa.forward(q, k, v, off, kernel=kern, scale=scale)
        dq, _, _, do = dsa.backward(q, k, v, off, lse, dout, kernel=kern, scale=scale)
        return out, lse, dq, do

    out, lse, dq, do = both(k, v, dout, scale)
    # V 2^100 times as large and dout 2^-70 times: da, and with it dq and d_offsets, 2^30 times
    o, s, g, d = both(k, v * up, dout * down, scale)
    assert torch.equal(o, out * up) and torch.equal(s, lse)
    assert torch.equal(g, dq * (up * down)) and torch.equal(d, do * (up * down))
    o, s, g, d = both(k, v, dout * down, scale)
    assert torch.equal(g, dq * down) and torch.equal(d, do * down)
    # K 2^100 times as large and the scale 2^-100 times
    o, s, g, d = both(k * up, v, dout, scale / up)
    assert torch.equal(o, out) and torch.equal(s, lse)
    assert torch.equal(g, dq) and torch.equal(d, do)


@pytest.mark.parametrize("w,rounds", [(c[0], c[2]) for c in FINITE_CASES],
                         ids=lambda x: finite_id(x) if hasattr(x, "dtype") else str(x))
def test_a_small_weight_on_a_large_value_counts(w, rounds):
    """Offsets of 2^-10: the upper corner of all three axes has weight 2^-30, about 2^-35 of the
    row's sum with its softmax weight.  On a value of 2^36 it adds about 2 to a sum of size 1.
    The coefficients' products and sums are fp32 (2^-24 each); the bf16 output adds 2^-9."""
    import paper_2607_22696_amd as dsa
    bf = w.dtype == "bf16"
    q, k, v, off, _ = testgen.gen_inputs(w)
    dout = testgen.gen_tensor(w, testgen.TID_DOUT, w.qkv_shape(), w.dout, True)
    off = np.full_like(off, 2.0 ** -10)
    voxel = (0, 3, 8, 13, 0, 5)
    big = np.float32(2.0 ** 36)
    value = np.uint16(big.view(np.uint32) >> 16) if bf else big
    kern = (w.kt, w.kh, w.kw)
    qd, od, gd = to_device(q, bf), to_device(off, False), to_device(dout, bf)

    def check_near(name, got, ref, rel, small):
        got, ref = got.astype(np.float64)[..., 5], ref.reshape(got.shape)[..., 5]
        e = np.abs(got - ref) / (rel * np.abs(ref) + small)
        say(f"  {name}: {e.max():.3f} of the bound")
        assert e.max() <= 1.0, name

    v1 = v.copy()
    v1[voxel] = value
    out, lse = dsa.forward(qd, to_device(k, bf), to_device(v1, bf), od, kernel=kern)
    ref = oracle.forward(shape9(w), w.dtype, q, k, v1, off)[0]
    check_near("out", to_host(out), ref, 2.0 ** -8 if bf else 1e-5, 1e-5)
    if rounds == 0:  # the gathering dq subtracts Delta sum alpha k at the end: it cancels here
        return
    # K: channel 5 of q is 0, so that the logits stay as they are
    q0, k1 = q.copy(), k.copy()
    q0[..., 5] = 0
    k1[voxel] = value
    qd, kd, vd = to_device(q0, bf), to_device(k1, bf), to_device(v, bf)
    out, lse = dsa.forward(qd, kd, vd, od, kernel=kern)
    dq = dsa.backward(qd, kd, vd, od, lse, gd, kernel=kern)[0]
    ref = oracle.backward(shape9(w), w.dtype, q0, k1, v, off, dout)[0]
    check_near("dq", to_host(dq), ref, 2e-4, 2e-4)
