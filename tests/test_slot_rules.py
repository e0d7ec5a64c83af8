"""The dispatch rules of the distinct-voxel slots (csrc/slot_rules.h), compiled for the host: the
cases of test_gpu_slots.py take the code they are written for, and the workloads' calls the code that
was measured to be the faster one for them."""
import os
import subprocess

import pytest

import testgen
from tests import test_gpu_slots as slots

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HDR = os.path.join(ROOT, "paper_2607_22696_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "slot_rules.h"
using namespace dsa3d;
int main(int argc, char** argv) {
  const int D = atoi(argv[1]), bf16 = atoi(argv[2]), P = atoi(argv[4]);
  const long rows = atol(argv[3]);
  printf("%d %d %d\n", forward_rounds(D, bf16, rows, P, false), backward_rounds(D, bf16, rows, P),
         forward_rounds(D, bf16, rows, P, true));
}
"""


@pytest.fixture(scope="module")
def rounds(tmp_path_factory):
    d = tmp_path_factory.mktemp("slot_rules")
    src, exe = d / "r.cpp", d / "r"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", HDR, str(src), "-o", str(exe)])

    def ask(w):
        """(forward, backward, predicted-weights forward) rounds of workload w."""
        out = subprocess.check_output([str(exe), str(w.head_dim), str(int(w.dtype == "bf16")),
                                       str(w.queries), str(w.P)], text=True)
        return tuple(map(int, out.split()))
    return ask


def test_the_slot_tests_reach_their_kernels(rounds):
    for w, fwd, bwd in slots.CASES + slots.BOX_CASES + slots.FINITE_CASES + slots.MIXED_CASES:
        assert rounds(w)[:2] == (fwd, bwd), w.name
    for w, fwd in slots.PW_CASES:
        assert rounds(w)[2] == fwd, w.name
    reached = {(w.head_dim, w.dtype, "fwd", f) for w, f, b in slots.CASES} | {
        (w.head_dim, w.dtype, "bwd", b) for w, f, b in slots.CASES}
    for d, t in ((32, "f32"), (64, "f32"), (64, "bf16"), (128, "bf16")):
        assert (d, t, "fwd", 2) in reached and (d, t, "fwd", 5) in reached
    for at in ((32, "f32", "bwd", 5), (64, "f32", "bwd", 5), (128, "bf16", "bwd", 2),
               (128, "bf16", "bwd", 5)):
        assert at in reached


def test_workloads(rounds):
    w = testgen.WORKLOADS
    assert rounds(w["tiny_f32"]) == (2, 0, 2)
    assert rounds(w["fwdbwd_64x34x60"]) == (2, 0, 0)
    assert rounds(w["full_1080p_256f"]) == (2, 2, 2)
    assert rounds(w["paper_3x7x7_64x68x120"]) == (5, 5, 5)
    # few rows; rows of a size that the slots are not built for; few points
    few = w["fwdbwd_64x34x60"].with_grid(name="few", T=4, H=14, W=21, heads=2)
    assert rounds(few) == (0, 0, 0)
    tiny = w["tiny_f32"].with_grid(name="few32", T=3, H=12, W=20)
    assert rounds(tiny) == (0, 0, 0)
    assert rounds(tiny.with_grid(name="few32", kh=5, kw=5)) == (5, 5, 5)
    assert rounds(w["full_1080p_256f"].with_grid(name="f", dtype="f32")) == (0, 0, 0)
    assert rounds(w["full_1080p_256f"].with_grid(name="f", kt=1)) == (0, 0, 0)


def test_the_bench_counts_corner_loads_only_where_a_kernel_gathers(rounds):
    import bench
    for w in testgen.WORKLOADS.values():
        wide = w.offsets.kind == testgen.UNIFORM and w.offsets.b > 4
        fwd, bwd, _ = rounds(w)
        assert bench.loads_every_corner(w, "fwd_kernel") == (wide or fwd == 0), w.name
        for k in ("bwd_vpass_kernel", "bwd_kpass_kernel"):
            assert bench.loads_every_corner(w, k) == (wide or bwd == 0), w.name
