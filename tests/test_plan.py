"""How products are cut and which kernel form multiplies them (srq_plan.hpp): host arithmetic, compiled alone."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_00874_amd", "csrc")
I8, F8, BF16, F16C, F16W = range(5)
P256, P128, P128_G2, P128x192, P64, P64_G2, P64_G4 = range(7)

WRAP = """
#include "srq_plan.hpp"
using namespace srq;
extern "C" void plan(size_t P, size_t Q, size_t R, int pipe, unsigned* o) {
  const Plan pl = plan_for(P, Q, R, pipe);
  const Launch l = choose_launch(pl, P, Q, pipe == PIPE_BF16 ? 2 * R : R, pipe);
  o[0] = pl.nsplit; o[1] = l.form; o[2] = l.nsplit; o[3] = l.k_per_split;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(WRAP)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")],
                   check=True)
    lib = C.CDLL(str(d / "plan.so"))
    lib.plan.argtypes = [C.c_size_t] * 3 + [C.c_int, C.c_void_p]

    def f(P, Q, R, pipe):
        o = (C.c_uint * 4)()
        lib.plan(P, Q, R, pipe, o)
        return dict(planned_slices=o[0], form=o[1], slices=o[2], k_per_split=o[3])
    return f


def test_four_groups_are_for_binary32_sums(plan):
    # the int8 kernel of that form is not built: its sums are exact, two groups do
    forms = {pipe: {plan(P, Q, R, pipe)["form"] for P in (16, 48, 592, 2000, 5104) for Q in (64, 560, 1024)
                    for R in range(16, 12000, 592)} for pipe in range(5)}
    assert P64_G4 not in forms[I8] and P64_G4 not in forms[F8]
    assert all(P64_G4 in forms[pipe] for pipe in (BF16, F16C, F16W))
