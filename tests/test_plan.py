"""How products are cut and which kernel form multiplies them (srq_plan.hpp): host arithmetic, compiled alone."""
import ctypes as C
import os
import subprocess

import pytest

from gpu_util import GROUP_SHAPES, LARGE_MFMA_SHAPES, PAIR_SHAPES, RIDE_SHAPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_00874_amd", "csrc")
I8, F8, BF16, F16C, F16W = range(5)
P256, P128, P128_S2, P128_G2, P128x192, P64_G2, P64_G4 = range(7)

WRAP = """
#include <chrono>
#include "srq_plan.hpp"
using namespace srq;
extern "C" void plan(size_t P, size_t Q, size_t R, int pipe, int leaves, unsigned rides, unsigned* o) {
  const Plan pl = plan_for(P, Q, R, pipe);
  const Launch l = choose_launch(pl, P, Q, pipe == PIPE_BF16 ? 2 * R : R, pipe, leaves, rides);
  o[0] = pl.nsplit; o[1] = l.form; o[2] = l.nsplit; o[3] = l.k_per_split; o[4] = l.ring;
}
extern "C" void pair(size_t M, size_t N, size_t K, int pipe, unsigned* o) {
  const Pair p = choose_pair(M, N, K, pipe, plan_for(N, K, M, pipe), plan_for(M, K, N, pipe));
  const unsigned v[] = {(unsigned)p.form, p.weight_first, (unsigned)p.w.waves, p.w.nsplit, p.w.k_per_split, (unsigned)p.d.waves, p.d.nsplit, p.d.k_per_split};
  for (int i = 0; i < 8; ++i) o[i] = v[i];
}
extern "C" void large_mfma(size_t M, size_t N, size_t K, int pipe, unsigned* o) {
  const Plan w = plan_for(N, K, M, pipe), d = plan_for(M, K, N, pipe);
  const Pair p = choose_pair(M, N, K, pipe, w, d);
  const Launch lw = choose_launch(w, N, K, M, pipe, true, 0), ld = choose_launch(d, M, K, N, pipe, false, 0);
  const auto tiles = [](const Launch& l, size_t P, size_t Q) { return l.form == FORM_128x192 ? (P + 127) / 128 * ((Q + 191) / 192) * l.nsplit : 0; };
  const size_t v[] = {p.form, p.w.waves != p.d.waves, p.w.large_mfma, p.d.large_mfma, large_mfma_of_gradient(w, lw, true, N, K, M, pipe),
                      large_mfma_of_gradient(d, ld, false, M, K, N, pipe), tiles(lw, N, K), tiles(ld, M, K)};
  for (int i = 0; i < 8; ++i) o[i] = (unsigned)v[i];
}
// nanoseconds of the plans of a backward call, and of what chooses between one launch and two beside them
extern "C" void host_time(size_t M, size_t N, size_t K, int pipe, double* o) {
  const auto now = [] { return std::chrono::duration<double, std::nano>(std::chrono::steady_clock::now().time_since_epoch()).count(); };
  unsigned sum = 0;
  o[0] = o[1] = 1e30;
  for (int r = 0; r < 20; ++r) {
    const double start = now();
    Plan w, d;
    for (int i = 0; i < 100; ++i) {
      w = plan_for(N + i % 2 * 16, K, M, pipe), d = plan_for(M, K, N + i % 2 * 16, pipe);
      sum += w.nsplit + d.nsplit;
    }
    const double between = now();
    for (int i = 0; i < 100; ++i) sum += choose_pair(M, N + i % 2 * 16, K, pipe, w, d).form;
    const double end = now();
    if (between - start < o[0]) o[0] = between - start;
    if (end - between < o[1]) o[1] = end - between;
  }
  o[0] /= 100, o[1] /= 100, o[2] = sum;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(WRAP)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")],
                   check=True)
    lib = C.CDLL(str(d / "plan.so"))
    lib.plan.argtypes = [C.c_size_t] * 3 + [C.c_int, C.c_int, C.c_uint, C.c_void_p]
    lib.pair.argtypes = lib.large_mfma.argtypes = lib.host_time.argtypes = [C.c_size_t] * 3 + [C.c_int, C.c_void_p]

    def pair(M, N, K, pipe):
        o = (C.c_uint * 8)()
        lib.pair(M, N, K, pipe, o)
        return dict(zip(("form", "weight_first", "waves_w", "slices_w", "k_w", "waves_d", "slices_d", "k_d"), o))

    def f(P, Q, R, pipe, leaves=False, rides=0):
        o = (C.c_uint * 5)()
        lib.plan(P, Q, R, pipe, leaves, rides, o)
        return dict(planned_slices=o[0], form=o[1], slices=o[2], k_per_split=o[3], ring=o[4])
    f.pair, f.large_mfma, f.host_time = pair, lib.large_mfma, lib.host_time
    return f


def test_pairs_keep_the_sums_of_the_launches_they_replace(plan):
    # over random calls: a pair has the slices of the separate launches, and in binary32 as many partial sums in them; no pair for
    # bfloat16 operands or 256 x 256 tiles
    import random
    rng = random.Random(5)
    taken = 0
    for _ in range(4000):
        M, N, K = (16 * int(2 ** rng.uniform(0, 9)) for _ in range(3))
        for pipe in range(5):
            p = plan.pair(M, N, K, pipe)
            w, d = plan(N, K, M, pipe, True), plan(M, K, N, pipe)
            if pipe == BF16 or P256 in (w["form"], d["form"]):
                assert p["form"] == 0
            if p["form"] == 0:
                continue
            taken += 1
            for which, l in (("w", w), ("d", d)):
                assert (p["slices_" + which], p["k_" + which]) == (l["slices"], l["k_per_split"])
                if pipe != I8:
                    parts = 4 if l["form"] == P64_G4 else 2 if l["form"] in (P128_S2, P128_G2, P64_G2) else 1
                    assert p["waves_" + which] == parts
                assert p["waves_" + which] in ((1, 2) if p["form"] == 1 else (2, 4))
    assert taken > 4000


# a backward call makes its two plans once, and what is added to them is less than a microsecond (it was the time of two more plans)
@pytest.mark.parametrize("M,N,K,pipe", [(1008, 3072, 768, F16C), (4096, 2048, 2048, I8), (16384, 256, 256, F16W), (65536, 256, 512, F16W)])
def test_choosing_a_pair_costs_little_host_time(plan, M, N, K, pipe):
    ns = (C.c_double * 3)()
    plan.host_time(M, N, K, pipe, ns)
    print("ns of the plans and of the choice", M, N, K, pipe, list(ns)[:2])
    assert ns[1] < 1000


# integer products whose results are written for longer than they are multiplied (us of both in launches of their own, and in one launch
# of 64 x 64 and of 128 x 128 tiles, where these can be taken)
@pytest.mark.parametrize("M,N,K,apart,small,large", [
    (8192, 16, 4096, 42.6, 47.3, None), (16, 8192, 4096, 39.0, 44.0, None), (5648, 96, 10688, 69.5, 86.0, None),
    (96, 58384, 1104, 82.9, 96.4, None), (128, 10240, 3392, 47.7, 53.6, None), (80, 7600, 4000, 41.0, 44.3, None),
    (32768, 16, 1024, 64.2, 43.3, None), (99808, 16, 256, 86.7, 47.0, None), (65536, 32, 512, 94.5, 52.9, None),
    (672, 16, 61424, 61.0, 49.8, None), (4096, 64, 8192, 44.1, 37.2, None), (48, 1328, 20560, 38.9, 31.6, None),
    (80, 768, 22816, 26.4, 22.5, None), (12912, 16, 1088, 28.1, 22.3, None),
    (2496, 192, 10192, 44.0, 43.4, 33.4), (240, 2928, 6736, 40.5, 37.2, 30.6), (192, 1360, 10512, 27.5, 25.4, 20.8),
    (192, 256, 114336, 58.9, 67.5, 54.5), (160, 1984, 3584, 15.5, 12.7, 16.7), (1024, 3632, 1088, 30.1, 22.6, 29.6)])
def test_pairs_of_large_results_take_the_tiles_that_write_them_faster(plan, M, N, K, apart, small, large):
    times = {0: apart, 1: large, 2: small}
    form = plan.pair(M, N, K, I8)["form"]
    assert times[form] == min(t for t in times.values() if t)


def test_pair_shapes_cover_the_forms(plan):
    seen = {pipe: {(p["form"], p["waves_w"], p["waves_d"], p["weight_first"], p["slices_w"] > 1, p["slices_d"] > 1)
                   for p in (plan.pair(*s, pipe) for s in PAIR_SHAPES)} for pipe in (I8, F8, F16C)}
    for pipe in seen:
        assert {f[0] for f in seen[pipe]} >= {1, 2} and {f[3] for f in seen[pipe]} == {0, 1}
        assert any(f[4] for f in seen[pipe]) and any(f[5] for f in seen[pipe])
    assert {f[1:3] for f in seen[F16C] if f[0] == 1} == {(1, 1), (1, 2), (2, 1), (2, 2)}
    assert {f[1:3] for f in seen[F16C] if f[0] == 2} == {(2, 2), (2, 4), (4, 2), (4, 4)}


def test_four_groups_are_for_binary32_sums(plan):
    # the int8 kernel of that form is not built: its sums are exact, two groups do
    forms = {pipe: {plan(P, Q, R, pipe)["form"] for P in (16, 48, 592, 2000, 5104) for Q in (64, 560, 1024)
                    for R in range(16, 12000, 592)} for pipe in range(5)}
    assert P64_G4 not in forms[I8] and P64_G4 not in forms[F8]
    assert all(P64_G4 in forms[pipe] for pipe in (BF16, F16C, F16W))


LAUNCH = 1.5  # us that the rule counts for the launch that sums slices

# products that one pass of 64 x 64 tiles makes slower (us as planned, in one pass, each repeated in a graph), and others that it makes faster
@pytest.mark.parametrize("P,Q,R,pipe,planned,once", [
    (4496, 96, 7456, I8, 16.8, 19.8), (576, 2048, 6000, I8, 22.2, 29.9), (64, 6000, 10192, I8, 21.7, 26.6),
    (192, 160, 2240, F16C, 7.6, 8.2), (3776, 32, 2768, F16C, 8.4, 9.5), (256, 256, 2048, F16C, 7.3, 7.7),
    (4432, 208, 2720, BF16, 18.6, 21.7), (1152, 1616, 11408, F8, 46.4, 55.4), (1008, 224, 10240, I8, 14.7, 19.0),
    (640, 992, 7168, I8, 17.2, 13.4), (1008, 768, 3072, I8, 13.7, 7.1), (1008, 768, 3072, F16C, 15.8, 10.2),
    (512, 1024, 4096, F16C, 15.6, 12.2), (16, 5632, 5632, I8, 11.4, 9.8), (32, 5632, 2048, I8, 6.5, 5.4),
    (1024, 2048, 2048, F16C, 17.4, 12.4), (1024, 2048, 2048, BF16, 21.8, 15.3), (256, 6528, 96, F8, 5.5, 4.6),
    # with the quantizers before it
    (48, 1072, 1664, BF16, 19.2, 20.2), (176, 208, 2928, I8, 19.5, 20.6), (32, 320, 2816, I8, 11.54, 11.57), (240, 240, 3984, I8, 19.8, 27.2),
    (144, 1440, 2448, I8, 15.1, 14.4), (496, 304, 6864, I8, 17.3, 32.3), (48, 2848, 4592, I8, 20.8, 23.7), (144, 1648, 4816, F16C, 23.8, 27.9),
    (32, 2496, 2112, I8, 14.6, 13.1), (80, 4320, 2512, I8, 24.0, 19.5), (96, 544, 2112, BF16, 13.3, 15.8), (352, 272, 6704, I8, 15.3, 24.4),
    (288, 384, 3600, I8, 15.1, 19.7), (64, 80, 8176, I8, 13.6, 24.2), (848, 320, 3408, F16C, 17.2, 21.8)])
def test_one_pass_only_where_it_is_faster(plan, P, Q, R, pipe, planned, once):
    p = plan(P, Q, R, pipe)
    sliced = p["planned_slices"] > 1
    assert (p["form"] in (P64_G2, P64_G4) and p["slices"] == 1) == (once < planned + sliced * LAUNCH)


# the ring of 64 x 64 tiles as planned, with a CU each (us of quantizer and product with three stages, with four)
@pytest.mark.parametrize("P,Q,R,pipe,three,four", [
    (128, 1136, 992, I8, 9.48, 9.18), (128, 1760, 1280, I8, 10.49, 10.25), (16, 80, 1296, I8, 9.11, 8.39),
    (160, 224, 144, I8, 6.99, 7.07), (192, 128, 144, I8, 6.96, 7.10), (192, 1040, 160, BF16, 7.56, 7.60),
    (16, 2720, 304, F16C, 7.86, 7.95), (288, 96, 384, F16C, 8.24, 8.37)])
def test_ring_of_small_tiles(plan, P, Q, R, pipe, three, four):
    p = plan(P, Q, R, pipe)
    assert p["form"] == P64_G2 and p["ring"] == (3 if three < four else 4)


# weight gradients whose slice sum runs beside the next launch: N x K, contraction M (us of both products of the backward call with
# the weight gradient in slices, in one pass)
@pytest.mark.parametrize("M,N,K,pipe,sliced,once", [
    (1088, 208, 336, BF16, 7.9, 8.9), (976, 208, 560, BF16, 8.0, 8.9), (1808, 528, 256, F16W, 9.9, 12.2),
    (1376, 624, 256, F16W, 9.3, 10.4), (2048, 192, 352, F16C, 9.7, 11.8), (2432, 304, 288, F16C, 10.5, 13.0),
    (3968, 128, 960, I8, 11.2, 13.5), (5824, 960, 1216, I8, 34.0, 39.3), (4240, 7360, 224, F16C, 45.3, 50.0),
    (5776, 2544, 736, F16W, 57.4, 63.7),
    (1744, 1872, 384, F16W, 18.3, 15.9), (2432, 1440, 384, F16W, 19.0, 16.4), (2736, 432, 1312, F16C, 22.1, 17.8),
    (3888, 160, 2768, I8, 25.9, 21.6), (1520, 1216, 1104, F16W, 22.6, 19.0)])
def test_one_pass_where_the_slice_sum_is_left_to_a_later_launch(plan, M, N, K, pipe, sliced, once):
    assert (plan(N, K, M, pipe, True)["slices"] == 1) == (once < sliced)


LDS_OF_A_CU = 160 << 10
QUANTIZER_LDS = 64 * (128 + 2) * 2   # a workgroup of the kernel that writes transposed operands


@pytest.mark.parametrize("pipe", range(5))
def test_groups_of_waves_leave_lds_for_quantizers_of_another_stream(plan, pipe):
    # what srq.h tells callers of the phase entry points; the forms without groups that they stand in for left as much
    edge = {P128_G2: 128, P64_G2: 64, P64_G4: 64}
    seen = set()
    for P in (16, 80, 656, 1264, 2048, 2672, 5104, 9200):
        for Q in (64, 304, 704, 1536, 2080, 3232):
            for R in (16, 144, 1040, 2672, 5424, 6128, 11408):
                for leaves in (False, True):
                    p = plan(P, Q, R, pipe, leaves)
                    if p["form"] in edge:
                        e = edge[p["form"]]
                        lds, tiles = p["ring"] * 2 * e * 128, -(-P // e) * -(-Q // e) * p["slices"]
                        room = LDS_OF_A_CU - min(-(-tiles // 256), LDS_OF_A_CU // lds) * lds
                        assert room >= 3 * QUANTIZER_LDS, (P, Q, R, leaves, p)
                        seen.add((p["form"], p["ring"]))
    assert {(P128_G2, 3), (P64_G2, 3), (P64_G2, 4)} <= seen


# input gradients that carry the slice sum of the weight gradient (us of both products without groups of waves, with)
@pytest.mark.parametrize("M,N,K,pipe,plain,groups", [
    (5328, 3104, 736, F16C, 58.1, 64.1), (7296, 1968, 448, F16C, 37.6, 41.5), (6416, 2496, 560, F16W, 48.8, 52.8),
    (3824, 9344, 192, I8, 39.5, 41.9), (6064, 1488, 320, I8, 25.1, 27.7),
    (4304, 320, 288, F16W, 15.6, 17.0), (9504, 544, 112, F16C, 17.5, 19.1), (2320, 96, 560, BF16, 10.9, 11.4),
    (6784, 4016, 432, F16C, 60.7, 56.9), (6512, 5264, 480, F16W, 81.9, 76.6), (10304, 5440, 288, I8, 65.0, 61.9),
    (5248, 3008, 448, I8, 36.5, 31.8), (2816, 272, 368, I8, 11.6, 10.0), (4832, 1488, 320, F16C, 27.5, 23.6),
    (9360, 2528, 176, I8, 33.7, 29.0)])
def test_launches_that_carry_a_slice_sum_leave_room_for_it(plan, M, N, K, pipe, plain, groups):
    rides = plan(N, K, M, pipe, leaves=True)["slices"]
    assert rides > 1
    assert (plan(M, K, N, pipe, rides=rides)["form"] in (P128_G2, P64_G2, P64_G4)) == (groups < plain)


@pytest.mark.parametrize("pipe", [F8, BF16, F16C, F16W])
def test_no_binary32_sum_is_longer_than_a_slice_of_the_plan_and_uncut_sums_are_halved(plan, pipe):
    groups = {P256: 1, P128: 1, P128_S2: 2, P128_G2: 2, P128x192: 1, P64_G2: 2, P64_G4: 4}
    element = 2 if pipe == BF16 else 1
    for P in (16, 80, 656, 1264, 2048, 5104):
        for Q in (64, 304, 704, 2080):
            for R in (16, 144, 400, 688, 1040, 2672, 5424, 6128):
                for leaves in (False, True):
                    p = plan(P, Q, R, pipe, leaves)
                    part = min(p["k_per_split"], element * R) / groups[p["form"]]
                    whole = plan(P, Q, R, pipe, leaves, rides=5)
                    # with a sum on board: the same slices in as many parts, so the same result
                    assert (p["slices"], p["k_per_split"], groups[p["form"]]) == (whole["slices"], whole["k_per_split"],
                                                                                  groups[whole["form"]])
                    assert part <= element * R / p["planned_slices"] + 128
                    if p["form"] in (P64_G2, P64_G4):
                        assert part <= max(64, element * R / 2)


def test_gpu_tests_reach_every_form(plan):
    # (form, stages of the ring, sliced) that the shapes of the GPU tests take, on each pipeline
    seen = {pipe: set() for pipe in range(5)}
    carried = {pipe: set() for pipe in range(5)}
    for pipe in range(5):
        for P, Q, R in GROUP_SHAPES:
            p = plan(P, Q, R, pipe)
            seen[pipe].add((p["form"], p["ring"], p["slices"] > 1))
        for M, N, K in RIDE_SHAPES:
            rides = plan(N, K, M, pipe, True)["slices"]
            if rides > 1 and plan.pair(M, N, K, pipe)["form"] == 0:  # (in one launch the sums follow on their own)
                p = plan(M, K, N, pipe, rides=rides)
                carried[pipe].add((p["form"], p["slices"] > 1))
    for pipe in range(5):
        ring = 3 if pipe in (F16C, F16W) else 4
        assert {(P64_G2, 3, False), (P64_G2, ring, True), (P128_G2, 3, False), (P128_G2, 3, True)} <= seen[pipe], pipe
    for pipe in (I8, F16C, F8):
        assert (P64_G2, 4, False) in seen[pipe]
    for pipe in (F16C, F16W):
        assert {(P64_G4, 5, False), (P64_G4, 3, False)} <= seen[pipe]
    assert {(P64_G2, False), (P128, False), (P128_G2, False)} <= carried[I8]
    assert {(P64_G2, False), (P128_S2, False), (P128_G2, False)} <= carried[F8]
    for pipe in (F16C, F16W):
        assert {(P64_G2, False), (P128_S2, False), (P128_G2, False)} <= carried[pipe]


def test_mfma_tiles_of_gradients_on_wide_tiles(plan):
    # 32 x 32 alone with up to 256 tiles of 128 x 192, beside two sets of a pair with up to 512; 16 x 16 in a pair of one set each.  A
    # gradient in a call of its own has those of the pair
    seen = set()
    for M, N, K in LARGE_MFMA_SHAPES:
        o = (C.c_uint * 8)()
        plan.large_mfma(M, N, K, F16C, o)
        form, mixed, *values = o
        for gradient, paired, alone, tiles in zip(("weight", "input"), *(values[i:i + 2] for i in (0, 2, 4))):
            assert alone == (0 < tiles <= (256 if not form else 512 if mixed else 0)), (M, N, K, gradient)
            assert not form or paired == alone
            if tiles:
                seen.add((gradient, (tiles > 256) + (tiles > 512), "mixed" if form and mixed else "pair" if form else "alone"))
    want = {(n, beside) for n in range(3) for beside in ("alone", "pair", "mixed")}
    assert seen == {(gradient,) + s for gradient in ("weight", "input") for s in want}, seen ^ {(g,) + s for g in ("weight", "input") for s in want}
