"""The weight-only objective (Sec. 3.2: quantized weights, full-precision activations and
gradients) through the C ABI against the oracle's binary64 definition: Y = A Q(W)^T and
dA = dY Q(W), every weight format, binary32 and bfloat16 row operands."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import DEV, KINDS, check_product, host_src, say
from paper_2511_00874_amd import lib as L
from paper_2511_00874_amd import synth

pytestmark = pytest.mark.gpu

NOQ = L.Quant(L.NONE, 1.0)


def _case(M, N, K, kind, bf16_rows, bf16_w, seed):
    A = synth.gaussian_torch((M, K), 1.0, seed, DEV)
    dY = synth.gaussian_torch((M, N), 1e-3, seed + 1, DEV)
    W = synth.gaussian_torch((N, K), 0.02, seed + 2, DEV)
    if bf16_rows:
        A, dY = A.to(torch.bfloat16), dY.to(torch.bfloat16)
    if bf16_w:
        W = W.to(torch.bfloat16)
    sW = float(L.sr_absmax_scale(W, kind).cpu()[0])
    return A, dY, W, sW


@pytest.mark.parametrize("bf16_rows", [False, True])
@pytest.mark.parametrize("kind", KINDS)
def test_forward_and_input_gradient_match_the_definition(kind, bf16_rows):
    # ragged: edge tiles in both output dimensions, contraction tails (208 = 128 + 80)
    M, N, K = 272, 144, 208
    A, dY, W, sW = _case(M, N, K, kind, bf16_rows, bf16_w=(kind == L.INT4), seed=50 + kind)
    qW = L.Quant(kind, sW, seed=9, counter_offset=77)
    oq = oracle.Quant(kind, sW, seed=9, counter_offset=77)
    say("weight-only", L.KIND_NAMES[kind], "bf16 rows" if bf16_rows else "fp32 rows", M, N, K)
    Y = L.sr_linear_fwd(A, W, NOQ, qW).cpu().numpy()
    ref, ab = oracle.linear_fwd_weight_only(host_src(A), host_src(W), oq, want_abs=True)
    check_product(Y, ref, ab, "Y")
    dA = L.sr_linear_bwd_data(dY, W, NOQ, qW).cpu().numpy()
    ref, ab = oracle.linear_bwd_data_weight_only(host_src(dY), host_src(W), oq, want_abs=True)
    check_product(dA, ref, ab, "dA")


def test_binary32_operand_is_split_exactly():
    # integers up to 2^24 - 1 need all 24 significand bits: with W = identity (on the int8 grid
    # at scale 1) the product returns A itself, bit for bit, only if the three planes sum to it
    M, K = 64, 64
    g = torch.Generator(device=DEV).manual_seed(3)
    A = torch.randint(-(1 << 24) + 1, 1 << 24, (M, K), device=DEV, generator=g).float()
    A[0, :8] = torch.tensor([0.0, -0.0, 1.0, 2.0 ** -126, 16777215.0, -16777215.0, 3.0e38, 1.0 + 2.0 ** -23], device=DEV)
    W = torch.eye(K, device=DEV)
    Y = L.sr_linear_fwd(A, W, NOQ, L.Quant(L.INT8, 1.0, seed=1))
    bad = (Y != A).nonzero().cpu().numpy()
    say("mismatches", [(int(i), int(j), float(A[i, j]), float(Y[i, j])) for i, j in bad[:10]])
    assert torch.equal(Y, A)
    # the stated limit: the bf16 matrix pipeline takes subnormal numbers as zero
    A[0, 3] = 2.0 ** -140
    Y = L.sr_linear_fwd(A, W, NOQ, L.Quant(L.INT8, 1.0, seed=1))
    assert float(Y[0, 3]) == 0.0 and torch.equal(Y[1:], A[1:])


def test_long_contraction_is_split_and_accumulated():
    # few tiles, long contraction: the three plane products each run in slices and accumulate
    M, N, K = 128, 128, 16384
    A, dY, W, sW = _case(M, N, K, L.E5M2, False, False, seed=70)
    qW, oq = L.Quant(L.E5M2, sW, seed=2), oracle.Quant(L.E5M2, sW, seed=2)
    Y = L.sr_linear_fwd(A, W, NOQ, qW).cpu().numpy()
    ref, ab = oracle.linear_fwd_weight_only(host_src(A), host_src(W), oq, want_abs=True)
    check_product(Y, ref, ab, "Y")


def test_gpt2_mlp_shape_int8_weights():
    M, N, K = 8192, 3072, 768
    A, dY, W, sW = _case(M, N, K, L.INT8, False, False, seed=80)
    qW, oq = L.Quant(L.INT8, sW, seed=4, counter_offset=5), oracle.Quant(L.INT8, sW, seed=4, counter_offset=5)
    Y = L.sr_linear_fwd(A, W, NOQ, qW).cpu().numpy()
    ref, ab = oracle.linear_fwd_weight_only(host_src(A), host_src(W), oq, want_abs=True)
    check_product(Y, ref, ab, "Y")
    dA = L.sr_linear_bwd_data(dY, W, NOQ, qW).cpu().numpy()
    ref, ab = oracle.linear_bwd_data_weight_only(host_src(dY), host_src(W), oq, want_abs=True)
    check_product(dA, ref, ab, "dA")


# binary32 rows: less than a tile, edges of the 64- and 128-wide tiles, contractions that end inside a
# stage of 32 elements, one stage, a sliced contraction whose last slice is short, many tiles
@pytest.mark.parametrize("M,N,K", [(16, 16, 16), (64, 64, 48), (80, 112, 32), (144, 272, 80), (128, 128, 4112),
                                   (48, 2064, 1040), (2064, 2064, 144)])
def test_binary32_rows_at_the_edges_of_tiles_stages_and_slices(M, N, K):
    A, dY, W, sW = _case(M, N, K, L.E4M3, False, True, seed=90)
    qW, oq = L.Quant(L.E4M3, sW, seed=6, counter_offset=3), oracle.Quant(L.E4M3, sW, seed=6, counter_offset=3)
    say("binary32 rows", M, N, K)
    Y = L.sr_linear_fwd(A, W, NOQ, qW).cpu().numpy()
    ref, ab = oracle.linear_fwd_weight_only(host_src(A), host_src(W), oq, want_abs=True)
    check_product(Y, ref, ab, "Y")
    dA = L.sr_linear_bwd_data(dY, W, NOQ, qW).cpu().numpy()
    ref, ab = oracle.linear_bwd_data_weight_only(host_src(dY), host_src(W), oq, want_abs=True)
    check_product(dA, ref, ab, "dA")
    # a non-finite value reaches its own row of the result and no other
    clean = torch.from_numpy(Y).to(DEV)
    A[M // 2, K - 1] = float("inf")
    Y = L.sr_linear_fwd(A, W, NOQ, qW)
    assert bool(torch.isnan(Y[M // 2]).all())
    keep = torch.arange(M, device=DEV) != M // 2
    assert torch.equal(Y[keep], clean[keep])


# 128 x 128 tiles multiply in MFMA tiles of 32 x 32 up to 256 of them, of 16 x 16 beyond: 256 and 272 tiles with one set of sums, and
# slices with two sets, few and many; the last rows and columns end inside a tile
@pytest.mark.parametrize("M,N,K", [(2048, 2048, 144), (2064, 2032, 144), (544, 976, 4576), (944, 2208, 1664)])
def test_binary32_rows_on_both_sizes_of_mfma_tiles(M, N, K):
    A, _, W, sW = _case(M, N, K, L.INT8, False, True, seed=95)
    say("binary32 rows, MFMA tiles", M, N, K)
    Y = L.sr_linear_fwd(A, W, NOQ, L.Quant(L.INT8, sW, seed=6, counter_offset=3)).cpu().numpy()
    ref, ab = oracle.linear_fwd_weight_only(host_src(A), host_src(W), oracle.Quant(L.INT8, sW, seed=6, counter_offset=3), want_abs=True)
    check_product(Y, ref, ab, "Y")


# contractions that one bfloat16 product over the three parts side by side would leave whole (the first two) and
# would cut into 2, 2, 3, 6, 7 and 11 slices
@pytest.mark.parametrize("M,N,K", [(256, 256, 256), (2064, 1040, 272), (1200, 608, 400), (8192, 768, 3072),
                                   (1888, 416, 544), (688, 720, 1152), (736, 688, 1744), (432, 576, 2320)])
def test_binary32_rows_are_no_less_precise_than_their_parts_side_by_side(M, N, K):
    # grid values and scale 1: the quantizer passes W through.  Both forms multiply the same exact parts and sum in
    # binary32, this one with no more roundings at the size of the sum; over 6 x 10^4 outputs and more the 2-norm of the
    # error is no larger but for chance, which is below 1 %
    rng = torch.Generator().manual_seed(K)
    W = torch.randn((N, K), generator=rng).to(torch.float8_e4m3fn).float()
    A, part, parts = torch.randn((M, K), generator=rng), None, []
    rest = A.clone()
    for _ in range(3):
        part = (rest.view(torch.int32) & -65536).view(torch.float32)
        parts.append(part)
        rest = rest - part
    assert not rest.any()
    say("error of", M, N, K)
    got = L.sr_linear_fwd(A.to(DEV), W.to(DEV), NOQ, L.Quant(L.E4M3, 1.0, seed=1))
    side = L.sr_gemm_bf16(torch.cat(parts, 1).to(DEV, torch.bfloat16), torch.cat([W] * 3, 1).to(DEV, torch.bfloat16))
    ref = (A.double() @ W.double().T).to(DEV)
    err, err_side = ((p.double() - ref).norm().item() for p in (got, side))
    assert err <= 1.05 * err_side, (err / ref.norm().item(), err_side / ref.norm().item())


def test_where_the_identity_quantizer_is_not_accepted():
    A = torch.zeros((16, 16), device=DEV)
    q8 = L.Quant(L.INT8, 1.0)
    with pytest.raises(RuntimeError):
        L.sr_linear_fwd(A, A, q8, NOQ)            # W must be quantized
    with pytest.raises(RuntimeError):
        L.sr_linear_bwd_weight(A, A, NOQ, q8)     # no quantized operand: not this library's product
    with pytest.raises(RuntimeError):
        L.sr_quantize(A, NOQ)
