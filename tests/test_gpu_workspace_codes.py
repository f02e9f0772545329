"""The quantized operands the linear entry points leave in the caller's workspace, compared bit for
bit with the oracle's codes: these come from the kernel that quantizes all operands of a call in one
launch (same-layout, transposing, two-output and bfloat16-valued forms), not from sr_quantize.

Workspace layout (pieces aligned to 256 bytes): forward  [Q(A) M x K | Q(W) N x K | slices];
whole backward pass  [Q(dY) M x N | Q(W)^T K x N | slices | Q(dY)^T N x M | Q(A)^T K x M | slices].
An operand is one byte per element (integer formats: the value; a 4-bit dY from a binary32 source is
stored two per byte for the products that run on 256 x 256 tiles; E5M2 when every operand
of the call is E5M2: the code) or the grid value as bfloat16."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_00874_amd import lib as L
from paper_2511_00874_amd import synth
from gpu_util import KINDS, host_src, say, to_dev

pytestmark = pytest.mark.gpu


def _up(n):
    return (n + 255) // 256 * 256


def _form(kind):
    """(element size, slice-workspace query) of the stored form when all operands have this kind."""
    if kind in (L.INT8, L.INT4):
        return 1, lambda P, Q, R: L.sr_gemm_workspace_bytes(P, Q, R)
    if kind == L.E5M2:
        return 1, lambda P, Q, R: L.raw.sr_gemm_e5m2_workspace_bytes(P, Q, R)
    return 2, lambda P, Q, R: L.raw.sr_gemm_bf16_workspace_bytes(P, Q, R)


def _expect(t, kind, q, transpose, es, mode=oracle.SR):
    codes = oracle.quantize(host_src(t), kind, q.scale, q.seed, q.counter_offset, mode)
    if transpose:
        codes = np.ascontiguousarray(codes.T)
    if es == 1:
        return codes.reshape(-1)
    vals = oracle.decode_array(kind, codes).astype(np.float32)   # every grid value is a bfloat16 number
    return torch.from_numpy(vals).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint8).reshape(-1)


def _piece(ws, off, n):
    return ws[off:off + n].cpu().numpy()


def _run(M, N, K, kind, seed, w_bf16):
    A, W, dY = synth.single_layer(M, N, K, seed, std_dy=1e-3)
    A, W, dY = to_dev(A), to_dev(W, w_bf16), to_dev(dY)
    qs, off = {}, 0
    for name, t in (("A_fwd", A), ("W_fwd", W), ("dY", dY), ("W_bwd", W), ("A_bwd", A)):
        qs[name] = oracle.Quant(kind, oracle.absmax_scale(host_src(t), kind), seed, off)
        off += (t.numel() + 7) // 8
    lq = {n: L.Quant(kind, q.scale, q.seed, q.counter_offset) for n, q in qs.items()}
    es, slices = _form(kind)

    ws = torch.zeros(L.sr_linear_workspace_bytes(L.OP_FWD, M, N, K), dtype=torch.uint8, device=A.device)
    L.sr_linear_fwd(A, W, lq["A_fwd"], lq["W_fwd"], workspace=ws)
    assert np.array_equal(_piece(ws, 0, M * K * es), _expect(A, kind, qs["A_fwd"], False, es)), "Q(A) forward"
    assert np.array_equal(_piece(ws, _up(M * K * es), N * K * es), _expect(W, kind, qs["W_fwd"], False, es)), "Q(W) forward"

    ws = torch.zeros(L.sr_linear_workspace_bytes(L.OP_BWD, M, N, K), dtype=torch.uint8, device=A.device)
    L.sr_linear_bwd(dY, W, A, lq["dY"], lq["W_bwd"], lq["A_bwd"], workspace=ws)
    o_dy = 0
    o_wt = o_dy + _up(M * N * es)
    o_dyt = o_wt + _up(K * N * es) + _up(slices(M, K, N))
    o_at = o_dyt + _up(N * M * es)
    assert np.array_equal(_piece(ws, o_dy, M * N * es), _expect(dY, kind, qs["dY"], False, es)), "Q(dY)"
    assert np.array_equal(_piece(ws, o_wt, K * N * es), _expect(W, kind, qs["W_bwd"], True, es)), "Q(W)^T"
    assert np.array_equal(_piece(ws, o_dyt, N * M * es), _expect(dY, kind, qs["dY"], True, es)), "Q(dY)^T"
    assert np.array_equal(_piece(ws, o_at, K * M * es), _expect(A, kind, qs["A_bwd"], True, es)), "Q(A)^T"


@pytest.mark.parametrize("kind", KINDS)
def test_ragged_layer_every_format(kind):
    say("workspace codes", L.KIND_NAMES[kind])
    _run(272, 144, 208, kind, seed=3, w_bf16=True)


@pytest.mark.parametrize("kind", [L.INT8, L.E5M2])
def test_gpt2_fc1_benchmark_formats(kind):
    say("workspace codes fc1", L.KIND_NAMES[kind])
    _run(8192, 3072, 768, kind, seed=10, w_bf16=False)


def test_many_row_bands_with_a_ragged_last_group():
    # the transposing quantizer walks its tiles in groups of 32 bands of 128 rows: 37 full bands and
    # a band of 16 rows make one full group and one of six bands, the last of them partial
    say("workspace codes, 4752 rows")
    _run(4752, 144, 208, L.INT8, seed=5, w_bf16=True)


# Launches whose quantizers all round to nearest, and launches of both modes: the mode is a branch of a job, and saved float codes have a
# kernel of their own only where both quantizers round stochastically; the sources span
# 40 binades with zeros of both signs, infinities and NaN, so that a quad holds numbers that the 8-bit conversions round,
# subnormals of the grid and numbers that underflow, and the scale is not that of the largest element (saturation).
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("modes", [(L.SR, L.SR, L.SR), (L.RTN, L.RTN, L.RTN), (L.SR, L.RTN, L.SR)])
def test_codes_of_mixed_rounding_and_wide_ranges(kind, modes):
    M, N, K, seed = 144, 80, 208, 21
    say("workspace codes, modes", L.KIND_NAMES[kind], modes)
    rng = np.random.default_rng(kind)

    def wide(shape):
        x = (rng.standard_normal(shape) * np.exp2(rng.uniform(-38, 2, shape))).astype(np.float32)
        flat = x.reshape(-1)
        at = rng.permutation(flat.size)[:96]
        flat[at] = np.resize(np.float32([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-40, -1e-40, 3e38]), 96)
        return x

    A, W, dY = to_dev(wide((M, K))), to_dev(wide((N, K)), True), to_dev(wide((M, N)))
    oq, lq, off = {}, {}, 0
    for name, t, mode in (("dY", dY, modes[0]), ("W", W, modes[1]), ("A", A, modes[2])):
        scale = float(np.float32(2.0 / L.QMAX[kind]))
        oq[name] = oracle.Quant(kind, scale, seed, off)
        lq[name] = L.Quant(kind, scale, seed, off, round_mode=mode)
        off += (t.numel() + 7) // 8
    es, slices = _form(kind)
    mode_of = dict(zip(("dY", "W", "A"), modes))
    ws = torch.zeros(L.sr_linear_workspace_bytes(L.OP_BWD, M, N, K), dtype=torch.uint8, device=A.device)
    L.sr_linear_bwd(dY, W, A, lq["dY"], lq["W"], lq["A"], workspace=ws)
    o_wt = _up(M * N * es)
    o_dyt = o_wt + _up(K * N * es) + _up(slices(M, K, N))
    o_at = o_dyt + _up(N * M * es)
    for what, name, t, off_b, tr in (("Q(dY)", "dY", dY, 0, False), ("Q(W)^T", "W", W, o_wt, True),
                                     ("Q(dY)^T", "dY", dY, o_dyt, True), ("Q(A)^T", "A", A, o_at, True)):
        want = _expect(t, kind, oq[name], tr, es, mode_of[name])
        got = _piece(ws, off_b, want.size)
        if es == 2:  # NaN has a payload of its own in each
            got, want = (x.view(np.uint16) for x in (got, want))
            nan = (want & 0x7FFF) > 0x7F80
            assert np.all((got[nan] & 0x7FFF) > 0x7F80)
            got, want = got[~nan], want[~nan]
        assert np.array_equal(got, want), what
    # integer codes in the source layout beside the transposed ones (the stash call): both of A's quantizers
    q8 = L.Quant(L.INT8, 0.02, seed, 5000, round_mode=modes[1])
    q8w = L.Quant(L.INT8, 0.02, seed, 9000, round_mode=modes[0])
    ws = torch.zeros(L.sr_linear_workspace_bytes(L.OP_FWD_STASH, M, N, K), dtype=torch.uint8, device=A.device)
    _, stash = L.sr_linear_fwd_stash(A, W, q8, q8w, lq["A"], lq["W"], workspace=ws)
    q = oracle.Quant(L.INT8, 0.02, seed, 5000)
    assert np.array_equal(_piece(ws, 0, M * K), _expect(A, L.INT8, q, False, 1, modes[1])), "Q(A) forward"
    if es == 1:
        assert np.array_equal(_piece(stash, 0, M * K), _expect(A, kind, oq["A"], True, 1, modes[2])), "stash"


# rows and columns that end inside a tile, in its first half and by one group of 16; one tile and several bands; the scale takes some
# elements into the subnormals of the formats and some to saturation
@pytest.mark.parametrize("M,N,K,kind", [(16, 16, 16, L.E5M2), (80, 1040, 144, L.E5M2), (2192, 208, 336, L.E5M2),
                                        (4240, 16, 80, L.E5M2), (272, 1040, 528, L.E4M3), (2096, 144, 464, L.E4M3)])
@pytest.mark.parametrize("fwd", [L.INT8, L.INT4])
def test_stash_codes_of_two_quantizers(M, N, K, kind, fwd):
    say("stash, two quantizers", M, N, K, L.KIND_NAMES[kind], L.KIND_NAMES[fwd])
    rng = np.random.default_rng(M + N)
    A, W = ((rng.standard_normal(s) * np.exp2(rng.uniform(-24, 3, s))).astype(np.float32) for s in ((M, K), (N, K)))
    for w_bf16 in (True, False):
        tA, tW = to_dev(A, not w_bf16), to_dev(W, w_bf16)
        oq = [oracle.Quant(k, s, 17, 1000 * i) for i, (k, s) in enumerate(((fwd, 0.03), (fwd, 0.04), (kind, 0.01), (kind, 0.02)))]
        lq = [L.Quant(q.kind, q.scale, q.seed, q.counter_offset) for q in oq]
        ws = torch.zeros(L.sr_linear_workspace_bytes(L.OP_FWD_STASH, M, N, K), dtype=torch.uint8, device=tA.device)
        _, stash = L.sr_linear_fwd_stash(tA, tW, *lq, workspace=ws)
        assert np.array_equal(_piece(ws, 0, M * K), _expect(tA, fwd, oq[0], False, 1)), "Q(A)"
        assert np.array_equal(_piece(ws, _up(M * K), N * K), _expect(tW, fwd, oq[1], False, 1)), "Q(W)"
        assert np.array_equal(_piece(stash, 0, M * K), _expect(tA, kind, oq[2], True, 1)), "Q(A)^T"
        assert np.array_equal(_piece(stash, _up(2 * M * K), N * K), _expect(tW, kind, oq[3], True, 1)), "Q(W)^T"


def _spread(shape, rng, bf16):
    """Elements over 27 binades (some in the subnormals of the formats, some at saturation), one in 40 of them zeros of both signs,
    infinities, NaN, subnormals of binary32 and numbers near its end."""
    x = (rng.standard_normal(shape) * np.exp2(rng.uniform(-24, 3, shape))).astype(np.float32)
    flat = x.reshape(-1)
    at = rng.permutation(flat.size)[:flat.size // 40 + 8]
    flat[at] = np.resize(np.float32([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-40, -1e-40, 3e38, -3e38]), at.size)
    return to_dev(x, bf16)


# the quantizers of a backward call that round stochastically to bytes have a kernel of their own (tiles of 128 rows and 64 columns,
# steps of 64 and 128 rows, pieces of four): both sides of its edges and of the rule on binary32 rows 4096 and 8192 apart
# (2048 rows, and more; other multiples of 4096 have none); one format for all operands, and one for dY beside another for W and A
@pytest.mark.parametrize("M,N,K,kind,kind_dy", [
    (16, 16, 16, L.E5M2, L.E5M2), (80, 1040, 144, L.E5M2, L.E5M2), (144, 80, 4240, L.E5M2, L.E5M2), (2192, 208, 336, L.E5M2, L.E5M2),
    (2048, 4096, 16, L.E5M2, L.E5M2), (2064, 4096, 16, L.E5M2, L.E5M2), (2064, 8192, 16, L.E5M2, L.E5M2), (1040, 528, 272, L.E4M3, L.E4M3), (2064, 144, 464, L.E4M3, L.E4M3),
    (1040, 528, 272, L.E4M3, L.E5M2), (2064, 144, 464, L.E4M3, L.E5M2),
    (16, 16, 16, L.INT8, L.INT8), (144, 80, 4240, L.INT8, L.INT8), (2192, 208, 336, L.INT4, L.INT4), (2048, 4096, 16, L.INT8, L.INT8),
    (2064, 4096, 16, L.INT8, L.INT8), (2048, 8192, 16, L.INT8, L.INT8), (272, 1040, 528, L.INT4, L.INT4), (272, 1040, 528, L.INT8, L.INT4)])
@pytest.mark.parametrize("bf16", [False, True])
def test_backward_codes(M, N, K, kind, kind_dy, bf16):
    say("backward codes", M, N, K, L.KIND_NAMES[kind], L.KIND_NAMES[kind_dy], bf16)
    rng = np.random.default_rng(M + N + K)
    A, W, dY = (_spread(s, rng, bf16) for s in ((M, K), (N, K), (M, N)))
    assert L.E4M3 not in (kind, kind_dy) or M * N * K >= 2**27  # one byte an element
    oq = [oracle.Quant(k, s, 17, 1000 * i) for i, (k, s) in enumerate(((kind_dy, 0.01), (kind, 0.02), (kind, 0.015)))]
    qdY, qW, qA = (L.Quant(q.kind, q.scale, q.seed, q.counter_offset) for q in oq)
    ws = torch.zeros(L.sr_linear_workspace_bytes(L.OP_BWD_STASHED, M, N, K), dtype=torch.uint8, device=A.device)
    stash = torch.zeros(L.sr_linear_stash_bytes(M, N, K), dtype=torch.uint8, device=A.device)
    dA, dW = torch.empty((M, K), device=A.device), torch.empty((N, K), device=A.device)
    whole = torch.zeros(L.sr_linear_workspace_bytes(L.OP_BWD, M, N, K), dtype=torch.uint8, device=A.device)
    L.sr_linear_bwd(dY, W, A, qdY, qW, qA, out_dA=dA, out_dW=dW, workspace=whole, phase=L.PHASE_QUANTIZE)
    L.sr_linear_bwd_stashed(dY, stash, K, qdY, qW, qA, out_dA=dA, out_dW=dW, workspace=ws, phase=L.PHASE_QUANTIZE)
    slices = L.sr_gemm_workspace_bytes if kind in (L.INT8, L.INT4) else L.raw.sr_gemm_e5m2_workspace_bytes
    partial = _up(slices(M, K, N))
    assert L.E4M3 not in (kind, kind_dy) or partial == _up(L.raw.sr_gemm_bf16_workspace_bytes(M, K, N))  # (it may take that plan)
    o_wt = _up(M * N)
    o_dyt = o_wt + _up(K * N) + partial
    o_at = o_dyt + _up(N * M)
    for what, blob, off, t, q, tr in (("Q(dY)", whole, 0, dY, oq[0], False), ("Q(W)^T", whole, o_wt, W, oq[1], True),
                                      ("Q(dY)^T", whole, o_dyt, dY, oq[0], True), ("Q(A)^T", whole, o_at, A, oq[2], True),
                                      ("Q(dY), stashed", ws, 0, dY, oq[0], False), ("Q(dY)^T, stashed", ws, o_wt + partial, dY, oq[0], True)):
        assert np.array_equal(_piece(blob, off, t.numel()), _expect(t, q.kind, q, tr, 1)), what


# operands of a forward pass: chunks of 512 elements and what is left over, four loads of a bfloat16 source and fewer
@pytest.mark.parametrize("M,N,K,kind", [(16, 16, 16, L.INT8), (48, 80, 208, L.INT4), (272, 1040, 528, L.INT8), (16, 16, 16, L.E5M2),
                                        (48, 1040, 272, L.E5M2), (1040, 528, 272, L.E4M3), (272, 1040, 528, L.E4M3)])
@pytest.mark.parametrize("bf16", [False, True])
def test_forward_codes(M, N, K, kind, bf16):
    say("forward codes", M, N, K, L.KIND_NAMES[kind], bf16)
    rng = np.random.default_rng(M + N + K)
    A, W = (_spread(s, rng, b) for s, b in (((M, K), bf16), ((N, K), not bf16)))
    oq = [oracle.Quant(kind, s, 17, 1000 * i) for i, s in enumerate((0.01, 0.02))]
    lq = [L.Quant(q.kind, q.scale, q.seed, q.counter_offset, flags=L.FLAG_QUANTIZE_ONCE) for q in oq]
    ws = torch.zeros(L.sr_linear_workspace_bytes(L.OP_FWD, M, N, K), dtype=torch.uint8, device=A.device)
    L.sr_linear_fwd(A, W, *lq, out=torch.empty((M, N), device=A.device), workspace=ws, phase=L.PHASE_QUANTIZE)
    assert np.array_equal(_piece(ws, 0, M * K), _expect(A, kind, oq[0], False, 1)), "Q(A)"
    assert np.array_equal(_piece(ws, _up(M * K), N * K), _expect(W, kind, oq[1], False, 1)), "Q(W)"


def _nib16(codes):
    """Two 4-bit values per byte: byte j of every 8 holds elements j (low nibble) and j + 8 (high nibble)
    of a run of 16 along the last axis."""
    r = (codes.view(np.uint8) & 0x0F).reshape(codes.shape[0], -1, 2, 8)
    return (r[:, :, 0, :] | (r[:, :, 1, :] << 4)).reshape(codes.shape[0], -1)


# the benchmark's layer shape at 16384 tokens; ragged shapes whose products take the 256 x 256 tiles, with
# contractions that end half way through a 16-byte piece of packed values (length % 32 == 16), one of
# them long enough to be cut into slices
@pytest.mark.parametrize("M,N,K", [(16384, 2048, 2048), (8208, 1040, 4112), (32784, 2064, 1040), (6160, 1040, 4112)])
def test_four_bit_gradient_is_stored_two_per_byte_for_the_large_tile_products(M, N, K):
    # Llama formats (int4 dY, int8 elsewhere), binary32 dY: where a backward product runs on the 256 x 256
    # tiles its copy of Q(dY) is written two values per byte; elsewhere one per byte.  Either way the
    # values are the oracle's, and for the benchmark's layer shape both copies are packed.
    say("workspace codes, packed int4 dY", M, N, K)
    A, W, dY = synth.single_layer(M, N, K, 9, std_dy=1e-3)
    A, W, dY = to_dev(A), to_dev(W, True), to_dev(dY)
    q = {}
    off = 0
    for name, t, kind in (("dY", dY, L.INT4), ("W", W, L.INT8), ("A", A, L.INT8)):
        q[name] = oracle.Quant(kind, oracle.absmax_scale(host_src(t), kind), 4, off)
        off += (t.numel() + 7) // 8
    lq = {n: L.Quant(v.kind, v.scale, v.seed, v.counter_offset) for n, v in q.items()}
    ws = torch.zeros(L.sr_linear_workspace_bytes(L.OP_BWD, M, N, K), dtype=torch.uint8, device=A.device)
    dA, dW = L.sr_linear_bwd(dY, W, A, lq["dY"], lq["W"], lq["A"], workspace=ws)
    codes = oracle.quantize(host_src(dY), L.INT4, q["dY"].scale, q["dY"].seed, q["dY"].counter_offset)
    slices = L.sr_gemm_workspace_bytes
    o_dy = 0
    o_dyt = _up(M * N) + _up(K * N) + _up(slices(M, K, N))
    packed = []
    for name, off_b, c in (("Q(dY)", o_dy, codes), ("Q(dY)^T", o_dyt, np.ascontiguousarray(codes.T))):
        got = _piece(ws, off_b, M * N)
        if np.array_equal(got, c.reshape(-1)):
            packed.append(False)
        else:
            assert np.array_equal(got[:M * N // 2], _nib16(c).reshape(-1)), name
            packed.append(True)
    if (M, N, K) == (16384, 2048, 2048):
        assert packed == [True, True]
    assert any(packed)   # (which products take the large tiles is the cost model's choice; these shapes do today)
    # and the products from them are those of the separate calls (one value per byte) bit for bit
    assert torch.equal(dA, L.sr_linear_bwd_data(dY, W, lq["dY"], lq["W"]))
    assert torch.equal(dW, L.sr_linear_bwd_weight(dY, A, lq["dY"], lq["A"]))
    # accumulation onto the weight gradient (beta = 1) through the packed products and their slice sums
    acc = dW.clone()
    L.sr_linear_bwd(dY, W, A, lq["dY"], lq["W"], lq["A"], out_dA=dA, out_dW=acc, beta=1.0, workspace=ws)
    assert torch.equal(acc, dW + dW)
    say("   packed:", packed)
