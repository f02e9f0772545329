"""GPU parity of sr_quantize / sr_absmax_scale against the CPU oracle: codes bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_00874_amd import lib as L
from paper_2511_00874_amd import synth
from gpu_util import DEV, KINDS, host_src, oracle_codes, say, to_dev

pytestmark = pytest.mark.gpu


def _specials():
    tiny = np.float32(1e-40)  # subnormal in binary32
    v = [0.0, -0.0, np.nan, np.inf, -np.inf, tiny, -tiny, 1e-30, -1e-30, 3e38, -3e38,
         0.5, -0.5, 1.5, -1.5, 126.5, 127.0, 127.49, -127.5, 448.0, 449.0, 57344.0, 60000.0,
         2.0**-6, 2.0**-9, 2.0**-10, -(2.0**-10), 2.0**-14, 2.0**-16, 2.0**-17, -(2.0**-17),
         0.9999999, 1.0000001, 7.0, 7.5, -7.5, 15.99, 16.0, 255.9, 256.0]
    return np.array(v, dtype=np.float32)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mode", [L.SR, L.RTN])
def test_flat_codes_bit_exact_with_ragged_tail(kind, bf16, mode):
    n = 3 * 256 * 8 * 4 + 2 * 8 + 6      # several blocks, a short last group
    x = synth.gaussian((n,), 1.0, 7 + kind)
    x[:_specials().size] = _specials()
    xd = to_dev(x, bf16)
    scale = 0.037
    say("flat", L.KIND_NAMES[kind], "bf16" if bf16 else "f32", mode, n)
    got = L.sr_quantize(xd, L.Quant(kind, scale, seed=0xDEADBEEFCAFE1234, counter_offset=2**64 - 5,
                                    round_mode=mode)).cpu().numpy()
    want = oracle_codes(xd, kind, scale, 0xDEADBEEFCAFE1234, 2**64 - 5, mode)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("kind", KINDS)
def test_scale_one_specials_and_binade_edges(kind):
    # scale 1: the grid coordinate is the input itself
    x = np.concatenate([_specials(), -_specials(),
                        np.float32([oracle.decode(kind, c) for c in range(256)
                                    if np.isfinite(oracle.decode(kind, c))])])
    x = np.concatenate([x, np.nextafter(x, np.float32(np.inf)), np.nextafter(x, np.float32(-np.inf))])
    x = np.resize(x, (x.size + 7) // 8 * 8).astype(np.float32)
    xd = to_dev(x)
    for seed in (0, 1, 2):
        got = L.sr_quantize(xd, L.Quant(kind, 1.0, seed=seed)).cpu().numpy()
        assert np.array_equal(got, oracle_codes(xd, kind, 1.0, seed, 0)), seed


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("shape", [(128, 64), (130, 72), (300, 200), (2, 8), (1000, 8), (16, 1024)])
def test_transposed_codes_equal_the_same_codes_transposed(kind, shape):
    x = synth.gaussian(shape, 2.0, 3)
    xd = to_dev(x)
    scale = oracle.absmax_scale(x, kind)
    say("transpose", L.KIND_NAMES[kind], shape)
    got = L.sr_quantize(xd, L.Quant(kind, scale, seed=11, counter_offset=77), transpose_out=True).cpu().numpy()
    want = oracle_codes(xd, kind, scale, 11, 77, transpose=True)
    assert np.array_equal(got, want)
    # and the row-major call gives the very same codes (thresholds keyed by source index)
    got_rm = L.sr_quantize(xd, L.Quant(kind, scale, seed=11, counter_offset=77)).cpu().numpy()
    assert np.array_equal(got_rm, oracle_codes(xd, kind, scale, 11, 77))


@pytest.mark.parametrize("kind", KINDS)
def test_thresholds_scanned_on_hard_constants(kind):
    # each constant meets ~2^17 different thresholds: values whose fractional part is not a
    # binary32 number (negative coordinates), neighbours of 1/2 ulp traps, tiny magnitudes
    consts = np.float32([-0.3, 0.3, -0.7, -1e-3, (0.5 - 2.0**-25) / 65536.0, -(0.5 - 2.0**-25) / 65536.0,
                         -126.99999, 126.99999, -5.0000005, 2.0**-7 * 1.2345, -(2.0**-7) * 1.2345,
                         2.0**-17, -(2.0**-17), 1.0 - 2.0**-24, -(1.0 - 2.0**-24), 0.49999997])
    x = np.repeat(consts, 1 << 17)
    xd = to_dev(x)
    got = L.sr_quantize(xd, L.Quant(kind, 1.0, seed=77, counter_offset=5)).cpu().numpy()
    assert np.array_equal(got, oracle_codes(xd, kind, 1.0, 77, 5))
    got = L.sr_quantize(xd, L.Quant(kind, 1.0, round_mode=L.RTN)).cpu().numpy()
    assert np.array_equal(got, oracle_codes(xd, kind, 1.0, 0, 0, oracle.RTN))


# runs that start and end off every alignment, one tile and several, both tile heights (256 rows from 16384
# such tiles up), full and partial groups of 16 row bands, fewer rows than a word holds
@pytest.mark.parametrize("shape", [(1, 8), (3, 16), (5, 72), (129, 64), (257, 136), (2051, 200), (4098, 72),
                                   (524290, 8), (524288, 8), (525301, 8), (260, 16392),
                                   (4194306, 8)])
@pytest.mark.parametrize("bf16", [False, True])
def test_transposed_codes_at_odd_row_counts(shape, bf16):
    x = synth.gaussian(shape, 2.0, 3)
    flat = x.reshape(-1)
    flat[-min(flat.size, _specials().size):] = _specials()[:flat.size]
    xd = to_dev(x, bf16)
    for kind in (L.INT8, L.INT4, L.E4M3, L.E5M2, L.E4M1):
        if kind == L.INT4 and shape[0] % 2:
            continue  # two codes of a byte are neighbours in the output
        mode = L.RTN if shape[0] == 2051 else L.SR
        say("transpose", L.KIND_NAMES[kind], "bf16" if bf16 else "f32", shape)
        q = L.Quant(kind, 0.037, seed=0xDEADBEEFCAFE1234, counter_offset=2**64 - 5, round_mode=mode)
        guard = torch.full((x.size + 64,), 0xA5, dtype=torch.uint8, device=xd.device)
        n = x.size // 2 if kind == L.INT4 else x.size
        L.sr_quantize(xd, q, transpose_out=True, out=guard[:n])
        want = oracle_codes(xd, kind, 0.037, 0xDEADBEEFCAFE1234, 2**64 - 5, mode, transpose=True)
        assert np.array_equal(guard[:n].cpu().numpy(), want)
        assert bool((guard[n:] == 0xA5).all())


def test_bf16_transposed():
    x = synth.gaussian((256, 136), 0.02, 5)
    xd = to_dev(x, bf16=True)
    scale = oracle.absmax_scale(host_src(xd), L.INT8)
    got = L.sr_quantize(xd, L.Quant(L.INT8, scale, seed=3), transpose_out=True).cpu().numpy()
    assert np.array_equal(got, oracle_codes(xd, L.INT8, scale, 3, 0, transpose=True))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("bf16", [False, True])
def test_absmax_scale_and_device_scale_path(kind, bf16):
    x = synth.outlier_tensor_np(100003 * 2, 5)
    x[17] = np.nan
    x[18] = np.inf
    xd = to_dev(x, bf16)
    s_dev = L.sr_absmax_scale(xd, kind)
    want = oracle.absmax_scale(host_src(xd), kind)
    assert float(s_dev.item()) == want
    got = L.sr_quantize(xd, L.Quant(kind, s_dev, seed=9)).cpu().numpy()
    assert np.array_equal(got, oracle_codes(xd, kind, want, 9, 0))
    # host scale, same codes
    got2 = L.sr_quantize(xd, L.Quant(kind, want, seed=9)).cpu().numpy()
    assert np.array_equal(got, got2)


# the one-launch form up to 256 KiB, the three-launch form beyond it (one element more), a share per workgroup
# that ends in a partial piece, the change from many to few workgroups; the maximum at either end or nowhere
@pytest.mark.parametrize("n", [1, 7, 4095, 65536, 65537, 131072, 131073, 1048583, 4194311])
@pytest.mark.parametrize("bf16", [False, True])
def test_absmax_scale_finds_the_maximum_wherever_it_is(n, bf16):
    x = synth.gaussian((n,), 1e-3, 5)
    for where, v in ((0, 2.0), (n - 1, -3.0), (n // 2, 5.0), (None, 0.0)):
        y = np.zeros_like(x) if where is None else x.copy()
        if where is not None:
            y[where] = v
        say("absmax", n, "bf16" if bf16 else "f32", where)
        s = float(L.sr_absmax_scale(to_dev(y, bf16), L.INT8).item())
        assert s == (1.0 if where is None else float(np.float32(abs(v)) / np.float32(127)))


# E4M3 tensors of at least 2^22 elements take their codes from the conversion instructions, smaller ones do not: halves of a tensor,
# each below the line, against the whole; zeros, subnormals of the grid, NaN, Inf and saturating values among the elements
@pytest.mark.parametrize("rows,cols", [(2048, 2048), (2052, 2056), (2, (1 << 21) + 8), (4096, 4096)])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mode", [L.SR, L.RTN])
def test_large_e4m3_tensor_has_the_codes_of_its_halves(rows, cols, bf16, mode):
    say("E4M3 on both sides of 2^22 elements", rows, cols, bf16, mode)
    g = torch.Generator(DEV).manual_seed(7)
    x = torch.randn(rows, cols, device=DEV, generator=g) * torch.exp2(torch.rand(rows, cols, device=DEV, generator=g) * 24 - 20)
    x.view(-1)[::997] = float("nan")
    x.view(-1)[1::1009] = 0.0
    x.view(-1)[2::1013] = -0.0
    x.view(-1)[3::1019] = -float("inf")
    x = x.to(torch.bfloat16) if bf16 else x
    half = rows // 2
    q = [L.Quant(L.E4M3, 0.01, 3, o, round_mode=mode) for o in (0, half * cols // 8)]
    want = torch.cat([L.sr_quantize(x[:half], q[0]).view(half, cols), L.sr_quantize(x[half:], q[1]).view(half, cols)])
    assert torch.equal(L.sr_quantize(x, q[0]).view(rows, cols), want)
    assert torch.equal(L.sr_quantize(x, q[0], transpose_out=True).view(cols, rows), want.t())


# NaN of either sign in every place of a group of eight, alone and beside others, has the code 0 and leaves its neighbours theirs
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mode", [L.SR, L.RTN])
def test_codes_of_nan_in_every_place(kind, bf16, mode):
    x = synth.gaussian((1040, 72), 1.0, 11)
    flat = x.reshape(-1)
    for g in range(0, flat.size // 8, 3):
        flat[8 * g + g // 3 % 8] = np.nan if g % 2 else -np.nan
    flat[64:72] = np.nan
    flat[80:88:2] = -np.nan
    xd = to_dev(x, bf16)
    q = L.Quant(kind, 3.0 / L.QMAX[kind], 3, 7, round_mode=mode)
    say("NaN in every place", L.KIND_NAMES[kind], bf16, mode)
    assert np.array_equal(L.sr_quantize(xd, q).cpu().numpy(), oracle_codes(xd, kind, q.scale, 3, 7, mode))
    assert np.array_equal(L.sr_quantize(xd, q, transpose_out=True).cpu().numpy(),
                          oracle_codes(xd, kind, q.scale, 3, 7, mode, transpose=True))


# Codes that come out of the conversion instructions, about the smallest normal number of the grid: values of 2^-12 to 2^4 of it, of
# both signs, whose last bits decide ties of the 16 random bits, against the oracle; every rounding of a wave meets both rules
@pytest.mark.parametrize("kind,n", [(L.E5M2, 1 << 18), (L.E4M3, 1 << 22)])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mode", [L.SR, L.RTN])
def test_converted_codes_about_the_smallest_normal_number(kind, n, bf16, mode):
    say("codes about the smallest normal number", L.KIND_NAMES[kind], bf16, mode)
    least, step = (2.0 ** -6, 2.0 ** -9) if kind == L.E4M3 else (2.0 ** -14, 2.0 ** -16)
    rng = np.random.default_rng(kind)
    x = (least * rng.standard_normal(n, np.float32) * np.exp2(rng.uniform(-12, 4, n))).astype(np.float32)
    ties = rng.integers(-(1 << 22), 1 << 22, n // 4)  # multiples of 2^-17 and 2^-21 of the spacing of the subnormals
    x[::4] = ties.astype(np.float32) * np.float32(step * 2.0 ** -17)
    x[2::8] = ties[::2].astype(np.float32) * np.float32(step * 2.0 ** -21)
    x[1::997], x[3::1009], x[5::1013] = np.nan, 0.0, -0.0
    xd = to_dev(x, bf16)
    got = L.sr_quantize(xd, L.Quant(kind, 1.0, 5, 9, round_mode=mode)).cpu().numpy()
    assert np.array_equal(got, oracle_codes(xd, kind, 1.0, 5, 9, mode))


def _us_in_turn(calls, repeats=12):
    """Least us of each of some calls, two at a time in a graph, timed in turn: the clock of a GPU changes from one millisecond to the next."""
    graphs = []
    for f in calls:
        f()
        torch.cuda.synchronize()
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            f()
            f()
    times = [[] for _ in calls]
    for _ in range(repeats):
        for graph, ms in zip(graphs, times):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            end.synchronize()
            ms.append(start.elapsed_time(end))
    return [min(ms) * 500 for ms in times]


# E4M3 and E5M2 codes of a large tensor take no longer than the codes of E4M2, which no conversion makes, whatever the values: neither
# where 1 % of outliers or a range of 40 binades put nearly every wave among the subnormals, nor where half of the elements are
# zero.  (A tenth for the spread of such times; a loop over the elements of those waves took 1.25 to 1.8 times as long.)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("values", ["normal", "outliers", "half zero", "40 binades"])
def test_converted_codes_take_no_longer_than_code_by_code_whatever_the_values(bf16, transpose, values):
    rows, cols = 1 << 14, 1 << 13
    x = synth.outlier_tensor_torch(rows * cols, 5, DEV, outlier_frac=0.01 if values == "outliers" else 0.0).view(rows, cols)
    if values == "half zero":
        x = x.clamp_(min=0.0)
    elif values == "40 binades":
        x *= torch.exp2(-40 * torch.rand(rows, cols, device=DEV, generator=torch.Generator(DEV).manual_seed(6)))
    x = x.to(torch.bfloat16) if bf16 else x
    out = torch.empty(rows * cols, dtype=torch.uint8, device=DEV)
    q = {k: L.Quant(k, L.sr_absmax_scale(x, k), 3) for k in (L.E4M2, L.E4M3, L.E5M2)}
    us = _us_in_turn([lambda k=k: L.sr_quantize(x, q[k], transpose_out=transpose, out=out) for k in q])
    say("us of E4M2, E4M3, E5M2", bf16, transpose, values, us)
    assert max(us[1:]) <= 1.1 * us[0]


# Inf and NaN of every payload take no part, beside the largest finite value, in either half of a bfloat16 word; values whose
# neighbour in that word has all its bits set; nothing but Inf and NaN; batched and alone
@pytest.mark.parametrize("n", [2, 9, 4103, 65536, 262159])
@pytest.mark.parametrize("bf16", [False, True])
def test_absmax_scale_of_finite_values_beside_others(n, bf16):
    bits = [0x7F800000, 0xFF800000, 0x7FFF0000, 0xFF810000, 0x7FC00000, 0xFFFF0000]
    if not bf16:
        bits += [0x7F800001, 0xFFFFFFFF]
    others = np.array(bits, np.uint32).view(np.float32)
    for big in (np.uint32(0x7F7F0000).view(np.float32), np.float32(1.0), np.float32(2.0 ** -130), None):
        for at in (0, 1, n // 2, n - 1):
            y = np.resize(others, n)
            if big is not None:
                y[at] = -big if at % 2 else big
                y[(at + 1) % n] = np.float32(0.0) if at % 3 else others[-1]
            say("absmax beside Inf and NaN", n, "bf16" if bf16 else "f32", big, at)
            high = (y.view(np.uint32) >> 16).astype(np.uint16).view(np.int16)
            x = torch.from_numpy(high).view(torch.bfloat16).to(DEV) if bf16 else to_dev(y)
            want = 1.0 if big is None else max(float(np.float32(big) / np.float32(127)), 2.0 ** -100)
            out = torch.empty(1, device=DEV)
            L.sr_absmax_scales([(x, L.INT8, out)])
            assert float(L.sr_absmax_scale(x, L.INT8).item()) == want and float(out.item()) == want


@pytest.mark.parametrize("kind", [L.INT8, L.E5M2, L.E4M3])
def test_vanishing_tensor_gets_the_floored_scale_not_saturation(kind):
    # max|x| / Qmax below 2^-100: both absmax entry points floor the step there, and the codes
    # quantized with that device-resident scale are the oracle's (zeros and nearest neighbours)
    x = synth.gaussian((4096,), 2.0 ** -118, 7).astype(np.float32)
    xd = to_dev(x)
    want = oracle.absmax_scale(x, kind)
    assert want == 2.0 ** -100
    s1 = L.sr_absmax_scale(xd, kind)
    s2 = torch.empty(1, device=DEV)
    L.sr_absmax_scales([(xd, kind, s2)])
    assert float(s1.item()) == want and float(s2.item()) == want
    got = L.sr_quantize(xd, L.Quant(kind, s1, seed=4)).cpu().numpy()
    assert np.array_equal(got, oracle_codes(xd, kind, want, 4, 0))
    assert np.abs(oracle.decode_array(kind, got)).max() <= 1.0   # nowhere near Qmax


def test_batched_absmax_shares_passes_and_matches_oracle():
    A = to_dev(synth.gaussian((512, 96), 1.0, 1))
    W = to_dev(synth.gaussian((64, 96), 0.02, 2), bf16=True)
    dY = to_dev(synth.outlier_tensor_np(512 * 64, 3).reshape(512, 64))
    Z = torch.zeros(48, device=DEV)
    outs = torch.empty(6, device=DEV)
    reqs = [(A, L.INT8, outs[0:1]), (W, L.INT8, outs[1:2]), (A, L.E5M2, outs[2:3]), (W, L.E4M3, outs[3:4]),
            (dY, L.INT4, outs[4:5]), (Z, L.INT8, outs[5:6])]
    batch = L.AbsmaxBatch(reqs)
    for _ in range(2):   # the workspace needs no clearing between calls
        batch.run()
        got = outs.cpu().numpy()
        want = [oracle.absmax_scale(host_src(x), k) for x, k, _ in reqs]
        assert [float(g) for g in got] == want


def test_absmax_of_zeros_and_empty():
    z = torch.zeros(4096, device=DEV)
    assert float(L.sr_absmax_scale(z, L.INT8).item()) == 1.0
    e = torch.zeros(0, device=DEV)
    assert float(L.sr_absmax_scale(e, L.E4M3).item()) == 1.0
    out = L.sr_quantize(e, L.Quant(L.INT8, 1.0))
    assert out.numel() == 0


def test_statistics_on_gpu_match_the_paper_example():
    # 0.7 on the integer grid: up with probability 0.7 (worked example after Def. 3)
    x = torch.full((1 << 20,), 0.7, device=DEV)
    codes = L.sr_quantize(x, L.Quant(L.INT8, 1.0, seed=123)).cpu().numpy()
    assert set(np.unique(codes)) == {0, 1}
    assert abs(codes.mean() - 0.7) < 5 * np.sqrt(0.21 / codes.size)
    rtn = L.sr_quantize(x, L.Quant(L.INT8, 1.0, round_mode=L.RTN)).cpu().numpy()
    assert np.all(rtn == 1)


@pytest.mark.parametrize("kind", [L.INT8, L.INT4, L.E4M3, L.E5M2, L.E4M1])
def test_full_size_standalone_quantize_bit_exact(kind):
    # the 2^28-element workload of the standalone quantizer, in the launch shape bench.py times
    n = 1 << 28
    say("full-size", L.KIND_NAMES[kind], "generate")
    xd = synth.outlier_tensor_torch(n, 1234, DEV)
    s_dev = L.sr_absmax_scale(xd, kind)
    got = L.sr_quantize(xd, L.Quant(kind, s_dev, seed=42, counter_offset=1 << 40))
    torch.cuda.synchronize()
    x = xd.cpu().numpy()
    del xd
    say("full-size", L.KIND_NAMES[kind], "oracle")
    scale = oracle.absmax_scale(x, kind)
    assert float(s_dev.item()) == scale
    want = oracle.quantize(x, kind, scale, 42, 1 << 40)
    if kind == L.INT4:
        want = oracle.pack_int4(want)
    got = got.cpu().numpy()
    assert np.array_equal(got, want)


def test_more_than_2_to_32_elements():
    # element indices and Philox block numbers past 32 bits: 2^32 + 2^20 elements (17 GB of
    # binary32), checked on the slices around index 2^32 and at the end; the scale must find a
    # maximum planted past index 2^32
    n = (1 << 32) + (1 << 20)
    say("2^32 + 2^20 elements: generate")
    xd = torch.empty(n, dtype=torch.float32, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(77)
    for i in range(0, n, 1 << 30):
        xd[i:i + (1 << 30)].normal_(generator=g)
    xd[(1 << 32) + 12345] = -1000.0
    for kind in (L.INT8, L.INT4):
        s_dev = L.sr_absmax_scale(xd, kind)
        assert float(s_dev.item()) == float(np.float32(1000.0) / np.float32(oracle.qmax(kind)))
        batched = torch.empty(1, device=DEV)
        L.sr_absmax_scales([(xd, kind, batched)])
        assert torch.equal(batched, s_dev)
        scale = float(s_dev.item()) / 64  # a finer step than the planted maximum allows: more codes in use
        seed, off = 9, (1 << 63) - 5         # the block counter also crosses 2^63 here
        got = L.sr_quantize(xd, L.Quant(kind, scale, seed=seed, counter_offset=off))
        torch.cuda.synchronize()
        per_byte = 2 if kind == L.INT4 else 1
        for lo, hi in (((1 << 32) - (1 << 19), (1 << 32) + (1 << 19)), (n - (1 << 20), n), (0, 1 << 16)):
            x = xd[lo:hi].cpu().numpy()
            want = oracle.quantize(x, kind, scale, seed, off + lo // 8)
            if kind == L.INT4:
                want = oracle.pack_int4(want)
            assert np.array_equal(got[lo // per_byte:hi // per_byte].cpu().numpy(), want), (L.KIND_NAMES[kind], lo)
        del got
    # the same tensor as 65552 x 65536, transposed output: source rows past element 2^32 are the
    # last columns of the result
    rows, cols = 65552, 65536
    scale, seed, off = 0.125, 4, 1 << 50
    got = L.sr_quantize(xd.view(rows, cols), L.Quant(L.INT8, scale, seed=seed, counter_offset=off), transpose_out=True)
    torch.cuda.synchronize()
    for r in (0, 65535, 65536, 65551):
        want = oracle.quantize(xd[r * cols:(r + 1) * cols].cpu().numpy(), L.INT8, scale, seed, off + r * cols // 8)
        assert np.array_equal(got.view(cols, rows)[:, r].cpu().numpy(), want), r
