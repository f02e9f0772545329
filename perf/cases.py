"""Workloads for timing the SR-quantized linear layer through its public entry points.

`listed()` names the fixed cases, `draw(rng)` makes further ones of the same ranges, and
`prepare` / `run` / `work` / `tolerance` take any of them.  A case is a dict of plain values; "op" says
which use of the library it stands for:

  fwd          serving or a small layer: the scale of A, then Y = Q(A) Q(W)^T; W's scale is kept
  step         training step of one linear with the activation saved as codes: five scales, forward
               pass that writes the stash, backward pass that reads it
  step_plain   the same without a stash (formats the stash does not take): forward, then backward
  block        the linears of an MLP block in one step on two streams, the memory-bound half of every
               linear beside the products of the one before
  weight_only  quantized weights, full-precision activations and gradients: Y and dA
  quantize     one tensor: its scale, then its codes, in its own layout or transposed
  module       SRLinear through autograd: micro-batches forward and backward, then the weight update

Tokens are M, out features N, in features K.
"""
import math

import torch

from paper_2511_00874_amd import lib as L
from paper_2511_00874_amd import synth, train

DEV = "cuda:0"

# format sets of a training step: (forward A and W, backward A and W, output gradient)
FORMATS = {
    "int8_int4": (L.INT8, L.INT8, L.INT4),    # 8-bit integers, 4-bit output gradient
    "int8_e5m2": (L.INT8, L.E5M2, L.E5M2),    # integers forward, E5M2 backward, exact products
    "int8_e5m2_f8": (L.INT8, L.E5M2, L.E5M2),  # the same on the fp8 matrix pipeline
    "e4m3": (L.E4M3, L.E4M3, L.E4M3),         # E4M3 throughout, exact products
    "e4m3_e5m2": (L.E4M3, L.E4M3, L.E5M2),    # E4M3 with an E5M2 output gradient
}
STASHED = ("int8_int4", "int8_e5m2", "int8_e5m2_f8")
KINDS = {"int8": L.INT8, "int4": L.INT4, "e4m3": L.E4M3, "e5m2": L.E5M2, "e4m1": L.E4M1}
BLOCKS = {"gpt2": [(3072, 768), (768, 3072)], "llama": [(5632, 2048), (5632, 2048), (2048, 5632)]}
LR = 1e-4


def listed():
    return [
        # the smallest call: one small layer, where the launches are all there is
        {"name": "fwd_single_layer", "op": "fwd", "M": 64, "N": 128, "K": 128, "kind": "int8", "w_bf16": False},
        # a few sequences through a wide layer with bfloat16 weights
        {"name": "fwd_serve_wide", "op": "fwd", "M": 32, "N": 5632, "K": 2048, "kind": "int8", "w_bf16": True},
        # a short, ragged batch of the GPT-2 MLP
        {"name": "step_gpt2_fc1_ragged", "op": "step", "M": 1008, "N": 3072, "K": 768, "formats": "int8_e5m2",
         "w_bf16": False},
        # the GPT-2 MLP at its training batch (8 sequences of 1024)
        {"name": "step_gpt2_fc2", "op": "step", "M": 8192, "N": 768, "K": 3072, "formats": "int8_e5m2",
         "w_bf16": False},
        # an attention projection of the Llama-shaped layer on the smallest batch of the token sweep
        {"name": "step_llama_qkvo_4k", "op": "step", "M": 4096, "N": 2048, "K": 2048, "formats": "int8_int4",
         "w_bf16": True},
        # the largest: the down projection at the largest single-GPU batch
        {"name": "step_llama_down_64k", "op": "step", "M": 65536, "N": 2048, "K": 5632, "formats": "int8_int4",
         "w_bf16": True},
        # the 4-exponent-bit floats of the paper's experiments
        {"name": "step_e4m3_4k", "op": "step_plain", "M": 4096, "N": 2048, "K": 2048, "formats": "e4m3",
         "w_bf16": True},
        # a whole MLP block on two streams
        {"name": "block_llama_mlp_8k", "op": "block", "M": 8192, "block": "llama", "formats": "int8_int4",
         "w_bf16": True},
        # weight-only objective on the GPT-2 MLP, binary32 activations and gradients
        {"name": "weight_only_gpt2_fc1", "op": "weight_only", "M": 8192, "N": 3072, "K": 768, "kind": "int8",
         "a_bf16": False, "w_bf16": True},
        # a large tensor with outliers, the standalone quantizer's benchmark
        {"name": "quantize_int8_2p28", "op": "quantize", "rows": 1, "cols": 1 << 28, "kind": "int8", "bf16": False,
         "transpose": False, "rtn": False},
        # an odd matrix turned on the way
        {"name": "quantize_e5m2_turned", "op": "quantize", "rows": 12289, "cols": 3080, "kind": "e5m2", "bf16": True,
         "transpose": True, "rtn": False},
        # the autograd face: two micro-batches and the update
        {"name": "module_qkvo_micro2", "op": "module", "M": 4096, "N": 2048, "K": 2048, "micro": 2,
         "objective": "five"},
    ]


def _log_int(rng, lo, hi, multiple):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(multiple, int(v / multiple + 0.5) * multiple)


LARGEST = 65536.0 * 2048 * 5632  # M N K of the largest listed case


def draw(rng):
    op = rng.choice(["fwd", "fwd", "step", "step", "step", "step", "step_plain", "step_plain", "block", "weight_only",
                     "quantize", "quantize", "module"])
    if op == "fwd":
        return {"op": op, "M": _log_int(rng, 16, 512, 16), "N": _log_int(rng, 128, 5632, 16),
                "K": _log_int(rng, 128, 5632, 16), "kind": rng.choice(["int8", "int8", "e5m2", "e4m3"]),
                "w_bf16": rng.random() < 0.5}
    if op in ("step", "step_plain"):
        while True:
            M, N, K = _log_int(rng, 64, 65536, 16), _log_int(rng, 256, 5632, 16), _log_int(rng, 256, 5632, 16)
            if M * N * K <= (LARGEST if op == "step" else LARGEST / 4):
                break
        return {"op": op, "M": M, "N": N, "K": K,
                "formats": rng.choice(list(STASHED)) if op == "step" else rng.choice(["e4m3", "e4m3_e5m2", "int8_e5m2"]),
                "w_bf16": rng.random() < 0.5}
    if op == "block":
        return {"op": op, "M": _log_int(rng, 512, 16384, 16), "block": rng.choice(["gpt2", "llama"]),
                "formats": rng.choice(["int8_int4", "int8_e5m2"]), "w_bf16": rng.random() < 0.5}
    if op == "weight_only":
        return {"op": op, "M": _log_int(rng, 256, 16384, 16), "N": _log_int(rng, 256, 4096, 16),
                "K": _log_int(rng, 256, 4096, 16), "kind": rng.choice(["int8", "int4", "e4m3"]),
                "a_bf16": rng.random() < 0.3, "w_bf16": rng.random() < 0.7}
    if op == "module":
        return {"op": op, "M": _log_int(rng, 256, 16384, 16), "N": _log_int(rng, 256, 4096, 16),
                "K": _log_int(rng, 256, 4096, 16), "micro": rng.choice([1, 2, 4]),
                "objective": rng.choice(["five", "five", "qat"])}
    transpose = rng.random() < 0.4
    kind = rng.choice(["int8", "int4", "e4m3", "e5m2", "e4m1"])
    if transpose:
        rows, cols = _log_int(rng, 64, 65536, 2 if kind == "int4" else 1), _log_int(rng, 64, 4096, 8)
    else:
        rows, cols = 1, _log_int(rng, 1 << 12, 1 << 28, 2 if kind == "int4" else 1)
    return {"op": "quantize", "rows": rows, "cols": cols, "kind": kind, "bf16": rng.random() < 0.4,
            "transpose": transpose, "rtn": rng.random() < 0.2}


class _Linear:
    """Tensors, scales, quantizers, outputs and workspaces of one linear in a training step."""

    def __init__(self, M, N, K, formats, w_bf16, seed, stash):
        fwd, bwd, grad = FORMATS[formats]
        flag = L.FLAG_F8_PIPELINE if formats.endswith("_f8") else 0
        self.K, self.stashed = K, stash
        self.A = synth.gaussian_torch((M, K), 1.0, seed, DEV)
        self.W = synth.gaussian_torch((N, K), 0.02, seed + 1, DEV, torch.bfloat16 if w_bf16 else None)
        self.dY = synth.gaussian_torch((M, N), 1e-3, seed + 2, DEV)
        self.scales = torch.empty(5, dtype=torch.float32, device=DEV)
        self.q, requests, offset = [], [], 0
        for i, (t, kind) in enumerate(((self.A, fwd), (self.W, fwd), (self.A, bwd), (self.W, bwd), (self.dY, grad))):
            s = self.scales[i:i + 1]
            self.q.append(L.Quant(kind, s, seed=seed, counter_offset=offset, flags=flag if i >= 2 else 0))
            requests.append((t, kind, s))
            offset += (t.numel() + 7) // 8
        self.absmax = L.AbsmaxBatch(requests)
        self.Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
        self.dA = torch.empty((M, K), dtype=torch.float32, device=DEV)
        self.dW = torch.empty((N, K), dtype=torch.float32, device=DEV)
        ops = (L.OP_FWD_STASH, L.OP_BWD_STASHED) if stash else (L.OP_FWD, L.OP_BWD)
        self.ws_fwd, self.ws_bwd = (torch.empty(L.sr_linear_workspace_bytes(op, M, N, K), dtype=torch.uint8, device=DEV)
                                    for op in ops)
        self.stash = torch.empty(L.sr_linear_stash_bytes(M, N, K), dtype=torch.uint8, device=DEV) if stash else None

    def forward(self, phase=L.PHASE_BOTH):
        qA, qW, qAb, qWb, _ = self.q
        if self.stashed:
            L.sr_linear_fwd_stash(self.A, self.W, qA, qW, qAb, qWb, stash=self.stash, out=self.Y,
                                  workspace=self.ws_fwd, phase=phase)
        else:
            L.sr_linear_fwd(self.A, self.W, qA, qW, out=self.Y, workspace=self.ws_fwd)

    def backward(self, phase=L.PHASE_BOTH):
        _, _, qAb, qWb, qdY = self.q
        if self.stashed:
            L.sr_linear_bwd_stashed(self.dY, self.stash, self.K, qdY, qWb, qAb, out_dA=self.dA, out_dW=self.dW,
                                    workspace=self.ws_bwd, phase=phase)
        else:
            L.sr_linear_bwd(self.dY, self.W, self.A, qdY, qWb, qAb, out_dA=self.dA, out_dW=self.dW,
                            workspace=self.ws_bwd)

    def outputs(self):
        return self.Y, self.dA, self.dW


class _Bag:
    pass


def prepare(case, seed):
    op = case["op"]
    if op in ("step", "step_plain"):
        return op, _Linear(case["M"], case["N"], case["K"], case["formats"], case["w_bf16"], seed, op == "step")
    if op == "block":
        s = _Bag()
        s.layers = [_Linear(case["M"], N, K, case["formats"], case["w_bf16"], seed + 100 * i, True)
                    for i, (N, K) in enumerate(BLOCKS[case["block"]])]
        s.mem, s.mat = torch.cuda.Stream(), torch.cuda.Stream()
        s.events = [(torch.cuda.Event(), torch.cuda.Event()) for _ in s.layers]
        return op, s
    s = _Bag()
    if op == "quantize":
        n = case["rows"] * case["cols"]
        s.x = synth.outlier_tensor_torch(n, seed, DEV)
        if case["bf16"]:
            s.x = s.x.to(torch.bfloat16)
        if case["rows"] > 1:
            s.x = s.x.view(case["rows"], case["cols"])
        s.kind, s.transpose = KINDS[case["kind"]], case["transpose"]
        s.scale = torch.empty(1, dtype=torch.float32, device=DEV)
        s.q = L.Quant(s.kind, s.scale, seed=seed, counter_offset=1 << 40, round_mode=L.RTN if case["rtn"] else L.SR)
        s.codes = torch.empty(n // 2 if s.kind == L.INT4 else n, dtype=torch.uint8, device=DEV)
        return op, s
    M, N, K = case["M"], case["N"], case["K"]
    if op == "module":
        s.layer = train.SRLinear(K, N, seed, device=DEV, objective=case["objective"])
        s.x = [synth.gaussian_torch((M, K), 1.0, seed + 10 + 2 * i, DEV).requires_grad_() for i in range(case["micro"])]
        s.dy = [synth.gaussian_torch((M, N), 1e-3, seed + 11 + 2 * i, DEV) for i in range(case["micro"])]
        return op, s
    kind = KINDS[case["kind"]]
    s.A = synth.gaussian_torch((M, K), 1.0, seed, DEV, torch.bfloat16 if case.get("a_bf16") else None)
    s.W = synth.gaussian_torch((N, K), 0.02, seed + 1, DEV, torch.bfloat16 if case["w_bf16"] else None)
    s.sw = L.sr_absmax_scale(s.W, kind)
    s.qW = L.Quant(kind, s.sw, seed=seed, counter_offset=(M * K + 7) // 8)
    s.Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    if op == "fwd":
        s.kind, s.sa = kind, torch.empty(1, dtype=torch.float32, device=DEV)
        s.qA = L.Quant(kind, s.sa, seed=seed)
        s.ws = torch.empty(L.sr_linear_workspace_bytes(L.OP_FWD, M, N, K), dtype=torch.uint8, device=DEV)
        return op, s
    s.dY = synth.gaussian_torch((M, N), 1e-3, seed + 2, DEV, torch.bfloat16 if case["a_bf16"] else None)
    s.dA = torch.empty((M, K), dtype=torch.float32, device=DEV)
    s.ws = torch.empty(max(L.sr_linear_workspace_bytes(o, M, N, K)
                           for o in (L.OP_FWD_WEIGHT_ONLY, L.OP_BWD_DATA_WEIGHT_ONLY)), dtype=torch.uint8, device=DEV)
    return op, s


def run(state):
    op, s = state
    if op == "fwd":
        L.sr_absmax_scale(s.A, s.kind, out=s.sa)
        return L.sr_linear_fwd(s.A, s.W, s.qA, s.qW, out=s.Y, workspace=s.ws)
    if op in ("step", "step_plain"):
        s.absmax.run()
        s.forward()
        s.backward()
        return s.outputs()
    if op == "block":
        cur = torch.cuda.current_stream()
        s.mem.wait_stream(cur)
        s.mat.wait_stream(cur)
        for layer, (forward_ready, backward_ready) in zip(s.layers, s.events):
            with torch.cuda.stream(s.mem):
                layer.absmax.run()
                layer.forward(L.PHASE_QUANTIZE)
                forward_ready.record()
                layer.backward(L.PHASE_QUANTIZE)
                backward_ready.record()
            with torch.cuda.stream(s.mat):
                s.mat.wait_event(forward_ready)
                layer.forward(L.PHASE_PRODUCT)
                s.mat.wait_event(backward_ready)
                layer.backward(L.PHASE_PRODUCT)
        cur.wait_stream(s.mem)
        cur.wait_stream(s.mat)
        return [layer.outputs() for layer in s.layers]
    if op == "quantize":
        L.sr_absmax_scale(s.x, s.kind, out=s.scale)
        return L.sr_quantize(s.x, s.q, transpose_out=s.transpose, out=s.codes), s.scale
    if op == "weight_only":
        L.sr_linear_fwd(s.A, s.W, train.NOQ, s.qW, out=s.Y, workspace=s.ws)
        L.sr_linear_bwd_data(s.dY, s.W, train.NOQ, s.qW, out=s.dA, workspace=s.ws)
        return s.Y, s.dA
    results = []
    for x, dy in zip(s.x, s.dy):
        y = s.layer(x)
        results.append((y.detach(), torch.autograd.grad(y, x, dy)[0]))
    s.layer.update(LR)
    return results, s.layer.dW, s.layer.weight


def work(case):
    op = case["op"]
    if op == "quantize":
        n = case["rows"] * case["cols"]
        return {"bytes": n * (2 if case["bf16"] else 4) + (n // 2 if case["kind"] == "int4" else n), "flops": 0}
    if op == "block":
        shapes = [(case["M"], N, K) for N, K in BLOCKS[case["block"]]]
    else:
        shapes = [(case["M"], case["N"], case["K"])] * case.get("micro", 1)
    total = {"bytes": 0, "flops": 0}
    for M, N, K in shapes:
        ea, ew = 2 if case.get("a_bf16") else 4, 2 if case.get("w_bf16") else 4
        if op == "fwd":
            total["bytes"] += ea * M * K + ew * N * K + 4 * M * N
            total["flops"] += 2 * M * N * K
        elif op == "weight_only":
            total["bytes"] += ea * (M * K + M * N) + ew * N * K + 4 * (M * N + M * K)
            total["flops"] += 4 * M * N * K
        else:  # A, W, dY in, Y, dA, dW out
            total["bytes"] += 4 * 2 * (M * K + M * N) + ew * N * K + 4 * N * K
            total["flops"] += 6 * M * N * K
    if op == "module":  # one gradient buffer and one weight for all micro-batches; the update reads and writes it
        N, K, micro = case["N"], case["K"], case["micro"]
        total["bytes"] += N * K * (4 + 2 + 2 - (4 + 4) * micro)
    return total


def tolerance(case):
    """About four times what the path differs by from the binary64 product of the same operands (the
    contraction length at most 16384; it grows like its square root)."""
    op = case["op"]
    if op == "quantize":
        return "exact"
    if op == "weight_only":  # three bfloat16 planes per activation: 3.6e-7, largest 2.5e-6
        return {"rel": 1.5e-6, "max": 1e-5}
    if op == "module":  # sums as below; a weight on the edge between two bfloat16 numbers may take the other one
        return {"rel": 2e-5, "max": 1e-2}
    kinds = [KINDS[case["kind"]]] if op == "fwd" else FORMATS[case["formats"]]
    if all(k in (L.INT8, L.INT4) for k in kinds):
        return "exact"  # integer sums, one scaling
    if case.get("formats", "").endswith("_f8"):  # the fp8 pipeline aligns groups of products: 9e-6, largest 1.2e-4
        return {"rel": 4e-5, "max": 5e-4}
    return {"rel": 8e-7, "max": 4e-6}  # exact products, binary32 sums: 1e-7, largest 6e-7


# ---- the same in 64 bits, from the definition: nothing below uses the package's arithmetic --------------
# kind: (fraction bits, smallest exponent, largest value); integer grids have spacing 1
_GRID = {L.INT8: (None, 0, 127.0), L.INT4: (None, 0, 7.0), L.E4M3: (3, -6, 448.0), L.E5M2: (2, -14, 57344.0)}


def _r16(n, seed, offset):
    """16 random bits of elements 0 .. n-1: Philox4x32-10, block offset + i // 8, slice i % 8."""
    low = 0xFFFFFFFF
    block = torch.arange((n + 7) // 8, dtype=torch.int64, device=DEV) + offset
    c0, c1 = block & low, (block >> 32) & low
    c2, c3 = torch.zeros_like(c0), torch.zeros_like(c0)
    k0, k1 = seed & low, (seed >> 32) & low
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # modulo 2^64: the high half is exact after the mask
        c0, c1, c2, c3 = ((p1 >> 32) & low) ^ c1 ^ k0, p1 & low, ((p0 >> 32) & low) ^ c3 ^ k1, p0 & low
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return torch.stack([w >> s & 0xFFFF for w in (c0, c1, c2, c3) for s in (0, 16)], 1).reshape(-1)[:n]


def _scale(x, kind):
    return float((x.abs().max().float().cpu() / _GRID[kind][2]).item())


def _quantized(x, kind, seed, offset):
    """x on its grid, in binary64 (scale included)."""
    m, emin, qmax = _GRID[kind]
    s = _scale(x, kind)
    inv = float((torch.tensor(1.0) / torch.tensor(s)).item())
    t = (x.float() * inv).clamp(-qmax, qmax).double()
    d = 1.0 if m is None else torch.exp2((torch.frexp(t).exponent - 1).clamp(min=emin).double() - m)
    y = t / d
    low = y.floor()
    eps = (_r16(x.numel(), seed, offset).view(x.shape).double() + 0.5) / 65536
    return (low + (y - low >= eps)) * d * s


def _exact_step(M, N, K, formats, w_bf16, seed):
    fwd, bwd, grad = FORMATS[formats]
    A = synth.gaussian_torch((M, K), 1.0, seed, DEV)
    W = synth.gaussian_torch((N, K), 0.02, seed + 1, DEV, torch.bfloat16 if w_bf16 else None)
    dY = synth.gaussian_torch((M, N), 1e-3, seed + 2, DEV)
    q, offset = [], 0
    for t, kind in ((A, fwd), (W, fwd), (A, bwd), (W, bwd), (dY, grad)):
        q.append(_quantized(t, kind, seed, offset))
        offset += (t.numel() + 7) // 8
    return q[0] @ q[1].t(), q[4] @ q[3], q[4].t() @ q[2]


def _exact_module(case, seed):
    M, N, K = case["M"], case["N"], case["K"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    W = (torch.randn((N, K), device=DEV, generator=g) * 0.02).to(torch.bfloat16)
    qat = case["objective"] == "qat"
    results, dW, position, wb, ab = [], 0.0, 0, (N * K + 7) // 8, (M * K + 7) // 8
    for i in range(case["micro"]):
        x = synth.gaussian_torch((M, K), 1.0, seed + 10 + 2 * i, DEV)
        dy = synth.gaussian_torch((M, N), 1e-3, seed + 11 + 2 * i, DEV)
        if qat:
            wq = _quantized(W, L.E5M2, seed, position)
            y, a = x.double() @ wq.t(), _quantized(x, L.E5M2, seed, position + wb)
            position += wb + ab
        else:
            y = _quantized(x, L.INT8, seed, position + wb) @ _quantized(W, L.INT8, seed, position).t()
            a = _quantized(x, L.E5M2, seed, position + wb + ab)
            wq = _quantized(W, L.E5M2, seed, position + wb + 2 * ab)
            position += 2 * wb + 2 * ab
        d = _quantized(dy, L.E5M2, seed, position)
        position += (M * N + 7) // 8
        results.append((y, d @ wq))
        dW = dW + d.t() @ a
    return results, dW, None  # the weight is rounded to bfloat16 with random thresholds


def exact(case, seed):
    op = case["op"]
    if op == "quantize":
        n = case["rows"] * case["cols"]
        x = synth.outlier_tensor_torch(n, seed, DEV)
        if case["bf16"]:
            x = x.to(torch.bfloat16)
        qmax = {"int8": 127.0, "int4": 7.0, "e4m3": 448.0, "e5m2": 57344.0, "e4m1": 384.0}[case["kind"]]
        return None, (x.abs().max().double() / qmax).view(1)
    if op in ("step", "step_plain"):
        return _exact_step(case["M"], case["N"], case["K"], case["formats"], case["w_bf16"], seed)
    if op == "block":
        return [_exact_step(case["M"], N, K, case["formats"], case["w_bf16"], seed + 100 * i)
                for i, (N, K) in enumerate(BLOCKS[case["block"]])]
    if op == "module":
        return _exact_module(case, seed)
    M, N, K, kind = case["M"], case["N"], case["K"], KINDS[case["kind"]]
    A = synth.gaussian_torch((M, K), 1.0, seed, DEV, torch.bfloat16 if case.get("a_bf16") else None)
    W = synth.gaussian_torch((N, K), 0.02, seed + 1, DEV, torch.bfloat16 if case["w_bf16"] else None)
    wq = _quantized(W, kind, seed, (M * K + 7) // 8)
    if op == "fwd":
        return _quantized(A, kind, seed, 0) @ wq.t()
    dY = synth.gaussian_torch((M, N), 1e-3, seed + 2, DEV, torch.bfloat16 if case["a_bf16"] else None)
    return A.double() @ wq.t(), dY.double() @ wq
