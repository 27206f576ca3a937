"""Performance cases of the fused low-bit linear: what a user's program has the
library do, through the Python binding of the C ABI, over the sizes it is used
at.

Every case draws its inputs on the GPU from the seed (synth.device_layer: the
token streams, outlier channels, channel scaling and gains of a world-action
DiT's linears), prepares the int4 weights once as a program does when it loads
a model, and allocates the workspace and outputs a program keeps.

kinds
  layer    one fused linear (sq_linear_w4a8 / sq_linear_w4a4), called eagerly
  block    the four linears (qkv, out, up, down) of `layers` DiT blocks, every
           block with its own weights.  With graph = True the calls are one
           captured HIP graph, as a serving loop with few tokens per call runs
           them; else they are called eagerly
  chain    the MLP's direct chain: the up projection whose epilogue applies
           GELU and writes the down projection's codes, then the down
           projection's GEMM
  calib    activation calibration of one linear (Eq. 9): the fp64 target, then
           the objective of a batch of candidates
  scaling  shared channel scaling of one linear (Eq. 7): the full-precision
           target, then the objective of a list of exponents, weights packed
           for each

fields: tokens (rows), hidden / mlp or K / N, bits (of the activations), group
(input channels per weight step; 0: one step per output channel), static
(per-step threshold instead of a per-token range), out (output type).
"""
from __future__ import annotations

import math

import torch

from paper_2609_39056_amd import binding as B
from paper_2609_39056_amd import synth

STEPS = 10  # denoising steps of the gain tables
STEP = 3    # the step that is run
OUT = {"f32": B.SQ_OUT_F32, "bf16": B.SQ_OUT_BF16, "f16": B.SQ_OUT_F16}


def listed():
    return [
        # the smallest call: the 256 x 256 layer of the tests, one eager call
        dict(name="tiny_layer", kind="layer", tokens=88, K=256, N=256, bits=8, group=128, static=False, out="bf16"),
        # a denoising step that runs the action tokens only: 28 blocks of the 2B class, weights from HBM
        dict(name="action_2b", kind="block", layers=28, graph=True, tokens=64, hidden=2048, mlp=8192, bits=8,
             group=128, static=False, out="bf16"),
        # the same with 4-bit activations and the most tokens that still count as few
        dict(name="action_2b_a4", kind="block", layers=28, graph=True, tokens=128, hidden=2048, mlp=8192, bits=4,
             group=128, static=False, out="bf16"),
        # a batch of 8 samples' proprioception and action tokens: between the few-token and the large regime
        dict(name="batch_2b", kind="block", layers=7, graph=True, tokens=768, hidden=2048, mlp=8192, bits=8, group=128,
             static=False, out="bf16"),
        # one 2B-class block, one sample: 4096 video + 32 proprioception + 64 action tokens
        dict(name="block_2b", kind="block", layers=1, graph=False, tokens=4192, hidden=2048, mlp=8192, bits=8,
             group=128, static=False, out="bf16"),
        # the same in W4A4
        dict(name="block_2b_a4", kind="block", layers=1, graph=False, tokens=4192, hidden=2048, mlp=8192, bits=4,
             group=128, static=False, out="bf16"),
        # the benchmark's block: 14B class, 8192 + 64 + 128 tokens
        dict(name="block_14b", kind="block", layers=1, graph=False, tokens=8384, hidden=5120, mlp=13824, bits=8,
             group=128, static=False, out="bf16"),
        # the same with the paper's weight format, one step per output channel, and its static ranges
        dict(name="block_14b_channel", kind="block", layers=1, graph=False, tokens=8384, hidden=5120, mlp=13824,
             bits=8, group=0, static=True, out="bf16"),
        # a column shard (one of 8) of the 14B up projection, an odd token count, fp32 out
        dict(name="shard_odd", kind="layer", tokens=2731, K=5120, N=1728, bits=8, group=128, static=False, out="f32"),
        # up -> GELU -> down of the 2B class in one chain
        dict(name="chain_2b", kind="chain", tokens=4192, hidden=2048, mlp=8192, bits=8, group=128, out="bf16"),
        # calibration of the 2B up projection, one step per channel, a batch of candidates (offline)
        dict(name="calib_2b", kind="calib", tokens=4192, K=2048, N=8192, bits=8, group=0, candidates=16),
        # the channel scaling's objective over exponents for the 2B output projection, W4A4 (offline)
        dict(name="scaling_2b", kind="scaling", tokens=1048, K=2048, N=2048, bits=4, group=128, exponents=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: token counts from 1 to 8384, channels from
    256 to 13824, both activation widths, weight groups and output types."""
    kind = rng.choice(["layer", "layer", "layer", "block", "block", "chain", "calib", "scaling"])
    bits, group = rng.choice([8, 8, 4]), rng.choice([128, 128, 0])
    if kind == "layer":
        return dict(kind=kind, tokens=_log_int(rng, 1, 8384), K=128 * _log_int(rng, 2, 108),
                    N=64 * _log_int(rng, 4, 216), bits=bits, group=group, static=rng.random() < 0.3,
                    out=rng.choice(["bf16", "bf16", "f32", "f16"]))
    if kind == "block":
        few = rng.random() < 0.6
        hidden = rng.choice([1024, 1536, 2048, 2560])
        return dict(kind=kind, layers=4 if few else 1, graph=few,
                    tokens=_log_int(rng, 16, 1024) if few else _log_int(rng, 1024, 6000), hidden=hidden,
                    mlp=hidden * rng.choice([3, 4]), bits=bits, group=group, static=rng.random() < 0.3, out="bf16")
    if kind == "chain":
        hidden = rng.choice([1024, 1536, 2048, 3072])
        return dict(kind=kind, tokens=_log_int(rng, 16, 6000), hidden=hidden, mlp=hidden * rng.choice([3, 4]),
                    bits=bits, group=group, out=rng.choice(["bf16", "f32"]))
    K, N = 128 * _log_int(rng, 4, 32), 64 * _log_int(rng, 8, 64)
    tokens = _log_int(rng, 200, 4192)
    if kind == "calib":
        return dict(kind=kind, tokens=tokens, K=K, N=N, bits=bits, group=group, candidates=rng.randint(2, 16))
    return dict(kind=kind, tokens=tokens, K=K, N=N, bits=bits, group=group, exponents=rng.randint(2, 8))


# ------------------------------------------------------------------ inputs
def _streams(tokens):
    """(video, proprioception, action) tokens: few tokens are the action
    stream alone, more are mixed as in the 2B and 14B configurations."""
    if tokens <= 128:
        return (0, 0, tokens)
    proprio, action = tokens // 131, tokens // 65
    return (tokens - proprio - action, proprio, action)


def _linears(case):
    """(K, N) of every linear of the case, in call order."""
    if case["kind"] == "block":
        h, m = case["hidden"], case["mlp"]
        return [(h, 3 * h), (h, h), (h, m), (m, h)] * case["layers"]
    if case["kind"] == "chain":
        return [(case["hidden"], case["mlp"]), (case["mlp"], case["hidden"])]
    return [(case["K"], case["N"])]


def _group(case, K):
    return case["group"] or K


def _inputs(case, seed, i, K, N):
    """Device tensors of linear i: x, tok2stream, w (fp32 [N, K]), d, dinv,
    bias, gamma [STEPS, S], clip [STEPS] (about the 0.999 quantile of |X D^-1|)."""
    d = synth.device_layer(K, N, _streams(case["tokens"]), T=STEPS, seed=seed * 1009 + i)
    rms = (d["x"].float() * d["dinv"]).square().mean().sqrt()
    d["clip"] = (3.3 * rms * torch.linspace(0.9, 1.1, STEPS, device=rms.device)).contiguous()
    return d


def _act(case, d, bits, static):
    return B.ActParams(tok2stream=d["tok2stream"], gamma=d["gamma"], step=STEP, act_bits=bits, dinv=d["dinv"],
                       range_mode=B.SQ_RANGE_STATIC if static else B.SQ_RANGE_DYNAMIC, clip=d["clip"])


def _chain_clip(d):
    """Per-step thresholds of the down projection's input GELU(Y_up), of order
    of the up projection's output (X W has a spread of about one)."""
    return torch.linspace(2.0, 4.0, STEPS, device=d["gamma"].device)


def _omega(S):
    return torch.full((S,), 1.0 / S, dtype=torch.float64, device="cuda")


def _candidates(case, d, seed):
    """Gains within a factor 2 of one and thresholds around the table's."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    C, S = case["candidates"], d["gamma"].shape[1]
    gamma = torch.exp((torch.rand((C, S), generator=g, device="cuda") - 0.5) * 1.3)
    clip = d["clip"][STEP] * torch.exp((torch.rand((C,), generator=g, device="cuda") - 0.5) * 0.8)
    return gamma.contiguous(), clip.contiguous()


def _alphas(case):
    n = case["exponents"]
    return [0.25 + 0.5 * i / max(1, n - 1) for i in range(n)]


# ------------------------------------------------------------------ prepare and run
def prepare(case, seed):
    M, kind = case["tokens"], case["kind"]
    dims = _linears(case)
    if kind in ("layer", "block"):
        bits = case["bits"]
        ws = torch.empty(max(B.sq_workspace_bytes(B.SQ_VARIANT_FUSED, M, K, N, bits) for K, N in set(dims)),
                         dtype=torch.uint8, device="cuda")
        call = B.sq_linear_w4a8 if bits == 8 else B.sq_linear_w4a4
        outs = {}
        for K, N in dims:
            outs[(K, N)] = torch.empty((dims.count((K, N)), M, N), dtype=B.OUT_DTYPES[OUT[case["out"]]], device="cuda")
        calls, at = [], {}
        for i, (K, N) in enumerate(dims):
            d = _inputs(case, seed, i, K, N)
            w = B.prepare_weight(d["w"], d["d"], _group(case, K), d["bias"])
            n = at[(K, N)] = at.get((K, N), -1) + 1
            calls.append((d["x"], _act(case, d, bits, case["static"]), w, outs[(K, N)][n]))
        state = dict(call=call, calls=calls, out=OUT[case["out"]], ws=ws, outs=list(outs.values()), graph=None)
        if case.get("graph"):
            _eager(state)  # the first call, before the capture
            torch.cuda.synchronize()
            state["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(state["graph"]):
                _eager(state)
        return state
    if kind == "chain":
        bits = case["bits"]
        (K, N), (K2, N2) = dims
        up, down = _inputs(case, seed, 0, K, N), _inputs(case, seed, 1, K2, N2)
        down["clip"] = _chain_clip(down)
        wide = bits == 4 and M > 128  # the 4-bit codes then take the fp8 form
        qx = torch.empty((M, N if bits == 8 or wide else N // 2), dtype=torch.int8 if bits == 8 else torch.uint8,
                         device="cuda")
        if bits == 8:
            scale = torch.empty((M,), dtype=torch.float32, device="cuda")
        else:
            scale = torch.empty((M, N // 64), dtype=torch.float32 if wide else torch.float16, device="cuda")
        kc = torch.empty((M, N // 64), dtype=torch.float32, device="cuda") if wide else None
        return dict(kind=kind, bits=bits, x=up["x"], act=_act(case, up, bits, False),
                    w=B.prepare_weight(up["w"], up["d"], _group(case, K), up["bias"]),
                    act2=_act(case, down, bits, True),
                    w2=B.prepare_weight(down["w"], down["d"], _group(case, K2), down["bias"]), qx=qx, scale=scale,
                    kc=kc, ws=B.alloc_workspace(B.SQ_VARIANT_FUSED, M, K, N, bits),
                    ws2=B.alloc_workspace(B.SQ_VARIANT_GEMM, M, K2, N2, bits), out=OUT[case["out"]],
                    y=torch.empty((M, N2), dtype=B.OUT_DTYPES[OUT[case["out"]]], device="cuda"))
    (K, N), = dims
    d = _inputs(case, seed, 0, K, N)
    S = d["gamma"].shape[1]
    state = dict(kind=kind, d=d, S=S, bits=case["bits"], omega=_omega(S),
                 y_ref=torch.empty((M, N), dtype=torch.float64, device="cuda"))
    if kind == "calib":
        state["gamma"], state["clip"] = _candidates(case, d, seed)
        state["w"] = B.prepare_weight(d["w"], d["d"], _group(case, K))
        state["objective"] = torch.empty((case["candidates"],), dtype=torch.float64, device="cuda")
        ws = B.sq_calib_workspace_bytes(M, K, N, case["bits"], S)
    else:
        state["group"], state["alphas"] = _group(case, K), _alphas(case)
        state["objective"] = torch.empty((case["exponents"],), dtype=torch.float64, device="cuda")
        ws = B.sq_calib_scaling_workspace_bytes(M, K, N, state["group"], case["bits"], S)
    state["ws"] = torch.empty(ws, dtype=torch.uint8, device="cuda")
    return state


def _eager(state):
    for x, act, w, y in state["calls"]:
        state["call"](x, act, w, y, state["out"], state["ws"])


def run(state):
    if "calls" in state:
        if state["graph"] is not None:
            state["graph"].replay()
        else:
            _eager(state)
        return state["outs"]
    s = state
    if s["kind"] == "chain":
        if s["bits"] == 8:
            B.sq_linear_w4a8_gelu_quant(s["x"], s["act"], s["w"], s["act2"], s["qx"], s["scale"], s["ws"])
            B.sq_gemm_w4a8(s["qx"], s["scale"], s["w2"], s["y"], s["out"], s["ws2"])
        else:
            B.sq_linear_w4a4_gelu_quant(s["x"], s["act"], s["w"], s["act2"], s["qx"], s["scale"], s["kc"], s["ws"])
            if s["kc"] is not None:
                B.sq_gemm_w4a4_fp8(s["qx"], s["scale"], s["kc"], s["act2"], s["w2"], s["y"], s["out"], s["ws2"])
            else:
                B.sq_gemm_w4a4(s["qx"], s["scale"], s["act2"], s["w2"], s["y"], s["out"], s["ws2"])
        return {"codes": s["qx"], "scale": s["scale"], "y": s["y"]}
    d = s["d"]
    if s["kind"] == "calib":
        B.sq_calib_reference(d["x"], d["dinv"], s["w"], s["y_ref"])
        B.sq_calib_objective(d["x"], d["tok2stream"], s["S"], d["dinv"], s["bits"], s["w"], s["y_ref"], s["gamma"],
                             s["clip"], s["omega"], s["objective"], s["ws"])
    else:
        B.sq_calib_fp_reference(d["x"], d["w"], s["y_ref"])
        B.sq_calib_scaling_objective(d["x"], d["tok2stream"], s["S"], s["omega"], d["w"], s["group"], s["bits"],
                                     s["y_ref"], s["alphas"], s["objective"], s["ws"])
    return {"y_ref": s["y_ref"], "objective": s["objective"]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    M, kind = case["tokens"], case["kind"]
    size = {"f32": 4, "bf16": 2, "f16": 2}.get(case.get("out"), 4)
    nbytes = flops = 0
    for i, (K, N) in enumerate(_linears(case)):
        weight = N * K // 2 + (K // _group(case, K)) * N * 2 + N * 2
        x_in = M * K * 2 if kind != "chain" or i == 0 else 0  # the chain's second input is the first's output
        y_out = M * N * size if kind != "chain" or i == 1 else M * N
        evals = 1 + case.get("candidates", 0) + case.get("exponents", 0)  # the target, then every candidate
        if kind in ("calib", "scaling"):  # the target is written once; x, w and it are read by the objective
            weight = weight if kind == "calib" else N * K * 4
            y_out = M * N * 8
        nbytes += x_in + weight + y_out + M * 4 + K * 4
        flops += 2 * M * N * K * evals
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the fused and the unfused path (the same sums in
    another order) differ by: fp32 1.7e-7 (rel) and 2.2e-6 (max); 16-bit
    outputs by one unit of the type where a sum crosses a rounding boundary
    (bf16 3.7e-5, f16 9.2e-6); the chain's codes follow the up projection's
    bf16 rounding (2e-7 of the codes, 9.3e-5 in y); the objectives carry the
    fp32 rounding of the candidates' outputs (1e-7 against 64 bits)."""
    if case["kind"] == "chain":
        return {"rel": 4e-4, "max": 0.03, "differ": 1e-5}
    if case["kind"] in ("calib", "scaling"):
        return {"rel": 4e-7, "max": 4e-6}
    return {"f32": {"rel": 7e-7, "max": 1e-5}, "bf16": {"rel": 1.5e-4, "max": 0.009},
            "f16": {"rel": 4e-5, "max": 0.0012}}[case["out"]]


# ------------------------------------------------------------------ the same in 64 bits
def _div(a, b):
    """The correctly rounded fp32 quotient (fp64 carries enough digits)."""
    return (a.double() / b).float()


def _reciprocal(v):
    """fp32 1 / v, 0 where that is infinite."""
    r = _div(torch.ones_like(v), v.double())
    return torch.where(torch.isinf(r), torch.zeros_like(r), r)


def _weight64(w, d, group):
    """Q(D W) as the header defines it: w' = w d and the step in fp32 and fp16,
    codes in [-7, 7]; returns code * step in fp64 [N, K]."""
    N, K = w.shape
    wp = (w * d).view(N, K // group, group)
    step = _div(wp.abs().amax(dim=2, keepdim=True), 7.0).half().float()
    inv = _reciprocal(step)
    code = torch.round(torch.clamp(wp * inv, -7.0, 7.0))
    return (code.double() * step.double()).view(N, K)


def _quant64(x, dinv, g, bits, clip):
    """Codes * step / gain of the activation quantizer, fp64 [M, K]: the codes
    by the header's fp32 sequence, everything after them in fp64.  clip None:
    the range of the row (8-bit) or of the 64-group (4-bit)."""
    M, K = x.shape
    xt = x.float() * dinv
    qmax, width = (127.0, K) if bits == 8 else (7.0, 64)
    xt = xt.view(M, K // width, width)
    c = xt.abs().amax(dim=2, keepdim=True) if clip is None else clip.view(1, 1, 1).expand(M, K // width, 1)
    delta = _div(c, qmax)
    if bits == 4:
        delta = delta.half().float()
    inv = _reciprocal(delta)
    t = (xt * g.view(M, 1, 1)) * inv
    q = torch.round(torch.clamp(t, -qmax, qmax))
    return (q.double() * delta.double() / g.double().view(M, 1, 1)).view(M, K)


def _linear64(x, d, w64, bits, clip):
    g = d["gamma"][STEP][d["tok2stream"].long()]
    return _quant64(x, d["dinv"], g, bits, clip) @ w64.t()


def _stream_error64(e, d, omega):
    """sum_s omega_s / n_s * ||e_s||^2"""
    row = e.square().sum(dim=1)
    ids = d["tok2stream"].long()
    n = torch.bincount(ids, minlength=omega.numel()).double()
    return (row * omega[ids] / n[ids]).sum()


def exact(case, seed):
    kind, dims = case["kind"], _linears(case)
    if kind in ("layer", "block"):
        outs = {}
        for i, (K, N) in enumerate(dims):
            d = _inputs(case, seed, i, K, N)
            y = _linear64(d["x"], d, _weight64(d["w"], d["d"], _group(case, K)), case["bits"],
                          d["clip"][STEP] if case["static"] else None)
            outs.setdefault((K, N), []).append(y + d["bias"].double())
        return [torch.stack(v) for v in outs.values()]
    if kind == "chain":
        (K, N), (K2, N2) = dims
        up, down = _inputs(case, seed, 0, K, N), _inputs(case, seed, 1, K2, N2)
        down["clip"] = _chain_clip(down)
        h = _linear64(up["x"], up, _weight64(up["w"], up["d"], _group(case, K)), case["bits"], None)
        h = (h + up["bias"].double()).to(torch.bfloat16).double()
        h = (0.5 * h * (1.0 + torch.erf(h / math.sqrt(2.0)))).to(torch.bfloat16)
        y = _linear64(h, down, _weight64(down["w"], down["d"], _group(case, K2)), case["bits"], down["clip"][STEP])
        return {"codes": None, "scale": None, "y": y + down["bias"].double()}
    (K, N), = dims
    d = _inputs(case, seed, 0, K, N)
    omega = _omega(d["gamma"].shape[1])
    objective = []
    if kind == "calib":
        w64 = _weight64(d["w"], d["d"], _group(case, K))
        y_ref = (d["x"].float() * d["dinv"]).double() @ w64.t()
        gamma, clip = _candidates(case, d, seed)
        for c in range(case["candidates"]):
            y = _quant64(d["x"], d["dinv"], gamma[c][d["tok2stream"].long()], case["bits"], clip[c]) @ w64.t()
            objective.append(_stream_error64(y - y_ref, d, omega))
    else:
        y_ref = d["x"].double() @ d["w"].double().t()
        ax, aw = d["x"].float().abs().amax(dim=0).double(), d["w"].abs().amax(dim=0).double()
        one = torch.ones_like(d["tok2stream"], dtype=torch.float32)
        for alpha in _alphas(case):
            alpha = float(torch.tensor(alpha, dtype=torch.float32))
            v = torch.where((ax > 0) & (aw > 0), ax.pow(alpha) / aw.pow(1.0 - alpha), torch.ones_like(ax))
            s = v.clamp(2.0**-6, 2.0**6).float()
            y = _quant64(d["x"], _div(torch.ones_like(s), s.double()), one, case["bits"], None) @ _weight64(d["w"], s, _group(case, K)).t()
            objective.append(_stream_error64(y - y_ref, d, omega))
    return {"y_ref": y_ref, "objective": torch.stack(objective)}
