"""The work whose speed this repository cares about, as cases with their inputs, one pass each, and their floors.

The cases follow what a user of the library runs through its public entry points: the quantized mixer on whole
sequences (prefill) and on one token per sequence with carried state (generation), the whole model around the
mixer (time to first token, time per output token), and the calibration that produces scales and int8 weights.
Shapes are the ones the repository is configured, tested and benchmarked at: the 130M layer (d_model 768), the
2.8B layer (d_model 2560, alone and as a stack of 64 with vocabulary 50280) and the Jamba-shaped layer (d_model
4096).  `listed` fixes twelve points; `draw` gives others of the same ranges.

Inputs are made on the GPU from the seed: dense weights N(0, 0.02^2), A_log[d, n] = log(n + 1), time-step bias the
inverse softplus of a log-uniform step in [1e-3, 1e-1], hidden input N(0, 1) with a few channels 50 to 100 times
larger; scales and int8 weights come from the library's own calibration on a small batch of the same distribution.
"""
import math

import torch

import paper_2410_13229_amd as Q

DEV = "cuda:0"
#          d_model, d_inner, dt_rank, outlier channels, their gain
SHAPES = {"130m": (768, 1536, 48, 4, 50.0), "2p8b": (2560, 5120, 160, 4, 50.0), "jamba": (4096, 8192, 256, 8, 100.0)}
N, W = 16, 4
VOCAB, EPS = 50280, 1e-5
PERCENTILE = 99.999
MAX_OPS, MAX_CALIBRATE_OPS = 3.5e12, 6e10  # a drawn case stays at or below the largest listed ones


def listed():
    return [
        # smallest call: one token of one sequence through one small layer; launches and latency
        {"name": "decode_130m_b1", "path": "mixer_decode", "shape": "130m", "batch": 1, "grid": "static"},
        # serving: a generation step of 64 sequences through the 2.8B layer
        {"name": "decode_2p8b_b64", "path": "mixer_decode", "shape": "2p8b", "batch": 64, "grid": "static"},
        # short prompt through the small layer
        {"name": "prefill_130m_1x256", "path": "mixer_prefill", "shape": "130m", "batch": 1, "length": 256,
         "grid": "static", "state": False},
        # the headline workload: one 2048-token prompt through the 2.8B layer
        {"name": "prefill_2p8b_1x2048", "path": "mixer_prefill", "shape": "2p8b", "batch": 1, "length": 2048,
         "grid": "static", "state": False},
        # a few prompts of an odd length, their recurrent states kept for generation
        {"name": "prefill_2p8b_3x701", "path": "mixer_prefill", "shape": "2p8b", "batch": 3, "length": 701,
         "grid": "static", "state": True},
        # a batch of long prompts (one layer of the 64-layer configuration)
        {"name": "prefill_2p8b_4x4096", "path": "mixer_prefill", "shape": "2p8b", "batch": 4, "length": 4096,
         "grid": "static", "state": True},
        # long context through the widest layer
        {"name": "prefill_jamba_1x16384", "path": "mixer_prefill", "shape": "jamba", "batch": 1, "length": 16384,
         "grid": "static", "state": True},
        # the scan input in E4M3 codes, the most accurate of the alternative 8-bit formats
        {"name": "prefill_2p8b_e4m3_1x1024", "path": "mixer_prefill", "shape": "2p8b", "batch": 1, "length": 1024,
         "grid": "e4m3", "state": False},
        # time to first token: embedding, two blocks of the stack, final norm and head (two, because in a deeper
        # stack one int8 code that rounds the other way grows to the size of the quantization noise, and the outputs
        # of two correct programs can no longer be compared: 0.03 of the logits after 6 blocks, 0.15 after 64)
        {"name": "model_prefill_1x512", "path": "model_prefill", "shape": "2p8b", "batch": 1, "length": 512, "layers": 2},
        # time per output token of the 64-block model, one user
        {"name": "model_decode_b1", "path": "model_decode", "shape": "2p8b", "batch": 1, "layers": 64},
        # time per output token of the 64-block model, a serving batch
        {"name": "model_decode_b64", "path": "model_decode", "shape": "2p8b", "batch": 64, "layers": 64},
        # scales and int8 weights of one 2.8B layer from the stated 4 x 256 calibration batch
        {"name": "calibrate_2p8b_4x256", "path": "calibrate", "shape": "2p8b", "batch": 4, "length": 256},
    ]


def _log_int(rng, lo, hi):
    """An integer whose logarithm is uniform over [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choices(["mixer_prefill", "mixer_decode", "model_prefill", "model_decode", "calibrate"],
                       weights=[9, 5, 1, 2, 1])[0]
    while True:
        c = {"path": path, "shape": rng.choice(["130m", "2p8b", "2p8b", "jamba"])}
        if path in ("model_prefill", "model_decode"):
            c["shape"], c["layers"] = "2p8b", 2 if path == "model_prefill" else 64
        if path == "mixer_prefill":
            c["length"] = _log_int(rng, 16, 16384)
            c["batch"] = _log_int(rng, 1, max(1, min(64, 16384 // c["length"])))
            c["grid"] = rng.choices(["static", "e4m3", "log2", "asym", "dynamic", "hadamard"], weights=[10, 2, 1, 1, 1, 1])[0]
            c["state"] = rng.random() < 0.5
        elif path == "mixer_decode":
            c["batch"] = _log_int(rng, 1, 256)
            c["grid"] = rng.choices(["static", "e4m3", "log2", "asym", "dynamic", "hadamard"], weights=[10, 1, 1, 1, 1, 1])[0]
        elif path == "model_prefill":
            c["length"] = _log_int(rng, 16, 4096)
            c["batch"] = _log_int(rng, 1, max(1, 4096 // c["length"]))
        elif path == "model_decode":
            c["batch"] = _log_int(rng, 1, 64)
        else:
            c["length"] = _log_int(rng, 32, 256)
            c["batch"] = rng.randint(1, 4)
        if work(c)["flops"] <= (MAX_CALIBRATE_OPS if path == "calibrate" else MAX_OPS):
            return c


class _Dims:
    """What the binding reads a layer's sizes from."""

    def __init__(self, shape):
        self.d_model, self.d_inner, self.dt_rank, self.outliers, self.gain = SHAPES[shape]
        self.d_state, self.d_conv = N, W


def _fp_weights(d, g):
    """fp32 master weights of one layer."""
    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV) * 0.02

    Dm, Di, R = d.d_model, d.d_inner, d.dt_rank
    dt = torch.exp(torch.rand(Di, generator=g, device=DEV) * (math.log(1e-1) - math.log(1e-3)) + math.log(1e-3))
    return {"W_in": normal(2 * Di, Dm), "conv_w": normal(Di, W), "conv_b": torch.zeros(Di, device=DEV),
            "W_x": normal(R + 2 * N, Di), "W_dt": normal(Di, R), "dt_bias": dt + torch.log(-torch.expm1(-dt)),
            "A_log": torch.log(torch.arange(1, N + 1, device=DEV, dtype=torch.float32)).repeat(Di, 1),
            "D": torch.ones(Di, device=DEV), "W_out": normal(Dm, Di)}


def _q_buffers(d):
    """Device buffers for one layer's int8 weights."""
    Dm, Di, R = d.d_model, d.d_inner, d.dt_rank
    q = {k: torch.empty(s, dtype=torch.int8, device=DEV)
         for k, s in {"W_in": (2 * Di, Dm), "conv_w": (Di, W), "W_x": (R + 2 * N, Di), "W_dt": (Di, R), "A": (Di, N),
                      "D": (Di,), "W_outH": (Dm, Di)}.items()}
    q["conv_b"] = torch.empty(Di, dtype=torch.float32, device=DEV)
    q["dt_bias"] = torch.empty(Di, dtype=torch.float32, device=DEV)
    return q


def _hidden(d, g, *shape):
    u = torch.randn((*shape, d.d_model), generator=g, device=DEV)
    u[..., torch.randperm(d.d_model, generator=g, device=DEV)[:d.outliers]] *= d.gain
    return u.half()


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def _calibrated(s, d, g, grid):
    """Quantized weights and scales of one layer on the given grid of the scan input."""
    nb, Lc = 2, 128
    fw, calib = _fp_weights(d, g), _hidden(d, g, nb, Lc)
    q, cws = _q_buffers(d), _bytes(Q.quamba_calibrate_workspace_bytes(d, nb, Lc))
    nx, extra = d.dt_rank + 2 * N, None
    if grid == "asym":
        keep = torch.empty(nx, dtype=torch.int32, device=DEV)
        sc, extra = Q.quamba_calibrate_xasym(d, fw, calib, nb, Lc, PERCENTILE, q, keep, cws)
    elif grid == "hadamard":
        keep = torch.empty((nx, d.d_inner), dtype=torch.int8, device=DEV)
        sc, extra = Q.quamba_calibrate_hadx(d, fw, calib, nb, Lc, PERCENTILE, q, keep, cws)
    elif grid in ("e4m3", "log2"):
        keep = torch.empty((nx, d.d_inner), dtype=torch.int16, device=DEV)
        sc, extra = Q.quamba_calibrate_xfmt(d, fw, calib, nb, Lc, Q.XFMT_E4M3 if grid == "e4m3" else Q.XFMT_LOG2,
                                            PERCENTILE, q, keep, cws)
    else:
        keep = None
        sc = Q.quamba_calibrate(d, fw, calib, nb, Lc, PERCENTILE, q, cws)
    s.update(dims=Q.make_dims(d), q=Q.make_qweights(q), sc=sc, extra=extra, grid=grid, keep=(q, keep))


def _mixer_workspace(d, batch, length, grid):
    size = {"hadamard": Q.quamba_hadx_workspace_bytes, "dynamic": Q.quamba_xdyn_workspace_bytes}
    return _bytes(size.get(grid, Q.quamba_workspace_bytes)(d, batch, length))


def _model(s, d, g, n_layers):
    """A stack of blocks with embedding and head, every block calibrated on the unquantized forward of the blocks before it."""
    nb, Lc = 2, 64
    E = (torch.randn((VOCAB, d.d_model), generator=g, device=DEV) * 0.02).half()
    norms = (1.0 + 0.1 * torch.randn((n_layers + 1, d.d_model), generator=g, device=DEV)).half()
    res = E[torch.randint(0, VOCAB, (nb * Lc,), generator=g, device=DEV)].float()
    out, cws, layers = torch.zeros_like(res), _bytes(Q.quamba_calibrate_workspace_bytes(d, nb, Lc)), []
    for i in range(n_layers):
        q = _q_buffers(d)
        sc = Q.quamba_calibrate_block(d, _fp_weights(d, g), norms[i], EPS, res, out, nb, Lc, PERCENTILE, q, cws)
        layers.append((q, sc, norms[i]))
    s["model"] = Q.make_model(d, E, norms[n_layers], layers, EPS)
    s["keep"] = (E, norms, layers)


def prepare(case, seed):
    d = _Dims(case["shape"])
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    s = {"path": case["path"], "batch": case["batch"], "length": case.get("length", 1)}
    b, L, Dm, Di = s["batch"], s["length"], d.d_model, d.d_inner
    if s["path"] == "calibrate":
        s.update(dims=d, fw=_fp_weights(d, g), calib=_hidden(d, g, b, L), q=_q_buffers(d),
                 ws=_bytes(Q.quamba_calibrate_workspace_bytes(d, b, L)))
    elif s["path"] == "mixer_prefill":
        _calibrated(s, d, g, case["grid"])
        s.update(u=_hidden(d, g, b, L), out=torch.empty((b, L, Dm), dtype=torch.float16, device=DEV),
                 ssm=torch.zeros((b, Di, N), device=DEV) if case["state"] else None,
                 conv=torch.empty((b, Di, W - 1), dtype=torch.float16, device=DEV),
                 ws=_mixer_workspace(d, b, L, case["grid"]))
    elif s["path"] == "mixer_decode":
        _calibrated(s, d, g, case["grid"])
        s.update(u=_hidden(d, g, b), out=torch.empty((b, Dm), dtype=torch.float16, device=DEV),
                 ssm=torch.randn((b, Di, N), generator=g, device=DEV) * 0.1,
                 conv=(torch.randn((b, Di, W - 1), generator=g, device=DEV) * 2.2).half(),
                 ws=_mixer_workspace(d, b, 1, case["grid"]))
    else:
        nl = case["layers"]
        _model(s, d, g, nl)
        m = s["model"]
        s.update(logits=torch.empty((b, VOCAB), device=DEV), next=torch.empty(b, dtype=torch.int32, device=DEV),
                 ssm=torch.empty((nl, b, Di, N), device=DEV),
                 conv=torch.empty((nl, b, Di, W - 1), dtype=torch.float16, device=DEV),
                 ws=_bytes(Q.quamba_model_workspace_bytes(m, b, L)))
        prompt = L if s["path"] == "model_prefill" else 16
        s["tokens"] = torch.randint(0, VOCAB, (b, prompt), generator=g, device=DEV, dtype=torch.int32)
        if s["path"] == "model_decode":  # generation goes on from real states: a short prompt first
            s["tokens_in"] = torch.empty(b, dtype=torch.int32, device=DEV)
            ws = _bytes(Q.quamba_model_workspace_bytes(m, b, prompt))
            Q.quamba_model_prefill(m, s["tokens"], b, prompt, None, s["tokens_in"], s["ssm"], s["conv"], ws)
    s["stream"] = torch.cuda.current_stream().cuda_stream
    return s


def run(s):
    path, b, L, st = s["path"], s["batch"], s["length"], s["stream"]
    if path == "calibrate":
        sc = Q.quamba_calibrate(s["dims"], s["fw"], s["calib"], b, L, PERCENTILE, s["q"], s["ws"], st)
        return {"weights": s["q"], "scales": Q.scales_to_dict(sc)}
    if path == "model_prefill":  # a sampling program: it takes the logits and picks the token itself
        Q.quamba_model_prefill(s["model"], s["tokens"], b, L, s["logits"], None, s["ssm"], s["conv"], s["ws"], st)
        return {"logits": s["logits"], "ssm": s["ssm"], "conv": s["conv"]}
    if path == "model_decode":  # greedy: logits and the chosen token
        Q.quamba_model_decode(s["model"], s["tokens_in"], b, s["logits"], s["next"], s["ssm"], s["conv"], s["ws"], st)
        return {"logits": s["logits"], "next": s["next"], "ssm": s["ssm"], "conv": s["conv"]}
    if path == "mixer_prefill":
        if s["ssm"] is not None:
            s["ssm"].zero_()  # fresh sequences
        head, tail = (s["dims"], s["q"], s["sc"]), (s["u"], b, L, s["out"], s["ssm"], s["conv"], None)
        calls = {"static": Q.quamba_mixer_prefill, "asym": Q.quamba_mixer_prefill_xasym, "hadamard": Q.quamba_mixer_prefill_hadx,
                 "dynamic": Q.quamba_mixer_prefill_xdyn}
        call = calls.get(s["grid"], Q.quamba_mixer_prefill_xfmt)
    else:
        head, tail = (s["dims"], s["q"], s["sc"]), (s["u"], b, s["out"], s["ssm"], s["conv"], None)
        calls = {"static": Q.quamba_mixer_decode, "asym": Q.quamba_mixer_decode_xasym, "hadamard": Q.quamba_mixer_decode_hadx,
                 "dynamic": Q.quamba_mixer_decode_xdyn}
        call = calls.get(s["grid"], Q.quamba_mixer_decode_xfmt)
    if s["extra"] is not None:
        head += (s["extra"],)
    tail += {"hadamard": (None,), "dynamic": (None, None)}.get(s["grid"], ())
    call(*head, *tail, s["ws"], st)
    return {"out": s["out"], "ssm": s["ssm"], "conv": s["conv"]}


def work(case):
    """Bytes: int8 weights, inputs, outputs and states once each.  Operations: the four projections, the causal conv,
    one scan update per (token, channel, state) of exponential, multiply and two multiply-adds, the Hadamard butterflies."""
    d = _Dims(case["shape"])
    b, L, Dm, Di, R = case["batch"], case.get("length", 1), d.d_model, d.d_inner, d.dt_rank
    M, nx = b * L, R + 2 * N
    params = 2 * Di * Dm + nx * Di + Di * R + Dm * Di
    small = Di * (W + N + 1 + 8)
    per_token = 2 * params + Di * (2 * W + 7 * N + math.log2(Di))
    states = b * Di * (N * 4 + (W - 1) * 2)
    path = case["path"]
    if path == "calibrate":  # the fp32 forward (no output projection), the transform of W_out, the int8 weights
        return {"bytes": 5 * params + small + M * Dm * 2,
                "flops": M * (per_token - 2 * Dm * Di) + Dm * Di * math.log2(Di)}
    if path == "mixer_prefill":
        return {"bytes": params + small + M * Dm * 4 + (states if case["state"] else b * Di * (W - 1) * 2), "flops": M * per_token}
    if path == "mixer_decode":
        return {"bytes": params + small + M * Dm * 4 + 2 * states, "flops": M * per_token}
    head = VOCAB * Dm * 2 + b * VOCAB * 4
    passes = 1 if path == "model_prefill" else 2  # a prompt's states are written, a step's are read and written
    nl = case["layers"]
    return {"bytes": nl * (params + small + passes * states) + head + M * (4 + 2 * Dm),
            "flops": nl * M * per_token + 2 * b * VOCAB * Dm}


def tolerance(case):
    """Four times what a second order of the floating-point work showed.

    Prefill was compared between the two forms of the scan (chunked, one sweep): the fp16 output moves by 1.1e-4 to
    2.1e-4 (2-norm; 0.016 of the rms at most) because a few of the int8 codes in front of the output projection round
    the other way, the states by 9e-7.  A generation step from states 3e-7 apart: 4.8e-4 and 0.008.  Two blocks: 2.5e-3
    and 0.09 in the states of the second.  Calibration was compared with its forward pass in 64 bits: scales 2.0e-6,
    2.7e-6 of the codes of the folded output weight."""
    if case["path"] == "calibrate":
        return {"rel": 8e-6, "max": 8e-6, "differ": 1.1e-5}
    if case["path"] == "model_prefill":
        return {"rel": 1e-2, "max": 0.36}
    return {"rel": 2e-3, "max": 0.064, "differ": 0.0 if case["path"] != "model_decode" else 1e-2}
