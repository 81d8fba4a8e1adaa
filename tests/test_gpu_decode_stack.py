"""Generation of a stack in one launch: the bits of the launch-by-launch form, at the edges of its column groups and widths, with its
work items kept or taken from the counter, replayed from a graph, and with two steps in flight at once."""
import pytest
import torch

import paper_2410_13229_amd as Q
import workloads as W
from gpu_util import empty, workspace

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
VOCAB = 97


def _model(Dm, Di, R, n_layers, seed):
    """A calibrated stack with random weights, everything on the GPU."""
    d = W.tiny_config(name="stack", d_model=Dm, d_inner=Di, dt_rank=R, batch=1, seqlen=1, config_id=97)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV)

    E, norms = (normal(VOCAB, Dm) * 0.5).half(), (1 + 0.1 * normal(n_layers + 1, Dm)).half()
    nb, Lc, layers = 1, 24, []
    res = E[torch.randint(0, VOCAB, (nb * Lc,), generator=g, device=DEV)].float()
    out, ws = torch.zeros_like(res), workspace(Q.quamba_calibrate_workspace_bytes(d, nb, Lc))
    for i in range(n_layers):
        fw = {"W_in": normal(2 * Di, Dm) * Dm ** -0.5, "conv_w": normal(Di, 4) * 0.5, "conv_b": normal(Di) * 0.1,
              "W_x": normal(R + 32, Di) * Di ** -0.5, "W_dt": normal(Di, R) * R ** -0.5, "dt_bias": normal(Di) - 3.0,
              "A_log": torch.log(torch.arange(1, 17, device=DEV, dtype=torch.float32)).repeat(Di, 1), "D": normal(Di),
              "W_out": normal(Dm, Di) * Di ** -0.5}
        q = {k: torch.empty(s, dtype=torch.int8, device=DEV)
             for k, s in {"W_in": (2 * Di, Dm), "conv_w": (Di, 4), "W_x": (R + 32, Di), "W_dt": (Di, R), "A": (Di, 16), "D": (Di,),
                          "W_outH": (Dm, Di)}.items()}
        q["conv_b"], q["dt_bias"] = empty((Di,), torch.float32), empty((Di,), torch.float32)
        sc = Q.quamba_calibrate_block(d, fw, norms[i], 1e-5, res, out, nb, Lc, 99.999, q, ws)
        layers.append((q, sc, norms[i]))
    return d, Q.make_model(d, E, norms[n_layers], layers, 1e-5), (E, norms, layers)


def _states(d, n_layers, Bt, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return (torch.randn((n_layers, Bt, d.d_inner, 16), generator=g, device=DEV) * 0.1,
            (torch.randn((n_layers, Bt, d.d_inner, 3), generator=g, device=DEV) * 0.5).half())


def _steps(d, m, n_layers, Bt, hook, steps=2, fill=0):
    ssm, conv = _states(d, n_layers, Bt, 5)
    ws = workspace(Q.quamba_model_workspace_bytes(m, Bt, 1))
    ws.fill_(fill)  # words of an earlier step, or anything else
    tok = torch.arange(Bt, dtype=torch.int32, device=DEV) * 40 + 3
    logits, got = empty((Bt, VOCAB), torch.float32), []
    Q.quamba_debug_set_decode_stack(hook)
    try:
        for _ in range(steps):
            Q.quamba_model_decode(m, tok, Bt, logits, tok, ssm, conv, ws)
            got += [logits.clone(), tok.clone()]
    finally:
        Q.quamba_debug_set_decode_stack(0)
    return got + [ssm, conv]


@pytest.mark.parametrize("Dm,Di,R,n_layers,Bt", [
    (80, 1536, 16, 3, 1),     # fewer columns than workgroups, Hadamard items that leave a wave half empty
    (64, 1536, 16, 3, 1),     # 12 items of x_proj watch 7 lines of the residual stream
    (704, 1536, 256, 3, 2),   # 72 watch 71
    (208, 1536, 48, 2, 2),    # a ragged last group of out_proj columns
    (768, 1536, 48, 23, 1),   # more blocks than descriptors in one launch
    (1024, 2048, 64, 2, 2),   # an order that is a power of two
    (1280, 2560, 256, 2, 1),  # the widest dt_rank
    (1536, 3072, 96, 2, 2),
    (2048, 4096, 128, 2, 1),
    (2560, 5120, 160, 2, 1),  # every CU
    (2560, 5120, 160, 2, 2),
    (2560, 1536, 16, 2, 2),   # as many workgroups for out_proj as there are CUs
])
def test_one_launch_gives_the_bits_of_separate_launches(Dm, Di, R, n_layers, Bt):
    """Integer sums and the same fp32 operations in the same order: equal, not close."""
    d, m, keep = _model(Dm, Di, R, n_layers, Dm + Di + Bt)
    assert Q.quamba_debug_decode_stack_served(d, n_layers, Bt)
    want = _steps(d, m, n_layers, Bt, 1)
    assert torch.isfinite(want[0]).all() and want[0].std() > 0
    for hook, fill in ((0, 0), (0, 255), (2, 1)):
        print("decode stack", Dm, Di, Bt, "hook", hook, flush=True)
        for a, b in zip(_steps(d, m, n_layers, Bt, hook, fill=fill), want):
            assert torch.equal(a, b)
    del keep


@pytest.mark.parametrize("Dm,Di,R,n_layers,Bt", [
    (2576, 1536, 16, 2, 2),   # more out_proj columns than 256 workgroups take
    (3072, 1536, 16, 2, 2),
    (3088, 1536, 16, 2, 1),   # more than role A's registers hold of a weight row
    (768, 1536, 272, 2, 1),   # dt_rank
    (96, 192, 16, 2, 1), (1024, 8192, 64, 2, 1),  # widths that are not built
    (2048, 4096, 128, 2, 2),  # two sequences of this width
    (768, 1536, 48, 1, 1),    # one block
    (768, 1536, 48, 2, 3),    # three sequences
])
def test_other_shapes_run_launch_by_launch(Dm, Di, R, n_layers, Bt):
    d, m, keep = _model(Dm, Di, R, n_layers, 16)
    assert not Q.quamba_debug_decode_stack_served(d, n_layers, Bt)
    for a, b in zip(_steps(d, m, n_layers, Bt, 0, fill=255), _steps(d, m, n_layers, Bt, 1)):
        assert torch.equal(a, b)
    del keep


def test_generation_from_a_graph():
    d, m, keep = _model(768, 1536, 48, 4, 11)
    assert Q.quamba_debug_decode_stack_served(d, 4, 1)
    outs = []
    for hook, graph in ((1, 0), (0, 0), (0, 1), (0, 1)):
        ssm, conv = _states(d, 4, 1, 5)
        ws, toks = workspace(Q.quamba_model_workspace_bytes(m, 1, 1)), empty((9, 1), torch.int32)
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        Q.quamba_debug_set_decode_stack(hook)
        try:
            Q.quamba_model_generate(m, torch.tensor([3], dtype=torch.int32, device=DEV), 1, 9, toks, ssm, conv, ws, graph,
                                    stream.cuda_stream)
            torch.cuda.synchronize()
        finally:
            Q.quamba_debug_set_decode_stack(0)
        outs.append((toks.clone(), ssm.clone(), conv.clone()))
    for o in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(o, outs[0]))
    del keep


def test_two_steps_in_flight():
    """Two streams, states and workspaces of their own, their launches interleaved: neither step waits for the other's workgroups."""
    d, m, keep = _model(2560, 5120, 160, 2, 12)
    assert Q.quamba_debug_decode_stack_served(d, 2, 1)
    want = _steps(d, m, 2, 1, 1, steps=6)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    runs = []
    for s in streams:
        ssm, conv = _states(d, 2, 1, 5)
        runs.append((torch.full((1,), 3, dtype=torch.int32, device=DEV), empty((1, VOCAB), torch.float32), ssm, conv,
                     workspace(Q.quamba_model_workspace_bytes(m, 1, 1))))
    torch.cuda.synchronize()
    for _ in range(6):
        for s, (tok, logits, ssm, conv, ws) in zip(streams, runs):
            Q.quamba_model_decode(m, tok, 1, logits, tok, ssm, conv, ws, s.cuda_stream)
    torch.cuda.synchronize()
    for tok, logits, ssm, conv, _ in runs:
        assert torch.equal(logits, want[-4]) and torch.equal(tok, want[-3])
        assert torch.equal(ssm, want[-2]) and torch.equal(conv, want[-1])
    del keep


@pytest.mark.parametrize("Bt", [1, 2])
def test_four_users_for_many_steps(Bt):
    """Four streams that keep the GPU full, so that the launches of a step start piecemeal and hold one another up: a workgroup
    may be late at any word of the hand-over."""
    n, steps = 16, 40
    d, m, keep = _model(2560, 5120, 160, n, 14)
    assert Q.quamba_debug_decode_stack_served(d, n, Bt)
    want = _steps(d, m, n, Bt, 1, steps=steps)
    for rep in range(4):
        streams, runs = [torch.cuda.Stream() for _ in range(4)], []
        for _ in streams:
            ssm, conv = _states(d, n, Bt, 5)
            runs.append((torch.arange(Bt, dtype=torch.int32, device=DEV) * 40 + 3, empty((Bt, VOCAB), torch.float32), ssm, conv,
                         workspace(Q.quamba_model_workspace_bytes(m, Bt, 1))))
        torch.cuda.synchronize()
        for _ in range(steps):
            for s, (tok, logits, ssm, conv, ws) in zip(streams, runs):
                Q.quamba_model_decode(m, tok, Bt, logits, tok, ssm, conv, ws, s.cuda_stream)
        torch.cuda.synchronize()
        print("four users", Bt, "repetition", rep, flush=True)
        for tok, logits, ssm, conv, _ in runs:
            assert torch.equal(logits, want[-4]) and torch.equal(tok, want[-3])
            assert torch.equal(ssm, want[-2]) and torch.equal(conv, want[-1])
    del keep


@pytest.mark.parametrize("Dm,Di,R,Bt", [(768, 1536, 48, 1), (1024, 2048, 64, 2)])
def test_a_step_that_gives_up_says_so_and_the_next_one_is_whole(Dm, Di, R, Bt):
    """The first input of the chain is held back, so that every bounded wait behind it runs out: NaN and -1, nothing finite."""
    d, m, keep = _model(Dm, Di, R, 3, 15)
    assert Q.quamba_debug_decode_stack_served(d, 3, Bt)
    want = _steps(d, m, 3, Bt, 1)
    ssm, conv = _states(d, 3, Bt, 5)
    ws = workspace(Q.quamba_model_workspace_bytes(m, Bt, 1))
    first = torch.arange(Bt, dtype=torch.int32, device=DEV) * 40 + 3
    tok, logits, toks = first.clone(), empty((Bt, VOCAB), torch.float32), empty((3, Bt), torch.int32)
    Q.quamba_debug_set_decode_stack(3)
    try:
        Q.quamba_model_decode(m, tok, Bt, logits, tok, ssm, conv, ws)
        assert torch.isnan(logits).all() and (tok == -1).all()
        Q.quamba_model_generate(m, first, Bt, 1, toks, ssm, conv, ws, 0)
        assert (toks[0] == -1).all()
    finally:
        Q.quamba_debug_set_decode_stack(0)
    got = []
    ssm, conv = _states(d, 3, Bt, 5)
    tok = first.clone()
    for _ in range(2):
        Q.quamba_model_decode(m, tok, Bt, logits, tok, ssm, conv, ws)
        got += [logits.clone(), tok.clone()]
    for a, b in zip(got + [ssm, conv], want):
        assert torch.equal(a, b)
    del keep


@pytest.mark.parametrize("Bt", [3, 20, 70, 130])  # both, both, both with more than 64 sequences, out_proj alone
def test_weights_read_ahead_change_nothing(Bt):
    """A stack whose weights exceed the last-level cache (the same block seven times: 280 MB): norm and Hadamard launches with workgroups that
    read ahead, against the blocks one by one through their own entry points."""
    d, m, keep = _model(2560, 5120, 160, 1, 13)
    E, norms, layers = keep
    n = 7
    m = Q.make_model(d, E, norms[1], layers * n, 1e-5)
    got = _steps(d, m, n, Bt, 0, steps=1)
    ssm, conv = _states(d, n, Bt, 5)
    tok = torch.arange(Bt, dtype=torch.int32, device=DEV) * 40 + 3
    res, out = E[tok.long().clamp(0, VOCAB - 1)].contiguous(), torch.zeros((Bt, 2560), dtype=torch.float16, device=DEV)
    u_q, ws = empty((Bt, 2560), torch.int8), workspace(Q.quamba_workspace_bytes(d, Bt, 1))
    q, sc, norm = layers[0]
    for l in range(n):
        Q.quamba_add_rmsnorm_quant(out, res, norm, 1e-5, Q.scales_to_dict(sc)["inv_s_u"], u_q, Bt, 2560)
        Q.quamba_mixer_decode_q(d, q, sc, u_q, Bt, out, ssm[l], conv[l], None, ws)
    y, logits = empty((Bt, 2560), torch.float16), empty((Bt, VOCAB), torch.float32)
    Q.quamba_final_norm(out, res, norms[1], 1e-5, Bt, 1, 2560, y)
    Q.quamba_lm_head(y, E, Bt, VOCAB, 2560, logits)
    assert torch.equal(got[0], logits) and torch.equal(got[2], ssm) and torch.equal(got[3], conv)
