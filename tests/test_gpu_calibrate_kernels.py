"""The fp32 kernels under calibration at the edges of their tiles, against the same forward in 64 bits."""
import math

import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import Q, dev, empty, host, rel_err, torch, workspace

pytestmark = pytest.mark.gpu


def _case(Dm, Di, R, nb, L):
    cfg = W.tiny_config(name="tk", d_model=Dm, d_inner=Di, dt_rank=R, config_id=95)
    return cfg, W.make_weights(cfg, randomize_bias=True), W.make_hidden(cfg, batch=nb, seqlen=L, stream=12)


# Products of fewer than 128 tiles run in 32 x 32 blocks, others in tiles of 128 x 64 (more than 64 rows), 64 x 128 (33 to
# 64) or 32 x 256 (up to 32); above 64 rows tiles of 128 x 96, 128 x 128 or 128 x 160 where they come out even over the CUs.
@pytest.mark.parametrize("Dm,Di,R,nb,L", [
    # 32 x 32 blocks throughout
    (48, 16, 16, 1, 1),        # half a block of channels, one token, K = 16 and 48: a part of a slice
    (80, 320, 48, 1, 31),      # one row block, not full
    (64, 192, 16, 1, 33),      # one row past a block
    (64, 192, 16, 2, 32),      # whole row blocks; exactly one block of tokens
    (80, 320, 48, 5, 13),      # 65 rows
    (768, 1536, 48, 3, 43),    # 129 rows; in_proj: 128 x 64 tiles, 48 x 2 of them too few, K = 1536 in the blocks
    # 128 x 64 tiles
    (768, 1536, 48, 3, 100),   # in_proj: 48 x 3 tiles, 300 rows
    (48, 1536, 48, 5, 130),    # in_proj and dt_proj: 650 rows, K = 48: a slice and a half
    (1040, 192, 16, 7, 131),   # out_proj: 917 rows, 1040 columns (a quarter of the last tile)
    # 128 x 96, 128 x 128 and 128 x 160 tiles
    (48, 5120, 16, 1, 129),    # in_proj: 107 x 2 of 96 columns, 64 in the last, one row in the second row block
    (80, 5120, 16, 2, 128),    # whole row blocks
    (10256, 16, 16, 5, 130),   # out_proj: 650 rows, 81 x 6 of 128 columns, 16 in the last
    (48, 5120, 16, 5, 151),    # in_proj: 755 rows, 128 columns
    (80, 5120, 16, 3, 131),    # in_proj: 393 rows, 64 x 4 of 160 columns
    (10192, 16, 16, 7, 130),   # out_proj: 910 rows, 64 x 8 of 160 columns, 112 in the last
    # 64 x 128 tiles: in_proj to 16384 columns
    (48, 8192, 16, 1, 33),
    (80, 8192, 16, 3, 21),     # 63 rows
    (48, 8192, 16, 2, 32),     # 64 rows
    (16272, 16, 16, 1, 40),    # out_proj: 16272 columns (16 of the last tile's 128), K = 16
    # 32 x 256 tiles: in_proj to 32768 columns
    (48, 16384, 16, 1, 1),
    (80, 16384, 16, 1, 31),
    (48, 16384, 16, 2, 16),    # 32 rows
    (32528, 16, 16, 1, 20),    # out_proj: 32528 columns (16 of the last tile's 256)
])
def test_fp32_forward_at_tile_edges(Dm, Di, R, nb, L):
    """fp32 sums of up to 16384 products against fp64: errors of about sqrt(K) 2^-24 per sum, 128 x 6e-8 = 7.7e-6 at most and
    2.4e-6 at 1536 of the sum's scale, through three projections and a decaying recurrence: 1e-5 of the largest output."""
    cfg, w, u = _case(Dm, Di, R, nb, L)
    want = O.fp_forward(w, u)["out"].reshape(nb * L, Dm)
    fw = {k: dev(v) for k, v in w.items()}
    out = empty((nb * L, Dm), torch.float32)
    Q.quamba_mixer_fp32(cfg, fw, dev(u), nb, L, out, workspace(Q.quamba_calibrate_workspace_bytes(cfg, nb, L)))
    assert rel_err(host(out), want) <= 1e-5


def test_calibration_takes_unaligned_master_weights():
    """Master weights promise four-byte alignment only (W_out sixteen), code buffers none: the same codes and scales."""
    cfg, w, u = _case(80, 320, 48, 2, 19)
    ws = workspace(Q.quamba_calibrate_workspace_bytes(cfg, 2, 19))
    got = []
    for shift in (0, 1):
        fw = {}
        for k, v in w.items():
            buf = torch.empty(v.size + 4, dtype=torch.float32, device="cuda:0")
            at = buf[(shift if k != "W_out" else 0):][:v.size]
            at.copy_(dev(np.ascontiguousarray(v, np.float32)).reshape(-1))
            fw[k] = at.view(v.shape)
        out_q = {}
        for k, shape in (("W_in", (640, 80)), ("conv_w", (320, 4)), ("W_x", (80, 320)), ("W_dt", (320, 48)), ("A", (320, 16)),
                         ("D", (320,)), ("W_outH", (80, 320)), ("conv_b", (320,)), ("dt_bias", (320,))):
            f32 = k in ("conv_b", "dt_bias")
            buf = torch.zeros(math.prod(shape) + 4, dtype=torch.float32 if f32 else torch.int8, device="cuda:0")
            out_q[k] = buf[shift:][:math.prod(shape)].view(shape)
        sc = Q.scales_to_dict(Q.quamba_calibrate(cfg, fw, dev(u), 2, 19, 99.9, out_q, ws))
        got.append((sc, {k: host(v) for k, v in out_q.items()}))
    assert got[0][0] == got[1][0]
    for k in got[0][1]:
        assert np.array_equal(got[0][1][k], got[1][1][k]), k


@pytest.mark.parametrize("Dm,Di,R,nb,L", [
    (80, 320, 48, 3, 47),     # 32 x 32 blocks on both sides, at other rows of a block
    (768, 1536, 48, 6, 43),   # in_proj 128 x 64 against 32 x 32
    (48, 1536, 48, 5, 130),   # in_proj and dt_proj
    (1040, 192, 16, 7, 131),  # out_proj
    (80, 8192, 16, 2, 32),    # in_proj 64 x 128 against 32 x 32
    (80, 16384, 16, 2, 20),   # in_proj 64 x 128 against 32 x 256
    (80, 16384, 16, 4, 30),   # in_proj 128 x 64 against 32 x 256
])
def test_order_of_the_fp32_sums_does_not_depend_on_the_tile(Dm, Di, R, nb, L):
    """Every fp32 output is one chain of multiply-adds over K, so a sequence gives the same bits alone and in a batch: scales, and
    with them int8 codes, do not move with the batch's shape."""
    cfg, w, u = _case(Dm, Di, R, nb, L)
    fw = {k: dev(v) for k, v in w.items()}
    ws = workspace(Q.quamba_calibrate_workspace_bytes(cfg, nb, L))
    whole, one = empty((nb, L, Dm), torch.float32), empty((1, L, Dm), torch.float32)
    Q.quamba_mixer_fp32(cfg, fw, dev(u), nb, L, whole, ws)
    for b in range(nb):
        Q.quamba_mixer_fp32(cfg, fw, dev(np.ascontiguousarray(u[b:b + 1])), 1, L, one, ws)
        assert np.array_equal(host(one)[0], host(whole)[b])


def _left_in_workspace(ws, cfg, M):
    """u, x_pre | z, x, dt_low | B | C, dt and g of the fp32 forward, in the order in which the workspace holds them."""
    at, got = 0, []
    for cols in (cfg.d_model, 2 * cfg.d_inner, cfg.d_inner, cfg.dt_rank + 32, cfg.d_inner, cfg.d_inner):
        n = M * cols
        got.append(host(ws[4 * at:4 * (at + n)].view(torch.float32)).reshape(M, cols))
        at += (n + 63) // 64 * 64
    return got


def _chain(a, w):
    """sum_k a[m, k] w[n, k] with k in order, one rounding to fp32 per multiply-add: the product of two fp32 values is exact
    in 64 bits of significand, and so is its sum with an fp32 value but for a tie in one of about 2^40 steps."""
    acc = np.zeros((a.shape[0], w.shape[0]), np.float32)
    a, w = a.astype(np.longdouble), w.astype(np.longdouble)
    for k in range(a.shape[1]):
        acc = (a[:, k, None] * w[None, :, k] + acc.astype(np.longdouble)).astype(np.float32)
    return acc


@pytest.mark.parametrize("Dm,Di,R,nb,L", [(80, 320, 48, 1, 31), (48, 1536, 48, 5, 130), (80, 8192, 16, 2, 32), (80, 16384, 16, 1, 20),
                                             (48, 5120, 16, 1, 130), (80, 5120, 16, 5, 130), (48, 5120, 16, 7, 141)])
def test_fp32_sums_run_over_k_in_order(Dm, Di, R, nb, L):
    """Each projection of the forward against the chain on the host, bit for bit, at rows and columns of every part of a tile."""
    cfg, w, u = _case(Dm, Di, R, nb, L)
    M = nb * L
    ws = workspace(Q.quamba_calibrate_workspace_bytes(cfg, nb, L))
    out = empty((M, Dm), torch.float32)
    Q.quamba_mixer_fp32(cfg, {k: dev(v) for k, v in w.items()}, dev(u), nb, L, out, ws)
    u32, xz, x, dbc, dt, g = _left_in_workspace(ws, cfg, M)
    for name, a, wt, got in (("in_proj", u32, w["W_in"], xz), ("x_proj", x, w["W_x"], dbc), ("dt_proj", dbc[:, :R], w["W_dt"], dt),
                             ("out_proj", g, w["W_out"], host(out))):
        rows = np.unique(np.linspace(0, M - 1, 23).astype(int))
        cols = np.unique(np.linspace(0, wt.shape[0] - 1, 61).astype(int))
        assert np.array_equal(got[np.ix_(rows, cols)], _chain(a[rows], np.asarray(wt, np.float32)[cols])), name


@pytest.mark.parametrize("M,workgroups", [(1, 256), (1027, 256), (1028, 257), (2048, 512), (3068, 767), (3100, 768)])
def test_percentile_of_many_values(M, workgroups):
    """The same at every size of the grid that counts: its least, one more, and its most."""
    cfg, w, u = _case(16, 5120, 16, 1, M)
    assert Q.quamba_debug_percentile_workgroups(M * 5120) == workgroups
    ws = workspace(Q.quamba_calibrate_workspace_bytes(cfg, 1, M))
    q = {k: empty(s, torch.int8) for k, s in (("W_in", (10240, 16)), ("conv_w", (5120, 4)), ("W_x", (48, 5120)), ("W_dt", (5120, 16)),
                                              ("A", (5120, 16)), ("D", (5120,)), ("W_outH", (16, 5120)))}
    q["conv_b"], q["dt_bias"] = empty((5120,), torch.float32), empty((5120,), torch.float32)
    fw = {k: dev(v) for k, v in w.items()}
    for percentile in (0.37, 99.999):
        sc = Q.scales_to_dict(Q.quamba_calibrate(cfg, fw, dev(u), 1, M, percentile, q, ws))
        x = np.abs(_left_in_workspace(ws, cfg, M)[2]).reshape(-1)
        rank = max(int(math.ceil(percentile * x.size / 100.0)), 1) - 1
        v = np.partition(x, rank)[rank]
        assert v > 0 and np.float32(sc["s_x"]) == np.float32(np.float64(v) / 127.0)


@pytest.mark.parametrize("kind", ["plain", "ties", "zero"])
@pytest.mark.parametrize("percentile", [1e-7, 0.37, 50.0, 99.9, 99.999, 100.0])
def test_percentile_picks_the_value_of_its_rank(kind, percentile):
    """s_x is the value of rank ceil(p n / 100) of |x| over 127, exactly; ranks 1 and n are among them."""
    nb, L = 3, 19
    cfg, w, u = _case(80, 320, 48, nb, L)
    if kind != "plain":  # x = silu(conv_b): few values, or none but zero
        w["conv_w"] = np.zeros_like(w["conv_w"])
        w["conv_b"] = (np.resize([0.5, -0.25, 1.0, 0.5, 0.0, -3.0], w["conv_b"].shape) * (kind == "ties")).astype(np.float32)
    ws = workspace(Q.quamba_calibrate_workspace_bytes(cfg, nb, L))
    q = {k: empty(s, torch.int8) for k, s in (("W_in", (640, 80)), ("conv_w", (320, 4)), ("W_x", (80, 320)), ("W_dt", (320, 48)),
                                              ("A", (320, 16)), ("D", (320,)), ("W_outH", (80, 320)))}
    q["conv_b"], q["dt_bias"] = empty((320,), torch.float32), empty((320,), torch.float32)
    sc = Q.scales_to_dict(Q.quamba_calibrate(cfg, {k: dev(v) for k, v in w.items()}, dev(u), nb, L, percentile, q, ws))
    x = np.sort(np.abs(_left_in_workspace(ws, cfg, nb * L)[2]).reshape(-1))
    v = x[max(int(math.ceil(percentile * x.size / 100.0)), 1) - 1]
    want = np.float32(np.float64(v) / 127.0) if v > 0 else np.float32(1.0)
    assert np.float32(sc["s_x"]) == want
    assert (kind != "zero") or want == 1.0
