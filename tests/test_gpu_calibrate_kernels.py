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


@pytest.mark.parametrize("Dm,Di,R,nb,L", [
    (48, 16, 16, 1, 1),      # half a block of channels, one token, K = 16 and 48: a part of a slice
    (80, 320, 48, 1, 31),    # one row tile of 32, not full
    (64, 192, 16, 1, 33),    # 64-row tiles
    (64, 192, 16, 2, 32),    # exactly one 64-row tile; exactly one block of tokens
    (80, 320, 48, 5, 13),    # 65 rows: 128-row tiles
    (768, 1536, 48, 3, 43),  # 129 rows; skinny outputs of a long K
])
def test_fp32_forward_at_tile_edges(Dm, Di, R, nb, L):
    """fp32 sums of up to 1536 products against fp64: errors of about sqrt(K) 2^-24 per sum, 40 x 6e-8 = 2.4e-6 of the
    sum's scale, through three projections and a decaying recurrence: 1e-5 of the largest output."""
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


@pytest.mark.parametrize("Dm,Di,R,nb,L", [(80, 320, 48, 3, 47), (768, 1536, 48, 6, 43)])
def test_order_of_the_fp32_sums_does_not_depend_on_the_tile(Dm, Di, R, nb, L):
    """Every fp32 output is one chain of multiply-adds over K, so a sequence gives the same bits alone (32- or 64-row tiles, the
    skinny form) and in a batch (128-row tiles): scales, and with them int8 codes, do not move with the batch's shape."""
    cfg, w, u = _case(Dm, Di, R, nb, L)
    fw = {k: dev(v) for k, v in w.items()}
    ws = workspace(Q.quamba_calibrate_workspace_bytes(cfg, nb, L))
    whole, one = empty((nb, L, Dm), torch.float32), empty((1, L, Dm), torch.float32)
    Q.quamba_mixer_fp32(cfg, fw, dev(u), nb, L, whole, ws)
    for b in range(nb):
        Q.quamba_mixer_fp32(cfg, fw, dev(np.ascontiguousarray(u[b:b + 1])), 1, L, one, ws)
        assert np.array_equal(host(one)[0], host(whole)[b])
