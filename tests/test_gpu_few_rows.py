"""Generation with a few sequences: the launches that carry a neighbour's work give the bits of the separate kernels."""
import numpy as np
import pytest

import oracle as O  # noqa: F401  (the workloads build on it)
import workloads as W
from gpu_util import Q, dev, empty, host, make_taps, oracle_setup, qweights_to_dev, torch, workspace

pytestmark = pytest.mark.gpu


def _step(cfg, qd, sc, u, Bt, names):
    g = np.random.default_rng(3)
    ssm = dev((g.standard_normal((Bt, cfg.d_inner, 16)) * 0.1).astype(np.float32))
    cs = dev((g.standard_normal((Bt, cfg.d_inner, 3)) * 0.5).astype(np.float16))
    out = empty((Bt, cfg.d_model), torch.float16)
    Q.quamba_mixer_decode(cfg, qd, sc, dev(u[:, 0]), Bt, out, ssm, cs, make_taps(cfg, Bt, names) if names else None,
                          workspace(Q.quamba_workspace_bytes(cfg, Bt, 1)))
    return host(out).view(np.uint16), host(ssm), host(cs).view(np.uint16)


@pytest.mark.parametrize("Dm,Di,Bt", [
    (80, 1536, 1),   # 96 items: half of the second wave has none
    (208, 1536, 3),  # column groups that are not a multiple of eight
    (96, 2560, 2),   # 160 items: two and a half waves
    (128, 1024, 1),  # whole waves
])
def test_fused_launches_give_the_bits_of_the_separate_kernels(Dm, Di, Bt):
    """Integer sums and the same fp32 operations in the same order: equal, not close.  The u_q tap takes the quantization out of
    in_proj's launch, the gH_f32 tap the Hadamard transform out of out_proj's."""
    cfg = W.tiny_config(name="few", d_model=Dm, d_inner=Di, dt_rank=16, batch=Bt, seqlen=1, config_id=96)
    _, qw, sc = oracle_setup(cfg)
    qd, u = qweights_to_dev(qw), W.make_hidden(cfg, batch=Bt, seqlen=1, stream=13)
    want = _step(cfg, qd, sc, u, Bt, ["u_q", "gH_f32"])
    for names in (None, ["u_q"], ["gH_f32"], ["gH_q"]):
        for a, b in zip(_step(cfg, qd, sc, u, Bt, names), want):
            assert np.array_equal(a, b), names


@pytest.mark.parametrize("Dm,Di,Bt", [(768, 1536, 1), (208, 1536, 3), (1280, 2560, 2)])
def test_fused_out_proj_rounds_the_product_before_the_conversion(Dm, Di, Bt):
    """out = fp16(fp32(sum * m_out)).  With m_out a power of two over 3, rounded up to fp32, sums of 3 b have products that fp32
    rounds to b, halfway between two halves for every fourth b or so: rounded once they go up, rounded twice to even."""
    cfg = W.tiny_config(name="few", d_model=Dm, d_inner=Di, dt_rank=16, batch=Bt, seqlen=1, config_id=96)
    _, qw, sc = oracle_setup(cfg)
    qd, u = qweights_to_dev(qw), W.make_hidden(cfg, batch=Bt, seqlen=1, stream=13)
    m = np.float32(2.0 ** -14 / 3)
    sc = {**sc, "m_out": float(m), "inv_s_y": 8.0 * sc["inv_s_y"]}  # large codes: sums that spread over many of these b
    taps = make_taps(cfg, Bt, ["acc_out"])
    g = np.random.default_rng(3)
    ssm = (g.standard_normal((Bt, Di, 16)) * 0.1).astype(np.float32)
    cs = (g.standard_normal((Bt, Di, 3)) * 0.5).astype(np.float16)
    out, ws = empty((Bt, Dm), torch.float16), workspace(Q.quamba_workspace_bytes(cfg, Bt, 1))
    Q.quamba_mixer_decode(cfg, qd, sc, dev(u[:, 0]), Bt, out, dev(ssm), dev(cs), taps, ws)  # the tap takes the separate kernels
    acc, separate = host(taps["acc_out"]), host(out).view(np.uint16)
    want = (acc.astype(np.float32) * m).astype(np.float16).view(np.uint16)
    once = (acc.astype(np.float64) * np.float64(m)).astype(np.float16).view(np.uint16)
    assert np.count_nonzero(want != once) >= 5  # the inputs tell the two roundings apart
    Q.quamba_mixer_decode(cfg, qd, sc, dev(u[:, 0]), Bt, out, dev(ssm), dev(cs), None, ws)
    assert np.array_equal(separate, want) and np.array_equal(host(out).view(np.uint16), want)
