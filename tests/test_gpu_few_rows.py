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
