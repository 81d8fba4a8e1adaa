"""The 128 x 96 tiles of the int8 GEMM: ragged edges against the oracle, and the sums where the planner takes them."""
import numpy as np
import pytest

import oracle as O
from gpu_util import Q, dev, empty, host, torch, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(128, 96, 256), (129, 100, 512), (300, 700, 768), (37, 604, 1280), (257, 332, 2560)])
def test_tiles_of_128_by_96_forced_onto_ragged_shapes(M, N, K):
    """One to ten slices of K, rows and columns past the last whole tile: integer sums, hence equal codes and halves."""
    rng = np.random.default_rng(M + N + K)
    A, Wt = (rng.integers(-128, 128, s, dtype=np.int8) for s in ((M, K), (N, K)))
    acc_ref = O.int_matmul(A, Wt)
    mult = np.array([3.1e-5, 7.7e-5, 1.9e-4], dtype=np.float32)
    e0, e1 = N // 16 * 4, N // 8 * 4
    want = np.concatenate([O.requant_acc(acc_ref[:, a:b], m) for a, b, m in ((0, e0, mult[0]), (e0, e1, mult[1]), (e1, N, mult[2]))], axis=1)
    acc, out, outh = empty((M, N), torch.int32), empty((M, N), torch.int8), empty((M, N), torch.float16)
    Q.quamba_debug_set_gemm_variant(14)
    try:
        Q.quamba_gemm_i8(dev(A), K, dev(Wt), K, M, N, K, e0, e1, mult, out, None, N, acc)
        Q.quamba_gemm_i8(dev(A), K, dev(Wt), K, M, N, K, N, N, mult, None, outh, N, None)
    finally:
        Q.quamba_debug_set_gemm_variant(-1)
    assert np.array_equal(host(acc), acc_ref) and np.array_equal(host(out), want)
    assert np.array_equal(host(outh).view(np.uint16), (acc_ref.astype(np.float32) * mult[0]).astype(np.float16).view(np.uint16))


@pytest.mark.parametrize("M,N,K,taken", [(896, 2560, 5120, False), (897, 2560, 5120, True), (1152, 2560, 5120, True),
                                         (1153, 2560, 5120, False), (520, 4096, 8192, True)])
def test_planned_tiles_give_the_sums_of_the_64_by_64_ones(M, N, K, taken):
    """Either side of the row counts at which the planner changes over (189 and 270 tiles are outside its range)."""
    assert (Q.quamba_debug_gemm_kind(M, N, K) == 14) == taken
    g = torch.Generator(device="cuda:0").manual_seed(M)
    A, Wt = (torch.randint(-128, 128, s, dtype=torch.int8, device="cuda:0", generator=g) for s in ((M, K), (N, K)))
    mult, ws, got = np.array([1e-5] * 3, dtype=np.float32), workspace(Q.quamba_gemm_workspace_bytes(M, N, K)), []
    for kind in (-1, 5):
        Q.quamba_debug_set_gemm_variant(kind)
        try:
            got.append(empty((M, N), torch.float16))
            Q.quamba_gemm_i8(A, K, Wt, K, M, N, K, N, N, mult, None, got[-1], N, None, ws)
        finally:
            Q.quamba_debug_set_gemm_variant(-1)
    assert torch.equal(got[0], got[1])
