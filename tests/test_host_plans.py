"""Sizes and kernel choices that the library decides on the host: no GPU."""
import pytest

import paper_2410_13229_amd as Q
import workloads as W


@pytest.mark.parametrize("Dm,Di,R,nb,L", [(16, 16, 16, 1, 1), (80, 320, 48, 3, 19), (2560, 5120, 160, 4, 256)])
def test_calibration_takes_a_workspace_of_its_buffers_alone(Dm, Di, R, nb, L):
    """Input, x_pre | z, x, dt_low | B | C, dt, g and H g over the batch, the folded weight, A, 32 slots, one histogram and
    the clip search's area: a workspace that a program allocated once for a layer and batch stays large enough."""
    cfg = W.tiny_config(name="ws", d_model=Dm, d_inner=Di, dt_rank=R, config_id=94)
    M = nb * L
    words = [M * Dm, M * 2 * Di, M * Di, M * (R + 32), M * Di, M * Di, M * Di, Dm * Di, Di * 16, 32]
    want = sum((4 * n + 255) // 256 * 256 for n in words) + 256 * 8 + (Q.quamba_clip_search_workspace_bytes() + 255) // 256 * 256
    assert Q.quamba_calibrate_workspace_bytes(cfg, nb, L) <= want


@pytest.mark.parametrize("M,N,K,tiles", [
    (960, 288, 8192, 1), (961, 192, 4096, 1), (1216, 192, 5120, 1), (1216, 288, 8192, 1), (1217, 288, 5120, 5),
    (1024, 128, 8192, 2), (1088, 80, 8192, 2), (1216, 288, 3072, 5),   # two column groups, shallow K
    (16385, 192, 5120, 3), (20480, 288, 8192, 5), (16385, 80, 1536, 2),  # two row tiles per wave
    (8128, 192, 5120, 3),
])
def test_column_groups_of_xfmt_proj_are_spread_where_that_was_measured_to_pay(M, N, K, tiles):
    assert Q.quamba_debug_xfmt_column_tiles(M, N, K) == tiles


@pytest.mark.parametrize("M,N,K,taken", [
    (896, 2560, 5120, False), (897, 2560, 5120, True), (1152, 2560, 5120, True), (1153, 2560, 5120, False),
    (512, 4096, 8192, False), (513, 4096, 8192, True), (640, 4096, 8192, True), (641, 4096, 8192, False),
    (1408, 1712, 5632, True), (576, 4096, 4864, False), (1056, 2048, 4096, False), (1088, 2048, 4096, False), (1024, 3072, 768, False),
    (129, 9216, 4096, False), (160, 9376, 4608, False), (447, 4672, 5632, False), (319, 6416, 7168, False),  # one round of 64 x 64
    (130, 11264, 5376, False), (448, 5072, 4352, False), (288, 6608, 5120, False),  # little more than one
])
def test_128_by_96_tiles_are_taken_where_that_was_measured_to_pay(M, N, K, taken):
    assert (Q.quamba_debug_gemm_kind(M, N, K) == 14) == taken


@pytest.mark.parametrize("batch,L,Dm,Di,ahead", [
    (1, 512, 2560, 5120, True), (2, 256, 2560, 5120, True), (4, 512, 2560, 5120, True), (1, 256, 6144, 4096, True),
    (3, 512, 2560, 5120, False), (2, 512, 6144, 4096, False), (1, 256, 4096, 8192, False),  # no idle CUs in the last round
    (4, 1024, 768, 1536, False), (2, 512, 2048, 4096, False),                               # weights of 1 and 8 MB
    (1, 16, 6144, 2560, False), (1, 20, 6144, 2560, True),                                  # one state per lane: 47 ns a token
    (1, 4, 2560, 5120, True), (1, 1, 2560, 5120, False), (1, 16, 6144, 4096, False),        # scans shorter than the read
    (1, 1456, 2560, 5120, True), (1, 4096, 2560, 5120, False), (1, 1024, 6144, 4096, False),  # chunked scans
    (16, 32, 2560, 5120, True), (64, 16, 2560, 5120, True), (64, 1, 2560, 5120, False), (6, 96, 2560, 5120, False),
    (8, 512, 2560, 5120, False), (52, 9, 4096, 8192, False),                                # sweeps of many rounds
])
def test_last_block_reads_ahead_only_where_that_was_measured_to_pay(batch, L, Dm, Di, ahead):
    assert Q.quamba_debug_last_block_reads_ahead(batch, L, Dm, Di) == ahead


@pytest.mark.parametrize("n_layers,batch,Dm,Di,R,in_proj,out_proj", [
    (64, 64, 2560, 5120, 160, 2560 * 5120, 2560 * 5120), (64, 128, 2560, 5120, 160, 2560 * 5120, 2560 * 5120),
    (64, 129, 2560, 5120, 160, 0, 2560 * 5120), (64, 512, 2560, 5120, 160, 0, 2560 * 5120),  # too many sequences beside the norm
    (14, 3, 2048, 4096, 128, 2048 * 4096, 2048 * 4096),                                       # half of in_proj, not all
    (4, 64, 4096, 8192, 256, 16 << 20, 0), (4, 65, 4096, 8192, 256, 16 << 20, 4096 * 8192),   # 33 MB outlast a short Hadamard launch
    (6, 3, 3072, 6144, 192, 16 << 20, 3072 * 6144), (3, 256, 5120, 10240, 320, 0, 5120 * 10240),
    (6, 3, 2560, 5120, 160, 0, 0), (7, 3, 2560, 5120, 160, 2560 * 5120, 2560 * 5120),         # the stack stays in the cache, or not
])
def test_generation_reads_weights_ahead_where_that_was_measured_to_pay(n_layers, batch, Dm, Di, R, in_proj, out_proj):
    got = [Q.quamba_debug_decode_reads_ahead(n_layers, batch, Dm, Di, R, k) for k in (0, 1)]
    assert got == [in_proj, out_proj]
