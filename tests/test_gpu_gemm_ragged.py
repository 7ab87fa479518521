"""GPU parity of the 256-row bf16 kernel where rows are no multiple of 128 bytes or columns no multiple of four (gemm.hip, RAGGED).

Every width, with k ending 1 to 7 chunks of 16 bytes into the last slot, that slot first, last or in the middle of the walk (the
start of the walk follows the tile row), a single slot, fewer rows and columns than a tile, and columns whose rows start on 8, 4
or 2 bytes.  Bar: 6e-3 of the scale (fp32 accumulation, one rounding to bf16).
"""
import numpy as np
import pytest
import torch

from oracle import dense as OD
from paper_2410_07531_amd import binding as rov
from paper_2410_07531_amd import workloads as wl

SHAPES = [(300, 1000, 1000), (257, 131, 72), (700, 514, 184), (256, 256, 8), (1, 1, 120), (1100, 333, 136), (513, 258, 64), (530, 1001, 1024)]


def test_which_products_take_it():
    tile = lambda M, N, K, tb=True, dt=rov.BF16: rov.gemm_tile(M, N, K, dt, tb)
    for M, N, K, cols in ((6935, 8514, 5960, 256), (7296, 4090, 4096, 256), (6798, 14336, 1000, 256), (3761, 14336, 4088, 224)):
        assert tile(M, N, K) == (rov.GEMM_256_ROWS, 256, cols, 1, 16), (M, N, K)
    for args in ((6935, 8514, 5956), (6935, 8512, 5960, False), (300, 1000, 1000), (4554, 1024, 1000)):
        assert tile(*args)[0] == rov.GEMM_SMALL_TILES, args
    assert tile(6000, 4098, 24)[0] == rov.GEMM_256_ROWS and tile(6000, 4099, 8)[0] == rov.GEMM_ANY_SHAPE


@pytest.mark.gpu
@pytest.mark.parametrize("cols", [128, 160, 192, 224, 256])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_ragged_256_row_tiles_match_oracle(M, N, K, cols):
    print("gemm ragged", M, N, K, cols, flush=True)
    rng = np.random.default_rng(M * 131 + N * 17 + K)
    a, w = wl.gemm_operands(rng, M, K, N)
    A, W = torch.from_numpy(a).to(torch.bfloat16), torch.from_numpy(w).to(torch.bfloat16)

    def behind(t):   # NaN behind the operands stays out of the result
        buf = torch.full((t.numel() + 4096,), float("nan"), dtype=t.dtype, device="cuda")
        buf[:t.numel()] = t.flatten().cuda()
        return buf[:t.numel()].view(t.shape)

    frame = torch.full((M * N + 128,), 3.0, dtype=torch.bfloat16, device="cuda")
    C = frame[64:64 + M * N].view(M, N)
    prev = rov.set_gemm_tile_cols(cols)
    try:
        assert rov.gemm_tile(M, N, K, rov.BF16) == (rov.GEMM_256_ROWS, 256, cols, 1, 16)
        rov.gemm(behind(A), behind(W), C=C, scaleA=0.5, scaleB=4.0)
        torch.cuda.synchronize()
    finally:
        rov.set_gemm_tile_cols(prev)
    assert bool((frame[:64] == 3.0).all()) and bool((frame[64 + M * N:] == 3.0).all())
    rows = sorted(set(r for r in (0, 1, 127, 128, 255, 256, 511, 512, M // 2, M - 2, M - 1) if 0 <= r < M))
    ref = 2.0 * OD.gemm(A[rows].float().numpy().astype(np.float64), W.float().numpy().astype(np.float64), transB=True)
    got = C[rows].float().cpu().numpy().astype(np.float64)
    err = float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))
    assert err <= 6e-3, err
