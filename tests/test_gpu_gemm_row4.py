"""GPU parity of the small-tile bf16 products whose rows start on 4 bytes only (gemm_ring.hip, the forms for longer sums).

A 16-byte load that holds the end of a row brings the next row's first values along; they are cleared in LDS.  The rows
reach every form at sums that end 2, 4 or 6 values into 16 bytes, in a slot's first or second part, with walks over k that
begin at, before and behind that slot, and with columns past the edge.  Bars as in test_gpu_gemm_ring.py: 6e-3 of the scale.
"""
import os
import re

import numpy as np
import pytest
import torch

from oracle import dense as OD
from paper_2410_07531_amd import binding as rov
from paper_2410_07531_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASES = [
    # M, N, K, transB; the tile: rows, columns, parts of k, bytes that rows start on
    (100, 1002, 1026, True, (64, 32, 4, 4)),
    (257, 4090, 2050, True, (128, 64, 2, 4)),
    (500, 6146, 2154, True, (128, 128, 2, 4)),
    (1100, 4090, 1070, True, (192, 128, 2, 4)),
    (1100, 4092, 1022, True, (192, 128, 2, 4)),          # columns in whole groups of four
    (130, 1002, 1092, False, (64, 64, 4, 4)),
    (257, 4094, 1090, False, (128, 64, 2, 4)),
    (900, 4090, 518, False, (128, 128, 2, 4)),
    (1530, 4090, 580, False, (192, 128, 2, 4)),
    (1530, 4090, 584, False, (192, 128, 2, 4)),          # A's rows on 16 bytes, the weights' on 4
]


def test_row4_cases_reach_every_form():
    seen = set()
    for M, N, K, transB, tile in CASES:
        assert rov.gemm_tile(M, N, K, rov.BF16, transB) == (rov.GEMM_SMALL_TILES,) + tile, (M, N, K, transB)
        seen.add((transB,) + tile)
    src = open(os.path.join(ROOT, "paper_2410_07531_amd", "csrc", "gemm_ring.hip")).read()
    table = re.findall(r"^\s*\{ROV_BF16, (\d), (\d+), (\d), (\d+), (\d+), .*, kRow4Slots\},$", src, flags=re.M)
    forms = {(kn == "0", int(bm), int(bn), int(ks), int(row)) for kn, row, ks, bm, bn in table}
    assert len(forms) == len(table) == 8 and seen == forms, seen ^ forms


def _operands(M, N, K, transB):
    rng = np.random.default_rng(M * 131 + N * 17 + K)
    a, w = wl.gemm_operands(rng, M, K, N)
    if not transB:
        w = np.ascontiguousarray(w.T)
    return torch.from_numpy(a).to(torch.bfloat16), torch.from_numpy(w).to(torch.bfloat16)


def _behind(t, fill, n=4096):
    buf = torch.full((t.numel() + n,), fill, dtype=t.dtype, device="cuda")
    buf[:t.numel()] = t.flatten().cuda()
    return buf[:t.numel()].view(t.shape)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,transB,tile", CASES)
def test_row4_tiles_match_oracle(M, N, K, transB, tile):
    print("gemm row4", M, N, K, transB, tile, flush=True)
    assert rov.gemm_tile(M, N, K, rov.BF16, transB) == (rov.GEMM_SMALL_TILES,) + tile
    A, W = _operands(M, N, K, transB)
    frame = torch.full((M * N + 128,), 3.0, dtype=torch.bfloat16, device="cuda")
    C = frame[64:64 + M * N].view(M, N)
    rov.gemm(_behind(A, float("nan")), _behind(W, float("nan")), C=C, transB=transB, scaleA=0.5, scaleB=4.0)
    torch.cuda.synchronize()
    assert bool((frame[:64] == 3.0).all()) and bool((frame[64 + M * N:] == 3.0).all())
    rows = sorted(set(r for r in (0, 1, 63, 64, 127, 128, 191, 192, 255, 256, 511, 512, M // 2, M - 2, M - 1) if 0 <= r < M))
    ref = 2.0 * OD.gemm(A[rows].float().numpy().astype(np.float64), W.float().numpy().astype(np.float64), transB=transB)
    got = C[rows].float().cpu().numpy().astype(np.float64)
    err = float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))
    assert err <= 6e-3, err


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,transB,dtype", [(70, 98, 102, True, "bf16"), (300, 258, 1026, True, "bf16"), (300, 258, 1026, False, "bf16"),
                                                (70, 45, 37, True, "f32"), (300, 131, 1001, False, "f32")])
def test_values_of_the_next_row_stay_there(M, N, K, transB, dtype):
    # infinities at the start of A's (and [N, K] weights') rows, where the last load of the row before them reaches
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    A = torch.ones((M, K), dtype=dt, device="cuda")
    W = torch.ones((N, K) if transB else (K, N), dtype=dt, device="cuda")
    rows, cols = [3, 64, M - 1], [7, 65 % N, N - 1] if transB else []
    A[rows, :4] = float("inf")
    if transB:
        W[cols, :4] = float("inf")
    C = rov.gemm(A, W, transB=transB).float()
    exp = torch.full((M, N), float(K), device="cuda").to(dt).float()
    exp[rows] = float("inf")
    exp[:, cols] = float("inf")
    assert torch.equal(C, exp)
