"""GPU parity of the small-tile GEMM kernels (gemm_ring.hip) at the sizes where they can go wrong.

The rows reach every tile and operand form, and assert which one: tiles of 32 to 192 rows, k split between the waves of a
workgroup or not, [K, N] weights, rows that start on 16 or only on 4 bytes, a last slot of k that is
partly filled, rows and columns past the edge, output rows that take no vector store.  Reference:
the float64 oracle on sampled rows (first, last, tile edges), all columns.

Bars: bf16 and fp8 6e-3 of the result's scale (fp32 accumulation and one rounding to bf16, 2^-9, with room
for the maximum), fp32 1e-5 (sums of at most 4096 terms of like size: sqrt(4096) * 2^-24 = 4e-6).
"""
import numpy as np
import pytest
import torch

from oracle import dense as OD
from oracle import numerics as ON
from paper_2410_07531_amd import binding as rov
from paper_2410_07531_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, M, N, K, transB; the tile: rows, columns, parts of k, bytes of a lane's load
    ("bf16", 100, 4096, 2048, True, (64, 32, 4, 16)),
    ("bf16", 250, 4096, 2112, True, (64, 64, 2, 16)),   # two 128-byte parts per slot, odd number of parts
    ("bf16", 333, 4096, 2048, True, (128, 64, 2, 16)),
    ("bf16", 500, 6144, 2176, True, (128, 128, 2, 16)),
    ("bf16", 1100, 4100, 2048, True, (192, 128, 2, 16)),   # ragged columns
    ("bf16", 1000, 6144, 2048, True, (128, 192, 2, 16)),
    ("bf16", 70, 1000, 448, True, (64, 64, 1, 16)),
    ("bf16", 700, 4096, 1024, True, (128, 128, 1, 16)),
    ("bf16", 1, 4, 64, True, (64, 64, 1, 16)),   # smallest
    ("bf16", 129, 65, 8, True, (64, 32, 4, 16)),   # one chunk of k, odd number of columns
    ("bf16", 333, 1001, 1000, True, (64, 32, 4, 16)),   # last slot partly filled, scalar stores
    ("bf16", 65, 130, 102, True, (64, 64, 2, 4)),
    ("bf16", 64, 64, 64, False, (64, 64, 4, 16)),   # one tile, one slot
    ("bf16", 257, 4096, 1032, False, (128, 64, 2, 16)),   # last slot of one chunk
    ("bf16", 1000, 1000, 72, False, (64, 64, 4, 16)),   # ragged everywhere
    ("bf16", 900, 4096, 264, False, (128, 128, 2, 16)),   # last slot of one chunk
    ("bf16", 900, 6144, 256, False, (192, 128, 2, 16)),
    ("bf16", 3000, 4096, 256, False, (192, 128, 2, 16)),
    ("bf16", 130, 98, 34, False, (64, 64, 2, 4)),
    ("fp8", 100, 4096, 512, True, (64, 64, 1, 16)),
    ("fp8", 333, 4096, 640, True, (128, 64, 1, 16)),
    ("fp8", 500, 8192, 384, True, (128, 128, 1, 16)),
    ("fp8", 77, 131, 144, True, (64, 64, 1, 16)),   # last slot partly filled, scalar stores
    ("f32", 256, 256, 256, True, (32, 32, 4, 16)),
    ("f32", 1, 1, 1, True, (32, 32, 4, 4)),   # smallest
    ("f32", 1000, 1024, 260, True, (64, 64, 2, 16)),   # last slot of one chunk
    ("f32", 33, 47, 131, True, (32, 32, 4, 4)),
    ("f32", 900, 1025, 513, True, (64, 64, 2, 4)),
    ("f32", 100, 36, 68, False, (32, 32, 4, 16)),
    ("f32", 1024, 1024, 64, False, (64, 64, 2, 16)),
    ("f32", 65, 33, 35, False, (32, 32, 4, 4)),
    ("f32", 957, 1027, 67, False, (64, 64, 2, 4)),
]


def _operands(dtype, M, N, K, transB):
    rng = np.random.default_rng(M * 131 + N * 17 + K)
    a, w = wl.gemm_operands(rng, M, K, N)
    if not transB:
        w = np.ascontiguousarray(w.T)
    if dtype == "fp8":
        A = torch.from_numpy(a * np.float32(16)).to(torch.float8_e4m3fn).view(torch.uint8)
        W = torch.from_numpy(w * np.float32(256)).to(torch.float8_e4m3fn).view(torch.uint8)
        return A.cuda(), W.cuda(), ON.e4m3_decode(A.numpy()), ON.e4m3_decode(W.numpy())
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    A, W = torch.from_numpy(a).to(dt), torch.from_numpy(w).to(dt)
    return A.cuda(), W.cuda(), A.float().numpy().astype(np.float64), W.float().numpy().astype(np.float64)


DTYPES = {"bf16": rov.BF16, "fp8": rov.FP8_E4M3, "f32": rov.F32}


@pytest.mark.parametrize("dtype,M,N,K,transB,tile", CASES)
def test_small_tiles_match_oracle(dtype, M, N, K, transB, tile):
    print("gemm ring", dtype, M, N, K, transB, tile, flush=True)
    assert rov.gemm_tile(M, N, K, DTYPES[dtype], transB) == (rov.GEMM_SMALL_TILES,) + tile
    if dtype != "fp8":       # what an earlier workgroup left in LDS must not reach a partly filled slot
        dt = torch.bfloat16 if dtype == "bf16" else torch.float32
        nan = torch.full((512, 512), float("nan"), dtype=dt, device="cuda")
        rov.gemm(nan, nan, transB=transB)
    A, W, a, w = _operands(dtype, M, N, K, transB)
    odt = torch.float32 if dtype == "f32" else torch.bfloat16
    # a frame of known values around the result: nothing outside it is written
    frame = torch.full((M * N + 128,), 3.0, dtype=odt, device="cuda")
    C = frame[64:64 + M * N].view(M, N)
    rov.gemm(A, W, C=C, transB=transB, scaleA=0.5, scaleB=4.0)
    torch.cuda.synchronize()
    assert bool((frame[:64] == 3.0).all()) and bool((frame[64 + M * N:] == 3.0).all())
    rows = sorted(set(r for r in (0, 1, 31, 32, 63, 64, 127, 128, 191, 192, 255, 256, M // 2, M - 2, M - 1) if 0 <= r < M))
    ref = 2.0 * OD.gemm(a[rows], w, transB=transB)
    got = C[rows].float().cpu().numpy().astype(np.float64)
    err = float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))
    assert err <= (1e-5 if dtype == "f32" else 6e-3), err


@pytest.mark.parametrize("dtype,M,N,K,transB", [
    ("bf16", 70, 36, 64, True), ("bf16", 333, 4096, 2112, True), ("bf16", 65, 130, 102, True), ("bf16", 257, 264, 72, False),
    ("fp8", 77, 131, 144, True), ("f32", 33, 36, 36, True), ("f32", 33, 47, 131, True), ("f32", 65, 36, 68, False),
])
def test_memory_behind_the_operands_is_not_part_of_the_result(dtype, M, N, K, transB):
    # rows past the edge, the partly filled last slot and the loads issued past the end of the walk over k (all of them,
    # where the ring has more slots than the sum) lie outside the operands' ranges: NaN behind A and W changes nothing
    print("gemm ring behind", dtype, M, N, K, transB, flush=True)
    A, W, _, _ = _operands(dtype, M, N, K, transB)

    def framed(t, fill):
        buf = torch.full((t.numel() + 64 * K + 4096,), fill, dtype=t.dtype, device="cuda")
        buf[:t.numel()] = t.flatten()
        return buf[:t.numel()].view(t.shape)

    nan = 0x7F if dtype == "fp8" else float("nan")
    C = rov.gemm(framed(A, nan), framed(W, nan), transB=transB)
    C0 = rov.gemm(framed(A, 0), framed(W, 0), transB=transB)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(C.float()).all()) and torch.equal(C, C0)


@pytest.mark.parametrize("dtype,M,N,K,tile", [
    ("bf16", 300, 2048, 1024, (64, 64)), ("bf16", 700, 4096, 512, (128, 128)),
    ("fp8", 300, 2048, 4096, (64, 64)), ("fp8", 333, 4096, 640, (128, 64)), ("fp8", 500, 8192, 384, (128, 128)),
])
def test_unsplit_small_tiles_give_the_256_row_kernels_bits(dtype, M, N, K, tile):
    print("gemm ring bits", dtype, M, N, K, tile, flush=True)
    assert rov.gemm_tile(M, N, K, DTYPES[dtype])[:4] == (rov.GEMM_SMALL_TILES,) + tile + (1,)
    A, W, _, _ = _operands(dtype, M, N, K, True)
    C = rov.gemm(A, W)
    prev = rov.set_gemm_tile_cols(128)
    try:
        assert rov.gemm_tile(M, N, K, DTYPES[dtype])[0] == rov.GEMM_256_ROWS
        C2 = rov.gemm(A, W)
        torch.cuda.synchronize()
    finally:
        rov.set_gemm_tile_cols(prev)
    assert torch.equal(C.view(torch.int16), C2.view(torch.int16))


def test_long_sums_have_the_same_bits_at_every_forced_width():
    # from K = 2048 on the small tiles may add partial sums over k: the default product is then another rounding of the same
    # sum, while the forced widths keep one order, whatever M is
    M, N, K = 333, 4096, 4096
    assert rov.gemm_tile(M, N, K, rov.BF16) == (rov.GEMM_SMALL_TILES, 128, 64, 2, 16)
    A, W, _, _ = _operands("bf16", M, N, K, True)
    got = {}
    for cols in (0, 128, 160, 192, 224, 256):
        prev = rov.set_gemm_tile_cols(cols)
        try:
            got[cols] = rov.gemm(A, W)
            if cols == 256:
                part = rov.gemm(A[:100], W)
        finally:
            rov.set_gemm_tile_cols(prev)
    torch.cuda.synchronize()
    for cols in (160, 192, 224, 256):
        assert torch.equal(got[cols], got[128]), cols
    assert torch.equal(part, got[128][:100])
    # fp32 sums of 4096 terms in two orders: 4e-6 of the scale apart (see above) and then rounded to bf16, so that a few
    # results on the edge between two neighbours differ by one of 2^-8
    far = (got[0].float() - got[128].float()).abs()
    assert float((far > 0).float().mean()) < 0.02
    assert bool((far <= 2.0 ** -7 * got[128].float().abs() + 1e-5 * got[128].float().abs().max()).all())


def test_fp32_product_keeps_infinities_and_nan_in_their_rows():
    # a non-finite operand reaches the outputs of its own row or column only
    A = torch.ones((70, 37), device="cuda")
    W = torch.ones((45, 37), device="cuda")
    A[3, 36] = float("inf")
    W[7, 0] = float("nan")
    C = rov.gemm(A, W)
    exp = torch.full((70, 45), 37.0, device="cuda")
    exp[3] = float("inf")
    exp[:, 7] = float("nan")
    assert torch.equal(torch.nan_to_num(C, nan=-1.0), torch.nan_to_num(exp, nan=-1.0))


@pytest.mark.parametrize("K", [3840, 3842])
@pytest.mark.parametrize("transB", [True, False])
def test_fp32_tiles_of_both_sizes_round_alike(K, transB):
    # The error of a long sum grows with the root of its chain of additions: k / 4 terms with either tile.  Over 65536 results and more its norm
    # scatters by under 2 %; chains of k / 2 would show as a ratio of 1.41.
    err = {}
    for M, N, tile in ((256, 256, (32, 32, 4)), (2048, 2048, (64, 64, 2))):
        assert rov.gemm_tile(M, N, K, rov.F32, transB)[1:4] == tile
        g = torch.Generator("cuda").manual_seed(K + M)
        A = torch.randn(M, K, device="cuda", generator=g)
        W = torch.randn(*((N, K) if transB else (K, N)), device="cuda", generator=g)
        ref = A.double() @ (W.double().t().contiguous() if transB else W.double())
        C = rov.gemm(A, W, transB=transB)
        err[tile[0]] = float((C.double() - ref).norm() / ref.norm())
    assert err[64] <= 1.15 * err[32], err


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("M,N,K", [
    (300, 14336, 128),       # ragged rows
    (2900, 2820, 1024),      # ragged columns (five blocks: last tile 20 of 80)
    (2304, 3300, 256),       # nine tile rows: every start of the walk over k
    (70, 4, 128),            # one tile, four columns: fewer than one block
    (257, 60, 256),          # fewer columns than one wave's half of any tile
])
def test_dual_tiles_of_every_width_give_the_same_bits(dtype, M, N, K):
    # every width forced, and the one chosen from the shape, against the widest (whose parity has its own tests)
    print("dual", dtype, M, N, K, flush=True)
    A, Wg, _, _ = _operands(dtype, M, N, K, True)
    g = torch.Generator("cuda").manual_seed(N)
    Wu = Wg[torch.randperm(N, device="cuda", generator=g)].contiguous()
    run = (lambda: rov.gemm_swiglu(A, Wg, Wu)) if dtype == "bf16" else (lambda: rov.gemm_swiglu_fp8(A, Wg, Wu, 1 / 16, 1 / 64, 1 / 64, 0.25))
    got = {}
    for cols in (0, 128, 160, 192, 224, 256):
        prev = rov.set_gemm_tile_cols(cols)
        try:
            assert cols == 0 or rov.gemm_swiglu_tile_cols(M, N, K, DTYPES[dtype]) == cols // 2
            got[cols] = run()
            torch.cuda.synchronize()
        finally:
            rov.set_gemm_tile_cols(prev)
    for cols in (0, 128, 160, 192, 224):
        assert torch.equal(got[cols], got[256]), cols
    assert got[256].float().abs().max() > 0


@pytest.mark.parametrize("dtype,M,N,K,transB", [("bf16", 333, 4096, 4096, True), ("bf16", 1000, 1000, 2056, False),
                                                ("f32", 256, 256, 1000, True), ("fp8", 333, 4096, 640, True)])
def test_split_sums_repeat_bit_for_bit(dtype, M, N, K, transB):
    # the parts of k are added in a fixed order: repeated calls, on other streams and beside other work too, give the same bits
    A, W, _, _ = _operands(dtype, M, N, K, transB)
    ref = rov.gemm(A, W, transB=transB)
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [torch.full_like(ref, 7.0) for _ in range(24)]
    torch.cuda.synchronize()
    for i, C in enumerate(outs):
        rov.gemm(A, W, C=C, transB=transB, stream=streams[i % 3])
    torch.cuda.synchronize()
    assert all(torch.equal(C, ref) for C in outs)
