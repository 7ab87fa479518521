"""The C-ABI library loads and exports every symbol include/rov.h declares (no GPU needed)."""
import ctypes
import os
import re

from paper_2410_07531_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "rov.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(rov_[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_are_exported_and_bound():
    names = _declared()
    assert "rov_dropout_mask_generate" in names and "rov_gemm" in names
    assert os.path.exists(binding.LIB_PATH), "build the library first (__graft_entry__.build())"
    lib = ctypes.CDLL(binding.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), "librov.so does not export %s" % n
    assert sorted(binding.SIGNATURES) == names


def test_host_only_entry_points():
    L = binding.load()
    assert L.rov_version().startswith(b"rov")
    assert binding.mask_words(1, 2, 128) == 2 * 4 * 4 * 16
    assert binding.mask_words(1, 1, 70) == 3 * 3 * 16
    assert binding.mask_words(0, 1, 70) == 0
    assert binding.mask_philox_calls(1, 2, 128) == 64 * 128
    assert binding.mask_philox_calls(1, 1, 70) == 64 * 36
    assert binding.mask_philox_calls(1, 1, 1) == 64 * 4
    assert binding.mask_shape(2, 3, 70) == (2, 3, 3, 3, 16)
    assert L.rov_last_hip_error() == 0


def test_gemm_tile_width_rule():
    # host logic: the width that leaves least of the last round of workgroups empty (256 compute
    # units), widest on ties; the limiter model's copy of the rule must agree with the library's
    from paper_2410_07531_amd import limiter_model as LM
    assert binding.gemm_tile_cols(2048, 14336) == 224      # 448 tiles of 256 -> 512 tiles of 224: two full rounds
    assert binding.gemm_tile_cols(2048, 6144) == 192       # 192 tiles -> 256 tiles: one full round
    assert binding.gemm_tile_cols(2048, 4096) == 128
    assert binding.gemm_tile_cols(8192, 8192) == 256 and binding.gemm_tile_cols(16384, 14336) == 256
    assert binding.gemm_tile_cols(1, 4) == 128             # one tile either way: the narrowest is the cheapest
    for M in (1, 256, 300, 2048, 4096, 8192, 16384):
        for N in range(4, 20000, 364):
            assert binding.gemm_tile_cols(M, N) == LM.gemm_tile_cols(LM.MI355X, M, N), (M, N)
    for esz, dt in ((2, binding.BF16), (1, binding.FP8_E4M3)):
        for M in (1, 70, 300, 949, 2000, 2048, 2900, 4096, 16384):
            for N in (4, 300, 2816, 2820, 8192, 14336, 28672):
                for K in (128, 1024, 4096):
                    assert binding.gemm_swiglu_tile_cols(M, N, K, dt) == 16 * LM.dual_tile_blocks(LM.MI355X, M, N, K, esz), (M, N, K, dt)
    # what the model prices as a 256-row kernel is one, in the workloads that it is applied to
    for S in (2048, 4096, 8192, 16384, 32768):
        for N, K in ((6144, 4096), (4096, 4096), (4096, 14336)):
            assert binding.gemm_tile(S, N, K, binding.BF16)[:3] == (binding.GEMM_256_ROWS, 256, LM.gemm_tile_cols(LM.MI355X, S, N))
    L = binding.load()
    assert L.rov_gemm_tile_cols(0, 8) == binding.ERR_INVALID and L.rov_gemm_tile_cols(8, -1) == binding.ERR_INVALID
    prev = binding.set_gemm_tile_cols(160)
    try:
        assert binding.gemm_tile_cols(8192, 8192) == 160
    finally:
        binding.set_gemm_tile_cols(prev)
    assert binding.gemm_tile_cols(8192, 8192) == 256


def test_kernel_choice_queries():
    # host logic: what the launches choose, so that a test can assert the kernel that it means to reach
    B = binding
    assert B.gemm_tile(16384, 14336, 4096, B.BF16) == (B.GEMM_256_ROWS, 256, 256, 1, 16)
    assert B.gemm_tile(333, 4096, 2048, B.BF16) == (B.GEMM_SMALL_TILES, 128, 64, 2, 16)
    assert B.gemm_tile(65, 130, 102, B.BF16) == (B.GEMM_SMALL_TILES, 64, 64, 2, 4)
    assert B.gemm_tile(77, 130, 101, B.BF16) == (B.GEMM_ANY_SHAPE, 64, 64, 1, 2)      # rows off 4 bytes
    assert B.gemm_tile(256, 256, 256, B.FP8_E4M3, transB=False)[0] == B.GEMM_ANY_SHAPE
    for cols in (128, 160, 192, 224, 256):
        prev = B.set_gemm_tile_cols(cols)
        try:
            assert B.gemm_tile(333, 4096, 2048, B.BF16) == (B.GEMM_256_ROWS, 256, cols, 1, 16)
            assert B.gemm_swiglu_tile_cols(333, 4096, 2048, B.FP8_E4M3) == cols // 2
        finally:
            B.set_gemm_tile_cols(prev)
    assert B.gemm_swiglu_tile_cols(2000, 14336, 4096, B.BF16) == 112
    for bad in ((0, 4, 4, B.BF16), (4, 4, 4, 7)):
        try:
            B.gemm_tile(*bad)
            assert False
        except B.RovError as e:
            assert e.code == B.ERR_INVALID
    assert B.attention_key_parts(1, 32, 16384, 128, B.BF16, False) == 1
    assert B.attention_key_parts(1, 2, 128, 64, B.BF16, True) == 4
    assert [B.attention_key_parts(1, 2, 128, d, B.F32, False) for d in (40, 64, 128, 100, 136)] == [8, 8, 4, 0, 0]
    assert B.attention_key_parts(1, 2, 128, 96, B.BF16, False) == 0
    chunks = lambda H, S: (B.mask_words(1, H, S) + 63) // 64
    assert B.overlap_mask_chunks(0.0, B.BF16, 1, 8, 512) == 0
    assert B.overlap_mask_chunks(1e15, B.BF16, 1, 32, 16384) == chunks(32, 16384)
    assert B.overlap_mask_chunks(1e9, B.BF16, 1, 32, 16384) == -1
    assert 0 < B.overlap_mask_chunks(4e9, B.BF16, 1, 8, 1024) < chunks(8, 1024)


def test_small_tile_cases_reach_every_form():
    # every row of the small-tile GEMM's parity tests names the tile that it reaches (the tests assert it); together they are
    # all the forms that the launch chooses from
    import test_gpu_gemm_ring as T
    import test_gpu_gemm_row4 as T4
    seen = set()
    for dtype, M, N, K, transB, tile in T.CASES + [("bf16",) + case for case in T4.CASES]:
        assert binding.gemm_tile(M, N, K, T.DTYPES[dtype], transB) == (binding.GEMM_SMALL_TILES,) + tile, (dtype, M, N, K)
        seen.add((dtype, transB) + tile)
    src = open(os.path.join(ROOT, "paper_2410_07531_amd", "csrc", "gemm_ring.hip")).read()
    table = re.findall(r"^\s*\{ROV_(BF16|FP8_E4M3|F32), (\d), (\d+), (\d), (\d+), (\d+), ", src, flags=re.M)
    forms = {({"BF16": "bf16", "FP8_E4M3": "fp8", "F32": "f32"}[t], kn == "0", int(bm), int(bn), int(ks), int(vec))
             for t, kn, vec, ks, bm, bn in table}
    assert len(forms) == len(table) == 33 and seen == forms, seen ^ forms


def test_small_tiles_only_where_they_are_sooner():
    # products that were measured 5 to 28 % slower with small tiles than with the 256-row kernel, and some that are faster
    B = binding
    for dt, M, N, K in ((B.FP8_E4M3, 400, 10240, 8192), (B.FP8_E4M3, 700, 8192, 8192), (B.FP8_E4M3, 1200, 4096, 14336),
                        (B.FP8_E4M3, 300, 14336, 4096), (B.FP8_E4M3, 950, 5120, 8192), (B.BF16, 600, 10240, 8192),
                        (B.BF16, 1600, 10240, 8192), (B.BF16, 3000, 8192, 8192), (B.BF16, 3600, 5120, 8192),
                        (B.BF16, 1100, 7168, 7168), (B.BF16, 1100, 14336, 4096)):
        assert B.gemm_tile(M, N, K, dt)[0] == B.GEMM_256_ROWS, (dt, M, N, K)
    for dt, M, N, K in ((B.BF16, 333, 4096, 4096), (B.BF16, 512, 4096, 14336), (B.BF16, 1000, 6144, 4096), (B.BF16, 1024, 4096, 4096),
                        (B.FP8_E4M3, 300, 4096, 14336), (B.FP8_E4M3, 512, 4096, 4096)):
        assert B.gemm_tile(M, N, K, dt)[0] == B.GEMM_SMALL_TILES, (dt, M, N, K)


def test_fp32_products_take_the_tile_that_is_sooner():
    # measured 9 to 14 % slower with 32 x 32 tiles, and 8 to 20 % slower with 64 x 64
    B = binding
    for M, N, K, tb in ((2922, 3880, 3800, False), (2414, 2500, 1304, False), (1497, 4040, 1796, False), (930, 2024, 1756, False), (550, 1732, 1780, False),
                        (1972, 984, 1680, False), (376, 2652, 1972, True), (2048, 4096, 4096, True)):
        assert B.gemm_tile(M, N, K, B.F32, tb)[1:3] == (64, 64), (M, N, K, tb)
    for M, N, K, tb in ((256, 256, 256, True), (442, 1176, 2640, True), (430, 1484, 932, True), (676, 1686, 1034, False), (1214, 449, 1049, True),
                        (1023, 1340, 672, False), (1939, 1164, 1220, False)):
        assert B.gemm_tile(M, N, K, B.F32, tb)[1:3] == (32, 32), (M, N, K, tb)


def test_very_short_sums_take_the_any_shape_kernel():
    # sums of a few terms into large outputs were measured up to 1.7 times as long with the small tiles, the longer ones below up to twice
    # as long with the any-shape kernel
    B = binding
    for dt, M, N, K, tb in ((B.BF16, 1500, 4098, 2, True), (B.BF16, 6000, 4096, 2, False), (B.BF16, 4154, 3759, 2, True), (B.BF16, 6000, 4098, 6, False),
                            (B.F32, 5000, 6001, 2, True), (B.FP8_E4M3, 6000, 1001, 16, True), (B.FP8_E4M3, 5368, 4803, 16, True)):
        assert B.gemm_tile(M, N, K, dt, tb)[0] == B.GEMM_ANY_SHAPE, (dt, M, N, K, tb)
    for dt, M, N, K, tb in ((B.BF16, 1500, 4098, 102, True), (B.BF16, 1500, 1000, 30, False), (B.BF16, 6000, 1000, 8, True),
                            (B.F32, 200, 1000, 40, True), (B.F32, 1500, 1000, 102, False), (B.F32, 6000, 4098, 200, True),
                            (B.FP8_E4M3, 6000, 1001, 48, True), (B.FP8_E4M3, 1500, 4096, 112, True),
                            (B.BF16, 1500, 4098, 30, False), (B.BF16, 4176, 5322, 68, True), (B.BF16, 2757, 6526, 44, True), (B.BF16, 2265, 4366, 34, False),
                            (B.F32, 1500, 4098, 30, True), (B.F32, 6000, 4096, 16, True), (B.F32, 6000, 4098, 62, False), (B.F32, 3166, 1195, 65, False)):
        assert B.gemm_tile(M, N, K, dt, tb)[0] == B.GEMM_SMALL_TILES, (dt, M, N, K, tb)


def test_key_parts_leave_full_chips_alone():
    # causal problems that fill the chip take workgroups of 256 rows: with two key parts these shapes were measured 2 to 20 %
    # slower (stored mask and no dropout); and short ones keep their split
    parts = lambda B, H, S, d: binding.attention_key_parts(B, H, S, d, binding.BF16, True)
    for B, H, S, d in ((2, 32, 7232, 64), (2, 32, 3000, 64), (1, 32, 8192, 64), (4, 32, 2500, 64), (1, 16, 6000, 128),
                       (1, 24, 3500, 128), (2, 20, 1700, 128), (2, 32, 4096, 128)):
        assert parts(B, H, S, d) == 1, (B, H, S, d)
    assert parts(2, 32, 384, 128) < 4 and parts(4, 32, 333, 64) < 4
    for B, H, S, d in ((1, 2, 33, 64), (2, 16, 1000, 64), (1, 32, 512, 128), (1, 16, 2048, 128)):
        assert parts(B, H, S, d) == 4, (B, H, S, d)
    assert parts(1, 32, 2048, 128) == 2 and parts(1, 32, 4096, 64) == 2


def test_fp32_attention_of_a_few_rows_takes_a_row_a_wave():
    # even with tiles of 16 rows or sooner up to 4 tokens, 1.2 to 1.9 times as fast as tiles of 32 rows for a few tokens of many heads; and
    # slower elsewhere (tiles of 16 rows: 1 x 16 x 64 4.7 us against 5.2, 1 x 37 x 128 6.2 against 8.7, 32 x 57 x 96 6.3 against 13.6)
    waves = lambda heads, S, d: binding.attention_key_parts(1, heads, S, d, binding.F32, False)
    for heads, S, d in ((1, 1, 8), (1, 4, 64), (8, 4, 128), (300, 3, 128), (256, 9, 64), (512, 9, 40), (512, 8, 128), (512, 4, 32)):
        assert waves(heads, S, d) == 0, (heads, S, d)
    for heads, S, d in ((1, 5, 64), (1, 16, 64), (1, 33, 128), (8, 32, 96), (32, 16, 128), (128, 8, 64), (1, 65, 8), (2, 128, 64), (32, 64, 128),
                        (128, 48, 64), (512, 32, 128), (512, 33, 64), (32, 56, 96)):
        assert waves(heads, S, d) == (8 if d <= 64 else 4), (heads, S, d)


def test_fp32_query_tiles_of_16_rows_only_where_they_are_sooner():
    # without the causal mask these problems, of 144 to 192 tiles of 32 rows, were measured 1.04 to 1.5 times as long with tiles of 16
    rows = lambda B, H, S, d, causal: binding.attention_tile_rows(B, H, S, d, binding.F32, causal)
    for B, H, S, d in ((1, 3, 1616, 128), (2, 3, 763, 128), (1, 1, 5106, 8), (1, 1, 5597, 64), (2, 1, 2725, 32), (2, 6, 493, 128), (1, 6, 788, 32),
                       (1, 8, 687, 8), (1, 16, 313, 128), (1, 32, 134, 128)):
        assert rows(B, H, S, d, False) == 32 and rows(B, H, S, d, True) == 16, (B, H, S, d)
    for B, H, S, d in ((1, 2, 128, 64), (1, 2, 400, 128), (1, 16, 256, 64), (1, 5, 816, 128), (2, 16, 139, 64), (1, 32, 168, 8)):
        assert rows(B, H, S, d, False) == 16 and rows(B, H, S, d, True) == 16, (B, H, S, d)
    assert rows(2, 8, 1000, 64, True) == 32 and rows(1, 1, 1, 8, True) == 1
    assert binding.attention_tile_rows(1, 32, 16384, 128, binding.BF16, False) == 256
    assert binding.attention_tile_rows(1, 2, 128, 64, binding.BF16, True) == 64 and binding.attention_tile_rows(1, 2, 128, 96, binding.BF16, True) == 1
    assert binding.load().rov_attention_tile_rows(1, 2, 0, 64, binding.F32, 0) == binding.ERR_INVALID


def test_key_parts_never_ask_for_more_workgroups_than_a_grid_holds():
    # 2^30 (batch, head) pairs (views with zero strides) fit the grid with 256 rows a workgroup or one row a wave, which
    # is what such calls are accepted for, but not with the 32, 64 or 128 rows of the finer forms
    B = H = 32768
    assert binding.attention_key_parts(B, H, 64, 64, binding.F32, False) == 0
    assert binding.attention_key_parts(B, H, 32, 64, binding.F32, False) == 8
    assert binding.attention_key_parts(B // 4, H, 96, 64, binding.F32, False) == 8
    for d in (64, 128):
        for causal in (False, True):
            assert binding.attention_key_parts(B, H, 256, d, binding.BF16, causal) == 1


def test_no_oracle_on_the_product_path():
    # the package must never import the oracle (and the oracle never the package)
    pkg = os.path.join(ROOT, "paper_2410_07531_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                src = open(os.path.join(dirpath, f)).read()
                assert not re.search(r"^\s*(from|import)\s+oracle\b", src, flags=re.M), f
                assert "liboracle" not in src and "philox_oracle" not in src, f
    for f in os.listdir(os.path.join(ROOT, "oracle")):
        if f.endswith((".py", ".c")):
            src = open(os.path.join(ROOT, "oracle", f)).read()
            assert not re.search(r"^\s*(from|import)\s+paper_2410_07531_amd\b", src, flags=re.M), f
            assert "librov" not in src, f
