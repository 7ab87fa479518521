"""GPU parity for the schedules and the transformer block.

The three schedules must give the same attention output bit for bit (same mask bits, same
kernels' arithmetic), and each matches the oracle within the bf16 bar (2e-2 of the output scale).
"""
import numpy as np
import pytest
import torch

from oracle import dense as OD
from oracle import philox as OP
from paper_2410_07531_amd import binding as rov
from paper_2410_07531_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _f64(t):
    return t.float().cpu().numpy().astype(np.float64)


def _dev(x, dtype=torch.bfloat16):
    return torch.from_numpy(x).to(dtype).cuda()


@pytest.mark.parametrize("dtype,B,S,H,Hkv,d,gemm", [
    (torch.float32, 1, 128, 2, 2, 64, (256, 256, 256)),        # tiny workload
    (torch.bfloat16, 1, 512, 4, 2, 128, (512, 256, 768)),
])
def test_layer_step_three_schedules(dtype, B, S, H, Hkv, d, gemm):
    rng = np.random.default_rng(11)
    q, k, v = wl.qkv(rng, B, S, H, Hkv, d)
    Q, K, V = _dev(q, dtype), _dev(k, dtype), _dev(v, dtype)
    M, Kd, N = gemm
    a, w = wl.gemm_operands(rng, M, Kd, N)
    A, W = _dev(a, dtype), _dev(w, dtype)
    p, seed, offset = 0.1, wl.SEED, wl.OFFSET
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    outs, cs = [], []
    for sched in (rov.SCHED_SEQUENTIAL, rov.SCHED_FUSED, rov.SCHED_OVERLAP):
        print("layer_step", dtype, sched, flush=True)
        O = torch.zeros_like(Q)
        C = torch.zeros((M, N), dtype=torch.float32 if dtype == torch.float32 else torch.bfloat16, device="cuda")
        mask = torch.full(rov.mask_shape(B, H, S), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda")  # poison
        torch.cuda.synchronize()
        gd = [rov.make_gemm_desc(A, W, C)]
        ad = rov.make_attn_desc(Q, K, V, O, p)
        for _ in range(2):   # twice: the second pass reuses the events and the mask buffer
            rov.layer_step(sched, gd, ad, seed, offset, None if sched == rov.SCHED_FUSED else mask, main, side)
        torch.cuda.synchronize()
        outs.append(O)
        cs.append(C)
        if sched != rov.SCHED_FUSED:
            assert np.array_equal(mask.cpu().numpy().view(np.uint64), OP.dropout_mask(seed, offset, B, H, S, p))
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert torch.equal(cs[0], cs[1]) and torch.equal(cs[0], cs[2])
    keep = OP.unpack_keep(OP.dropout_mask(seed, offset, B, H, S, p), S)
    ref = OD.attention_dropout(_f64(Q), _f64(K), _f64(V), keep, p)
    tol = 2e-2 if dtype == torch.bfloat16 else 1e-4
    assert np.max(np.abs(_f64(outs[0]) - ref)) / np.max(np.abs(ref)) <= tol
    refc = OD.gemm(_f64(A), _f64(W), transB=True)
    assert np.max(np.abs(_f64(cs[0]) - refc)) / np.max(np.abs(refc)) <= (6e-3 if dtype == torch.bfloat16 else 1e-5)


@pytest.mark.parametrize("M,N,K,B,H,S", [
    (600, 1000, 448, 1, 2, 256),      # ragged tile edges, odd slot count; 24 tiles, 128 chunks: the waves beside the tiles get most of them
    (256, 128, 64, 2, 4, 1024),       # one tile, one slot-step: nearly the whole mask (8192 chunks) is left to the launch behind
    (2048, 2048, 1024, 1, 1, 64),     # 128 tiles, one chunk: most RNG waves find the queue empty
    (512, 512, 256, 1, 3, 320),       # 75 chunks over 8 tiles
])
def test_gemm_rng_single_kernel_matches_oracle(M, N, K, B, H, S):
    # the wave-specialised single kernel (paper Sec. 6.1): its GEMM against the oracle, its mask bit
    # for bit against the oracle's, twice in a row (the queue slot changes, the result must not)
    print("gemm_rng_fused", M, N, K, B, H, S, flush=True)
    rng = np.random.default_rng(M + N + K + S)
    a, w = wl.gemm_operands(rng, M, K, N)
    A, W = _dev(a, torch.bfloat16), _dev(w, torch.bfloat16)
    p, seed, offset = 0.1, wl.SEED, wl.CARRY_OFFSET - 2048          # some chunks cross 2^32
    words = OP.dropout_mask(seed, offset, B, H, S, p)
    refc = OD.gemm(_f64(A), _f64(W), transB=True)
    st = torch.cuda.Stream()
    for rep in range(2):
        C = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
        mask = torch.full(rov.mask_shape(B, H, S), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda")   # poison
        torch.cuda.synchronize()
        rov.gemm_rng_fused(A, W, seed, offset, B, H, S, p, C=C, mask=mask, stream=st)
        torch.cuda.synchronize()
        assert np.array_equal(mask.cpu().numpy().view(np.uint64), words), rep
        assert np.max(np.abs(_f64(C) - refc)) / np.max(np.abs(refc)) <= 6e-3, rep
    # same bits as the two-kernel path's GEMM with the same tile
    prev = rov.set_gemm_tile_cols(128)
    try:
        C2 = rov.gemm(A, W, transB=True)
        torch.cuda.synchronize()
    finally:
        rov.set_gemm_tile_cols(prev)
    assert torch.equal(C, C2)


def test_gemm_rng_single_kernel_argument_errors():
    A = torch.zeros((256, 64), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((128, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(rov.RovError):
        rov.gemm_rng_fused(A, W, 1, 0, 1, 1, 48, 0.1)              # S % 32 != 0
    with pytest.raises(rov.RovError):
        rov.gemm_rng_fused(A, W, 1, 0, 1, 1, 64, 1.0)              # p outside [0, 1)
    with pytest.raises(rov.RovError):
        rov.gemm_rng_fused(A[:, :32], W[:, :32].contiguous(), 1, 0, 1, 1, 64, 0.1)   # K % 64 != 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("sched", [rov.SCHED_SEQUENTIAL, rov.SCHED_FUSED, rov.SCHED_OVERLAP])
def test_layer_step_replays_from_a_captured_graph(sched):
    # a caller may record the step into a HIP graph (the library allocates nothing, synchronises
    # nothing and clears its work queue with a kernel): every replay, with eager steps and
    # synchronisations between the replays, must reproduce the eager result
    B, S, H, Hkv, d = 1, 320, 4, 2, 128
    rng = np.random.default_rng(31)
    q, k, v = wl.qkv(rng, B, S, H, Hkv, d)
    Q, K, V = [_dev(x, torch.bfloat16) for x in (q, k, v)]
    a, w = wl.gemm_operands(rng, 512, 256, 768)
    A, W = _dev(a, torch.bfloat16), _dev(w, torch.bfloat16)
    p, seed, offset = 0.1, wl.SEED, 1280
    O = torch.zeros_like(Q)
    C = torch.zeros((512, 768), dtype=torch.bfloat16, device="cuda")
    mask = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    gd, ad = [rov.make_gemm_desc(A, W, C)], rov.make_attn_desc(Q, K, V, O, p)

    def step():
        rov.layer_step(sched, gd, ad, seed, offset, None if sched == rov.SCHED_FUSED else mask, main, side)

    torch.cuda.synchronize()
    step()
    torch.cuda.synchronize()
    O_ref, C_ref, m_ref = O.clone(), C.clone(), mask.clone()
    if sched != rov.SCHED_FUSED:
        assert np.array_equal(m_ref.cpu().numpy().view(np.uint64), OP.dropout_mask(seed, offset, B, H, S, p))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=main):
        step()
    torch.cuda.synchronize()
    for r in range(4):
        print("graph replay", sched, r, flush=True)
        O.zero_()
        C.zero_()
        mask.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(main):
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, O_ref) and torch.equal(C, C_ref), r
        if sched != rov.SCHED_FUSED:
            assert torch.equal(mask, m_ref), r
        step()                       # eager work between the replays
        torch.cuda.synchronize()


def test_layer_step_overlap_from_two_host_threads():
    # two host threads enqueue overlap steps at the same time, each on its own pair of streams with its own
    # buffers and seed (ctypes releases the interpreter lock during the calls).  The library serialises the
    # enqueue phase of its schedule entry points and shares one set of fork / join events between them (and the work-queue
    # slots of larger masks: test_gpu_mask_queue.py): every thread must end with the oracle's mask for its seed and with the outputs a
    # single-threaded run gives, bit for bit.
    import threading
    B, H, Hkv, d = 1, 4, 2, 128
    cases = [dict(S=512, gemm=(256, 128, 256), seed=wl.SEED),            # RNG outlasts the GEMM: split, helper launch
             dict(S=256, gemm=(1024, 512, 1024), seed=wl.SEED + 77)]     # RNG fits beside the GEMM: plain launch
    p, reps = 0.1, 12
    for i, c in enumerate(cases):
        rng = np.random.default_rng(50 + i)
        q, k, v = wl.qkv(rng, B, c["S"], H, Hkv, d)
        a, w = wl.gemm_operands(rng, *c["gemm"])
        c["Q"], c["K"], c["V"], c["A"], c["W"] = [_dev(x) for x in (q, k, v, a, w)]
        c["main"], c["side"] = torch.cuda.Stream(), torch.cuda.Stream()

    def run(c, tag):
        M, Kd, N = c["gemm"]
        O = torch.zeros_like(c["Q"])
        C = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
        mask = torch.full(rov.mask_shape(B, H, c["S"]), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        gd = [rov.make_gemm_desc(c["A"], c["W"], C)]
        ad = rov.make_attn_desc(c["Q"], c["K"], c["V"], O, p)
        try:
            for _ in range(reps):
                rov.layer_step(rov.SCHED_OVERLAP, gd, ad, c["seed"], wl.OFFSET, mask, c["main"], c["side"])
        except Exception as e:      # a thread's exception would otherwise be lost
            c[tag] = e
            return
        c[tag] = (O, C, mask)

    print("two threads: single-threaded reference runs", flush=True)
    for c in cases:
        run(c, "ref")
    torch.cuda.synchronize()
    print("two threads: concurrent runs", flush=True)
    threads = [threading.Thread(target=run, args=(c, "got")) for c in cases]
    for t in threads:
        t.start()
    for t in threads:
        t.join(120)
        assert not t.is_alive()
    torch.cuda.synchronize()
    for c in cases:
        assert not isinstance(c["ref"], Exception), c["ref"]
        assert not isinstance(c["got"], Exception), c["got"]
        (O0, C0, m0), (O1, C1, m1) = c["ref"], c["got"]
        words = OP.dropout_mask(c["seed"], wl.OFFSET, B, H, c["S"], p)
        assert np.array_equal(m0.cpu().numpy().view(np.uint64), words)
        assert np.array_equal(m1.cpu().numpy().view(np.uint64), words)
        assert torch.equal(O0, O1) and torch.equal(C0, C1)
        keep = OP.unpack_keep(words, c["S"])
        ref = OD.attention_dropout(_f64(c["Q"]), _f64(c["K"]), _f64(c["V"]), keep, p)
        assert np.max(np.abs(_f64(O1) - ref)) / np.max(np.abs(ref)) <= 2e-2


@pytest.mark.parametrize("rounds", [3, 5, 7, 10])
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float32, 64)])
def test_layer_step_rounds_three_schedules(rounds, dtype, d):
    # fewer Philox rounds (paper Sec. 5.2): the mask kernel and the fused attention must still drop
    # the same elements, those of the oracle's mask with that round count
    B, S, H, Hkv = 1, 320, 2, 1
    rng = np.random.default_rng(21)
    q, k, v = wl.qkv(rng, B, S, H, Hkv, d)
    Q, K, V = _dev(q, dtype), _dev(k, dtype), _dev(v, dtype)
    a, w = wl.gemm_operands(rng, 256, 256, 256)
    A, W = _dev(a, dtype), _dev(w, dtype)
    p, seed, offset = 0.3, 77, wl.CARRY_OFFSET - 640        # the mask's calls cross 2^32
    words = OP.dropout_mask(seed, offset, B, H, S, p, rounds=rounds)
    if rounds != 10:
        assert not np.array_equal(words, OP.dropout_mask(seed, offset, B, H, S, p))
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    for sched in (rov.SCHED_SEQUENTIAL, rov.SCHED_FUSED, rov.SCHED_OVERLAP):
        print("layer_step_rounds", rounds, dtype, sched, flush=True)
        O = torch.zeros_like(Q)
        C = torch.zeros((256, 256), dtype=dtype, device="cuda")
        mask = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        rov.layer_step(sched, [rov.make_gemm_desc(A, W, C)], rov.make_attn_desc(Q, K, V, O, p), seed, offset,
                       None if sched == rov.SCHED_FUSED else mask, main, side, rounds=rounds)
        torch.cuda.synchronize()
        outs.append(O)
        if sched != rov.SCHED_FUSED:
            assert np.array_equal(mask.cpu().numpy().view(np.uint64), words)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    ref = OD.attention_dropout(_f64(Q), _f64(K), _f64(V), OP.unpack_keep(words, S), p)
    tol = 2e-2 if dtype == torch.bfloat16 else 1e-4
    assert np.max(np.abs(_f64(outs[0]) - ref)) / np.max(np.abs(ref)) <= tol
    # the stand-alone attention entry point with a round count: same bits as the mask of that count
    O2 = rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, rounds=rounds)
    torch.cuda.synchronize()
    assert torch.equal(O2, outs[0])


@pytest.mark.parametrize("bits", [8, 16, 32])
@pytest.mark.parametrize("dtype,d,S", [(torch.bfloat16, 128, 320), (torch.bfloat16, 64, 200), (torch.float32, 64, 100)])
def test_layer_step_bits_three_schedules(bits, dtype, d, S):
    # narrower random numbers (paper Sec. 5.2): the mask kernel writes the oracle's mask of that width,
    # and the three schedules (the fused kernel draws the same fields itself) drop exactly its elements
    B, H, Hkv = 1, 2, 2
    rng = np.random.default_rng(22)
    q, k, v = wl.qkv(rng, B, S, H, Hkv, d)
    Q, K, V = _dev(q, dtype), _dev(k, dtype), _dev(v, dtype)
    a, w = wl.gemm_operands(rng, 256, 256, 256)
    A, W = _dev(a, dtype), _dev(w, dtype)
    p, seed, offset = 0.1, 78, wl.CARRY_OFFSET - 320          # the calls cross 2^32
    words = OP.dropout_mask_bits(seed, offset, B, H, S, p, bits)
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    for sched in (rov.SCHED_SEQUENTIAL, rov.SCHED_FUSED, rov.SCHED_OVERLAP):
        print("layer_step_bits", bits, dtype, sched, flush=True)
        O = torch.zeros_like(Q)
        C = torch.zeros((256, 256), dtype=dtype, device="cuda")
        mask = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        rov.layer_step(sched, [rov.make_gemm_desc(A, W, C)], rov.make_attn_desc(Q, K, V, O, p), seed, offset,
                       None if sched == rov.SCHED_FUSED else mask, main, side, bits=bits)
        torch.cuda.synchronize()
        if sched != rov.SCHED_FUSED:
            assert np.array_equal(mask.cpu().numpy().view(np.uint64), words)
        outs.append(O)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    ref = OD.attention_dropout(_f64(Q), _f64(K), _f64(V), OP.unpack_keep(words, S), p)
    tol = 2e-2 if dtype == torch.bfloat16 else 1e-4
    assert np.max(np.abs(_f64(outs[0]) - ref)) / np.max(np.abs(ref)) <= tol
    O2 = rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, bits=bits)
    torch.cuda.synchronize()
    assert torch.equal(O2, outs[0])
    with pytest.raises(rov.RovError):
        rov.layer_step(rov.SCHED_OVERLAP, [], rov.make_attn_desc(Q, K, V, O, p), seed, offset, mask, main, side,
                       bits=12)
    with pytest.raises(rov.RovError):
        rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, bits=4)


def test_layer_step_rounds_rejects_other_counts():
    Q = torch.zeros((1, 64, 1, 64), dtype=torch.bfloat16, device="cuda")
    O = torch.zeros_like(Q)
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    mask = torch.zeros(rov.mask_shape(1, 1, 64), dtype=torch.int64, device="cuda")
    for bad in (0, 4, 6, 11, -7):
        with pytest.raises(rov.RovError):
            rov.layer_step(rov.SCHED_OVERLAP, [], rov.make_attn_desc(Q, Q, Q, O, 0.1), 1, 0, mask, main, side,
                           rounds=bad)
        with pytest.raises(rov.RovError):
            rov.attention_fwd_dropout(Q, Q, Q, 0.1, seed=1, offset=0, rounds=bad)


def test_layer_step_invalid_arguments():
    Q = torch.zeros((1, 64, 2, 64), dtype=torch.bfloat16, device="cuda")
    O = torch.zeros_like(Q)
    ad = rov.make_attn_desc(Q, Q, Q, O, 0.1)
    s = torch.cuda.Stream()
    with pytest.raises(rov.RovError):
        rov.layer_step(rov.SCHED_OVERLAP, [], ad, 1, 0, None, s, torch.cuda.Stream())      # mask missing
    mask = torch.zeros(rov.mask_shape(1, 2, 64), dtype=torch.int64, device="cuda")
    with pytest.raises(rov.RovError):
        rov.layer_step(rov.SCHED_OVERLAP, [], ad, 1, 0, mask, s, s)                        # same stream
    with pytest.raises(rov.RovError):
        rov.layer_step(7, [], ad, 1, 0, mask, s, torch.cuda.Stream())


def _block_setup(B, S, H, Hkv, d, hidden, ffn, seed):
    rng = np.random.default_rng(seed)
    w = wl.block_weights(rng, H, Hkv, d, hidden, ffn)
    # non-trivial norm weights so that a dropped scale would show
    w["norm1"] = (1.0 + 0.1 * rng.standard_normal(hidden)).astype(np.float32)
    w["norm2"] = (1.0 + 0.1 * rng.standard_normal(hidden)).astype(np.float32)
    for kname in ("wqkv", "wo", "wg", "wu", "wd"):
        w[kname] = w[kname] * np.float32(3.0)     # sd 0.06: keeps every stage's contribution visible
    x = wl.block_input(rng, B, S, hidden)
    wd = {k_: _dev(v_) for k_, v_ in w.items()}
    return _dev(x), wd


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,S,H,Hkv,d", [(1, 256, 4, 2, 128),
                                         (2, 200, 6, 3, 64)])     # two batches, ragged sequence, head dimension 64
def test_block_forward_three_schedules_match_oracle(causal, B, S, H, Hkv, d):
    hidden, ffn = 512, 1024
    p, seed, offset = 0.1, wl.SEED, 640
    x, wd = _block_setup(B, S, H, Hkv, d, hidden, ffn, 21)
    cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, p, causal=causal)
    weights = rov.make_block_weights(wd)
    ws = torch.empty(rov.block_workspace_bytes(cfg, B, S, 0), dtype=torch.uint8, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    ys = {}
    for name, sched, ready in (("seq", rov.SCHED_SEQUENTIAL, False), ("fused", rov.SCHED_FUSED, False),
                               ("ovl_first", rov.SCHED_OVERLAP, False), ("ovl_steady", rov.SCHED_OVERLAP, True)):
        print("block", name, causal, flush=True)
        y = torch.zeros_like(x)
        mask = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
        nxt = torch.zeros_like(mask) if name == "ovl_steady" else None
        if ready:
            rov.dropout_mask_generate(seed, offset, B, H, S, p, out=mask)
        torch.cuda.synchronize()
        rov.block_forward(weights, x, y, cfg, sched, seed, offset, None if sched == rov.SCHED_FUSED else mask,
                          ws, main, side, mask_ready=ready, next_mask=nxt)
        torch.cuda.synchronize()
        ys[name] = y
        if nxt is not None:
            exp = OP.dropout_mask(seed, offset + OP.mask_philox_calls(B, H, S), B, H, S, p)
            got = nxt.cpu().numpy().view(np.uint64)
            if causal:      # only the tiles causal attention reads are guaranteed
                T = (S + 31) // 32
                lower = np.tril(np.ones((T, T), dtype=bool))
                assert np.array_equal(got[:, :, lower], exp[:, :, lower])
            else:
                assert np.array_equal(got, exp)
    for name in ("fused", "ovl_first", "ovl_steady"):
        assert torch.equal(ys["seq"], ys[name]), name
    keep = OP.unpack_keep(OP.dropout_mask(seed, offset, B, H, S, p), S)
    ocfg = dict(H=H, Hkv=Hkv, d=d, eps=1e-5, rope_theta=500000.0, p=p, causal=causal)
    ref = OD.block_forward(_f64(x), {k_: _f64(v_) for k_, v_ in wd.items()}, ocfg, keep)
    got = _f64(ys["seq"])
    assert np.max(np.abs(got - ref)) / np.max(np.abs(ref)) <= 2e-2
    # the block is not the identity: the residual branches are visible at this tolerance
    assert np.max(np.abs(ref - _f64(x))) / np.max(np.abs(ref)) > 0.1


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("rows", [-1, 64, 160, 320])
def test_block_forward_hybrid_equals_the_other_schedules(rows, causal):
    # hybrid: stored bits for the first R query rows, in-kernel Philox for the rest; R forced to
    # none, a part (tile-aligned and not), and all of S = 320: always the sequential schedule's bits,
    # both when the block makes its own mask and in steady state (mask made by the block before)
    B, S, H, Hkv, d, hidden, ffn = 1, 320, 4, 2, 128, 512, 1024
    p, seed, offset = 0.1, wl.SEED, 640
    x, wd = _block_setup(B, S, H, Hkv, d, hidden, ffn, 23)
    cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, p, causal=causal)
    weights = rov.make_block_weights(wd)
    ws = torch.empty(rov.block_workspace_bytes(cfg, B, S, 0), dtype=torch.uint8, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    calls = rov.mask_philox_calls(B, H, S)
    y_seq, y_seq2 = torch.zeros_like(x), torch.zeros_like(x)
    m = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    rov.block_forward(weights, x, y_seq, cfg, rov.SCHED_SEQUENTIAL, seed, offset, m, ws, main, side)
    rov.block_forward(weights, x, y_seq2, cfg, rov.SCHED_SEQUENTIAL, seed, offset + calls, m, ws, main, side)
    torch.cuda.synchronize()
    prev = rov.set_block_hybrid_mask_rows(rows)
    try:
        R = rov.block_hybrid_mask_rows(cfg, B, S)
        assert R == (0 if rows < 0 else rows - rows % 32)
        y1, y2 = torch.zeros_like(x), torch.zeros_like(x)
        m0 = torch.full(rov.mask_shape(B, H, S), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda")
        m1 = torch.full_like(m0, 0x2AAAAAAAAAAAAAAA)
        torch.cuda.synchronize()
        print("hybrid", rows, causal, "first block", flush=True)
        rov.block_forward(weights, x, y1, cfg, rov.SCHED_HYBRID, seed, offset, m0, ws, main, side, next_mask=m1)
        torch.cuda.synchronize()
        print("hybrid", rows, causal, "steady state", flush=True)
        rov.block_forward(weights, x, y2, cfg, rov.SCHED_HYBRID, seed, offset + calls, m1, ws, main, side,
                          mask_ready=True, next_mask=m0)
        torch.cuda.synchronize()
    finally:
        rov.set_block_hybrid_mask_rows(prev)
    assert torch.equal(y1, y_seq) and torch.equal(y2, y_seq2)
    if 0 < R:
        # the rows that were stored are those of the full mask of the next layer
        full = OP.dropout_mask(seed, offset + calls, B, H, S, p)             # [B, H, T, T, 16]
        got = m1.cpu().numpy().view(np.uint64).reshape(-1)[: B * H * (R // 32) * (S // 32) * 16]
        got = got.reshape(B, H, R // 32, S // 32, 16)
        if causal and R == S:     # the whole-mask kernel skips the tiles causal attention never reads
            lower = np.tril(np.ones((S // 32, S // 32), dtype=bool))
            assert np.array_equal(got[:, :, lower], full[:, :, lower])
        else:
            assert np.array_equal(got, full[:, :, : R // 32])


def test_block_hybrid_rows_rule():
    # host rule: everything fits at the benchmark's 16K block, a part at 32K, in steps of 2048 rows
    cfg = rov.make_block_cfg(32, 8, 128, 4096, 14336, 0.1)
    assert rov.block_hybrid_mask_rows(cfg, 1, 2048) == 2048
    assert rov.block_hybrid_mask_rows(cfg, 1, 8192) == 8192
    r32 = rov.block_hybrid_mask_rows(cfg, 1, 32768)
    assert 0 < r32 < 32768 and r32 % 2048 == 0
    r64 = rov.block_hybrid_mask_rows(cfg, 1, 65536)
    assert 0 <= r64 < 65536 and r64 % 2048 == 0 and r64 / 65536 < r32 / 32768


def test_block_forward_same_bits_for_every_gemm_tile_width():
    # the residual and SwiGLU epilogues of every width of the matrix-core GEMM kernel: the block's
    # output must not depend on the width (same k order per element, same epilogue arithmetic)
    B, S, H, Hkv, d, hidden, ffn = 1, 320, 4, 2, 128, 512, 1088
    p, seed, offset = 0.1, wl.SEED, 64
    x, wd = _block_setup(B, S, H, Hkv, d, hidden, ffn, 22)
    cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, p)
    weights = rov.make_block_weights(wd)
    ws = torch.empty(rov.block_workspace_bytes(cfg, B, S, 0), dtype=torch.uint8, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    ys = {}
    for cols in (0, 128, 160, 192, 224, 256):
        print("block width", cols, flush=True)
        y = torch.zeros_like(x)
        torch.cuda.synchronize()
        prev = rov.set_gemm_tile_cols(cols)
        try:
            rov.block_forward(weights, x, y, cfg, rov.SCHED_FUSED, seed, offset, None, ws, main, side)
            torch.cuda.synchronize()
        finally:
            rov.set_gemm_tile_cols(prev)
        ys[cols] = y
    for cols in (128, 160, 192, 224, 256):
        assert torch.equal(ys[0], ys[cols]), cols
    keep = OP.unpack_keep(OP.dropout_mask(seed, offset, B, H, S, p), S)
    ocfg = dict(H=H, Hkv=Hkv, d=d, eps=1e-5, rope_theta=500000.0, p=p, causal=False)
    ref = OD.block_forward(_f64(x), {k_: _f64(v_) for k_, v_ in wd.items()}, ocfg, keep)
    assert np.max(np.abs(_f64(ys[256]) - ref)) / np.max(np.abs(ref)) <= 2e-2


def test_block_workspace_and_argument_errors():
    B, S, H, Hkv, d, hidden, ffn = 1, 64, 2, 2, 64, 128, 256
    x, wd = _block_setup(B, S, H, Hkv, d, hidden, ffn, 3)
    cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, 0.1)
    weights = rov.make_block_weights(wd)
    need = rov.block_workspace_bytes(cfg, B, S, 0)
    T = B * S
    assert need >= 2 * T * (2 * hidden + (H + 2 * Hkv) * d + H * d + ffn)     # h, x2, qkv, att, u
    ws = torch.empty(need - 256, dtype=torch.uint8, device="cuda")
    y = torch.full_like(x, 5.0)
    mask = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    with pytest.raises(rov.RovError) as e:
        rov.block_forward(weights, x, y, cfg, rov.SCHED_SEQUENTIAL, 1, 0, mask, ws, s1, s2)
    assert e.value.code == rov.ERR_WORKSPACE
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    with pytest.raises(rov.RovError):
        rov.block_forward(weights, x, y, cfg, rov.SCHED_SEQUENTIAL, 1, 0, None, ws, s1, s2)     # mask missing
    with pytest.raises(rov.RovError):
        rov.block_forward(weights, x, y, cfg, rov.SCHED_SEQUENTIAL, 1, 0, mask, ws, s1, s2, next_mask=mask.clone())
    torch.cuda.synchronize()
    assert bool((y == 5.0).all())


@pytest.mark.parametrize("causal", [False, True])
def test_block_forward_fp8_matches_oracle(causal):
    # fp8 block: e4m3 weights with per-tensor scales, the four activations quantised where they are
    # produced (normalisation kernel, attention epilogue, FC1 epilogue); against the oracle's fp8 block
    from oracle import numerics as ON
    B, S, H, Hkv, d, hidden, ffn = 1, 256, 4, 2, 128, 512, 1024
    p, seed, offset = 0.1, wl.SEED, 1920
    rng = np.random.default_rng(27)
    w = wl.block_weights(rng, H, Hkv, d, hidden, ffn)
    w["norm1"] = (1.0 + 0.1 * rng.standard_normal(hidden)).astype(np.float32)
    w["norm2"] = (1.0 + 0.1 * rng.standard_normal(hidden)).astype(np.float32)
    x = wl.block_input(rng, B, S, hidden)
    wq, ws, wdev = {}, {}, {}
    for name in ("wqkv", "wo", "wg", "wu", "wd"):
        wq[name], ws[name] = ON.e4m3_quantise(w[name] * np.float32(3.0))    # sd 0.06: every stage stays visible
        wdev[name] = torch.from_numpy(wq[name]).cuda()
    for name in ("norm1", "norm2"):
        wdev[name] = _dev(w[name])
        wq[name] = _f64(wdev[name])
    X = _dev(x)
    act = [float(np.float32(v)) for v in (6.0 / 448.0, 6.0 / 448.0, 6.0 / 448.0, 16.0 / 448.0)]
    cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, p, causal=causal, dtype=rov.FP8_E4M3, act_scale=act)
    weights = rov.make_block_weights(wdev, ws)
    wsb = torch.empty(rov.block_workspace_bytes(cfg, B, S, 0), dtype=torch.uint8, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    ys = {}
    for name, sched, ready in (("seq", rov.SCHED_SEQUENTIAL, False), ("fused", rov.SCHED_FUSED, False),
                               ("ovl_first", rov.SCHED_OVERLAP, False), ("ovl_steady", rov.SCHED_OVERLAP, True)):
        print("fp8 block", name, causal, flush=True)
        y = torch.zeros_like(X)
        mask = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
        nxt = torch.zeros_like(mask) if name == "ovl_steady" else None
        if ready:
            rov.dropout_mask_generate(seed, offset, B, H, S, p, out=mask)
        torch.cuda.synchronize()
        rov.block_forward(weights, X, y, cfg, sched, seed, offset, None if sched == rov.SCHED_FUSED else mask,
                          wsb, main, side, mask_ready=ready, next_mask=nxt)
        torch.cuda.synchronize()
        ys[name] = y
    for name in ("fused", "ovl_first", "ovl_steady"):
        assert torch.equal(ys["seq"], ys[name]), name
    keep = OP.unpack_keep(OP.dropout_mask(seed, offset, B, H, S, p), S)
    ocfg = dict(H=H, Hkv=Hkv, d=d, eps=1e-5, rope_theta=500000.0, p=p, causal=causal)
    ref = OD.block_forward_fp8(_f64(X), wq, ws, act, ocfg, keep)
    got = _f64(ys["seq"])
    # Tolerance of the fp8 block (derived, not the single-GEMM bar): two faithful evaluations differ
    # upstream by rounding (bf16 probabilities inside attention, fp32 against float64), and every
    # quantiser turns a relative difference delta into a different code for about delta / 2^-4 of its
    # elements, each then off by one code step (2^-3 of its value at most); the flips compound through
    # the three quantisers that follow attention (measured: 11 % of the h2 codes, 40 % of the u codes).
    # The result carries noise of the size of the quantisation noise itself: a few percent of the
    # output's rms, up to about 5 % of its maximum over 10^5 outputs.
    err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
    rms = np.sqrt(np.mean((got - ref) ** 2)) / np.sqrt(np.mean(ref ** 2))
    print("fp8 block error: max", err, "rms", rms, flush=True)
    assert err <= 8e-2 and rms <= 6e-2, (err, rms)
    # not the identity, and not the block without activation quantisation
    assert np.max(np.abs(ref - _f64(X))) / np.max(np.abs(ref)) > 0.1


def test_block_forward_fp8_quantisers_on_structured_weights():
    # Every quantiser and scale of the fp8 block, checked tightly: weights chosen so that everything
    # upstream of a quantiser is exact on both sides and no code can flip through rounding noise.
    # Wq = Wk = 0 (uniform attention: probabilities 1/S, exact in bf16), Wv and Wo pick single features
    # (one e4m3 code 1.0 per row), power-of-two scales: q|k|v, the attention output's codes and the
    # residual stream x2 are then identical on both sides, and RMSNorm / FC1 / FC2 see identical inputs.
    from oracle import numerics as ON
    B, S, H, Hkv, d, hidden, ffn = 1, 256, 4, 2, 128, 512, 1024
    p, seed, offset = 0.1, wl.SEED, 2560
    rng = np.random.default_rng(29)
    w = wl.block_weights(rng, H, Hkv, d, hidden, ffn)
    x = wl.block_input(rng, B, S, hidden)
    one = 0x38                                                     # e4m3 code of 1.0
    qkv_n = (H + 2 * Hkv) * d
    wqkv = np.zeros((qkv_n, hidden), dtype=np.uint8)
    vrows = np.arange((H + Hkv) * d, qkv_n)
    wqkv[vrows, rng.permutation(hidden)[: len(vrows)]] = one       # v feature r = one feature of h1
    wo = np.zeros((hidden, H * d), dtype=np.uint8)
    wo[np.arange(hidden), rng.permutation(H * d)[:hidden] if H * d >= hidden else rng.integers(0, H * d, hidden)] = one
    wq = {"wqkv": wqkv, "wo": wo}
    ws = {"wqkv": 1.0, "wo": 1.0}
    for name in ("wg", "wu", "wd"):
        wq[name], ws[name] = ON.e4m3_quantise(w[name] * np.float32(3.0))
    wdev = {n: torch.from_numpy(wq[n]).cuda() for n in ("wqkv", "wo", "wg", "wu", "wd")}
    for name in ("norm1", "norm2"):
        wn = (1.0 + 0.1 * rng.standard_normal(hidden)).astype(np.float32)
        wdev[name] = _dev(wn)
        wq[name] = _f64(wdev[name])
    X = _dev(x)
    act = [2.0 ** -6, 2.0 ** -8, 2.0 ** -6, 2.0 ** -5]             # h1 up to 7, a (a mean) well below 1.75, h2 up to 7, u up to 14
    cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, p, causal=False, dtype=rov.FP8_E4M3, act_scale=act)
    wsb = torch.empty(rov.block_workspace_bytes(cfg, B, S, 0), dtype=torch.uint8, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    y = torch.zeros_like(X)
    mask = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    rov.block_forward(rov.make_block_weights(wdev, ws), X, y, cfg, rov.SCHED_OVERLAP, seed, offset, mask, wsb, main, side)
    torch.cuda.synchronize()
    keep = OP.unpack_keep(OP.dropout_mask(seed, offset, B, H, S, p), S)
    ocfg = dict(H=H, Hkv=Hkv, d=d, eps=1e-5, rope_theta=500000.0, p=p, causal=False)
    ref = OD.block_forward_fp8(_f64(X), wq, ws, act, ocfg, keep)
    got = _f64(y)
    err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
    rms = np.sqrt(np.mean((got - ref) ** 2)) / np.sqrt(np.mean(ref ** 2))
    print("fp8 block, structured weights: max", err, "rms", rms, flush=True)
    assert err <= 2e-2 and rms <= 3e-3, (err, rms)
    # the quantisers matter at this tolerance: the same block without them is much further away
    noq = OD.block_forward(_f64(X), {n: (ON.e4m3_decode(wq[n]) * ws[n] if n in ws else wq[n]) for n in wq}, ocfg, keep)
    assert np.max(np.abs(noq - ref)) / np.max(np.abs(ref)) > 4 * max(err, 5e-3)


def test_block_forward_fp8_error_paths():
    B, S, H, Hkv, d, hidden, ffn = 1, 64, 2, 1, 128, 256, 256
    wdev = {n: torch.zeros(s_, dtype=torch.uint8, device="cuda") for n, s_ in
            (("wqkv", ((H + 2 * Hkv) * d, hidden)), ("wo", (hidden, H * d)), ("wg", (ffn, hidden)),
             ("wu", (ffn, hidden)), ("wd", (hidden, ffn)))}
    wdev["norm1"] = torch.ones(hidden, dtype=torch.bfloat16, device="cuda")
    wdev["norm2"] = torch.ones(hidden, dtype=torch.bfloat16, device="cuda")
    X = torch.zeros((B, S, hidden), dtype=torch.bfloat16, device="cuda")
    y = torch.full_like(X, 2.0)
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    good_ws = {n: 1.0 for n in ("wqkv", "wo", "wg", "wu", "wd")}
    for act, wsc, code in (([1.0, 0.0, 1.0, 1.0], good_ws, rov.ERR_INVALID),
                           ([1.0] * 4, dict(good_ws, wd=-1.0), rov.ERR_INVALID)):
        cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, 0.1, dtype=rov.FP8_E4M3, act_scale=act)
        wsb = torch.empty(rov.block_workspace_bytes(cfg, B, S, 0), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        with pytest.raises(rov.RovError) as e:
            rov.block_forward(rov.make_block_weights(wdev, wsc), X, y, cfg, rov.SCHED_FUSED, 1, 0, None, wsb, main, side)
        assert e.value.code == code
    # hidden not a multiple of 128
    cfg = rov.make_block_cfg(H, Hkv, d, 192, ffn, 0.1, dtype=rov.FP8_E4M3, act_scale=[1.0] * 4)
    wsb = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    with pytest.raises(rov.RovError) as e:
        rov.block_forward(rov.make_block_weights(wdev, good_ws), X[:, :, :192].contiguous(), y[:, :, :192].contiguous(),
                          cfg, rov.SCHED_FUSED, 1, 0, None, wsb, main, side)
    assert e.value.code == rov.ERR_UNSUPPORTED
    torch.cuda.synchronize()
    assert bool((y == 2.0).all())


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("tiny_grid", [False, True])
def test_block_forward_deferred_join_over_three_layers(causal, tiny_grid):
    # a stack of blocks on one stream pair: every block leaves the next layer's mask in flight
    # (ROV_SCHED_OVERLAP_DEFERRED) and the following one finishes and joins it beside its QKV GEMM
    # (mask_ready = ROV_MASK_IN_FLIGHT).  Outputs and masks are those of the sequential schedule.
    B, S, H, Hkv, d, hidden, ffn = 1, 320, 4, 2, 128, 512, 1024
    p, seed, offset = 0.1, wl.SEED, 4480
    x, wd = _block_setup(B, S, H, Hkv, d, hidden, ffn, 31)
    cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, p, causal=causal)
    weights = rov.make_block_weights(wd)
    ws = torch.empty(rov.block_workspace_bytes(cfg, B, S, 0), dtype=torch.uint8, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    calls = rov.mask_philox_calls(B, H, S)
    # (masks of this size are split between the two RNG launches beforehand; with a grid of one workgroup for either of
    # them each runs on for long.  The work queue: test_gpu_mask_queue.py)
    prev = rov.set_rng_max_workgroups(1) if tiny_grid else None
    try:
        y_seq = []
        m = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        for layer in range(3):
            y = torch.zeros_like(x)
            rov.block_forward(weights, x, y, cfg, rov.SCHED_SEQUENTIAL, seed, offset + layer * calls, m, ws, main, side)
            torch.cuda.synchronize()
            y_seq.append(y)
        masks = [torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda") for _ in range(2)]
        ys = [torch.zeros_like(x) for _ in range(3)]
        torch.cuda.synchronize()
        # layer 0 makes its own mask; layers 1 and 2 find theirs in flight
        rov.block_forward(weights, x, ys[0], cfg, rov.SCHED_OVERLAP_DEFERRED, seed, offset, masks[0], ws, main, side,
                          mask_ready=rov.MASK_NOT_READY, next_mask=masks[1])
        rov.block_forward(weights, x, ys[1], cfg, rov.SCHED_OVERLAP_DEFERRED, seed, offset + calls, masks[1], ws, main, side,
                          mask_ready=rov.MASK_IN_FLIGHT, next_mask=masks[0])
        rov.block_forward(weights, x, ys[2], cfg, rov.SCHED_OVERLAP, seed, offset + 2 * calls, masks[0], ws, main, side,
                          mask_ready=rov.MASK_IN_FLIGHT, next_mask=None)
        torch.cuda.synchronize()
    finally:
        if tiny_grid:
            rov.set_rng_max_workgroups(prev)
    for layer in range(3):
        assert torch.equal(ys[layer], y_seq[layer]), layer
    T = S // 32
    lower = np.tril(np.ones((T, T), dtype=bool))
    for buf, layer in ((masks[1], 1), (masks[0], 2)):
        exp = OP.dropout_mask(seed, offset + layer * calls, B, H, S, p)
        got = buf.cpu().numpy().view(np.uint64)
        if causal:
            assert np.array_equal(got[:, :, lower], exp[:, :, lower]), layer
        else:
            assert np.array_equal(got, exp), layer
    # a mask that nobody left in flight, or one described differently, is refused and nothing runs
    y = torch.full_like(x, 5.0)
    for off in (offset, offset + calls):
        with pytest.raises(rov.RovError) as e:
            rov.block_forward(weights, x, y, cfg, rov.SCHED_OVERLAP, seed, off, masks[1], ws, main, side,
                              mask_ready=rov.MASK_IN_FLIGHT)
        assert e.value.code == rov.ERR_INVALID
    torch.cuda.synchronize()
    assert bool((y == 5.0).all())


@pytest.mark.parametrize("tiny_grid", [False, True])
def test_mask_finish_completes_a_mask_left_in_flight(tiny_grid):
    # the last block of a stack called with ROV_SCHED_OVERLAP_DEFERRED leaves a mask that no block will
    # claim: while it is in flight every other use of the buffer is refused; rov_mask_finish completes it
    # (bit-exact against the oracle) and gives the buffer back
    B, S, H, Hkv, d, hidden, ffn = 1, 320, 4, 2, 128, 512, 1024
    p, seed, offset = 0.1, wl.SEED, 96
    x, wd = _block_setup(B, S, H, Hkv, d, hidden, ffn, 37)
    cfg = rov.make_block_cfg(H, Hkv, d, hidden, ffn, p)
    weights = rov.make_block_weights(wd)
    ws = torch.empty(rov.block_workspace_bytes(cfg, B, S, 0), dtype=torch.uint8, device="cuda")
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    calls = rov.mask_philox_calls(B, H, S)
    masks = [torch.full(rov.mask_shape(B, H, S), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda") for _ in range(2)]
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    # (a fixed split, with one workgroup for either launch; the work queue: test_gpu_mask_queue.py)
    prev = rov.set_rng_max_workgroups(1) if tiny_grid else None
    try:
        print("mask_finish: deferred block", tiny_grid, flush=True)
        rov.block_forward(weights, x, y, cfg, rov.SCHED_OVERLAP_DEFERRED, seed, offset, masks[0], ws, main, side,
                          mask_ready=rov.MASK_NOT_READY, next_mask=masks[1])
        # in flight: not usable as a ready mask, not as a target, and only finishable once
        y2 = torch.full_like(x, 5.0)
        for kw in (dict(mask=masks[1], mask_ready=rov.MASK_READY, next_mask=None),
                   dict(mask=masks[1], mask_ready=rov.MASK_NOT_READY, next_mask=None),
                   dict(mask=masks[0], mask_ready=rov.MASK_READY, next_mask=masks[1])):
            with pytest.raises(rov.RovError) as e:
                rov.block_forward(weights, x, y2, cfg, rov.SCHED_OVERLAP, seed, offset + calls, kw["mask"], ws, main, side,
                                  mask_ready=kw["mask_ready"], next_mask=kw["next_mask"])
            assert e.value.code == rov.ERR_INVALID
        with pytest.raises(rov.RovError) as e:
            rov.mask_finish(masks[1], side)            # the stream the RNG runs on cannot be the one that waits for it
        assert e.value.code == rov.ERR_INVALID
        print("mask_finish: finish", flush=True)
        rov.mask_finish(masks[1], main)
        with pytest.raises(rov.RovError) as e:
            rov.mask_finish(masks[1], main)
        assert e.value.code == rov.ERR_INVALID
        with pytest.raises(rov.RovError):
            rov.mask_finish(masks[0], main)            # never was in flight
        main.synchronize()                             # the main stream alone: it has joined the side stream
    finally:
        if tiny_grid:
            rov.set_rng_max_workgroups(prev)
    assert bool((y2 == 5.0).all())
    assert np.array_equal(masks[1].cpu().numpy().view(np.uint64), OP.dropout_mask(seed, offset + calls, B, H, S, p))
    # the buffer is an ordinary ready mask again
    y3 = torch.zeros_like(x)
    y_seq = torch.zeros_like(x)
    rov.block_forward(weights, x, y3, cfg, rov.SCHED_OVERLAP, seed, offset + calls, masks[1], ws, main, side,
                      mask_ready=rov.MASK_READY)
    m = torch.zeros(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
    rov.block_forward(weights, x, y_seq, cfg, rov.SCHED_SEQUENTIAL, seed, offset + calls, m, ws, main, side)
    torch.cuda.synchronize()
    assert torch.equal(y3, y_seq)
