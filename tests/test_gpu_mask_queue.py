"""Masks shared between two RNG launches across calls: left in flight by a deferred block, by a fixed split or through a work
queue, claimed by the following block or finished by hand; queue slots used from two host threads; a queue in a graph.

The masks are those of one launch of the mask kernel (whose bits the oracle pins; the last head is held against the oracle
here too), the outputs those of the sequential schedule, bit for bit.  Every test asserts from the library's own rule
that its masks take the path it is about.
"""
import threading

import numpy as np
import pytest
import torch

from oracle import philox as OP
from paper_2410_07531_amd import binding as rov
from paper_2410_07531_amd import workloads as wl

pytestmark = pytest.mark.gpu

QUEUE = dict(S=8192, H=12, Hkv=4, d=64, hidden=512, ffn=1024)      # 196608 chunks: a queue
SPLIT = dict(S=1000, H=12, Hkv=4, d=64, hidden=256, ffn=128)       # 3072 chunks: a fixed split


def _block(c, causal, seed):
    rng = np.random.default_rng(seed)
    w = wl.block_weights(rng, c["H"], c["Hkv"], c["d"], c["hidden"], c["ffn"])
    wd = {k: torch.from_numpy(v * np.float32(3.0) if k[0] == "w" else v).bfloat16().cuda() for k, v in w.items()}
    x = torch.from_numpy(wl.block_input(rng, 1, c["S"], c["hidden"])).bfloat16().cuda()
    cfg = rov.make_block_cfg(c["H"], c["Hkv"], c["d"], c["hidden"], c["ffn"], 0.1, causal=causal)
    ws = torch.empty(rov.block_workspace_bytes(cfg, 1, c["S"], 0), dtype=torch.uint8, device="cuda")
    return x, wd, cfg, ws


def _chunks(c):
    return (rov.mask_words(1, c["H"], c["S"]) + 63) // 64


def _shares(c, causal):
    """Chunks of the small grid beside the QKV product, and beside all four products of a deferred block."""
    S, qkv = c["S"], (c["H"] + 2 * c["Hkv"]) * c["d"]
    own = 2.0 * S * qkv * c["hidden"]
    rest = 2.0 * S * c["hidden"] * (c["H"] * c["d"] + 3 * c["ffn"])
    return [rov.overlap_mask_chunks(f, rov.BF16, 1, c["H"], S, causal) for f in (own, own + rest)]


def _single_launch(c, causal, seed, offset):
    ref = torch.full(rov.mask_shape(1, c["H"], c["S"]), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda")
    gen = rov.dropout_mask_generate_causal if causal else rov.dropout_mask_generate
    return gen(seed, offset, 1, c["H"], c["S"], 0.1, out=ref)


def _check_mask(mask, c, causal, seed, offset):
    torch.cuda.synchronize()
    ref = _single_launch(c, causal, seed, offset)
    torch.cuda.synchronize()
    T = (c["S"] + 31) // 32
    lower = torch.tril(torch.ones(T, T, dtype=torch.bool, device="cuda")) if causal else torch.ones(T, T, dtype=torch.bool, device="cuda")
    assert torch.equal(mask[:, :, lower], ref[:, :, lower])
    first = (c["H"] - 1) * T * T * 16
    exp = OP.dropout_mask(seed, offset + 64 * (first // 4), 1, 1, c["S"], 0.1)[0, 0]
    got = mask[0, c["H"] - 1].cpu().numpy().view(np.uint64)
    lo = lower.cpu().numpy()
    assert np.array_equal(got[lo], exp[lo])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("kind", ["split", "queue"])
def test_masks_left_in_flight_between_three_layers(kind, causal):
    c = QUEUE if kind == "queue" else SPLIT
    shares = _shares(c, causal)
    print("in flight", kind, causal, shares, flush=True)
    assert all(s == -1 for s in shares) if kind == "queue" else all(0 < s < _chunks(c) for s in shares)
    seed, offset = wl.SEED, 2**32 - 4480
    x, wd, cfg, ws = _block(c, causal, 31)
    weights = rov.make_block_weights(wd)
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    calls = rov.mask_philox_calls(1, c["H"], c["S"])
    y_seq, m = [], torch.zeros(rov.mask_shape(1, c["H"], c["S"]), dtype=torch.int64, device="cuda")
    for layer in range(3):
        y = torch.zeros_like(x)
        torch.cuda.synchronize()
        rov.block_forward(weights, x, y, cfg, rov.SCHED_SEQUENTIAL, seed, offset + layer * calls, m, ws, main, side)
        torch.cuda.synchronize()
        y_seq.append(y)
    masks = [torch.full_like(m, 0x2AAAAAAAAAAAAAAA) for _ in range(2)]
    for _ in range(2):           # the second pass reuses queue slots and buffers
        ys = [torch.zeros_like(x) for _ in range(3)]
        torch.cuda.synchronize()
        rov.trace_read()
        rov.trace_enable(True, [rov.TRACE_RNG, rov.TRACE_RNG_HELPER])
        try:
            rov.block_forward(weights, x, ys[0], cfg, rov.SCHED_OVERLAP_DEFERRED, seed, offset, masks[0], ws, main, side,
                              next_mask=masks[1])
            rov.block_forward(weights, x, ys[1], cfg, rov.SCHED_OVERLAP_DEFERRED, seed, offset + calls, masks[1], ws, main, side,
                              mask_ready=rov.MASK_IN_FLIGHT, next_mask=masks[0])
            rov.block_forward(weights, x, ys[2], cfg, rov.SCHED_OVERLAP, seed, offset + 2 * calls, masks[0], ws, main, side,
                              mask_ready=rov.MASK_IN_FLIGHT)
        finally:
            rov.trace_enable(False)
        torch.cuda.synchronize()
        kinds = [k for k, _ in rov.trace_read()]
        assert kinds.count(rov.TRACE_RNG) == 3 and kinds.count(rov.TRACE_RNG_HELPER) == 3
        for layer in range(3):
            assert torch.equal(ys[layer], y_seq[layer]), layer
    _check_mask(masks[1], c, causal, seed, offset + calls)
    _check_mask(masks[0], c, causal, seed, offset + 2 * calls)


@pytest.mark.parametrize("kind", ["split", "queue"])
def test_mask_finish_of_a_shared_mask(kind):
    c = QUEUE if kind == "queue" else SPLIT
    print("mask_finish", kind, flush=True)
    assert (_shares(c, False)[1] == -1) == (kind == "queue") and _shares(c, False)[1] < _chunks(c)
    seed, offset = wl.SEED, 96
    x, wd, cfg, ws = _block(c, False, 37)
    weights = rov.make_block_weights(wd)
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    calls = rov.mask_philox_calls(1, c["H"], c["S"])
    masks = [torch.full(rov.mask_shape(1, c["H"], c["S"]), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda") for _ in range(2)]
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    rov.block_forward(weights, x, y, cfg, rov.SCHED_OVERLAP_DEFERRED, seed, offset, masks[0], ws, main, side, next_mask=masks[1])
    with pytest.raises(rov.RovError) as e:           # in flight: no one else's target
        rov.block_forward(weights, x, y, cfg, rov.SCHED_OVERLAP, seed, offset + calls, masks[0], ws, main, side,
                          mask_ready=rov.MASK_READY, next_mask=masks[1])
    assert e.value.code == rov.ERR_INVALID
    rov.mask_finish(masks[1], main)
    main.synchronize()                               # the main stream alone: it has joined the side stream
    _check_mask(masks[1], c, False, seed, offset + calls)
    with pytest.raises(rov.RovError) as e:
        rov.mask_finish(masks[1], main)
    assert e.value.code == rov.ERR_INVALID


def _step(c, causal, seed, M):
    g = torch.Generator("cuda").manual_seed(seed)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g).bfloat16()
    q = dict(Q=r(1, c["S"], c["H"], c["d"]), K=r(1, c["S"], c["Hkv"], c["d"]), V=r(1, c["S"], c["Hkv"], c["d"]),
             A=r(M, 512), W=r(512, 512), main=torch.cuda.Stream(), side=torch.cuda.Stream(), causal=causal, seed=seed)
    assert rov.overlap_mask_chunks(2.0 * M * 512 * 512, rov.BF16, 1, c["H"], c["S"], causal) == -1
    return q


def _run_step(s, c, O, C, mask):
    rov.layer_step(rov.SCHED_OVERLAP, [rov.make_gemm_desc(s["A"], s["W"], C)],
                   rov.make_attn_desc(s["Q"], s["K"], s["V"], O, 0.1, causal=s["causal"]), s["seed"], 640, mask, s["main"], s["side"])


def _buffers(s, c):
    return (torch.zeros_like(s["Q"]), torch.zeros((s["A"].shape[0], 512), dtype=torch.bfloat16, device="cuda"),
            torch.full(rov.mask_shape(1, c["H"], c["S"]), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda"))


def test_queues_from_two_host_threads():
    # both threads' masks go through queue slots of the one pool, over more calls than it has slots
    c, reps = QUEUE, 40
    steps = [_step(c, False, 1234, 512), _step(c, True, 77, 2048)]
    for s in steps:
        s["ref"] = _buffers(s, c)
        torch.cuda.synchronize()
        _run_step(s, c, *s["ref"])
        torch.cuda.synchronize()
        s["got"] = _buffers(s, c)
    torch.cuda.synchronize()
    errors = []

    def work(s):
        try:
            for _ in range(reps):
                _run_step(s, c, *s["got"])
        except Exception as e:      # a thread's exception would otherwise be lost
            errors.append(e)

    print("queues: two threads", flush=True)
    threads = [threading.Thread(target=work, args=(s,)) for s in steps]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
        assert not t.is_alive()
    torch.cuda.synchronize()
    assert not errors, errors
    for s in steps:
        for a, b in zip(s["ref"], s["got"]):
            assert torch.equal(a, b)
        _check_mask(s["got"][2], c, s["causal"], s["seed"], 640)


def test_queue_in_a_captured_graph():
    # the queue is cleared by a kernel of the graph: every replay starts with a full queue, eager steps in between
    c = QUEUE
    s = _step(c, False, 5, 512)
    O, C, mask = _buffers(s, c)
    torch.cuda.synchronize()
    _run_step(s, c, O, C, mask)
    torch.cuda.synchronize()
    ref = [t.clone() for t in (O, C, mask)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s["main"]):
        _run_step(s, c, O, C, mask)
    torch.cuda.synchronize()
    for r in range(4):
        print("queue graph replay", r, flush=True)
        for t in (O, C, mask):
            t.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(s["main"]):
            graph.replay()
        torch.cuda.synchronize()
        for t, e in zip((O, C, mask), ref):
            assert torch.equal(t, e), r
        _run_step(s, c, O, C, mask)
        torch.cuda.synchronize()
    _check_mask(mask, c, False, s["seed"], 640)
