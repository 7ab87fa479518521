#!/usr/bin/env python3
"""Benchmark of the RNG/GEMM-overlap hot path on one MI355X.

Headline workload: the full Llama-3-8B transformer block forward (RMSNorm, QKV, RoPE, GQA attention
with dropout p = 0.1, O-proj, SwiGLU FFN), B = 1, S = 16384, bf16, overlap schedule in steady state:
this layer's keep-mask (32 x 16384 x 16384 bits, 1 GiB) was generated during the previous call, and
the next layer's mask is generated by the stand-alone Philox4x32-10 kernel on a side stream beside
this block's PROJ / FC1 / FC2 GEMMs (`rov_block_forward`, ROV_SCHED_OVERLAP).  A "step" is one such
block forward: every part of the hot path runs once (Philox mask, GEMMs, stream join, attention that
drops with the mask).  Inputs are synthetic (seeded N(0,1) activations, N(0,0.02) weights) and
resident in HBM before the timed region.

One JSON line is printed.  `value` is the first half of the metric, the stand-alone RNG kernel's mask
rate on this workload's mask (Gbit/s); the second half, the block under the three schedules and
overlap's two speedups, is in `block`.  `ms_per_step` is the overlap block step.  `roofline` is that
of the step's dominant kernel (the attention kernel that reads the mask), from HIP events recorded
around it on its stream inside the timed region; `roofline_by_kernel` has the step's other kernels.
`cpu_baseline` is the CPU oracle timed on this machine's host cores on a bounded sample of the same block.
"""
import argparse
import ctypes
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0       # MI355X dense bf16 MFMA (published)
PEAK_FP8_TFLOPS = 5000.0        # dense fp8 MFMA (published)
# Nominal VALU peak in lane-instructions per second: 256 CU x 4 SIMD x 32 lanes/clk x 2.4 GHz, the
# issue rate behind the published 157.3 TFLOP/s fp32 (one FMA = 2 flop per lane-instruction).  No
# integer instruction reaches it on this chip: a dependent-free stream of v_add_u32 measures 58 T/s
# (rov_valu_probe, 8 waves per SIMD), three-input xors 37 T/s, 32x32->64 multiply-adds 28 T/s.
PEAK_INT32_LANE_OPS = 256 * 4 * 32 * 2.4e9 / 1e12      # 78.6 T lane-instructions/s
# Philox4x32-10 call, counted two ways: algorithmic 32-bit results (20 wide multiplies x 2 halves,
# 40 two-input xors, 4 compares) and VALU instructions the kernel issues per call (18 v_mad_u64_u32,
# 15 v_bitop3, 4 v_xor, 4 v_cmp, 4 v_mov_b64, 1 v_add; SQ_INSTS_VALU reads 46.5 per wave-call)
INT32_RESULTS_PER_CALL = 84
VALU_INSTS_PER_CALL = 46.5
# Memory traffic per launch at this workload from rocprofv3 --pmc FETCH_SIZE and WRITE_SIZE (KiB per dispatch), as
# bytes.  Calibration on a 1 GiB device copy in the same run: WRITE_SIZE reads 1048576 KiB (x1.00), FETCH_SIZE
# 524311 KiB (x2.00: requests wider than 64 bytes are counted as 64).  The keep words reach attention through
# the scalar cache in 64-byte requests, which the counter sizes correctly: mask-mode attention reads
# 1049119 KiB more than the no-dropout kernel for a 1048576 KiB mask, so that part is taken x1.00.  The
# counters sit between L2 and the fabric; the 256 MiB memory-side cache lies behind them, so HBM reads
# are at most these figures.
_KIB = 1024
TRAFFIC = {"attention_mask": (2 * 1114234 + 1049119 + 131077) * _KIB,     # K/V/Q x2.00, keep words x1.00, O written
           "mask_kernel": (45 + 1048576) * _KIB,                          # writes = bits / 8 exactly
           "gemm_swiglu": (2 * 2935458 + 458753) * _KIB,
           "gemm_down": (2 * 1456557 + 131110) * _KIB,
           "gemm_qkv": (2 * 611749 + 196773) * _KIB,
           "gemm_o": (2 * 408145 + 131110) * _KIB}
# VALU occupancy of the stand-alone mask kernel from rocprofv3 --pmc: SQ_ACTIVE_INST_VALU (1561919488, in units
# of four cycles) x 4 / (4 SIMDs x SQ_BUSY_CU_CYCLES 1579185055): the share of SIMD cycles in which a VALU
# instruction is in flight.  SQ_INSTS_VALU reads 1561788416 = 46.5 per wave-call.
RNG_VALU_BUSY_COUNTER = 1561919488 / 1579185055


# ---------------------------------------------------------------------------------------------- timing helpers
def median_ms(fn, warm, iters, sync, ev_pair, inner=10):
    """Median over `iters` batches of the per-call time of `inner` back-to-back calls (HIP events on
    the current stream), so that launch latency after an idle queue is not billed to the kernel."""
    for _ in range(warm):
        fn()
    sync()
    ts = []
    for _ in range(iters):
        a, b = ev_pair()
        a.record()
        for _ in range(inner):
            fn()
        b.record()
        b.synchronize()
        ts.append(a.elapsed_time(b) / inner)
    return float(np.median(ts))


def once_ms(fn, ev_pair):
    """One call between two events on the current stream."""
    a, b = ev_pair()
    a.record()
    fn()
    b.record()
    b.synchronize()
    return a.elapsed_time(b)


def stabilise(fn, ev_pair, batch=3, tol=0.02, max_batches=20):
    """Runs batches of `batch` calls until two consecutive batch times agree within `tol` (the clock
    and power state have settled), whatever --warmup says.  Returns (batches run, last per-call ms)."""
    prev = None
    t = 0.0
    for i in range(max_batches):
        a, b = ev_pair()
        a.record()
        for _ in range(batch):
            fn()
        b.record()
        b.synchronize()
        t = a.elapsed_time(b) / batch
        if prev is not None and abs(t - prev) <= tol * prev:
            return i + 1, t
        prev = t
    return max_batches, t


def interleaved_medians(fns, iters, ev_pair, sync, after=None):
    """Each callable once per round, `iters` rounds, so that every quantity in a ratio was measured
    in the same clock and power state as its partner.  after[name](): optional per-call hook (reads a
    trace) whose return value is collected.  Returns ({name: median ms}, {name: [hook values]})."""
    ts = {k: [] for k in fns}
    extra = {k: [] for k in fns}
    sync()
    for _ in range(iters):
        for k, fn in fns.items():
            ts[k].append(once_ms(fn, ev_pair))
            if after and k in after:
                extra[k].append(after[k]())
    return {k: float(np.median(v)) for k, v in ts.items()}, extra


def trace_by_kind(rov):
    out = {}
    for kind, ms in rov.trace_read():
        out.setdefault(kind, []).append(ms)
    return out


# ---------------------------------------------------------------------------------------------- RNG ceiling
def valu_probe_ceiling(torch, rov, sync):
    """Issue cost (ns per wave64 instruction per SIMD, 8 waves per SIMD) of the instruction kinds the
    mask kernel is made of, measured now on this device, and the call rate that the sum of its instruction
    mix at those costs gives: 18 wide multiply-adds, 15 three-input xors, 4 + 1 simple ops and 4 compares,
    each with the one-lane move of its ballot (priced as the probed compare + lane write), per call.  An
    estimate, no bound: in the kernel the scalar unit and the multiplier overlap work that the
    single-class streams serialise."""
    L = rov.load()
    props = torch.cuda.get_device_properties(0)
    n_simd = props.multi_processor_count * 4
    wgs, iters = props.multi_processor_count * 8, 1000
    out = torch.zeros(wgs * 4 * 2, dtype=torch.int64, device="cuda")
    ns = {}
    for kind, name in ((0, "mad64_plus_add"), (3, "xor3"), (4, "add"), (5, "cmp_writelane_plus_add")):
        def fn():
            rov._check(L.rov_valu_probe(kind, iters, wgs, ctypes.c_void_p(out.data_ptr()), rov._stream_ptr(None)),
                       "rov_valu_probe")
        for _ in range(2):
            fn()
        sync()
        ts = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fn()
            b.record()
            b.synchronize()
            ts.append(a.elapsed_time(b))
        wave_insts = wgs * 4 * iters * 4 * 8                      # per launch (probe: 8 chains x 4 x iters)
        ns[name] = min(ts) * 1e6 / (wave_insts / n_simd)          # ns per wave-instruction per SIMD
    add = ns["add"]
    mad, xor3, cmpw = ns["mad64_plus_add"] - add, ns["xor3"], ns["cmp_writelane_plus_add"] - add
    ns_per_wave_call = 18 * mad + 15 * xor3 + 5 * add + 4 * cmpw
    gcalls = 64.0 * n_simd / ns_per_wave_call                     # 64 calls per wave-call, per ns -> Gcalls/s
    return {"ns_per_wave_instruction_per_simd": {"mad_u64_u32": mad, "bitop3_xor3": xor3, "add": add,
                                                 "cmp_plus_writelane": cmpw},
            "ns_per_wave_call": ns_per_wave_call, "ceiling_gcalls_s": gcalls}


def rng_roofline(ncalls, t_ms, probe):
    """The VALU roofline of the stand-alone mask kernel in three forms: issued instructions against the nominal
    lane-instruction peak, the call rate against the sum of its mix at the probed costs, and the counter reading."""
    calls_s = ncalls / (t_ms * 1e-3)
    issued = calls_s * VALU_INSTS_PER_CALL / 1e12
    return {"bound": "alu", "unit": "T int32 lane-instructions/s",
            "achieved": issued, "peak": PEAK_INT32_LANE_OPS, "frac": issued / PEAK_INT32_LANE_OPS,
            "peak_derivation": "peak = 256 CU x 4 SIMD x 32 lanes/clk x 2.4 GHz (the lane-instruction rate behind the "
                               "published 157.3 TFLOP/s fp32); achieved = calls/s x 46.5 VALU instructions issued per call "
                               "(SQ_INSTS_VALU per wave-call). Integer instructions cannot reach that peak on this chip "
                               "(measured: add 58 T/s, xor3 37 T/s, mad_u64_u32 28 T/s).  frac_of_probe_ceiling is the call "
                               "rate against the sum of this kernel's own instruction mix at the probed issue rates: an "
                               "estimate, above 1 where the kernel overlaps classes that the probes run one by one; "
                               "valu_busy_counter says how full the issue slots are",
            "frac_of_probe_ceiling": (calls_s / 1e9) / probe["ceiling_gcalls_s"] if probe else None,
            "probe": probe,
            "valu_busy_counter": RNG_VALU_BUSY_COUNTER,
            "algorithmic": {"int32_results_per_call": INT32_RESULTS_PER_CALL,
                            "achieved_T_results_s": calls_s * INT32_RESULTS_PER_CALL / 1e12,
                            "frac_of_78.6T_nominal_32_lanes_per_clk": calls_s * INT32_RESULTS_PER_CALL / 1e12 / 78.6},
            "traffic": TRAFFIC["mask_kernel"]}


# ---------------------------------------------------------------------------------------------- block (8B-shaped, 16384 tokens)
class Block:
    """The Llama-3-8B block workload on the device: weights, input, two mask buffers, workspace."""

    def __init__(self, torch, rov, wl, seq_len=None, causal=False, ci=4):
        """ci = 4: the Llama-3-8B block in bf16; ci = 3: the 70B-shaped layer as an fp8 block (e4m3 weights
        and activations, per-tensor scales: weights amax / 448, activations fixed at the amax the shapes give)."""
        c = wl.CONFIGS[ci]
        self.fp8 = c["dtype"] == "fp8"
        self.B, self.H, self.Hkv, self.d, self.p = c["B"], c["H"], c["Hkv"], c["d"], c["p"]
        self.hidden, self.ffn = c["hidden"], c["ffn"]
        self.S = c["S"] if seq_len is None else int(seq_len)
        B, H, Hkv, S, d, hidden, ffn = self.B, self.H, self.Hkv, self.S, self.d, self.hidden, self.ffn
        gen = torch.Generator(device="cuda")
        gen.manual_seed(1000 + ci)
        bf = torch.bfloat16

        def randn(*shape, sd=1.0):
            return (torch.randn(*shape, device="cuda", generator=gen) * sd).to(bf)

        self.wts = dict(norm1=torch.ones(hidden, device="cuda", dtype=bf), norm2=torch.ones(hidden, device="cuda", dtype=bf),
                        wqkv=randn((H + 2 * Hkv) * d, hidden, sd=0.02), wo=randn(hidden, H * d, sd=0.02),
                        wg=randn(ffn, hidden, sd=0.02), wu=randn(ffn, hidden, sd=0.02), wd=randn(hidden, ffn, sd=0.02))
        self.x = randn(B, S, hidden)
        self.y = torch.empty_like(self.x)
        self.torch, self.rov, self.wl = torch, rov, wl
        self.w_scale, self.act_scale = None, None
        if self.fp8:
            self.w_scale = {}
            for name in ("wqkv", "wo", "wg", "wu", "wd"):
                t = self.wts[name].float()
                sc = float(t.abs().max()) / 448.0
                self.wts[name] = (t / sc).to(torch.float8_e4m3fn).view(torch.uint8)
                self.w_scale[name] = sc
            self.act_scale = [v / 448.0 for v in (6.0, 8.0, 6.0, 32.0)]
        self.weights = rov.make_block_weights(self.wts, self.w_scale)
        self.m0 = torch.empty(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
        self.m1 = torch.empty_like(self.m0)
        self.off1 = rov.mask_philox_calls(B, H, S)
        self.set_causal(causal)
        self.ws = torch.empty(rov.block_workspace_bytes(self.cfg, B, S, 0), dtype=torch.uint8, device="cuda")
        self.layer = 0
        self.in_flight = False
        self.deferred = True     # steady state of a layer stack: the next mask is joined by the next block
        self.nbits = B * H * S * S
        T = B * S
        self.gemm_flops = {"qkv": 2.0 * T * (H + 2 * Hkv) * d * hidden, "o": 2.0 * T * hidden * H * d,
                           "swiglu": 2.0 * 2.0 * T * ffn * hidden, "down": 2.0 * T * hidden * ffn}
        self.attn_flops = 4.0 * B * H * S * S * d

    def set_causal(self, causal):
        self.causal = causal
        self.cfg = self.rov.make_block_cfg(self.H, self.Hkv, self.d, self.hidden, self.ffn, self.p, causal=causal,
                                           dtype=self.rov.FP8_E4M3 if self.fp8 else self.rov.BF16,
                                           act_scale=self.act_scale)

    def prime(self, main_s):
        """Mask of layer 0 into m0, so that the first overlap call finds its mask ready."""
        self.settle()
        self.layer = 0
        self.rov.dropout_mask_generate(self.wl.SEED, 0, self.B, self.H, self.S, self.p, out=self.m0, stream=main_s)

    def seq(self, main_s, side_s):
        self.rov.block_forward(self.weights, self.x, self.y, self.cfg, self.rov.SCHED_SEQUENTIAL, self.wl.SEED, 0,
                               self.m0, self.ws, main_s, side_s)

    def fus(self, main_s, side_s):
        self.rov.block_forward(self.weights, self.x, self.y, self.cfg, self.rov.SCHED_FUSED, self.wl.SEED, 0, None,
                               self.ws, main_s, side_s)

    def ovl(self, main_s, side_s, sched=None):
        """Steady state: this layer's mask was produced during the previous call, the next one's is produced now."""
        cur, nxt = (self.m0, self.m1) if self.layer % 2 == 0 else (self.m1, self.m0)
        ready = self.rov.MASK_IN_FLIGHT if self.in_flight else self.rov.MASK_READY
        if sched is None:
            sched = self.rov.SCHED_OVERLAP_DEFERRED if self.deferred else self.rov.SCHED_OVERLAP
        self.rov.block_forward(self.weights, self.x, self.y, self.cfg, sched, self.wl.SEED,
                               self.layer * self.off1, cur, self.ws, main_s, side_s, mask_ready=ready, next_mask=nxt)
        self.in_flight = sched == self.rov.SCHED_OVERLAP_DEFERRED
        self._streams = (main_s, side_s)
        self.layer += 1

    def settle(self):
        """Joins a mask left in flight by the last deferred call (one plain overlap call consumes it)."""
        if self.in_flight:
            self.ovl(*self._streams, sched=self.rov.SCHED_OVERLAP)

    def ovl_chain(self, main_s, side_s, n):
        """n consecutive blocks of a layer stack: every block leaves the next mask in flight for its successor;
        the last one joins its own, so that nothing is in flight afterwards."""
        for i in range(n):
            self.ovl(main_s, side_s, sched=None if i + 1 < n else self.rov.SCHED_OVERLAP)

    def norng(self, main_s, side_s):
        """The same block with no RNG anywhere: mask ready, no next mask (what overlap would cost if the RNG were free)."""
        cur = self.m0 if self.layer % 2 == 0 else self.m1
        self.rov.block_forward(self.weights, self.x, self.y, self.cfg, self.rov.SCHED_OVERLAP, self.wl.SEED,
                               self.layer * self.off1, cur, self.ws, main_s, side_s, mask_ready=True, next_mask=None)


GEMM_NAMES = ("qkv", "o", "swiglu", "down")       # launch order of the block's GEMMs


CHAIN = 4     # blocks per timed sample of a schedule: a short layer stack


def block_schedules(blk, rov, main_s, side_s, sync, ev_pair, iters):
    """The three schedules and the RNG-free block, interleaved, each sample a stack of CHAIN blocks
    (per-block time = sample / CHAIN): the overlap schedule's steady state spans block boundaries (a
    block's mask is finished beside the next block's QKV GEMM).  GEMM and RNG times inside the overlap
    and the RNG-free block from the library's kernel trace (events on the kernels' own streams); for
    the overlap schedule from the stack's inner blocks."""
    def hook():
        t = trace_by_kind(rov)
        return {"gemm": t.get(rov.TRACE_GEMM, []), "rng": t.get(rov.TRACE_RNG, []),
                "helper": t.get(rov.TRACE_RNG_HELPER, []), "attention": t.get(rov.TRACE_ATTENTION, [])}

    def rep(fn):
        def run():
            for _ in range(CHAIN):
                fn(main_s, side_s)
        return run

    blk.settle()
    fns = {"sequential": rep(blk.seq), "fused": rep(blk.fus), "norng": rep(blk.norng),
           "overlap": lambda: blk.ovl_chain(main_s, side_s, CHAIN)}
    rov.trace_enable(True, [rov.TRACE_GEMM, rov.TRACE_RNG, rov.TRACE_RNG_HELPER, rov.TRACE_ATTENTION])
    rov.trace_read()
    med, extra = interleaved_medians(fns, iters, ev_pair, sync, after={k: hook for k in fns})
    rov.trace_enable(False)
    rov.trace_read()
    med = {k: v / CHAIN for k, v in med.items()}

    def per_block(records, key, n, inner_only=False):
        """median over samples and blocks of the n records of `key` each block contributes"""
        rows = []
        for r in records:
            if len(r[key]) != n * CHAIN:
                continue
            blocks = [r[key][i * n:(i + 1) * n] for i in range(CHAIN)]
            rows += blocks[1:-1] if inner_only else blocks
        return [float(np.median([b[i] for b in rows])) for i in range(n)] if rows else None

    g_alone = per_block(extra["norng"], "gemm", 4)
    g_ovl = per_block(extra["overlap"], "gemm", 4, inner_only=True)
    rng_seq = per_block(extra["sequential"], "rng", 1)
    attn_ovl = per_block(extra["overlap"], "attention", 1, inner_only=True)
    # RNG launches of an overlap stack: CHAIN - 1 small grids (blocks 0 .. CHAIN-2 start the next mask) and as
    # many helper launches (each in the block after, or at the stack's end)
    rng_in = [float(np.median([np.median(r["rng"]) for r in extra["overlap"] if r["rng"]]))] if any(r["rng"] for r in extra["overlap"]) else None
    helper = [float(np.median([np.median(r["helper"]) for r in extra["overlap"] if r["helper"]]))] if any(r["helper"] for r in extra["overlap"]) else None
    return med, g_alone, g_ovl, rng_in, helper, rng_seq, attn_ovl


# ---------------------------------------------------------------------------------------------- main
def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the causal block, the S=2048 layer step and the 70B fp8 layer in `extras`")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU-oracle baseline")
    ap.add_argument("--all-configs", action="store_true",
                    help="instead of the benchmark line: one result record per workload (the five configurations) "
                         "under --out-dir, plus the scaling-law check between them")
    ap.add_argument("--out-dir", default=os.path.join(ROOT, "gpurun_out"), help="where --all-configs writes its records")
    ap.add_argument("--seq-sweep", action="store_true",
                    help="instead of the benchmark line: the Llama-3-8B block (non-causal) under the three schedules "
                         "at S = 2048 ... 32768 beside the limiter model's prediction and region, one JSON object")
    ap.add_argument("--kernels-only-fp8", action="store_true",
                    help="for profilers: the calibration copy, then the Llama-3-70B-shaped fp8 block (T=8192) three times "
                         "under the sequential schedule (every kernel alone), three times fused, and a chain of four "
                         "overlap blocks; no JSON")
    ap.add_argument("--kernels-only", action="store_true",
                    help="for profilers: a 1 GiB device copy (counter calibration), then every kernel of the "
                         "S=16384 block alone and the overlap block step, 3 times each; no JSON")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build measures one GPU only (the path has no cross-GPU step); run with --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2410_07531_amd import binding as rov
    from paper_2410_07531_amd import workloads as wl

    rov.load()
    torch.cuda.set_device(0)
    sync = torch.cuda.synchronize
    main_s, side_s = torch.cuda.Stream(), torch.cuda.Stream()

    def ev_pair():
        return torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    if args.seq_sweep:
        return seq_sweep(torch, rov, wl, main_s, side_s, sync, ev_pair)
    if args.all_configs:
        return all_configs(torch, rov, wl, main_s, side_s, sync, ev_pair, args.out_dir)
    if args.kernels_only:
        return kernels_only(torch, rov, wl, main_s, side_s, sync)
    if args.kernels_only_fp8:
        return kernels_only_fp8(torch, rov, wl, main_s, side_s, sync)

    blk = Block(torch, rov, wl)
    B, H, Hkv, S, d, p = blk.B, blk.H, blk.Hkv, blk.S, blk.d, blk.p
    nbits, ncalls = blk.nbits, blk.nbits // 4
    hidden_, ffn_ = blk.hidden, blk.ffn
    sync()   # inputs were produced on torch's current stream; the library runs on main_s / side_s

    with torch.cuda.stream(main_s):
        blk.prime(main_s)
        # ---- warm-up that does not trust --warmup: until two consecutive batches agree within 2 %
        n_batches, _ = stabilise(lambda: blk.ovl(main_s, side_s), ev_pair)
        for _ in range(args.warmup):
            blk.ovl(main_s, side_s)
        sync()
        # ---- timed region: K overlap block steps; only the dominant kernel carries trace events
        rov.trace_enable(True, [rov.TRACE_ATTENTION])
        rov.trace_read()
        sync()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            blk.ovl(main_s, side_s)
        sync()
        t1 = time.perf_counter()
        rov.trace_enable(False)
        attn_in_step = float(np.mean([ms for kind, ms in rov.trace_read() if kind == rov.TRACE_ATTENTION]))
        ms_per_step = (t1 - t0) * 1e3 / args.steps
        blk.settle()

        # ---- schedules and the RNG-free block, interleaved (same clock state for both sides of every ratio)
        med, g_alone, g_ovl, rng_in, helper, rng_seq, attn_ovl = block_schedules(blk, rov, main_s, side_s, sync, ev_pair, 9)

        # ---- stand-alone kernels on this workload
        t_rng = median_ms(lambda: rov.dropout_mask_generate(wl.SEED, 0, B, H, S, p, out=blk.m1, stream=main_s),
                          3, 9, sync, ev_pair, inner=3)
        blk.prime(main_s)
        Q = (torch.randn(B, S, H, d, device="cuda") ).to(torch.bfloat16)
        Kt = (torch.randn(B, S, Hkv, d, device="cuda")).to(torch.bfloat16)
        V = (torch.randn(B, S, Hkv, d, device="cuda")).to(torch.bfloat16)
        O = torch.empty_like(Q)
        sync()
        fa = {"none": lambda: rov.attention_fwd_dropout(Q, Kt, V, 0.0, O=O, stream=main_s),
              "mask": lambda: rov.attention_fwd_dropout(Q, Kt, V, p, mask=blk.m0, O=O, stream=main_s),
              "fused": lambda: rov.attention_fwd_dropout(Q, Kt, V, p, seed=wl.SEED, offset=0, O=O, stream=main_s)}
        for f in fa.values():
            f()
        t_attn, _ = interleaved_medians(fa, 7, ev_pair, sync)
        del Q, Kt, V, O
        probe = valu_probe_ceiling(torch, rov, sync)

    t_seq, t_fus, t_ovl, t_norng = med["sequential"], med["fused"], med["overlap"], med["norng"]
    # the GEMMs a mask runs beside in steady state: PROJ, FC1 (gate + up), FC2 of the block before its attention and
    # the QKV GEMM of its own block (the deferred join), i.e. all four of every block
    beside = [0, 1, 2, 3]
    gemm = {}
    for i, name in enumerate(GEMM_NAMES):
        fl = blk.gemm_flops[name]
        gemm[name] = {"alone_ms": g_alone[i], "in_overlap_block_ms": g_ovl[i], "rng_co_running": i in beside,
                      "alone_tflops": fl / g_alone[i] / 1e9, "in_overlap_block_tflops": fl / g_ovl[i] / 1e9,
                      "mfma_frac_alone": fl / g_alone[i] / 1e9 / PEAK_BF16_TFLOPS,
                      "mfma_frac_in_overlap_block": fl / g_ovl[i] / 1e9 / PEAK_BF16_TFLOPS,
                      "slowdown": g_ovl[i] / g_alone[i] - 1.0}
    sum_alone = sum(g_alone[i] for i in beside)
    sum_ovl = sum(g_ovl[i] for i in beside)
    rng_total_in = rng_in[0] if rng_in else None
    block = {
        "sequential_ms": t_seq, "fused_ms": t_fus, "overlap_ms": t_ovl, "without_rng_ms": t_norng,
        "speedup_overlap_vs_sequential": t_seq / t_ovl, "speedup_overlap_vs_fused": t_fus / t_ovl,
        # R16 on the whole block: the share of the stand-alone RNG time that no longer shows in the block
        "rng_hidden_fraction_whole_block": 1.0 - max(t_ovl - t_norng, 0.0) / t_rng,
        # the same on the region the RNG overlaps: (GEMMs beside the RNG + helper launch) against the same GEMMs alone
        "rng_hidden_fraction_gemm_region": 1.0 - max(sum_ovl + (helper[0] if helper else 0.0) - sum_alone, 0.0) / t_rng,
        "gemm_slowdown_beside_rng": sum_ovl / sum_alone - 1.0,
        "gemm_slowdown_all_four": sum(g_ovl) / sum(g_alone) - 1.0,
        "rng_beside_gemms_ms": rng_total_in, "rng_helper_launch_ms": helper[0] if helper else None,
        "rng_rate_beside_gemms_vs_alone": (t_rng / rng_total_in) if rng_total_in else None,
        "rng_in_sequential_block_ms": rng_seq[0] if rng_seq else None,
        "attention_in_overlap_block_ms": attn_ovl[0] if attn_ovl else None,
        "gemm": gemm,
        "paper_context_gh100_fp8_philox7": {"speedup_vs_sequential": 1.26, "speedup_vs_fused": 1.22,
                                            "gemm_slowdown": 0.04, "rng_rate_beside_gemm": 0.5},
    }
    attention = {"none_ms": t_attn["none"], "mask_ms": t_attn["mask"], "fused_ms": t_attn["fused"],
                 "none_tflops": blk.attn_flops / t_attn["none"] / 1e9, "mask_tflops": blk.attn_flops / t_attn["mask"] / 1e9,
                 "fused_tflops": blk.attn_flops / t_attn["fused"] / 1e9,
                 "dropping_overhead": t_attn["mask"] / t_attn["none"] - 1.0,
                 "fused_overhead": t_attn["fused"] / t_attn["none"] - 1.0,
                 "paper_context_gh100_dropping_overhead": 0.12}
    rng_alone = {"ms": t_rng, "gbit_s": nbits / t_rng / 1e6, "gcalls_s": ncalls / t_rng / 1e6,
                 "roofline": rng_roofline(ncalls, t_rng, probe)}

    def mfma_roofline(kernel, flops, ms, key):
        return {"bound": "mfma", "kernel": kernel, "achieved": flops / ms / 1e9, "peak": PEAK_BF16_TFLOPS,
                "unit": "TFLOP/s", "frac": flops / ms / 1e9 / PEAK_BF16_TFLOPS, "traffic": TRAFFIC[key]}

    def tn_label(M, N, K):
        # the launch picks the kernel and its tile per shape; ask the library what it runs
        kernel, rows, cols = rov.gemm_tile(M, N, K, rov.BF16)[:3]
        name = "gemm_tn_kernel<%d, false>" % (cols // 32) if kernel == rov.GEMM_256_ROWS else "gemm_ring_kernel (tile %dx%d)" % (rows, cols)
        return "%s %dx%dx%d (RNG co-running)" % (name, M, N, K)

    T_tok = B * S
    roofline_by_kernel = {
        "gemm_swiglu": mfma_roofline("gemm_swiglu_kernel<%d> (gate and up projections, SwiGLU in the accumulators; RNG co-running)"
                                     % (rov.gemm_swiglu_tile_cols(T_tok, ffn_, hidden_, rov.BF16) // 16),
                                     blk.gemm_flops["swiglu"], g_ovl[2], "gemm_swiglu"),
        "gemm_down": mfma_roofline(tn_label(T_tok, hidden_, ffn_), blk.gemm_flops["down"], g_ovl[3], "gemm_down"),
        "gemm_qkv": mfma_roofline(tn_label(T_tok, (H + 2 * Hkv) * d, hidden_), blk.gemm_flops["qkv"], g_ovl[0], "gemm_qkv"),
        "gemm_o": mfma_roofline(tn_label(T_tok, hidden_, H * d), blk.gemm_flops["o"], g_ovl[1], "gemm_o"),
        "mask_kernel_alone": rng_alone["roofline"],
    }
    extras = {"warmup_batches_until_stable": n_batches, "attention_alone_s16k": attention, "rng_alone_s16k": rng_alone,
              "mask_bits_per_whole_step_gbit_s": nbits / ms_per_step / 1e6}

    from paper_2410_07531_amd import limiter_model as LM
    bm = LM.block(LM.MI355X, B, S, H, Hkv, d, blk.hidden, blk.ffn, False)
    block["limiter_model_ms"] = {"sequential": bm["baseline"] * 1e3, "fused": bm["fusion"] * 1e3,
                                 "overlap": bm["overlap"] * 1e3, "rng_exposed": bm["rng_exposed"] * 1e3}
    T_ = B * S
    extras["limiter_model_vs_measured_ms"] = {
        "rng": [LM.t_rng(LM.MI355X, B, H, S)["time"] * 1e3, t_rng],
        "attention_none": [LM.t_attention(LM.MI355X, B, H, S, d, "none")["time"] * 1e3, t_attn["none"]],
        "attention_mask": [LM.t_attention(LM.MI355X, B, H, S, d, "mask")["time"] * 1e3, t_attn["mask"]],
        "attention_fused": [LM.t_attention(LM.MI355X, B, H, S, d, "fused")["time"] * 1e3, t_attn["fused"]],
        "gemm_qkv": [LM.t_gemm(LM.MI355X, T_, (H + 2 * Hkv) * d, hidden_)["time"] * 1e3, g_alone[0]],
        "gemm_o": [LM.t_gemm(LM.MI355X, T_, hidden_, H * d)["time"] * 1e3, g_alone[1]],
        "gemm_swiglu": [LM.t_gemm(LM.MI355X, T_, ffn_, hidden_, dual=True)["time"] * 1e3, g_alone[2]],
        "gemm_down": [LM.t_gemm(LM.MI355X, T_, hidden_, ffn_)["time"] * 1e3, g_alone[3]],
        "note": "[model, measured]; counts x probed chip properties, no per-kernel factor (paper Sec. 3)"}

    if not args.no_extras:
        with torch.cuda.stream(main_s):
            blk.set_causal(True)
            blk.prime(main_s)
            for _ in range(2):
                blk.ovl(main_s, side_s)
            cm, cg_alone, cg_ovl, *_ = block_schedules(blk, rov, main_s, side_s, sync, ev_pair, 5)
            t_rng_c = median_ms(lambda: rov.dropout_mask_generate_causal(wl.SEED, 0, B, H, S, p, out=blk.m1, stream=main_s),
                                2, 7, sync, ev_pair, inner=3)
            blk.prime(main_s)
        extras["block_causal"] = {"sequential_ms": cm["sequential"], "fused_ms": cm["fused"], "overlap_ms": cm["overlap"],
                                  "without_rng_ms": cm["norng"],
                                  "speedup_overlap_vs_sequential": cm["sequential"] / cm["overlap"],
                                  "speedup_overlap_vs_fused": cm["fused"] / cm["overlap"],
                                  # the causal mask holds only the tiles causal attention reads: about half the Philox calls
                                  "rng_alone_ms": t_rng_c,
                                  "rng_hidden_fraction_whole_block": 1.0 - max(cm["overlap"] - cm["norng"], 0.0) / t_rng_c,
                                  "gemm_slowdown_beside_rng": sum(cg_ovl) / sum(cg_alone) - 1.0}
    del blk
    torch.cuda.empty_cache()
    if not args.no_extras:
        # the 70B-shaped layer as one fp8 block (e4m3 GEMM operands, quantising epilogues), steady state
        b8 = Block(torch, rov, wl, ci=3)
        sync()
        with torch.cuda.stream(main_s):
            b8.prime(main_s)
            stabilise(lambda: b8.ovl(main_s, side_s), ev_pair)
            m8, ga8, go8, ri8, he8, _, _ = block_schedules(b8, rov, main_s, side_s, sync, ev_pair, 5)
            t_rng8 = median_ms(lambda: rov.dropout_mask_generate(wl.SEED, 0, b8.B, b8.H, b8.S, b8.p, out=b8.m1, stream=main_s),
                               2, 5, sync, ev_pair, inner=2)
        fl8 = sum(b8.gemm_flops.values())
        extras["block_llama3_70b_fp8_s8k"] = {
            "sequential_ms": m8["sequential"], "fused_ms": m8["fused"], "overlap_ms": m8["overlap"], "without_rng_ms": m8["norng"],
            "speedup_overlap_vs_sequential": m8["sequential"] / m8["overlap"], "speedup_overlap_vs_fused": m8["fused"] / m8["overlap"],
            "rng_alone_ms": t_rng8, "rng_hidden_fraction_whole_block": 1.0 - max(m8["overlap"] - m8["norng"], 0.0) / t_rng8,
            "gemms_alone_ms": dict(zip(GEMM_NAMES, ga8)), "gemms_in_overlap_block_ms": dict(zip(GEMM_NAMES, go8)),
            "gemms_alone_tflops": fl8 / sum(ga8) / 1e9, "gemms_fp8_mfma_frac_alone": fl8 / sum(ga8) / 1e9 / PEAK_FP8_TFLOPS,
            "gemm_slowdown_beside_rng": sum(go8[1:]) / sum(ga8[1:]) - 1.0,
            "rng_beside_gemms_ms": ri8[0] if ri8 else None, "rng_helper_launch_ms": he8[0] if he8 else None}
        del b8
        torch.cuda.empty_cache()
        extras["layer_llama3_8b_s2k"] = bench_layer_config(torch, rov, wl, 1, main_s, side_s, sync, ev_pair, iters=15)
        extras["layer_llama3_70b_fp8_s8k"] = bench_layer_config(torch, rov, wl, 3, main_s, side_s, sync, ev_pair, iters=5,
                                                              variants=True)

    cpu = None if args.no_cpu else cpu_baseline(wl)

    out = {
        "metric": "RNG mask Gbit/s + Transformer-block speedup: overlap vs sequential/fused",
        "value": nbits / t_rng / 1e6,
        "unit": "Gbit/s",
        "value_definition": "stand-alone Philox4x32-10 mask kernel on this workload's 32x16384x16384-bit mask; the "
                            "block speedups are in `block`",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic",
        "config": {"workload": "llama3_8b_block_s16k: full Llama-3-8B block forward, B=1 S=16384 H=32 (8 KV heads) d=128 "
                               "hidden=4096 ffn=14336 bf16 p=0.1 non-causal; overlap schedule in steady state (this layer's "
                               "mask ready, next layer's 32x16384x16384-bit mask generated on the side stream beside the "
                               "PROJ / FC1 / FC2 GEMMs and the next block's RMSNorm and QKV GEMM, joined before that block's attention)",
                   "schedule": "overlap", "seed": wl.SEED, "offset": wl.OFFSET},
        "roofline": dict(mfma_roofline("attn_bf16_kernel<128, 1, 8, MODE_MASK> (flash-attention forward that drops with the "
                                       "stored mask), inside the timed overlap block steps", blk_attn_flops(B, H, S, d),
                                       attn_in_step, "attention_mask"),
                         share_of_step=attn_in_step / ms_per_step,
                         algorithmic_bytes=(2 * B * S * H * d + 2 * B * S * Hkv * d) * 2 + nbits // 8,
                         traffic_note="FETCH_SIZE + WRITE_SIZE per launch, calibrated on a 1 GiB copy; L2-miss traffic to the "
                                      "fabric (K and V are re-read by the 64 query blocks of the 4 heads that share them; 87 % of "
                                      "those re-reads hit L2), an upper bound on HBM bytes: 0.8 TB/s, a tenth of the HBM peak"),
        "roofline_by_kernel": roofline_by_kernel,
        "block": block,
        "cpu_baseline": cpu,
        "extras": extras,
    }
    print(json.dumps(out))


def blk_attn_flops(B, H, S, d):
    return 4.0 * B * H * S * S * d


# ---------------------------------------------------------------------------------------------- one layer-step workload
def bench_layer_config(torch, rov, wl, ci, main_s, side_s, sync, ev_pair, iters=9, variants=False):
    """Workloads 1-4: the GEMMs of the configuration, the keep-mask of its attention and the attention,
    under the three schedules (`rov_layer_step`: the paper's silicon experiment, Sec. 6.1, with every
    GEMM of the configuration beside the RNG).  Inputs are drawn on the device."""
    c = wl.CONFIGS[ci]
    B, H, Hkv, S, d, p = c["B"], c["H"], c["Hkv"], c["S"], c["d"], c["p"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 + ci)
    kind = c["dtype"]
    act_dt = torch.float32 if kind == "fp32" else torch.bfloat16

    def quant(x):
        scale = float(x.abs().max()) / 448.0
        return (x / scale).to(torch.float8_e4m3fn), scale

    descs, keep, flops = [], [], []
    shapes = list(c["gemms"])
    if kind == "fp8":
        shapes = shapes + [("ffn_gate",) + tuple(c["gemms"][2][1:])]      # gate and up both run
    for _, M, K, N in shapes:
        a = torch.randn(M, K, device="cuda", generator=gen)
        w = torch.randn(N, K, device="cuda", generator=gen) * 0.02
        if kind == "fp8":
            a, sa = quant(a)
            w, sw = quant(w)
        else:
            a, w, sa, sw = a.to(act_dt), w.to(act_dt), 1.0, 1.0
        C = torch.empty((M, N), dtype=torch.float32 if kind == "fp32" else torch.bfloat16, device="cuda")
        descs.append(rov.make_gemm_desc(a, w, C, scaleA=sa, scaleB=sw))
        keep += [a, w, C]
        flops.append(2.0 * M * N * K)
    Q = torch.randn(B, S, H, d, device="cuda", generator=gen).to(act_dt)
    Kt = torch.randn(B, S, Hkv, d, device="cuda", generator=gen).to(act_dt)
    V = torch.randn(B, S, Hkv, d, device="cuda", generator=gen).to(act_dt)
    O = torch.empty_like(Q)
    mask = torch.empty(rov.mask_shape(B, H, S), dtype=torch.int64, device="cuda")
    ad = rov.make_attn_desc(Q, Kt, V, O, p)
    nbits = B * H * S * S
    flop = float(sum(flops))
    peak = PEAK_FP8_TFLOPS if kind == "fp8" else PEAK_BF16_TFLOPS
    attn_flops = 4.0 * B * H * S * S * d
    sync()   # the inputs were produced on torch's current stream

    def step(sched, **kw):
        rov.layer_step(sched, descs, ad, wl.SEED, 0, None if sched == rov.SCHED_FUSED else mask, main_s, side_s, **kw)

    def gemms_only():
        for g in descs:
            rov.gemm_desc(g, stream=main_s)

    def norng():     # the same GEMMs and attention with the mask already in HBM
        gemms_only()
        rov.attention_fwd_dropout(Q, Kt, V, p, mask=mask, O=O, stream=main_s)

    res = {"workload": c["name"], "B": B, "H": H, "Hkv": Hkv, "S": S, "d": d, "p": p, "dtype": kind,
           "gemms": [{"name": n, "M": M, "K": K, "N": N} for n, M, K, N in shapes], "mask_bits": nbits}
    with torch.cuda.stream(main_s):
        rov.dropout_mask_generate(wl.SEED, 0, B, H, S, p, out=mask, stream=main_s)
        stabilise(lambda: step(rov.SCHED_OVERLAP), ev_pair)

        def hook():
            t = trace_by_kind(rov)
            return {"gemm": t.get(rov.TRACE_GEMM, []), "rng": t.get(rov.TRACE_RNG, []),
                    "helper": t.get(rov.TRACE_RNG_HELPER, []), "attention": t.get(rov.TRACE_ATTENTION, [])}

        fns = {"rng": lambda: rov.dropout_mask_generate(wl.SEED, 0, B, H, S, p, out=mask, stream=main_s),
               "gemms": gemms_only,
               "attn_none": lambda: rov.attention_fwd_dropout(Q, Kt, V, 0.0, O=O, stream=main_s),
               "attn_mask": lambda: rov.attention_fwd_dropout(Q, Kt, V, p, mask=mask, O=O, stream=main_s),
               "attn_fused": lambda: rov.attention_fwd_dropout(Q, Kt, V, p, seed=wl.SEED, offset=0, O=O, stream=main_s),
               "sequential": lambda: step(rov.SCHED_SEQUENTIAL), "fused": lambda: step(rov.SCHED_FUSED),
               "norng": norng, "overlap": lambda: step(rov.SCHED_OVERLAP)}
        for f in fns.values():
            f()
        rov.trace_enable(True)
        rov.trace_read()
        med, extra = interleaved_medians(fns, iters, ev_pair, sync, after={k: hook for k in fns})
        rov.trace_enable(False)
        rov.trace_read()
        n = len(descs)
        rows = [r for r in extra["overlap"] if len(r["gemm"]) == n]
        g_in = float(np.median([sum(r["gemm"]) for r in rows]))
        rng_in = float(np.median([sum(r["rng"]) for r in rows]))
        helper = [sum(r["helper"]) for r in rows if r["helper"]]
        helper_ms = float(np.median(helper)) if helper else 0.0
        res.update({
            "rng_alone": {"ms": med["rng"], "gbit_s": nbits / med["rng"] / 1e6, "gcalls_s": nbits / 4 / med["rng"] / 1e6},
            "gemms_alone": {"ms": med["gemms"], "tflops": flop / med["gemms"] / 1e9, "mfma_frac": flop / med["gemms"] / 1e9 / peak},
            "gemms_beside_rng": {"ms": g_in, "tflops": flop / g_in / 1e9, "mfma_frac": flop / g_in / 1e9 / peak,
                                 "slowdown_vs_alone": g_in / med["gemms"] - 1.0},
            "rng_beside_gemms": {"ms": rng_in, "helper_launch_ms": helper_ms, "rate_vs_alone": med["rng"] / rng_in},
            # hidden = 1 - (T[GEMM || RNG] - T[GEMM]) / T[RNG] on the region (GEMMs beside the RNG + the full-speed
            # helper launch), and on the whole step against the same step with the mask already in HBM
            "rng_hidden_fraction_gemm_region": 1.0 - max(g_in + helper_ms - med["gemms"], 0.0) / med["rng"],
            "rng_hidden_fraction_whole_step": 1.0 - max(med["overlap"] - med["norng"], 0.0) / med["rng"],
            "attention": {"none_ms": med["attn_none"], "mask_ms": med["attn_mask"], "fused_ms": med["attn_fused"],
                          "mask_tflops": attn_flops / med["attn_mask"] / 1e9,
                          "dropping_overhead": med["attn_mask"] / med["attn_none"] - 1.0},
            "step_ms": {"sequential": med["sequential"], "fused": med["fused"], "overlap": med["overlap"],
                        "without_rng": med["norng"]},
            "speedup_overlap_vs_sequential": med["sequential"] / med["overlap"],
            "speedup_overlap_vs_fused": med["fused"] / med["overlap"],
        })
        if variants:
            # fewer Philox rounds and narrower random numbers per element (paper Sec. 5.2; its silicon numbers are for 7 rounds)
            var = {}
            for key, kw in (("philox_7", dict(rounds=7)), ("philox_5", dict(rounds=5)), ("philox_3", dict(rounds=3)),
                            ("bits_16", dict(bits=16)), ("bits_8", dict(bits=8))):
                if "rounds" in kw:
                    rng_fn = lambda kw=kw: rov.dropout_mask_generate(wl.SEED, 0, B, H, S, p, out=mask, rounds=kw["rounds"], stream=main_s)
                else:
                    rng_fn = lambda kw=kw: rov.dropout_mask_generate_bits(wl.SEED, 0, B, H, S, p, kw["bits"], out=mask, stream=main_s)
                vf = {"rng": rng_fn, "sequential": lambda kw=kw: step(rov.SCHED_SEQUENTIAL, **kw),
                      "fused": lambda kw=kw: step(rov.SCHED_FUSED, **kw), "overlap": lambda kw=kw: step(rov.SCHED_OVERLAP, **kw)}
                for f in vf.values():
                    f()
                m, _ = interleaved_medians(vf, iters, ev_pair, sync)
                var[key] = {"rng_ms": m["rng"], "sequential_ms": m["sequential"], "fused_ms": m["fused"], "overlap_ms": m["overlap"],
                            "speedup_overlap_vs_sequential": m["sequential"] / m["overlap"],
                            "speedup_overlap_vs_fused": m["fused"] / m["overlap"],
                            "rng_hidden_fraction_whole_step": (m["sequential"] - m["overlap"]) / m["rng"]}
            res["rng_variants"] = var
    del keep, descs, Q, Kt, V, O, mask
    torch.cuda.empty_cache()
    return res


def all_configs(torch, rov, wl, main_s, side_s, sync, ev_pair, outdir):
    """One record per workload under `outdir` and the scaling laws of paper Sec. 4.1 between them
    (RNG time ~ B*H*S^2, GEMM time ~ M*N*K, attention time ~ B*H*S^2*d)."""
    os.makedirs(outdir, exist_ok=True)
    recs = []
    for ci in range(4):
        print("all-configs: workload", ci + 1, wl.CONFIGS[ci]["name"], file=sys.stderr, flush=True)
        r = bench_layer_config(torch, rov, wl, ci, main_s, side_s, sync, ev_pair, iters=7)
        recs.append(r)
        json.dump(r, open(os.path.join(outdir, "bench_config%d_%s.json" % (ci + 1, r["workload"])), "w"), indent=1)
    print("all-configs: workload 5 (block)", file=sys.stderr, flush=True)
    blk = Block(torch, rov, wl)
    sync()
    with torch.cuda.stream(main_s):
        blk.prime(main_s)
        stabilise(lambda: blk.ovl(main_s, side_s), ev_pair)
        med, g_alone, g_ovl, rng_in, helper, rng_seq, attn_ovl = block_schedules(blk, rov, main_s, side_s, sync, ev_pair, 7)
        t_rng = median_ms(lambda: rov.dropout_mask_generate(wl.SEED, 0, blk.B, blk.H, blk.S, blk.p, out=blk.m1, stream=main_s),
                          2, 7, sync, ev_pair, inner=3)
    flop = sum(blk.gemm_flops.values())
    r5 = {"workload": wl.CONFIGS[4]["name"], "B": blk.B, "H": blk.H, "Hkv": blk.Hkv, "S": blk.S, "d": blk.d, "p": blk.p,
          "dtype": "bf16", "mask_bits": blk.nbits,
          "rng_alone": {"ms": t_rng, "gbit_s": blk.nbits / t_rng / 1e6, "gcalls_s": blk.nbits / 4 / t_rng / 1e6},
          "gemms_alone": {"ms": sum(g_alone), "tflops": flop / sum(g_alone) / 1e9, "mfma_frac": flop / sum(g_alone) / 1e9 / PEAK_BF16_TFLOPS,
                          "per_gemm_ms": dict(zip(GEMM_NAMES, g_alone))},
          "gemms_beside_rng": {"ms": sum(g_ovl), "tflops": flop / sum(g_ovl) / 1e9, "mfma_frac": flop / sum(g_ovl) / 1e9 / PEAK_BF16_TFLOPS,
                               "per_gemm_ms": dict(zip(GEMM_NAMES, g_ovl)),
                               "slowdown_vs_alone": sum(g_ovl) / sum(g_alone) - 1.0},
          "rng_beside_gemms": {"ms": rng_in[0], "helper_launch_ms": helper[0] if helper else 0.0, "rate_vs_alone": t_rng / rng_in[0]},
          "rng_hidden_fraction_gemm_region": 1.0 - max(sum(g_ovl) + (helper[0] if helper else 0.0) - sum(g_alone), 0.0) / t_rng,
          "rng_hidden_fraction_whole_step": 1.0 - max(med["overlap"] - med["norng"], 0.0) / t_rng,
          "attention": {"mask_ms": attn_ovl[0], "mask_tflops": blk.attn_flops / attn_ovl[0] / 1e9},
          "step_ms": {"sequential": med["sequential"], "fused": med["fused"], "overlap": med["overlap"], "without_rng": med["norng"]},
          "speedup_overlap_vs_sequential": med["sequential"] / med["overlap"],
          "speedup_overlap_vs_fused": med["fused"] / med["overlap"]}
    recs.append(r5)
    cpu_baseline_masks(wl, recs)
    for ci, r in enumerate(recs):
        json.dump(r, open(os.path.join(outdir, "bench_config%d_%s.json" % (ci + 1, r["workload"])), "w"), indent=1)
    # scaling laws: time per unit of work should be flat across the workloads that fill the device
    law = []
    for r in recs:
        gf = sum(2.0 * g["M"] * g["N"] * g["K"] for g in r["gemms"]) if "gemms" in r else flop
        law.append({"workload": r["workload"],
                    "rng_ps_per_bit": r["rng_alone"]["ms"] * 1e9 / r["mask_bits"],
                    "gemm_ps_per_kflop": r["gemms_alone"]["ms"] * 1e9 / (gf / 1e3),
                    "attention_mask_ps_per_kflop": r["attention"]["mask_ms"] * 1e9 / (4.0 * r["B"] * r["H"] * r["S"] ** 2 * r["d"] / 1e3)})
    summary = {"scaling_law_check_paper_sec_4_1": law,
               "note": "RNG ~ B*H*S^2, GEMM ~ M*N*K, attention ~ B*H*S^2*d: the per-unit times of workloads 2-5 agree to "
                       "within their tile-round effects; workload 1 (tiny) is launch-bound, and workload 4's GEMMs are fp8"}
    json.dump(summary, open(os.path.join(outdir, "bench_all_configs_summary.json"), "w"), indent=1)
    print(json.dumps({"all_configs": [r["workload"] for r in recs], "summary": summary}))


def seq_sweep(torch, rov, wl, main_s, side_s, sync, ev_pair):
    from paper_2410_07531_amd import limiter_model as LM
    c5 = wl.CONFIGS[4]
    out = {}
    for S_ in (2048, 4096, 8192, 16384, 32768):
        print("seq-sweep: S =", S_, file=sys.stderr, flush=True)
        blk = Block(torch, rov, wl, seq_len=S_)
        sync()
        with torch.cuda.stream(main_s):
            blk.prime(main_s)
            stabilise(lambda: blk.ovl(main_s, side_s), ev_pair)
            med, *_ = block_schedules(blk, rov, main_s, side_s, sync, ev_pair, 5)
            r = {"sequential_ms": med["sequential"], "fused_ms": med["fused"], "overlap_ms": med["overlap"],
                 "without_rng_ms": med["norng"],
                 "speedup_overlap_vs_sequential": med["sequential"] / med["overlap"],
                 "speedup_overlap_vs_fused": med["fused"] / med["overlap"]}
            rows = rov.block_hybrid_mask_rows(blk.cfg, blk.B, S_)
            r["hybrid_mask_rows"] = rows
            if 0 < rows < S_:
                blk.settle()
                blk.layer = 0
                rov.dropout_mask_generate_rows(wl.SEED, 0, blk.B, blk.H, S_, blk.p, 0, rows, out=blk.m0, stream=main_s)
                r["hybrid_ms"] = median_ms(lambda: blk.ovl(main_s, side_s, rov.SCHED_HYBRID), 2, 5, sync, ev_pair, inner=2)
            # the schedules drop the same elements: outputs agree bit for bit
            outs = []
            for fn in (blk.seq, blk.fus):
                sync()
                fn(main_s, side_s)
                sync()
                outs.append(blk.y.clone())
            blk.prime(main_s)
            sync()
            blk.ovl(main_s, side_s, sched=rov.SCHED_OVERLAP)
            sync()
            r["schedules_agree_bit_for_bit"] = bool(torch.equal(outs[0], outs[1]) and torch.equal(outs[0], blk.y))
        bm = LM.block(LM.MI355X, c5["B"], S_, c5["H"], c5["Hkv"], c5["d"], c5["hidden"], c5["ffn"], False)
        r["limiter_model_ms"] = {"sequential": bm["baseline"] * 1e3, "fused": bm["fusion"] * 1e3,
                                 "overlap": bm["overlap"] * 1e3, "rng": bm["rng"] * 1e3,
                                 "rng_exposed": bm["rng_exposed"] * 1e3}
        r["limiter_model_region"] = LM.region(LM.MI355X, c5["B"], c5["H"], S_, c5["d"], c5["hidden"], c5["ffn"])
        out["S=%d" % S_] = r
        del blk, outs
        torch.cuda.empty_cache()
    print(json.dumps({"seq_sweep_llama3_8b_block": out}))


def kernels_only(torch, rov, wl, main_s, side_s, sync):
    """For rocprofv3: a 1 GiB copy (counter calibration), each kernel of the S=16384 block alone and
    the overlap block step, three times each."""
    blk = Block(torch, rov, wl)
    B, H, Hkv, S, d, p, hidden, ffn = blk.B, blk.H, blk.Hkv, blk.S, blk.d, blk.p, blk.hidden, blk.ffn
    T = B * S
    bf = torch.bfloat16
    src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    a_h = torch.randn(T, hidden, device="cuda").to(bf)
    a_att = torch.randn(T, H * d, device="cuda").to(bf)
    a_u = torch.randn(T, ffn, device="cuda").to(bf)
    c_qkv = torch.empty(T, (H + 2 * Hkv) * d, dtype=bf, device="cuda")
    c_h = torch.empty(T, hidden, dtype=bf, device="cuda")
    c_u = torch.empty(T, ffn, dtype=bf, device="cuda")
    Q = torch.randn(B, S, H, d, device="cuda").to(bf)
    Kt = torch.randn(B, S, Hkv, d, device="cuda").to(bf)
    V = torch.randn(B, S, Hkv, d, device="cuda").to(bf)
    O = torch.empty_like(Q)
    sync()
    with torch.cuda.stream(main_s):
        for _ in range(3):
            dst.copy_(src)                                     # reads 1 GiB, writes 1 GiB
        for _ in range(3):
            rov.dropout_mask_generate(wl.SEED, 0, B, H, S, p, out=blk.m0, stream=main_s)
        for _ in range(3):
            rov.gemm(a_h, blk.wts["wqkv"], C=c_qkv, stream=main_s)
        for _ in range(3):
            rov.gemm(a_att, blk.wts["wo"], C=c_h, stream=main_s)
        for _ in range(3):
            rov.gemm_swiglu(a_h, blk.wts["wg"], blk.wts["wu"], C=c_u, stream=main_s)
        for _ in range(3):
            rov.gemm(a_u, blk.wts["wd"], C=c_h, stream=main_s)
        for _ in range(3):
            rov.attention_fwd_dropout(Q, Kt, V, 0.0, O=O, stream=main_s)
        for _ in range(3):
            rov.attention_fwd_dropout(Q, Kt, V, p, mask=blk.m0, O=O, stream=main_s)
        for _ in range(3):
            rov.attention_fwd_dropout(Q, Kt, V, p, seed=wl.SEED, offset=0, O=O, stream=main_s)
        sync()
        blk.prime(main_s)
        blk.ovl_chain(main_s, side_s, 4)
    sync()
    print("kernels-only run done", file=sys.stderr)


def kernels_only_fp8(torch, rov, wl, main_s, side_s, sync):
    """For rocprofv3: a 1 GiB copy (counter calibration), then the 70B-shaped fp8 block: sequential (each of its
    kernels runs alone: quantising RMSNorm, e4m3 GEMMs, RoPE, mask kernel, attention with e4m3 output, dual
    SwiGLU GEMM with e4m3 output), fused, and a chain of overlap blocks."""
    blk = Block(torch, rov, wl, ci=3)
    src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    sync()
    with torch.cuda.stream(main_s):
        for _ in range(3):
            dst.copy_(src)
        for _ in range(3):
            blk.seq(main_s, side_s)
        for _ in range(3):
            blk.fus(main_s, side_s)
        sync()
        blk.prime(main_s)
        blk.ovl_chain(main_s, side_s, 4)
    sync()
    print("kernels-only (fp8 block) run done", file=sys.stderr)


# ---------------------------------------------------------------------------------------------- CPU oracle
def cpu_baseline_masks(wl, recs):
    """The CPU oracle's mask of every workload, in full, timed beside the device's (--all-configs)."""
    from oracle import philox as OP
    for ci, r in enumerate(recs):
        c = wl.CONFIGS[ci]
        t0 = time.perf_counter()
        OP.dropout_mask(wl.SEED, wl.OFFSET, c["B"], c["H"], c["S"], c["p"])
        dt = time.perf_counter() - t0
        r["cpu_oracle_mask"] = {"s": dt, "gbit_s": r["mask_bits"] / dt / 1e9, "cores": OP.num_threads(), "kind": "oracle"}


def cpu_baseline(wl):
    """The oracle as it stands, timed on this machine's host cores on a bounded sample of the block step:
    the whole mask (all 32 heads), and the oracle's block on 2048 sampled token rows (QKV projection of every
    token, attention of the sampled rows against the full K, V of every head, the rest on those rows); each part extrapolated to the whole
    block by its work count."""
    import torch
    from oracle import dense as OD
    from oracle import numerics as ON
    from oracle import philox as OP
    ci = 4
    c = wl.CONFIGS[ci]
    B, H, Hkv, S, d, p, hidden, ffn = c["B"], c["H"], c["Hkv"], c["S"], c["d"], c["p"], c["hidden"], c["ffn"]
    nbits = B * H * S * S
    heads = H
    t0 = time.perf_counter()
    words = OP.dropout_mask(wl.SEED, wl.OFFSET, 1, heads, S, p)
    t_mask = (time.perf_counter() - t0) * (H / heads)
    rng = wl.rng_for(ci)
    nrows = 2048
    rows = wl.sample_rows(S, nrows)
    # dense part on a reduced block of the same shapes per token: all S tokens feed K and V, the
    # sampled rows go through every row-wise stage
    w = wl.block_weights(rng, H, Hkv, d, hidden, ffn)
    x = wl.block_input(rng, B, S, hidden)
    wr = {k: ON.bf16_round(v).astype(np.float64) for k, v in w.items()}
    xr = ON.bf16_round(x).astype(np.float64)
    # real keep bits for the first four heads, all-kept elsewhere: the oracle's work does not depend on the
    # bits, and unpacking all 32 heads would cost more host time than the sample itself
    keep = np.ones((B, H, S, S), dtype=bool)
    keep[:, :4] = OP.unpack_keep(words[:, :4], S)
    del words
    cfg = dict(H=H, Hkv=Hkv, d=d, eps=1e-5, rope_theta=500000.0, p=p, causal=False)
    t0 = time.perf_counter()
    OD.block_forward(xr, wr, cfg, keep, rows=rows)
    t_dense_sample = time.perf_counter() - t0
    # work of the sample: the QKV projection of all S tokens + everything after it for len(rows) tokens
    T = B * S
    full = 2.0 * T * ((H + 2 * Hkv) * d * hidden + hidden * H * d + 3 * ffn * hidden) + 4.0 * B * H * S * S * d
    sample = (2.0 * T * (H + 2 * Hkv) * d * hidden                        # the oracle projects every token to q, k, v
              + 2.0 * len(rows) * (hidden * H * d + 3 * ffn * hidden)
              + 4.0 * B * H * len(rows) * S * d)
    t_dense = t_dense_sample * full / sample
    total = t_mask + t_dense
    return {"value": nbits / t_mask / 1e9, "unit": "Gbit/s", "cores": max(OP.num_threads(), torch.get_num_threads()),
            "kind": "oracle",
            "sample": "mask: %d of %d heads of the 32x16384x16384-bit mask (%.2f s measured, %.1f s extrapolated to all "
                      "heads); block: the oracle's block_forward on %d sampled token rows with K, V of all %d tokens "
                      "(%.1f s measured, %.0f s extrapolated by flop count to the whole block)"
                      % (heads, H, t_mask * heads / H, t_mask, len(rows), S, t_dense_sample, t_dense),
            "block_step_s_extrapolated": total, "block_steps_per_s": 1.0 / total}


if __name__ == "__main__":
    main()
