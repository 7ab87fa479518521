"""Masks shared between the small grid beside the GEMMs and the launch behind them: the two launches of a fixed split
and of a work queue write every chunk exactly as one launch does."""
import numpy as np
import pytest
import torch

from oracle import philox as OP
from paper_2410_07531_amd import binding as rov
from paper_2410_07531_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,H,causal,M,share", [
    # share: chunks of 64 words that the small grid makes (of H * ceil(S/32)^2 / 4), -1: a work queue
    (512, 8, False, 16, 0),         # its share would be too small for a launch: one launch behind the GEMM
    (512, 8, False, 64, 33),
    (1024, 8, False, 2048, 1066),   # a part of the mask
    (1000, 8, True, 1024, 1066),    # ragged, causal: the cut falls inside a head
    (1024, 8, True, 1024, 1066),    # causal, workgroups left out of the grid of either share
    (2048, 4, False, 3000, 1562),
    (512, 2, False, 4096, 128),     # everything fits beside the GEMM: no second launch
    (8192, 12, True, 512, -1),
])
def test_overlap_masks_equal_the_single_launch(S, H, causal, M, share):
    print("mask split", S, H, causal, M, share, flush=True)
    B, d, K, p, seed, offset = 1, 64, 1024, 0.1, wl.SEED, 2**32 - 777
    g = torch.Generator("cuda").manual_seed(S)
    Q, Kt, V = (torch.randn(B, S, H, d, device="cuda", generator=g).bfloat16() for _ in range(3))
    A = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    W = torch.randn(K, K, device="cuda", generator=g).bfloat16()
    C, O = torch.empty(M, K, dtype=torch.bfloat16, device="cuda"), torch.empty_like(Q)
    gen = rov.dropout_mask_generate_causal if causal else rov.dropout_mask_generate
    ref = torch.full(rov.mask_shape(B, H, S), 0x2AAAAAAAAAAAAAAA, dtype=torch.int64, device="cuda")
    gen(seed, offset, B, H, S, p, out=ref)
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    T = (S + 31) // 32
    assert rov.overlap_mask_chunks(2.0 * M * K * K, rov.BF16, B, H, S, causal) == share
    launches = {0: [0, 1], (H * T * T + 3) // 4: [1, 0]}.get(share, [1, 1])      # small grid, full-speed launch
    for _ in range(2):
        mask = torch.full_like(ref, 0x2AAAAAAAAAAAAAAA)
        torch.cuda.synchronize()
        rov.trace_read()
        rov.trace_enable(True, [rov.TRACE_RNG, rov.TRACE_RNG_HELPER])
        try:
            rov.layer_step(rov.SCHED_OVERLAP, [rov.make_gemm_desc(A, W, C)], rov.make_attn_desc(Q, Kt, V, O, p, causal=causal),
                           seed, offset, mask, main, side)
        finally:
            rov.trace_enable(False)
        torch.cuda.synchronize()
        kinds = [k for k, _ in rov.trace_read()]
        assert [kinds.count(rov.TRACE_RNG), kinds.count(rov.TRACE_RNG_HELPER)] == launches
        assert torch.equal(mask, ref)
    first = (H - 1) * T * T * 16
    exp = OP.dropout_mask(seed, offset + 64 * (first // 4), 1, 1, S, p)[0, 0]
    got = mask[0, H - 1].cpu().numpy().view(np.uint64)
    lower = np.tril(np.ones((T, T), dtype=bool)) if causal else np.ones((T, T), dtype=bool)
    assert np.array_equal(got[lower], exp[lower])
