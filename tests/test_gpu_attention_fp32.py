"""GPU parity of fp32 attention: the kernel on the matrix instructions and, for a few rows, the one-row-per-wave kernel.

Sizes at which the former can go wrong: tiles of 32 partly filled, fewer key tiles than waves,
head dimensions that fill a feature tile, a part of one, or several; causal and not; grouped keys; strided
views.  The rows assert which of the two they reach.  Reference: the float64 oracle; bar 1e-4 of the result's scale (hardware exp2, fp32 sums).
"""
import numpy as np
import pytest
import torch

from oracle import dense as OD
from oracle import philox as OP
from paper_2410_07531_amd import binding as rov
from paper_2410_07531_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-4


def _err(got, ref):
    # (a fully dropped result is all zeros on both sides)
    return float(np.max(np.abs(got.double().cpu().numpy() - ref)) / max(np.max(np.abs(ref)), 1e-30))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,S,H,Hkv,d,waves", [
    (1, 1, 1, 1, 8, 0), (1, 4, 2, 1, 32, 0), (2, 9, 128, 32, 40, 0), (2, 12, 100, 50, 128, 0),   # few rows: one row a wave
    (1, 5, 1, 1, 8, 8), (1, 33, 2, 1, 32, 8), (1, 40, 2, 2, 128, 4),       # tiles of 16 rows
    (8, 20, 64, 16, 8, 8), (4, 33, 16, 4, 32, 8), (8, 32, 32, 32, 128, 4),  # one or two key tiles, many heads
    (2, 65, 8, 4, 40, 8), (1, 300, 4, 2, 64, 8), (1, 97, 3, 3, 80, 4), (1, 70, 2, 2, 96, 4), (2, 129, 2, 1, 128, 4), (1, 100, 2, 2, 104, 4),
])
def test_fp32_matches_oracle(B, S, H, Hkv, d, waves, causal):
    print("attn fp32", B, S, H, Hkv, d, causal, flush=True)
    assert rov.attention_key_parts(B, H, S, d, rov.F32, causal) == waves
    p, seed, offset = 0.2, wl.SEED, 2**32 - 200        # call numbers carry into the second counter word
    q, k, v = wl.qkv(np.random.default_rng(S + d), B, S, H, Hkv, d)
    Q, K, V = (torch.from_numpy(x).cuda() for x in (q, k, v))
    keep = OP.unpack_keep(OP.dropout_mask(seed, offset, B, H, S, p), S)
    mask = rov.dropout_mask_generate(seed, offset, B, H, S, p)
    O = {"mask": rov.attention_fwd_dropout(Q, K, V, p, mask=mask, causal=causal),
         "fused": rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, causal=causal),
         "none": rov.attention_fwd_dropout(Q, K, V, 0.0, causal=causal), "rows": torch.full_like(Q, 7.0)}
    for q0 in range(0, S, 64):
        part = rov.dropout_mask_generate_rows(seed, offset, B, H, S, p, q0, 64)
        rov.attention_fwd_dropout_rows(Q, K, V, p, q0, 64, O["rows"], mask_rows=part, causal=causal)
    torch.cuda.synchronize()
    assert torch.equal(O["mask"], O["fused"]) and torch.equal(O["mask"], O["rows"])
    f64 = [x.astype(np.float64) for x in (q, k, v)]
    assert _err(O["mask"], OD.attention_dropout(*f64, keep, p, causal=causal)) <= TOL
    assert _err(O["none"], OD.attention_dropout(*f64, None, 0.0, causal=causal)) <= TOL


@pytest.mark.parametrize("H,rows", [(2, 16), (80, 32)])     # query tiles of either height
@pytest.mark.parametrize("rounds,bits", [(7, 32), (3, 32), (10, 16), (10, 8)])
def test_fp32_fused_variants_draw_the_mask_kernels_bits(rounds, bits, H, rows):
    B, S, d, p, seed, offset = 1, 90, 64, 0.3, 77, 640
    assert rov.attention_tile_rows(B, H, S, d, rov.F32, False) == rows
    Q, K, V = (torch.from_numpy(x).cuda() for x in wl.qkv(np.random.default_rng(1), B, S, H, H, d))
    if bits == 32:
        mask = rov.dropout_mask_generate(seed, offset, B, H, S, p, rounds=rounds)
        fused = rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, rounds=rounds)
    else:
        mask = rov.dropout_mask_generate_bits(seed, offset, B, H, S, p, bits)
        fused = rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, bits=bits)
    assert torch.equal(fused, rov.attention_fwd_dropout(Q, K, V, p, mask=mask))


@pytest.mark.parametrize("H,rows", [(2, 16), (80, 32)])
def test_fp32_strided_views(H, rows):
    # Q, K, V as slices of one projection output; a row stride that is no multiple of 4 takes the general kernel
    B, S, d = 1, 70, 64
    assert rov.attention_tile_rows(B, H, S, d, rov.F32, True) == rows
    for pad in (0, 1):
        x = torch.randn(B, S, 3 * H * d + pad, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
        Q, K, V = (x[..., i * H * d:(i + 1) * H * d].unflatten(-1, (H, d)) for i in range(3))
        O = torch.empty(B, S, H, d, device="cuda")
        rov.attention_fwd_dropout(Q, K, V, 0.0, causal=True, O=O)
        ref = OD.attention_dropout(*(t.double().cpu().numpy() for t in (Q, K, V)), None, 0.0, causal=True)
        assert _err(O, ref) <= TOL


@pytest.mark.parametrize("H,rows", [(1, 16), (80, 32)])
def test_fp32_causal_rows_never_see_later_values(H, rows):
    # non-finite keys and values reach the rows that admit them and no other
    B, S, d = 1, 96, 64
    assert rov.attention_key_parts(B, H, S, d, rov.F32, True) == 8 and rov.attention_tile_rows(B, H, S, d, rov.F32, True) == rows
    g = torch.Generator("cuda").manual_seed(9)
    Q, K, V = (torch.randn(B, S, H, d, device="cuda", generator=g) for _ in range(3))
    ref = rov.attention_fwd_dropout(Q, K, V, 0.0, causal=True)
    V2, K2 = V.clone(), K.clone()
    V2[0, 40, 0, 3] = float("inf")
    K2[0, 77, 0, 0] = float("nan")
    O = rov.attention_fwd_dropout(Q, K2, V2, 0.0, causal=True)
    torch.cuda.synchronize()
    assert torch.allclose(O[0, :40, 0], ref[0, :40, 0], rtol=1e-5, atol=1e-6)
    assert bool((O[0, 40:77, 0, 3] == float("inf")).all())
    others = [i for i in range(d) if i != 3]
    assert torch.allclose(O[0, 40:77, 0, others], ref[0, 40:77, 0, others], rtol=1e-5, atol=1e-6)
    assert bool(torch.isnan(O[0, 77:, 0]).all())
    assert torch.equal(O[0, :, 1:], ref[0, :, 1:])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("S,H,d", [(1, 1, 8), (20, 256, 8), (33, 128, 40), (60, 128, 64), (97, 2, 128)])
def test_fp32_rows_behind_the_last_key_are_not_part_of_the_result(S, H, d, causal):
    # K and V end inside a tile of 32 keys and what lies behind them in memory is NaN: the loads stay in the rows
    # [0, S) (the row of a load is clamped to the last one, the rest is outside its buffer's range)
    print("attn fp32 rows behind", S, H, d, causal, flush=True)
    assert (rov.attention_key_parts(1, H, S, d, rov.F32, causal) != 0) == (S > 1)
    g = torch.Generator("cuda").manual_seed(S)
    buf = [torch.full((1, S + 40, H, d), float("nan"), device="cuda") for _ in range(3)]
    Q, K, V = (x[:, :S] for x in buf)
    for x in (Q, K, V):
        x.copy_(torch.randn(1, S, H, d, device="cuda", generator=g))
    frame = torch.full((1, S + 40, H, d), 7.0, device="cuda")
    rov.attention_fwd_dropout(Q, K, V, 0.0, causal=causal, O=frame[:, :S])
    torch.cuda.synchronize()
    ref = OD.attention_dropout(*(t.double().cpu().numpy() for t in (Q, K, V)), None, 0.0, causal=causal)
    assert _err(frame[:, :S], ref) <= TOL
    assert bool((frame[:, S:] == 7.0).all())
