"""GPU parity of fp32 attention in its two tile heights: 16 query rows where 32-row tiles are few, 32 rows elsewhere.

Sizes at which they can go wrong: sequences that end 1, 15, 16 or 17 keys into a tile, fewer key blocks than waves, head
dimensions that end in the first or second half of a 16-feature chunk, grouped keys, ranges of rows, non-finite values under keys
that a query does not admit.  Reference: the float64 oracle; bar 1e-4 of the result's scale (hardware exp2, fp32 sums).
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


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,S,H,Hkv,d,rows", [
    (1, 65, 2, 1, 32, (16, 16)), (1, 79, 2, 2, 48, (16, 16)), (1, 80, 1, 1, 8, (16, 16)), (1, 81, 3, 3, 72, (16, 16)), (1, 113, 2, 1, 120, (16, 16)),
    (2, 129, 4, 2, 128, (16, 16)), (1, 190, 6, 2, 88, (16, 16)), (1, 300, 2, 2, 64, (16, 16)), (4, 70, 32, 8, 64, (32, 32)), (2, 129, 32, 8, 96, (32, 32)),
    (3, 97, 20, 20, 128, (32, 32)), (2, 128, 16, 4, 64, (16, 16)), (2, 129, 16, 4, 40, (16, 16)), (1, 257, 17, 17, 40, (32, 16)),   # 256, 288, 289 tiles of 16 rows
])
def test_both_tile_heights_match_oracle(B, S, H, Hkv, d, rows, causal):
    print("attn fp32 q16", B, S, H, Hkv, d, causal, flush=True)
    assert rov.attention_tile_rows(B, H, S, d, rov.F32, causal) == rows[causal]
    p, seed, offset = 0.2, wl.SEED, 2**32 - 200
    q, k, v = wl.qkv(np.random.default_rng(S + d), B, S, H, Hkv, d)
    Q, K, V = (torch.from_numpy(x).cuda() for x in (q, k, v))
    keep = OP.unpack_keep(OP.dropout_mask(seed, offset, B, H, S, p), S)
    mask = rov.dropout_mask_generate(seed, offset, B, H, S, p)
    O = {"mask": rov.attention_fwd_dropout(Q, K, V, p, mask=mask, causal=causal),
         "fused": rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, causal=causal),
         "none": rov.attention_fwd_dropout(Q, K, V, 0.0, causal=causal), "rows": torch.full_like(Q, 7.0)}
    for q0 in range(0, S, 32):
        part = rov.dropout_mask_generate_rows(seed, offset, B, H, S, p, q0, 32)
        rov.attention_fwd_dropout_rows(Q, K, V, p, q0, 32, O["rows"], mask_rows=part, causal=causal)
    torch.cuda.synchronize()
    assert torch.equal(O["mask"], O["fused"]) and torch.equal(O["mask"], O["rows"])
    f64 = [x.astype(np.float64) for x in (q, k, v)]
    err = lambda got, ref: float(np.max(np.abs(got.double().cpu().numpy() - ref)) / np.max(np.abs(ref)))
    assert err(O["mask"], OD.attention_dropout(*f64, keep, p, causal=causal)) <= TOL
    assert err(O["none"], OD.attention_dropout(*f64, None, 0.0, causal=causal)) <= TOL


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("H,rows", [(2, 16), (80, 32)])
def test_narrow_fields_are_the_mask_kernels(bits, H, rows):
    B, S, d, p, seed, offset = 1, 83, 40, 0.3, 77, 640
    assert rov.attention_tile_rows(B, H, S, d, rov.F32, False) == rows
    Q, K, V = (torch.from_numpy(x).cuda() for x in wl.qkv(np.random.default_rng(1), B, S, H, H, d))
    mask = rov.dropout_mask_generate_bits(seed, offset, B, H, S, p, bits)
    a = rov.attention_fwd_dropout(Q, K, V, p, mask=mask)
    b = rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, bits=bits)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("S,bad", [(67, 40), (67, 66), (130, 129), (130, 17)])
def test_values_of_inadmissible_keys_stay_out(S, bad):
    # causal: queries before key `bad` do not see its infinite value; memory behind the last key is NaN
    g = torch.Generator().manual_seed(S)
    Q, K = (torch.randn(1, S, 2, 64, generator=g).cuda() for _ in range(2))
    buf = torch.full((S * 2 * 64 + 4096,), float("nan"), device="cuda")
    buf[:S * 128] = torch.randn(S * 128, generator=g).cuda()
    V = buf[:S * 128].view(1, S, 2, 64)
    ref = rov.attention_fwd_dropout(Q, K, V, 0.0, causal=True)
    V[0, bad] = float("inf")
    O = rov.attention_fwd_dropout(Q, K, V, 0.0, causal=True)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(ref).all())
    assert float((O[0, :bad] - ref[0, :bad]).abs().max()) <= TOL * float(ref.abs().max())
    assert not bool(torch.isfinite(O[0, bad]).any())
