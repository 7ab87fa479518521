"""GPU parity of the matrix-core attention kernel where its workgroups split the keys between waves.

Short sequences, few heads and causal masks take workgroups of 128 or 64 query rows whose waves share the
keys and merge their partial results; larger problems take 256 rows and no split.  The rows reach every split at
both head dimensions, causal and not, and assert which one they reach; among them are key parts that lie beyond the sequence, row tiles past its end and causal parts without a
single admissible key.  Reference: the float64 oracle on sampled rows; bar 2e-2 of the result's scale as for
every bf16 attention test (probabilities rounded to bf16, 2^-9, one rounding of the result).
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


@pytest.mark.parametrize("B,S,H,Hkv,d,causal,parts", [
    (1, 33, 2, 1, 128, True, 4),     # 64 rows a workgroup; the second row tile has one row, two key parts none
    (1, 33, 2, 1, 64, False, 4),
    (2, 130, 3, 3, 128, False, 4),   # a second LDS tile with two keys
    (1, 257, 4, 2, 64, True, 4),     # ragged, third LDS tile with one key
    (1, 700, 24, 8, 128, False, 2),  # 128 rows
    (1, 1001, 32, 8, 64, False, 2),
    (2, 1025, 16, 4, 128, True, 2),  # causal, one row past a tile
    (2, 1000, 32, 8, 64, True, 2),
    (2, 1025, 16, 4, 64, True, 4),
    (1, 1500, 24, 8, 128, False, 1),  # 256 rows
    (1, 2001, 32, 8, 64, False, 1),
    (2, 2048, 24, 8, 128, True, 1),  # causal: waves that leave the walk early
    (4, 1279, 32, 8, 64, True, 1),
])
def test_split_keys_match_oracle_and_agree(B, S, H, Hkv, d, causal, parts):
    print("attention key parts", B, S, H, Hkv, d, causal, parts, flush=True)
    assert rov.attention_key_parts(B, H, S, d, rov.BF16, causal) == parts
    p, seed, offset = 0.1, wl.SEED, 96
    rng = np.random.default_rng(S + d)
    Q, K, V = (torch.from_numpy(x).bfloat16().cuda() for x in wl.qkv(rng, B, S, H, Hkv, d))
    mask = rov.dropout_mask_generate(seed, offset, B, H, S, p)
    O = {m: torch.full_like(Q, 7.0) for m in ("mask", "fused", "none", "rows")}
    rov.attention_fwd_dropout(Q, K, V, p, mask=mask, causal=causal, O=O["mask"])
    rov.attention_fwd_dropout(Q, K, V, p, seed=seed, offset=offset, causal=causal, O=O["fused"])
    rov.attention_fwd_dropout(Q, K, V, 0.0, causal=causal, O=O["none"])
    for q0 in range(0, S, 96):       # row ranges that cut every workgroup size
        part = rov.dropout_mask_generate_rows(seed, offset, B, H, S, p, q0, 96)
        rov.attention_fwd_dropout_rows(Q, K, V, p, q0, 96, O["rows"], mask_rows=part, causal=causal)
    torch.cuda.synchronize()
    assert torch.equal(O["mask"], O["fused"]) and torch.equal(O["mask"], O["rows"])
    rows = sorted(set(r for r in (0, 1, 31, 32, 63, 64, 127, 128, 255, 256, S // 2, S - 2, S - 1) if 0 <= r < S))
    T = (S + 31) // 32
    for b, h in ((0, 0), (B - 1, H - 1)):
        first = (b * H + h) * T * T * 16
        words = OP.dropout_mask(seed, offset + 64 * (first // 4), 1, 1, S, p)
        keep = OP.unpack_keep(words, S)
        q, k, v = _f64(Q[b:b + 1, :, h:h + 1]), _f64(K[b:b + 1, :, h // (H // Hkv):][:, :, :1]), _f64(V[b:b + 1, :, h // (H // Hkv):][:, :, :1])
        for m, kp, pp in (("mask", keep, p), ("none", None, 0.0)):
            ref = OD.attention_dropout(q, k, v, kp, pp, causal=causal, rows=rows)[0, :, 0]
            got = _f64(O[m][b, rows, h])
            assert np.max(np.abs(got - ref)) / np.max(np.abs(ref)) <= 2e-2, (m, b, h)


def test_key_parts_with_scores_far_apart():
    # the parts' exponent references differ by hundreds of log2 units: one part holds all the weight of a row
    B, S, H, d = 1, 256, 2, 128
    g = torch.Generator().manual_seed(3)
    Q = torch.randn(B, S, H, d, generator=g)
    K = torch.randn(B, S, H, d, generator=g)
    K[:, 96:128] = Q[:, 96:128] * 4.0            # keys of the last 32-key part of the first LDS tile
    V = torch.randn(B, S, H, d, generator=g)
    Q, K, V = (t.bfloat16().cuda() for t in (Q, K, V))
    O = rov.attention_fwd_dropout(Q, K, V, 0.0)
    ref = OD.attention_dropout(_f64(Q), _f64(K), _f64(V), None, 0.0, causal=False)
    assert np.max(np.abs(_f64(O) - ref)) / np.max(np.abs(ref)) <= 2e-2


@pytest.mark.parametrize("mode", ["mask", "fused", "none"])
def test_split_keys_repeat_bit_for_bit(mode):
    # the parts are merged in a fixed order: repeated calls, on other streams and beside other work too, give the same bits
    B, S, H, Hkv, d, causal, p = 2, 1000, 16, 4, 64, True, 0.1
    assert rov.attention_key_parts(B, H, S, d, rov.BF16, causal) == 4
    Q, K, V = (torch.from_numpy(x).bfloat16().cuda() for x in wl.qkv(np.random.default_rng(4), B, S, H, Hkv, d))
    mask = rov.dropout_mask_generate(wl.SEED, 96, B, H, S, p)
    kw = dict(p=0.0) if mode == "none" else dict(p=p, mask=mask if mode == "mask" else None, seed=wl.SEED, offset=96)
    ref = rov.attention_fwd_dropout(Q, K, V, causal=causal, **kw)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [torch.full_like(Q, 7.0) for _ in range(24)]
    torch.cuda.synchronize()
    for i, O in enumerate(outs):
        rov.attention_fwd_dropout(Q, K, V, causal=causal, O=O, stream=streams[i % 3], **kw)
    torch.cuda.synchronize()
    assert all(torch.equal(O, ref) for O in outs)
