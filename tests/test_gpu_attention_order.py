"""Causal attention in the orders of its workgroups: every query block is computed once, whatever the order.

Problems with 1.1 to 2.6 workgroups a compute unit (d = 64: the first round of workgroups comes in reversed order there, but for the last one in two
modes: more than two a compute unit, under 1000 tokens), heads that are
and are not a multiple of eight, workgroups that are no multiple of eight.  A range of rows has fewer workgroups, in the other order: the rows
put together agree bit for bit; and the first group of heads agrees with float64 (bar 2e-2 of the scale, that of every bf16 attention test).
"""
import numpy as np
import pytest
import torch

from oracle import dense as OD
from oracle import philox as OP
from paper_2410_07531_amd import binding as rov
from paper_2410_07531_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["none", "mask", "fused"])
@pytest.mark.parametrize("B,S,H,Hkv", [(2, 427, 32, 8), (1, 1495, 12, 4), (3, 700, 9, 3), (2, 1250, 16, 4), (2, 613, 32, 8)])
def test_every_block_once(B, S, H, Hkv, mode):
    d, p, seed, offset = 64, 0.1, wl.SEED, 640
    ks = rov.attention_key_parts(B, H, S, d, rov.BF16, True)
    n = -(-S // (256 // ks)) * B * H
    print("attn order", B, S, H, mode, n, flush=True)
    assert 282 <= n <= 665
    q, k, v = wl.qkv(np.random.default_rng(S), B, S, H, Hkv, d)
    Q, K, V = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (q, k, v))
    pr = 0.0 if mode == "none" else p
    mask = rov.dropout_mask_generate(seed, offset, B, H, S, p) if mode == "mask" else None
    O = rov.attention_fwd_dropout(Q, K, V, pr, mask=mask, seed=seed, offset=offset, causal=True, O=torch.full_like(Q, 7.0))
    R = torch.full_like(Q, 7.0)
    step = 256
    for q0 in range(0, S, step):
        part = rov.dropout_mask_generate_rows(seed, offset, B, H, S, p, q0, step) if mode == "mask" else None
        rov.attention_fwd_dropout_rows(Q, K, V, pr, q0, step, R, mask_rows=part, seed=seed, offset=offset, causal=True)
    torch.cuda.synchronize()
    assert torch.equal(O, R)
    group = H // Hkv
    keep = None if mode == "none" else OP.unpack_keep(OP.dropout_mask(seed, offset, 1, group, S, p), S)
    f64 = [x.float().cpu().numpy().astype(np.float64) for x in (Q[:1, :, :group], K[:1, :, :1], V[:1, :, :1])]
    ref = OD.attention_dropout(*f64, keep, pr, causal=True)
    got = O[:1, :, :group].float().cpu().numpy().astype(np.float64)
    assert float(np.max(np.abs(got - ref)) / np.max(np.abs(ref))) <= 2e-2
