"""Kernels at the edges of their tiles and of their dispatch rules, against plain 64-bit torch."""
import math

import pytest
import torch

from paper_2609_34555_amd import pulse as P

from parity import say

pytestmark = pytest.mark.gpu
D = 128
DEV = "cuda"


def _paged(ctx, hkv, bs, dtype, gen):
    """Random resident KV: (pool [slots][2][hkv][bs*128], table, ctx_len, total blocks), slots shuffled."""
    n = [-(-x // bs) for x in ctx]
    total, mb = max(1, sum(n)), max(1, max(n))
    pool = torch.randn((total, 2, hkv, bs * D), generator=gen, device=DEV, dtype=dtype)
    slots = torch.randperm(total, generator=gen, device=DEV).int()
    table = torch.full((len(ctx), mb), -1, dtype=torch.int32, device=DEV)
    o = 0
    for r, k in enumerate(n):
        table[r, :k] = slots[o:o + k]
        o += k
    return pool, table, torch.tensor(ctx, dtype=torch.int32, device=DEV), n, mb


MAM_CASES = [
    # contexts, hq, hkv, bs, dtype, sink, local: one workgroup per head; a partial block and an empty request;
    # several workgroups whose last holds one token; 64 blocks per wave and many heads; G = 16
    ([1, 31, 33], 8, 2, 16, "bf16", 1, 2),
    ([0, 255, 256, 257], 4, 4, 16, "f16", 0, 0),
    ([16 * 256 * 3 + 1, 5], 4, 1, 16, "bf16", 1, 8),
    ([2048 * 32, 2047 * 32 + 1], 16, 1, 32, "bf16", 1, 4),
    ([64 * 64 * 4 + 63] * 9, 64, 64, 64, "f16", 2, 3),
    ([70, 4096], 8, 8, 64, "bf16", 3, 100),
]


@pytest.mark.parametrize("ctx,hq,hkv,bs,dt,ns,nl", MAM_CASES)
def test_mam_edges(ctx, hq, hkv, bs, dt, ns, nl):
    say(f"\n[gpu] mam ctx={ctx[:3]} hq={hq} hkv={hkv} bs={bs}")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(sum(ctx) + bs)
    dtype = torch.bfloat16 if dt == "bf16" else torch.float16
    pool, table, ctx_len, n, mb = _paged(ctx, hkv, bs, dtype, gen)
    B, G = len(ctx), hq // hkv
    q = 2 * torch.randn((B, hq, D), generator=gen, device=DEV, dtype=dtype)
    sh = P.make_shape(hq, hkv, D, bs, P.PULSE_BF16 if dt == "bf16" else P.PULSE_F16)
    out = torch.full((B, hkv), -1.0, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    nb = P.pulse_mam_workspace_bytes(sh, B, mb)
    ws = torch.full((nb,), 255, dtype=torch.uint8, device=DEV)  # NaN patterns: every partial read must have been written
    P.pulse_mam(sh, q, pool, pool.shape[0], table, mb, ctx_len, B, ns, nl, D ** -0.5, out, st, ws, nb)
    want = torch.zeros((B, hkv), dtype=torch.float64)
    for r in range(B):
        if not ctx[r]:
            continue
        b = pool[table[r, : n[r]].long()]
        t0, t1 = ns * bs, min(ctx[r], max(n[r] - nl, 0) * bs)
        for h in range(hkv):
            K = b[:, 0, h].reshape(-1, D)[: ctx[r]].double()
            p = torch.softmax(q[r, h * G:(h + 1) * G].double() @ K.T / math.sqrt(D), 1)
            want[r, h] = p[:, t0:max(t0, t1)].sum(1).mean()
    assert st.item() == 0
    # logits to about 128 * 2^-24 * |logit|, sums over a lane's tokens and the merges: below 1e-5 of a value in [0, 1]
    err = (out.double().cpu() - want).abs().max().item()
    say(f"  max err {err:.1e}")
    assert err < 1e-5
