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


@pytest.mark.parametrize("ctx", [100, 4096])  # one workgroup per head, several
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_mam_of_non_finite_keys_is_nan(ctx, bad):
    """A key that makes a logit NaN or infinite makes its head's mass NaN, in no other head."""
    say(f"\n[gpu] mam non-finite ctx={ctx} {bad}")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(ctx)
    pool, table, ctx_len, n, mb = _paged([ctx, ctx], 2, 16, torch.bfloat16, gen)
    q = torch.rand((2, 8, D), generator=gen, device=DEV).add(0.5).bfloat16()
    pool[table[1, 3].long(), 0, 1, 5 * D:6 * D] = bad  # request 1, head 1, token 5 of block 3
    sh = P.make_shape(8, 2, D, 16, P.PULSE_BF16)
    out = torch.zeros((2, 2), device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    nb = P.pulse_mam_workspace_bytes(sh, 2, mb)
    ws = torch.zeros(nb, dtype=torch.uint8, device=DEV)
    P.pulse_mam(sh, q, pool, pool.shape[0], table, mb, ctx_len, 2, 1, 2, D ** -0.5, out, st, ws, nb)
    assert st.item() == 0
    assert out.isnan().cpu().tolist() == [[False, False], [False, True]]


# Whole parts of a context whose every logit is NaN: the last workgroup's only token, a wave's blocks, a
# workgroup's, several workgroups' (those that a thread of the merge starts with), everything; first and last.
@pytest.mark.parametrize("ctx,lo,hi", [(257, 256, 257), (257, 0, 64), (257, 0, 256), (200, 0, 64), (4096, 0, 64),
                                       (4096, 0, 256), (4096, 3840, 4096), (16384, 0, 8192), (300, 0, 300)])
@pytest.mark.parametrize("what", ["key", "query"])
def test_mam_nan_parts(ctx, lo, hi, what):
    """A NaN logit makes its head's mass NaN wherever in the merge it stands, in no other head or request."""
    say(f"\n[gpu] mam NaN {what} ctx={ctx} {lo}..{hi}")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(ctx + lo)
    pool, table, ctx_len, n, mb = _paged([ctx, ctx], 2, 16, torch.bfloat16, gen)
    q = torch.randn((2, 8, D), generator=gen, device=DEV, dtype=torch.bfloat16)
    sh = P.make_shape(8, 2, D, 16, P.PULSE_BF16)
    if what == "key":  # tokens lo..hi of request 1, head 1
        for t in range(lo, hi):
            pool[table[1, t // 16].long(), 0, 1, (t % 16) * D] = float("nan")
    else:
        q[1, 6, 5] = float("nan")  # a query of head 1: every logit of it
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    nb = P.pulse_mam_workspace_bytes(sh, 2, mb)
    ws = torch.zeros(nb, dtype=torch.uint8, device=DEV)
    for ns, nl in ((1, 2), (n[0], 0)):  # with middle blocks; without any the mass is 0 whatever the logits are
        out = torch.full((2, 2), -1.0, device=DEV)
        P.pulse_mam(sh, q, pool, pool.shape[0], table, mb, ctx_len, 2, ns, nl, D ** -0.5, out, st, ws, nb)
        assert st.item() == 0
        if ns == 1:
            assert out.isnan().cpu().tolist() == [[False, False], [False, True]]
        else:
            assert (out == 0).all()


# Rows of the FFN products per tile count (16, 32, 64 and beyond), hidden sizes below one group of
# K steps, with a last step of 8 elements, and on either side of the two-tile rule (512 column tiles).
FFN_CASES = [(1, 8, 2, 1, 100), (16, 24, 4, 2, 33), (17, 136, 8, 8, 16), (32, 1000, 4, 4, 300), (33, 512, 6, 3, 20),
             (70, 264, 2, 2, 5), (5, 8184, 2, 1, 40), (31, 8192 + 8, 4, 1, 64)]


@pytest.mark.parametrize("B,F,hq,hkv,ctx", FFN_CASES)
def test_normal_layer_edges(B, F, hq, hkv, ctx):
    from paper_2609_34555_amd.harness import NormalBatch
    from paper_2609_34555_amd import workloads as W
    from parity import build

    say(f"\n[gpu] normal layer B={B} F={F} hq={hq} hkv={hkv} ctx={ctx}")
    spec, seed = W.custom("light", [200], Hq=4, Hkv=2, bs=16, k_mid=2)
    w, st = build(spec, seed)
    st.reset()
    normal = NormalBatch(B=B, ctx=ctx, n_layers=1, Hq=hq, Hkv=hkv, d_ff=F, seed=B + F)
    cmp_, io = torch.cuda.Stream(), torch.cuda.Stream()
    sched = P.IrqScheduler(cmp_, io)
    torch.cuda.synchronize()
    stats, _ = sched.step([st.layer_args()], normal.layers, mode="blocking")
    torch.cuda.synchronize()
    assert stats["normal_layers"] == 1 and normal.status() == 0 and st.status() == 0
    b = normal.bufs[0]
    x, wgu, wd = (b[k].double().cpu() for k in ("x", "w_gu", "w_down"))
    assert torch.equal(b["x"].view(B, hq, 128), b["out"].bfloat16())

    def close(got, want, mass, what):
        # one rounding to bf16 (8 significant bits: half a unit in the last place is at most 2^-8 of the
        # value), and fp32 sums of products of total size `mass`
        err = (got.double().cpu() - want).abs() - (2.0 ** -8 * want.abs() + 2.0 ** -20 * mass)
        say(f"  {what}: worst excess {err.max().item():.1e}")
        assert err.max().item() <= 0, what

    close(b["gu"], x @ wgu.T, x.abs() @ wgu.abs().T, "gu")
    g, u = b["gu"].double().cpu()[:, :F], b["gu"].double().cpu()[:, F:]
    close(b["h"], g * torch.sigmoid(g) * u, (g * u).abs(), "h")
    h = b["h"].double().cpu()
    close(b["y"], h @ wd.T, h.abs() @ wd.abs().T, "y")
    sched.destroy()


@pytest.mark.parametrize("ctx", [40, 900])  # one workgroup per head (it writes the output), several and a merge
@pytest.mark.parametrize("how", ["h on x", "h past x", "x in ws", "x on q", "x past q", "x on lse"])
def test_normal_layer_shared_buffers(ctx, how):
    """A layer whose x or h lies in memory that is read before it is written gives what separate buffers give."""
    from paper_2609_34555_amd.harness import NormalBatch
    from paper_2609_34555_amd import workloads as W
    from parity import build

    say(f"\n[gpu] normal layer ctx={ctx} {how}")
    spec, seed = W.custom("light", [200], Hq=4, Hkv=2, bs=16, k_mid=2)
    w, st = build(spec, seed)
    B, hq, F = 6, 8, 1032
    normal = NormalBatch(B=B, ctx=ctx, n_layers=1, Hq=hq, Hkv=2, d_ff=F, seed=3)
    b, layer = normal.bufs[0], normal.layers[0]
    nx, nh, nq = 2 * B * hq * D, 2 * B * F, 2 * B * hq * D
    cmp_, io = torch.cuda.Stream(), torch.cuda.Stream()
    sched = P.IrqScheduler(cmp_, io)

    def step():
        st.reset()
        torch.cuda.synchronize()
        sched.step([st.layer_args()], normal.layers, mode="blocking")
        torch.cuda.synchronize()
        assert normal.status() == 0 and st.status() == 0

    step()
    want = {k: b[k].clone() for k in ("out", "gu", "h", "y", "x")}
    mem = torch.full((nx + nh + nq + normal.ws_bytes + 4096,), 255, dtype=torch.uint8, device=DEV)
    q = b["q"].view(torch.uint8).view(-1)
    if how[0] == "h":
        layer.x, layer.h = mem.data_ptr(), mem.data_ptr() + (0 if how == "h on x" else nx // 2)
    elif how == "x in ws":
        layer.ws, layer.x = mem.data_ptr(), mem.data_ptr() + 1024
        assert nx + 1024 < normal.ws_bytes
    elif how == "x on lse":
        layer.lse = layer.x = mem.data_ptr()
    else:
        mem[:nq] = q
        layer.q, layer.x = mem.data_ptr(), mem.data_ptr() + (0 if how == "x on q" else nq // 2)
    step()
    for k in ("out", "gu", "y"):
        assert torch.equal(b[k], want[k]), k
    at = (layer.x if how[0] == "x" else layer.h) - mem.data_ptr()
    last = want["x" if how[0] == "x" else "h"]
    assert torch.equal(mem[at:at + 2 * last.numel()].view(torch.bfloat16), last.view(-1))
    sched.destroy()


# Selected blocks per request around the shares of the split plan: equal, one long request among short and
# empty ones, the plan's limit of 64 requests and one past it, many heads per KV head (4-wave workgroups).
PLAN_CASES = [
    ([128] * 4, 8, 2, 16, "bf16"), ([300, 0, 1, 2, 5], 8, 2, 16, "bf16"), ([0, 0, 0, 260], 4, 1, 16, "f16"),
    ([1, 97, 98, 99, 513], 32, 8, 16, "bf16"), ([40] * 63 + [200], 2, 1, 16, "f16"),
    ([40] * 64 + [200], 2, 1, 16, "bf16"), ([7, 150, 33], 32, 2, 32, "bf16"), ([3, 260, 0, 31], 12, 1, 64, "f16"),
    ([0, 0], 4, 2, 16, "bf16"), ([9] * 40 + [800], 8, 8, 32, "bf16"),
    # more than one round of workgroups whose last ones are light: equal counts, a host's split of one round and of
    # more, no room for a plan of one round, more heads than a round has workgroups, 4-wave workgroups
    ([129] * 12, 16, 8, 16, "bf16"), ([129] * 11 + [40], 16, 8, 16, "bf16"), ([129, 10, 3, 129] * 3, 16, 8, 16, "f16"),
    ([60] * 31 + [250], 8, 8, 16, "bf16"), ([600, 5], 257, 257, 16, "f16"), ([300, 20, 77, 0, 150], 48, 4, 16, "bf16"),
    ([700, 3, 41, 260, 0], 8, 8, 32, "bf16"), ([37, 1, 0, 12, 5, 9, 36], 8, 8, 64, "bf16"),
    ([2900, 17, 1400], 8, 1, 16, "f16"),
]


@pytest.mark.parametrize("cnt,hq,hkv,bs,dt", PLAN_CASES)
def test_attention_split_plan(cnt, hq, hkv, bs, dt):
    say(f"\n[gpu] split plan cnt={cnt[:5]}.. hq={hq} hkv={hkv} bs={bs}")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(sum(cnt) + bs + hq)
    dtype = torch.bfloat16 if dt == "bf16" else torch.float16
    B, G, k_max = len(cnt), hq // hkv, max(1, max(cnt))
    ctx = [(c + 3) * bs - (r % bs) for r, c in enumerate(cnt)]  # the last block is partial
    pool, table, ctx_len, n, mb = _paged(ctx, hkv, bs, dtype, gen)
    q = torch.randn((B, hq, D), generator=gen, device=DEV, dtype=dtype)
    sel = torch.full((B, k_max), -1, dtype=torch.int32, device=DEV)
    for r, c in enumerate(cnt):  # the last c blocks
        sel[r, :c] = torch.arange(n[r] - c, n[r], dtype=torch.int32, device=DEV)
    sel_cnt = torch.tensor(cnt, dtype=torch.int32, device=DEV)
    sh = P.make_shape(hq, hkv, D, bs, P.PULSE_BF16 if dt == "bf16" else P.PULSE_F16)
    nb = P.pulse_workspace_bytes(sh, B, k_max, 0)
    ws = torch.full((nb,), 255, dtype=torch.uint8, device=DEV)  # NaN patterns: every partial read was written
    out = torch.full((B, hq, D), float("nan"), device=DEV)
    lse = torch.full((B, hq), float("nan"), device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    P.pulse_sparse_decode_attn(sh, q, pool, pool.shape[0], table, mb, sel, sel_cnt, k_max, ctx_len, B, D ** -0.5, out,
                               lse, st, ws, nb)
    assert st.item() == 0
    for r, c in enumerate(cnt):
        if c == 0:
            assert (out[r] == 0).all() and (lse[r] == -math.inf).all()
            continue
        b = pool[table[r, n[r] - c: n[r]].long()]
        ok = torch.arange((n[r] - c) * bs, n[r] * bs, device=DEV) < ctx[r]
        for h in range(hkv):
            K = b[:, 0, h].reshape(-1, D)[ok].double()
            V = b[:, 1, h].view(-1, D, bs).transpose(1, 2).reshape(-1, D)[ok].double()
            s = q[r, h * G:(h + 1) * G].double() @ K.T / math.sqrt(D)
            # probabilities in two 16-bit parts (2^-16) and fp32 sums: 2^-14 of the values' size is well above both
            assert (out[r, h * G:(h + 1) * G] - torch.softmax(s, 1) @ V).abs().max() < 2.0 ** -14 * 5, (r, h)
            assert (lse[r, h * G:(h + 1) * G] - torch.logsumexp(s, 1)).abs().max() < 1e-5, (r, h)


@pytest.mark.parametrize("hkv", [1, 8, 257])
def test_average_of_no_blocks(hkv):
    """Requests without blocks select nothing, whatever the head count."""
    say(f"\n[gpu] average of no blocks hkv={hkv}")
    i32 = dict(dtype=torch.int32, device=DEV)
    sel, cnt, st = torch.full((2, 4), -7, **i32), torch.full((2,), 9, **i32), torch.zeros(1, **i32)
    pad = torch.zeros((2, hkv, D), dtype=torch.bfloat16, device=DEV)
    sh = P.make_shape(hkv, hkv, D, 16, P.PULSE_BF16)
    P.pulse_select_average(sh, pad, pad, torch.zeros(3, dtype=torch.int64, device=DEV), 2, 0, torch.ones(2, **i32), 1, 1,
                           4, sel, cnt, None, st, torch.zeros(256, dtype=torch.uint8, device=DEV), 256)
    assert st.item() == 0 and (cnt == 0).all() and (sel == -1).all()


# Average scores: one head, head counts that divide a workgroup's 16 pairs and that do not, more than 16
# heads, ragged and empty requests, and more digests than the one-launch limit (65536).
AVG_EDGES = [([300, 0, 17], 8, 1, "bf16"), ([700, 31, 0, 0, 650], 6, 3, "f16"), ([900, 2000], 32, 8, "bf16"),
             ([1, 16, 4000], 20, 5, "bf16"), ([500, 900], 34, 17, "f16"), ([131072, 7000], 32, 8, "bf16")]


@pytest.mark.parametrize("ctx,hq,hkv,dt", AVG_EDGES)
def test_average_scores_edges(ctx, hq, hkv, dt):
    say(f"\n[gpu] average ctx={ctx} hq={hq} hkv={hkv}")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(sum(ctx) + hq)
    dtype = torch.bfloat16 if dt == "bf16" else torch.float16
    B, G, bs, ns, nl = len(ctx), hq // hkv, 16, 1, 2
    n = [-(-x // bs) for x in ctx]
    off = [0]
    for k in n:
        off.append(off[-1] + k)
    total = off[-1]
    a = torch.randn((2, hkv, total, D), generator=gen, device=DEV, dtype=dtype)
    dig = torch.stack([a.amin(0), a.amax(0)], 2).contiguous()  # [hkv][total][2][128]
    q = torch.randn((B, hq, D), generator=gen, device=DEV, dtype=dtype)
    blk_off = torch.tensor(off, dtype=torch.int64, device=DEV)
    k_mid = torch.full((B,), 5, dtype=torch.int32, device=DEV)
    sel = torch.full((B, 8), -7, dtype=torch.int32, device=DEV)
    cnt = torch.zeros(B, dtype=torch.int32, device=DEV)
    scores = torch.full((total,), 1e9, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    sh = P.make_shape(hq, hkv, D, bs, P.PULSE_BF16 if dt == "bf16" else P.PULSE_F16)
    nb = P.pulse_average_workspace_bytes(sh, B, 8, total)
    ws = torch.full((nb,), 255, dtype=torch.uint8, device=DEV)
    P.pulse_select_average(sh, q, dig, blk_off, B, total, k_mid, ns, nl, 8, sel, cnt, scores, st, ws, nb)
    assert st.item() == 0
    for r in range(B):
        lo, hi = min(ns, n[r]), max(min(ns, n[r]), n[r] - nl)
        b0 = off[r]
        got = scores[b0:b0 + n[r]]
        assert (got[:lo] == 1e9).all() and (got[hi:] == 1e9).all()  # forced blocks are left as they are
        if hi <= lo:
            continue
        want = torch.zeros(hi - lo, dtype=torch.float64, device=DEV)
        mass = torch.zeros_like(want)
        for h in range(hkv):
            mn, mx = dig[h, b0 + lo:b0 + hi, 0].double(), dig[h, b0 + lo:b0 + hi, 1].double()
            for g in range(G):
                qq = q[r, h * G + g].double()
                want += mx @ qq.clamp(min=0) + mn @ qq.clamp(max=0)
                mass += torch.maximum(mx.abs(), mn.abs()) @ qq.abs()
        # fp32 sums of at most 128 G + Hkv terms: each within 2^-24 of a running sum no larger than the mass
        err = (got[lo:hi].double() * G * hkv - want).abs() - 2.0 ** -24 * (128 * G / 16 + 8 + hkv) * mass
        assert err.max().item() <= 0
        k = min(5, hi - lo)
        top = torch.sort(got[lo:hi], descending=True, stable=True).indices[:k] + lo
        ids = torch.cat([torch.arange(lo, device=DEV), top, torch.arange(hi, n[r], device=DEV)]).sort().values
        assert cnt[r].item() == len(ids) and torch.equal(sel[r, : len(ids)].long(), ids)


# Block counts around the one-wave selection (up to 512 blocks), its 64-block rounds and the general path, with
# every budget from none to all and blocks that are copies of one another (ties go to the lowest index).
@pytest.mark.parametrize("n", [[1, 2, 63, 64], [65, 127, 128, 0], [511, 512, 513, 3], [512] * 3, [200] * 4, [700, 40]])
@pytest.mark.parametrize("copies", [0, 1])
def test_select_block_counts(n, copies):
    say(f"\n[gpu] select n={n} copies={copies}")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(sum(n) + copies)
    B, total, ns, nl, G = len(n), sum(n), 1, 2, 4
    off = [0]
    for k in n:
        off.append(off[-1] + k)
    a = torch.randn((2, total, D), generator=gen, device=DEV, dtype=torch.bfloat16)
    if copies:  # few distinct blocks
        a = a[:, torch.randint(0, max(1, total // 16), (total,), generator=gen, device=DEV)]
    dig = torch.stack([a.amin(0), a.amax(0)], 1).contiguous()
    q = torch.randn((B, G, D), generator=gen, device=DEV, dtype=torch.bfloat16)
    blk_off = torch.tensor(off, dtype=torch.int64, device=DEV)
    sh = P.make_shape(G, 1, D, 16, P.PULSE_BF16)
    k_max = max(n)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    nb = P.pulse_workspace_bytes(sh, B, k_max, total)
    ws = torch.zeros(nb, dtype=torch.uint8, device=DEV)
    for share in (0.0, 0.02, 0.3, 0.97, 1.0):
        k_mid = torch.tensor([int(share * x) for x in n], dtype=torch.int32, device=DEV)
        sel = torch.full((B, k_max), -7, dtype=torch.int32, device=DEV)
        cnt = torch.full((B,), -7, dtype=torch.int32, device=DEV)
        scores = torch.zeros(total, device=DEV)
        P.pulse_select_solohead(sh, q, dig, blk_off, B, total, 0, k_mid, ns, nl, k_max, sel, cnt, scores, st, ws, nb)
        assert st.item() == 0
        for r in range(B):
            lo, hi = min(ns, n[r]), max(min(ns, n[r]), n[r] - nl)
            k = min(int(share * n[r]), hi - lo)
            s = scores[off[r] + lo: off[r] + hi]
            top = torch.sort(s, descending=True, stable=True).indices[:k] + lo
            ids = torch.cat([torch.arange(lo, device=DEV), top, torch.arange(hi, n[r], device=DEV)]).sort().values
            assert cnt[r].item() == len(ids), (share, r)
            assert torch.equal(sel[r, : len(ids)].long(), ids) and (sel[r, len(ids):] == -1).all(), (share, r)


# The plan beside the selection: runs of missing blocks across the one-wave path's 64-block rounds, the general
# path's waves (64), rounds (1024) and tiles (8192), on either side of the 512 blocks where the paths part.
@pytest.mark.parametrize("n", [[63, 64, 65], [127, 128, 129, 0, 1], [510, 511, 512], [513, 512, 514], [1023, 1025, 2050],
                               [8191, 8193], [8193, 300, 9000]])
@pytest.mark.parametrize("share", [1.0, 0.4])
def test_select_plan_counts(n, share):
    say(f"\n[gpu] select plan n={n} share={share}")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(sum(n))
    B, H, total, ns, nl, G, n_slots = len(n), 2, sum(n), 1, 2, 4, 1000
    off = [0]
    for k in n:
        off.append(off[-1] + k)
    a = torch.randn((2, H * total, D), generator=gen, device=DEV, dtype=torch.bfloat16)
    dig = torch.stack([a.amin(0), a.amax(0)], 1).contiguous()
    q = torch.randn((B, H * G, D), generator=gen, device=DEV, dtype=torch.bfloat16)
    i32 = dict(dtype=torch.int32, device=DEV)
    blk_off = torch.tensor(off, dtype=torch.int64, device=DEV)
    mb, k_max = max(n), max(n)
    table = torch.randint(0, n_slots, (B, mb), generator=gen, **i32)
    for at in range(0, mb, 64):  # missing around every 64th block, and a long run over several rounds
        table[:, max(0, at - 3):at + at // 64 % 5] = -1
    table[:, 300:480] = -1
    table[:, 1000:1300] = -1
    sh = P.make_shape(H * G, H, D, 16, P.PULSE_BF16)
    nb = P.pulse_headwise_workspace_bytes(sh, B, k_max, total)
    ws = torch.zeros(nb, dtype=torch.uint8, device=DEV)

    def select(k_mid, k_max, table):
        sel, cnt = torch.full((H, B, k_max), -7, **i32), torch.full((H, B), -7, **i32)
        miss, run, st = torch.full((H, B), -7, **i32), torch.full((H, B), -7, **i32), torch.zeros(1, **i32)
        P.pulse_select_headwise(sh, q, dig, blk_off, B, total, torch.tensor(k_mid, **i32), ns, nl, k_max, table, mb,
                                n_slots, sel, cnt, miss, run, st, ws, nb)
        return sel.cpu(), cnt.cpu(), miss.cpu(), run.cpu(), st.item()

    k_mid = [int(share * x) for x in n]
    sel, cnt, miss, run, st = select(k_mid, k_max, table)
    assert st == 0
    tab = table.cpu()
    for h in range(H):
        for r in range(B):
            forced = len(set(range(min(ns, n[r]))) | set(range(max(0, n[r] - nl), n[r])))
            c = forced + min(k_mid[r], n[r] - forced)
            assert cnt[h, r] == c and (sel[h, r, c:] == -1).all()
            ids = sel[h, r, :c].long()
            m = ids[tab[r, ids] < 0]
            assert miss[h, r] == len(m), (h, r)
            assert run[h, r] == int((m[1:] != m[:-1] + 1).sum()) + (len(m) > 0), (h, r)
    # a selected entry past the pool is reported, an unselected one is not
    bad = table.clone()
    big = max(range(B), key=lambda r: n[r])
    bad[big, n[big] - 1] = n_slots  # a local block
    assert select(k_mid, k_max, bad)[4] == P.PULSE_ERR_BAD_INDEX
    bad = table.clone()
    bad[big, n[big] // 2] = n_slots
    assert select([0] * B, k_max, bad)[4] == 0
    # one block too many: that request (and any other of its count) is empty, the rest are as they were
    limit = int(cnt[0, big]) - 1
    full = (sel, cnt, miss, run)
    sel, cnt, miss, run, st = select(k_mid, limit, table)
    assert st == P.PULSE_ERR_SELECT_OVERFLOW
    for r in range(B):
        if full[1][0, r] > limit:
            assert (cnt[:, r] == 0).all() and (sel[:, r] == -1).all() and (miss[:, r] == 0).all() and (run[:, r] == 0).all()
        else:
            assert torch.equal(sel[:, r], full[0][:, r, :limit])
            assert all(torch.equal(a[:, r], b[:, r]) for a, b in zip((cnt, miss, run), full[1:]))


# The layer-step on requests past the one-wave selection: lengths for which the loads at equal-length offsets
# are right for requests 0 and 3 and wrong for 1 and 2, then lengths on both sides of 512 blocks and of a tile.
@pytest.mark.parametrize("n", [[800, 1120, 480, 800], [600, 500, 513, 512], [8300, 700, 100]])
@pytest.mark.parametrize("fault", ["none", "overflow", "entry past pool"])
def test_chained_layer_longer_requests(n, fault):
    from oracle import pulse_oracle as O
    from paper_2609_34555_amd import workloads as W
    from parity import (assert_attention_close, assert_recall_equal, assert_selection_ok, build, full_check,
                        oracle_attention, oracle_recall, oracle_selection)
    import numpy as np

    say(f"\n[gpu] chained n={n} {fault}")
    spec, seed = W.custom("longer", [16 * x - r for r, x in enumerate(n)], Hq=4, Hkv=1, bs=16, dtype="bf16",
                          k_mid=[20, 40, 9, 50][:len(n)], n_sink=1, n_local=8, resident_frac=0.1, heavy_per_req=6)
    w, st = build(spec, seed, k_max=48 if fault == "overflow" else None)
    if fault == "none":
        full_check(w, st, chained=True)
        return
    st.reset()
    table0 = w.table0.copy()
    if fault == "entry past pool":
        table0[0, n[0] - 1] = w.n_slots  # a local block, always selected
        st.table.copy_(torch.from_numpy(table0))
    st.decode_layer()
    torch.cuda.synchronize()
    code, ocode = ((P.PULSE_ERR_SELECT_OVERFLOW, O.ERR_SELECT_OVERFLOW) if fault == "overflow"
                   else (P.PULSE_ERR_BAD_INDEX, O.ERR_BAD_INDEX))
    assert st.status() == code
    gidx, gcnt = st.selection()
    dig = st.digests.cpu().numpy().view(np.uint16)[: w.total_blocks]
    rc, oidx, ocnt, osc = oracle_selection(w, dig, k_max=st.k_max)
    assert_selection_ok(w, gidx, gcnt, oidx, ocnt, osc)
    rr, table, pool, fh, stats = oracle_recall(w, gidx, gcnt, table0=table0)
    assert (rc if fault == "overflow" else rr) == ocode
    assert_recall_equal(st, table, pool, fh, stats)
    if fault == "overflow":
        assert gcnt[1] == 0 and stats[0] > 0
        assert_attention_close(st, *oracle_attention(w, pool, table, gidx, gcnt))


def test_irq_blocking_step_follows_io_stream_work():
    """The blocking step's recalls read what the I/O stream's earlier work wrote to the host store."""
    from paper_2609_34555_amd import workloads as W
    from parity import build
    import numpy as np

    say("\n[gpu] blocking step behind I/O stream work")
    spec, seed = W.custom("behind", [640], Hq=4, Hkv=2, bs=16, k_mid=6)
    w, st = build(spec, seed)
    st.reset()
    cmp_, io = torch.cuda.Stream(), torch.cuda.Stream()
    sched = P.IrqScheduler(cmp_, io)
    host = torch.from_numpy(w.kv.view(np.int16))
    new = torch.full_like(host, 0x3C00, device=DEV)  # every key and value the same
    a = torch.randn((4096, 4096), device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.stream(io):
        for _ in range(20):  # some milliseconds of work ahead of the store's update
            a = (a @ a).clamp(-1, 1)
        host.copy_(new, non_blocking=True)
    assert not io.query()
    sched.step([st.layer_args()], [], mode="blocking")
    torch.cuda.synchronize()
    assert st.status() == 0 and st.recall_stats()[0] > 0
    table = st.table_np()[0]
    slots = [int(table[j]) for j in range(w.max_blocks) if table[j] >= 0 and w.table0[0, j] < 0]
    assert len(slots) == st.recall_stats()[0]
    assert (st.pool_np()[slots] == 0x3C00).all()
    sched.destroy()
