"""GPU parity of softmax_prefix_step (exact softmax over a KV cache plus the
block) against the fp64 oracle, and its reduction to the hybrid step."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_06628_amd import binding as hb
from paper_2608_06628_amd import synth
from _helpers import act, announce, assert_close, check_outputs, f32, host, i32

pytestmark = pytest.mark.gpu

CASES = [
    # (B, Hq, Hkv, d, L, dtype, Pmax, plens)
    (1, 1, 1, 64, 8, "f32", 32, [32]),
    (2, 4, 2, 64, 8, "f32", 100, [100, 0]),
    (3, 8, 2, 128, 32, "f32", 300, [300, 17, 64]),
    (2, 16, 4, 128, 32, "bf16", 4096, [4096, 1000]),
    (3, 4, 4, 128, 16, "bf16", 777, [0, 777, 5]),
    (2, 8, 1, 64, 32, "bf16", 2048, [2048, 1536]),
    (2, 4, 2, 128, 7, "bf16", 96, [96, 200]),   # prefix_len above max is clamped
    # the copy-ring kernel at d=64 with 4 heads per KV head, and at d=128 with 8;
    # 3 heads per KV head take the register-staged kernel
    (2, 8, 2, 64, 16, "bf16", 500, [500, 260]),
    (1, 8, 1, 128, 32, "bf16", 5000, [4900]),
    (2, 6, 2, 64, 32, "bf16", 1000, [1000, 33]),
]


@pytest.mark.parametrize("case", CASES, ids=lambda s: "x".join(map(str, s[:7])))
def test_softmax_prefix(case):
    B, Hq, Hkv, d, L, dt, Pmax, plens = case
    dims = synth.Dims(B=B, Hq=Hq, Hkv=Hkv, d=d, L=L, F=32, dtype=dt)
    announce(f"softmax_prefix {case}")
    q, k, v = synth.block_qkv(dims, 71, 1.0)
    kc, vc = synth.prefix_kv(B, Pmax, Hkv, d, 72, 1.0, dt)
    pl = np.array(plens, np.int32)
    args = (act(q, dt), act(k, dt), act(v, dt), act(kc, dt), act(vc, dt), i32(pl))
    ref = oracle.softmax_prefix(q, k, v, kc, vc, np.minimum(pl, Pmax))
    check_outputs(lambda o32: hb.softmax_prefix_step(*args, out_f32=o32), ref, dt,
                  f"softmax_prefix {case[:7]}")


def test_no_prefix_equals_hybrid_with_empty_state():
    dims = synth.Dims(B=2, Hq=16, Hkv=4, d=128, L=32, F=64, dtype="bf16")
    announce("softmax_prefix P=0 vs hybrid empty state")
    q, k, v = synth.block_qkv(dims, 81, 1.0)
    Wt, alpha = synth.feature_weights(dims, 82, 83)
    qd, kd, vd = act(q, "bf16"), act(k, "bf16"), act(v, "bf16")
    kc = torch.zeros((2, 0, 4, 128), dtype=torch.bfloat16, device="cuda")
    S = torch.zeros((2, 16, 128, 128), device="cuda")
    z = torch.zeros((2, 16, 128), device="cuda")
    ref = oracle.softmax_prefix(q, k, v, np.zeros((2, 0, 4, 128)), np.zeros((2, 0, 4, 128)),
                                np.zeros(2, np.int32))
    check_outputs(lambda o32: hb.softmax_prefix_step(qd, kd, vd, kc, kc, i32([0, 0]),
                                                     out_f32=o32), ref, "bf16", "softmax P=0")
    check_outputs(lambda o32: hb.hybrid_attn_step(qd, kd, vd, act(Wt, "bf16"), f32(alpha), S, z,
                                                  out_f32=o32), ref, "bf16", "hybrid empty state")


RANGES = [
    # lengths far apart, in calls small enough that the host cuts every request
    # into ranges of the same number of whole tiles;
    # (B, Hq, Hkv, d, L, dtype, Pmax, lengths or a seed)
    (5, 8, 2, 128, 32, "bf16", 6016, [6016, 0, 31, 3000, 4097]),    # 4 heads per KV head
    (3, 2, 2, 64, 9, "bf16", 3008, [3008, 1, 1600]),                # one wave per workgroup
    (3, 4, 2, 128, 1, "bf16", 2080, [65, 2080, 1024]),
    (2, 8, 1, 128, 32, "bf16", 4096, [4096, 700]),                  # 8 heads per KV head
    (3, 6, 2, 64, 32, "bf16", 2048, [2048, 2017, 5]),               # register-staged kernel
    (3, 4, 2, 64, 5, "f32", 2048, [2048, 1, 1500]),
    # tiles per range around the copy ring's depth and its remainders
    (7, 4, 1, 128, 32, "bf16", 544, [0, 32, 64, 96, 128, 160, 544]),
    # more requests than the plan stages in LDS at once
    (300, 4, 1, 64, 3, "bf16", 1088, 5),
    (2100, 1, 1, 64, 2, "bf16", 544, 6),                            # a range per request at most
    # more ranges than fit one round, so the plan is made from the lengths; in
    # most of these it finds that a range per request is enough (for plans of
    # several see PLANNED)
    (40, 8, 8, 64, 9, "bf16", 544, 7),
    (40, 32, 8, 128, 32, "bf16", 544, 8),
    (20, 64, 8, 64, 32, "bf16", 544, 9),
    # (the same in bf16: BF16_ROWS)
    (40, 24, 8, 64, 32, "f32", 544, 10),
    (40, 8, 8, 64, 5, "f32", 544, 11),
]


@pytest.mark.parametrize("case", RANGES, ids=lambda s: "x".join(map(str, s[:7])))
def test_softmax_prefix_mixed_lengths(case):
    B, Hq, Hkv, d, L, dt, Pmax, plens = case
    dims = synth.Dims(B=B, Hq=Hq, Hkv=Hkv, d=d, L=L, F=32, dtype=dt)
    announce(f"softmax_prefix ranges {case}")
    if isinstance(plens, int):
        plens = np.random.default_rng(plens).integers(0, Pmax + 1, B)
    pl = np.array(plens, np.int32)
    q, k, v = synth.block_qkv(dims, 91, 1.0)
    kc, vc = synth.prefix_kv(B, Pmax, Hkv, d, 92, 1.0, dt)
    kd, vd = act(kc, dt), act(vc, dt)
    args = (act(q, dt), act(k, dt), act(v, dt))
    ref = oracle.softmax_prefix(q, k, v, kc, vc, pl)
    check_outputs(lambda o32: hb.softmax_prefix_step(*args, kd, vd, i32(pl), out_f32=o32), ref, dt,
                  f"softmax_prefix ranges {case[:7]}")
    # the paged cache follows the same plan: the same bits
    pages = (B * Pmax // 32, 32, Hkv, d)
    table = torch.arange(pages[0], dtype=torch.int32, device="cuda").view(B, -1)
    a = hb.softmax_prefix_step(*args, kd, vd, i32(pl), out_f32=True)
    b = hb.softmax_prefix_step_paged(*args, kd.view(pages), vd.view(pages), table, i32(pl),
                                     out_f32=True)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def _weights_error(q, k, v, P, splits):
    """The attention of q [B][L][Hq][d] over k, v [B][N][Hkv][d] in 64 bits, and
    the same with bf16 weights relative to the running maximum, tile by tile of
    32 keys, of `splits` equal cuts of the keys (whole tiles)."""
    B, L, Hq, d = q.shape
    N, Hkv = k.shape[1:3]
    G = Hq // Hkv
    qh = q.double().permute(0, 2, 1, 3).reshape(B, Hkv, G * L, d)
    kh, vh = (x.double().permute(0, 2, 1, 3) for x in (k, v))
    s = torch.matmul(qh, kh.transpose(-1, -2).contiguous()) * (np.log2(np.e) / np.sqrt(d))
    exact = torch.matmul(torch.softmax(s * np.log(2.0), -1), vh)
    cut = -(-(-(-N // splits)) // 32) * 32
    num, den = 0.0, 0.0
    for lo in range(0, N, cut):
        x = s[..., lo:lo + cut]
        run = torch.nn.functional.pad(x, (0, -x.shape[-1] % 32), value=-1e30)
        run = run.unflatten(-1, (-1, 32)).amax(-1).cummax(-1).values
        ref = run.repeat_interleave(32, -1)[..., :x.shape[-1]]
        p = torch.exp2(x - ref).float().to(torch.bfloat16).double() * torch.exp2(ref - s.amax(-1, True))
        num, den = num + torch.matmul(p, vh[:, :, lo:lo + cut]), den + p.sum(-1, True)
    back = lambda x: x.reshape(B, Hq, L, d).permute(0, 2, 1, 3)
    return back(exact), back(num / den)


@pytest.mark.parametrize("B,Hq,Hkv,L,P", [(16, 32, 32, 4, 4096), (32, 48, 16, 4, 4096)],
                         ids=["ring", "staged"])
def test_softmax_prefix_long_ranges_round_no_worse(B, Hq, Hkv, L, P):
    """The rounding of the weights to bf16 costs no more than with the equal
    cuts of the longest prefix into up to 2048 workgroups, however long the
    ranges of a call that needs fewer are."""
    d = 64
    announce(f"softmax_prefix rounding of long ranges {B}x{Hq}x{Hkv}x{P}")
    g = torch.Generator(device="cuda").manual_seed(301)
    rnd = lambda *n: torch.randn(n, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v = rnd(B, L, Hq, d), rnd(B, L, Hkv, d), rnd(B, L, Hkv, d)
    kc, vc = rnd(B, P, Hkv, d), rnd(B, P, Hkv, d)
    out = hb.softmax_prefix_step(q, k, v, kc, vc, i32([P] * B), out_f32=True)
    splits = max(1, min(-(-2048 // (B * Hkv)), -(-(P + L) // 512)))
    exact, cuts = _weights_error(q, torch.cat([kc, k], 1), torch.cat([vc, v], 1), P, splits)
    rms = lambda x: float((x - exact).square().mean().sqrt() / exact.square().mean().sqrt())
    here, bound = rms(out.double()), rms(cuts)
    print(f"[rounding] {here:.3e}, equal cuts {bound:.3e}")
    assert here <= bound


def test_softmax_prefix_time_per_request_is_constant():
    """A request's time in a call of many short ones does not grow with their
    number (every workgroup once walked all lengths: 4 times the bound here)."""
    Hkv, d, L, P = 8, 64, 4, 32
    announce("softmax_prefix time per request")
    us = {}
    for B in (512, 8192):
        x = torch.randn((B, P, Hkv, d), device="cuda").to(torch.bfloat16)
        args = (x[:, :L].contiguous(),) * 3 + (x, x, i32([P] * B))
        out = hb.softmax_prefix_step(*args)
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda._sleep(200000)
            a.record()
            for _ in range(5):
                hb.softmax_prefix_step(*args, out=out)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 200)
        us[B] = best
    print(f"[time] {us}")
    assert us[8192] <= 2 * 16 * us[512]


def _softmax64(q, k, v, kc, vc, pl):
    """The attention in 64 bits (lengths pl of the cache, then the block), and the
    spread sum(p |v - out|) / sum(p) of every output: what weights off by a
    relative e each can move it by is e / (1 - e) of that."""
    B, L, Hq, d = q.shape
    Hkv = k.shape[2]
    G = Hq // Hkv
    out, spread = (torch.empty(q.shape, dtype=torch.float64, device="cuda") for _ in range(2))
    for b, n in enumerate(pl):
        kb, vb = (torch.cat([c[b, :n], x[b]]).double().transpose(0, 1) for c, x in ((kc, k), (vc, v)))
        qb = q[b].double().transpose(0, 1).reshape(Hkv, G * L, d)
        p = torch.softmax(torch.matmul(qb, kb.transpose(1, 2).contiguous()) / np.sqrt(d), -1)
        o = torch.matmul(p, vb.contiguous())
        # (over the value columns, in slices)
        sp = torch.stack([(p * (vb[:, None, :, c] - o[:, :, None, c]).abs()).sum(-1) for c in range(d)], -1)
        out[b], spread[b] = (x.reshape(Hq, L, d).transpose(0, 1) for x in (o, sp))
    return out, spread


def _check_rounded_weights(got, out, spread, dt, what):
    """fp32: 1e-5.  bf16: the weights' rounding, at most 2^-8 each, and fp32
    sums."""
    err = (got.double() - out).abs()
    tol = 2 ** -8 / (1 - 2 ** -8) * spread + 1e-5 if dt == "bf16" else torch.full_like(err, 1e-5)
    print(f"[parity] {what}: max abs err {float(err.max()):.3e}, of the bound {float((err / tol).max()):.2f}; "
          f"2e-2 rms is {2e-2 * float(out.square().mean().sqrt()):.2e}")
    assert (err <= tol).all()


BF16_ROWS = [(40, 24, 8, 64, 32, 544, 10), (40, 8, 8, 64, 5, 544, 11)]


@pytest.mark.parametrize("case", BF16_ROWS, ids=lambda s: "x".join(map(str, s)))
def test_softmax_prefix_few_keys_bf16(case):
    """Rows that few keys carry, where the rounding of single weights shows."""
    B, Hq, Hkv, d, L, Pmax, seed = case
    announce(f"softmax_prefix few keys {case}")
    pl = np.random.default_rng(seed).integers(0, Pmax + 1, B)
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *n: torch.randn(n, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v = rnd(B, L, Hq, d), rnd(B, L, Hkv, d), rnd(B, L, Hkv, d)
    kc, vc = rnd(B, Pmax, Hkv, d), rnd(B, Pmax, Hkv, d)
    got = hb.softmax_prefix_step(q, k, v, kc, vc, i32(pl), out_f32=True)
    _check_rounded_weights(got, *_softmax64(q, k, v, kc, vc, pl.tolist()), "bf16", f"few keys {case}")


PLANNED = [
    # (B, Hq, Hkv, d, L, dtype, Pmax, the longest request's ranges: at least)
    # one request of Pmax keys among short ones: the plan alone cuts it
    (24, 8, 8, 64, 4, "bf16", 4096, 5),       # one wave; 3 rounds < B * n_split
    (24, 16, 8, 64, 9, "bf16", 4096, 5),
    (24, 16, 4, 128, 32, "bf16", 4096, 5),
    (24, 16, 2, 128, 32, "bf16", 4096, 5),    # 8 heads per KV head
    (24, 12, 4, 64, 32, "bf16", 4096, 5),     # register-staged
    (24, 8, 8, 64, 5, "f32", 4096, 5),
    (24, 16, 4, 128, 5, "f32", 4096, 3),
    (300, 6, 2, 64, 3, "bf16", 1184, 2),      # more requests than are staged in LDS
    # more requests than three rounds: only the last candidate fits, whole requests
    (50, 32, 32, 64, 3, "bf16", 800, 1),
]


@pytest.mark.parametrize("case", PLANNED, ids=lambda s: "x".join(map(str, s)))
def test_softmax_prefix_planned_ranges(case):
    """Calls that the device plans, contiguous and over permuted pages: the same
    bits, within the bound, and the first request's number of ranges, read off
    the partial results that they leave in the workspace (the second request, of
    one range, leaves none)."""
    B, Hq, Hkv, d, L, dt, Pmax, least = case
    announce(f"softmax_prefix planned {case}")
    act_t = torch.bfloat16 if dt == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(311)
    rnd = lambda *n: torch.randn(n, generator=g, device="cuda").to(act_t)
    pl = np.random.default_rng(312).integers(0, 64, B)
    pl[0], pl[1] = Pmax, 3
    if least > 1:
        pl[B // 2], pl[-1] = Pmax // 2 + 7, Pmax - 31
    q, k, v = rnd(B, L, Hq, d), rnd(B, L, Hkv, d), rnd(B, L, Hkv, d)
    kc, vc = rnd(B, Pmax, Hkv, d), rnd(B, Pmax, Hkv, d)
    dims = hb.make_dims(B, Hq, Hkv, d, L, 64, hb.HYB_BF16 if dt == "bf16" else hb.HYB_F32, 1)
    ws = torch.full((hb.workspace_bytes(dims, hb.OP_SOFTMAX_PREFIX, Pmax) // 4,), float("nan"), device="cuda")
    got = hb.softmax_prefix_step(q, k, v, kc, vc, i32(pl), out_f32=True, ws=ws)
    torch.cuda.synchronize()
    _check_rounded_weights(got, *_softmax64(q, k, v, kc, vc, pl.tolist()), dt, f"planned {case}")
    per = ws.numel() // (B * Hq * L * (d + 2))      # ranges per request that fit
    sums = ws[B * per * Hq * L * d:].view(B * per, -1)
    written = ~torch.isnan(sums).all(1)
    n = int((~written).nonzero()[0]) if not bool(written.all()) else B * per
    print(f"[ranges] the first request: {n or 1}, written in all: {int(written.sum())} of {B * per}")
    assert max(n, 1) >= least and (least > 1 or not written.any())
    page = 32
    order = torch.randperm(B * Pmax // page, generator=g, device="cuda")
    pool = [torch.empty((order.numel(), page, Hkv, d), dtype=act_t, device="cuda") for _ in range(2)]
    for dst, src in zip(pool, (kc, vc)):
        dst[order] = src.view(dst.shape)
    paged = hb.softmax_prefix_step_paged(q, k, v, *pool, order.to(torch.int32).view(B, -1), i32(pl), out_f32=True)
    torch.cuda.synchronize()
    assert torch.equal(got, paged)


def test_softmax_prefix_captured_plan():
    """A captured call plans its ranges anew from the lengths of each replay.
    The shape (6 heads per KV head) has no other test, so this is the first use
    of its kernels: what they ask of the runtime is asked under capture."""
    B, Hq, Hkv, d, L, Pmax = 24, 12, 2, 128, 7, 2048
    announce("softmax_prefix captured plan")
    g = torch.Generator(device="cuda").manual_seed(321)
    rnd = lambda *n: torch.randn(n, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v = rnd(B, L, Hq, d), rnd(B, L, Hkv, d), rnd(B, L, Hkv, d)
    kc, vc = rnd(B, Pmax, Hkv, d), rnd(B, Pmax, Hkv, d)
    pl, out = i32(np.zeros(B)), torch.zeros_like(q)
    dims = hb.make_dims(B, Hq, Hkv, d, L, 64, hb.HYB_BF16, 1)
    ws = torch.empty(hb.workspace_bytes(dims, hb.OP_SOFTMAX_PREFIX, Pmax), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        hb.softmax_prefix_step(q, k, v, kc, vc, pl, out=out, ws=ws)
    for i in range(4):
        lens = np.random.default_rng(322 + i).integers(0, 64, B)
        lens[i] = Pmax
        pl.copy_(i32(lens))
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, hb.softmax_prefix_step(q, k, v, kc, vc, i32(lens)))
        _check_rounded_weights(hb.softmax_prefix_step(q, k, v, kc, vc, i32(lens), out_f32=True),
                               *_softmax64(q, k, v, kc, vc, lens.tolist()), "bf16", f"captured {i}")
