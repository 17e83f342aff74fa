"""Grids that leave most of the chip idle: one strip of 32 rows a workgroup, whose waves share
the other side's subtiles.  And, at the same lengths with more heads, the 128-row blocks that larger grids take."""
import math

import numpy as np
import pytest
import torch

from helpers import check_grad, check_m, dev, fwd_bound, nan_bytes, to64
from test_gpu_exhausted import gen, mixed, mixed_grouped, sb  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def run(sb, oracle, gen, H, Hkv, T, d, kv_heads, seed):
    """kv heads by turns near, sharp and far (a group's first query head sees them so); every gradient of the
    stated ones against the oracle, with a workspace that reads as NaN where nothing was written."""
    G = H // Hkv
    q0, k, v = mixed(gen, 1, Hkv, T, d, seed=seed + T)
    g, q, _ = gen.gaussian(1, H, T, d, seed=seed + T + 1, dtype="bf16")
    q = q.clone()
    q[:, ::G] = q0
    r = gen.remainder_embedding(H, d, seed=seed + 2)
    qd, kd, vd, gd, rd = dev(q, k, v, g, r)
    _, m = sb.sb_attn_fwd_gqa(qd, kd, vd, r=rd)
    ws = nan_bytes(sb.sb_attn_bwd_workspace_bytes(1, H, T, d))
    got = sb.sb_attn_bwd_gqa(qd, kd, vd, m, gd, r=rd, workspace=ws)
    torch.cuda.synchronize()
    for h in kv_heads:
        s, h = slice(h * G, (h + 1) * G), slice(h, h + 1)
        ref = oracle.bwd_gqa(to64(q[:, s]), to64(k[:, h]), to64(v[:, h]), to64(g[:, s]), r=to64(r[s]))
        for name, a, x in zip(("dq", "dk", "dv", "dr"), (got[0][:, s], got[1][:, h], got[2][:, h], got[3][s]), ref):
            check_grad(f"{name} kv head {h.start}", to64(a), x)


@pytest.mark.parametrize("T", [65, 96, 97, 128, 255, 257, 1000])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_strips(sb, oracle, gen, T, d):
    run(sb, oracle, gen, 3, 3, T, d, range(3), seed=0)


@pytest.mark.parametrize("H,Hkv,T", [(6, 3, 200), (16, 2, 97), (15, 3, 321)])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_strips_of_groups(sb, oracle, gen, H, Hkv, T, d):
    run(sb, oracle, gen, H, Hkv, T, d, range(Hkv), seed=40)


@pytest.mark.parametrize("H,Hkv,T", [(2, 2, 2049), (4, 2, 2111), (3, 1, 2080)])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_strips_of_two_words(sb, oracle, gen, H, Hkv, T, d):
    """More than 64 strips of queries reach a strip of keys, in some heads; in the near one none of the second 64 does."""
    run(sb, oracle, gen, H, Hkv, T, d, range(Hkv), seed=60)


@pytest.mark.parametrize("H,Hkv,T", [(21, 21, 993), (15, 15, 2200), (11, 11, 3105), (72, 24, 1750)])
@pytest.mark.parametrize("d", [32, 64])
def test_strips_of_four_waves(sb, oracle, gen, H, Hkv, T, d):
    """Enough strips for the workgroups of four waves, in the query-stationary pass or (the groups) the key-stationary one."""
    run(sb, oracle, gen, H, Hkv, T, d, range(3), seed=70)


@pytest.mark.parametrize("d", [32, 64, 128])
def test_longest_strips(sb, oracle, gen, d):
    """128 subtiles a row, for which the kernels' arrays have room, and one more; the most rows that strips take, and one more, which takes the
    128-row blocks."""
    for T in (4096, 4097, 8192, 8193):
        q, k, v = mixed(gen, 1, 3, T, d, seed=T)
        g = gen.gaussian(1, 3, T, d, seed=T + 1, dtype="bf16")[0]
        h = slice(2, 3)                                    # the far one
        qd, kd, vd, gd = dev(q[:, h], k[:, h], v[:, h], g[:, h])
        _, m = sb.sb_attn_fwd_train(qd, kd, vd)
        ws = nan_bytes(sb.sb_attn_bwd_workspace_bytes(1, 1, T, d))
        got = sb.sb_attn_bwd(qd, kd, vd, m, gd, workspace=ws)
        torch.cuda.synchronize()
        for name, a, r in zip(("dq", "dk", "dv"), got, oracle.bwd(*(to64(t[:, h]) for t in (q, k, v, g)))):
            check_grad(f"{name} T {T}", to64(a), r)


def weights_of_the_last_rows(sb, q, k, v):
    """Of the last d rows of every head the weights that enter dV = A^T dO, each a bfloat16 (dO has one 1 in each of
    these rows, in a column of its own), the same in fp64, and the bits of their stick that the rows use up."""
    _, H, T, d = q.shape
    q, k, v = dev(q, k, v)
    _, m = sb.sb_attn_fwd_train(q, k, v)
    g = torch.zeros_like(q)
    rows = torch.arange(T - d, T, device="cuda")
    g[0, :, rows, torch.arange(d, device="cuda")] = 1.0
    _, _, dv = sb.sb_attn_bwd(q, k, v, m, g)
    z = q[0, :, rows].double() @ k[0].double().transpose(1, 2).contiguous() / math.sqrt(d)
    seen = torch.arange(T, device="cuda") < rows[:, None]
    sp = torch.where(seen, torch.nn.functional.softplus(z, threshold=1e9), 0.0)
    a = torch.where(seen, torch.exp(z - sp.flip(-1).cumsum(-1).flip(-1)), 0.0)
    return dv[0].transpose(1, 2).double(), a, sp.sum(-1) / math.log(2)


# the share with softplus totals summed up from the diagonal, and with carries counted down from m and left so: 9.4e-4, 1.55e-3;
# 1.29e-3, 2.22e-3; 9.0e-4, 1.85e-3; 2.20e-3, 3.22e-3 (other inputs of the kind: within a fifth).  The bound lies between the two
@pytest.mark.parametrize("H,T,d,share", [(8, 1000, 128, 1.2e-3), (4, 2000, 128, 1.7e-3), (8, 1000, 64, 1.3e-3), (2, 4000, 32, 2.7e-3)])
def test_weights_of_rows_that_are_nearly_exhausted(sb, gen, H, T, d, share):
    """Rows that use up most of 160 bits of their stick, whose m is known to some 1e-5 only: the weights next to the diagonal
    are as good as sums over the keys nearer than theirs.  Counted are those that round to another bfloat16 than in fp64."""
    mean = math.log(120 * math.log(2) / T) - 0.5                # of the logits, for 120 bits a row
    got, a, bits = weights_of_the_last_rows(sb, *gen.biased_gaussian(1, H, T, d, seed=T, shift=mean))
    assert 60 < bits.mean() < 150 and bits.max() < 160
    big = a > 2.0 ** -12
    assert (got != a.float().bfloat16().double())[big].double().mean() <= share


# H12 T3200 at d = 64: workgroups of four waves, which have room for 96 carries in place of 128
@pytest.mark.parametrize("H,T,d", [(1, 4000, 32), (1, 4200, 32), (1, 8192, 32), (1, 4200, 64), (1, 8192, 64), (1, 4200, 128), (1, 8192, 128), (12, 3200, 64)])
def test_sharp_and_far_rows_in_one_strip(sb, oracle, gen, H, T, d):
    """Every other row is exhausted within a few keys and goes on to tens of thousands of bits, those between them never are: no
    start is found, in the longer ones not even looked for to the end, and the sharp rows' carries come down from there."""
    q, k, v = gen.biased_gaussian(1, H, T, d, seed=T, shift=-6.0)
    x = gen.scaled_gaussian(1, H, T, d, seed=T + 1, gain=1.0)[0][:, :, 1::2] * 20.0
    x[..., -1] = 0.0
    q[:, :, 1::2] = x
    got, a, bits = weights_of_the_last_rows(sb, q, k, v)
    sharp = torch.arange(T - d, T, device="cuda") % 2 == 1
    assert bits[:, sharp].min() > 20000 and bits[:, ~sharp].max() < 160
    big = a > 2.0 ** -12
    # half a unit of 8 bits, and what fp32 leaves in exponents made of numbers up to some 100
    assert ((got - a) / a).abs()[big].max() <= 2.0 ** -8 + 1e-4
    g = gen.gaussian(1, H, T, d, seed=T + 2, dtype="bf16")[0]
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_fwd_train(qd, kd, vd)
    got = sb.sb_attn_bwd(qd, kd, vd, m, gd, workspace=nan_bytes(sb.sb_attn_bwd_workspace_bytes(1, H, T, d)))
    h = slice(H - 1, H)
    for name, x, ref in zip(("dq", "dk", "dv"), got, oracle.bwd(*(to64(t[:, h]) for t in (q, k, v, g)))):
        check_grad(name, to64(x[:, h]), ref)


@pytest.mark.parametrize("H,Hkv,T,d", [(66, 66, 129, 64), (66, 66, 257, 32), (42, 42, 193, 128), (42, 42, 255, 128), (90, 45, 200, 128),
                                       (132, 66, 130, 64), (150, 150, 129, 128), (150, 150, 65, 32)])
def test_blocks_of_larger_grids(sb, oracle, gen, H, Hkv, T, d):
    run(sb, oracle, gen, H, Hkv, T, d, (0, 1, 2, Hkv - 1), seed=80)


@pytest.mark.parametrize("d", [64, 128])
def test_packed(sb, oracle, gen, d):
    """Sequences of all kinds of lengths in one small grid: none, one row, one strip, a strip and a row, many."""
    lens = [1, 0, 32, 33, 64, 65, 96, 300]
    q, k, v = mixed(gen, 1, 3, sum(lens), d, seed=7)
    g = gen.gaussian(1, 3, sum(lens), d, seed=8, dtype="bf16")[0]
    q, k, v, g = (t[0] for t in (q, k, v, g))
    cu = torch.tensor(np.cumsum([0] + lens), dtype=torch.int32)
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_varlen_fwd(qd, kd, vd, cu.cuda(), max(lens))
    got = sb.sb_attn_varlen_bwd(qd, kd, vd, m, gd, cu.cuda(), max(lens))
    torch.cuda.synchronize()
    for i, n in enumerate(lens):
        s = slice(int(cu[i]), int(cu[i]) + n)
        if n:
            for name, a, r in zip(("dq", "dk", "dv"), got, oracle.bwd(*(to64(t[:, s]) for t in (q, k, v, g)))):
                check_grad(f"{name} of {n}", to64(a[:, s]), r)


def beyond_small_grids(T):
    """How many times three heads of T rows are beyond the forward's largest small grid, 1000 strips."""
    return 1000 // (3 * ((T + 31) // 32)) + 1


@pytest.mark.parametrize("T", [65, 96, 97, 128, 129, 255, 257, 321, 500, 1000, 4096])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward_strips(sb, oracle, gen, T, d):
    """o of a small grid is what the 128-row blocks of a large one give, bit for bit; o and m against the oracle."""
    q, k, v = mixed(gen, 1, 3, T, d, seed=300 + T)
    r = gen.remainder_embedding(3, d, seed=9)
    qd, kd, vd, rd = dev(q, k, v, r)
    o, m = sb.sb_attn_fwd_gqa(qd, kd, vd, r=rd)
    o2 = sb.sb_attn_fwd(qd, kd, vd)
    times = beyond_small_grids(T)
    many = [torch.cat([t] * times) for t in (qd, kd, vd)]
    om, mm = sb.sb_attn_fwd_gqa(*many, r=rd)
    torch.cuda.synchronize()
    for i in (0, times - 1):
        assert torch.equal(o, om[i:i + 1])
        assert torch.allclose(m, mm[i:i + 1], rtol=1e-5, atol=1e-4)      # sums in another order behind exhausted rows
    assert torch.equal(o2, sb.sb_attn_fwd(*many)[:1])
    if T <= 1000:
        ref, rem = oracle.fwd(to64(q), to64(k), to64(v), r=to64(r))
        assert np.all(np.abs(to64(o) - ref) <= fwd_bound(ref, to64(v)))
        check_m(to64(m), rem)


@pytest.mark.parametrize("H,T", [(10, 2500), (10, 2753), (11, 2273), (10, 3008)])
def test_forward_strips_of_four_waves(sb, oracle, gen, H, T):
    """d = 32, enough strips for the workgroups of four waves (two batch entries: 128-row blocks, which give the same o): rows that end within a subtile, heads
    that are exhausted within a round and heads that never are."""
    d = 32
    q, k, v = mixed(gen, 1, H, T, d, seed=500 + T)
    r = gen.remainder_embedding(H, d, seed=10)
    qd, kd, vd, rd = dev(q, k, v, r)
    o, m = sb.sb_attn_fwd_gqa(qd, kd, vd, r=rd)
    o2 = sb.sb_attn_fwd(qd, kd, vd)
    om, mm = sb.sb_attn_fwd_gqa(*(torch.cat([t] * 2) for t in (qd, kd, vd)), r=rd)
    assert torch.equal(o, om[:1]) and torch.allclose(m, mm[:1], rtol=1e-5, atol=1e-4)
    assert torch.equal(o2, sb.sb_attn_fwd(*(torch.cat([t] * 2) for t in (qd, kd, vd)))[:1])
    h = slice(0, 3)
    ref, rem = oracle.fwd(*(to64(t[:, h]) for t in (q, k, v)), r=to64(r[h]))
    assert np.all(np.abs(to64(o[:, h]) - ref) <= fwd_bound(ref, to64(v[:, h])))
    check_m(to64(m[:, h]), rem)


# last pairs of one row, of one strip, of one row behind a whole strip; shared kv heads
@pytest.mark.parametrize("H,Hkv,T,d", [(10, 10, 2500, 64), (12, 12, 2080, 64), (10, 5, 2529, 64), (9, 9, 3489, 64), (10, 10, 3009, 64),
                                       (12, 12, 1057, 128), (8, 8, 2000, 128), (10, 10, 1600, 128), (12, 4, 1281, 128), (2, 2, 8190, 128)])
def test_forward_two_strips(sb, oracle, gen, H, Hkv, T, d):
    """Two strips a workgroup, without m: o is what the 128-row blocks of twice as large a grid give, bit for bit, and what is given with m; with a remainder bias
    as well, and against the oracle.  Heads that are exhausted within a round, both strips or one after the other, and heads that never are."""
    q, k, v, _ = mixed_grouped(gen, 1, H, Hkv, T, d, seed=700 + T)
    r = gen.remainder_embedding(H, d, seed=11)
    qd, kd, vd, rd = dev(q, k, v, r)
    twice = [torch.cat([t] * 2) for t in (qd, kd, vd)]
    for bias in (None, rd):
        o = sb.sb_attn_fwd_gqa(qd, kd, vd, r=bias, want_m=False)
        assert torch.equal(o, sb.sb_attn_fwd_gqa(qd, kd, vd, r=bias)[0])
        assert torch.equal(o, sb.sb_attn_fwd_gqa(*twice, r=bias, want_m=False)[:1])
    h, G = slice(0, min(3, Hkv)), H // Hkv
    heads = slice(0, h.stop * G)
    if T <= 4000:
        ref = oracle.fwd_gqa(to64(q[:, heads]), to64(k[:, h]), to64(v[:, h]), r=to64(r[heads]))[0]
        assert np.all(np.abs(to64(o[:, heads]) - ref) <= fwd_bound(ref, to64(v[:, h])))


TWO_STRIPS_LENS = [2500, 33, 64, 65, 1, 0, 31, 96, 97]


@pytest.mark.parametrize("H,d", [(9, 64), (5, 128)])
def test_forward_two_strips_packed(sb, gen, H, d):
    """Sequences of all kinds of lengths, two strips a workgroup: each as it is alone."""
    lens = TWO_STRIPS_LENS
    q, k, v = dev(*(t[0] for t in mixed(gen, 1, H, sum(lens), d, seed=18)))
    cu = torch.tensor(np.cumsum([0] + lens), dtype=torch.int32).cuda()
    o = torch.full_like(q, float("nan"))
    sb.sb_attn_varlen_fwd(q, k, v, cu, max(lens), o=o, want_m=False)
    at = 0
    for n in lens:
        s = slice(at, at + n)
        at += n
        if n:
            assert torch.equal(o[:, s], sb.sb_attn_fwd_train(*(t[None, :, s].contiguous() for t in (q, k, v)))[0][0]), n


@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward_packed(sb, gen, d):
    """Sequences of all kinds of lengths in one small grid: each as it is alone."""
    lens = [1, 0, 32, 33, 64, 65, 96, 400]
    q, k, v = (t[0] for t in mixed(gen, 1, 3, sum(lens), d, seed=17))
    cu = torch.tensor(np.cumsum([0] + lens), dtype=torch.int32)
    qd, kd, vd = dev(q, k, v)
    o, m = sb.sb_attn_varlen_fwd(qd, kd, vd, cu.cuda(), max(lens))
    for i, n in enumerate(lens):
        s = slice(int(cu[i]), int(cu[i]) + n)
        if n:
            o1, m1 = sb.sb_attn_fwd_train(*(t[None, :, s].contiguous() for t in (qd, kd, vd)))
            assert torch.equal(o[:, s], o1[0]) and torch.allclose(m[:, s], m1[0], rtol=1e-5, atol=1e-4)


@pytest.mark.parametrize("lens,H,Hkv,max_T", [
    ([0] * 3 + [1, 33] * 32 + [0, 300, 31], 2, 2, 300),                # 70 sequences: more than a wave looks at at a time
    ([2, 0, 34] * 21 + [1, 400] + [0] * 70, 1, 1, 400),                # the 64th and the 65th of 135; nothing behind them
    ([100] * 13, 4, 2, 1300),                                          # a maximum that no sequence comes near
])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_packed_places(sb, oracle, gen, lens, H, Hkv, max_T, d):
    """A workgroup finds its sequence and strip among many, and among empty ones: o is every sequence's alone,
    bit for bit, and every gradient the oracle's."""
    q0, k, v = mixed(gen, 1, Hkv, sum(lens), d, seed=27)
    g, q, _ = gen.gaussian(1, H, sum(lens), d, seed=28, dtype="bf16")
    q = q.clone()
    q[:, ::H // Hkv] = q0
    q, k, v, g = (t[0] for t in (q, k, v, g))
    r = gen.remainder_embedding(H, d, seed=29)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    qd, kd, vd, gd, rd, cud = dev(q, k, v, g, r, torch.from_numpy(cu))
    o, m = sb.sb_attn_varlen_fwd(qd, kd, vd, cud, max_T, r=rd)
    ws = nan_bytes(sb.sb_attn_varlen_bwd_workspace_bytes(len(lens), H, sum(lens), max_T, d))
    got = sb.sb_attn_varlen_bwd(qd, kd, vd, m, gd, cud, max_T, r=rd, workspace=ws)
    for a, n in zip(cu, lens):
        s = slice(int(a), int(a) + n)
        if n:
            o1, m1 = sb.sb_attn_fwd_gqa(*(t[None, :, s].contiguous() for t in (qd, kd, vd)), r=rd)
            assert torch.equal(o[:, s], o1[0]) and torch.allclose(m[:, s], m1[0], rtol=1e-5, atol=1e-4)
    ref = oracle.bwd_varlen(to64(q), to64(k), to64(v), to64(g), cu, r=to64(r))
    for name, a, x in zip(("dq", "dk", "dv", "dr"), got, ref):
        check_grad(name, to64(a), x)


@pytest.mark.parametrize("B,H,T,d", [(1, 1, 321, 32), (1, 3, 1500, 32), (1, 1, 65, 64), (2, 1, 700, 64), (1, 1, 8192, 64), (1, 8, 1024, 128), (1, 8, 1025, 128)])
@pytest.mark.parametrize("shift", [-3.0, -6.0])
def test_halting_strips(sb, gen, B, H, T, d, shift):
    """A halting sweep of a small grid, against the whole one: off by at most eps max|v| and a rounding of each to bfloat16, whatever is
    skipped; the same to the bit where tiles are counted (by blocks), and as the whole one where nothing may be skipped."""
    q, k, v = dev(*gen.biased_gaussian(B, H, T, d, seed=T, shift=shift, dtype="bf16"))
    whole = sb.sb_attn_fwd(q, k, v)
    for eps in (1e-2, 1e-6):
        o = sb.sb_attn_fwd_halt(q, k, v, eps)
        assert (o.float() - whole.float()).abs().max() <= eps * v.float().abs().max() + 2.0 ** -8 * whole.float().abs().max(), eps
        counts = torch.zeros(2, dtype=torch.int64, device="cuda")
        assert torch.equal(o, sb.sb_attn_fwd_halt(q, k, v, eps, tile_counts=counts))
        swept, all_of_them = counts.tolist()
        assert 0 < swept <= all_of_them == B * H * sum((min(T, 128 * i + 128) + 62) // 64 for i in range((T + 127) // 128))
    k[..., -1] = -200.0 * d ** 0.5                            # logits of -200 and below: no stick is used up
    q[..., -1] = 1.0
    k[..., :-1] = 0.0
    counts = torch.zeros(2, dtype=torch.int64, device="cuda")
    o = sb.sb_attn_fwd_halt(q, k, v, 1e-6)
    assert torch.equal(o, sb.sb_attn_fwd(q, k, v)) and torch.equal(o, sb.sb_attn_fwd_halt(q, k, v, 1e-6, tile_counts=counts))
