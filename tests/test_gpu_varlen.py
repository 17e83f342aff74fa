"""GPU parity of the packed variable-length entry points (sequences packed along T attend
only inside themselves) against the CPU float64 oracle, through the C ABI.  Tolerances as
for the plain path: forward 2e-2 max abs; gradients max(2e-2, 2^-8 * max|ref|) per tensor."""
import numpy as np
import pytest
import torch

from helpers import check_grad, BF16_TOL, check_m, dev, max_abs, nan_bytes, to64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2410_17980_amd import binding
    binding.load(build_if_missing=False)
    return binding


@pytest.fixture(scope="module")
def gen():
    from paper_2410_17980_amd import inputs
    return inputs


def packed(gen, H, Hkv, lens, d, seed, kind="gaussian", **kw):
    """q, k, v, dout packed [H, Ttot, d] and the int32 offsets."""
    Ttot = sum(lens)
    f = getattr(gen, kind)
    q, _, _, g = f(1, H, Ttot, d, seed=seed, with_dout=True, **kw)
    _, k, v, _ = f(1, Hkv, Ttot, d, seed=seed + 1, with_dout=True, **kw)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return q[0], k[0], v[0], g[0], cu


def check(sb, oracle, q, k, v, g, cu, max_T=None, r=None):
    lens = np.diff(cu)
    max_T = int(lens.max()) if max_T is None else max_T
    qd, kd, vd, gd = dev(q, k, v, g)
    cud = torch.from_numpy(cu).cuda()
    rd = r.cuda() if r is not None else None
    o, m = sb.sb_attn_varlen_fwd(qd, kd, vd, cud, max_T, r=rd)
    ws = nan_bytes(sb.sb_attn_varlen_bwd_workspace_bytes(len(cu) - 1, q.shape[0], q.shape[1], max_T, q.shape[2]))
    grads = sb.sb_attn_varlen_bwd(qd, kd, vd, m, gd, cud, max_T, r=rd, workspace=ws)
    torch.cuda.synchronize()
    r64 = to64(r) if r is not None else None
    ref, rem = oracle.fwd_varlen(to64(q), to64(k), to64(v), cu, r=r64)
    err = max_abs(to64(o), ref)
    print(f"fwd err {err:.3e}")
    assert err <= BF16_TOL
    check_m(to64(m), rem)
    refs = oracle.bwd_varlen(to64(q), to64(k), to64(v), to64(g), cu, r=r64)
    assert len(grads) == len(refs)
    for name, a, rf in zip(("dq", "dk", "dv", "dr"), grads, refs):
        a = to64(a)
        assert a.shape == rf.shape, name
        check_grad(name, a, rf)
    return o, m, grads


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("lens", [[200], [1, 2, 3], [130, 0, 77, 1, 300], [64, 128, 256], [33, 500, 31], [65, 129, 1, 257]])
def test_length_mixes(sb, oracle, gen, lens, d):
    check(sb, oracle, *packed(gen, 3, 3, lens, d, seed=sum(lens) + d))


def test_grouped_heads_and_remainder_bias(sb, oracle, gen):
    q, k, v, g, cu = packed(gen, 6, 2, [150, 90, 260], 64, seed=7, kind="biased_gaussian", shift=-4.0)
    check(sb, oracle, q, k, v, g, cu, r=gen.remainder_embedding(6, 64, seed=8))


def test_long_range_inside_sequences(sb, oracle, gen):
    check(sb, oracle, *packed(gen, 2, 2, [700, 450], 128, seed=9, kind="biased_gaussian", shift=-6.0))


def test_sharp_sequences_take_the_redo(sb, oracle, gen):
    check(sb, oracle, *packed(gen, 2, 1, [260, 140], 128, seed=10, kind="scaled_gaussian", gain=12.0))


def test_loose_length_bound_gives_the_same_result(sb, oracle, gen):
    q, k, v, g, cu = packed(gen, 2, 2, [100, 40, 160], 128, seed=11)
    o1, m1, g1 = check(sb, oracle, q, k, v, g, cu)
    o2, m2, g2 = check(sb, oracle, q, k, v, g, cu, max_T=300)
    assert torch.equal(o1, o2) and torch.equal(m1, m2)
    for a, b in zip(g1, g2):
        assert torch.equal(a, b)


@pytest.mark.parametrize("H,lens", [(3, [0] * 3 + [1, 128, 129, 0, 300, 127]), (1, [0] * 4 + [1, 0, 129, 33])])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_bias_gradient_of_many_sequences(sb, oracle, gen, H, lens, d):
    """Chunks of 128 rows at the sequences' ends, none for empty ones, more sequences than a wave has lanes, and a bound on their
    lengths that leaves room for many times as many; blocks and (one head) strips."""
    lens = lens * 9
    q, k, v, g, cu = packed(gen, H, H, lens, d, seed=12, kind="biased_gaussian", shift=-4.0)
    check(sb, oracle, q, k, v, g, cu, max_T=1400, r=gen.remainder_embedding(H, d, seed=13))


def test_equal_lengths_match_the_batched_call(sb, gen):
    """Packing B equal sequences gives, bit for bit, the batched entry points' results."""
    B, H, T, d = 3, 2, 200, 128
    q, k, v, g = gen.gaussian(B, H, T, d, seed=12, with_dout=True)
    qd, kd, vd, gd = dev(q, k, v, g)
    o, m = sb.sb_attn_fwd_train(qd, kd, vd)
    dq, dk, dv = sb.sb_attn_bwd(qd, kd, vd, m, gd)
    pack = lambda t: t.transpose(0, 1).reshape(H, B * T, d).contiguous()
    cu = torch.arange(0, (B + 1) * T, T, dtype=torch.int32, device="cuda")
    o2, m2 = sb.sb_attn_varlen_fwd(pack(qd), pack(kd), pack(vd), cu, T)
    dq2, dk2, dv2 = sb.sb_attn_varlen_bwd(pack(qd), pack(kd), pack(vd), m2, pack(gd), cu, T)
    torch.cuda.synchronize()
    assert torch.equal(o2, pack(o)) and torch.equal(m2, m.transpose(0, 1).reshape(H, B * T))
    assert torch.equal(dq2, pack(dq)) and torch.equal(dk2, pack(dk)) and torch.equal(dv2, pack(dv))


def test_argument_errors(sb, gen):
    q, k, v, g, cu = packed(gen, 2, 2, [40, 50], 64, seed=13)
    qd, kd, vd = dev(q, k, v)
    cud = torch.from_numpy(cu).cuda()
    with pytest.raises(sb.SbAttnError):
        sb.sb_attn_varlen_fwd(qd, kd, vd, cud, 0)
    with pytest.raises(sb.SbAttnError):
        sb.sb_attn_varlen_fwd(qd, kd, vd, cud, 91)
    with pytest.raises(sb.SbAttnError):
        sb.sb_attn_varlen_fwd(qd, kd, vd, cud.to(torch.int64), 50)


# lengths of 1 to 5 blocks and a long one, so that blocks are looked up by their length; 1, 2 and 4 sequences to a lane, and more than a
# wave holds; blocks that end with the sequence, empty sequences, one that takes everything
BY_LENGTH = {
    "few": [1900, 5, 128, 0, 384, 385, 127, 1, 640, 33],
    "64": [1700] + [1 + 37 * i % 200 for i in range(63)],
    "65": [1 + 53 * i % 200 for i in range(64)] + [2000],
    "200": [1 + 11 * i % 90 for i in range(120)] + [3000] + [0, 129] * 40,
    "300": [20] * 150 + [2800] + [9] * 149,
    "first": [4000] + [0] * 9,
}


@pytest.mark.parametrize("H,Hkv,d", [(16, 16, 32), (9, 9, 64), (12, 12, 128), (4, 4, 64), (24, 12, 128), (20, 5, 32)])
@pytest.mark.parametrize("lens", BY_LENGTH)
def test_blocks_by_length(sb, lens, H, Hkv, d):
    """Every block is found once: all rows are written, and as by a call for each sequence alone.  The weights are those of the same
    tiles in the same order, so o is the same to the bit where that call takes blocks as well; it may take strips, which round
    the partial sums of m differently (some 2^-20 of its size) and, with their other carries, the bfloat16 operands of the gradients: two
    results within the gradients' tolerance differ by at most twice that."""
    lens = BY_LENGTH[lens]
    T, g = sum(lens), torch.Generator(device="cuda").manual_seed(7)
    q, do = (torch.randn(H, T, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn(Hkv, T, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    far, of = (6.0 * d ** 0.5) ** 0.5, H // Hkv
    for h in range(2, Hkv, 3):                               # logits around -6: weights that reach over hundreds of keys
        q[h * of:(h + 1) * of, :, -1], k[h, :, -1] = far, -far
    cu = torch.tensor([0] + lens, device="cuda").cumsum(0).int()
    o, m = torch.full_like(q, float("nan")), torch.full((H, T), float("nan"), device="cuda")
    grads = [torch.full(x.shape, float("nan"), device="cuda") for x in (q, k, v)]
    sb.sb_attn_varlen_fwd(q, k, v, cu, max(lens), o=o, m=m)
    sb.sb_attn_varlen_bwd(q, k, v, m, do, cu, max(lens), dq=grads[0], dk=grads[1], dv=grads[2])
    assert torch.isfinite(m).all()
    assert (m[2 * of, sum(lens[:lens.index(max(lens))]) + 500] > -4.0).all()      # more than 1 % of the stick after 500 keys
    at, worst = 0, 0.0
    for n in lens:
        x = slice(at, at + n)
        at += n
        if n == 0 or (n < 100 and x.start % 3):              # (of the many short ones, some)
            continue
        one = [t[None, :, x].contiguous() for t in (q, k, v)]
        o1, m1 = sb.sb_attn_fwd_gqa(*one, want_m=True)
        assert torch.equal(o[:, x], o1[0]), n
        assert torch.allclose(m[:, x], m1[0], rtol=1e-5, atol=1e-5), n
        ref = sb.sb_attn_bwd_gqa(*one, m1, do[None, :, x].contiguous())
        for a, b in zip(grads, ref):
            assert (a[:, x] - b[0]).abs().max() <= 2 * max(2e-2, 2.0 ** -8 * b.abs().max()), n
            # every head for itself, far ones with their small gradients as well: two results of bfloat16 operands, 2^-9 off each
            off, size = (a[:, x] - b[0]).flatten(1).norm(dim=1), b[0].flatten(1).norm(dim=1)
            worst = max(worst, float((off / size.clamp(min=1e-30)).max()))
            assert (off <= 2.0 ** -8 * size).all(), (n, float((off / size).max()))
    print(f"worst head {worst:.2e}")
    assert all(torch.isfinite(a).all() for a in grads) and torch.isfinite(o.float()).all()
