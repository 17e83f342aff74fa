"""GPU parity where the stick is used up long before key 0: the kernels stop forming weights once
every row of a block is exhausted (they are zero from there on), so these sizes put the end of the
sweep at every place it can fall relative to the unrolled loop and the last tile."""
import numpy as np
import pytest
import torch

from helpers import check_grad, check_m, dev, fwd_bound, nan_bytes, to64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2410_17980_amd import binding
    binding.load(build_if_missing=False)      # the built library must be there
    return binding


@pytest.fixture(scope="module")
def gen():
    from paper_2410_17980_amd import inputs
    return inputs


def mixed(gen, B, H, T, d, seed):
    """Heads by turns: exhausted within ~130 keys, within a few (sharp, chains out of range), never."""
    q, k, v = gen.gaussian(B, H, T, d, seed=seed, dtype="bf16")
    _, k30, _ = gen.scaled_gaussian(B, H, T, d, seed, gain=30.0)
    qb, kb, _ = gen.biased_gaussian(B, H, T, d, seed=seed, shift=-6.0, dtype="bf16")
    q, k = q.clone(), k.clone()
    k[:, 1::3] = k30[:, 1::3]
    q[:, 2::3], k[:, 2::3] = qb[:, 2::3], kb[:, 2::3]
    return q, k, v


@pytest.mark.parametrize("T", [257, 383, 449, 511, 640, 705, 1025, 1300])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward(sb, oracle, gen, T, d):
    q, k, v = mixed(gen, 1, 3, T, d, seed=500 + T)
    qd, kd, vd = dev(q, k, v)
    o, m = sb.sb_attn_fwd_train(qd, kd, vd)
    o2 = sb.sb_attn_fwd(qd, kd, vd)
    torch.cuda.synchronize()
    ref, rem = oracle.fwd(to64(q), to64(k), to64(v))
    assert torch.equal(o, o2)
    assert np.all(np.abs(to64(o) - ref) <= fwd_bound(ref, to64(v)))
    check_m(to64(m), rem)


def test_m_without_underflow(sb, gen):
    """m beyond float64's range of the remainder itself: the softplus sum in float64."""
    q, k, v = mixed(gen, 1, 3, 1500, 64, seed=9)
    _, m = sb.sb_attn_fwd_train(*dev(q, k, v))
    z = to64(q) @ np.swapaxes(to64(k), -1, -2) / 8.0
    sp = np.tril(np.logaddexp(0.0, z), -1)
    ref = -sp.sum(-1)
    assert np.all(np.abs(to64(m) - ref) <= 2e-3 + 1e-4 * np.abs(ref))


@pytest.mark.parametrize("T", [257, 320, 353, 385, 449, 577, 641, 1283])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_m_of_short_tails(sb, gen, T, d):
    """m over 0 to 18 tiles behind the end of the weights, odd and even, whose keys the waves of a block
    share, with one to four waves' rows in the last block.  A logit is a sum of d products in fp32, a
    softplus total one of T logits' worth: both a few 2^-24 of their terms, 1e-5 in all."""
    q, k, v = mixed(gen, 2, 3, T, d, seed=900 + T)
    _, m = sb.sb_attn_fwd_train(*dev(q, k, v))
    z = to64(q) @ np.swapaxes(to64(k), -1, -2) / np.sqrt(d)
    ref = -np.tril(np.logaddexp(0.0, z), -1).sum(-1)
    assert np.all(np.abs(to64(m) - ref) <= 1e-4 + 1e-5 * np.abs(ref))


@pytest.mark.parametrize("H,T", [(1, 130), (9, 300), (65, 300), (3, 8200)])
def test_every_block_once(sb, gen, H, T):
    """The shares of the launch (heads over XCDs, single blocks or pairs) cover every row: equal to
    one launch per head, which takes another share."""
    q, k, v = dev(*mixed(gen, 1, H, T, 32, seed=77))
    o, m = sb.sb_attn_fwd_train(q, k, v)
    for h in {0, H // 2, H - 1}:
        oh, mh = sb.sb_attn_fwd_train(*(t[:, h:h + 1].contiguous() for t in (q, k, v)))
        assert torch.equal(o[:, h:h + 1], oh) and torch.equal(m[:, h:h + 1], mh)


@pytest.mark.parametrize("T", [511, 512, 577, 705, 1025, 1300])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_backward(sb, oracle, gen, T, d):
    q, k, v = mixed(gen, 1, 3, T, d, seed=600 + T)
    g = gen.gaussian(1, 3, T, d, seed=601 + T, dtype="bf16")[0]
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_fwd_train(qd, kd, vd)
    ws = nan_bytes(sb.sb_attn_bwd_workspace_bytes(1, 3, T, d))
    got = sb.sb_attn_bwd(qd, kd, vd, m, gd, workspace=ws)
    torch.cuda.synchronize()
    for name, a, r in zip(("dq", "dk", "dv"), got, oracle.bwd(*(to64(t) for t in (q, k, v, g)))):
        for h in range(3):
            check_grad(f"{name} head {h}", to64(a)[:, h], r[:, h])


@pytest.mark.parametrize("d", [64, 128])
def test_backward_far_queries_come_back(sb, oracle, gen, d):
    """Rows 1024..1151 reach all keys, the rows before them only near ones: the query blocks that
    reach a key block are not contiguous."""
    T = 1300
    q, k, v, g = gen.gaussian(1, 1, T, d, seed=8, dtype="bf16", with_dout=True)
    q, k = q.clone(), k.clone()
    q[..., 0], k[..., 0] = 0.0, -4.0
    q[..., 1024:1152, :] *= 0.25
    q[..., 1024:1152, 0] = 2.0 * d ** 0.5
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_fwd_train(qd, kd, vd)
    ws = nan_bytes(sb.sb_attn_bwd_workspace_bytes(1, 1, T, d))
    got = sb.sb_attn_bwd(qd, kd, vd, m, gd, workspace=ws)
    torch.cuda.synchronize()
    for name, a, r in zip(("dq", "dk", "dv"), got, oracle.bwd(*(to64(t) for t in (q, k, v, g)))):
        check_grad(name, to64(a), r)


@pytest.mark.parametrize("H,Hkv,T,d", [(6, 3, 256, 128), (6, 3, 257, 64), (34, 2, 600, 32), (12, 3, 1536, 128), (12, 3, 1537, 128),
                                       (6, 3, 1793, 64), (3, 3, 2048, 32), (51, 3, 3000, 64), (3, 3, 33025, 128),
                                       # spread over the chip with m beyond 512 keys; without it from 513, 1025 or 1281 keys on at
                                       # d = 128, 64, 32; both up to 34 MB in all
                                       (6, 3, 512, 128), (34, 2, 513, 64), (6, 3, 513, 128), (51, 3, 1025, 32),
                                       (34, 2, 1024, 64), (6, 3, 1025, 64), (34, 2, 1280, 32), (51, 3, 1281, 32),
                                       (6, 3, 24001, 128), (51, 3, 46000, 64), (6, 6, 47000, 32)])
def test_decode(sb, oracle, gen, H, Hkv, T, d):
    """Caches at the edges of the passes and of the ways to split them, groups of 1 to 17 heads; without m
    (exhausted heads may finish early) and with it (no head does)."""
    q = gen.gaussian(1, H, 1, d, seed=T)[0][:, :, 0].clone()
    qk, k, v = mixed(gen, 1, Hkv, T, d, seed=T + 1)
    G = H // Hkv
    for h in range(2, Hkv, 3):
        q[:, h * G:(h + 1) * G] = qk[:, h, -1:].expand(-1, G, -1)
    r = gen.remainder_embedding(H, d, seed=3)
    ref, rem = oracle.decode(*(to64(t) for t in (q, k, v)), r=to64(r))
    ws = nan_bytes(sb.load().sb_attn_decode_workspace_bytes(1, H, T, d))
    qd, kd, vd, rd = dev(q, k, v, r)
    o = sb.sb_attn_decode(qd, kd, vd, r=rd, workspace=ws)
    o2, m = sb.sb_attn_decode(qd, kd, vd, r=rd, workspace=ws, want_m=True)
    torch.cuda.synchronize()
    for x in (o, o2):
        assert np.all(np.abs(to64(x) - ref) <= fwd_bound(ref, to64(v)))
    check_m(to64(m), rem)


@pytest.mark.parametrize("T", [449, 512, 577])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_backward_of_more_blocks_than_cus(sb, oracle, gen, T, d):
    """Grids beyond the small ones take other key-stationary kernels: 97 heads of 4 or 5 key blocks."""
    H = 97
    q, k, v = mixed(gen, 1, H, T, d, seed=700 + T)
    g = gen.gaussian(1, H, T, d, seed=701 + T, dtype="bf16")[0]
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_fwd_train(qd, kd, vd)
    got = sb.sb_attn_bwd(qd, kd, vd, m, gd, workspace=nan_bytes(sb.sb_attn_bwd_workspace_bytes(1, H, T, d)))
    torch.cuda.synchronize()
    for h in (0, 1, 2, 95, 96):
        one = (to64(t[:, h:h + 1]) for t in (q, k, v, g))
        for name, a, r in zip(("dq", "dk", "dv"), got, oracle.bwd(*one)):
            check_grad(f"{name} head {h}", to64(a)[:, h], r[:, 0])


@pytest.mark.parametrize("T", [129, 193, 1024, 1025, 1153, 1216])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_halt_after_the_first_tile_behind_the_band(sb, gen, T, d):
    """N(0,1) logits leave less than 2^-20 after 64 keys (about 74 bits are used up; the sum of 64 terms
    of mean 1.16 and deviation 0.9 stays above 20 in every row).  So a block takes its diagonal band and
    the one tile behind it, and no more."""
    H, eps = 4, 2.0 ** -20
    q, k, v = dev(*gen.gaussian(1, H, T, d, seed=800 + T, dtype="bf16"))
    tc = torch.zeros(2, dtype=torch.int64, device="cuda")
    sb.sb_attn_fwd_halt(q, k, v, eps, tile_counts=tc)
    full = want = 0
    for Q0 in range(0, T, 128):
        ntile = (min(T, Q0 + 128) - 1 + 63) // 64
        ndiag = max(0, ntile - Q0 // 64)
        full += ntile
        want += min(ntile, ndiag + 1)
    swept, of = tc.tolist()
    assert of == H * full
    ragged = T % 128 != 0                        # the last block, whose band may be one tile: a trip more
    assert H * want <= swept <= H * (want + 2 * ragged), (swept, H * want)


def mixed_grouped(gen, B, H, Hkv, T, d, seed):
    """kv heads by turns as in mixed(); of the query heads on a far one every second is near all the same."""
    qk, k, v = mixed(gen, B, Hkv, T, d, seed)
    q, _, _, g = gen.gaussian(B, H, T, d, seed=seed + 5, dtype="bf16", with_dout=True)
    q, G = q.clone(), H // Hkv
    for h in range(2, Hkv, 3):
        q[:, h * G:(h + 1) * G] = qk[:, h:h + 1]
        q[:, h * G + 1:(h + 1) * G:2, :, d - 1] = 0.0
    return q, k, v, g


def check_heads(got, refs):
    for name, a, r in zip(("dq", "dk", "dv", "dr"), got, refs):
        a, heads = to64(a), r.shape[-3] if name != "dr" else 1
        for h in range(heads):
            check_grad(f"{name} head {h}", a[..., h, :, :] if name != "dr" else a, r[..., h, :, :] if name != "dr" else r)


def test_mixed_grouped_reaches(gen):
    """The inputs do what the tests below need: of two query heads on one far kv head one is exhausted
    within 400 keys, the other keeps most of its stick."""
    q, k, _, _ = mixed_grouped(gen, 1, 6, 3, 600, 64, seed=1)
    sp = lambda h: np.logaddexp(0.0, to64(q[0, h, -1]) @ to64(k[0, 2]).T / 8.0)
    assert sp(4)[200:].sum() < 10.0 and sp(5)[200:].sum() > 112.0


@pytest.mark.parametrize("T", [1025, 1300])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_backward_grouped_with_bias(sb, oracle, gen, T, d):
    """Every query head of a group has a start tile of its own."""
    q, k, v, g = mixed_grouped(gen, 1, 6, 3, T, d, seed=900 + T)
    r = gen.remainder_embedding(6, d, seed=3)
    qd, kd, vd, gd, rd = dev(q, k, v, g, r)
    o, m = sb.sb_attn_fwd_gqa(qd, kd, vd, r=rd)
    got = sb.sb_attn_bwd_gqa(qd, kd, vd, m, gd, r=rd, workspace=nan_bytes(sb.sb_attn_bwd_workspace_bytes(1, 6, T, d)))
    torch.cuda.synchronize()
    q64, k64, v64, g64, r64 = (to64(t) for t in (q, k, v, g, r))
    ref, rem = oracle.fwd_gqa(q64, k64, v64, r=r64)
    assert np.all(np.abs(to64(o) - ref) <= fwd_bound(ref, v64))
    check_m(to64(m), rem)
    check_heads(got, oracle.bwd_gqa(q64, k64, v64, g64, r=r64))


@pytest.mark.parametrize("lens,max_T", [([1100, 40, 0, 1300, 513], 1300), ([700, 1025], 1725)])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_backward_packed(sb, oracle, gen, lens, max_T, d):
    """Start tiles of sequences that lie one behind the other, also with a bound that is too long."""
    H, Hkv, Ttot = 6, 3, sum(lens)
    q, k, v, g = (t[0] for t in mixed_grouped(gen, 1, H, Hkv, Ttot, d, seed=950 + d))
    r = gen.remainder_embedding(H, d, seed=4)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    qd, kd, vd, gd, rd = dev(q, k, v, g, r)
    cud = torch.from_numpy(cu).cuda()
    o, m = sb.sb_attn_varlen_fwd(qd, kd, vd, cud, max_T, r=rd)
    ws = nan_bytes(sb.sb_attn_varlen_bwd_workspace_bytes(len(lens), H, Ttot, max_T, d))
    got = sb.sb_attn_varlen_bwd(qd, kd, vd, m, gd, cud, max_T, r=rd, workspace=ws)
    torch.cuda.synchronize()
    q64, k64, v64, g64, r64 = (to64(t) for t in (q, k, v, g, r))
    ref, rem = oracle.fwd_varlen(q64, k64, v64, cu, r=r64)
    assert np.all(np.abs(to64(o) - ref) <= fwd_bound(ref, v64))
    check_m(to64(m), rem)
    check_heads(got, oracle.bwd_varlen(q64, k64, v64, g64, cu, r=r64))


@pytest.mark.parametrize("B,H,Hkv,T", [(8, 16, 16, 640), (8, 16, 16, 1025), (16, 16, 8, 700), (2, 20, 20, 1000), (1, 32, 32, 1100)])
def test_backward_of_many_heads(sb, oracle, gen, B, H, Hkv, T):
    """d = 128: from 128 kv heads on blocks in pairs; 320 and 288 blocks of 128 keys, more than CUs but
    short heads; heads of all reaches at both ends of the grid."""
    d = 128
    q, k, v, g = mixed_grouped(gen, B, H, Hkv, T, d, seed=1000 + T)
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_fwd_gqa(qd, kd, vd)
    got = sb.sb_attn_bwd_gqa(qd, kd, vd, m, gd, workspace=nan_bytes(sb.sb_attn_bwd_workspace_bytes(B, H, T, d)))
    torch.cuda.synchronize()
    G = H // Hkv
    for b, h in ((0, 0), (0, 1), (0, 2), (B // 2, 2), (B - 1, Hkv - 2), (B - 1, Hkv - 1)):
        qs, ks = slice(h * G, (h + 1) * G), slice(h, h + 1)
        one = oracle.bwd_gqa(*(to64(t) for t in (q[b:b + 1, qs], k[b:b + 1, ks], v[b:b + 1, ks], g[b:b + 1, qs])))
        check_heads((got[0][b:b + 1, qs], got[1][b:b + 1, ks], got[2][b:b + 1, ks]), one)


@pytest.mark.parametrize("T", [300, 385, 895, 960])
def test_second_block_of_a_pair(sb, oracle, gen, T):
    """d = 128, 128 heads in whole rounds of pairs: the second block is fetched while the first ends, after 15, 13,
    11, ... tiles of 64 rows; with a block of one row, with rows past the end, with a middle block alone."""
    B, H, d = 8, 16, 128
    q, k, v = mixed(gen, B, H, T, d, seed=2000 + T)
    g = gen.gaussian(B, H, T, d, seed=2001 + T, dtype="bf16")[0]
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_fwd_train(qd, kd, vd)
    got = sb.sb_attn_bwd(qd, kd, vd, m, gd, workspace=nan_bytes(sb.sb_attn_bwd_workspace_bytes(B, H, T, d)))
    torch.cuda.synchronize()
    for b, h in ((0, 0), (0, 1), (0, 2), (3, 5), (7, 15)):
        one = oracle.bwd(*(to64(t[b:b + 1, h:h + 1]) for t in (q, k, v, g)))
        check_heads([t[b:b + 1, h:h + 1] for t in got], one)


@pytest.mark.parametrize("T", [449, 513, 700, 1057])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_starts_of_all_distances(sb, oracle, gen, T, d):
    """Heads whose rows are exhausted after 4 strips of 32 keys, 5, ... up to more than there are: the search for
    the backward's start finds it in each of its steps, at its limit, and not at all."""
    B, H = 1, 64
    q, k, v, g = (gen.gaussian(B, H, T, d, seed=3000 + T + i, dtype="bf16")[0].clone() for i in range(4))
    for h in range(H):
        f = (4.0 * h / H * d ** 0.5) ** 0.5                 # logits shifted by 0 ... -4
        q[:, h, :, d - 1], k[:, h, :, d - 1] = f, -f
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_fwd_train(qd, kd, vd)
    got = sb.sb_attn_bwd(qd, kd, vd, m, gd, workspace=nan_bytes(sb.sb_attn_bwd_workspace_bytes(B, H, T, d)))
    torch.cuda.synchronize()
    for h in range(0, H, 6):
        one = oracle.bwd(*(to64(t[:, h:h + 1]) for t in (q, k, v, g)))
        check_heads([t[:, h:h + 1] for t in got], one)
