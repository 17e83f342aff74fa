"""The backward's kernels for blocks of 128 rows against the oracle: grids just beyond those that take a strip
of 32 rows a workgroup, with the kernels named in block_shapes.py (checked against the library's rules in
test_routes.py).  Heads by turns near, sharp and far, some of them compared; the workspace reads as NaN where nothing
was written.  Tolerances as in test_gpu_backward.py, see check() for the one addition."""
import numpy as np
import pytest
import torch

import block_shapes
from helpers import GRAD_REL, check_grad, check_m, dev, fwd_bound, nan_bytes, to64
from test_gpu_exhausted import gen, mixed, mixed_grouped, sb  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def some(Hkv):
    """kv heads of every kind at both ends of the grid and in its middle."""
    return sorted({0, 1, 2, Hkv // 2, Hkv - 2, Hkv - 1} & set(range(Hkv)))


def rounding_of_dz(q, k, v, g, r):
    """2^-8 |dZ| |K| / sqrt(d) and 2^-8 |dZ|^T |Q| / sqrt(d) of one head: the most that rounding every dZ to bf16
    (half a unit of its 8 bits) moves an entry of dq and of dk."""
    T, d = q.shape
    z = q @ k.T / np.sqrt(d)
    seen = np.tril(np.ones((T, T), dtype=bool), -1)
    sp = np.where(seen, np.logaddexp(0.0, z), 0.0)
    G = np.where(seen, np.exp(z - np.cumsum(sp[:, ::-1], 1)[:, ::-1]), 0.0) * (g @ v.T)
    left = np.cumsum(G, 1) + (np.exp(-sp.sum(1)) * (g @ r))[:, None] if r is not None else np.cumsum(G, 1)
    dz = np.abs(np.where(seen, G - left / (1.0 + np.exp(-z)), 0.0)) * 2.0 ** -8 / np.sqrt(d)
    return dz @ np.abs(k), dz.T @ np.abs(q)


def check(name, got, ref, bound):
    """check_grad, or element by element the bound that bound() derives: far heads have one column of q and of k in
    which all entries are alike (5.8 in size at d = 32), where the roundings of dZ add up while the dZ themselves
    cancel.  At H24 Hkv8 T1300 d32, head 7, rounding a float64 dZ moves dq by 0.02137 with the largest entry at 5.247
    (2^-8 of it 0.0205)."""
    try:
        check_grad(name, got, ref)
    except AssertionError:
        if bound is None or not np.all(np.isfinite(got)):
            raise
        assert np.all(np.abs(got - ref) <= bound() + GRAD_REL * np.abs(ref)), name


def compare(oracle, got, q, k, v, g, r, cu=None):
    """got, all on the host: dq, dk, dv[, dr] of [B, H, T, d], or of a packed [H, Ttot, d] with offsets."""
    if cu is not None:
        q, k, v, g, got = q[None], k[None], v[None], g[None], [t[None] for t in got[:3]] + list(got[3:])
    B, Hkv, G = k.shape[0], k.shape[1], q.shape[1] // k.shape[1]
    for b, h in {(b, h) for b in (0, B - 1) for h in some(Hkv)}:
        s, t = slice(h * G, (h + 1) * G), slice(h, h + 1)
        one = [to64(x[b:b + 1, y]) for x, y in ((q, s), (k, t), (v, t), (g, s))]
        r64 = to64(r[s]) if r is not None else None
        ref = oracle.bwd_gqa(*one, r=r64) if cu is None else [x[None] for x in oracle.bwd_varlen(*(x[0] for x in one), cu, r=r64)]
        spans = [slice(0, one[0].shape[2])] if cu is None else [slice(x, y) for x, y in zip(cu[:-1], cu[1:]) if y > x]

        def bound(heads, which):
            out = np.zeros(one[0].shape[2:])
            for n in spans:
                for i in heads:
                    out[n] += rounding_of_dz(one[0][0, i, n], one[1][0, 0, n], one[2][0, 0, n], one[3][0, i, n], r64[i] if r is not None else None)[which]
            return out
        for i in range(G):
            check(f"dq[{b}] kv head {h}, {i}", to64(got[0][b, h * G + i]), ref[0][0, i], lambda: bound([i], 0))
        check(f"dk[{b}] kv head {h}", to64(got[1][b, h]), ref[1][0, 0], lambda: bound(range(G), 1))
        check(f"dv[{b}] kv head {h}", to64(got[2][b, h]), ref[2][0, 0], None)
        if r is not None and B == 1:
            check_grad(f"dr kv head {h}", to64(got[3][s]), ref[3] if cu is None else ref[3][0])


def batched(sb, gen, oracle, shape, bias=False, inputs=None):
    B, H, Hkv, T, d = shape[:5]
    Hkv = Hkv or H
    q, k, v, g = inputs or mixed_grouped(gen, B, H, Hkv, T, d, seed=4000 + T + d)
    r = gen.remainder_embedding(H, d, seed=5) if bias else None
    qd, kd, vd, gd = dev(q, k, v, g)
    rd = r.cuda() if bias else None
    _, m = sb.sb_attn_fwd_gqa(qd, kd, vd, r=rd)
    got = sb.sb_attn_bwd_gqa(qd, kd, vd, m, gd, r=rd, workspace=nan_bytes(sb.sb_attn_bwd_workspace_bytes(B, H, T, d)))
    compare(oracle, [t.cpu() for t in got], q, k, v, g, r)


@pytest.mark.parametrize("shape", block_shapes.LOOPS, ids=block_shapes.name)
def test_loop_boundaries(sb, oracle, gen, shape):
    batched(sb, gen, oracle, shape)


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("shape", block_shapes.LONG + block_shapes.GROUPED, ids=block_shapes.name)
def test_starts_and_groups(sb, oracle, gen, shape, bias):
    batched(sb, gen, oracle, shape, bias)


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("shape", block_shapes.PACKED + block_shapes.ALIKE, ids=block_shapes.name)
def test_packed(sb, oracle, gen, shape, bias):
    B, H, Hkv, max_T, d, lens = shape[:6]
    Ttot = sum(lens)
    q, k, v, g = (t[0] for t in mixed_grouped(gen, 1, H, Hkv, Ttot, d, seed=5000 + d))
    r = gen.remainder_embedding(H, d, seed=6) if bias else None
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    qd, kd, vd, gd, cud = dev(q, k, v, g, torch.from_numpy(cu))
    rd = r.cuda() if bias else None
    o, m = sb.sb_attn_varlen_fwd(qd, kd, vd, cud, max_T, r=rd)
    ws = nan_bytes(sb.sb_attn_varlen_bwd_workspace_bytes(B, H, Ttot, max_T, d))
    got = sb.sb_attn_varlen_bwd(qd, kd, vd, m, gd, cud, max_T, r=rd, workspace=ws)
    compare(oracle, [t.cpu() for t in got], q, k, v, g, r, cu)
    G = H // Hkv
    for h in some(Hkv):
        s = slice(h * G, (h + 1) * G)
        ref, rem = oracle.fwd_varlen(to64(q[s]), to64(k[h:h + 1]), to64(v[h:h + 1]), cu, r=to64(r[s]) if bias else None)
        assert np.all(np.abs(to64(o[s]) - ref) <= fwd_bound(ref, to64(v)))
        check_m(to64(m[s]), rem)


def random_shapes():
    rng = np.random.default_rng(20241018)
    out = []
    for i in range(18):
        d, T = int(rng.choice([32, 64, 128])), int(rng.integers(65, 641))
        limit = 256 if d == 128 or T <= 341 else 3 * T // 4
        H = block_shapes.above(limit, block_shapes.strips(T)) + int(rng.integers(0, 40))
        out.append((1, H, H, T, d, None, ("plain", "sharp", "biased")[i % 3]))
    return out


@pytest.mark.parametrize("shape", random_shapes(), ids=lambda s: "H%d_T%d_d%d_%s" % (s[1], s[3], s[4], s[6]))
def test_random_shapes(sb, oracle, gen, shape):
    B, H, _, T, d, _, kind = shape
    g = gen.gaussian(B, H, T, d, seed=6001 + T, dtype="bf16", with_dout=True)[3]
    if kind == "sharp":
        q, k, v = gen.scaled_gaussian(B, H, T, d, seed=6000 + T, gain=8.0, dtype="bf16")
    elif kind == "biased":
        q, k, v = gen.biased_gaussian(B, H, T, d, seed=6000 + T, shift=-5.0, dtype="bf16")
    else:
        q, k, v = gen.gaussian(B, H, T, d, seed=6000 + T, dtype="bf16")
    batched(sb, gen, oracle, shape, inputs=(q, k, v, g))


@pytest.mark.parametrize("H,d", [(19, 64), (48, 64), (19, 32), (7, 128), (28, 128)])
def test_far_queries_come_back(sb, oracle, gen, H, d):
    """Rows 1024..1151 reach all keys, the rows before them only near ones: the query blocks that
    reach a key block are not contiguous."""
    T = 1300
    q, k, v, g = gen.gaussian(1, H, T, d, seed=8, dtype="bf16", with_dout=True)
    q, k = q.clone(), k.clone()
    q[..., 0], k[..., 0] = 0.0, -4.0
    q[..., 1024:1152, :] *= 0.25
    q[..., 1024:1152, 0] = 2.0 * d ** 0.5
    batched(sb, gen, oracle, (1, H, H, T, d), inputs=(q, k, v, g))


@pytest.mark.parametrize("H,T,d", [(24, 333, 128), (66, 449, 64), (30, 1300, 32), (128, 449, 128)])
def test_split_passes_equal_the_whole(sb, gen, H, T, d):
    """sb_attn_bwd_dq followed by sb_attn_bwd_dkdv on one workspace is sb_attn_bwd, bit for bit."""
    q, k, v, g = dev(*mixed_grouped(gen, 1, H, H, T, d, seed=21))
    _, m = sb.sb_attn_fwd_train(q, k, v)
    want = sb.sb_attn_bwd(q, k, v, m, g)
    dq, ws = sb.sb_attn_bwd_dq(q, k, v, m, g)
    for a, b in zip((dq, *sb.sb_attn_bwd_dkdv(q, k, v, g, ws)), want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("T", [257, 320, 353, 385, 449, 577, 641, 1283])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward_and_m_of_short_tails(sb, oracle, gen, T, d):
    """The lengths and the bound on m of test_gpu_exhausted.py, where the forward takes blocks of 128 rows."""
    H = block_shapes.above(512, block_shapes.strips(T))
    q, k, v = mixed(gen, 1, H, T, d, seed=900 + T)
    o, m = sb.sb_attn_fwd_train(*dev(q, k, v))
    for h in some(H):
        q64, k64, v64 = (to64(t[0, h]) for t in (q, k, v))
        ref = -np.tril(np.logaddexp(0.0, q64 @ k64.T / np.sqrt(d)), -1).sum(-1)
        assert np.all(np.abs(to64(m[0, h]) - ref) <= 1e-4 + 1e-5 * np.abs(ref))
        ref, _ = oracle.fwd(q64, k64, v64)
        assert np.all(np.abs(to64(o[0, h]) - ref) <= fwd_bound(ref, v64))
