"""Key-stationary pass of grouped heads whose query heads are several workgroups' (key_plan() in csrc/sb_share.h), against the oracle as in
test_gpu_blocks.py, twice on one workspace, which at first reads as NaN; the plans named here are asked for in test_routes.py."""
import numpy as np
import pytest
import torch

from helpers import dev, nan_bytes
from test_gpu_blocks import compare
from test_gpu_exhausted import gen, mixed_grouped, sb  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

APART, ALIKE, LONG, HARDLY = [2, 700, 1025, 31, 129], [900, 1100, 1000, 1041], [1665, 1700, 1600, 1641], [1409, 0, 33, 1, 1280]
# B, H, Hkv, T, d, lengths or None, kernel, parts, beyond
SHAPES = [(1, 12, 3, 462, 128, None, "strips", 2, 8), (2, 8, 1, 535, 32, None, "strips", 2, 8), (1, 16, 2, 449, 64, None, "strips", 2, 8),
          (1, 24, 3, 1500, 128, None, "strips", 2, 8), (1, 24, 3, 1300, 128, None, "strips", 4, 8), (1, 9, 3, 1889, 128, None, "strips", 1, 0),
          (1, 9, 3, 1500, 128, None, "strips", 3, 8), (1, 32, 4, 1300, 64, None, "strips", 1, 0), (1, 32, 4, 1130, 64, None, "strips", 2, 8),
          (1, 32, 4, 1130, 32, None, "strips", 2, 8), (2, 8, 1, 1035, 32, None, "strips", 4, 8), (1, 16, 2, 1099, 64, None, "strips", 4, 8),
          (1, 38, 19, 2000, 128, None, "128 keys", 2, 16), (1, 120, 30, 1665, 64, None, "one group", 2, 16), (1, 96, 48, 1409, 64, None, "one group", 1, 16),
          (1, 164, 41, 1665, 32, None, "one group", 2, 16),
          (5, 16, 4, 1887, 128, APART, "strips", 1, 0), (5, 8, 1, 1887, 128, APART, "strips", 8, 8), (5, 26, 13, 1887, 128, APART, "128 keys", 2, 16),
          (5, 132, 33, 1887, 64, APART, "one group", 2, 16), (5, 164, 82, 1887, 32, APART, "one group", 1, 16), (4, 40, 4, 1100, 128, ALIKE, "strips", 1, 0),
          (4, 8, 1, 1100, 64, ALIKE, "strips", 2, 8), (4, 8, 4, 1700, 128, LONG, "128 keys", 2, 16), (4, 40, 10, 1700, 64, LONG, "one group", 2, 16),
          (4, 44, 11, 1700, 32, LONG, "one group", 2, 16), (5, 90, 30, 1409, 128, HARDLY, "128 keys", 1, 16), (5, 36, 18, 1700, 128, HARDLY, "128 keys", 2, 16)]


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%d_H%d_Hkv%d_T%d_d%d%s" % (*s[:5], "_packed" if s[5] else ""))
def test_parts(sb, oracle, gen, shape, bias):
    B, H, Hkv, T, d, lens = shape[:6]
    q, k, v, g = mixed_grouped(gen, 1 if lens else B, H, Hkv, sum(lens) if lens else T, d, seed=7000 + T + d)
    r = gen.remainder_embedding(H, d, seed=9) if bias else None
    rd, cu = r.cuda() if bias else None, None
    if lens:
        q, k, v, g = (t[0] for t in (q, k, v, g))
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        qd, kd, vd, gd, cud = dev(q, k, v, g, torch.from_numpy(cu))
        _, m = sb.sb_attn_varlen_fwd(qd, kd, vd, cud, T, r=rd)
        ws = nan_bytes(sb.sb_attn_varlen_bwd_gqa_workspace_bytes(B, H, Hkv, sum(lens), T, d))
        go = lambda w: sb.sb_attn_varlen_bwd(qd, kd, vd, m, gd, cud, T, r=rd, workspace=w)
    else:
        qd, kd, vd, gd = dev(q, k, v, g)
        _, m = sb.sb_attn_fwd_gqa(qd, kd, vd, r=rd)
        ws = nan_bytes(sb.sb_attn_bwd_gqa_workspace_bytes(B, H, Hkv, T, d))
        go = lambda w: sb.sb_attn_bwd_gqa(qd, kd, vd, m, gd, r=rd, workspace=w)
    got = go(ws)
    for a, b, c in zip(got, go(ws), go(None)):
        assert torch.equal(a, b) and torch.equal(a, c)
    compare(oracle, [t.cpu() for t in got], q, k, v, g, r, cu)


@pytest.mark.parametrize("far", [0, 71])
def test_any_head_of_a_large_group_counts(sb, gen, far):
    """72 query heads to a kv head, more than a wave has lanes, one of them far: its blocks are shared out all the same, as the counts at the end of the
    workspace say, and the sums are those of the call without parts, each of 72 heads' times 3300 queries' terms added up in another order."""
    B, H, Hkv, T, d = 1, 72, 1, 3300, 32
    q, k, v, g = gen.gaussian(B, H, T, d, seed=5, dtype="bf16", with_dout=True)
    k, v = k[:, :Hkv].clone(), v[:, :Hkv].contiguous()
    f = (6.0 * d ** 0.5) ** 0.5
    q[..., d - 1] = 0.0
    q[:, far, :, d - 1], k[..., d - 1] = f, -f
    qd, kd, vd, gd = dev(q, k, v, g)
    _, m = sb.sb_attn_fwd_gqa(qd, kd, vd)
    need = sb.sb_attn_bwd_gqa_workspace_bytes(B, H, Hkv, T, d)
    strips = (T + 31) // 32
    parts = (need - sb.sb_attn_bwd_workspace_bytes(B, H, T, d)) // (8 * B * Hkv * T * d)
    assert parts > 1
    ws = nan_bytes(need)
    got = sb.sb_attn_bwd_gqa(qd, kd, vd, m, gd, workspace=ws)
    one = sb.sb_attn_bwd_gqa(qd, kd, vd, m, gd, workspace=nan_bytes(sb.sb_attn_bwd_workspace_bytes(B, H, T, d)))
    torch.cuda.synchronize()
    counts = ws[-4 * strips:].view(torch.int32)
    assert (counts[:strips // 2] == parts).all(), counts
    assert torch.equal(got[0], one[0])
    for a, b in zip(got[1:], one[1:]):
        assert (a - b).norm() <= 1e-5 * b.norm()


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[5] is None and s[6] != "strips" and s[7] > 1], ids=lambda s: "B%d_H%d_Hkv%d_T%d_d%d" % s[:5])
def test_near_blocks_are_not_shared_out(sb, gen, shape):
    """Rows of N(0,1) reach less than a dozen strips of 32 keys: no part of their blocks ever comes to be counted."""
    B, H, Hkv, T, d = shape[:5]
    q, k, v, g = gen.gaussian(B, H, T, d, seed=6, dtype="bf16", with_dout=True)
    qd, kd, vd, gd = dev(q, k[:, :Hkv], v[:, :Hkv], g)
    _, m = sb.sb_attn_fwd_gqa(qd, kd, vd)
    ws = nan_bytes(sb.sb_attn_bwd_gqa_workspace_bytes(B, H, Hkv, T, d))
    sb.sb_attn_bwd_gqa(qd, kd, vd, m, gd, workspace=ws)
    torch.cuda.synchronize()
    assert not ws[-4 * B * Hkv * ((T + 31) // 32):].view(torch.int32).any()
