"""Calls whose work takes more threads than one HIP launch holds (2^32): they go out as several."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2410_17980_amd import binding
    binding.load(build_if_missing=False)
    return binding


def test_f32_rows(sb):
    """2^27 rows, 16 to a workgroup of 512 threads: exactly one launch more than fits."""
    H, T, d = 1 << 23, 16, 32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    x = torch.randn(1, H, T, d, generator=gen, device="cuda")
    o = torch.full_like(x, float("nan"))
    sb.sb_attn_fwd_f32(x, x, x, o=o)
    assert torch.isfinite(o).all()
    for h in (0, H // 2 - 1, H // 2, H - 9, H - 2):
        y = x[:, h:h + 2].contiguous()
        assert torch.equal(o[:, h:h + 2], sb.sb_attn_fwd_f32(y, y, y)), h


@pytest.mark.parametrize("d", [32, 128])
def test_packed_blocks(sb, d):
    """2^16 sequences of one row and one of 2^14, two heads: over 2^24 blocks of 256 threads.  The long
    sequence, last in the batch, as if it were alone; the others have nothing to attend to."""
    H, n1, T = 2, 1 << 16, 1 << 14
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    q, k, v, g = (torch.randn(H, n1 + T, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    q[1, :, d - 1], k[1, :, d - 1] = 4.0, -0.375 * d ** 0.5 * 4.0       # one head with logits around -6: reaches far
    r = torch.randn(H, d, generator=gen, device="cuda").to(torch.bfloat16)
    cu = torch.arange(n1 + 2, dtype=torch.int32, device="cuda")
    cu[-1] = n1 + T
    one = [x[:, n1:].contiguous()[None] for x in (q, k, v, g)]
    o, m = sb.sb_attn_varlen_fwd(q, k, v, cu, T, r=r)
    o1, m1 = sb.sb_attn_fwd_rb(*one[:3], r)
    assert torch.equal(o[:, n1:], o1[0]) and torch.equal(m[:, n1:], m1[0])
    assert torch.equal(o[:, :n1], r[:, None].expand(H, n1, d)) and not m[:, :n1].any()
    grads = sb.sb_attn_varlen_bwd(q, k, v, m, g, cu, T, r=r)
    alone = sb.sb_attn_bwd_rb(*one[:3], r, m1, one[3])
    for name, a, b in zip(("dq", "dk", "dv"), grads, alone):
        assert not a[:, :n1].any(), name
        # other kernel variants for the two calls: sums in another order
        assert (a[:, n1:] - b[0]).norm() <= 1e-4 * b.norm(), name
    dr = (m.double().exp()[..., None] * g.double()).sum(1)
    assert (grads[3] - dr).norm() <= 1e-4 * dr.norm()
