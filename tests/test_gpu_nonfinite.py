"""NaN and infinities in the inputs reach every result that weighs them.  Through a zero weight (masked
inside the 32 x 32 strip on the diagonal, or of a row that has used up its stick) they may or may not:
such a row is either spoilt or exactly what it is without them."""
import pytest
import torch

from helpers import dev

pytestmark = pytest.mark.gpu

T, AT = 1500, 700
STRIP = AT // 32 * 32                                            # first row of the strip on the diagonal


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


def heads(gen, d, seed=3):
    """A head that is exhausted within some 140 keys and one that never is."""
    q, k, v, g = gen.gaussian(1, 2, T, d, seed=seed, dtype="bf16", with_dout=True)
    qb, kb, _ = gen.biased_gaussian(1, 2, T, d, seed=seed, shift=-6.0, dtype="bf16")
    q, k = q.clone(), k.clone()
    q[:, 1], k[:, 1] = qb[:, 1], kb[:, 1]
    return dev(q, k, v, g)


def rows(x):
    return x.reshape(2, T, -1)


def check(clean, spoilt, reach, rounding=0.0):
    """rows before the strip as they were; behind AT `reach` rows spoilt at least (head 1: all); the others either way"""
    clean, spoilt = rows(clean), rows(spoilt)
    bad = ~torch.isfinite(spoilt).all(-1)
    same = ((clean - spoilt).abs().float() <= rounding * (1.0 + clean.abs().float())).all(-1)
    assert same[:, :STRIP].all()
    assert bad[0, AT + 1:AT + 1 + reach].all() and bad[1, AT + 1:].all()
    assert (bad | same).all()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward(sb, gen, d, value):
    q, k, v, _ = heads(gen, d)
    o, m = sb.sb_attn_fwd_train(q, k, v)
    vx = v.clone()
    vx[:, :, AT, 5] = value
    check(o, sb.sb_attn_fwd(q, k, vx), 8)
    ox, mx = sb.sb_attn_fwd_train(q, k, vx)
    check(o, ox, 8)
    assert torch.equal(m, mx)
    # a NaN among a wave's logits sends its other rows into the log form too: other roundings of weights and o
    kx = k.clone()
    kx[:, :, AT] = float("nan")
    check(o, sb.sb_attn_fwd(q, kx, v), 8, rounding=2.0 ** -7)
    ox, mx = sb.sb_attn_fwd_train(q, kx, v)
    check(o, ox, 8, rounding=2.0 ** -7)
    assert torch.allclose(m[:, :, :AT + 1], mx[:, :, :AT + 1], rtol=1e-4, atol=1e-3)
    assert (mx[:, :, AT + 1:] < m[:, :, AT + 1:] - 80.0).all()      # a NaN logit counts as 128 in base 2


@pytest.mark.parametrize("d", [32, 64, 128])
def test_backward(sb, gen, d):
    """A row of dout that is not finite spoils its row of dq, and dk and dv of the keys that it weighs."""
    q, k, v, g = heads(gen, d)
    r = gen.remainder_embedding(2, d, seed=4).cuda()
    _, m = sb.sb_attn_fwd_rb(q, k, v, r)
    gx = g.clone()
    gx[:, :, AT, 5] = float("nan")
    clean, spoilt = sb.sb_attn_bwd_rb(q, k, v, r, m, g), sb.sb_attn_bwd_rb(q, k, v, r, m, gx)
    bad = ~torch.isfinite(rows(spoilt[0])).all(-1)
    assert bad[:, AT].all() and not bad[:, :AT].any() and not bad[:, AT + 1:].any()
    for a, b in zip(clean[1:3], spoilt[1:3]):
        bad = ~torch.isfinite(rows(b)).all(-1)
        assert bad[0, AT - 8:AT].all() and bad[1, :AT].all() and not bad[:, STRIP + 32:].any()
        assert (bad | (rows(a) == rows(b)).all(-1)).all()
    assert torch.isfinite(spoilt[3][:, :5]).all() and not torch.isfinite(spoilt[3][1, 5])   # head 0: exp(m) is zero there


@pytest.mark.parametrize("want_m", [False, True])
def test_decode(sb, gen, want_m):
    q, k, v, _ = heads(gen, 64)
    k, v = (torch.cat([t, t], 2) for t in (k, v))                # beyond what one launch takes
    qn = q[:, :, -1].contiguous()
    call = lambda vv: sb.sb_attn_decode(qn, k, vv, want_m=want_m)
    o = call(v)
    for at, reach in ((2 * T - 2, (0, 1)), (AT, (1,))):
        vx = v.clone()
        vx[:, :, at, 5] = float("nan")
        ox = call(vx)
        (a, m), (b, mx) = (o, ox) if want_m else ((o, None), (ox, None))
        assert m is None or torch.equal(m, mx)
        for h in (0, 1):
            assert not torch.isfinite(b[0, h, 5]) or (h not in reach and torch.equal(a[0, h], b[0, h]))
            assert torch.equal(a[0, h, :5], b[0, h, :5]) and torch.equal(a[0, h, 6:], b[0, h, 6:])


class Many:
    """The library with every call's two heads `times` over, so that a call takes the kernels of larger grids: results of
    the first two, those of the last two the same bit for bit."""
    def __init__(self, sb, times):
        self.sb, self.times = sb, times

    def __getattr__(self, name):
        def call(*tensors):
            out = getattr(self.sb, name)(*(t.repeat(*((self.times, 1) if t.dim() == 2 else (1, self.times) + (1,) * (t.dim() - 2))) for t in tensors))
            return tuple(map(self.two, out)) if isinstance(out, tuple) else self.two(out)
        return call

    def two(self, x):
        heads = (lambda a, b: x[a:b]) if x.dim() == 2 else (lambda a, b: x[:, a:b].contiguous())
        first, last = heads(None, 2), heads(-2, None)
        assert torch.equal(first.isfinite(), last.isfinite()) and torch.equal(first.nan_to_num(), last.nan_to_num())
        return first


# (d, times over, key-stationary pass); the other passes take blocks of 128 rows.  test_routes.py asks the library's rules
GRIDS = [(32, 9, "two groups"), (32, 22, "one group"), (64, 9, "two groups"), (64, 22, "one group"),
         (128, 9, "64 keys"), (128, 17, "128 keys"), (128, 64, "pairs")]


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward_blocks(sb, gen, d, value):
    test_forward(Many(sb, GRIDS[0][1]), gen, d, value)


@pytest.mark.parametrize("d,times", [g[:2] for g in GRIDS])
def test_backward_blocks(sb, gen, d, times):
    test_backward(Many(sb, times), gen, d)
