"""Calls on a stream= of their own: what they allocate belongs to that stream, and is not handed on
while the stream that was current, or the call's own, still has work that uses it."""
import pytest
import torch

from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2410_17980_amd import binding
    binding.load(build_if_missing=False)
    return binding


@pytest.fixture(scope="module")
def calls(sb):
    """name -> call(stream=...) that leaves every output and workspace to the library."""
    from paper_2410_17980_amd import inputs as gen
    B, H, T, d = 1, 6, 700, 128
    q, k, v, g = dev(*gen.gaussian(B, H, T, d, seed=5, with_dout=True))
    kv = [t[:, ::3].contiguous() for t in (k, v)]
    r = gen.remainder_embedding(H, d, seed=6).cuda()
    cu = torch.tensor([0, 300, T], dtype=torch.int32, device="cuda")
    one = [t[0].contiguous() for t in (q, k, v, g)]
    qd = q[:, :, -1].contiguous()
    x = [t.float() for t in (q, k, v)]
    _, m = sb.sb_attn_fwd_train(q, k, v)
    _, mp = sb.sb_attn_varlen_fwd(*one[:3], cu, 400)
    _, mr = sb.sb_attn_fwd_gqa(q, *kv, r=r)
    _, ws = sb.sb_attn_bwd_dq(q, k, v, m, g)
    torch.cuda.synchronize()
    return {
        "fwd": lambda **kw: (sb.sb_attn_fwd(q, k, v, **kw),),
        "fwd_halt": lambda **kw: (sb.sb_attn_fwd_halt(q, k, v, 1e-6, **kw),),
        "fwd_train": lambda **kw: sb.sb_attn_fwd_train(q, k, v, **kw),
        "fwd_f32": lambda **kw: sb.sb_attn_fwd_f32(*x, want_m=True, **kw),
        "fwd_gqa": lambda **kw: sb.sb_attn_fwd_gqa(q, *kv, r=r, **kw),
        "bwd": lambda **kw: sb.sb_attn_bwd(q, k, v, m, g, **kw),
        "bwd_gqa": lambda **kw: sb.sb_attn_bwd_gqa(q, *kv, mr, g, r=r, **kw),
        "bwd_dq": lambda **kw: sb.sb_attn_bwd_dq(q, k, v, m, g, **kw),
        "bwd_dkdv": lambda **kw: sb.sb_attn_bwd_dkdv(q, k, v, g, ws, **kw),
        "varlen_fwd": lambda **kw: sb.sb_attn_varlen_fwd(*one[:3], cu, 400, **kw),
        "varlen_bwd": lambda **kw: sb.sb_attn_varlen_bwd(*one[:3], mp, one[3], cu, 400, **kw),
        "decode": lambda **kw: sb.sb_attn_decode(qd, k, v, want_m=True, **kw),
        "diag_fwd_tri": lambda **kw: sb.sb_diag_fwd_tri(q, k, v, **kw),
    }


NAMES = ("fwd", "fwd_halt", "fwd_train", "fwd_f32", "fwd_gqa", "bwd", "bwd_gqa", "bwd_dq", "bwd_dkdv", "varlen_fwd",
         "varlen_bwd", "decode", "diag_fwd_tri")
BUSY = 100_000_000        # clocks: about 0.05 s


def values(name, got):
    """The results proper: of bwd_dq's workspace only what the key-stationary pass reads is written."""
    return got[:1] if name == "bwd_dq" else got


def memory_of(stream):
    return [(s["address"], s["address"] + s["total_size"]) for s in torch.cuda.memory_snapshot() if s["stream"] == stream.cuda_stream]


@pytest.mark.parametrize("name", NAMES)
def test_outputs_do_not_take_memory_that_is_still_written(sb, calls, name):
    """Memory freed on the current stream, with a write to it still queued there, is not a result's."""
    call = calls[name]
    want = [t.clone() for t in call()]
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda._sleep(BUSY)
    for t in want:                                   # the sizes that the call will ask for
        for _ in range(3):
            torch.empty_like(t).fill_(77)
    got = call(stream=side)
    torch.cuda.synchronize()
    blocks = memory_of(side)
    for a in got:
        assert any(lo <= a.data_ptr() < hi for lo, hi in blocks)
    for a, b in zip(values(name, got), values(name, want)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("name", NAMES)
def test_dropped_outputs_wait_for_their_readers(sb, calls, name):
    """A result that is dropped while the current stream has a read of it queued is not the next call's memory."""
    call = calls[name]
    want = call()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    got = call(stream=side)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda._sleep(BUSY)
    copies = [t.clone() for t in got]
    held = {t.data_ptr() for t in got}
    del got
    again = call(stream=side)
    assert not held & {t.data_ptr() for t in again}
    torch.cuda.synchronize()
    for a, b in zip(values(name, copies), values(name, want)):
        assert torch.equal(a, b)


def test_measurements_read_their_own_stream(sb):
    """The clock of a launch on a busy stream is read after that launch, not beside it."""
    from paper_2410_17980_amd import inputs as gen
    q, k, v = dev(*gen.gaussian(1, 4, 300, 128, seed=8))
    o, m = sb.sb_attn_fwd_train(q, k, v)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(BUSY)
    assert 300.0 < sb.sb_diag_fwd_clock(q, k, v, o, m, stream=side) < 2600.0
    with torch.cuda.stream(side):
        torch.cuda._sleep(BUSY)
    assert sb.sb_diag_stream_read(torch.ones(1 << 20, device="cuda"), iters=2, stream=side) > 0.0
    tf, mhz = sb.sb_diag_mfma_rate(q.reshape(-1).repeat(8).contiguous(), iters=50, stream=side)
    assert tf > 0.0 and 300.0 < mhz < 2600.0
