"""The library launches kernels on the caller's stream and nothing else (no allocation, no
memset, no synchronisation), so a training step or a decode call can be captured in a HIP
graph.  Replays are checked against the eager results, with eager work between them."""
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
def gen():
    from paper_2410_17980_amd import inputs
    return inputs


def test_training_step_in_a_graph(sb, gen):
    B, H, T, d = 2, 4, 700, 128
    q, k, v, g = dev(*gen.gaussian(B, H, T, d, seed=1, sharp_half=True, with_dout=True))
    r = gen.remainder_embedding(H, d, seed=2).cuda()
    o = torch.empty_like(q)
    m = torch.empty(B, H, T, dtype=torch.float32, device="cuda")
    dq, dk, dv = (torch.empty(B, H, T, d, dtype=torch.float32, device="cuda") for _ in range(3))
    dr = torch.empty(H, d, dtype=torch.float32, device="cuda")
    ws = torch.empty(sb.sb_attn_bwd_workspace_bytes(B, H, T, d), dtype=torch.uint8, device="cuda")

    def step():
        sb.sb_attn_fwd_rb(q, k, v, r, o=o, m=m)
        sb.sb_attn_bwd_rb(q, k, v, r, m, g, dq=dq, dk=dk, dv=dv, dr=dr, workspace=ws)

    step()
    torch.cuda.synchronize()
    want = [t.clone() for t in (o, m, dq, dk, dv, dr)]

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()                                   # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for rep in range(3):
        for t in (o, m, dq, dk, dv, dr):
            t.fill_(float("nan") if t.is_floating_point() else 0)
        ws.random_(0, 255)                       # the workspace's previous contents must not matter
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name, a, b in zip(("o", "m", "dq", "dk", "dv", "dr"), (o, m, dq, dk, dv, dr), want):
            assert torch.equal(a, b), f"replay {rep}: {name} differs from the eager result"
        sb.sb_attn_fwd(q, k, v)                  # eager work between the replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("B,H,Hkv,T,d", [(1, 12, 3, 462, 128), (1, 24, 3, 1500, 128), (1, 38, 19, 2000, 128), (1, 120, 30, 1665, 64)])
def test_parts_of_grouped_heads_in_a_graph(sb, B, H, Hkv, T, d):
    """Plans of more than one part (test_gpu_parts.py), whose counts every replay finds as something left them."""
    from test_gpu_exhausted import mixed_grouped
    from paper_2410_17980_amd import inputs
    q, k, v, g = dev(*mixed_grouped(inputs, B, H, Hkv, T, d, seed=T + d))
    _, m = sb.sb_attn_fwd_gqa(q, k, v)
    out = [torch.empty(x.shape, dtype=torch.float32, device="cuda") for x in (q, k, v)]
    ws = torch.empty(sb.sb_attn_bwd_gqa_workspace_bytes(B, H, Hkv, T, d), dtype=torch.uint8, device="cuda")

    def step():
        sb.sb_attn_bwd_gqa(q, k, v, m, g, dq=out[0], dk=out[1], dv=out[2], workspace=ws)

    step()
    torch.cuda.synchronize()
    want = [t.clone() for t in out]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for rep in range(3):
        for t in out:
            t.fill_(float("nan"))
        ws.random_(0, 255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name, a, b in zip(("dq", "dk", "dv"), out, want):
            assert torch.equal(a, b), f"replay {rep}: {name} differs from the eager result"


def test_decode_in_a_graph(sb, gen):
    B, H, Hkv, T, d = 2, 8, 2, 3000, 128
    q, _, _ = gen.gaussian(B, H, 1, d, seed=3)
    _, k, v = gen.gaussian(B, Hkv, T, d, seed=4)
    q, k, v = dev(q[:, :, 0].contiguous(), k, v)
    o = torch.empty_like(q)
    ws = torch.empty(sb.load().sb_attn_decode_workspace_bytes(B, H, T, d), dtype=torch.uint8, device="cuda")
    sb.sb_attn_decode(q, k, v, o=o, workspace=ws)
    torch.cuda.synchronize()
    want = o.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sb.sb_attn_decode(q, k, v, o=o, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        sb.sb_attn_decode(q, k, v, o=o, workspace=ws)
    for rep in range(3):
        o.zero_()
        ws.random_(0, 255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, want), f"replay {rep}"


def test_workspace_lives_as_long_as_the_stream_needs_it(sb, gen):
    """A call on a stream of its own returns before its kernels have run, and gives its workspace back to
    torch's allocator: what the current stream allocates and writes meanwhile must be other memory."""
    B, H, T, d = 1, 4, 700, 64
    q, k, v, g = dev(*gen.gaussian(B, H, T, d, seed=5, with_dout=True))
    qd, _, _ = dev(*gen.gaussian(B, H, 1, d, seed=6))
    kd, vd = (t.expand(4, H, T, d).transpose(0, 1).reshape(B, H, 4 * T, d).contiguous() for t in (k, v))
    qd = qd[:, :, 0].contiguous()
    cu = torch.tensor([0, 300, T], dtype=torch.int32, device="cuda")
    one = [t[0].contiguous() for t in (q, k, v, g)]
    o, m = sb.sb_attn_fwd_train(q, k, v)
    _, mp = sb.sb_attn_varlen_fwd(*one[:3], cu, 400)
    side = torch.cuda.Stream()
    calls = ((sb.sb_attn_bwd_workspace_bytes(B, H, T, d), lambda **kw: sb.sb_attn_bwd(q, k, v, m, g, **kw)),
             (sb.sb_attn_varlen_bwd_workspace_bytes(2, H, T, 400, d),
              lambda **kw: sb.sb_attn_varlen_bwd(*one[:3], mp, one[3], cu, 400, **kw)),
             (sb.load().sb_attn_decode_workspace_bytes(B, H, 4 * T, d),
              lambda **kw: (sb.sb_attn_decode(qd, kd, vd, **kw),)))
    for need, call in calls:
        want = call()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            torch.cuda._sleep(200_000_000)       # about 0.1 s: the call's kernels wait behind it
        got = call(stream=side)
        for _ in range(4):
            torch.empty(need, dtype=torch.uint8, device="cuda").fill_(0xFF)
        torch.cuda.synchronize()
        segment = [s for s in torch.cuda.memory_snapshot() if s["stream"] == side.cuda_stream]
        assert sum(s["total_size"] for s in segment) >= need
        for a, b in zip(got, want):
            assert torch.equal(a, b)
