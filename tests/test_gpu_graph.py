"""The attention entry points allocate nothing and take a stream, so a forward+backward step can
be captured into a HIP graph and replayed (run with -m gpu)."""
import numpy as np
import pytest
import torch

from paper_2506_19852_amd import binding as rb

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _randn_bf16(shape, seed):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return torch.randn(shape, generator=g).to(torch.bfloat16).to(DEV)


@pytest.mark.parametrize("flags", [0, rb.RADIAL_MASK_TOKEN_EXACT])
def test_forward_backward_replay_matches_eager(flags):
    f, s, block, B, H, D = 10, 160, 128, 1, 4, 128
    N = f * s
    print(f"graph replay flags={flags}", flush=True)
    scale = 1.0 / np.sqrt(D)
    mask = rb.radial_mask_build(f, s, block, 1, rb.RADIAL_MASK_TRANSPOSE | flags)
    q, k, v, do = (_randn_bf16((B, H, N, D), 90 + i) for i in range(4))
    out = torch.empty_like(q)
    lse = torch.empty((B, H, N), dtype=torch.float32, device=DEV)
    dq, dk, dv = (torch.empty_like(q) for _ in range(3))
    ws = torch.empty(rb.radial_attn_bwd_workspace(B, H, N, D, mask), dtype=torch.uint8, device=DEV)

    def step():
        rb.radial_attn_fwd(q, k, v, out, lse, mask, scale)
        rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, mask, scale, ws)

    step()                                      # warm-up outside the capture (one-time kernel attributes)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):                        # new inputs in place, replay, compare with an eager run
        for t, seed in zip((q, k, v, do), range(4)):
            t.copy_(_randn_bf16((B, H, N, D), 200 + 10 * rep + seed))
        for t in (out, dq, dk, dv):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in (out, lse, dq, dk, dv)]
        step()
        torch.cuda.synchronize()
        for a, b, nm in zip(got, (out, lse, dq, dk, dv), ("O", "LSE", "dQ", "dK", "dV")):
            assert torch.equal(a, b), f"replay {rep}: {nm} differs from the eager run"
    mask.free()


# few heads and an odd last block of text tokens; many heads
@pytest.mark.parametrize("heads, frames, tokens, extra", [(8, 17, 1000, 226), (40, 12, 1366, 0)])
def test_pairs_of_blocks_replay_matches_eager(heads, frames, tokens, extra):
    """Launches whose workgroups take two blocks each, forward (bf16 and 8-bit scores) and dK/dV."""
    from test_gpu_pair_rules import pairs_of
    print(f"graph replay of pairs H={heads} {frames}x{tokens}+{extra}", flush=True)
    N, D = frames * tokens + extra, 128
    scale = 1.0 / np.sqrt(D)
    mask = rb.radial_mask_build(frames, tokens, 128, 1, rb.RADIAL_MASK_TRANSPOSE, extra_tokens=extra)
    gen = torch.Generator(device=DEV).manual_seed(heads)
    q, k, v, do = (torch.randn((1, heads, N, D), device=DEV, generator=gen).bfloat16() for _ in range(4))
    assert pairs_of(rb, mask, q, k, v, scale)[1] > 0.5      # most blocks: this is a launch of pairs
    out, out8, dq, dk, dv = (torch.empty_like(q) for _ in range(5))
    lse, lse8 = (torch.empty((1, heads, N), dtype=torch.float32, device=DEV) for _ in range(2))
    codes = [torch.empty(q.shape, dtype=torch.uint8, device=DEV) for _ in range(2)]
    scales = [torch.empty((1, heads, -(-N // 128)), dtype=torch.float32, device=DEV) for _ in range(2)]
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, heads, N, D, mask), dtype=torch.uint8, device=DEV)
    results = (out, lse, out8, lse8, dq, dk, dv)

    def step():
        rb.radial_attn_fwd(q, k, v, out, lse, mask, scale)
        for x, c, s in zip((q, k), codes, scales):
            rb.radial_quantize_fp8(x, 128, c, s)
        rb.radial_attn_fwd_fp8(codes[0], scales[0], codes[1], scales[1], v, out8, lse8, mask, scale)
        rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, mask, scale, ws)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        for t in (q, k, v, do):
            t.copy_(torch.randn(t.shape, device=DEV, generator=gen))
        for t in results:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in results]
        step()
        torch.cuda.synchronize()
        for a, b, name in zip(got, results, ("O", "LSE", "O of 8-bit scores", "LSE of 8-bit scores", "dQ", "dK", "dV")):
            assert torch.isfinite(b).all() and torch.equal(a, b), f"replay {rep}: {name} differs from the eager run"
    mask.free()
