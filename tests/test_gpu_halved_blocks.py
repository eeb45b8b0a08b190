"""Launches a little above whole rounds of 256 blocks of 128, whose last blocks are taken in halves: one to 128 of them and
one more (not halved), ragged ends in either half, lists of 0 entries, of one (a group without any), of a few and of all
blocks, the token rule, against float64."""
import numpy as np
import pytest

from test_gpu_list_split import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H, nb, cut", [(1, 257, 1), (5, 53, 100), (8, 33, 33), (6, 64, 0), (5, 77, 64), (8, 65, 127), (13, 20, 63), (20, 26, 65)])
@pytest.mark.parametrize("rule", [False, True])
def test_forward_and_backward_match_float64(D, H, nb, cut, rule):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"D={D} H={H} nb={nb} cut={cut} rule={rule}", flush=True)
    block, N = 128, 128 * nb - cut
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, do = (torch.randn((1, N, H, D), device="cuda", generator=g).bfloat16().transpose(1, 2) for _ in range(4))
    scale = D ** -0.5
    if rule:
        frames, s = N // 150, 150
        m = rb.radial_mask_build(frames, s, block, 1, rb.RADIAL_MASK_TRANSPOSE | rb.RADIAL_MASK_TOKEN_EXACT, extra_tokens=N - frames * s)

        def visible(rows):
            pos = torch.arange(N, device="cuda")
            fr, text = pos // s, pos >= frames * s
            at = pos - fr * s
            d = (fr[rows, None] - fr[None]).abs()
            b = 2 ** torch.floor(torch.log2(d.clamp(min=1).double())).long()
            w = s // b
            near = torch.where(w >= 1, (at[rows, None] - at[None]).abs() <= w - 1, (at[rows, None] == at[None]) & (d % (-(-b // s)) == 0))
            return near | (fr < 1)[None] | text[None] | text[rows, None]
    else:
        rng = np.random.default_rng(N)
        lists = [np.sort(rng.choice(nb, size=(nb if r == 3 else (9, 0, 1, 4, 5)[r % 5]), replace=False)) for r in range(nb)]
        row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in lists])]).astype(np.int32)
        m = rb.radial_mask_from_csr(N, block, row_ptr, np.concatenate(lists).astype(np.int32), rb.RADIAL_MASK_TRANSPOSE)
        bm = torch.zeros((nb, nb), dtype=torch.bool)
        for r, c in enumerate(lists):
            bm[r, c.astype(np.int64)] = True
        bm = bm.cuda()

        def visible(rows):
            return bm[rows // block].repeat_interleave(block, 1)[:, :N]
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    for h in {0, H - 1}:
        K, V = k[0, h].double(), v[0, h].double()
        rk, rv, some = torch.zeros_like(K), torch.zeros_like(V), torch.zeros(N, dtype=torch.bool, device="cuda")
        ro, rl, rq = torch.zeros_like(K), torch.zeros(N, dtype=torch.float64, device="cuda"), torch.zeros_like(K)
        for r0 in range(0, N, 4096):  # rows in parts: the score matrix of all of them is large
            rows = torch.arange(r0, min(N, r0 + 4096), device="cuda")
            vis = visible(rows)
            o, l, a, b, c = reference(q[0, h, rows], K, V, do[0, h, rows], vis, scale)
            some[rows] = vis.any(1)
            ro[rows], rl[rows], rq[rows] = o, l, a
            rk += b
            rv += c
        assert (lse[0, h][~some] == float("-inf")).all() and (out[0, h][~some] == 0).all()
        # lse is float32; out and the gradients carry two to three bf16 roundings (2^-9 each, of P or dS, of the result, and
        # of out inside delta)
        assert (lse[0, h][some].double() - rl[some]).abs().max() <= 1e-4
        for name, x, r in (("out", out[0, h], ro), ("dq", dq[0, h], rq), ("dk", dk[0, h], rk), ("dv", dv[0, h], rv)):
            assert torch.isfinite(x).all(), (name, h)
            assert (x.double() - r).norm() <= 8e-3 * r.norm() + 1e-6, (name, h, (x.double() - r).norm() / r.norm())
    m.free()
