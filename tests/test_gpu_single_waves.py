"""Launches small enough for one wave per group and 32 rows per workgroup: the largest of them and one item more, rows
that end inside a wave, lists that leave groups without an entry or give one of them a whole chunk of 64, against float64."""
import numpy as np
import pytest

from test_gpu_list_split import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("block, H, N, longest", [
    (64, 1, 33, 1), (64, 2, 31 * 64 + 1, 2), (64, 1, 128 * 64 - 33, 9), (64, 1, 129 * 64, 17), (64, 1, 99 * 64, 99),
    (128, 1, 97, 1), (128, 2, 3 * 128 + 33, 4), (128, 4, 16 * 128 - 95, 16), (128, 5, 13 * 128, 13)])
@pytest.mark.parametrize("rule", [False, True])
def test_forward_and_backward_match_float64(D, block, H, N, longest, rule):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"D={D} block={block} H={H} N={N} longest={longest} rule={rule}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, do = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(4))
    q = q * 2
    nb, scale = -(-N // block), D ** -0.5
    if rule:  # frames of 70 tokens, and text: every list has at least the sink's and the text's blocks
        if N < 140:
            pytest.skip("shorter than two frames")
        frames, s = N // 70, 70
        m = rb.radial_mask_build(frames, s, block, 1, rb.RADIAL_MASK_TRANSPOSE | rb.RADIAL_MASK_TOKEN_EXACT, extra_tokens=N - frames * s)
        pos = torch.arange(N, device="cuda")
        fr, text = pos // s, pos >= frames * s
        at, d = pos - fr * s, (fr[:, None] - fr[None]).abs()
        b = 2 ** torch.floor(torch.log2(d.clamp(min=1).double())).long()
        w = s // b
        near = torch.where(w >= 1, (at[:, None] - at[None]).abs() <= w - 1, (at[:, None] == at[None]) & (d % (-(-b // s)) == 0))
        vis = near | (fr < 1)[None] | text[None] | text[:, None]
    else:
        rng = np.random.default_rng(N)
        rows = [np.sort(rng.choice(nb, size=min(nb, (longest, 0, 1, 2, longest - 1)[r % 5]), replace=False)) for r in range(nb)]
        row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
        m = rb.radial_mask_from_csr(N, block, row_ptr, np.concatenate(rows).astype(np.int32), rb.RADIAL_MASK_TRANSPOSE)
        bm = torch.zeros((nb, nb), dtype=torch.bool)
        for r, c in enumerate(rows):
            bm[r, c.astype(np.int64)] = True
        vis = bm.cuda().repeat_interleave(block, 0).repeat_interleave(block, 1)[:N, :N]
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    some = vis.any(1)
    for h in {0, H - 1}:
        ref = reference(q[0, h], k[0, h], v[0, h], do[0, h], vis, scale)
        assert (lse[0, h][~some] == float("-inf")).all() and (out[0, h][~some] == 0).all()
        # lse is float32; out and the gradients carry two to three bf16 roundings (2^-9 each, of P or dS, of the result, and
        # of out inside delta)
        assert (lse[0, h][some].double() - ref[1][some]).abs().max() <= 1e-4 if some.any() else True
        for name, x, r in zip(("out", "dq", "dk", "dv"), (out[0, h], dq[0, h], dk[0, h], dv[0, h]), (ref[0], *ref[2:])):
            assert torch.isfinite(x).all(), (name, h)
            assert (x.double() - r).norm() <= 8e-3 * r.norm() + 1e-6, (name, h, (x.double() - r).norm() / r.norm())
    m.free()
