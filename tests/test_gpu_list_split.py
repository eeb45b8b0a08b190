"""Small launches, where several groups of waves share a block's list and merge their results: every form of
the dispatch (half blocks, four, two and one group), with lists that leave groups without an entry, ragged
ends, the token rule and rows far apart in scale, against float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def reference(q, k, v, do, vis, scale):
    q, k, v, do = (t.double() for t in (q, k, v, do))
    s = (scale * (q @ k.T)).masked_fill(~vis, float("-inf"))
    lse = s.logsumexp(1)
    p = (s - lse[:, None]).exp().nan_to_num(0.0)
    out = p @ v
    ds = p * (do @ v.T - (do * out).sum(1, keepdim=True))
    return out, lse, scale * (ds @ k), scale * (ds.T @ q), p.T @ do


# items = heads * blocks: block 128 changes at 128 and 256, block 64 at 256, 1200 and 1536
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("block, H, N, rule", [
    (128, 1, 1, False), (128, 2, 777, False), (128, 8, 16 * 128, True), (128, 3, 43 * 128 - 1, False), (128, 4, 64 * 128, False),
    (128, 9, 29 * 128 - 90, False), (64, 1, 65, False), (64, 4, 64 * 64, True), (64, 5, 52 * 64 - 31, False),
    (64, 24, 50 * 64 + 3, False), (64, 25, 61 * 64, False), (64, 26, 61 * 64 - 63, True)])
def test_forward_and_backward_match_float64(D, block, H, N, rule):
    import torch
    from paper_2506_19852_amd import binding as rb
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, do = (torch.randn((1, H, N, D), device="cuda", generator=g) for _ in range(4))
    q, k, v, do = (t.bfloat16() for t in (q * 2, k, v, do))
    nb = -(-N // block)
    scale = D ** -0.5
    if rule:
        frames = max(1, N // 128)
        s = N // frames
        flags = rb.RADIAL_MASK_TRANSPOSE | rb.RADIAL_MASK_TOKEN_EXACT
        m = rb.radial_mask_build(frames, s, block, 1, flags, extra_tokens=N - frames * s)
        pos = torch.arange(N, device="cuda")
        fr, text = pos // s, pos >= frames * s
        at, d = pos - fr * s, (fr[:, None] - fr[None]).abs()
        b = torch.ones_like(d)
        for e in range(1, 12):
            b = torch.where(d >= (1 << e), torch.full_like(b, 1 << e), b)
        w = s // b
        near = torch.where(w >= 1, (at[:, None] - at[None]).abs() <= w - 1, (at[:, None] == at[None]) & (d % (-(-b // s)) == 0))
        vis = near | (fr < 1)[None] | text[None] | text[:, None]
    else:  # lists of 0, 1, 2, 3, 5, ... entries: some groups get none
        rng = np.random.default_rng(N)
        rows = [np.sort(rng.choice(nb, size=min(nb, (0, 1, 2, 3, 5, nb)[r % 6] if nb > 2 else nb), replace=False)) for r in range(nb)]
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
    for h in sorted({0, H // 2, H - 1}):
        ref = reference(q[0, h], k[0, h], v[0, h], do[0, h], vis, scale)
        got = (out[0, h], lse[0, h], dq[0, h], dk[0, h], dv[0, h])
        some = vis.any(1)
        assert (got[1][~some] == float("-inf")).all() and (got[0][~some] == 0).all()
        # lse is float32; out and the gradients carry two to three bf16 roundings (2^-9 each, of P or dS, of
        # the result, and of out inside delta)
        assert (got[1][some].double() - ref[1][some]).abs().max() <= 1e-4 if some.any() else True
        for x, r in zip((got[0], *got[2:]), (ref[0], *ref[2:])):
            assert torch.isfinite(x).all()
            assert (x.double() - r).norm() <= 8e-3 * r.norm() + 1e-6, (h, (x.double() - r).norm() / r.norm())
    m.free()


# Lists of at most two entries are walked by one group whatever the size of the launch.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("block, H, N", [(128, 2, 777), (128, 20, 11 * 128 + 1), (128, 9, 29 * 128 - 90), (64, 3, 333), (64, 24, 50 * 64 + 3), (64, 28, 80 * 64 - 5)])
def test_short_lists_match_float64(D, block, H, N):
    import torch
    from paper_2506_19852_amd import binding as rb
    nb = -(-N // block)
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v, do = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(4))
    rng = np.random.default_rng(N)
    rows = [np.sort(rng.choice(nb, size=r % 3, replace=False)) for r in range(nb)]
    row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    m = rb.radial_mask_from_csr(N, block, row_ptr, np.concatenate(rows).astype(np.int32), rb.RADIAL_MASK_TRANSPOSE)
    bm = torch.zeros((nb, nb), dtype=torch.bool)
    for r, c in enumerate(rows):
        bm[r, c.astype(np.int64)] = True
    vis = bm.cuda().repeat_interleave(block, 0).repeat_interleave(block, 1)[:N, :N]
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, D ** -0.5)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, D ** -0.5, ws)
    some = vis.any(1)
    for h in (0, H - 1):
        ref = reference(q[0, h], k[0, h], v[0, h], do[0, h], vis, D ** -0.5)
        assert (lse[0, h][~some] == float("-inf")).all() and (out[0, h][~some] == 0).all()
        # bounds as above
        assert (lse[0, h][some].double() - ref[1][some]).abs().max() <= 1e-4
        for name, x, r in zip(("out", "dq", "dk", "dv"), (out[0, h], dq[0, h], dk[0, h], dv[0, h]), (ref[0], *ref[2:])):
            assert torch.isfinite(x).all(), (name, h)
            assert (x.double() - r).norm() <= 8e-3 * r.norm() + 1e-6, (name, h, (x.double() - r).norm() / r.norm())
    m.free()


# Frames whose boundaries fall anywhere in a block; heads so that 8 blocks of 128 (16 of 64) take each form: half
# blocks, two groups, one; four groups, two, and from 1600 items one in every kernel that has that form.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("block, H", [(128, 4), (128, 20), (128, 40), (64, 4), (64, 20), (64, 100)])
@pytest.mark.parametrize("s", [65, 70, 79, 90, 93, 100, 333])
def test_token_rule_with_any_frame_length(D, block, H, s):
    import torch
    from oracle import build as obuild
    from paper_2506_19852_amd import binding as rb
    print(f"token rule s={s} block={block} H={H} D={D}", flush=True)
    frames = 1000 // s
    N = frames * s
    g = torch.Generator(device="cuda").manual_seed(s + H)
    q, k, v, do = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(4))
    scale = D ** -0.5
    m = rb.radial_mask_build(frames, s, block, 1, rb.RADIAL_MASK_TRANSPOSE | rb.RADIAL_MASK_TOKEN_EXACT)
    vis = torch.from_numpy(obuild.token_mask(frames, s, 1, 0, N, np.arange(N))).cuda()
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    for h in (0, H // 2, H - 1):
        ref = reference(q[0, h], k[0, h], v[0, h], do[0, h], vis, scale)
        # bounds as above
        assert (lse[0, h].double() - ref[1]).abs().max() <= 1e-4, h
        for name, x, r in zip(("out", "dq", "dk", "dv"), (out[0, h], dq[0, h], dk[0, h], dv[0, h]), (ref[0], *ref[2:])):
            assert torch.isfinite(x).all(), (name, h)
            assert (x.double() - r).norm() <= 8e-3 * r.norm(), (name, h, (x.double() - r).norm() / r.norm())
    m.free()


@pytest.mark.parametrize("H, N", [(1, 1), (2, 777), (4, 64 * 128 - 7), (5, 52 * 128)])
def test_8bit_scores_match_float64_on_the_codes(H, N):
    import torch
    from paper_2506_19852_amd import binding as rb
    D = block = 128
    nb = -(-N // block)
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    codes, scales = [], []
    for x in (q, k):
        codes.append(torch.empty((1, H, N, D), dtype=torch.uint8, device="cuda"))
        scales.append(torch.empty((1, H, nb), dtype=torch.float32, device="cuda"))
        rb.radial_quantize_fp8(x, block, codes[-1], scales[-1])
    q, k = (c.view(torch.float8_e4m3fn).double() * s.double().repeat_interleave(block, 2)[:, :, :N, None] for c, s in zip(codes, scales))
    rng = np.random.default_rng(N)
    rows = [np.sort(rng.choice(nb, size=min(nb, (0, 1, 2, 4, nb)[r % 5] if nb > 2 else nb), replace=False)) for r in range(nb)]
    row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    m = rb.radial_mask_from_csr(N, block, row_ptr, np.concatenate(rows).astype(np.int32))
    bm = torch.zeros((nb, nb), dtype=torch.bool)
    for r, c in enumerate(rows):
        bm[r, c.astype(np.int64)] = True
    vis = bm.cuda().repeat_interleave(block, 0).repeat_interleave(block, 1)[:N, :N]
    out = torch.full((1, H, N, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    rb.radial_attn_fwd_fp8(codes[0], scales[0], codes[1], scales[1], v, out, lse, m, D ** -0.5)
    some = vis.any(1)
    for h in {0, H - 1}:
        s = (D ** -0.5 * (q[0, h] @ k[0, h].T)).masked_fill(~vis, float("-inf"))
        ref_lse = s.logsumexp(1)
        ref = (s - ref_lse[:, None]).exp().nan_to_num(0.0) @ v[0, h].double()
        assert (lse[0, h][~some] == float("-inf")).all() and (out[0, h][~some] == 0).all()
        # the 8-bit matrix instruction's sums: 1e-4 of the scores; P and out are rounded to bf16 (2^-9 each)
        assert (lse[0, h][some].double() - ref_lse[some]).abs().max() <= 1e-3
        assert (out[0, h].double() - ref).norm() <= 8e-3 * ref.norm()
    m.free()
