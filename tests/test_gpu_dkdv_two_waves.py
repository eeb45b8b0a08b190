"""dK/dV of head dimension 64 with two waves per SIMD: beside dQ in one launch with every number of groups at both block sizes, and alone
above 1536 blocks, ragged ends, empty and short lists and the token rule, against float64."""
import numpy as np
import pytest

from test_gpu_list_split import reference

pytestmark = pytest.mark.gpu


# items = heads * blocks.  One launch, block 128: groups of one wave to 32 items, two groups to 256, one to 1536; block 64: groups of one
# wave to 64 items, two groups to 1536.  Above: alone, by one group or (block 64, long lists) two
@pytest.mark.parametrize("block, H, N, most", [
    (128, 5, 16 * 128 - 31, 16), (128, 8, 16 * 128, 4), (128, 8, 16 * 128 + 1, 9), (128, 16, 16 * 128, 3), (128, 17, 15 * 128 + 65, 15),
    (128, 40, 15 * 128 - 95, 1), (128, 11, 50 * 128 - 1, 50), (64, 9, 28 * 64 - 33, 28), (64, 9, 28 * 64, 7), (64, 13, 33 * 64 + 31, 12),
    (64, 18, 33 * 64, 3), (64, 30, 33 * 64 - 1, 33), (64, 60, 33 * 64 + 5, 5),
    (128, 100, 16 * 128 - 33, 16), (128, 110, 14 * 128 + 1, 1), (64, 18, 90 * 64 - 31, 90), (64, 50, 33 * 64, 33), (64, 100, 16 * 64 + 33, 2),
    (128, 2, 16 * 128 - 65, 9), (64, 2, 30 * 64 + 1, 30)])
@pytest.mark.parametrize("rule", [False, True])
def test_gradients_match_float64(block, H, N, most, rule):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"block={block} H={H} N={N} most={most} rule={rule}", flush=True)
    D = 64
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, do = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(4))
    nb, scale = -(-N // block), D ** -0.5
    if rule:
        frames, s = N // 90, 90
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
        rows = [np.sort(rng.choice(nb, size=min(nb, (most, 0, 1, most // 2)[r % 4]), replace=False)) for r in range(nb)]
        row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
        m = rb.radial_mask_from_csr(N, block, row_ptr, np.concatenate(rows).astype(np.int32), rb.RADIAL_MASK_TRANSPOSE)
        bm = torch.zeros((nb, nb), dtype=torch.bool)
        for r, c in enumerate(rows):
            bm[r, c.astype(np.int64)] = True
        vis = bm.cuda().repeat_interleave(block, 0).repeat_interleave(block, 1)[:N, :N]
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    for h in {0, H // 2, H - 1}:
        ref = reference(q[0, h], k[0, h], v[0, h], do[0, h], vis, scale)
        # the gradients carry three bf16 roundings (2^-9 each: of P or dS, of the result, and of out inside delta)
        for name, x, r in zip(("dk", "dv"), (dk[0, h], dv[0, h]), ref[3:]):
            assert torch.isfinite(x).all(), (name, h)
            assert (x.double() - r).norm() <= 8e-3 * r.norm() + 1e-6, (name, h, (x.double() - r).norm() / r.norm())
    m.free()
