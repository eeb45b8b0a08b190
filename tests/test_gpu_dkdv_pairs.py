"""dK/dV of head dimension 128 and blocks of 128, where two waves share 32 keys, beside dQ in one launch (65 to 1536 blocks) and
alone (above): lists of no entry, of one and of two (its second wave is a stage behind), of 64, 65 and 130 (the chunks in which a
wave reads its list), ragged ends that leave waves without keys, and the token rule, where whole pairs skip stages,
against float64."""
import numpy as np
import pytest

from test_gpu_list_split import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H, N, most", [(9, 15 * 128 - 31, 15), (3, 43 * 128 - 97, 1), (9, 16 * 128, 2), (2, 65 * 128 + 1, 64), (2, 65 * 128, 65),
                                        (1, 130 * 128 - 64, 130), (7, 19 * 128 + 33, 3),
                                        (110, 14 * 128 - 31, 14), (110, 14 * 128 + 33, 1), (24, 65 * 128, 65), (24, 65 * 128 + 1, 64)])  # alone
@pytest.mark.parametrize("rule", [0, 90, 700])
def test_gradients_match_float64(H, N, most, rule):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"H={H} N={N} most={most} rule={rule}", flush=True)
    D, block = 128, 128
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, do = (torch.randn((1, N, H, D), device="cuda", generator=g).bfloat16().transpose(1, 2) for _ in range(4))
    nb, scale = -(-N // block), D ** -0.5
    if rule:  # tokens per frame
        frames, s = N // rule, rule
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
        rows = [np.sort(rng.choice(nb, size=min(nb, (most, 0, 1, most, most // 2)[r % 5]), replace=False)) for r in range(nb)]
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
    for h in {0, H - 1}:
        ref = reference(q[0, h], k[0, h], v[0, h], do[0, h], vis, scale)
        # the gradients carry three bf16 roundings (2^-9 each: of P or dS, of the result, and of out inside delta)
        for name, x, r in zip(("dk", "dv"), (dk[0, h], dv[0, h]), ref[3:]):
            assert torch.isfinite(x).all(), (name, h)
            assert (x.double() - r).norm() <= 8e-3 * r.norm() + 1e-6, (name, h, (x.double() - r).norm() / r.norm())
    m.free()
