"""8-bit scores of small launches: four parts per block (to 64 blocks), two (to 128), none above; lists that leave groups
without an entry, ragged ends in every part; and the quantiser on blocks that end anywhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H, N, most", [(1, 31, 1), (1, 128 + 33, 2), (4, 16 * 128 - 65, 16), (4, 16 * 128, 3), (5, 13 * 128 - 127, 13), (8, 16 * 128 - 1, 9), (3, 43 * 128, 43)])
def test_forward_matches_float64_on_the_codes(H, N, most):
    import torch
    from oracle import quant as oq
    from paper_2506_19852_amd import binding as rb
    print(f"H={H} N={N} most={most}", flush=True)
    D = block = 128
    nb = -(-N // block)
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    codes, scales = [], []
    for x in (q, k):
        codes.append(torch.empty((1, H, N, D), dtype=torch.uint8, device="cuda"))
        scales.append(torch.empty((1, H, nb), dtype=torch.float32, device="cuda"))
        rb.radial_quantize_fp8(x, block, codes[-1], scales[-1])
    ref_codes, ref_scales = oq.quantize_blocks(q[0, H - 1].float().cpu().numpy(), block)
    assert np.array_equal(codes[0][0, H - 1].cpu().numpy(), ref_codes) and np.array_equal(scales[0][0, H - 1].cpu().numpy(), ref_scales)
    q, k = (c.view(torch.float8_e4m3fn).double() * s.double().repeat_interleave(block, 2)[:, :, :N, None] for c, s in zip(codes, scales))
    rng = np.random.default_rng(N)
    rows = [np.sort(rng.choice(nb, size=min(nb, (most, 0, 1, 2, most - 1)[r % 5]), replace=False)) for r in range(nb)]
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
        assert (lse[0, h][some].double() - ref_lse[some]).abs().max() <= 1e-3 if some.any() else True
        assert (out[0, h].double() - ref).norm() <= 8e-3 * ref.norm() + 1e-6
    m.free()
