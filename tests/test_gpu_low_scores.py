"""Forward over pairs of neighbouring query blocks, bf16 and 8-bit scores, where scores of some rows overflow to -inf: in the first half of a
stage, in whole key blocks and in all keys of a row, while other rows of the same wave have finite ones.  Such keys weigh nothing."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# by slices (two blocks per head; lists that share most entries), and by length
@pytest.mark.parametrize("H, nb, cut, kind", [(140, 2, 5, "all"), (20, 131, 97, "near"), (9, 115, 31, "all")])
@pytest.mark.parametrize("codes", [False, True])
def test_rows_without_a_score_so_far(H, nb, cut, kind, codes):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"H={H} nb={nb} cut={cut} {kind} codes={codes}", flush=True)
    D, N, scale = 128, 128 * nb - cut, 128 ** -0.5
    rng = np.random.default_rng(nb)
    bm = np.ones((nb, nb), dtype=bool)
    if kind == "near":  # neighbouring lists share most entries and have some alone
        bm = np.repeat(rng.random(((nb + 1) // 2, nb)) < 0.8, 2, axis=0)[:nb] ^ (rng.random((nb, nb)) < 0.1)
        bm[6:8] = [[c == 3 for c in range(nb)], [c in (3, 5) for c in range(nb)]]  # all that the first of these names is -inf for some of its rows
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v = (torch.randn((1, H, N, D), device="cuda", generator=g) for _ in range(3))
    i = torch.arange(N, device="cuda")
    # rows 3, 10, 17, ...: -3e40, beyond float32, for the first 48 keys of every block and all keys of every third
    q[..., 0] = torch.where(i % 7 == 3, 3e20, 1e-20)
    k[..., 0] = torch.where((i % 128 < 48) | (i // 128 % 3 == 0) & (nb > 2), -1e20, 0.0)
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    m = rb.radial_mask_from_csr(N, 128, np.concatenate([[0], np.cumsum(bm.sum(1))]).astype(np.int32), np.nonzero(bm)[1].astype(np.int32))
    out = torch.full_like(q, float("nan"))
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    if codes:
        c = [torch.empty((1, H, N, D), dtype=torch.uint8, device="cuda") for _ in range(2)]
        s = [torch.empty((1, H, nb), dtype=torch.float32, device="cuda") for _ in range(2)]
        for x, xc, xs in zip((q, k), c, s):
            rb.radial_quantize_fp8(x, 128, xc, xs)
        rb.radial_attn_fwd_fp8(c[0], s[0], c[1], s[1], v, out, lse, m, scale)
        q, k = (xc.view(torch.float8_e4m3fn).double() * xs.double().repeat_interleave(128, 2)[:, :, :N, None] for xc, xs in zip(c, s))
    else:
        rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    torch.cuda.synchronize()
    visible = torch.from_numpy(bm).cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)[:N, :N]
    for h in sorted({0, H // 2, H - 1}):
        x = q[0, h].double() @ k[0, h].double().T
        x = (scale * x).masked_fill(~visible | (x < -torch.finfo(torch.float32).max), float("-inf"))
        ref_lse = x.logsumexp(1)
        ref = (x - ref_lse[:, None]).exp().nan_to_num(0.0) @ v[0, h].double()
        none = torch.isneginf(ref_lse)
        assert none.any() == (kind == "near") and not none.all()
        assert torch.isneginf(lse[0, h][none]).all() and (out[0, h][none] == 0).all()
        # sums in float32, the 8-bit matrix instruction's: 1e-4 of the scores; P and the result are rounded to bf16, 2^-9 each
        assert (lse[0, h].double() - ref_lse)[~none].abs().max() <= (1e-4 if codes else 1e-5) * (1 + ref_lse[~none].abs().max())
        for r in range(0, N, 128):
            assert (out[0, h, r:r + 128].double() - ref[r:r + 128]).norm() <= 8e-3 * ref[r:r + 128].norm() + 1e-6, (h, r // 128)
    m.free()
