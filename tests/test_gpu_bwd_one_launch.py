"""Backward where dK/dV and dQ are one launch: the sizes where its form changes (D 64: 128 parts of 32 rows, 256 blocks, 1536
blocks; D 128: 128 parts of 64 rows, 1536 blocks of 128), ragged ends, empty and short lists and the token rule, against
float64."""
import numpy as np
import pytest

from test_gpu_list_split import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D, block, H, N, most", [(64, *c) for c in [
    (64, 1, 40, 1), (64, 2, 32 * 64 - 1, 32), (64, 5, 13 * 64 - 33, 13), (64, 8, 32 * 64, 7), (64, 13, 20 * 64 + 31, 12), (64, 48, 32 * 64, 5),
    (64, 53, 29 * 64 - 63, 29), (128, 1, 100, 1), (128, 4, 8 * 128 - 95, 8), (128, 3, 11 * 128, 5), (128, 16, 16 * 128 - 1, 9),
    (128, 17, 15 * 128 + 65, 15), (128, 96, 16 * 128, 4), (128, 53, 29 * 128 - 33, 11)]] + [(128, *c) for c in [
    (64, 1, 40, 1), (64, 4, 32 * 64 - 33, 32), (64, 3, 43 * 64 + 1, 9), (128, 1, 100, 1), (128, 4, 16 * 128 - 95, 16), (128, 5, 13 * 128, 3),
    (128, 16, 16 * 128 - 1, 9), (128, 17, 15 * 128 + 65, 15), (128, 48, 32 * 128 - 31, 4), (128, 53, 29 * 128 - 33, 11)]])
@pytest.mark.parametrize("rule", [False, True])
def test_gradients_match_float64(D, block, H, N, most, rule):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"D={D} block={block} H={H} N={N} most={most} rule={rule}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, do = (torch.randn((1, N, H, D), device="cuda", generator=g).bfloat16().transpose(1, 2) for _ in range(4))
    nb, scale = -(-N // block), D ** -0.5
    if rule and N >= 180:
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
        for name, x, r in zip(("dq", "dk", "dv"), (dq[0, h], dk[0, h], dv[0, h]), ref[2:]):
            assert torch.isfinite(x).all(), (name, h)
            assert (x.double() - r).norm() <= 8e-3 * r.norm() + 1e-6, (name, h, (x.double() - r).norm() / r.norm())
    m.free()


@pytest.mark.parametrize("D, block, H, nb", [(64, 64, 2, 9), (64, 64, 16, 30), (64, 128, 16, 16), (64, 128, 17, 30), (128, 64, 4, 32), (128, 128, 4, 9),
                                             (128, 128, 17, 30)])
@pytest.mark.parametrize("shared", ["q", "dout", "packed"])
def test_dq_in_the_memory_of_q_or_dout(D, block, H, nb, shared):
    """dK/dV reads all rows of Q and dO, so dQ must not replace them while it runs."""
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"D={D} block={block} H={H} nb={nb} shared={shared}", flush=True)
    N, scale = nb * block - 17, D ** -0.5
    g = torch.Generator(device="cuda").manual_seed(N)
    packed = torch.randn((1, N, 4, H, D), device="cuda", generator=g).bfloat16()  # q, k, v, dout side by side
    q, k, v, do = (packed[:, :, i].transpose(1, 2) for i in range(4))
    if shared != "packed":
        q, do = q.contiguous(), do.contiguous()
    m = rb.radial_mask_build_dense(N, block, rb.RADIAL_MASK_TRANSPOSE)
    out, dq, dk, dv, dk2, dv2 = (torch.empty((1, H, N, D), dtype=torch.bfloat16, device="cuda") for _ in range(6))
    lse = torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    into = do if shared == "dout" else q
    rb.radial_attn_bwd(q, k, v, out, do, lse, into, dk2, dv2, m, scale, ws)
    # sums in another order, then one bf16 rounding (2^-9) of dS and one of the result
    for name, x, y in (("dq", into, dq), ("dk", dk2, dk), ("dv", dv2, dv)):
        assert (x.double() - y.double()).norm() <= 8e-3 * y.double().norm(), name
    m.free()


@pytest.mark.parametrize("D, block, H, nb, cut", [(64, 64, 2, 30, 33), (64, 64, 9, 32, 1), (64, 64, 24, 32, 0), (64, 128, 4, 13, 65), (64, 128, 8, 16, 0), (64, 128, 8, 17, 100),
                                                  (128, 64, 9, 13, 31), (128, 64, 3, 100, 5), (128, 128, 4, 13, 65), (128, 128, 8, 16, 0), (128, 128, 8, 17, 100), (128, 128, 9, 32, 1)])
@pytest.mark.parametrize("rule", [False, True])
def test_dq_in_the_memory_of_dout_on_ragged_lists(D, block, H, nb, cut, rule):
    """Every form that the kernels take one after the other in small launches: lists of no entry, of one, of a few and of all
    blocks, rows that end in either half of a block, and the token rule."""
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"D={D} block={block} H={H} nb={nb} cut={cut} rule={rule}", flush=True)
    N, scale = nb * block - cut, D ** -0.5
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v, do = (torch.randn((1, N, H, D), device="cuda", generator=g).bfloat16().transpose(1, 2) for _ in range(4))
    if rule:
        m = rb.radial_mask_build(N // 90, 90, block, 1, rb.RADIAL_MASK_TRANSPOSE | rb.RADIAL_MASK_TOKEN_EXACT, extra_tokens=N % 90)
    else:
        rng = np.random.default_rng(N)
        rows = [np.sort(rng.choice(nb, size=(nb, 0, 1, 5, 12)[r % 5], replace=False)) for r in range(nb)]
        row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
        m = rb.radial_mask_from_csr(N, block, row_ptr, np.concatenate(rows).astype(np.int32), rb.RADIAL_MASK_TRANSPOSE)
    out, dq, dk, dv, dk2, dv2 = (torch.full_like(q, float("nan")) for _ in range(6))
    lse = torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    rb.radial_attn_bwd(q, k, v, out, do, lse, do, dk2, dv2, m, scale, ws)
    # sums in another order, then one bf16 rounding (2^-9) of dS and one of the result
    for name, x, y in (("dq", do, dq), ("dk", dk2, dk), ("dv", dv2, dv)):
        assert torch.isfinite(x).all() and (x.double() - y.double()).norm() <= 8e-3 * y.double().norm(), name
    m.free()


@pytest.mark.parametrize("D, block, H, nb", [(64, 64, 2, 9), (64, 128, 17, 30), (128, 64, 4, 32), (128, 128, 4, 9), (128, 128, 17, 30)])
@pytest.mark.parametrize("beside", ["q", "dout"])
def test_dq_beside_q_or_dout_in_one_buffer(D, block, H, nb, beside):
    """A slice of a packed buffer that shares no element with q and dout: same kernels, same bits, and the other slices stay."""
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"D={D} block={block} H={H} nb={nb} beside={beside}", flush=True)
    N, scale = nb * block - 17, D ** -0.5
    g = torch.Generator(device="cuda").manual_seed(N)
    packed = torch.randn((1, N, 4, H, D), device="cuda", generator=g).bfloat16()
    slices = [packed[:, :, i].transpose(1, 2) for i in range(4)]
    k, v, other = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    q, do = (slices[1], other) if beside == "q" else (other, slices[1])
    m = rb.radial_mask_build_dense(N, block, rb.RADIAL_MASK_TRANSPOSE)
    out, dq, dk, dv, dk2, dv2 = (torch.empty((1, H, N, D), dtype=torch.bfloat16, device="cuda") for _ in range(6))
    lse = torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    before = packed.clone()
    rb.radial_attn_bwd(q, k, v, out, do, lse, slices[2], dk2, dv2, m, scale, ws)
    for name, x, y in (("dq", slices[2], dq), ("dk", dk2, dk), ("dv", dv2, dv), *((f"slice {i}", packed[:, :, i], before[:, :, i]) for i in (0, 1, 3))):
        assert torch.equal(x, y), name
    m.free()
