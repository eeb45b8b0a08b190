"""At the edges of the rules that choose between single blocks and pairs of them, against float64: the forward, bf16 and 8-bit scores, and dK/dV; few blocks and
short lists by slices, long neighbours, lists with little in common, batches, peaked rows, dq in the memory of q or dout."""
import numpy as np
import pytest

from test_gpu_list_split import reference
from test_gpu_two_blocks import check

pytestmark = pytest.mark.gpu


def band(nb, width):
    """`width` neighbouring blocks a row."""
    first = np.minimum(np.maximum(np.arange(nb) - width // 2, 0), nb - width)
    return [np.arange(f, f + width) for f in first]


# fewer than 8 blocks on either side of a rule; 40 heads of 128 blocks are by slices, of 18 slices start workgroups without work
EDGES = [(127, 4, 3, 7), (128, 4, 4, 90), (199, 5, 2, 64), (200, 5, 5, 1), (199, 6, 6, 33), (200, 6, 2, 0), (300, 3, 3, 127), (140, 7, 7, 5), (140, 2, 1, 3),
         (40, 128, 27, 31), (40, 128, 28, 97), (149, 18, 2, 65)]


@pytest.mark.parametrize("H, nb, width, cut", EDGES)
def test_bf16(H, nb, width, cut):
    from paper_2506_19852_amd import binding as rb
    print(f"H={H} nb={nb} width={width} cut={cut}", flush=True)
    check(rb, 1, H, 128 * nb - cut, band(nb, width), "bnhd" if H % 2 else "bhnd", 2.0, H + nb)


@pytest.mark.parametrize("H, nb, width, cut", [e for e in EDGES if e[1] < 8] + [(40, 128, 2, 31), (149, 18, 2, 65)])
def test_8_bit_scores(H, nb, width, cut):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"8 bits H={H} nb={nb} width={width} cut={cut}", flush=True)
    D, N = 128, 128 * nb - cut
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    codes = [torch.empty((1, H, N, D), dtype=torch.uint8, device="cuda") for _ in range(2)]
    scales = [torch.empty((1, H, nb), dtype=torch.float32, device="cuda") for _ in range(2)]
    for x, c, s in zip((q, k), codes, scales):
        rb.radial_quantize_fp8(x, 128, c, s)
    lists = band(nb, width)
    bm = torch.zeros((nb, nb), dtype=torch.bool)
    for r, c in enumerate(lists):
        bm[r, torch.from_numpy(c)] = True
    m = rb.radial_mask_from_csr(N, 128, np.arange(nb + 1, dtype=np.int32) * width, np.concatenate(lists).astype(np.int32))
    out = torch.full((1, H, N, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    rb.radial_attn_fwd_fp8(codes[0], scales[0], codes[1], scales[1], v, out, lse, m, D ** -0.5)
    vis = bm.cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)[:N, :N]
    for h in sorted({0, 1, H // 2, H - 9, H - 8, H - 1}):
        qd, kd = (c[0, h].view(torch.float8_e4m3fn).double() * s[0, h].double().repeat_interleave(128)[:N, None] for c, s in zip(codes, scales))
        ref, ref_lse = reference(qd, kd, v[0, h], torch.zeros_like(qd), vis, D ** -0.5)[:2]
        # the 8-bit matrix instruction's sums: 1e-4 of the scores; P and out are rounded to bf16 (2^-9 each)
        assert (lse[0, h].double() - ref_lse).abs().max() <= 1e-4 * (1 + ref_lse.abs().max())
        for r in range(0, N, 128):
            assert (out[0, h, r:r + 128].double() - ref[r:r + 128]).norm() <= 8e-3 * ref[r:r + 128].norm() + 1e-6, (h, r // 128)
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    m.free()


def pairs_of(rb, m, q, k, v, scale):
    """The share of second blocks that began when their neighbour ended: all of those in pairs, hardly any other.  The traced launch gives the same output."""
    import torch
    _, H, N, _ = q.shape
    nb = -(-N // 128)
    out, traced = torch.empty_like(q), torch.empty_like(q)
    rb.radial_attn_fwd(q, k, v, out, None, m, scale)
    trace = torch.zeros((rb.radial_attn_fwd_trace_records(1, H, m), 3), dtype=torch.int64, device="cuda")
    rb.radial_attn_fwd_trace(q, k, v, traced, None, m, scale, trace)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), traced.view(torch.int16))
    t = trace.cpu().numpy()
    assert np.sum(t[:, 1] != 0) == H * nb
    return out, np.sum((t[8:, 0] == t[:-8, 1]) & (t[8:, 0] != 0)) / (H * (nb // 2))    # a pair's records are 8 apart


# entries that neighbouring rows share: none, an eighth, a quarter of 32 of them, all
@pytest.mark.parametrize("common", [0, 4, 8, 32])
def test_lists_with_little_in_common(common):
    import torch
    from paper_2506_19852_amd import binding as rb
    H, nb, D = 40, 128, 128
    lists = []
    for r in range(nb):
        own = 64 * (r % 2) + (r // 2 + np.arange(32 - common)) % 64      # the two halves of the blocks in turn
        both = (64 + r // 2 + np.arange(32 - common, 32)) % 64 if common else np.zeros(0, dtype=np.int64)
        lists.append(np.unique(np.concatenate([own, both])))
        assert len(lists[r]) >= 32 - common
    m = rb.radial_mask_from_csr(128 * nb, 128, np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32), np.concatenate(lists).astype(np.int32))
    g = torch.Generator(device="cuda").manual_seed(common)
    q, k, v = (torch.randn((1, H, 128 * nb, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    out, seconds = pairs_of(rb, m, q, k, v, D ** -0.5)
    assert seconds > 0.5 if common >= 8 else seconds < 0.1, seconds
    vis = torch.zeros((nb, nb), dtype=torch.bool)
    for r, c in enumerate(lists):
        vis[r, torch.from_numpy(c)] = True
    vis = vis.cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)
    for h in (0, H - 1):
        ref = reference(q[0, h], k[0, h], v[0, h], torch.zeros_like(q[0, h]), vis, D ** -0.5)[0]
        assert (out[0, h].double() - ref).norm() <= 8e-3 * ref.norm()    # P and out are rounded to bf16 (2^-9 each)
    m.free()


@pytest.mark.parametrize("how", ["csr", "radial"])
@pytest.mark.parametrize("full", [1, 2])
def test_two_long_neighbours(how, full):
    """Text rows see every block: where two of them are neighbours, one workgroup would have both for longer than the rest of the launch takes.  In
    pairs, and only there, a block begins when its neighbour ends."""
    import torch
    from paper_2506_19852_amd import binding as rb
    H, D, nb = (40, 128, 128) if how == "csr" else (1, 128, 1126 + full)
    N = 128 * nb
    if how == "csr":
        lists = band(nb, 32)
        for r in range(nb - full, nb):
            lists[r] = np.arange(nb)
        m = rb.radial_mask_from_csr(N, 128, np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32), np.concatenate(lists).astype(np.int32))
    else:   # 1125 blocks of video; text in block 1125, which has a neighbour that is video, 1126 and 1127, which are neighbours
        m = rb.radial_mask_build(40, 3600, 128, 1, 0, extra_tokens=N - 40 * 3600)
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    out, seconds = pairs_of(rb, m, q, k, v, D ** -0.5)
    assert seconds > 0.5 if full == 1 else seconds < 0.1, seconds
    h, rows = H - 1, slice(N - 128, N)
    s = (D ** -0.5 * (q[0, h, rows].double() @ k[0, h].double().T)).softmax(1)   # the last block's list is full
    ref = s @ v[0, h].double()
    # P and out are rounded to bf16 (2^-9 each)
    assert (out[0, h, rows].double() - ref).norm() <= 8e-3 * ref.norm()
    m.free()


@pytest.mark.parametrize("how", ["csr", "radial"])
def test_long_list_of_an_odd_last_block_is_among_the_first(how):
    """In order of length the workgroups of the last block, which has no neighbour, are among the first eight ranks where its list is full, though two of the others are longer.
    They are the ones whose second record is missing."""
    import torch
    from paper_2506_19852_amd import binding as rb
    H, D, nb = (9, 128, 131) if how == "csr" else (4, 128, 269)
    N = 128 * nb if how == "csr" else 24 * 1420 + 226
    if how == "csr":
        lists = band(nb, 80)
        lists[-1] = np.arange(nb)
        m = rb.radial_mask_from_csr(N, 128, np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32), np.concatenate(lists).astype(np.int32))
    else:
        m = rb.radial_mask_build(24, 1420, 128, 1, 0, extra_tokens=226)
    row_ptr, _ = rb.radial_mask_copy_to_host(m)
    n = np.diff(row_ptr)
    assert len(n) == nb and n[-1] == nb and n[-1] < np.sort(n[0:-1:2] + n[1::2])[10]
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    trace = torch.zeros((rb.radial_attn_fwd_trace_records(1, H, m), 3), dtype=torch.int64, device="cuda")
    rb.radial_attn_fwd_trace(q, k, v, torch.empty_like(q), None, m, D ** -0.5, trace)
    torch.cuda.synchronize()
    used = (trace[:, 1] != 0).cpu().numpy()
    assert used.sum() == H * nb
    first = used[:16 * H].reshape(H, 2, 8)      # the first 8 * H workgroups, eight at a time
    assert first[:, 0].all() and (~first[:, 1]).sum() == H
    m.free()


# dK/dV above 1536 blocks: lists of 6 and 7, 3 and 7 blocks, slices with gaps
@pytest.mark.parametrize("B, H, nb, width, cut, gain, dq_in", [(2, 260, 3, 3, 127, 4.0, None), (1, 230, 7, 6, 33, 1.0, "dout"), (2, 115, 7, 7, 1, 4.0, "q"), (2, 20, 40, 6, 64, 4.0, "q"),
                                                               (2, 20, 40, 7, 95, 4.0, "dout"), (1, 400, 4, 1, 3, 4.0, "q"), (2, 150, 9, 2, 65, 4.0, "dout"), (3, 8, 131, 40, 31, 4.0, "q")])
def test_key_blocks(B, H, nb, width, cut, gain, dq_in):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"keys B={B} H={H} nb={nb} width={width} cut={cut} gain={gain} dq in {dq_in}", flush=True)
    D, N = 128, 128 * nb - cut
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, do = (torch.randn((B, N, H, D), device="cuda", generator=g).transpose(1, 2) for _ in range(4))
    q, k, v, do = (q * gain).bfloat16(), k.bfloat16(), v.bfloat16(), do.bfloat16()
    lists = band(nb, width)
    m = rb.radial_mask_from_csr(N, 128, np.arange(nb + 1, dtype=np.int32) * width, np.concatenate(lists).astype(np.int32), rb.RADIAL_MASK_TRANSPOSE)
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(B, H, N, D, m), dtype=torch.uint8, device="cuda")
    scale = D ** -0.5
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    if dq_in:
        shared = {"q": q, "dout": do, dq_in: (q if dq_in == "q" else do).clone(memory_format=torch.preserve_format)}
        again = [torch.full_like(q, float("nan")) for _ in range(2)]
        rb.radial_attn_bwd(shared["q"], k, v, out, shared["dout"], lse, shared[dq_in], *again, m, scale, ws)
        for x, y in zip((dq, dk, dv), (shared[dq_in], *again)):
            assert torch.equal(x, y)
    vis = torch.zeros((nb, nb), dtype=torch.bool)
    for r, c in enumerate(lists):
        vis[r, torch.from_numpy(c)] = True
    vis = vis.cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)[:N, :N]
    for bh in sorted({0, H - 1, (B - 1) * H, B * H - 9, B * H - 8, B * H - 1}):
        b, h = divmod(bh, H)
        want = reference(q[b, h], k[b, h], v[b, h], do[b, h], vis, scale)[2:]
        for name, x, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), want):
            # P and dS are rounded to bf16 between the products and the results once more, 2^-9 each; delta comes from the rounded output
            assert (x[b, h].double() - ref).norm() <= 1.2e-2 * ref.norm() + 1e-6, (bh, name, float((x[b, h].double() - ref).norm() / ref.norm()))
    assert all(torch.isfinite(x).all() for x in (dq, dk, dv))
    m.free()
