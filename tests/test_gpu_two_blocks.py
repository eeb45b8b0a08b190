"""Forward over pairs of neighbouring query blocks (head dimension 128, blocks of 128): heads by slices and by length, odd and even numbers of
blocks, ragged ends in either half of a stage, neighbouring lists that are equal, overlap, have nothing in common or are empty, lists of
more entries than a wave looks at together, strided tensors, against float64."""
import numpy as np
import pytest

from test_gpu_list_split import reference

pytestmark = pytest.mark.gpu


def make_lists(nb, kind, seed):
    rng = np.random.default_rng(seed)
    lists = []
    for r in range(nb):
        if kind == "mixed":   # pairs: overlapping, nothing in common, first empty, second empty, equal
            p, odd = r // 2 % 5, r % 2
            some = np.sort(np.random.default_rng(seed + r // 2).choice(nb, size=max(1, nb // 2), replace=False))
            if p == 0:
                some = np.sort(rng.choice(nb, size=max(1, 2 * nb // 3), replace=False))
            elif p == 1:
                some = some[odd::2]
            elif p == 2 and not odd or p == 3 and odd:
                some = some[:0]
            lists.append(some)
        elif kind == "near":  # neighbours share most entries and have some alone
            some = np.random.default_rng(seed + r // 2).random(nb) < 0.8
            lists.append(np.flatnonzero(some ^ (rng.random(nb) < 0.1)))
        else:
            lists.append(np.arange(nb))
    return lists


def check(rb, B, H, N, lists, layout, gain, seed):
    import torch
    nb, D = -(-N // 128), 128
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = (B, N, H, D) if layout == "bnhd" else (B, H, N, D)
    q, k, v = (torch.randn(shape, device="cuda", generator=g) for _ in range(3))
    q, k, v = ((x * f).bfloat16() for x, f in ((q, gain), (k, 1.0), (v, 1.0)))
    if layout == "bnhd":
        q, k, v = (x.transpose(1, 2) for x in (q, k, v))
    row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in lists])]).astype(np.int32)
    m = rb.radial_mask_from_csr(N, 128, row_ptr, np.concatenate(lists).astype(np.int32))
    out = torch.full_like(q, float("nan"))
    lse = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, D ** -0.5)
    again, lse_again = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
    rb.radial_attn_fwd(q, k, v, again, lse_again, m, D ** -0.5)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), again.view(torch.int16)) and torch.equal(lse, lse_again)
    bm = torch.zeros((nb, nb), dtype=torch.bool)
    for r, c in enumerate(lists):
        bm[r, torch.from_numpy(c.astype(np.int64))] = True
    visible = bm.cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)[:N, :N]
    seen = visible.any(dim=1)
    # every head of a launch by itself: heads are compared with each other's sums only through the reference
    for bh in sorted({0, 1, B * H // 2, B * H - 2, B * H - 1} & set(range(B * H))):
        b, h = divmod(bh, H)
        ro, rl = reference(q[b, h], k[b, h].double(), v[b, h].double(), torch.zeros_like(q[b, h]), visible, D ** -0.5)[:2]
        o, l = out[b, h].double(), lse[b, h].double()
        # P and the result are rounded to bf16: 2^-9 of the values summed and of the sum, twice that for the order of the sums
        bound = 2 * 2.0 ** -9 * (v[b, h].double().abs().amax(dim=0)[None] + ro.abs()) + 1e-6
        assert ((o - ro).abs() <= bound)[seen].all(), (bh, float((o - ro)[seen].abs().max()))
        # on long flat lists that is as much as the values themselves: the rounding errors of a block of rows taken together, 2^-9 of P and of the result each
        for r in range(0, N, 128):
            assert (o - ro.nan_to_num(0.0))[r:r + 128].norm() <= 8e-3 * ro[r:r + 128].nan_to_num(0.0).norm() + 1e-6, (bh, r // 128)
        assert (l - rl).abs()[seen].max() <= 1e-5 * (1 + rl[seen].abs().max()) if seen.any() else True
        assert (o[~seen] == 0).all() and torch.isneginf(l[~seen]).all()
    # heads in between: no block is left out or written from another head's rows
    assert torch.isfinite(out).all() and torch.isfinite(lse[:, :, seen]).all()
    m.free()


# heads x blocks, tokens missing in the last block: by slices (few blocks, many heads), of 1 to 7 blocks (of 3 and 7 single blocks, of 5 either)
@pytest.mark.parametrize("B, H, nb, cut", [(1, 300, 1, 60), (2, 80, 2, 0), (1, 120, 3, 127), (3, 23, 5, 64), (1, 61, 7, 33), (2, 70, 4, 65), (1, 240, 5, 64), (3, 70, 6, 33)])
@pytest.mark.parametrize("kind", ["mixed", "all"])
@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
def test_few_blocks_by_slices(B, H, nb, cut, kind, layout):
    from paper_2506_19852_amd import binding as rb
    print(f"B={B} H={H} nb={nb} cut={cut} {kind} {layout}", flush=True)
    check(rb, B, H, 128 * nb - cut, make_lists(nb, kind, nb + H), layout, 1.0, H + nb)


# by slices with lists of more than 64 and 128 entries, peaked rows; by length in whole rounds of pairs, single blocks and halves (of 130 and 101 blocks with lists of 64
# and more only: "near")
@pytest.mark.parametrize("H, nb, cut, kind, gain", [(20, 131, 97, "mixed", 4.0), (20, 131, 31, "all", 1.0), (8, 130, 1, "mixed", 1.0), (9, 115, 95, "all", 2.0), (14, 101, 0, "mixed", 4.0),
                                                    (9, 130, 1, "near", 1.0), (14, 101, 31, "near", 4.0), (40, 128, 64, "near", 1.0)])
def test_long_lists(H, nb, cut, kind, gain):
    from paper_2506_19852_amd import binding as rb
    print(f"H={H} nb={nb} cut={cut} {kind} gain={gain}", flush=True)
    lists = make_lists(nb, kind, nb + H)
    check(rb, 1, H, 128 * nb - cut, lists, "bnhd", gain, H + nb)


@pytest.mark.parametrize("H, nb, cut, kind, gain", [(300, 1, 60, "mixed", 1.0), (120, 3, 127, "mixed", 4.0), (61, 7, 33, "all", 1.0), (20, 131, 97, "mixed", 4.0), (8, 130, 1, "mixed", 1.0), (14, 101, 0, "all", 2.0),
                                                    (140, 4, 95, "mixed", 4.0), (240, 5, 33, "mixed", 1.0), (9, 130, 1, "near", 4.0), (40, 128, 64, "near", 1.0)])
def test_8_bit_scores(H, nb, cut, kind, gain):
    """The same launches on codes of Q and K with a scale per block, against float64 on the codes."""
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"8 bits H={H} nb={nb} cut={cut} {kind} gain={gain}", flush=True)
    D, N = 128, 128 * nb - cut
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v = (torch.randn((1, H, N, D), device="cuda", generator=g) for _ in range(3))
    # blocks far apart in scale: either block of a pair and every key block has its own
    spread = (2.0 ** torch.randint(-2, 3, (1, H, nb, 1), device="cuda", generator=g)).repeat_interleave(128, 2)[:, :, :N]
    q, k, v = (q * gain).bfloat16(), (k * spread).bfloat16(), v.bfloat16()
    codes = [torch.empty((1, H, N, D), dtype=torch.uint8, device="cuda") for _ in range(2)]
    scales = [torch.empty((1, H, nb), dtype=torch.float32, device="cuda") for _ in range(2)]
    for x, c, s in zip((q, k), codes, scales):
        rb.radial_quantize_fp8(x, 128, c, s)
    lists = make_lists(nb, kind, nb + H)
    row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in lists])]).astype(np.int32)
    m = rb.radial_mask_from_csr(N, 128, row_ptr, np.concatenate(lists).astype(np.int32))
    out = torch.full((1, H, N, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    rb.radial_attn_fwd_fp8(codes[0], scales[0], codes[1], scales[1], v, out, lse, m, D ** -0.5)
    bm = torch.zeros((nb, nb), dtype=torch.bool)
    for r, c in enumerate(lists):
        bm[r, torch.from_numpy(c.astype(np.int64))] = True
    vis = bm.cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)[:N, :N]
    some = vis.any(1)
    for h in sorted({0, 1, H // 2, H - 2, H - 1}):
        qd, kd = (c[0, h].view(torch.float8_e4m3fn).double() * s[0, h].double().repeat_interleave(128)[:N, None] for c, s in zip(codes, scales))
        ref, ref_lse = reference(qd, kd, v[0, h], torch.zeros_like(qd), vis, D ** -0.5)[:2]
        assert (lse[0, h][~some] == float("-inf")).all() and (out[0, h][~some] == 0).all()
        if some.any():
            # the 8-bit matrix instruction's sums: 1e-4 of the scores; P and out are rounded to bf16 (2^-9 each)
            assert (lse[0, h][some].double() - ref_lse[some]).abs().max() <= 1e-4 * (1 + ref_lse[some].abs().max())
            assert (out[0, h].double() - ref).norm() <= 8e-3 * ref.norm() + 1e-6
    assert torch.isfinite(out).all() and torch.isfinite(lse[:, :, some]).all()
    m.free()


@pytest.mark.parametrize("H, nb", [(136, 4), (120, 3), (20, 131)])
def test_trace_of_pairs(H, nb):
    """One record for each head and block, taken with its neighbour, alone or in halves; the same results.  A workgroup's second block begins when its first ends."""
    import torch
    from paper_2506_19852_amd import binding as rb
    D = 128
    N = 128 * nb - 5
    m = rb.radial_mask_build_dense(N, 128, 0)
    q, k, v = (torch.randn((1, H, N, D), device="cuda").bfloat16() for _ in range(3))
    outs = [torch.empty_like(q) for _ in range(2)]
    lses = [torch.empty((1, H, N), dtype=torch.float32, device="cuda") for _ in range(2)]
    rb.radial_attn_fwd(q, k, v, outs[0], lses[0], m, D ** -0.5)
    trace = torch.zeros((rb.radial_attn_fwd_trace_records(1, H, m), 3), dtype=torch.int64, device="cuda")
    rb.radial_attn_fwd_trace(q, k, v, outs[1], lses[1], m, D ** -0.5, trace)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16)) and torch.equal(*lses)
    t = trace.cpu().numpy()
    used = t[:, 1] != 0
    assert int(used.sum()) == H * nb
    assert np.all(t[used, 1] >= t[used, 0]) and np.all(t[~used] == 0)
    in_pairs = int(np.sum((t[8:, 0] == t[:-8, 1]) & (t[8:, 0] != 0)))   # a pair's records are 8 apart; a tick is 10 ns
    assert in_pairs >= H * nb // 4 if nb != 3 else in_pairs < 8
    # by the workgroup that wrote it: workgroups go round the XCDs, from whichever the launch begins at; but for the last pairs in halves where their number is no multiple of 8
    assert np.bincount((np.flatnonzero(used) - (t[used, 2] >> 32 & 0xf)) & 7).max() >= 0.95 * H * nb
    m.free()
