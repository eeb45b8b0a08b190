"""Infinities and NaN in single rows of one head's inputs, in the kernels over pairs of query blocks (bf16 and 8-bit scores) and of key blocks: the outputs that
float64 gives as not finite are not, and every row that does not see the row in question keeps its bits."""
import numpy as np
import pytest

from test_gpu_two_blocks import make_lists

pytestmark = pytest.mark.gpu

HEAD, ROW = 5, 3 * 128 + 77


def launches(H, nb, cut):
    import torch
    from paper_2506_19852_amd import binding as rb
    D, N = 128, 128 * nb - cut
    g = torch.Generator(device="cuda").manual_seed(nb)
    x = {n: torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for n in ("q", "k", "v", "do")}
    bm = np.zeros((nb, nb), dtype=bool)
    for r, c in enumerate(make_lists(nb, "near", nb)):
        bm[r, c] = True
    bm[8:11] = bm[:, 8:11] = False     # blocks that see nothing of the others
    bm[[8, 9, 10], [8, 9, 10]] = True
    bm[6, 3], bm[7, 3] = True, False   # of two neighbours one sees the row
    bm[3, 6], bm[3, 7] = True, False
    m = rb.radial_mask_from_csr(N, 128, np.concatenate([[0], np.cumsum(bm.sum(1))]).astype(np.int32), np.nonzero(bm)[1].astype(np.int32), rb.RADIAL_MASK_TRANSPOSE)
    return rb, torch, x, bm, m, D ** -0.5


def untouched(torch, clean, got, rows_touched):
    """Other heads, and rows of other blocks, bit for bit."""
    same = (clean.view(torch.int16) == got.view(torch.int16)).all(-1) if clean.dtype == torch.bfloat16 else clean == got
    keep = torch.ones_like(same)
    keep[0, HEAD, rows_touched] = False
    assert same[keep].all()


# 20 heads of 131 blocks: both go by slices; 9 x 130 the forward by length
@pytest.mark.parametrize("H, nb, cut", [(20, 131, 97), (9, 130, 1)])
@pytest.mark.parametrize("what", ["q", "k", "v"])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("codes", [False, True])
def test_forward(H, nb, cut, what, value, codes):
    rb, torch, x, bm, m, scale = launches(H, nb, cut)
    print(f"H={H} nb={nb} {what} {value} codes={codes}", flush=True)
    N = x["q"].shape[2]

    def run():
        out, lse = torch.empty_like(x["v"]), torch.empty(x["v"].shape[:3], dtype=torch.float32, device="cuda")
        if not codes:
            rb.radial_attn_fwd(x["q"], x["k"], x["v"], out, lse, m, scale)
            return out, lse
        c = [torch.empty(out.shape, dtype=torch.uint8, device="cuda") for _ in range(2)]
        s = [torch.empty((1, H, nb), dtype=torch.float32, device="cuda") for _ in range(2)]
        for t, tc, ts in zip((x["q"], x["k"]), c, s):
            rb.radial_quantize_fp8(t, 128, tc, ts)
        rb.radial_attn_fwd_fp8(c[0], s[0], c[1], s[1], x["v"], out, lse, m, scale)
        return out, lse

    clean = run()
    assert all(torch.isfinite(t).all() for t in clean)
    x[what][0, HEAD, ROW, 9] = value
    out, lse = run()
    block = torch.from_numpy(bm[:, ROW // 128].copy() if what != "q" else np.arange(nb) == ROW // 128).cuda()
    sees = block.repeat_interleave(128)[:N]
    for before, after in zip(clean, (out, lse)):
        untouched(torch, before, after, sees)
    if what == "v":    # every row that sees the key, in that column only; the weights stay
        assert not torch.isfinite(out[0, HEAD, sees, 9]).any() and torch.equal(clean[1], lse)
        other = torch.arange(128, device="cuda") != 9
        assert torch.equal(out[..., other], clean[0][..., other])
    elif not codes:    # the row itself, or each of those that see the key: a weight of inf / inf, but for -inf scores, which weigh nothing
        s = x["q"][0, HEAD].double() @ x["k"][0, HEAD].double().T
        s = s.masked_fill(~torch.from_numpy(bm).cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)[:N, :N], float("-inf"))
        bad = (torch.isnan(s) | torch.isposinf(s)).any(1)
        assert not torch.isfinite(out[0, HEAD][bad]).any() and torch.isfinite(out[0, HEAD][~bad]).all() and bad.any()
    m.free()


@pytest.mark.parametrize("what", ["q", "k", "v", "do"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_backward(what, value):
    rb, torch, x, bm, m, scale = launches(20, 131, 97)
    print(f"{what} {value}", flush=True)
    N = x["q"].shape[2]
    out, lse = torch.empty_like(x["q"]), torch.empty(x["q"].shape[:3], dtype=torch.float32, device="cuda")
    rb.radial_attn_fwd(x["q"], x["k"], x["v"], out, lse, m, scale)
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, 20, N, 128, m), dtype=torch.uint8, device="cuda")

    def run():
        d = [torch.empty_like(out) for _ in range(3)]
        rb.radial_attn_bwd(x["q"], x["k"], x["v"], out, x["do"], lse, *d, m, scale, ws)
        return d

    clean = run()
    assert all(torch.isfinite(t).all() for t in clean)
    x[what][0, HEAD, ROW, 9] = value
    got = run()
    at = ROW // 128
    if what in ("k", "v"):     # query blocks that list the key block, and the key block
        query, key = bm[:, at], np.arange(131) == at
    else:                      # the query block, and the key blocks that it lists
        query, key = np.arange(131) == at, bm[at]
    for d, blocks in zip(range(3), (query, key, key)):
        untouched(torch, clean[d], got[d], torch.from_numpy(blocks.copy()).cuda().repeat_interleave(128)[:N])
    if what == "do":
        assert not torch.isfinite(got[0][0, HEAD, ROW]).any()
        seen = torch.from_numpy(key.copy()).cuda().repeat_interleave(128)[:N]
        assert not torch.isfinite(got[1][0, HEAD, seen]).any() and not torch.isfinite(got[2][0, HEAD, seen, 9]).any()
    m.free()
