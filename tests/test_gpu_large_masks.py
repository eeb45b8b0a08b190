"""Masks of more than 16 384 blocks: their lists are counted, scanned and filled by kernels of their own, and their
launches have no order by list length.  16 385 frames of 64 tokens in 64-token blocks, so that a block is a frame and
a block pair is listed by the frames' distance alone."""
import numpy as np
import pytest

from oracle import mask as om

pytestmark = pytest.mark.gpu
F, S = 16385, 64


@pytest.fixture(scope="module")
def lists():
    """(row_ptr, col_idx, col_ptr, row_idx) from the definition, sink 1."""
    # a pair of frames has a visible pair of tokens iff it has one at equal positions (any position: here 0)
    by_distance = np.array([om.token_visible(F, S, 0, 0, d, 0, 0) for d in range(F)])
    both = np.concatenate([by_distance[:0:-1], by_distance])   # index d + F - 1, d = key - query
    rows, cols = [], []
    for i in range(F):
        r = both[F - 1 - i: 2 * F - 1 - i].copy()
        r[0] = True                                              # key frame 0 is the sink
        rows.append(np.flatnonzero(r).astype(np.int32))
        cols.append(np.flatnonzero(both[F - 1 - i: 2 * F - 1 - i]).astype(np.int32) if i else np.arange(F, dtype=np.int32))
    ptr = lambda x: np.concatenate([[0], np.cumsum([len(r) for r in x])]).astype(np.int32)
    return ptr(rows), np.concatenate(rows), ptr(cols), np.concatenate(cols)


def test_lists_forward_and_backward(lists):
    import torch
    from paper_2506_19852_amd import binding as rb
    row_ptr, col_idx, col_ptr, row_idx = lists
    plain = rb.radial_mask_build(F, S, 64, 1)
    for got, want in zip(rb.radial_mask_copy_to_host(plain), (row_ptr, col_idx)):
        assert np.array_equal(got, want)
    plain.free()
    m = rb.radial_mask_build(F, S, 64, 1, rb.RADIAL_MASK_TRANSPOSE)
    for got, want in zip((*rb.radial_mask_copy_to_host(m), *rb.radial_mask_copy_transpose_to_host(m)), lists):
        assert np.array_equal(got, want)
    print("lists compared", flush=True)
    given = rb.radial_mask_from_csr(F * S, 64, row_ptr, col_idx, rb.RADIAL_MASK_TRANSPOSE)
    for got, want in zip(rb.radial_mask_copy_transpose_to_host(given), (col_ptr, row_idx)):
        assert np.array_equal(got, want)

    D, n, scale = 64, F * S, 64 ** -0.5
    g = torch.Generator(device="cuda").manual_seed(7)
    q, k, v, do = (torch.randn((1, 1, n, D), device="cuda", generator=g).bfloat16() for _ in range(4))
    out, again, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(5))
    lse = torch.full((1, 1, n), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, 1, n, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, again, None, given, scale)
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    assert torch.equal(out.view(torch.int16), again.view(torch.int16))
    for t in (out, lse, dq, dk, dv):
        assert torch.isfinite(t).all()
    print("forward and backward ran", flush=True)
    tokens = lambda blocks: (torch.from_numpy(blocks.astype(np.int64)).cuda()[:, None] * S + torch.arange(S, device="cuda")).flatten()
    h = [t[0, 0].double() for t in (q, k, v, do)]
    delta = (h[3] * out[0, 0].double()).sum(1)
    for b in (0, 1, F // 3, F - 1):
        at = slice(b * S, (b + 1) * S)
        keys = tokens(col_idx[row_ptr[b]:row_ptr[b + 1]])
        s = scale * (h[0][at] @ h[1][keys].T)
        ref_lse = s.logsumexp(1)
        p = (s - ref_lse[:, None]).exp()
        ref = p @ h[2][keys]
        ds = p * (h[3][at] @ h[2][keys].T - (h[3][at] * ref).sum(1, keepdim=True))
        # lse is float32; out and the gradients carry two to three bf16 roundings (2^-9 each)
        assert (lse[0, 0, at].double() - ref_lse).abs().max() <= 1e-4
        for name, x, r in (("out", out, ref), ("dq", dq, scale * (ds @ h[1][keys]))):
            assert (x[0, 0, at].double() - r).norm() <= 8e-3 * r.norm(), (name, b)
        if b == 0:
            continue                                              # the sink's column lists every row: a million queries
        rows = tokens(row_idx[col_ptr[b]:col_ptr[b + 1]])
        p = (scale * (h[0][rows] @ h[1][at].T) - lse[0, 0, rows].double()[:, None]).exp()
        ds = p * (h[3][rows] @ h[2][at].T - delta[rows][:, None])
        for name, x, r in (("dv", dv, p.T @ h[3][rows]), ("dk", dk, scale * (ds.T @ h[0][rows]))):
            assert (x[0, 0, at].double() - r).norm() <= 8e-3 * r.norm(), (name, b)
    m.free()
    given.free()
