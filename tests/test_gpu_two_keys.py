"""dK and dV over pairs of neighbouring key blocks (head dimension 128, blocks of 128, above 1536 blocks): heads by slices and by length, odd and
even numbers of blocks, ragged ends of queries and keys, neighbouring transposed lists that are equal, overlap, have nothing in common or are
empty (the last three one block at a time), lists of more entries than a wave looks at together, strided tensors, against float64."""
import numpy as np
import pytest

from test_gpu_list_split import reference
from test_gpu_two_blocks import make_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H, nb, cut, kind, layout", [
    (1600, 1, 60, "all", "bhnd"), (800, 2, 1, "mixed", "bnhd"), (530, 3, 127, "all", "bhnd"), (320, 5, 64, "mixed", "bhnd"), (225, 7, 33, "all", "bnhd"),
    (20, 131, 97, "near", "bnhd"), (13, 130, 1, "near", "bhnd"), (16, 101, 0, "all", "bnhd"), (20, 131, 31, "mixed", "bhnd")])
def test_gradients_match_float64(H, nb, cut, kind, layout):
    import torch
    from paper_2506_19852_amd import binding as rb
    print(f"H={H} nb={nb} cut={cut} {kind} {layout}", flush=True)
    D, N = 128, 128 * nb - cut
    g = torch.Generator(device="cuda").manual_seed(N + H)
    shape = (1, N, H, D) if layout == "bnhd" else (1, H, N, D)
    q, k, v, do = (torch.randn(shape, device="cuda", generator=g).bfloat16() for _ in range(4))
    if layout == "bnhd":
        q, k, v, do = (x.transpose(1, 2) for x in (q, k, v, do))
    if kind == "near":  # neighbouring key blocks' lists share most entries and have some alone
        rng = np.random.default_rng(nb)
        bm = np.repeat(rng.random(((nb + 1) // 2, nb)) < 0.8, 2, axis=0)[:nb] ^ (rng.random((nb, nb)) < 0.1)
    else:
        bm = np.zeros((nb, nb), dtype=bool)
        for key, rows in enumerate(make_lists(nb, kind, nb + H)):
            bm[key, rows] = True
    bm = bm.T  # rows: query blocks
    row_ptr = np.concatenate([[0], np.cumsum(bm.sum(1))]).astype(np.int32)
    m = rb.radial_mask_from_csr(N, 128, row_ptr, np.nonzero(bm)[1].astype(np.int32), rb.RADIAL_MASK_TRANSPOSE)
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.full((1, H, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, N, D, m), dtype=torch.uint8, device="cuda")
    scale = D ** -0.5
    rb.radial_attn_fwd(q, k, v, out, lse, m, scale)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, scale, ws)
    again = [torch.full_like(q, float("nan")) for _ in range(3)]
    rb.radial_attn_bwd(q, k, v, out, do, lse, *again, m, scale, ws)
    torch.cuda.synchronize()
    for x, y in zip((dq, dk, dv), again):
        assert torch.isfinite(x).all() and torch.equal(x.view(torch.int16), y.view(torch.int16))
    visible = torch.from_numpy(bm.copy()).cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)[:N, :N]
    for h in sorted({0, 1, H // 2, H - 2, H - 1}):
        want = reference(q[0, h], k[0, h].double(), v[0, h].double(), do[0, h], visible, scale)[2:]
        for name, x, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), want):
            # P and dS are rounded to bf16 between the products and the results once more, 2^-9 each; delta comes from the rounded output
            assert (x[0, h].double() - ref).norm() <= 1.2e-2 * ref.norm() + 1e-6, (h, name, float((x[0, h].double() - ref).norm() / ref.norm()))
            unlisted = ~visible.any(0) if name != "dq" else ~visible.any(1)
            assert (x[0, h][unlisted] == 0).all()
    m.free()
