"""Which workgroup takes which (head, block): launches whose heads are taken by slices, by falling list
length, or some each way give every head the result it has when it is computed alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# Up to 8 heads: all by length; above: the last 8 by length, the rest by slices.
@pytest.mark.parametrize("B, H, N, extra", [(1, 3, 2085, 70), (1, 8, 1000, 0), (1, 19, 1313, 0), (2, 11, 2048, 33), (1, 1, 1, 0)])
def test_every_head_gets_its_own_result(B, H, N, extra):
    import torch
    from paper_2506_19852_amd import binding as rb
    D = 128
    n = N + extra
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v, do = (torch.randn((B, H, n, D), device="cuda", generator=g).bfloat16() for _ in range(4))
    frames = 4 if N >= 4 else 1
    m = rb.radial_mask_build(frames, N // frames, 128, 1, rb.RADIAL_MASK_TRANSPOSE, extra_tokens=n - frames * (N // frames))

    def step(q, k, v, do):
        q, k, v, do = (t.contiguous() for t in (q, k, v, do))
        b, h = q.shape[:2]
        out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
        lse = torch.full((b, h, n), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.empty(rb.radial_attn_bwd_workspace(b, h, n, D, m), dtype=torch.uint8, device="cuda")
        rb.radial_attn_fwd(q, k, v, out, lse, m, D ** -0.5)
        rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, D ** -0.5, ws)
        return out, lse, dq, dk, dv

    got = step(q, k, v, do)
    for b, h in {(0, 0), (0, H // 2), (B - 1, H - 1), (B - 1, H // 3)}:
        one = step(*(t[b:b + 1, h:h + 1] for t in (q, k, v, do)))
        for name, x, y in zip(("out", "lse", "dq", "dk", "dv"), got, one):
            x, y = x[b, h].double(), y[0, 0].double()
            assert torch.isfinite(x).all(), (name, b, h)
            # the same products in another order of summation: a bf16 rounding of P and of the result each way
            assert (x - y).norm() <= 2 ** -7 * y.norm() + 1e-12, (name, b, h)
    m.free()


def test_order_covers_all_blocks_of_caller_lists():
    """Lists of equal length, empty lists and one full list, through a caller's CSR."""
    import torch
    from paper_2506_19852_amd import binding as rb
    block, nb, D = 64, 37, 64
    n = nb * block - 5
    rows = [[] if r % 7 == 3 else (list(range(nb)) if r == 20 else [r, min(r + 1, nb - 1)][: 1 if r == nb - 1 else 2]) for r in range(nb)]
    row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    m = rb.radial_mask_from_csr(n, block, row_ptr, np.array(sum(rows, []), dtype=np.int32))
    g = torch.Generator(device="cuda").manual_seed(4)
    q, k, v = (torch.randn((1, 2, n, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    out = torch.full_like(q, float("nan"))
    rb.radial_attn_fwd(q, k, v, out, None, m, D ** -0.5)
    for r, cols in enumerate(rows):
        rs = slice(r * block, min(n, (r + 1) * block))
        if not cols:
            assert (out[:, :, rs] == 0).all()
            continue
        keys = torch.cat([torch.arange(c * block, min(n, (c + 1) * block), device="cuda") for c in cols])
        for h in range(2):
            p = torch.softmax(q[0, h, rs].double() @ k[0, h, keys].double().T * D ** -0.5, dim=1)
            ref = p @ v[0, h, keys].double()
            assert ((out[0, h, rs].double() - ref).abs() <= 1e-2 + 1e-2 * ref.abs()).all(), r
    m.free()


@pytest.mark.parametrize("block, H, N", [(128, 20, 12 * 128), (64, 20, 12 * 64 - 5), (64, 85, 3 * 64), (64, 40, 12 * 64)])
def test_small_launches_of_many_heads_start_no_idle_workgroups(block, H, N):
    """Up to 256 (head, block) items, 512 in blocks of 64, the records of the traced forward are those of the first `items` workgroups."""
    import torch
    from paper_2506_19852_amd import binding as rb
    D, nb = 128, -(-N // block)
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((1, H, N, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    m = rb.radial_mask_build_dense(N, block)
    out = torch.full_like(q, float("nan"))
    lse = torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    trace = torch.zeros((rb.radial_attn_fwd_trace_records(1, H, m), 3), dtype=torch.int64, device="cuda")
    rb.radial_attn_fwd_trace(q, k, v, out, lse, m, D ** -0.5, trace)
    used = torch.nonzero(trace[:, 1]).flatten()
    assert used.numel() == H * nb and int(used.max()) == H * nb - 1
    for h in (0, H // 2, H - 1):
        ref = torch.softmax(q[0, h].double() @ k[0, h].double().T * D ** -0.5, dim=1) @ v[0, h].double()
        assert (out[0, h].double() - ref).norm() <= 8e-3 * ref.norm(), h   # P and out rounded to bf16
    m.free()
