"""Small sequences in launches of many heads: above 256 blocks of 128 tokens, and above 1536 of 64, one group of waves
walks each list, as in every real layer.  The shapes whose edges matter (ragged ends, one token, frames that end
anywhere in a block, several frames in a block, text tokens), both memory orders, outputs between guard bands, sampled
heads against float64."""
import numpy as np
import pytest
import torch

from oracle import build as obuild
from oracle import mask as om
from paper_2506_19852_amd import binding as rb

from test_gpu_bwd import _guarded, _guards_intact
from test_gpu_list_split import reference

pytestmark = pytest.mark.gpu


def visible(f, s, extra, block, rule):
    n = f * s + extra
    if rule:
        return torch.from_numpy(om.token_mask_rows_with_text(f, s, 1, np.arange(n), extra)).cuda()
    bitmap, _ = obuild.mask_scan(f, s, block, 1, extra_tokens=extra)
    return torch.from_numpy(bitmap).cuda().repeat_interleave(block, 0).repeat_interleave(block, 1)[:n, :n]


@pytest.mark.parametrize("rule", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("f, s, extra, block", [
    (5, 200, 0, 128), (3, 333, 0, 128), (7, 100, 0, 128), (12, 70, 33, 128), (33, 64, 0, 128), (1, 65, 0, 128), (9, 93, 150, 128),
    (7, 100, 0, 64), (12, 70, 33, 64), (1, 65, 0, 64), (5, 129, 1, 64)])
def test_forward_and_backward(f, s, extra, block, D, rule):
    n = f * s + extra
    nb = -(-n // block)
    H = (256 if block == 128 else 1536) // nb + 1
    print(f"unsplit f={f} s={s} extra={extra} block={block} D={D} H={H} token rule={rule}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + D)
    shape = (1, n, H, D) if D == 128 else (1, H, n, D)
    view = (lambda t: t.transpose(1, 2)) if D == 128 else (lambda t: t)
    q, k, v, do = (view(torch.randn(shape, device="cuda", generator=g).bfloat16()) for _ in range(4))
    nbytes = H * n * D * 2
    bufs = {nm: _guarded(nbytes, 0xFF) for nm in ("out", "dq", "dk", "dv")}      # 0xFFFF is a bf16 NaN
    out, dq, dk, dv = (view(bufs[nm][1].view(torch.bfloat16).view(shape)) for nm in ("out", "dq", "dk", "dv"))
    lse_whole, lse_bytes = _guarded(H * n * 4, 0xFF)
    lse = lse_bytes.view(torch.float32).view(1, H, n)
    m = rb.radial_mask_build(f, s, block, 1, rb.RADIAL_MASK_TRANSPOSE | (rb.RADIAL_MASK_TOKEN_EXACT if rule else 0), extra_tokens=extra)
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, n, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, D ** -0.5)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, D ** -0.5, ws)
    torch.cuda.synchronize()
    for nm, (whole, _) in bufs.items():
        assert _guards_intact(whole, nbytes), nm
    assert _guards_intact(lse_whole, H * n * 4)
    for t in (out, lse, dq, dk, dv):
        assert torch.isfinite(t).all()
    vis = visible(f, s, extra, block, rule)
    for h in sorted({0, H // 2, H - 9, H - 8, H - 1} & set(range(H))):
        ref = reference(q[0, h], k[0, h], v[0, h], do[0, h], vis, D ** -0.5)
        # lse is float32; out and the gradients carry two to three bf16 roundings (2^-9 each, of P or dS, of the
        # result, and of out inside delta)
        assert (lse[0, h].double() - ref[1]).abs().max() <= 1e-4, h
        for name, x, r in zip(("out", "dq", "dk", "dv"), (out[0, h], dq[0, h], dk[0, h], dv[0, h]), (ref[0], *ref[2:])):
            assert (x.double() - r).norm() <= 8e-3 * r.norm(), (name, h, (x.double() - r).norm() / r.norm())
    m.free()


@pytest.mark.parametrize("D", [64, 128])
def test_one_token(D):
    """out = v and dv = dout exactly, lse = scale q.k, dq = dk = 0 to the rounding of two float32 sums."""
    H = 257
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v, do = (torch.randn((1, H, 1, D), device="cuda", generator=g).bfloat16() for _ in range(4))
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.full((1, H, 1), float("nan"), dtype=torch.float32, device="cuda")
    m = rb.radial_mask_build(1, 1, 128, 1, rb.RADIAL_MASK_TRANSPOSE)
    ws = torch.empty(rb.radial_attn_bwd_workspace(1, H, 1, D, m), dtype=torch.uint8, device="cuda")
    rb.radial_attn_fwd(q, k, v, out, lse, m, D ** -0.5)
    rb.radial_attn_bwd(q, k, v, out, do, lse, dq, dk, dv, m, D ** -0.5, ws)
    assert torch.equal(out, v) and torch.equal(dv, do)
    assert (lse[..., 0].double() - D ** -0.5 * (q.double() * k.double()).sum(3)[..., 0]).abs().max() <= 1e-4
    # dS = P (dP - delta), where dP and delta are the same D products summed in float32 in two orders: each sum is off by at
    # most D 2^-24 of the sum of their magnitudes, and P, dS and the result round by 2^-9 at most
    ds = 2 * D * 2.0 ** -24 * (do.double() * v.double()).abs().sum(3, keepdim=True) * 1.01
    assert (dq.double().abs() <= D ** -0.5 * ds * k.double().abs()).all() and (dk.double().abs() <= D ** -0.5 * ds * q.double().abs()).all()
    m.free()


@pytest.mark.parametrize("f, s, sink", [(6, 200, 1), (5, 333, 0), (3, 128, 1), (1, 50, 1), (40, 3, 0), (2, 300, 5)])
def test_8bit_scores(f, s, sink):
    D = block = 128
    n = f * s
    nb = -(-n // block)
    H = 256 // nb + 1
    print(f"unsplit 8-bit f={f} s={s} H={H}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((1, H, n, D), device="cuda", generator=g).bfloat16() for _ in range(3))
    codes, scales = [], []
    for x in (q, k):
        codes.append(torch.empty((1, H, n, D), dtype=torch.uint8, device="cuda"))
        scales.append(torch.empty((1, H, nb), dtype=torch.float32, device="cuda"))
        rb.radial_quantize_fp8(x, block, codes[-1], scales[-1])
    m = rb.radial_mask_build(f, s, block, sink)
    whole, payload = _guarded(H * n * D * 2, 0xFF)
    out = payload.view(torch.bfloat16).view(1, H, n, D)
    lse = torch.full((1, H, n), float("nan"), dtype=torch.float32, device="cuda")
    rb.radial_attn_fwd_fp8(codes[0], scales[0], codes[1], scales[1], v, out, lse, m, D ** -0.5)
    torch.cuda.synchronize()
    assert _guards_intact(whole, H * n * D * 2)
    bitmap, _ = obuild.mask_scan(f, s, block, sink)
    vis = torch.from_numpy(bitmap).cuda().repeat_interleave(block, 0).repeat_interleave(block, 1)[:n, :n]
    for h in (0, H - 1):
        qd, kd = (c[0, h].view(torch.float8_e4m3fn).double() * sc[0, h].double().repeat_interleave(block)[:n, None] for c, sc in zip(codes, scales))
        x = (D ** -0.5 * (qd @ kd.T)).masked_fill(~vis, float("-inf"))
        ref_lse = x.logsumexp(1)
        ref = (x - ref_lse[:, None]).exp() @ v[0, h].double()
        # the 8-bit matrix instruction's sums: 1e-4 of the scores; P and out are rounded to bf16 (2^-9 each)
        assert (lse[0, h].double() - ref_lse).abs().max() <= 1e-3
        assert (out[0, h].double() - ref).norm() <= 8e-3 * ref.norm()
    m.free()
