"""The work a user of this library has it do, as timed cases.

A case is one pass through the public entry points of `paper_2506_19852_amd.binding`:

  fwd    one attention layer on a block list that the program keeps (denoising step of a video model);
  train  forward and backward of one layer (tuning step): out, lse, dq, dk, dv;
  fp8    quantise q and k, then the forward with 8-bit scores (what a layer does on each call, since
         q and k are new each time);
  shape  a new video shape arrives: build its block lists, then the forward of the first layer on them.

Inputs are iid N(0,1) in bf16, as in the repository's workloads (the rotary embedding applied there
rotates pairs of iid normals and leaves their distribution as it is, so it is not repeated here).
`gain` scales q: 1 gives the flat softmax of such inputs, larger values the peaked rows that trained
heads show.  `layout` is the memory order: "bhnd" (contiguous [B, H, N, D]) or "bnhd" (the
[B, N, H, D] tensors that projection layers produce, seen as [B, H, N, D] through strides).
"""
import math

import numpy as np
import torch

from paper_2506_19852_amd import binding as rb

DEVICE = "cuda:0"


def _case(kind, f, s, **kw):
    c = {"kind": kind, "B": 1, "H": 1, "D": 128, "frames": f, "tokens_per_frame": s, "block": 128, "sink_frames": 1,
         "extra_tokens": 0, "width_num": 1, "width_den": 1, "token_rule": False, "dense": False, "layout": "bhnd", "gain": 1.0}
    c.update(kw)
    return c


def listed():
    return [
        # The repository's tiny workload: 2 048 tokens, two heads.  Latency and launches are all there is.
        _case("fwd", 8, 256, name="tiny_fwd", H=2, D=64, block=64),
        # Tuning step of a small model (head dimension 64, 64-token blocks) on a clip of ragged size.
        _case("train", 8, 333, name="small_train", H=4, D=64, block=64, layout="bnhd"),
        # A short clip on one of eight GPUs that share 40 heads (5 each), conditional and unconditional
        # branch in one batch.
        _case("fwd", 9, 1560, name="clip_fwd", B=2, H=5, layout="bnhd", gain=2.0),
        # 480p, 21 latent frames, a whole 40-head layer.
        _case("fwd", 21, 1560, name="wan480p_fwd", H=40),
        # The same layer with the all-ones list: full attention, as the first denoising steps use it.
        _case("fwd", 21, 1560, name="wan480p_dense_fwd", H=40, dense=True),
        # 720p, default length, a whole 24-head layer: the benchmark's headline.
        _case("fwd", 33, 3600, name="hunyuan720p_fwd", H=24),
        # 720p, four times longer: the largest forward.
        _case("fwd", 129, 3600, name="hunyuan720p_4x_fwd", H=24),
        # 720p with prompt tokens behind the video and the sparsity knob, three heads of a layer shared
        # by eight GPUs.
        _case("fwd", 33, 3600, name="text_fwd", H=3, extra_tokens=226, width_num=13, width_den=20, layout="bnhd", gain=2.0),
        # 8-bit scores on the same share of heads.
        _case("fp8", 33, 3600, name="fp8_scores_fwd", H=3),
        # Tuning step under the token rule, five of 40 heads.
        _case("train", 21, 1560, name="token_rule_train", H=5, token_rule=True, layout="bnhd"),
        # 480p, four times longer, whole layer, forward and backward: the tuning workload.
        _case("train", 81, 1560, name="wan480p_4x_train", H=40),
        # First layer of a short clip whose shape is new, five of 40 heads: list construction and forward.
        _case("shape", 9, 1560, name="new_shape_fwd", H=5),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# Largest drawn case: all-ones flops of a call, forward (backward: 2.5 times more).  The largest listed
# case does 5.9e14 on its list.
_DRAW_FLOPS = 3.0e14


def draw(rng):
    while True:
        kind = rng.choice(("fwd", "fwd", "fwd", "train", "train", "train", "fp8", "shape"))
        f, s = _log_int(rng, 2, 129), _log_int(rng, 64, 3600)
        c = _case(kind, f, s, sink_frames=rng.choice((1, 1, 1, 0, 2)), B=rng.choice((1, 1, 2)),
                  H=_log_int(rng, 1, 40), layout=rng.choice(("bhnd", "bnhd")), gain=rng.choice((1.0, 1.0, 2.0, 4.0)))
        if kind != "fp8":
            c.update(D=rng.choice((64, 128, 128, 128)), block=rng.choice((64, 128, 128, 128)), token_rule=rng.random() < 0.25)
            c["dense"] = not c["token_rule"] and rng.random() < 0.15
        if not c["dense"]:
            if rng.random() < 0.3:
                c["extra_tokens"] = rng.randint(1, 512)
            if rng.random() < 0.3:
                c["width_num"], c["width_den"] = rng.choice(((13, 20), (1, 2), (3, 2)))
        n = f * s + c["extra_tokens"]
        if 4.0 * c["D"] * n * n * c["B"] * c["H"] * (3.5 if kind == "train" else 1.0) <= _DRAW_FLOPS:
            return c


def _n_tokens(c):
    return c["frames"] * c["tokens_per_frame"] + (0 if c["dense"] else c["extra_tokens"])


def _build_mask(c, transpose):
    flags = rb.RADIAL_MASK_TRANSPOSE if transpose else 0
    if c["dense"]:
        return rb.radial_mask_build_dense(_n_tokens(c), c["block"], flags)
    if c["token_rule"]:
        flags |= rb.RADIAL_MASK_TOKEN_EXACT
    return rb.radial_mask_build(c["frames"], c["tokens_per_frame"], c["block"], c["sink_frames"], flags,
                                width_num=c["width_num"], width_den=c["width_den"], extra_tokens=c["extra_tokens"])


def _empty(c):
    B, H, N, D = c["B"], c["H"], _n_tokens(c), c["D"]
    if c["layout"] == "bnhd":
        return torch.empty((B, N, H, D), dtype=torch.bfloat16, device=DEVICE).transpose(1, 2)
    return torch.empty((B, H, N, D), dtype=torch.bfloat16, device=DEVICE)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    x = {}
    for name in ("q", "k", "v") + (("dout",) if c["kind"] == "train" else ()):
        x[name] = _empty(c).normal_(0.0, c["gain"] if name == "q" else 1.0, generator=gen)
    st = {"case": c, "scale": 1.0 / math.sqrt(c["D"]), "mask": _build_mask(c, c["kind"] == "train"), "out": _empty(c), **x}
    B, H, N, D = c["B"], c["H"], _n_tokens(c), c["D"]
    st["lse"] = torch.empty((B, H, N), dtype=torch.float32, device=DEVICE)
    if c["kind"] == "train":
        st.update(dq=_empty(c), dk=_empty(c), dv=_empty(c),
                  workspace=torch.empty(rb.radial_attn_bwd_workspace(B, H, N, D, st["mask"]), dtype=torch.uint8, device=DEVICE))
    if c["kind"] == "fp8":
        for t in ("q", "k"):
            st[t + "8"] = torch.empty((B, H, N, D), dtype=torch.uint8, device=DEVICE)
            st[t + "s"] = torch.empty((B, H, (N + c["block"] - 1) // c["block"]), dtype=torch.float32, device=DEVICE)
    return st


def run(state):
    st = state
    kind = st["case"]["kind"]
    if kind == "shape":  # the build waits for the stream, so nothing uses the previous shape's lists any more
        previous, st["mask"] = st["mask"], _build_mask(st["case"], False)
        previous.free()
    if kind == "fp8":
        block = st["case"]["block"]
        rb.radial_quantize_fp8(st["q"], block, st["q8"], st["qs"])
        rb.radial_quantize_fp8(st["k"], block, st["k8"], st["ks"])
        rb.radial_attn_fwd_fp8(st["q8"], st["qs"], st["k8"], st["ks"], st["v"], st["out"], st["lse"], st["mask"], st["scale"], code_block=block)
        return {n: st[n] for n in ("out", "lse", "q8", "qs", "k8", "ks")}
    rb.radial_attn_fwd(st["q"], st["k"], st["v"], st["out"], st["lse"], st["mask"], st["scale"])
    if kind != "train":
        return {"out": st["out"], "lse": st["lse"]}
    rb.radial_attn_bwd(st["q"], st["k"], st["v"], st["out"], st["dout"], st["lse"], st["dq"], st["dk"], st["dv"], st["mask"],
                       st["scale"], st["workspace"])
    return {n: st[n] for n in ("out", "lse", "dq", "dk", "dv")}


def _token_pairs(c):
    """Visible token pairs of the radial mask (what the token rule asks for)."""
    f, s = c["frames"], c["tokens_per_frame"]
    num, den, sink, extra = c["width_num"], c["width_den"], c["sink_frames"], c["extra_tokens"]
    total = 0
    for d in range(f):
        if d < 2:
            w = s
        else:
            b = 1 << (d.bit_length() - 1)
            w = min(s, s * num // (den * b))
            if w < 1:
                w = 1 if d % -(-b * den // (s * num)) == 0 else 0
        pairs = s + 2 * ((w - 1) * s - (w - 1) * w // 2) if w >= 1 else 0  # |k - l| <= w - 1
        key_after = max(0, f - d - sink)                       # key frame j = i + d, not a sink
        key_before = max(0, f - d - sink) if d > 0 else 0      # key frame j = i - d >= sink
        if d > 0:
            key_after = sum(1 for j in range(sink, f) if j - d >= 0)
        total += pairs * (key_after + key_before)
    total += min(sink, f) * s * f * s
    return total + extra * (2 * f * s + extra)


def _listed_pairs(c):
    """(token pairs of the listed blocks, listed block pairs)."""
    n, blk = _n_tokens(c), c["block"]
    nb = (n + blk - 1) // blk
    if c["dense"]:
        return n * n, nb * nb
    mask = _build_mask(c, False)
    row_ptr, col_idx = rb.radial_mask_copy_to_host(mask)
    mask.free()
    size = np.full(nb, blk, dtype=np.int64)
    size[-1] = n - (nb - 1) * blk
    return int(np.repeat(size, np.diff(row_ptr)) @ size[col_idx]), int(row_ptr[-1])


def work(case):
    c = case
    n = _n_tokens(c)
    pairs, blocks = _listed_pairs(c)
    if c["token_rule"]:
        pairs = _token_pairs(c)
    heads = c["B"] * c["H"]
    tensor = 2.0 * heads * n * c["D"]
    lse = 4.0 * heads * n
    forward = 4.0 * c["D"] * pairs * heads
    if c["kind"] == "train":  # q, k, v, dout read once, out, dq, dk, dv written once; 2 + 5 products
        return {"bytes": 8 * tensor + lse, "flops": 3.5 * forward}
    if c["kind"] == "fp8":    # q, k, v read once, out and the codes of q and k written once
        return {"bytes": 5 * tensor + lse, "flops": forward}
    lists = 4.0 * (blocks + (n + c["block"] - 1) // c["block"] + 1) if c["kind"] == "shape" else 0.0
    return {"bytes": 4 * tensor + lse + lists, "flops": forward}


def tolerance(case):
    """Outputs are bf16 and P and dS are rounded to bf16 between the two products.  Measured against
    float64 over these ranges: relative 2-norm error at most 2.3e-3 (out) and 3.8e-3 (gradients at
    gain 4), largest single difference 1.3e-2 (forward) and 6.2e-2 (gradients) of the value or the root
    mean square; about four times that is allowed.  lse is float32 and agrees to 2e-6; codes of the
    8-bit scores have to be the same."""
    if case["kind"] == "train":
        return {"rel": 1.5e-2, "max": 0.25}
    return {"rel": 1e-2, "max": 5e-2}


# Token pairs of all heads up to which `exact` is computed (a few seconds; a training step costs three times more).
_EXACT_PAIRS = 5.0e10


def _half_widths(c):
    """Largest |k - l| that frames at distance 0 .. f-1 see of each other, -1: nothing."""
    s, num, den = c["tokens_per_frame"], c["width_num"], c["width_den"]
    hw = []
    for d in range(c["frames"]):
        b = 1 << max(d.bit_length() - 1, 0)
        w = s if d < 2 else min(s, s * num // (den * b))
        hw.append(w - 1 if w >= 1 else (0 if d % -(-b * den // (s * num)) == 0 else -1))
    return hw


def _seen(c, r0, r1, hw):
    """[r1 - r0, N] bool: which keys the tokens r0 .. r1-1 attend (r0 is the first token of a block)."""
    n, s, blk = _n_tokens(c), c["tokens_per_frame"], c["block"]
    if c["dense"]:
        return torch.ones((r1 - r0, n), dtype=torch.bool, device=DEVICE)
    pos = torch.arange(n, dtype=torch.int32, device=DEVICE)
    frame, text = pos // s, pos >= c["frames"] * s
    at = pos - frame * s
    distance = (frame[r0:r1, None] - frame[None]).abs().clamp(max=c["frames"] - 1)
    vis = (at[r0:r1, None] - at[None]).abs() <= hw[distance]
    vis |= (frame < c["sink_frames"])[None] | text[None] | text[r0:r1, None]
    if c["token_rule"]:
        return vis
    nq, nk = -(-(r1 - r0) // blk), -(-n // blk)  # a block pair is listed if any token pair in it is visible
    padded = torch.zeros((nq * blk, nk * blk), dtype=torch.bool, device=DEVICE)
    padded[:r1 - r0, :n] = vis
    listed = padded.view(nq, blk, nk, blk).any(dim=3).any(dim=1)
    return listed.repeat_interleave(blk, 0).repeat_interleave(blk, 1)[:r1 - r0, :n]


def exact(case, seed):
    """The outputs of `run` in float64: the masks from their definition over token pairs, plain softmax attention."""
    c = case
    B, H, N, D = c["B"], c["H"], _n_tokens(c), c["D"]
    train, fp8 = c["kind"] == "train", c["kind"] == "fp8"
    if float(N) * N * B * H * (3.0 if train else 1.0) > _EXACT_PAIRS:
        return None
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    x = {}
    for name in ("q", "k", "v") + (("dout",) if train else ()):
        x[name] = _empty(c).normal_(0.0, c["gain"] if name == "q" else 1.0, generator=gen)
    res = {"out": torch.empty((B, H, N, D), dtype=torch.float64, device=DEVICE),
           "lse": torch.empty((B, H, N), dtype=torch.float64, device=DEVICE)}
    if train:
        res.update({n: torch.zeros((B, H, N, D), dtype=torch.float64, device=DEVICE) for n in ("dq", "dk", "dv")})
    if fp8:  # codes: x / scale in 8 bits (4 exponent, 3 mantissa bits), one scale per block; the scores are those of the codes
        blk = c["block"]
        nb = -(-N // blk)
        for t in ("q", "k"):
            wide = torch.zeros((B, H, nb * blk, D), dtype=torch.float32, device=DEVICE)
            wide[:, :, :N] = x[t].float()
            amax = wide.abs().view(B, H, nb, blk * D).amax(dim=3)
            scales = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
            per_token = scales.repeat_interleave(blk, 2)[:, :, :N, None]
            codes = (wide[:, :, :N] / per_token).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
            res[t + "8"], res[t + "s"] = codes.view(torch.uint8), scales
            x[t] = codes.double() * per_token.double()
    scale = 1.0 / math.sqrt(D)
    hw = torch.tensor(_half_widths(c), dtype=torch.int32, device=DEVICE)
    step = 8 * c["block"]
    for b in range(B):
        for r0 in range(0, N, step):
            r1 = min(N, r0 + step)
            hidden = ~_seen(c, r0, r1, hw)
            for h in range(H):
                q, k, v = x["q"][b, h, r0:r1].double(), x["k"][b, h].double(), x["v"][b, h].double()
                p = (scale * (q @ k.T)).masked_fill_(hidden, -math.inf)
                lse = torch.logsumexp(p, dim=1)
                p = p.sub_(lse[:, None]).exp_()
                out = p @ v
                res["out"][b, h, r0:r1], res["lse"][b, h, r0:r1] = out, lse
                if train:
                    g = x["dout"][b, h, r0:r1].double()
                    ds = p * (g @ v.T - (g * out).sum(dim=1, keepdim=True))
                    res["dv"][b, h] += p.T @ g
                    res["dq"][b, h, r0:r1] = scale * (ds @ k)
                    res["dk"][b, h] += scale * (ds.T @ q)
    return res
