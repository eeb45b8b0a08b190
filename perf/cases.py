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
