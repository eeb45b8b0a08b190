"""Masks of different shapes built by several host threads at a time, each on a stream of its own: the lists, and a forward on them,
are those of masks built one after the other."""
import threading

import numpy as np
import pytest

from paper_2506_19852_amd import binding as rb

pytestmark = pytest.mark.gpu

SHAPES = [(3, 100 + 37 * i, 64 if i % 2 else 128, (i % 3) * 19) for i in range(8)] + [(12, 8000, 128, 0), (21, 2500, 64, 5)]  # the last two: counted


def build(shape, stream):
    f, s, block, extra = shape
    return rb.radial_mask_build(f, s, block, 1, rb.RADIAL_MASK_TRANSPOSE, stream=stream, extra_tokens=extra)


def results(shape, mask, stream):
    import torch
    n = shape[0] * shape[1] + shape[3]
    lists = rb.radial_mask_copy_to_host(mask) + rb.radial_mask_copy_transpose_to_host(mask)
    with torch.cuda.stream(stream):
        g = torch.Generator(device="cuda").manual_seed(n)
        q = torch.randn((1, 1, n, 64), device="cuda", generator=g).bfloat16()
        out = torch.empty_like(q)
        rb.radial_attn_fwd(q, q, q, out, None, mask, 0.125)
        return lists, out.cpu()


def test_threads_build_what_one_builds():
    import torch
    streams = [torch.cuda.Stream() for _ in SHAPES]
    want = []
    for shape, stream in zip(SHAPES, streams):
        mask = build(shape, stream)
        want.append(results(shape, mask, stream))
        mask.free()
    start, wrong = threading.Barrier(len(SHAPES)), []

    def work(i):
        try:
            start.wait(60)
            for _ in range(6):
                mask = build(SHAPES[i], streams[i])
                lists, out = results(SHAPES[i], mask, streams[i])
                mask.free()
                if not all(np.array_equal(a, b) for a, b in zip(lists, want[i][0])) or not torch.equal(out, want[i][1]):
                    wrong.append(SHAPES[i])
        except Exception as e:
            wrong.append((SHAPES[i], repr(e)))
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(SHAPES))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not any(t.is_alive() for t in threads) and not wrong, wrong
