"""List construction on both sides of the size at which the storage is sized by counting (720 blocks), bit-exact
against the oracle's scan, and the launch partitions that come with it: every block of every head is worked on."""
import numpy as np
import pytest

from oracle import build as obuild
from oracle import mask as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames, s, block", [(1, 1, 64), (2, 70, 128), (5, 9216, 64), (5, 9229, 64), (7, 13166, 128)])
@pytest.mark.parametrize("transpose", [False, True])
def test_lists_and_partitions(frames, s, block, transpose):
    import torch
    from paper_2506_19852_amd import binding as rb
    n = frames * s
    m = rb.radial_mask_build(frames, s, block, 1, rb.RADIAL_MASK_TRANSPOSE if transpose else 0)
    bitmap, _ = obuild.mask_scan(frames, s, block, 1)
    row_ptr, col_idx = om.block_lists(bitmap)
    got_ptr, got_idx = rb.radial_mask_copy_to_host(m)
    assert np.array_equal(got_ptr, row_ptr) and np.array_equal(got_idx, col_idx)
    if transpose:
        col_ptr, row_idx = om.block_lists(np.ascontiguousarray(bitmap.T))
        got_ptr, got_idx = rb.radial_mask_copy_transpose_to_host(m)
        assert np.array_equal(got_ptr, col_ptr) and np.array_equal(got_idx, row_idx)
    # 9 heads: one by slices, eight by list length; q = 0 makes every output the mean of the listed values, here 1
    shape = (1, 9, n, 64)
    q, k = torch.zeros(shape, dtype=torch.bfloat16, device="cuda"), torch.ones(shape, dtype=torch.bfloat16, device="cuda")
    out = torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    rb.radial_attn_fwd(q, k, k, out, None, m, 0.125)
    assert (out == 1).all()
    m.free()
