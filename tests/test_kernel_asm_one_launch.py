"""The promises of the dK/dV kernel's hand-issued MFMAs (test_kernel_asm.py) where it shares a launch with dQ."""
import re

from test_kernel_asm import bwd_asm, check_kernel, instructions, kernels  # noqa: F401  (bwd_asm is a fixture)


def test_hand_issued_mfmas_keep_their_promises_beside_dq(bwd_asm):  # noqa: F811
    found = 0
    for name, body in kernels(bwd_asm, "radial_bwd_both_hand_kernel"):
        found += 1
        assert check_kernel(name, list(instructions(body))) > 0, name
    assert found == 4, found   # block in {64, 128} x token rule on / off


def test_backward_kernels_reserve_no_private_memory(bwd_asm):  # noqa: F811
    """Where one does, its first launch allocates some for the whole chip, which callers that cannot allocate or are near the end of the
    device's memory did not ask for."""
    sizes = re.findall(r"\.amdhsa_kernel (\S+).*?\.amdhsa_private_segment_fixed_size (\d+)", "\n".join(bwd_asm), re.S)
    assert len(sizes) > 40 and not [(name, size) for name, size in sizes if size != "0"]


def test_parts_of_a_common_launch_keep_their_scalars(bwd_asm):  # noqa: F811
    """Scalars written to vector lanes: a few (in pairs of waves under the token rule as many as alone), with or without the rule.  Not
    looked at in groups of one wave, where it is quicker to load what all parts need first."""
    found = 0
    for name, body in kernels(bwd_asm, "radial_bwd_both"):
        if "ELi4E" in name:
            continue
        found += 1
        spills = sum(1 for ins in instructions(body) if ins.startswith("v_writelane_b32"))
        assert spills <= 7, (name, spills)
    assert found == 20, found
