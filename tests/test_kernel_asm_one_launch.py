"""The promises of the dK/dV kernel's hand-issued MFMAs (test_kernel_asm.py) where it shares a launch with dQ."""
from test_kernel_asm import bwd_asm, check_kernel, instructions, kernels  # noqa: F401  (bwd_asm is a fixture)


def test_hand_issued_mfmas_keep_their_promises_beside_dq(bwd_asm):  # noqa: F811
    found = 0
    for name, body in kernels(bwd_asm, "radial_bwd_both_hand_kernel"):
        found += 1
        assert check_kernel(name, list(instructions(body))) > 0, name
    assert found == 4, found   # block in {64, 128} x token rule on / off
