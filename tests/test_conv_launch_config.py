"""Host-only: the rules by which the convolution passes choose their kernels, asked through w2l_conv1d_launch_config
(the functions that the entry points dispatch through)."""
import pytest

import paper_1812_07625_amd as P

FWD, BWD_DATA, BWD_WEIGHT = 0, 1, 2
REGISTERS, CHUNKS, PLAIN = 1, 2, 3
F32 = P.W2L_F32


def test_fp32_layers_take_the_unchecked_kernel_from_haloed_operands():
    shape = (4, 400, 256, 512, 11, 1, F32)
    assert [P.w2l_conv1d_launch_config(p, *shape)[0] for p in (FWD, BWD_DATA, BWD_WEIGHT)] == [PLAIN] * 3
    assert [P.w2l_conv1d_launch_config(p, *shape, False)[0] for p in (FWD, BWD_DATA)] == [CHUNKS] * 2


@pytest.mark.parametrize("pass_, shape", [
    (FWD, (1, 64, 5_700_000, 64, 3, 1)),          # 64 rows of w, 17.1 M values each: the last starts 4.3 GB behind the first
    (FWD, (64, 1024, 16416, 64, 1, 1024)),        # 64 rows of x in 64 utterances, 67 MB apart
    (BWD_DATA, (1, 64, 12_000_000, 64, 3, 1)),    # 32 rows of w, 36 M values each
    (BWD_DATA, (64, 1, 64, 1_200_000, 3, 1)),     # 64 rows of dy in 64 utterances of 17 frames
    (BWD_WEIGHT, (1, 64, 18_000_000, 64, 3, 1)),  # 32 frames of x
], ids=str)
def test_lines_too_far_apart_for_32_bit_offsets(pass_, shape):
    """The unchecked kernel keeps a lane's byte offset within its tile in 32 bits; lines further apart take the kernel
    that addresses with 64."""
    B, T, Cin, Cout, k, s = shape
    assert P.w2l_conv1d_launch_config(pass_, *shape, F32)[0] == CHUNKS
    # the same layer with its channels a hundredth as wide is near enough
    small = (B, T, max(64, Cin // 100 // 64 * 64), max(64, Cout // 100 // 64 * 64), k, s)
    assert P.w2l_conv1d_launch_config(pass_, *small, F32)[0] == PLAIN
