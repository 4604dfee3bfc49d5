"""Host-only: the rules by which the convolution passes choose their kernels, asked through w2l_conv1d_launch_config
(the functions that the entry points dispatch through)."""
import ctypes

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


STRIDED = [(B, T, cin, cout, k, s) for B, T in ((1, 200), (4, 400), (4, 1600), (16, 1600)) for cin, cout in ((64, 64), (256, 512), (1024, 1024))
           for k in (3, 11) for s in (1, 2, 4, 8)]


@pytest.mark.parametrize("dtype", [P.W2L_F32, P.W2L_BF16])
def test_planes_of_a_data_gradient_stay_within_their_bound(dtype):
    """Every split of the reduction leaves a plane of the whole dx, whatever the stride: 96 MB in all at most."""
    split = 0
    for B, T, cin, cout, k, s in STRIDED:
        cin += dtype == P.W2L_BF16                          # (a channel count that the bf16 kernels do not take)
        shape = (B, T, cin, cout, k, s, dtype)
        form, splits = P.w2l_conv1d_launch_config(BWD_DATA, *shape)
        assert form != 0 and (splits == 1 or splits * B * T * cin * 4 <= 96 << 20), (shape, splits)
        copy = (B * (T + 16) + 320) * cout * 4 if form == PLAIN else 0
        assert P.w2l_conv1d_bwd_data_workspace_bytes(*shape) <= copy + (96 << 20) + 512, shape
        split += s > 1 and splits > 1
    assert split >= 4


def test_many_short_utterances_do_not_walk():
    """The walk through the frames of a haloed layout counts 17 for every utterance of one frame: beyond 2^30 of them the
    weight gradient counts real frames."""
    assert P.w2l_conv1d_launch_config(BWD_WEIGHT, 1 << 27, 1, 4, 36, 3, 1, F32)[0] == CHUNKS
    assert P.w2l_conv1d_launch_config(BWD_WEIGHT, 1 << 20, 1, 4, 36, 3, 1, F32)[0] == PLAIN


def test_networks_on_two_streams_reserve_no_planes():
    """The 105M-parameter network keeps its bf16 weight gradients whole (their workgroups and the data gradients' share the
    chip from two streams): its workspace holds no planes for them (24 MB on either stream; 467 MB without)."""
    import workloads as W
    n = P.w2l_train_step_workspace_bytes(W.layers_105m(), 8, 1500, 93, P.W2L_BF16)
    assert 460e6 < n < 490e6, n


@pytest.mark.parametrize("pass_, shape, splits", [
    (FWD, (13, 1063, 512, 256, 5, 2), 4), (FWD, (3, 900, 512, 512, 7, 2), 4), (FWD, (8, 1063, 256, 512, 5, 2), 2),   # strided: dense operands
    (FWD, (2, 700, 512, 512, 19, 1), 7), (BWD_DATA, (2, 700, 512, 512, 19, 1), 7), (BWD_WEIGHT, (5, 1505, 80, 832, 19, 1), 4),  # a window wider than the halo
], ids=str)
def test_runs_fit_the_kernel_that_is_launched(pass_, shape, splits):
    """fp32 layers that are not brought into the haloed layout run on the fp32 instruction, and are split for its cost: the
    runs that their times were fitted with, not those of the kernel for haloed operands."""
    assert P.w2l_conv1d_launch_config(pass_, *shape, F32) == (CHUNKS, splits)


@pytest.mark.parametrize("pass_, shape, tile", [
    # a few panels a workgroup: what the kernel for bf16 terms adds to a launch is more than it saves
    (FWD, (9, 63, 64, 768, 11), (64, 0)), (FWD, (9, 1431, 64, 592, 1), (64, 0)), (BWD_DATA, (4, 1062, 160, 128, 3), (64, 0)),
    (BWD_DATA, (6, 249, 256, 448, 1), (64, 0)), (BWD_WEIGHT, (3, 148, 160, 384, 5), (64, 0)), (BWD_WEIGHT, (1, 583, 96, 512, 7), (64, 0)),
    # longer ones, few and many tiles
    (FWD, (4, 400, 256, 512, 11), (64, 1)), (BWD_DATA, (4, 400, 256, 512, 11), (64, 1)), (BWD_WEIGHT, (4, 200, 256, 512, 11), (64, 1)),
    (FWD, (16, 800, 256, 512, 11), (128, 1)), (BWD_DATA, (16, 800, 256, 512, 11), (128, 1)), (BWD_WEIGHT, (16, 800, 256, 512, 11), (128, 1)),
], ids=str)
def test_fp32_passes_alone_take_bf16_terms_where_that_is_faster(pass_, shape, tile):
    """By the times of either kernel, 6 to 24 % of a pass in the first group (the weight gradients: 5 % of their layer)."""
    assert P.w2l_conv1d_launch_tile(pass_, *shape, 1, F32) == tile


def test_strides_fold_only_for_the_matrix_kernels():
    """A strided bf16 weight gradient whose x is beyond the matrix kernels' 32-bit offsets is not copied into folded frames,
    which the other kernels cannot read."""
    copies = lambda T: P.w2l_conv1d_bwd_weight_workspace_bytes(64, T, 512, 64, 5, 2, P.W2L_BF16) > 64 * T * 512 * 2
    assert copies(8000) and not copies(40000)


def test_class_layer_launch_has_fewer_than_2_32_threads():
    """A thread of the class layer's launch has four frames of one group of channels, 32 groups a workgroup: networks of more
    frames than 2^32 threads have room for keep the launches that walk."""
    ok = P.raw._ZN3w2l16class_bwd_glu_okEiiiiii  # (B, pitch, slack, C, H, dtype)
    ok.restype = ctypes.c_bool
    assert ok(60000, 8940, 64, 2, 256, P.W2L_BF16) and not ok(60000, 8960, 64, 2, 256, P.W2L_BF16)
    assert ok(1 << 10, (1 << 19) - 1, 512, 29, 128, F32) and not ok(1 << 10, 1 << 19, 0, 29, 128, F32)


def _net(widths, k, feat=40, classes=29, stride=2, head=None):
    layers = [dict(k=k, stride=stride if i == 0 else 1, cin=c, cout=w, glu=1) for i, (c, w) in enumerate(zip([feat] + [w // 2 for w in widths[:-1]], widths))]
    if head:
        layers.append(dict(k=1, stride=1, cin=widths[-1] // 2, cout=head, glu=1))
    return layers + [dict(k=1, stride=1, cin=(head or widths[-1]) // 2, cout=classes, glu=0)]


def _widths(layers, B, T, dtype=P.W2L_BF16):
    got = [P.w2l_train_step_layer_config(layers, B, T, dtype, i) for i in range(len(layers))]
    for i in range(1, len(layers)):
        assert got[i][0] == got[i - 1][1] // 2
    assert got[0][0] == layers[0]["cin"] and got[-1][1] == layers[-1]["cout"]
    return [g[1] for g in got[:-1]]


@pytest.mark.parametrize("layers, B, T, widths", [
    (_net([500] * 4, 7), 4, 800, [512] * 4),
    (_net([210, 250], 5), 3, 260, [256, 256]),
    (_net([496, 240, 332], 3, 80), 4, 800, [512, 256, 384]),
    (_net([40] * 4, 7), 16, 1600, [64] * 4),                  # 2.2 times the products
    (_net([66] * 4, 7), 4, 800, [128] * 4),                   # 3.4 times, all halves 64
    (_net([448] * 4, 7, head=1000), 4, 800, [448] * 4 + [1024]),  # layers on the blocks keep their widths
    (_net([500] * 4, 7, classes=100), 4, 800, [512] * 4),
    (_net([240] * 4, 7), 2, 200, [256] * 4),                  # (data gradients only)
    # as they are: on the blocks; features of no whole four; nothing gained; narrow; few products; few frames
    (_net([512] * 4, 7), 4, 800, [512] * 4),
    (_net([500] * 4, 7, feat=42), 4, 800, [500] * 4),
    (_net([64] * 4, 7, head=200), 4, 800, [64] * 4 + [200]),
    (_net([496], 7), 16, 1600, [496]),
    (_net([24] * 4, 7), 16, 1600, [24] * 4),
    (_net([32] * 4, 13), 16, 1600, [32] * 4),
    (_net([140] * 4, 5), 1, 280, [140] * 4),
    (_net([500] * 4, 7), 1, 254, [500] * 4),
    # tensors beyond the matrix kernels' 32-bit offsets, at the wide width and at both
    (_net([1100] * 4, 5, stride=1), 64, 18000, [1100] * 4),
    (_net([1000] * 4, 5, stride=1), 64, 16600, [1000] * 4),
], ids=str)
def test_networks_stepped_at_rounded_up_widths(layers, B, T, widths):
    """bf16 networks off the matrix kernels' blocks are stepped at wider widths where that moves enough work to those
    kernels, and only there; fp32 ones, and networks with a layer without GLU, never."""
    assert _widths(layers, B, T) == widths
    assert _widths(layers, B, T, F32) == [l["cout"] for l in layers[:-1]]
    if len(layers) > 3:
        plain = [dict(l) for l in layers]
        plain[1].update(glu=0, cout=plain[1]["cout"] // 2)
        got = [P.w2l_train_step_layer_config(plain, B, T, P.W2L_BF16, i)[:2] for i in range(len(plain))]
        assert got == [(l["cin"], l["cout"]) for l in plain]
