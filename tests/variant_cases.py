"""Problem sizes (classes C, padded target length Lmax) that between them make w2l_ctc_fwd_bwd and
w2l_asg_fwd_bwd launch every variant of their lattice kernels, and layers that make the train step
launch every form of its shared gradient kernel; which variant a size takes is asked of the library's
own host-side query (w2l_ctc_launch_config / w2l_asg_launch_config / w2l_train_step_launch_config),
the function the entry points dispatch through."""

# CTC: (pairs per lane, frames per block) follows Lmax + 1 pairs: <= 208 -> (1,16), <= 220 -> (1,12),
# <= 416 -> (2,16), <= 440 -> (2,12), <= 832 -> (4,16), <= 880 -> (4,12), more -> (4,16) on more wavefronts;
# the score-table values per staging thread follow frames per block * the table's rows -- the classes, or one more than the
# longest target if that is fewer -- against the staging threads (256 beside up to four wavefronts, else all).
CTC_LMAX = [200, 215, 400, 436, 800, 870, 1100]
CTC_CLASSES = [29, 50, 100, 200]
CTC_CASES = [(c, l) for l in CTC_LMAX for c in CTC_CLASSES] + [(29, 60), (600, 20)]

# ASG: positions per lane / frames per block follow Lmax the same way (without the +1); 32 or 64 class
# lanes follow C; emission values staged per thread follow frames per block * C against the workgroup size.
ASG_CASES = [(c, l) for l in [90, 190, 205, 300, 380, 412, 500, 760, 828, 1100] for c in [8, 28, 40, 64]] + [(28, 250)]


# Gradients of a gated layer inside a bf16 train step, as w2l_train_step_launch_config names them: (B, T, k, cin, cout) of
# the middle layer of bwd_network(), one per data-gradient form (1 .. 6) and weight tile (0 .. 3) of the shared launch,
# with few multiplications, so that the fp64 oracle takes a second or two.
BWD_CASES = [
    (12, 34, 3, 1088, 256), (16, 1161, 3, 64, 256), (12, 1340, 3, 64, 384), (8, 372, 5, 800, 256),    # form 1: tiles 0 .. 3
    (4, 33, 3, 64, 64), (16, 132, 3, 1152, 192), (6, 568, 3, 816, 64), (16, 190, 3, 1464, 256),       # form 2
    (2, 65, 1, 72, 256), (3, 345, 1, 64, 1792), (16, 82, 3, 64, 896), (3, 44, 13, 1280, 128),         # form 3
    (8, 1422, 13, 64, 192), (8, 695, 11, 144, 256), (8, 1051, 11, 136, 320), (2, 66, 9, 1648, 2048),  # form 4
    (4, 33, 1, 64, 64), (1, 1299, 1, 1456, 192), (4, 449, 1, 1208, 192), (3, 1206, 1, 752, 1024),     # form 5
    (16, 1109, 1, 144, 64), (16, 339, 1, 704, 192), (16, 233, 1, 1328, 64), (16, 292, 1, 1024, 1024), # form 6
]


# fp32 layers (B, T, Cin, Cout, k) whose passes between them take every kernel for haloed operands (rows of its tile,
# products from bf16 terms or not, reduction split or not) in every pass, as w2l_conv1d_launch_tile names them; utterances
# of a few frames, of less than a panel of 32, and of several; few multiplications for the fp64 oracle.
F32_CASES = [
    (35, 2, 1088, 1600, 5), (22, 158, 352, 96, 7), (28, 76, 96, 1696, 3), (17, 31, 96, 1824, 7), (20, 1273, 92, 96, 3),
    (26, 24, 1280, 36, 13), (15, 3, 1216, 216, 11), (39, 6, 1120, 96, 9),   # weight gradients over short utterances
    (2, 1321, 32, 3104, 1), (3, 701, 512, 1088, 1), (2, 450, 1024, 96, 9), (1, 130, 1100, 1600, 3),
]


def f32_variants(P, B, T, cin, cout, k):
    """(rows, terms, split) of the three passes, None where the operands are not haloed."""
    out = []
    for p in (0, 1, 2):
        form, splits = P.w2l_conv1d_launch_config(p, B, T, cin, cout, k, 1, P.W2L_F32)
        out.append(P.w2l_conv1d_launch_tile(p, B, T, cin, cout, k, 1, P.W2L_F32) + (splits > 1,) if form == 3 else None)
    return out


def bwd_network(k, cin, cout):
    return [dict(k=3, stride=1, cin=16, cout=2 * cin, glu=1), dict(k=k, stride=1, cin=cin, cout=cout, glu=1),
            dict(k=1, stride=1, cin=cout // 2, cout=29, glu=0)]


def bwd_variant(P, B, T, k, cin, cout):
    data, _, tile, _ = P.w2l_train_step_launch_config(bwd_network(k, cin, cout), B, T, P.W2L_BF16, 1)
    return (data, tile)


def ctc_variant(P, C, Lmax):
    ppt, nq, blk, _ = P.w2l_ctc_launch_config(C, Lmax)
    return (ppt, nq, blk)


def asg_variant(P, C, Lmax):
    ppt, cmax, maxt, blk, nq, _ = P.w2l_asg_launch_config(C, Lmax)
    return (ppt, cmax, maxt, blk, nq)
