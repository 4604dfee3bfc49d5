"""Problem sizes (classes C, padded target length Lmax) that between them make w2l_ctc_fwd_bwd and
w2l_asg_fwd_bwd launch every variant of their lattice kernels, and layers that make the train step
launch every form of its shared gradient kernel; which variant a size takes is asked of the library's
own host-side query (w2l_ctc_launch_config / w2l_asg_launch_config / w2l_train_step_launch_config),
the function the entry points dispatch through."""

# CTC: (pairs per lane, frames per block) follows Lmax + 1 pairs: <= 208 -> (1,16), <= 220 -> (1,12),
# <= 416 -> (2,16), <= 440 -> (2,12), <= 832 -> (4,16), <= 880 -> (4,12), more -> (4,16) on more wavefronts;
# the score-table values per thread follow frames per block * C against the workgroup size.
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
