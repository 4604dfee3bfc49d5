"""Train steps whose middle layer takes each form of the shared gradient launch (six data-gradient forms, four weight
tiles), and one whose layers keep launches of their own, against the fp64 oracle; bounds of a whole bf16 step as in
test_gpu_parity.py.  Frame counts are mostly no multiple of any tile and targets short, so that the oracle stays cheap."""
import pytest

import workloads as W
from test_gpu_parity import check_train_step, oracle_train_step
from variant_cases import BWD_CASES, bwd_network, bwd_variant
from workloads.device import run_train_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_1812_07625_amd as P
    return P


@pytest.mark.parametrize("case", BWD_CASES, ids=lambda c: "x".join(map(str, c)))
def test_shared_gradient_launch(P, case):
    B, T, k, cin, cout = case
    i = BWD_CASES.index(case)
    assert bwd_variant(P, *case) == (1 + i // 4, i % 4)
    cfg = W.small_model(60 + i, B, max(20, T - T // 4), T, 16, bwd_network(k, cin, cout), True, 2, 8)
    check_train_step(run_train_step(P, cfg), oracle_train_step(cfg), "bf16")


def test_gradients_in_launches_of_their_own(P):
    """The second body layer's tiles would leave CUs waiting in a shared launch, so every layer keeps two streams: the
    first body layer's data gradient by two workgroups a tile and the third one's with the GLU backward in its epilogue."""
    widths = [(3, 320, 256), (7, 128, 128), (5, 64, 128)]
    layers = [dict(k=3, stride=1, cin=16, cout=640, glu=1)] + [dict(k=k, stride=1, cin=a, cout=b, glu=1) for k, a, b in widths]
    layers += [dict(k=1, stride=1, cin=64, cout=29, glu=0)]
    B, T = 16, 98
    assert [bwd_variant(P, B, T, *w)[0] for w in widths] == [1, 0, 2]      # each by itself
    assert all(P.w2l_train_step_launch_config(layers, B, T, P.W2L_BF16, i)[0] == 0 for i in range(5))
    cfg = W.small_model(90, B, 70, T, 16, layers, True, 2, 8)
    check_train_step(run_train_step(P, cfg), oracle_train_step(cfg), "bf16")


def test_bias_gradients_not_wanted(P):
    """A layer whose bias gradient is not wanted (NULL) keeps launches of its own between layers that share theirs; the
    other gradients are the oracle's, and what is not wanted stays as it was."""
    import numpy as np
    layers = [dict(k=5, stride=2, cin=40, cout=256, glu=1)] + [dict(k=5, stride=1, cin=128, cout=256, glu=1)] * 4
    layers += [dict(k=1, stride=1, cin=128, cout=29, glu=0)]
    assert all(P.w2l_train_step_launch_config(layers, 4, 301, P.W2L_BF16, i)[0] > 0 for i in range(1, 5))

    class Without:  # the binding, with some bias gradients left out
        def __init__(self, skip): self.skip = skip
        def __getattr__(self, name): return getattr(P, name)
        def w2l_train_step(self, layers, w, b, dw, db, *rest):
            return P.w2l_train_step(layers, w, b, dw, [None if i in self.skip else t for i, t in enumerate(db)], *rest)

    cfg = W.small_model(91, 4, 220, 301, 40, layers, True, 4, 20)
    ref = oracle_train_step(cfg)
    for skip in ((2,), (1, 3), (0, 4, 5), tuple(range(6))):
        got = run_train_step(Without(skip), cfg)
        for i in skip:
            assert np.isnan(got["db"][i]).all()
            got["db"][i] = ref["db"][i]
        check_train_step(got, ref, "bf16")


@pytest.mark.parametrize("classes, H, dtype", [
    (29, 8, "bf16"), (30, 72, "bf16"), (64, 128, "bf16"), (63, 136, "bf16"), (29, 264, "bf16"), (33, 520, "bf16"),  # 1 .. 16 groups of 8 channels, 17 ..
    (65, 64, "bf16"), (29, 44, "bf16"),                                        # matrix kernels: a class or channels too many
    (29, 4, "f32"), (29, 60, "f32"), (64, 64, "f32"), (30, 68, "f32"), (31, 132, "f32"), (65, 64, "f32"), (29, 42, "f32"),
])
@pytest.mark.parametrize("misaligned", [False, True])
def test_class_layer_backward(P, classes, H, dtype, misaligned):
    """The gradient through the classes' layer into the layer below: one launch up to 64 classes of whole 16-byte groups
    of channels (fp32 of so few values: up to 48), over blocks of 32 and 64 frames that end in the middle, also where the
    weights lie off a 16-byte address (bf16: over fewer frames than the matrix kernels take, whose forward pass reads them in
    16-byte pieces).  Bounds: a whole step's."""
    layers = [dict(k=3, stride=1, cin=16, cout=2 * H, glu=1), dict(k=1, stride=1, cin=H, cout=classes, glu=0)]
    T = 42 if misaligned and dtype == "bf16" else 61
    cfg = W.small_model(100 + H, 3, T - 11, T, 16, layers, dtype == "bf16", 2, 8)

    class Shifted:  # the binding, with the classes' weights one element behind where an allocation starts
        def __getattr__(self, name): return getattr(P, name)
        def w2l_train_step(self, layers, w, *rest):
            import torch
            room = torch.empty(w[-1].numel() + 1, dtype=w[-1].dtype, device=w[-1].device)
            room[1:] = w[-1].reshape(-1)
            return P.w2l_train_step(layers, w[:-1] + [room[1:].view(w[-1].shape)], *rest)

    check_train_step(run_train_step(Shifted() if misaligned else P, cfg), oracle_train_step(cfg), dtype)


@pytest.mark.parametrize("classes, H, frames", [(64, 132, 2650), (49, 128, 2750), (64, 132, 2400), (64, 124, 2750)])
def test_many_classes_fp32(P, classes, H, frames):
    """fp32 networks of 49 .. 64 classes on either side of 2^20 values of dh and of 128 channels: one launch, or launches of
    their own, through the class layer.  Bounds: a whole step's."""
    layers = [dict(k=1, stride=1, cin=16, cout=2 * H, glu=1), dict(k=1, stride=1, cin=H, cout=classes, glu=0)]
    cfg = W.small_model(110 + H, 3, frames - 11, frames, 16, layers, False, 2, 8)
    check_train_step(run_train_step(P, cfg), oracle_train_step(cfg), "f32")


@pytest.mark.parametrize("widths, k, stride, feat, frames", [
    ((210, 250), 5, 2, 40, 260),              # halves of 105 and 125: no multiple of anything
    ((496, 240, 332), 3, 1, 80, 131),         # whole chunks, no whole blocks; a half of 2 mod 4 (gradients copied one by one)
    ((256, 128, 192, 264), 3, 1, 12, 140),    # one layer off the blocks; features of a multiple of 4
    ((72,) * 30, 3, 1, 40, 150),              # more layers than a copying launch takes
])
def test_widths_off_the_matrix_blocks(P, widths, k, stride, feat, frames):
    """Networks whose layers are stepped with zeros in new channels give the oracle's outputs, loss and gradients; bounds of a
    whole bf16 step.  Twice, the second time in a workspace full of other bytes and without some bias gradients."""
    cin = [feat] + [w // 2 for w in widths[:-1]]
    layers = [dict(k=k, stride=stride if i == 0 else 1, cin=c, cout=w, glu=1) for i, (c, w) in enumerate(zip(cin, widths))]
    layers += [dict(k=1, stride=1, cin=widths[-1] // 2, cout=29, glu=0)]
    cfg = W.small_model(130 + k, 3, frames - 30, frames, feat, layers, True, 5, 20)
    wide = [P.w2l_train_step_layer_config(layers, 3, frames, P.W2L_BF16, i)[1] for i in range(len(layers))]
    assert any(w % 64 for w in widths) and wide[-1] == 29
    assert all(b % 64 == 0 and (b > a if a % 64 else b == a) for a, b in zip(widths, wide))
    plain = [dict(l) for l in layers]
    ref = oracle_train_step(cfg)
    check_train_step(run_train_step(P, cfg), ref, "bf16")

    class Without:  # the binding without the bias gradients of two layers, into a workspace full of NaN
        def __getattr__(self, name): return getattr(P, name)
        def w2l_train_step(self, layers, w, b, dw, db, *rest):
            rest[-1].fill_(255)
            return P.w2l_train_step(layers, w, b, dw, [None if i in (0, 1) else t for i, t in enumerate(db)], *rest)

    got = run_train_step(Without(), cfg)
    for i in (0, 1):
        got["db"][i] = ref["db"][i]
    check_train_step(got, ref, "bf16")
    assert layers == plain


def test_widths_off_the_matrix_blocks_many_classes(P):
    """The same with more classes than the class layer's own launch takes (their gradient stays on the fp32 instruction)."""
    layers = [dict(k=3, stride=1, cin=40, cout=250, glu=1), dict(k=3, stride=1, cin=125, cout=300, glu=1), dict(k=1, stride=1, cin=150, cout=100, glu=0)]
    assert [P.w2l_train_step_layer_config(layers, 4, 200, P.W2L_BF16, i)[1] for i in range(3)] == [256, 320, 100]
    cfg = W.small_model(180, 4, 160, 200, 40, layers, True, 5, 20)
    check_train_step(run_train_step(P, cfg), oracle_train_step(cfg), "bf16")


def _asg_step(P, layers, cfg, trans, targets, dtype):
    import torch
    from workloads.device import empty, to_dev, to_host
    code = P.W2L_BF16 if dtype == "bf16" else P.W2L_F32
    B, T, Lmax = cfg["B"], cfg["T"], targets.shape[1]
    dw, db = [empty(a.shape) for a in cfg["weights"]], [empty(a.shape) for a in cfg["biases"]]
    dtrans, loss, logits = empty(trans.shape), empty((B,)), empty((B, -(-T // layers[0]["stride"]), layers[-1]["cout"]))
    P.w2l_train_step_asg(layers, [to_dev(a, dtype) for a in cfg["weights"]], [to_dev(a) for a in cfg["biases"]], dw, db, to_dev(cfg["x"], dtype),
                         to_dev(cfg["in_len"]), to_dev(targets), to_dev(cfg["tgt_len"]), to_dev(trans), dtrans, loss, logits, 1.0,
                         P.workspace(P.w2l_train_step_asg_workspace_bytes(layers, B, T, Lmax, code)))
    torch.cuda.synchronize()
    return dict(loss=to_host(loss), logits=to_host(logits), dw=[to_host(t) for t in dw], db=[to_host(t) for t in db]), to_host(dtrans)


def test_widths_off_the_matrix_blocks_asg(P):
    """The same with the ASG criterion, at a stride, whose frame counts its kernels divide themselves."""
    import numpy as np
    import oracle
    from gpu_util import rel_l2
    layers = [dict(k=5, stride=2, cin=40, cout=250, glu=1), dict(k=5, stride=1, cin=125, cout=300, glu=1), dict(k=1, stride=1, cin=150, cout=28, glu=0)]
    assert [P.w2l_train_step_layer_config(layers, 4, 301, P.W2L_BF16, i)[1] for i in range(3)] == [256, 320, 28]
    cfg = W.small_model(181, 4, 200, 301, 40, layers, True, 5, 20)
    trans = (np.random.default_rng(182).standard_normal((28, 28)) * 0.5).astype(np.float32)
    targets = (cfg["targets"] % 28).astype(np.int32)
    got, dtrans = _asg_step(P, layers, cfg, trans, targets, "bf16")
    f64 = lambda a: np.asarray(a, dtype=np.float64)
    ref = oracle.train_step(layers, [f64(w) for w in cfg["weights"]], [f64(b) for b in cfg["biases"]], f64(cfg["x"]),
                            cfg["in_len"], targets, cfg["tgt_len"], 1.0, trans=f64(trans))
    check_train_step(got, ref, "bf16")
    assert rel_l2(dtrans, ref["dtrans"]) <= 2e-2


@pytest.mark.parametrize("what", ["weights", "gradients", "logits"])
def test_widths_off_the_matrix_blocks_off_16_bytes(P, what):
    """Tensors that a network stepped at rounded-up widths copies element by element where they lie off a 16-byte address (the
    layers' weights and their gradients, at widths that are whole groups of four), and the logits, which are then written in the
    workspace and copied: the bits are those of aligned tensors."""
    import numpy as np
    import torch
    layers = [dict(k=5, stride=1, cin=40, cout=232, glu=1), dict(k=5, stride=1, cin=116, cout=232, glu=1), dict(k=1, stride=1, cin=116, cout=29, glu=0)]
    assert [P.w2l_train_step_layer_config(layers, 3, 260, P.W2L_BF16, i)[1] for i in range(3)] == [256, 256, 29]
    cfg = W.small_model(183, 3, 200, 260, 40, layers, True, 5, 20)

    def off(t, copy):  # a tensor of t's shape one element behind where an allocation starts
        room = torch.full((t.numel() + 1,), float("nan"), dtype=t.dtype, device=t.device)[1:].view(t.shape)
        return room.copy_(t) if copy else room

    class Off:
        def __getattr__(self, name): return getattr(P, name)
        def w2l_train_step(self, layers, w, b, dw, db, x, n, tg, tl, loss, logits, *rest):
            w2 = [off(t, True) for t in w] if what == "weights" else w
            dw2 = [off(t, False) for t in dw] if what == "gradients" else dw
            z2 = off(logits, False) if what == "logits" else logits
            P.w2l_train_step(layers, w2, b, dw2, db, x, n, tg, tl, loss, z2, *rest)
            for a, c in zip(dw + [logits], dw2 + [z2]):
                a.copy_(c)

    got, ref = run_train_step(Off(), cfg), run_train_step(P, cfg)
    for a, b in zip([got["loss"], got["logits"]] + got["dw"] + got["db"], [ref["loss"], ref["logits"]] + ref["dw"] + ref["db"]):
        assert np.isfinite(b).all()
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_logits_where_the_caller_wants_them(P, dtype, aligned):
    """Written in place, or (off a 16-byte address) copied: the oracle's, and nothing behind them."""
    import torch
    layers = [dict(k=3, stride=2, cin=40, cout=128, glu=1), dict(k=1, stride=1, cin=64, cout=29, glu=0)]
    cfg = W.small_model(184, 3, 100, 131, 40, layers, dtype == "bf16", 3, 10)
    room = torch.full((3 * 66 * 29 + 64,), -7.0, device="cuda:0")[0 if aligned else 1:]

    class There:
        def __getattr__(self, name): return getattr(P, name)
        def w2l_train_step(self, layers, w, b, dw, db, x, n, tg, tl, loss, logits, *rest):
            z = room[:logits.numel()].view(logits.shape)
            P.w2l_train_step(layers, w, b, dw, db, x, n, tg, tl, loss, z, *rest)
            logits.copy_(z)

    check_train_step(run_train_step(There(), cfg), oracle_train_step(cfg), dtype)
    assert (room[3 * 66 * 29:] == -7.0).all()


def _helpers(P, layers, B, T, dtype):
    """which weight gradients run on the helper stream, and which layers share a launch for both"""
    code = P.W2L_BF16 if dtype == "bf16" else P.W2L_F32
    n = range(len(layers))
    return ([P.w2l_train_step_layer_config(layers, B, T, code, i)[2] for i in n], [int(P.w2l_train_step_launch_config(layers, B, T, code, i)[0] > 0) for i in n])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_two_streams_layers_without_glu(P, dtype):
    """Layers without a GLU, whose dh is their dy, beside weight gradients on the helper stream: the data gradients wait before
    they overwrite a buffer that such a weight gradient still reads."""
    import numpy as np
    layers = [dict(k=5, stride=2, cin=40, cout=64, glu=0), dict(k=3, stride=1, cin=64, cout=96, glu=1),
              dict(k=3, stride=1, cin=48, cout=256, glu=0), dict(k=11, stride=1, cin=256, cout=256, glu=0),
              dict(k=5, stride=1, cin=256, cout=256, glu=0), dict(k=3, stride=1, cin=256, cout=64, glu=1),
              dict(k=1, stride=1, cin=32, cout=29, glu=0)]
    assert _helpers(P, layers, 4, 233, dtype)[0] == [0, 1, 1, 1, 1, 1, 0]
    cfg = W.small_model(185, 4, 150, 233, 40, layers, dtype == "bf16", 5, 30)
    ref = oracle_train_step(cfg)
    a, b = run_train_step(P, cfg), run_train_step(P, cfg)
    check_train_step(a, ref, dtype)
    for u, v in zip(a["dw"] + a["db"], b["dw"] + b["db"]):
        assert np.array_equal(u, v)


def test_two_streams_beside_shared_launches(P):
    """A strided layer's long weight gradient on the helper stream between layers that share a launch for both gradients, and
    those on the helper stream too where their bias gradients are not wanted."""
    import numpy as np
    body = dict(k=5, stride=1, cin=128, cout=256, glu=1)
    layers = [dict(k=5, stride=2, cin=40, cout=256, glu=1), body, dict(k=9, stride=2, cin=128, cout=512, glu=1),
              dict(k=5, stride=1, cin=256, cout=256, glu=1), body, dict(k=1, stride=1, cin=128, cout=29, glu=0)]
    assert _helpers(P, layers, 4, 301, "bf16") == ([0, 0, 1, 0, 0, 0], [0, 1, 0, 1, 1, 0])
    cfg = W.small_model(186, 4, 220, 301, 40, layers, True, 4, 20)
    ref = oracle_train_step(cfg)

    class Without:
        def __init__(self, skip): self.skip = skip
        def __getattr__(self, name): return getattr(P, name)
        def w2l_train_step(self, layers, w, b, dw, db, *rest):
            return P.w2l_train_step(layers, w, b, dw, [None if i in self.skip else t for i, t in enumerate(db)], *rest)

    for skip in ((), (1,), (3, 4), (1, 2, 3, 4), tuple(range(6))):
        got = run_train_step(Without(skip), cfg)
        for i in skip:
            assert np.isnan(got["db"][i]).all()
            got["db"][i] = ref["db"][i]
        check_train_step(got, ref, "bf16")


def test_two_streams_fp32(P):
    """fp32 weight gradients on the helper stream, split ones and short ones among them, beside the caller's."""
    layers = [dict(k=5, stride=2, cin=40, cout=256, glu=1), dict(k=9, stride=1, cin=128, cout=512, glu=1), dict(k=3, stride=1, cin=256, cout=140, glu=1),
              dict(k=7, stride=1, cin=70, cout=256, glu=1), dict(k=1, stride=1, cin=128, cout=40, glu=0)]
    assert _helpers(P, layers, 4, 301, "f32") == ([0, 1, 1, 1, 1], [0] * 5)
    cfg = W.small_model(187, 4, 220, 301, 40, layers, False, 4, 20)
    check_train_step(run_train_step(P, cfg), oracle_train_step(cfg), "f32")


@pytest.mark.parametrize("width, classes", [(250, 100), (250, 29), (256, 29)])
def test_class_gradient_is_not_rounded(P, width, classes):
    """Where the class layer's weights are the same for all classes, the criterion's gradient, whose classes add up to zero in
    every frame, leaves nothing for the layers below: what arrives there is the error of that sum.  In fp32 that is about 1e-6
    of what unequal weights pass on; a gradient rounded to bf16 (2^-9 a class) leaves about 1e-3.  (250: a width that the
    step rounds up; 256 with more than 64 classes does round it.)"""
    import numpy as np
    layers = [dict(k=3, stride=1, cin=40, cout=width, glu=1), dict(k=3, stride=1, cin=width // 2, cout=width, glu=1),
              dict(k=1, stride=1, cin=width // 2, cout=classes, glu=0)]
    cfg = W.small_model(140, 4, 160, 200, 40, layers, True, 5, 20)
    unequal = run_train_step(P, cfg)
    cfg["weights"][-1] = np.broadcast_to(cfg["weights"][-1][:1], cfg["weights"][-1].shape).copy()
    equal = run_train_step(P, cfg)
    for i in range(2):
        assert np.linalg.norm(equal["dw"][i]) <= 5e-5 * np.linalg.norm(unequal["dw"][i]), i


@pytest.mark.parametrize("widths, k, frames", [
    ((250,) * 3, 3, 200),       # planes of sums finished by the GLU passes
    ((250,) * 3, 1, 200),       # GLU passes of their own
    ((750, 760, 700), 3, 3000), # GLU and GLU backward in the epilogues of the tiles
])
def test_infinities_stay_where_they_are(P, widths, k, frames):
    """A network of positive weights, stepped at rounded-up widths, carries an infinite feature to the logits of the frames
    around it as infinities of its real channels (0 times infinity in a new channel would make them NaN); the others are
    finite and right, within the rounding of a bf16 step's activations."""
    import numpy as np
    import oracle
    cin = [40] + [w // 2 for w in widths[:-1]]
    layers = [dict(k=k, stride=1, cin=c, cout=w, glu=1) for c, w in zip(cin, widths)] + [dict(k=1, stride=1, cin=widths[-1] // 2, cout=29, glu=0)]
    B = 4
    cfg = W.small_model(150 + k, B, frames, frames, 40, layers, True, 3, 10)
    cfg["x"] = np.abs(cfg["x"])
    cfg["weights"] = [np.abs(w) for w in cfg["weights"]]
    cfg["x"][1, frames // 2, 7] = np.inf
    h = cfg["x"][1].astype(np.float64)[None, frames // 2 - 20:frames // 2 + 20]   # (the frames that it can reach, and some more)
    for L, w, b in zip(layers, cfg["weights"], cfg["biases"]):
        h = oracle.conv1d_fwd(h, w.astype(np.float64), b.astype(np.float64), L["stride"])
        if L["glu"]:
            h = oracle.glu_fwd(h)
    got = run_train_step(P, cfg)["logits"]
    assert np.isfinite(np.delete(got, 1, 0)).all()
    reach = slice(frames // 2 - 10, frames // 2 + 10)
    got, ref = got[1, reach], h[0, 10:30]
    assert np.isposinf(ref).any() and np.isfinite(ref).any()
    np.testing.assert_array_equal(np.isposinf(got), np.isposinf(ref))
    assert not np.isnan(got).any()
    fin = np.isfinite(ref)
    assert np.linalg.norm(got[fin] - ref[fin]) <= 2e-2 * np.linalg.norm(ref[fin])


@pytest.mark.parametrize("widths, k, frames", [((250,) * 3, 3, 200), ((250,) * 3, 1, 200), ((750, 760, 700), 3, 3000)])
def test_infinite_gradients_stay_where_they_are(P, widths, k, frames):
    """The same on the way back: with positive weights and features and a class that no target has, whose gradient times its
    weights overflows in some frames, every term of the layers' gradients is positive, so they overflow but are no NaN."""
    import numpy as np
    cin = [40] + [w // 2 for w in widths[:-1]]
    layers = [dict(k=k, stride=1, cin=c, cout=w, glu=1) for c, w in zip(cin, widths)] + [dict(k=1, stride=1, cin=widths[-1] // 2, cout=29, glu=0)]
    cfg = W.small_model(160 + k, 4, frames, frames, 40, layers, True, 3, 10, zero_bias=True)
    assert cfg["targets"].max() <= 28
    cfg["targets"] = np.where(cfg["targets"] == 28, 1, cfg["targets"]).astype(np.int32)
    x = 0.5 + 0.5 * np.abs(cfg["x"]) / np.abs(cfg["x"]).max()
    mid = slice(frames // 2 - 5, frames // 2 + 5)
    x[:, mid] *= 4                                                   # gates stay far from where their slope is 0
    cfg["x"] = W.round_to_bf16(x.astype(np.float32))
    mean = lambda w: np.abs(w) / np.abs(w).sum((1, 2), keepdims=True)  # a layer's values are means of the last one's
    w = [mean(w) for w in cfg["weights"][:-1]]
    w[-1] = 0.002 * w[-1]
    last = np.zeros(cfg["weights"][-1].shape)
    last[28] = 10.0 / (0.0027 * last.shape[2])
    cfg["weights"] = [W.round_to_bf16(a.astype(np.float32)) for a in w + [last]]
    cfg["biases"][-1][28] = -5
    got = run_train_step(P, cfg, grad_scale=3e38)
    assert np.isfinite(got["logits"]).all() and np.isfinite(got["loss"]).all()
    for i in range(3):
        assert np.isposinf(got["dw"][i]).any(), i
        assert not np.isnan(got["dw"][i]).any() and not np.isnan(got["db"][i]).any(), i


@pytest.mark.parametrize("cout, k, stride", [(100, 5, 2), (150, 13, 2), (84, 1, 2), (100, 9, 4), (128, 5, 2)])
def test_strided_first_layer_of_any_width(P, cout, k, stride):
    """The first layer's weight gradient, whose stride folds into the channels only where the matrix kernels take the folded
    layer: right, and nothing written behind it.  (Too little work to be stepped at rounded-up widths.)"""
    import torch
    layers = [dict(k=k, stride=stride, cin=40, cout=cout, glu=1), dict(k=1, stride=1, cin=cout // 2, cout=29, glu=0)]
    cfg = W.small_model(170 + cout + k, 3, 150, 200, 40, layers, True, 3, 10)
    room = torch.full((cfg["weights"][0].size + 65536,), -7.0, device="cuda:0")

    class Guarded:  # the binding, with room of known contents behind the first layer's weight gradient
        def __getattr__(self, name): return getattr(P, name)
        def w2l_train_step(self, layers, w, b, dw, db, *rest):
            inner = room[:dw[0].numel()].view(dw[0].shape)
            P.w2l_train_step(layers, w, b, [inner] + dw[1:], db, *rest)
            dw[0].copy_(inner)

    check_train_step(run_train_step(Guarded(), cfg), oracle_train_step(cfg), "bf16")
    assert (room[cfg["weights"][0].size:] == -7.0).all()


@pytest.mark.parametrize("net, dtype", [("shared", "bf16"), ("two streams", "bf16"), ("shared", "f32"), ("rounded up", "bf16")])
def test_captured_step_replays_the_eager_one(P, net, dtype):
    """A train step recorded into a HIP graph leaves the eager step's bits at every replay, with eager work of the same
    kernels on other data, and synchronisations, in between."""
    import torch
    from workloads.device import empty, to_dev
    widths = dict([("shared", [(5, 128, 256)] * 3), ("two streams", [(3, 320, 256), (7, 128, 128), (5, 64, 128)]), ("rounded up", [(5, 125, 250)] * 3)])[net]
    layers = [dict(k=5, stride=1, cin=40, cout=2 * widths[0][1], glu=1)] + [dict(k=k, stride=1, cin=a, cout=b, glu=1) for k, a, b in widths]
    layers += [dict(k=1, stride=1, cin=widths[-1][2] // 2, cout=29, glu=0)]
    assert (P.w2l_train_step_layer_config(layers, 16, 98, P.W2L_BF16, 1)[1] != widths[0][2]) == (net == "rounded up")

    def state(seed):
        cfg = W.small_model(seed, 16, 70, 98, 40, layers, dtype == "bf16", 2, 8)
        code = P.W2L_BF16 if dtype == "bf16" else P.W2L_F32
        s = dict(w=[to_dev(a, dtype) for a in cfg["weights"]], b=[to_dev(a) for a in cfg["biases"]], dw=[empty(a.shape) for a in cfg["weights"]],
                 db=[empty(a.shape) for a in cfg["biases"]], loss=empty((16,)), logits=empty((16, 98, 29)))
        args = [to_dev(cfg["x"], dtype), to_dev(cfg["in_len"]), to_dev(cfg["targets"]), to_dev(cfg["tgt_len"])]
        s["ws"] = P.workspace(P.w2l_train_step_workspace_bytes(layers, 16, 98, cfg["targets"].shape[1], code))
        s["run"] = lambda: P.w2l_train_step(layers, s["w"], s["b"], s["dw"], s["db"], *args, s["loss"], s["logits"], cfg["blank"], 1.0, s["ws"])
        s["out"] = [s["loss"], s["logits"]] + s["dw"] + s["db"]
        return s

    a, other = state(95), state(96)
    other["run"]()
    a["run"]()
    torch.cuda.synchronize()
    ref = [t.clone() for t in a["out"]]
    assert all(torch.isfinite(t).all() for t in ref)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        a["run"]()
    for _ in range(4):
        for t in a["out"]:
            t.fill_(float("nan"))
        a["ws"].fill_(255)
        other["run"]()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(t, r) for t, r in zip(a["out"], ref))
