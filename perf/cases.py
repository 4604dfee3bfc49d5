"""The work that a user of this library has it do, as cases that can be timed and compared.

Six kinds of pass, each through the public entry points only:

  step     one training step of a conv-GLU network with its criterion (w2l_train_step or
           w2l_train_step_asg): the library's main use.  The networks are the three of this
           repository's configurations (tiny fp32, about 10M and about 105M parameters) or others of
           the same build: a first convolution, a body of equal ones, an optional 1x1 layer, the
           classes.
  layer    one gated layer by its single entry points -- convolution and GLU forward, GLU backward,
           data gradient, weight and bias gradient -- as a program does that sequences its own network.
  ctc      the CTC criterion alone, from logits in one call, or from log-probabilities with the
           log-softmax and its backward as calls of their own.
  asg      the ASG criterion alone.
  logmel   features of a batch of utterances.
  sgd      the optimiser's update of every parameter tensor of a network.

Inputs are made on the GPU from the seed; buffers, weights and workspaces are what a training program
keeps from step to step.
"""
import math

import numpy as np
import torch

import paper_1812_07625_amd as P

DEV = "cuda:0"


# ------------------------------------------------------------------------------------ the cases
def _step(name, B, T, feat, first_k, stride, width, body, body_k, head, classes, crit, dtype):
    return dict(name=name, kind="step", B=B, T=T, feat=feat, first_k=first_k, stride=stride, width=width, body=body,
                body_k=body_k, head=head, classes=classes, crit=crit, dtype=dtype)


def listed():
    return [
        # a training step of the 105M-parameter model: 8 utterances of up to 15 s, bf16, CTC
        _step("step 105M bf16", 8, 1500, 80, 13, 2, 1536, 8, 11, 2048, 29, "ctc", "bf16"),
        # a training step of the 10M-parameter model: 16 utterances of up to 16 s, bf16, CTC
        _step("step 10M bf16", 16, 1600, 40, 13, 2, 512, 6, 11, 1024, 29, "ctc", "bf16"),
        # the same model on the four utterances a GPU that a large job gives each, with ASG; an odd frame count,
        # as batches padded to their longest utterance have
        _step("step 10M bf16 asg odd", 4, 1237, 40, 13, 2, 512, 6, 11, 1024, 28, "asg", "bf16"),
        # the same model in full precision
        _step("step 10M f32", 4, 800, 40, 13, 2, 512, 6, 11, 1024, 29, "ctc", "f32"),
        # the smallest network, where launches and latency count
        _step("step tiny f32", 2, 100, 40, 5, 1, 128, 1, 5, 0, 29, "ctc", "f32"),
        # one large layer, called pass by pass
        dict(name="layer bf16", kind="layer", B=16, T=800, cin=512, cout=1024, k=11, stride=1, dtype="bf16"),
        # a small layer of odd sizes: widths off the powers of two, an odd number of frames
        dict(name="layer bf16 ragged", kind="layer", B=3, T=731, cin=200, cout=440, k=13, stride=1, dtype="bf16"),
        # the criterion of a grapheme model at batch 32
        dict(name="ctc", kind="ctc", B=32, T=750, classes=29, max_target=200, logits=True),
        # the criterion of a word-piece model on a few short utterances, log-softmax in calls of its own
        dict(name="ctc logprobs small", kind="ctc", B=4, T=187, classes=200, max_target=45, logits=False),
        # the criterion with learned transitions at batch 32
        dict(name="asg", kind="asg", B=32, T=750, classes=28, max_target=200),
        # features of 8 utterances of 10 to 15 s
        dict(name="logmel", kind="logmel", B=8, samples=240240, mels=80, dtype="bf16"),
        # the optimiser over the 105M-parameter model, tensor by tensor
        dict(name="sgd 105M", kind="sgd", feat=80, first_k=13, stride=2, width=1536, body=8, body_k=11, head=2048, classes=29),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A channel count: mostly a multiple of 64, as most networks have, or of 16, or only of 4."""
    unit = rng.choice((64, 64, 16, 4))
    return max(unit, int(round(_log(rng, lo, hi) / unit)) * unit)


def draw(rng):
    kind = rng.choice(("step",) * 5 + ("layer",) * 4 + ("ctc",) * 2 + ("asg", "logmel", "sgd"))
    while True:
        if kind == "step":
            crit = rng.choice(("ctc", "ctc", "asg"))
            classes = rng.choice((29, 29, _log(rng, 20, 240))) if crit == "ctc" else rng.choice((28, _log(rng, 20, 64)))
            c = _step("", _log(rng, 1, 16), _log(rng, 100, 1600), rng.choice((40, 80)), rng.choice((5, 7, 11, 13)), rng.choice((1, 2, 2)),
                      _width(rng, 128, 1536), rng.randint(1, 8), rng.choice((3, 5, 7, 11, 13)), rng.choice((0, _width(rng, 256, 2048))),
                      classes, crit, rng.choice(("bf16", "bf16", "bf16", "f32")))
            del c["name"]
            most = 3.8e12 if c["dtype"] == "bf16" else 8e10
        elif kind == "layer":
            c = dict(kind=kind, B=_log(rng, 1, 16), T=_log(rng, 50, 1600), cin=_width(rng, 40, 1024), cout=_width(rng, 64, 2048),
                     k=rng.choice((1, 3, 5, 7, 9, 11, 13)), stride=rng.choice((1, 1, 1, 2)), dtype=rng.choice(("bf16", "bf16", "bf16", "f32")))
            most = 1e12 if c["dtype"] == "bf16" else 8e10
        elif kind in ("ctc", "asg"):
            T = _log(rng, 50, 1600)
            c = dict(kind=kind, B=_log(rng, 1, 32), T=T, max_target=max(1, int(T * rng.uniform(0.05, 0.3))))
            if kind == "ctc":
                c.update(classes=rng.choice((29, _log(rng, 20, 240))), logits=rng.choice((True, True, False)))
            else:
                c.update(classes=rng.choice((28, _log(rng, 20, 64))))
            return c
        elif kind == "logmel":
            return dict(kind=kind, B=_log(rng, 1, 32), samples=_log(rng, 8000, 320000), mels=rng.choice((40, 80)), dtype=rng.choice(("bf16", "f32")))
        else:
            return dict(kind=kind, feat=rng.choice((40, 80)), first_k=rng.choice((5, 7, 11, 13)), stride=2, width=_width(rng, 128, 1536), body=rng.randint(1, 8),
                        body_k=rng.choice((3, 5, 7, 11, 13)), head=rng.choice((0, _width(rng, 256, 2048))), classes=29)
        if work(c)["flops"] <= most:
            return c


# ------------------------------------------------------------------------------------ shapes
def _layers(c):
    layers = [dict(k=c["first_k"], stride=c["stride"], cin=c["feat"], cout=c["width"], glu=1)]
    layers += [dict(k=c["body_k"], stride=1, cin=c["width"] // 2, cout=c["width"], glu=1)] * c["body"]
    last = c["width"] // 2
    if c["head"]:
        layers.append(dict(k=1, stride=1, cin=last, cout=c["head"], glu=1))
        last = c["head"] // 2
    return layers + [dict(k=1, stride=1, cin=last, cout=c["classes"], glu=0)]


def _frames(T, stride):
    return (T + stride - 1) // stride


def work(case):
    """What a pass cannot do without: arithmetic of the convolutions (padded frames included: their outputs are part of
    the result), recursions and transforms; every input read and every output written once."""
    kind = case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if kind == "step":
        B, T = case["B"], case["T"]
        byts, flops, t = B * T * case["feat"] * es, 0.0, T
        for i, L in enumerate(_layers(case)):
            t = _frames(t, L["stride"])
            n = L["k"] * L["cin"] * L["cout"]
            flops += 2.0 * B * t * n * (3 if i else 2)
            byts += n * (es + 4) + 8 * L["cout"]
        return dict(bytes=byts + 4 * B * t * case["classes"], flops=flops)
    if kind == "layer":
        B, T, cin, cout = case["B"], case["T"], case["cin"], case["cout"]
        t = _frames(T, case["stride"])
        n = case["k"] * cin * cout
        # x, y, h, dh, dy, dx once each, w read, dw, bias and db
        return dict(bytes=es * (2 * B * T * cin + B * t * (2 * cout + 2 * (cout // 2)) + n) + 4 * n + 8 * cout, flops=6.0 * B * t * n)
    if kind == "ctc":
        n = case["B"] * case["T"]
        # logits in, gradient out (and log-probabilities and their gradient where those are calls of their own)
        return dict(bytes=4.0 * n * case["classes"] * (2 if case["logits"] else 4), flops=n * (12.0 * (2 * case["max_target"] + 1) + 6.0 * case["classes"]))
    if kind == "asg":
        n, C = case["B"] * case["T"], case["classes"]
        return dict(bytes=8.0 * n * C + 8.0 * C * C, flops=n * (6.0 * C * C + 12.0 * case["max_target"]))
    if kind == "logmel":
        frames = case["B"] * max(0, 1 + (case["samples"] - 400) // 160)
        return dict(bytes=4.0 * case["B"] * case["samples"] + es * frames * case["mels"], flops=frames * (400 + 2.5 * 512 * 9 + 3 * 257 + 2 * 512))
    n, b = sum(L["k"] * L["cin"] * L["cout"] for L in _layers(case)), sum(L["cout"] for L in _layers(case))
    return dict(bytes=22.0 * n + 20.0 * b, flops=6.0 * (n + b))


def tolerance(case):
    """About four times the largest relative error seen over these ranges against the same pass in 64 bits (from the
    same bf16 operands): a bf16 step rounds the activations and gradients of up to eleven layers (8.6e-3), a bf16 layer
    two or three of them in a row (2.5e-3); the ASG gradient is the difference of two occupancies (2e-5)."""
    kind, bf16 = case["kind"], case.get("dtype") == "bf16"
    if kind == "step":
        if bf16:
            return dict(rel=2.5e-2, max=0.25)
        return dict(rel=1e-4, max=3e-3) if case["crit"] == "asg" else dict(rel=2e-5, max=2e-4)
    if kind == "layer":
        return dict(rel=1e-2, max=0.05) if bf16 else dict(rel=5e-6, max=1e-4)
    if kind == "logmel":
        return dict(rel=7e-3, max=1.6e-2) if bf16 else dict(rel=5e-6, max=1e-3)
    if kind == "sgd":
        return dict(rel=5e-5, max=1e-2)  # the bf16 copy: a value next to a tie may round the other way
    return dict(rel=1e-4, max=3e-3) if kind == "asg" else dict(rel=1e-5, max=1e-4)


# ------------------------------------------------------------------------------------ what a program has in hand
class _Inputs:
    """Random tensors from one seed, drawn on the GPU; lengths and labels, which a data loader would bring, from the host."""

    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)
        self.host = np.random.default_rng(seed)

    def normal(self, shape, std=1.0, dtype=torch.float32):
        return (torch.randn(shape, generator=self.gen, device=DEV) * std).to(dtype)

    def uniform(self, shape, bound, dtype=torch.float32):
        return ((torch.rand(shape, generator=self.gen, device=DEV) * 2 - 1) * bound).to(dtype)

    def lengths(self, B, T):
        """Of a length-sorted corpus: between two thirds of the longest and the longest, which is there."""
        n = self.host.integers(max(1, 2 * T // 3), T + 1, size=B).astype(np.int32)
        n[self.host.integers(B)] = T
        return n

    def labels(self, lens, most, first, classes, frames):
        """Targets of `lens` labels from [first, classes), no two neighbours equal (so that every target fits its frames)."""
        tg = np.zeros((len(lens), most), np.int32)
        for b, n in enumerate(lens):
            step = self.host.integers(1, classes - first, size=n)  # from one label to the next: never 0
            tg[b, :n] = first + (self.host.integers(classes - first) + np.cumsum(step)) % (classes - first)
        assert all(n <= f for n, f in zip(lens, frames))
        return tg


def _dev(a):
    return torch.from_numpy(a).to(DEV)


def _td(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _code(case):
    return P.W2L_BF16 if case["dtype"] == "bf16" else P.W2L_F32


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, _Inputs(seed))


def run(state):
    return _RUN[state["kind"]](state)


def _prepare_step(c, r):
    layers, td = _layers(c), _td(c)
    B, T = c["B"], c["T"]
    n = r.lengths(B, T)
    x = r.normal((B, T, c["feat"]))
    x *= (torch.arange(T, device=DEV)[None, :] < _dev(n)[:, None])[:, :, None]
    w, b = [], []
    for L in layers:
        bound = 1.0 / math.sqrt(L["k"] * L["cin"])
        w.append(r.uniform((L["cout"], L["k"], L["cin"]), bound, td))
        b.append(r.uniform((L["cout"],), bound))
    frames = (n + c["stride"] - 1) // c["stride"]
    tl = np.maximum(1, n // 16).astype(np.int32)
    tl = np.minimum(tl, frames).astype(np.int32)
    asg = c["crit"] == "asg"
    tg = r.labels(tl, int(tl.max()), 0 if asg else 1, c["classes"], frames)
    query = P.w2l_train_step_asg_workspace_bytes if asg else P.w2l_train_step_workspace_bytes
    s = dict(kind="step", asg=asg, layers=layers, w=w, b=b, dw=[torch.zeros(t.shape, device=DEV) for t in w], db=[torch.zeros_like(t) for t in b],
             x=x.to(td), n=_dev(n), tg=_dev(tg), tl=_dev(tl), loss=torch.zeros(B, device=DEV),
             logits=torch.zeros((B, _frames(T, c["stride"]), c["classes"]), device=DEV), ws=P.workspace(query(layers, B, T, tg.shape[1], _code(c))))
    if asg:
        s.update(trans=r.normal((c["classes"], c["classes"]), 0.5), dtrans=torch.zeros((c["classes"], c["classes"]), device=DEV))
    return s


def _run_step(s):
    if s["asg"]:
        P.w2l_train_step_asg(s["layers"], s["w"], s["b"], s["dw"], s["db"], s["x"], s["n"], s["tg"], s["tl"], s["trans"], s["dtrans"], s["loss"],
                             s["logits"], 1.0, s["ws"])
        return s["loss"], s["logits"], s["dw"], s["db"], s["dtrans"]
    P.w2l_train_step(s["layers"], s["w"], s["b"], s["dw"], s["db"], s["x"], s["n"], s["tg"], s["tl"], s["loss"], s["logits"], 0, 1.0, s["ws"])
    return s["loss"], s["logits"], s["dw"], s["db"]


def _prepare_layer(c, r):
    B, T, cin, cout, k, stride, td = c["B"], c["T"], c["cin"], c["cout"], c["k"], c["stride"], _td(c)
    t = _frames(T, stride)
    shape, out = (B, T, cin, cout, k, stride, _code(c)), lambda *n, dt=td: torch.zeros(n, dtype=dt, device=DEV)
    need = max(P.w2l_conv1d_fwd_workspace_bytes(*shape), P.w2l_conv1d_bwd_data_workspace_bytes(*shape), P.w2l_conv1d_bwd_weight_workspace_bytes(*shape))
    return dict(kind="layer", stride=stride, x=r.normal((B, T, cin), 1.0, td), w=r.normal((cout, k, cin), 1.0 / math.sqrt(k * cin), td),
                bias=r.uniform((cout,), 0.1), dh=r.normal((B, t, cout // 2), 1.0, td), y=out(B, t, cout), h=out(B, t, cout // 2), dy=out(B, t, cout),
                dx=out(B, T, cin), dw=out(cout, k, cin, dt=torch.float32), db=out(cout, dt=torch.float32), ws=P.workspace(need))


def _run_layer(s):
    P.w2l_conv1d_fwd(s["x"], s["w"], s["bias"], s["y"], s["stride"], s["ws"])
    P.w2l_glu_fwd(s["y"], s["h"])
    P.w2l_glu_bwd(s["y"], s["dh"], s["dy"])
    P.w2l_conv1d_bwd_data(s["dy"], s["w"], s["dx"], s["stride"], s["ws"])
    P.w2l_conv1d_bwd_weight(s["x"], s["dy"], s["dw"], s["db"], s["stride"], False, s["ws"])
    return s["y"], s["h"], s["dy"], s["dx"], s["dw"], s["db"]


def _prepare_criterion(c, r, first):
    B, T, C, most = c["B"], c["T"], c["classes"], c["max_target"]
    n = r.host.integers(max(1, T - T // 5), T + 1, size=B).astype(np.int32)
    tl = r.host.integers(max(1, most // 4), most + 1, size=B).astype(np.int32)
    tl = np.minimum(tl, n).astype(np.int32)
    return dict(z=r.normal((B, T, C), math.sqrt(2.0)), n=_dev(n), tl=_dev(tl), tg=_dev(r.labels(tl, most, first, C, n)), loss=torch.zeros(B, device=DEV),
                grad=torch.zeros((B, T, C), device=DEV))


def _prepare_ctc(c, r):
    s = _prepare_criterion(c, r, 1)
    s.update(kind="ctc", logits=c["logits"], ws=P.workspace(P.w2l_ctc_workspace_bytes(c["B"], c["T"], c["classes"], c["max_target"])))
    if not c["logits"]:
        s.update(lp=torch.zeros_like(s["z"]), dz=torch.zeros_like(s["z"]))
    return s


def _run_ctc(s):
    if s["logits"]:
        P.w2l_ctc_fwd_bwd(s["z"], True, s["tg"], s["n"], s["tl"], s["loss"], s["grad"], 0, 1.0, s["ws"])
        return s["loss"], s["grad"]
    P.w2l_logsoftmax_fwd(s["z"], s["lp"])
    P.w2l_ctc_fwd_bwd(s["lp"], False, s["tg"], s["n"], s["tl"], s["loss"], s["grad"], 0, 1.0, s["ws"])
    P.w2l_logsoftmax_bwd(s["lp"], s["grad"], s["dz"])
    return s["loss"], s["lp"], s["grad"], s["dz"]


def _prepare_asg(c, r):
    s = _prepare_criterion(c, r, 0)
    C = c["classes"]
    s.update(kind="asg", trans=r.normal((C, C), 0.5), dtrans=torch.zeros((C, C), device=DEV),
             ws=P.workspace(P.w2l_asg_workspace_bytes(c["B"], c["T"], C, c["max_target"])))
    return s


def _run_asg(s):
    P.w2l_asg_fwd_bwd(s["z"], s["trans"], s["tg"], s["n"], s["tl"], s["loss"], s["grad"], s["dtrans"], 1.0, s["ws"])
    return s["loss"], s["grad"], s["dtrans"]


def _prepare_logmel(c, r):
    """Speech-shaped signals: a voice of twelve harmonics under a slow envelope, and noise 30 dB below it."""
    B, N = c["B"], c["samples"]
    t = torch.arange(N, device=DEV, dtype=torch.float32) / 16000.0
    f0, rate = r.uniform((B, 1), 80.0) + 170.0, r.uniform((B, 1), 1.0) + 2.0
    phase = 2 * math.pi * f0 * t + 3.0 * torch.sin(2 * math.pi * rate * t)
    wav = sum(torch.sin(h * phase) / h for h in range(1, 13)) * (0.15 * (1 + torch.sin(2 * math.pi * 0.7 * rate * t))) + r.normal((B, N), 0.016)
    n = r.lengths(B, N)
    wav *= torch.arange(N, device=DEV)[None, :] < _dev(n)[:, None]
    T = max(1, P.w2l_logmel_num_frames(N))
    return dict(kind="logmel", wav=wav, n=_dev(n), feat=torch.zeros((B, T, c["mels"]), dtype=_td(c), device=DEV),
                feat_len=torch.zeros(B, dtype=torch.int32, device=DEV))


def _run_logmel(s):
    P.w2l_logmel_fwd(s["wav"], s["n"], s["feat"], s["feat_len"])
    return s["feat"], s["feat_len"]


def _prepare_sgd(c, r):
    tensors = []
    for L in _layers(c):
        bound = 1.0 / math.sqrt(L["k"] * L["cin"])
        for shape, low in (((L["cout"], L["k"], L["cin"]), True), ((L["cout"],), False)):
            w = r.uniform(shape, bound)
            tensors.append((w, torch.zeros_like(w), r.normal(shape, 0.1), torch.zeros(shape, dtype=torch.bfloat16, device=DEV) if low else None))
    return dict(kind="sgd", tensors=tensors)


def _run_sgd(s):
    for w, v, g, low in s["tensors"]:
        P.w2l_sgd_momentum_step(w, v, g, low, 1e-4, 0.9)
    return [(w, v, low) for w, v, _, low in s["tensors"]]


_PREPARE = dict(step=_prepare_step, layer=_prepare_layer, ctc=_prepare_ctc, asg=_prepare_asg, logmel=_prepare_logmel, sgd=_prepare_sgd)
_RUN = dict(step=_run_step, layer=_run_layer, ctc=_run_ctc, asg=_run_asg, logmel=_run_logmel, sgd=_run_sgd)
