"""The work that is measured: calls a user of the library makes through its binding.

Kinds of case (the "kind" of a case's dict):

- ``conv``: one conv2d layer.  passes = "step" is a training step of the layer,
  forward (bias and relu fused), backward_filter (which hands the relu-masked
  gradient over) and backward_data; "fwd" is the forward alone (scoring);
  "first" is forward and backward_filter (the first layer of a network needs no
  input gradient).
- ``lenet_train``: one SGD-momentum step of the LeNet-style network.
- ``lenet_score``: forward-only scoring of ``images`` images in minibatches.
- ``classifier``: one training step of the softmax classifier: affine forward,
  softmax + cross-entropy, affine backward, SGD with momentum.
- ``pool``: bias_add + relu of a conv output, then max-pool forward and backward.

Buffers, workspaces and parameters are allocated once, as a training loop keeps
them.  The backward passes of a conv layer take the relu mask (out_fwd) as an
input of its own: a mask computed by the forward under test would flip where a
pre-activation is within rounding of zero and make two correct results differ.
"""
import math

import torch
import torch.nn.functional as TF

from paper_1802_04647_amd import dmlnn
from paper_1802_04647_amd.lenet import PARAM_ORDER, LeNetScorer, LeNetTrainer

_DT = {"f64": torch.float64, "f32": torch.float32}
_LR, _MU = 0.01, 0.9
_MAX_PASS_FLOPS = 3e10   # of a drawn conv pass (the largest listed one: 5.9e10)


def listed():
    conv = dict(kind="conv")
    return [
        # A conv2_x layer of a ResNet at a full training batch: the benchmark's
        # layer, in the library's primary type and in fp32.  The largest calls.
        dict(conv, name="conv_resnet_f64", dtype="f64", N=256, C=64, H=56, W=56, F=64, K=3,
             stride=1, pad=1, passes="step"),
        dict(conv, name="conv_resnet_f32", dtype="f32", N=256, C=64, H=56, W=56, F=64, K=3,
             stride=1, pad=1, passes="step"),
        # The layer that halves the image and doubles the channels between two stages.
        dict(conv, name="conv_down_f64", dtype="f64", N=32, C=64, H=56, W=56, F=128, K=3,
             stride=2, pad=1, passes="step"),
        # A layer of a deep stage: many channels, small images.
        dict(conv, name="conv_deep_f32", dtype="f32", N=64, C=256, H=14, W=14, F=256, K=3,
             stride=1, pad=1, passes="step"),
        # A 1x1 (channel mixing) layer.
        dict(conv, name="conv_point_f32", dtype="f32", N=64, C=256, H=28, W=28, F=128, K=1,
             stride=1, pad=0, passes="step"),
        # A network's first layer: three channels, wide rows, a large filter.
        dict(conv, name="conv_first_f32", dtype="f32", N=32, C=3, H=224, W=224, F=64, K=7,
             stride=2, pad=3, passes="first"),
        # A small batch with nothing a power of two.
        dict(conv, name="conv_ragged_f64", dtype="f64", N=5, C=45, H=27, W=31, F=70, K=5,
             stride=1, pad=2, passes="step"),
        # The LeNet-style network's training step at the default batch: about
        # twenty short launches.
        dict(kind="lenet_train", name="lenet_train_f64", dtype="f64", batch=64),
        # Scoring with it over four streams.
        dict(kind="lenet_score", name="lenet_score_f32", dtype="f32", batch=64, images=1024),
        # The softmax classifier on MNIST-shaped rows: the smallest calls.
        dict(kind="classifier", name="classifier_small_f64", dtype="f64", N=64, D=784, M=10),
        # The same as the head of a large network: wide features, 1000 classes.
        dict(kind="classifier", name="classifier_large_f32", dtype="f32", N=512, D=2048, M=1000),
        # The stem's overlapping pool behind a separate bias and relu.
        dict(kind="pool", name="pool_f32", dtype="f32", N=32, C=64, H=112, W=112, K=3, stride=2,
             pad=1),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["conv", "conv", "conv", "conv", "conv", "lenet_train", "lenet_score",
                       "classifier", "classifier", "pool"])
    dtype = rng.choice(["f64", "f32"])
    if kind == "conv":
        while True:
            K = rng.choice([1, 3, 3, 3, 5, 7])
            c = dict(kind="conv", dtype=dtype, N=_log(rng, 1, 256), C=_log(rng, 1, 512),
                     H=_log(rng, 7, 224), F=_log(rng, 8, 512), K=K, stride=rng.choice([1, 1, 2]),
                     pad=rng.choice([K // 2, K // 2, 0]), passes=rng.choice(["step", "step", "fwd"]))
            c["W"] = max(7, c["H"] + rng.choice([0, 0, 0, 1, -1, 3]))
            if K >= 5 and c["C"] > 64:
                continue
            Ho, Wo = _out_hw(c)
            if Ho < 1 or Wo < 1:
                continue
            flops = 2.0 * c["N"] * c["F"] * Ho * Wo * c["C"] * K * K
            cells = c["N"] * max(c["C"] * c["H"] * c["W"], c["F"] * Ho * Wo)
            if 2e7 <= flops <= _MAX_PASS_FLOPS and cells <= 4e7:
                return c
    if kind == "lenet_train":
        return dict(kind=kind, dtype="f64", batch=_log(rng, 16, 160))
    if kind == "lenet_score":
        b = _log(rng, 16, 128)
        return dict(kind=kind, dtype=dtype, batch=b, images=b * rng.randint(4, 16))
    if kind == "classifier":
        return dict(kind=kind, dtype=dtype, N=_log(rng, 16, 1024), D=_log(rng, 64, 4096),
                    M=_log(rng, 2, 1024))
    while True:
        K = rng.choice([2, 3])
        c = dict(kind="pool", dtype=dtype, N=_log(rng, 1, 128), C=_log(rng, 8, 256),
                 H=_log(rng, 8, 112), K=K, stride=2, pad=rng.choice([0, K - 2]))
        c["W"] = max(8, c["H"] + rng.choice([0, 0, 1]))
        if 1e5 <= c["N"] * c["C"] * c["H"] * c["W"] <= 2.6e7:
            return c


def _out_hw(c):
    o = lambda n: (n + 2 * c["pad"] - c["K"]) // c["stride"] + 1  # noqa: E731
    return o(c["H"]), o(c["W"])


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _inputs(case, seed):
    """The inputs of a case, from the seed alone."""
    dev, dt = _device(), _DT[case["dtype"]]
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    n = lambda *s: torch.randn(*s, generator=gen, dtype=dt, device=dev)  # noqa: E731
    kind = case["kind"]
    if kind == "conv":
        N, C, H, W, F, K = (case[k] for k in ("N", "C", "H", "W", "F", "K"))
        Ho, Wo = _out_hw(case)
        d = dict(X=n(N, C * H * W).relu_(), W=n(F, C * K * K) * math.sqrt(2.0 / (C * K * K)),
                 b=0.1 * n(F))
        if case["passes"] != "fwd":
            d.update(dout=n(N, F * Ho * Wo), out_fwd=n(N, F * Ho * Wo).relu_())
        return d
    if kind in ("lenet_train", "lenet_score"):
        M = case["batch"] if kind == "lenet_train" else case["images"]
        # MNIST-shaped images: about 80% exact zeros, the rest uniform in [0, 1)
        u = torch.rand(M, 784, generator=gen, dtype=dt, device=dev)
        keep = torch.rand(M, 784, generator=gen, dtype=dt, device=dev) < 0.2
        p = {}
        for k, s, fan in (("W1", (32, 25), 25), ("W2", (64, 800), 800), ("W3", (3136, 512), 3136),
                          ("W4", (512, 10), 512)):
            p[k] = n(*s) * math.sqrt(2.0 / fan)
        for k, s in (("b1", (32,)), ("b2", (64,)), ("b3", (512,)), ("b4", (10,))):
            p[k] = 0.1 * n(*s)
        lab = torch.randint(0, 10, (M,), generator=gen, device=dev)
        return dict(X=u * keep, Y=TF.one_hot(lab, 10).to(dt), params=p)
    if kind == "classifier":
        N, D, M = case["N"], case["D"], case["M"]
        lab = torch.randint(0, M, (N,), generator=gen, device=dev)
        return dict(X=n(N, D).relu_(), Y=TF.one_hot(lab, M).to(dt),
                    W=n(D, M) * math.sqrt(2.0 / D), b=0.1 * n(M))
    N, C, H, W = (case[k] for k in ("N", "C", "H", "W"))
    Ho, Wo = _out_hw(case)
    return dict(X=n(N, C * H * W), b=0.1 * n(C), dout=n(N, C * Ho * Wo))


def prepare(case, seed):
    s = dict(case=case, **_inputs(case, seed))
    kind, dt = case["kind"], _DT[case["dtype"]]
    e = lambda *sh: torch.empty(*sh, dtype=dt, device="cuda")  # noqa: E731
    if kind == "conv":
        N, C, H, W, F, K = (case[k] for k in ("N", "C", "H", "W", "F", "K"))
        Ho, Wo = _out_hw(case)
        s["out"] = e(N, F * Ho * Wo)
        if case["passes"] != "fwd":
            nb = dmlnn.conv2d_backward_filter_workspace_size(dt, N, C, H, W, F, K, K,
                                                             case["stride"], case["pad"])
            s.update(ws=torch.empty(max(nb, 1), dtype=torch.uint8, device="cuda"),
                     dW=e(F, C * K * K), db=e(F))
        if case["passes"] == "step":
            s.update(g=e(N, F * Ho * Wo), dX=e(N, C * H * W))
    elif kind == "lenet_train":
        s["trainer"] = LeNetTrainer(s["params"], N=case["batch"], lr=_LR, mu=_MU, dtype=dt)
    elif kind == "lenet_score":
        s["scorer"] = LeNetScorer(s["params"], batch=case["batch"], streams=4, dtype=dt)
    elif kind == "classifier":
        N, D, M = case["N"], case["D"], case["M"]
        # parameters, gradients and velocities in one flat buffer each
        s["p"] = torch.cat([s.pop("W").reshape(-1), s.pop("b")])
        s.update(g=e(D * M + M), v=torch.zeros_like(s["p"]), scores=e(N, M), loss=e(1),
                 ds=e(N, M), dX=e(N, D),
                 wsa=torch.empty(dmlnn.affine_workspace_size(dt, N, D, M), dtype=torch.uint8,
                                 device="cuda"),
                 wss=torch.empty(dmlnn.softmax_xent_workspace_size(dt, N, M), dtype=torch.uint8,
                                 device="cuda"))
        for k in ("p", "g"):
            s[k + "_W"], s[k + "_b"] = s[k][:D * M].view(D, M), s[k][D * M:]
    else:
        N, C, H, W = (case[k] for k in ("N", "C", "H", "W"))
        Ho, Wo = _out_hw(case)
        s.update(act=e(N, C * H * W), out=e(N, C * Ho * Wo), dX=e(N, C * H * W),
                 argmax=torch.empty(N, C * Ho * Wo, dtype=torch.int32, device="cuda"))
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "conv":
        a = (c["C"], c["H"], c["W"], c["K"], c["K"], c["stride"], c["pad"])
        dmlnn.conv2d_forward(s["X"], s["W"], s["b"], *a, relu=True, out=s["out"])
        if c["passes"] == "fwd":
            return dict(out=s["out"])
        if c["passes"] == "first":
            dmlnn.conv2d_backward_filter(s["X"], s["dout"], s["out_fwd"], *a, c["F"],
                                         workspace=s["ws"], dW=s["dW"], db=s["db"])
            return dict(out=s["out"], dW=s["dW"], db=s["db"])
        dmlnn.conv2d_backward_filter(s["X"], s["dout"], s["out_fwd"], *a, c["F"],
                                     workspace=s["ws"], dW=s["dW"], db=s["db"], g_out=s["g"])
        dmlnn.conv2d_backward_data(s["W"], s["g"], None, *a, dX=s["dX"])
        return dict(out=s["out"], dW=s["dW"], db=s["db"], dX=s["dX"])
    if kind == "lenet_train":
        t = s["trainer"]
        loss = t.step(s["X"], s["Y"])
        return dict(loss=loss, grads=t.g_flat, params=t.p_flat)
    if kind == "lenet_score":
        return dict(probs=s["scorer"].score(s["X"]))
    if kind == "classifier":
        dmlnn.affine_fwd(s["X"], s["p_W"], s["p_b"], out=s["scores"], workspace=s["wsa"])
        dmlnn.softmax_xent(s["scores"], s["Y"], want_probs=False, loss=s["loss"],
                           dscores=s["ds"], workspace=s["wss"])
        dmlnn.affine_bwd(s["ds"], s["X"], s["p_W"], None, dX=s["dX"], dW=s["g_W"], db=s["g_b"],
                         workspace=s["wsa"])
        dmlnn.sgd_momentum_update(s["p"], s["g"], s["v"], _LR, _MU)
        return dict(scores=s["scores"], loss=s["loss"], dX=s["dX"], grads=s["g"], params=s["p"])
    a = (c["C"], c["H"], c["W"], c["K"], c["K"], c["stride"], c["pad"])
    dmlnn.bias_add_relu(s["X"], s["b"], c["C"], c["H"] * c["W"], out=s["act"])
    dmlnn.max_pool2d_fwd(s["act"], *a, out=s["out"], argmax=s["argmax"])
    dmlnn.max_pool2d_bwd(s["dout"], s["argmax"], *a, dX=s["dX"])
    return dict(act=s["act"], out=s["out"], argmax=s["argmax"], dX=s["dX"])


# LeNet per image: multiply-adds of conv1, conv2, affine 1, affine 2 and elements moved
_LENET_MACS = 32 * 784 * 25, 64 * 196 * 800, 3136 * 512, 512 * 10
_LENET_PARAMS = 32 * 25 + 32 + 64 * 800 + 64 + 3136 * 512 + 512 + 512 * 10 + 10


def work(case):
    z = 8 if case["dtype"] == "f64" else 4
    kind = case["kind"]
    if kind == "conv":
        N, C, H, W, F, K = (case[k] for k in ("N", "C", "H", "W", "F", "K"))
        Ho, Wo = _out_hw(case)
        n = {"fwd": 1, "first": 2, "step": 3}[case["passes"]]
        x, o, w = N * C * H * W, N * F * Ho * Wo, F * C * K * K
        return dict(flops=2.0 * n * o * C * K * K,
                    bytes=z * ({1: x + o + w, 2: x + 3 * o + 2 * w, 3: 2 * x + 3 * o + 2 * w}[n]))
    if kind == "lenet_train":
        c1, rest = _LENET_MACS[0], sum(_LENET_MACS[1:])
        # conv1 has no input gradient; parameters, velocities and gradients of the update
        return dict(flops=2.0 * case["batch"] * (2 * c1 + 3 * rest),
                    bytes=z * (case["batch"] * 794 + 5 * _LENET_PARAMS))
    if kind == "lenet_score":
        return dict(flops=2.0 * case["images"] * sum(_LENET_MACS),
                    bytes=z * (case["images"] * 794 + _LENET_PARAMS))
    if kind == "classifier":
        N, D, M = case["N"], case["D"], case["M"]
        return dict(flops=6.0 * N * D * M, bytes=z * (2 * N * D + 3 * N * M + 5 * (D * M + M)))
    N, C, H, W = (case[k] for k in ("N", "C", "H", "W"))
    Ho, Wo = _out_hw(case)
    x, o = N * C * H * W, N * C * Ho * Wo
    return dict(flops=0, bytes=z * (3 * x + 2 * o) + 4 * o)


def tolerance(case):
    """Against 64 bits the library is off by up to 5e-7 in fp32 (dW of the largest layer, a sum over
    802,816 pixels; the products of the other cases 1e-7 to 4e-7) and 1.5e-14 in fp64."""
    if case["kind"] == "pool":  # selections are exact; at most four gradients are summed (3e-8)
        return {"rel": 2e-7 if case["dtype"] == "f32" else 4e-16}
    return {"rel": 4e-6, "max": 2e-4} if case["dtype"] == "f32" else {"rel": 1e-13, "max": 4e-12}


# ------------------------------------------------------------------ reference in 64 bits
def _taps(case):
    return [(i, j) for i in range(case["K"]) for j in range(case["K"])]


def _conv_exact(case, d):
    """The layer's passes as one matrix product per filter tap."""
    N, C, H, W, F, K = (case[k] for k in ("N", "C", "H", "W", "F", "K"))
    S, P = case["stride"], case["pad"]
    Ho, Wo = _out_hw(case)
    Xp = TF.pad(d["X"].double().view(N, C, H, W), (P, P, P, P))
    Wt = d["W"].double().view(F, C, K, K)

    def window(t, i, j):
        return t[:, :, i:i + (Ho - 1) * S + 1:S, j:j + (Wo - 1) * S + 1:S]

    out = torch.zeros(F, N * Ho * Wo, dtype=torch.float64, device=Xp.device)
    flat = lambda t: t.transpose(0, 1).reshape(t.shape[1], -1).contiguous()  # noqa: E731
    for i, j in _taps(case):
        out += Wt[:, :, i, j].contiguous() @ flat(window(Xp, i, j))
    out = (out + d["b"].double()[:, None]).relu_()
    res = dict(out=out.view(F, N, Ho * Wo).transpose(0, 1).reshape(N, -1))
    if case["passes"] == "fwd":
        return res
    g = (d["dout"].double() * (d["out_fwd"] > 0)).view(N, F, Ho, Wo)
    gf = flat(g)
    dW = torch.empty(F, C, K, K, dtype=torch.float64, device=Xp.device)
    for i, j in _taps(case):
        dW[:, :, i, j] = gf @ flat(window(Xp, i, j)).t().contiguous()
    res.update(dW=dW.view(F, -1), db=g.sum((0, 2, 3)))
    if case["passes"] == "step":
        dXp = torch.zeros_like(Xp)
        for i, j in _taps(case):
            t = Wt[:, :, i, j].t().contiguous() @ gf
            window(dXp, i, j).add_(t.view(C, N, Ho, Wo).transpose(0, 1))
        res["dX"] = dXp[:, :, P:P + H, P:P + W].reshape(N, -1)
    return res


def _lenet(X, p):
    h = X.view(-1, 1, 28, 28)
    h = TF.max_pool2d(TF.conv2d(h, p["W1"].view(32, 1, 5, 5), p["b1"], padding=2).relu(), 2)
    h = TF.max_pool2d(TF.conv2d(h, p["W2"].view(64, 32, 5, 5), p["b2"], padding=2).relu(), 2)
    h = (h.flatten(1) @ p["W3"] + p["b3"]).relu()
    return h @ p["W4"] + p["b4"]


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "conv":
        return _conv_exact(case, d)
    if kind in ("lenet_train", "lenet_score"):  # on the CPU, in 64 bits
        X, Y = d["X"].double().cpu(), d["Y"].double().cpu()
        p = {k: v.double().cpu() for k, v in d["params"].items()}
        if kind == "lenet_score":
            return dict(probs=_lenet(X, p).softmax(1))
        for k in PARAM_ORDER:
            p[k].requires_grad_()
        loss = -(Y * _lenet(X, p).log_softmax(1)).sum() / X.shape[0]
        loss.backward()
        grads = torch.cat([p[k].grad.reshape(-1) for k in PARAM_ORDER])
        flat = torch.cat([p[k].detach().reshape(-1) for k in PARAM_ORDER])
        return dict(loss=loss.detach().view(1), grads=grads, params=flat - _LR * grads)
    if kind == "classifier":
        X, Y, W, b = (d[k].double() for k in ("X", "Y", "W", "b"))
        scores = X @ W + b
        loss = -(Y * scores.log_softmax(1)).sum() / X.shape[0]
        ds = (scores.softmax(1) - Y) / X.shape[0]
        grads = torch.cat([(X.t().contiguous() @ ds).reshape(-1), ds.sum(0)])
        params = torch.cat([W.reshape(-1), b]) - _LR * grads
        return dict(scores=scores, loss=loss.view(1), dX=ds @ W.t().contiguous(), grads=grads,
                    params=params)
    N, C, H, W, K = (case[k] for k in ("N", "C", "H", "W", "K"))
    S, P = case["stride"], case["pad"]
    Ho, Wo = _out_hw(case)
    # bias_add rounds once in the case's type; everything after it selects
    act = (d["X"].view(N, C, H, W) + d["b"].view(1, C, 1, 1)).relu_()
    out, idx = TF.max_pool2d(act.double(), K, S, P, return_indices=True)
    dX = torch.zeros(N, C, H * W, dtype=torch.float64, device=act.device)
    dX.scatter_add_(2, idx.view(N, C, -1), d["dout"].double().view(N, C, -1))
    argmax = idx.view(N, C, -1) + H * W * torch.arange(C, device=act.device).view(1, C, 1)
    return dict(act=act.double().view(N, -1), out=out.reshape(N, -1),
                argmax=argmax.reshape(N, -1).to(torch.int32), dX=dX.view(N, -1))
