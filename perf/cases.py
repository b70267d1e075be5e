"""The calls that a user of this framework times: whole requests through ``Ensemble.infer`` and
``Ensemble.model_logits`` (one handle per deployed ensemble, as a server keeps it, and a new batch
per call) and the combine of logits that a caller already holds.

The ensembles, their batch sizes and their subsets are those of the benchmark configurations: two toy
CNNs (fp32), three CIFAR ResNet-20s, ResNet-50 + VGG-16 + ResNet-101 with the subset / batch-size sweep
and the serving sizes, and four TextCNNs.  The models' weights are drawn once per process from fixed
seeds; requests are drawn from the case's seed.  Weights are bfloat16 values (they are the model);
requests are ordinary float32 values.  Batch-norm gains and classifier scales are those of a network
whose logits have a standard deviation of about two, so that probabilities are neither uniform nor
one-hot.
"""
import math

import torch

from paper_1804_06087_amd import binding
from workloads import gen, specs

# ensemble -> (model builders, precision, the largest batch its handle serves, input distribution)
ENSEMBLES = {
    "toy": ((specs.toy_cnn,) * 2, "fp32", 64, "uniform"),
    "cifar": ((specs.resnet20,) * 3, "bf16", 512, "uniform"),
    "imagenet": ((specs.resnet50, specs.vgg16, specs.resnet101), "bf16", 256, "normal"),
    "text": ((specs.textcnn,) * 4, "bf16", 512, "tokens"),
}
# residual networks: the gain of a block's last batch-norm; each model's classifier scale against He's
LAST_GAMMA = 0.25
FC_SCALE = {"toy": (2.0,) * 2, "cifar": (3.0,) * 3, "imagenet": (0.25, 0.6, 0.09), "text": (4.0,) * 4}


def listed():
    return [
        # the smallest request of all: two toy CNNs in fp32, eight images; launches and latency only
        dict(name="toy_fp32_b8", task="infer", ensemble="toy", mask=3, n=8),
        # CIFAR-sized ensemble at its configured batch
        dict(name="resnet20x3_b128", task="infer", ensemble="cifar", mask=7, n=128),
        # the sweep's lowest latency point: one image through one model
        dict(name="resnet50_b1", task="infer", ensemble="imagenet", mask=1, n=1),
        # a small request on two models: the weights' bytes and the launches count
        dict(name="resnet50_vgg16_b4", task="infer", ensemble="imagenet", mask=3, n=4),
        # the smallest serving batch through the whole ensemble
        dict(name="imagenet3_b16", task="infer", ensemble="imagenet", mask=7, n=16),
        # the headline: the whole ensemble at batch 64
        dict(name="imagenet3_b64", task="infer", ensemble="imagenet", mask=7, n=64),
        # the largest batch of the sweep
        dict(name="imagenet3_b256", task="infer", ensemble="imagenet", mask=7, n=256),
        # one model of an asynchronous deployment (each model its own server) at a serving size
        dict(name="vgg16_logits_b48", task="logits", ensemble="imagenet", model=1, n=48),
        # a queue's remainder: an odd batch through the deepest model alone
        dict(name="resnet101_logits_b27", task="logits", ensemble="imagenet", model=2, n=27),
        # sentiment ensemble at its configured batch
        dict(name="textcnn4_b512", task="infer", ensemble="text", mask=15, n=512),
        # a few sequences through one text model
        dict(name="textcnn_b3", task="infer", ensemble="text", mask=1, n=3),
        # logits of models that ran elsewhere, combined here (a memory-bound pass)
        dict(name="combine_mean_3x65536x1000", task="combine", how="mean", models=3, n=65536, classes=1000),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5))))))


def draw(rng):
    kind = rng.choice(("imagenet", "imagenet", "imagenet", "logits", "text", "text", "cifar", "toy", "combine"))
    if kind == "combine":
        return dict(task="combine", how=rng.choice(("mean", "vote")), models=rng.randint(2, 4),
                    n=_log_int(rng, 16, 32768), classes=_log_int(rng, 2, 1000))
    if kind == "logits":
        return dict(task="logits", ensemble="imagenet", model=rng.randrange(3), n=_log_int(rng, 1, 256))
    builders, _, most, _ = ENSEMBLES[kind]
    return dict(task="infer", ensemble=kind, mask=rng.randint(1, 2 ** len(builders) - 1), n=_log_int(rng, 1, most))


# ---------------------------------------------------------------- the deployed models

# first model seed of each ensemble: draws whose two best classes lie apart, as a trained classifier's do, so
# that a label depends on the request and the models and not on the last bit of a sum
SEEDS = {"toy": 1180, "cifar": 1060, "imagenet": 1080, "text": 1060}


def _parameters(name, spec, seed):
    """He-normal weights (embedding tables N(0, 0.1)), zero biases, random inference batch-norm, drawn layer
    by layer; the last batch-norm of a residual block has a small gain, as in a trained network."""
    g = torch.Generator(device="cuda").manual_seed(SEEDS[name] + seed)
    bf16 = ENSEMBLES[name][1] == "bf16"
    host = lambda t: t.float().cpu().numpy()  # noqa: E731
    out = []
    for i, L in enumerate(spec.layers):
        p = gen.LayerParams()
        if L.has_weight():
            std = 0.1 if L.op == specs.EMBEDDING else math.sqrt(2.0 / L.fan_in())
            if i == len(spec.layers) - 1:
                std *= FC_SCALE[name][seed]
            w = torch.randn(L.weight_shape(), generator=g, device="cuda") * std
            p.weight = host(w.bfloat16() if bf16 else w)
        if L.bias:
            p.bias = host(torch.zeros(L.c_out))
        if L.bn:
            p.bn_gamma = host(torch.full((L.c_out,), LAST_GAMMA if L.input2 >= 0 else 1.0))
            p.bn_beta = host(torch.zeros(L.c_out))
            p.bn_mean = host(torch.randn(L.c_out, generator=g, device="cuda") * 0.1)
            p.bn_var = host(torch.rand(L.c_out, generator=g, device="cuda") + 0.5)
        out.append(p)
    return gen.ModelParams(spec, out, seed, bf16)


_kept = {}


def _models(name):
    if ("models", name) not in _kept:
        all_specs = [b() for b in ENSEMBLES[name][0]]
        _kept["models", name] = all_specs, [_parameters(name, s, k) for k, s in enumerate(all_specs)]
    return _kept["models", name]


def _handle(name):
    """The ensemble's handle: a server creates it once and keeps it for every request."""
    if ("handle", name) not in _kept:
        all_specs, params = _models(name)
        _kept["handle", name] = binding.Ensemble(all_specs, params, ENSEMBLES[name][1], max_batch=ENSEMBLES[name][2])
    return _kept["handle", name]


# ---------------------------------------------------------------- requests

def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = case["n"]
    if case["task"] == "combine":
        return torch.randn((case["models"], n, case["classes"]), generator=g, device="cuda") * 2.0
    spec = ENSEMBLES[case["ensemble"]][0][0]()
    dist = ENSEMBLES[case["ensemble"]][3]
    if dist == "tokens":
        return torch.randint(0, spec.vocab, (n, spec.input_shape[0]), generator=g, device="cuda", dtype=torch.int32)
    shape = (n,) + tuple(spec.input_shape)
    return (torch.rand if dist == "uniform" else torch.randn)(shape, generator=g, device="cuda")


def prepare(case, seed):
    n = case["n"]
    s = {"case": case, "x": _inputs(case, seed), "handle": None}
    classes = case.get("classes")
    if case["task"] != "combine":
        s["handle"] = _handle(case["ensemble"])
        classes = _models(case["ensemble"])[0][0].n_classes
    s["out"] = torch.empty((n, classes), device="cuda")
    s["labels"] = torch.empty(n, dtype=torch.int32, device="cuda")
    return s


def run(state):
    case, x, out, labels = state["case"], state["x"], state["out"], state["labels"]
    if case["task"] == "combine":
        (binding.combine_mean if case["how"] == "mean" else binding.combine_vote)(x, out, labels)
        return {"out": out, "labels": labels}
    if case["task"] == "logits":
        state["handle"].model_logits(case["model"], x, case["n"], out)
        return {"logits": out}
    state["handle"].infer(x, case["n"], case["mask"], out, labels)
    return {"probs": out, "labels": labels}


# ---------------------------------------------------------------- what a pass cannot do without

def _selected(case):
    if case["task"] == "logits":
        return [case["model"]]
    return [m for m in range(len(ENSEMBLES[case["ensemble"]][0])) if case["mask"] >> m & 1]


def _model_work(spec, n, item):
    """(FLOPs, weight bytes) of one model on n requests; an embedding's rows are read once each at most."""
    shapes = {-1: tuple(spec.input_shape)}
    flops = weights = 0
    for i, L in enumerate(spec.layers):
        x = shapes[L.input]
        if L.op == specs.CONV2D:
            h, w = ((d + 2 * L.pad - k) // L.stride + 1 for d, k in ((x[1], L.kh), (x[2], L.kw)))
            shapes[i] = (L.c_out, h, w)
            flops += 2 * n * h * w * L.c_out * L.fan_in()
        elif L.op == specs.MAXPOOL2D:
            shapes[i] = (L.c_out,) + tuple((d + 2 * L.pad - L.kh) // L.stride + 1 for d in x[1:])
        elif L.op == specs.EMBEDDING:
            shapes[i] = (L.c_out, x[0])
            weights += min(L.c_in, n * x[0]) * L.c_out * item
        elif L.op == specs.CONV1D_MAXTIME:
            shapes[i] = (L.c_out,)
            flops += 2 * n * (x[1] - L.kw + 1) * L.c_out * L.fan_in()
        else:
            shapes[i] = (L.c_out,)
            flops += 2 * n * L.c_out * L.c_in if L.op == specs.FC else 0
        if L.has_weight() and L.op != specs.EMBEDDING:
            weights += math.prod(L.weight_shape()) * item
    return flops, weights


def work(case):
    n = case["n"]
    if case["task"] == "combine":
        values = case["models"] * n * case["classes"]
        return {"bytes": 4 * (values + n * case["classes"] + n), "flops": 0}
    builders, precision, _, _ = ENSEMBLES[case["ensemble"]]
    flops, nbytes = 0, 4 * n * math.prod(builders[0]().input_shape)
    for m in _selected(case):
        f, w = _model_work(builders[m](), n, 4 if precision == "fp32" else 2)
        flops, nbytes = flops + f, nbytes + w
    classes = builders[0]().n_classes
    return {"bytes": nbytes + 4 * n * (classes + (case["task"] == "infer")), "flops": flops}


def tolerance(case):
    if case["task"] == "combine":
        return "exact" if case["how"] == "vote" else {"rel": 2e-6, "differ": 0.0005}
    if case["ensemble"] == "toy":
        return {"rel": 4e-6, "differ": 0.0}
    return {"rel": 0.02, "max": 0.5, "differ": 0.01}


# ---------------------------------------------------------------- the same in 64 bits

def _conv64(x, w, stride, pad):
    """Convolution as a sum of one matrix product per kernel tap, a few images at a time."""
    n, c, h, wd = x.shape
    o, _, kh, kw = w.shape
    ho, wo = (h + 2 * pad - kh) // stride + 1, (wd + 2 * pad - kw) // stride + 1
    y = torch.empty((n, o, ho, wo), dtype=x.dtype, device=x.device)
    step = max(1, (1 << 26) // (max(c, o) * h * wd))
    for at in range(0, n, step):
        p = torch.nn.functional.pad(x[at:at + step], (pad, pad, pad, pad)).permute(1, 0, 2, 3).contiguous()
        b = p.shape[1]
        acc = torch.zeros((o, b * ho * wo), dtype=x.dtype, device=x.device)
        for u in range(kh):
            for v in range(kw):
                rows = p[:, :, u:u + stride * (ho - 1) + 1:stride, v:v + stride * (wo - 1) + 1:stride]
                acc.addmm_(w[:, :, u, v].contiguous(), rows.reshape(c, -1))
        y[at:at + step] = acc.view(o, b, ho, wo).permute(1, 0, 2, 3)
    return y


def _logits64(spec, params, x):
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda().double()  # noqa: E731
    last = {}
    for i, L in enumerate(spec.layers):
        last[L.input] = last[L.input2] = i
    t = {-1: x if spec.vocab else x.double()}
    for i, (L, p) in enumerate(zip(spec.layers, params.layers)):
        a, w, b = t[L.input], dev(p.weight), dev(p.bias)
        if L.op == specs.CONV2D:
            y = _conv64(a, w, L.stride, L.pad)
            if b is not None:
                y += b.view(-1, 1, 1)
            if L.bn:
                s = dev(p.bn_gamma) / torch.sqrt(dev(p.bn_var) + p.bn_eps)
                y = y.mul_(s.view(-1, 1, 1)).add_((dev(p.bn_beta) - dev(p.bn_mean) * s).view(-1, 1, 1))
            if L.input2 >= 0:
                y += t[L.input2]
            y = y.clamp_(min=0) if L.relu else y
        elif L.op == specs.MAXPOOL2D:
            q = torch.nn.functional.pad(a, (L.pad,) * 4, value=-math.inf)
            y = q.unfold(2, L.kh, L.stride).unfold(3, L.kw, L.stride).amax((-1, -2))
        elif L.op == specs.GLOBAL_AVGPOOL:
            y = a.mean((2, 3))
        elif L.op == specs.EMBEDDING:
            y = w[a.long()]                                     # [n, length, dim]
        elif L.op == specs.CONV1D_MAXTIME:
            m = a.shape[1] - L.kw + 1
            z = sum(a[:, k:k + m].reshape(-1, L.c_in) @ w[:, :, k].t().contiguous() for k in range(L.kw))
            z = (z + b).clamp_(min=0) if L.relu else z + b
            y = z.view(a.shape[0], m, -1).amax(1)
        elif L.op == specs.CONCAT:
            y = torch.cat((a, t[L.input2]), 1)
        else:
            y = a.reshape(a.shape[0], -1) @ w.t().contiguous() + b
            y = y.clamp_(min=0) if L.relu else y
        t[i] = y
        for k in [k for k in t if k >= 0 and k != i and last.get(k, -1) <= i]:
            del t[k]
    return t[len(spec.layers) - 1]


def exact(case, seed):
    x = _inputs(case, seed)
    if case["task"] == "combine":
        z = x.double()
        if case["how"] == "mean":
            p = torch.softmax(z, -1).mean(0)
            return {"out": p, "labels": p.argmax(-1).int()}
        votes = z.argmax(-1)                                     # [models, n]
        counts = torch.zeros(z.shape[1:], dtype=torch.float64, device=z.device)
        counts.scatter_add_(1, votes.t().contiguous(), torch.ones_like(votes.t(), dtype=torch.float64))
        order = torch.arange(len(votes), device=z.device).view(-1, 1)
        best = (counts.gather(1, votes.t()).t() * 64 - order).argmax(0)
        return {"out": counts / len(votes), "labels": votes.gather(0, best.view(1, -1))[0].int()}
    all_specs, params = _models(case["ensemble"])
    step = 64
    logits = [torch.cat([_logits64(all_specs[m], params[m], x[at:at + step]) for at in range(0, case["n"], step)])
              for m in _selected(case)]
    if case["task"] == "logits":
        return {"logits": logits[0]}
    p = sum(torch.softmax(z, -1) for z in logits) / len(logits)
    return {"probs": p, "labels": p.argmax(-1).int()}
