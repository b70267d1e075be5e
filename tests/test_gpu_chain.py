"""fp32 runs of layers in one launch against the layers apart and the oracle.

RAFIKI_CHAINS=0 runs every layer apart.  The chain sums the same products in groups of four and
the mean adds its positions in another order: both agree with the layers and the oracle to a
few units of 2^-24 of the sums of a few hundred values.  Cases
cover bands of one to all rows, odd maps whose pool drops a row and a column, a pool as the
last layer, channel counts below the storage padding, 1x1 layers, several members and a handle
whose other model needs the images staged.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads import Layer, ModelSpec, CONV2D, MAXPOOL2D, GLOBAL_AVGPOOL, FC
from paper_1804_06087_amd import Ensemble

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def conv(i, c_in, c_out, k, relu=True, s=1):
    return Layer(op=CONV2D, input=i, c_in=c_in, c_out=c_out, kh=k, kw=k, stride=s, pad=k // 2, relu=relu, bn=True)


def pool(i, c):
    return Layer(op=MAXPOOL2D, input=i, c_in=c, c_out=c, kh=2, kw=2, stride=2)


def model(layers, shape, classes=10, flatten=False):
    L = list(layers)
    c = L[-1].c_out
    if flatten:     # the chain's stored map itself, flattened: every element reaches the logits
        h, w = shape[1:]
        for lay in L:
            if lay.op == MAXPOOL2D:
                h, w = h // 2, w // 2
        L.append(Layer(op=FC, input=len(L) - 1, c_in=c * h * w, c_out=classes, bias=True))
    else:
        L.append(Layer(op=GLOBAL_AVGPOOL, input=len(L) - 1, c_in=c, c_out=c))
        L.append(Layer(op=FC, input=len(L) - 1, c_in=c, c_out=classes, bias=True))
    return ModelSpec("chain", L, classes, shape)


TOY = ([conv(-1, 3, 16, 3), pool(0, 16), conv(1, 16, 32, 3)], (3, 32, 32))
CASES = {
    "toy": TOY,
    "odd": ([conv(-1, 1, 5, 3), pool(0, 5), conv(1, 5, 12, 3, relu=False), conv(2, 12, 9, 1)], (1, 11, 7)),
    "pool_last": ([conv(-1, 3, 6, 3), conv(0, 6, 20, 3), pool(1, 20)], (3, 9, 14)),
    "one_row": ([conv(-1, 2, 4, 1), conv(0, 4, 70, 3)], (2, 1, 130)),
    "many_channels": ([conv(-1, 3, 24, 3), conv(0, 24, 40, 3)], (3, 12, 10)),
    "deep": ([conv(-1, 3, 8, 3)] + [conv(i, 8, 8, 3) for i in range(5)] + [pool(5, 8), conv(6, 8, 8, 3)], (3, 26, 20)),
}


def run(specs, params, x, n, mode, monkeypatch, precision="fp32"):
    monkeypatch.setenv("RAFIKI_CHAINS", mode)
    with Ensemble(specs, params, precision=precision, max_batch=n) as ens:
        C = specs[0].n_classes
        zs = []
        for m in range(len(specs)):
            out = torch.full((n, C), float("nan"), dtype=torch.float32, device=DEV)
            ens.model_logits(m, x, n, out)
            torch.cuda.synchronize()
            zs.append(out.cpu().numpy())
        probs = torch.empty((n, C), dtype=torch.float32, device=DEV)
        labels = torch.empty((n,), dtype=torch.int32, device=DEV)
        ens.infer(x, n, (1 << len(specs)) - 1, probs, labels)
        ens.use_graphs(True)
        again = torch.empty_like(probs)
        for _ in range(3):
            again.zero_()
            ens.infer(x, n, (1 << len(specs)) - 1, again, labels)
            torch.cuda.synchronize()
            assert torch.equal(again, probs)
        ens.use_graphs(False)
        ens.trace(True)
        ens.infer(x, n, (1 << len(specs)) - 1, probs, labels)
        kinds = [r["kind"] for r in ens.trace_read()]
    return zs, probs.cpu().numpy(), kinds


@pytest.mark.parametrize("n", [1, 3, 70])
@pytest.mark.parametrize("name", sorted(CASES))
def test_chain_matches_layers(name, n, monkeypatch):
    layers, shape = CASES[name]
    spec = model(layers, shape, flatten=True)
    params = [wl.gen_params(spec, s, False, "random") for s in (3, 4)]
    batch = wl.gen_images(n, shape, "normal", False, seed=n)
    x = torch.from_numpy(batch).to(DEV)
    z1, p1, k1 = run([spec] * 2, params, x, n, "1", monkeypatch)
    z0, p0, k0 = run([spec] * 2, params, x, n, "0", monkeypatch)
    # chain, FC, combine, both members at once; "deep" exceeds LDS and leaves a layer apart, or
    # more where its bands of one row would recompute too much
    assert "stage" in k0 and "stage" not in k1
    assert len(k1) > 4 if (name, n) == ("deep", 70) else len(k1) == (4 if name == "deep" else 3)
    # layers of at most 180 terms (2^-24 each, random signs) and an FC over the whole map
    for a, b in zip(z1, z0):
        assert np.abs(a - b).max() <= 4e-6 * np.abs(b).max()
    assert np.abs(p1 - p0).max() <= 1e-4
    if n == 3:
        ref = oracle.run_model(spec, params[0], batch)
        err1, err0 = np.abs(z1[0] - ref).max(), np.abs(z0[0] - ref).max()
        assert err1 <= 1e-5 * np.abs(ref).max() and err1 <= 4 * err0 + 1e-6 * np.abs(ref).max()


@pytest.mark.parametrize("name", ["toy", "odd", "one_row"])
def test_tail_matches_oracle(name, monkeypatch):
    layers, shape = CASES[name]
    spec = model(layers, shape, classes=7)
    params = [wl.gen_params(spec, s, False, "random") for s in (3, 4)]
    for n in (1, 9):
        batch = wl.gen_images(n, shape, "uniform", False, seed=n)
        x = torch.from_numpy(batch).to(DEV)
        z1, _, k1 = run([spec] * 2, params, x, n, "1", monkeypatch)
        z0, _, _ = run([spec] * 2, params, x, n, "0", monkeypatch)
        assert len(k1) == 3                                          # chain, mean + FC, combine
        for m in range(2):
            ref = oracle.run_model(spec, params[m], batch)
            tol = 2e-6 * np.abs(ref).max()       # sums of at most 396 terms in fp32: under 32 units of 2^-24
            assert np.abs(z1[m] - ref).max() <= tol and np.abs(z1[m] - z0[m]).max() <= tol


def test_mixed_handle_keeps_staging(monkeypatch):
    """A model whose first layer strides cannot chain: the handle stages and nothing changes."""
    a = model(*TOY)
    b = model([conv(-1, 3, 8, 3, s=2), conv(0, 8, 8, 3)], (3, 32, 32))
    params = [wl.gen_params(a, 1, False, "random"), wl.gen_params(b, 2, False, "random")]
    batch = wl.gen_images(4, (3, 32, 32), "uniform", False, seed=1)
    x = torch.from_numpy(batch).to(DEV)
    z1, _, k1 = run([a, b], params, x, 4, "1", monkeypatch)
    assert "stage" in k1
    for spec, p, z in zip((a, b), params, z1):
        ref = oracle.run_model(spec, p, batch)
        assert np.abs(z - ref).max() <= 1e-5 * np.abs(ref).max()


def test_deep_chain_shortens_for_large_batches(monkeypatch):
    """Six 3x3 layers whose bands are one row: all in one launch for few images, where latency
    counts; for many, where each band's halo is recomputed work, the last layers run apart."""
    layers = [conv(-1, 3, 8, 3)] + [conv(i, 8, 8, 3) for i in range(5)]
    spec = model(layers, (3, 26, 20))
    params = [wl.gen_params(spec, 3, False, "random")]
    launches = {}
    for n in (8, 512):
        x = torch.from_numpy(wl.gen_images(n, (3, 26, 20), "normal", False, seed=n)).to(DEV)
        z1, p1, k1 = run([spec], params, x, n, "1", monkeypatch)
        z0, p0, _ = run([spec], params, x, n, "0", monkeypatch)
        assert "stage" not in k1
        launches[n] = k1.count("conv_f32")
        # 72 to 576 terms a layer in fp32, six layers and the mean
        assert np.abs(z1[0] - z0[0]).max() <= 4e-6 * np.abs(z0[0]).max()
        assert np.abs(p1 - p0).max() <= 1e-4
    assert launches[8] == 2                 # the chain, and the mean with the FC
    assert launches[512] > launches[8]


@pytest.mark.parametrize("hw, c, classes, joined", [
    ((64, 64), 24, 1000, True), ((24, 24), 128, 10, True), ((7, 7), 64, 1000, True),
    ((32, 32), 96, 10, False), ((7, 7), 128, 1000, False), ((7, 7), 256, 1000, False), ((128, 128), 16, 10, False),
])
def test_tail_joins_small_means_only(hw, c, classes, joined, monkeypatch):
    """The mean and the FC share a launch only where one workgroup per request is not too little
    for them; either way the logits are those of the layers apart."""
    spec = model([conv(-1, 3, c, 1)], (3,) + hw, classes=classes)
    params = [wl.gen_params(spec, 3, False, "random")]
    x = torch.from_numpy(wl.gen_images(2, (3,) + hw, "uniform", False, seed=1)).to(DEV)
    z1, _, k1 = run([spec], params, x, 2, "1", monkeypatch)
    z0, _, k0 = run([spec], params, x, 2, "0", monkeypatch)
    assert k0 == ["stage", "conv_f32", "pool", "conv_f32", "combine"]
    assert k1 == (["stage", "conv_f32", "conv_f32", "combine"] if joined else k0)
    # means of 49 to 16,384 positive values in slices, in fp32
    assert np.abs(z1[0] - z0[0]).max() <= 4e-6 * np.abs(z0[0]).max()
