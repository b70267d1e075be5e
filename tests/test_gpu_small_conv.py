"""The small-tile convolution kernel gives the bits of the tiled kernel and its reduce launch.

RAFIKI_SMALL_TILES=1..4 runs every layer the kernel takes with one of its tiles, 0 none.  Each
probe ends in a global average pool and a random FC (itself one of the layers): equal logits
mean equal outputs.  Cases: K split over the waves in one round and in several, unsplit,
1 x 1 and 3 x 3, strides, residual, the fused 2x2 max-pool, ragged rows and channels, padded
storage channels, a single row, and a grouped launch.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads import Layer, ModelSpec, CONV2D, MAXPOOL2D, GLOBAL_AVGPOOL, FC
from paper_1804_06087_amd import Ensemble
from paper_1804_06087_amd.binding import tile_configs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def conv(i, c_in, c_out, k, s=1, relu=True, res=-1):
    return Layer(op=CONV2D, input=i, input2=res, c_in=c_in, c_out=c_out, kh=k, kw=k, stride=s, pad=k // 2,
                 relu=relu, bn=True)


CASES = {
    # 9 splits: one round of waves; residual in the epilogue
    "k2304_residual": ([conv(-1, 256, 256, 1, relu=False), conv(-1, 256, 256, 3, res=0)], (256, 14, 14), 1),
    # 18 splits: two rounds; rows 49 of 64
    "k4608_two_rounds": ([conv(-1, 512, 512, 3)], (512, 7, 7), 1),
    # unsplit, stride 2, channels of no 16-multiple (storage padded to 128), ragged rows
    "k256_s2_cout114": ([conv(-1, 256, 114, 1, s=2)], (256, 9, 7), 3),
    # unsplit 3x3, rows across images
    "k576": ([conv(-1, 64, 96, 3)], (64, 5, 3), 5),
    # storage padded past the last 16-channel block of the layer's channels: zeros there
    "cout520_storage576": ([conv(-1, 64, 520, 1), conv(0, 520, 64, 1)], (64, 4, 5), 2),
    # split K with the fused max-pool; windows ragged against the tile
    "pool2_split": ([conv(-1, 512, 96, 3), Layer(op=MAXPOOL2D, input=0, c_in=96, c_out=96, kh=2, kw=2, stride=2)],
                    (512, 6, 10), 3),
    # a long K of many rounds into few rows (an FC of a whole map)
    "fc_long": ([], (512, 7, 7), 3),
    # one row
    "one_row": ([conv(-1, 128, 72, 1)], (128, 1, 1), 1),
}


def build(name):
    layers, shape, n = CASES[name]
    L = list(layers)
    if L:
        c = L[-1].c_out
        L.append(Layer(op=GLOBAL_AVGPOOL, input=len(L) - 1, c_in=c, c_out=c))
        L.append(Layer(op=FC, input=len(L) - 1, c_in=c, c_out=10, bias=True))
    else:
        c = int(np.prod(shape))
        L.append(Layer(op=FC, input=-1, c_in=c, c_out=200, bias=True, relu=True))
        L.append(Layer(op=FC, input=0, c_in=200, c_out=10, bias=True))
    return ModelSpec("small", L, 10, shape), n


def run(specs, params, x, n, mode, monkeypatch):
    monkeypatch.setenv("RAFIKI_SMALL_TILES", mode)
    with Ensemble(specs, params, precision="bf16", max_batch=n) as ens:
        out = torch.full((n, 10), float("nan"), dtype=torch.float32, device=DEV)
        for _ in range(2):
            ens.model_logits(0, x, n, out)
        probs = torch.empty((n, 10), dtype=torch.float32, device=DEV)
        labels = torch.empty((n,), dtype=torch.int32, device=DEV)
        ens.infer(x, n, (1 << len(specs)) - 1, probs, labels)
        torch.cuda.synchronize()
        z = out.cpu().numpy().copy()
        ens.trace(True)
        ens.model_logits(0, x, n, out)
        recs = [r for r in ens.trace_read() if r["kind"] in ("conv_mfma", "splitk_reduce")]
    return z, probs.cpu().numpy(), recs


@pytest.mark.parametrize("name", sorted(CASES))
def test_small_tiles_bitwise(name, monkeypatch):
    spec, n = build(name)
    params = wl.gen_params(spec, 3, True, "random")
    params2 = wl.gen_params(spec, 4, True, "random")       # a second member: grouped launches
    batch = wl.gen_images(n, spec.input_shape, "normal", True, seed=2)
    x = torch.from_numpy(batch).to(DEV)
    z0, p0, r0 = run([spec, spec], [params, params2], x, n, "0", monkeypatch)
    first = len(tile_configs()) + 4
    assert all(r["tile_cfg"] < first for r in r0)
    for t in range(4):
        z, p, recs = run([spec, spec], [params, params2], x, n, str(t + 1), monkeypatch)
        used = [r for r in recs if r["tile_cfg"] == first + t]
        assert used and not any(r["kind"] == "splitk_reduce" for r in recs if r["tile_cfg"] >= first)
        assert [r["splits"] for r in recs if r["kind"] == "conv_mfma"] == \
            [r["splits"] for r in r0 if r["kind"] == "conv_mfma"]
        assert np.array_equal(z.view(np.uint32), z0.view(np.uint32)), t
        assert np.array_equal(p.view(np.uint32), p0.view(np.uint32)), t
    ref = oracle.run_model(spec, params, batch, act="bf16")
    assert np.abs(z0 - ref).max() <= 1e-2 * np.abs(ref).max()


@pytest.mark.parametrize("c_in, k, split", [(64, 1, False), (64, 3, False), (256, 3, True)])
def test_small_tiles_nonfinite(c_in, k, split, monkeypatch):
    """A positive NaN (of a layer's shift; arithmetic gives negative ones here) ends as in the launches
    that the tile stands for: kept by the unsplit kernel's ReLU, an integer maximum, and 0 after
    the reduce launch's.  The request holds infinities and a NaN, the residual their opposites."""
    L = [conv(-1, c_in, 96, 1, relu=False), conv(-1, c_in, 96, k, res=0),
         Layer(op=GLOBAL_AVGPOOL, input=1, c_in=96, c_out=96),
         Layer(op=FC, input=2, c_in=96, c_out=10, bias=True)]
    spec = ModelSpec("nonfinite", L, 10, (c_in, 6, 7))
    params = wl.gen_params(spec, 3, True, "random")
    P = params.layers
    P[0].weight[:, 3], P[1].weight[:, 3] = -1.0, 1.0
    for p in P[:2]:
        p.bn_gamma = np.abs(p.bn_gamma) + 0.1
    P[1].bn_beta[5] = np.nan
    batch = wl.gen_images(4, spec.input_shape, "normal", True, seed=2).copy()
    batch[1:, 3, 0, 0] = np.inf, -np.inf, np.nan
    x = torch.from_numpy(batch).to(DEV)
    z0, _, r0 = run([spec], [params], x, 4, "0", monkeypatch)
    assert any(r["splits"] > 1 for r in r0) == split and np.isnan(z0[0]).all() == (not split)
    ok = ~np.isnan(z0)
    for t in range(4):
        z, _, _ = run([spec], [params], x, 4, str(t + 1), monkeypatch)
        assert np.array_equal(np.isnan(z), np.isnan(z0)), t
        assert np.array_equal(z[ok].view(np.uint32), z0[ok].view(np.uint32)), t


@pytest.mark.parametrize("n, hw, c", [(1, (1, 1), 512), (3, (1, 3), 520), (2, (7, 7), 2048), (5, (8, 8), 648),
                                      (2, (5, 13), 512)])
def test_small_mean_keeps_its_order(n, hw, c):
    """The mean of few images over at most 64 positions (65: the general kernel): four slices of
    positions summed in order and folded in order, in fp32, bit for bit."""
    from paper_1804_06087_amd.binding import global_avgpool_nhwc_bf16
    rng = np.random.default_rng(c + n)
    x = wl.gen.round_bf16_rne_f32(rng.standard_normal((n,) + hw + (c,), dtype=np.float32))
    xt = torch.from_numpy(x).to(DEV).bfloat16()
    y = torch.empty((n, c), dtype=torch.bfloat16, device=DEV)
    global_avgpool_nhwc_bf16(xt, y)
    rows = x.reshape(n, -1, c)
    total = None
    for s in range(4):
        acc = np.zeros((n, c), np.float32)
        for p in range(s, rows.shape[1], 4):
            acc = acc + rows[:, p]
        total = acc if total is None else total + acc
    ref = wl.gen.round_bf16_rne_f32(total * (np.float32(1.0) / np.float32(rows.shape[1])))
    assert np.array_equal(y.float().cpu().numpy(), ref)
