"""Fused bottleneck launches are bitwise the layers run apart.

Each probe is a chain of bottleneck blocks that holds every form of the fused unit: 3x3 +
expansion + next reduction, expansion + next reduction (after a stride-2 3x3, which stays
apart) and 3x3 + expansion (the last block).  RAFIKI_FUSED_BLOCKS=64 / 32 run every unit fused
with that many pixels per workgroup, 0 runs every layer apart; a global average pool and a
random FC carry any changed element to the logits.  Sizes cover ragged tiles, tiles across
images, odd and non-square maps, the widest map a patch fits, one image, K split in partial
sums (small batches) and not (the largest).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads import Layer, ModelSpec, CONV2D, GLOBAL_AVGPOOL, FC
from paper_1804_06087_amd import Ensemble
from paper_1804_06087_amd.binding import tile_configs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def conv(i, c_in, c_out, k, s=1, relu=True, res=-1):
    return Layer(op=CONV2D, input=i, input2=res, c_in=c_in, c_out=c_out, kh=k, kw=k, stride=s, pad=k // 2,
                 relu=relu, bn=True)


def chain(mid, hw):
    """y0 -> block 1 (3x3 stride 1) -> block 2 (3x3 stride 2, projection) -> block 3, last."""
    L = [conv(-1, 8, 4 * mid, 1)]                            # 0: y0
    L.append(conv(0, 4 * mid, mid, 1))                       # 1: reduction
    L.append(conv(1, mid, mid, 3))                           # 2 \
    L.append(conv(2, mid, 4 * mid, 1, res=0))                # 3  > one unit
    L.append(conv(3, 4 * mid, mid, 1))                       # 4 /
    L.append(conv(4, mid, mid, 3, s=2))                      # 5: stride 2, apart
    L.append(conv(3, 4 * mid, 4 * mid, 1, s=2, relu=False))  # 6: projection
    L.append(conv(5, mid, 4 * mid, 1, res=6))                # 7 \  one unit
    L.append(conv(7, 4 * mid, mid, 1))                       # 8 /
    L.append(conv(8, mid, mid, 3))                           # 9 \  one unit
    L.append(conv(9, mid, 4 * mid, 1, res=7))                # 10 /
    L.append(Layer(op=GLOBAL_AVGPOOL, input=10, c_in=4 * mid, c_out=4 * mid))
    L.append(Layer(op=FC, input=11, c_in=4 * mid, c_out=24, bias=True))
    return ModelSpec(f"chain{mid}", L, 24, (8,) + hw)


def logits(spec, params, x, n, mode, monkeypatch):
    monkeypatch.setenv("RAFIKI_FUSED_BLOCKS", mode)
    with Ensemble([spec], [params], precision="bf16", max_batch=n) as ens:
        out = torch.empty((n, spec.n_classes), dtype=torch.float32, device=DEV)
        for _ in range(2):
            out.fill_(float("nan"))
            ens.model_logits(0, x, n, out)
        torch.cuda.synchronize()
        z = out.cpu().numpy().copy()
        ens.trace(True)
        ens.model_logits(0, x, n, out)
        recs = ens.trace_read()
        ens.trace(False)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), z.view(np.uint32))
    return z, recs


@pytest.mark.parametrize("mid, hw, n", [
    (64, (6, 56), 1), (64, (5, 7), 3), (64, (9, 56), 17),
    (128, (3, 28), 1), (128, (7, 9), 5), (128, (28, 28), 11),
    (256, (14, 14), 1), (256, (5, 3), 7), (256, (7, 14), 27), (256, (14, 14), 42),
])
def test_fused_blocks_bitwise(mid, hw, n, monkeypatch):
    spec = chain(mid, hw)
    params = wl.gen_params(spec, 5, True, "random")
    batch = wl.gen_images(n, spec.input_shape, "normal", True, seed=mid + n)
    x = torch.from_numpy(batch).to(DEV)
    apart, r0 = logits(spec, params, x, n, "0", monkeypatch)
    assert np.isfinite(apart).all()
    fused_ids = {"64": len(tile_configs()) + 1, "32": len(tile_configs()) + 2}
    assert not any(r["tile_cfg"] in fused_ids.values() for r in r0)
    for mode, tile in fused_ids.items():
        z, recs = logits(spec, params, x, n, mode, monkeypatch)
        assert sorted(r["layer"] for r in recs if r["tile_cfg"] == tile) == [2, 3, 4, 7, 8, 9, 10]
        assert sum(r["flops"] for r in recs) == pytest.approx(sum(r["flops"] for r in r0))
        assert np.array_equal(z.view(np.uint32), apart.view(np.uint32)), mode
    if n * hw[0] * hw[1] <= 1024:
        ref = oracle.run_model(spec, params, batch, act="bf16")
        assert np.abs(apart - ref).max() <= 2e-2 * np.abs(ref).max()


def test_forced_without_tuning(monkeypatch):
    """RAFIKI_FUSED_BLOCKS=32 / 64 fuse every unit with RAFIKI_AUTOTUNE=0 as well; without it, or with
    any other value, an untuned handle runs the layers apart.  A tuned one takes other values as 1."""
    spec = chain(128, (7, 9))
    params = wl.gen_params(spec, 5, True, "random")
    x = torch.from_numpy(wl.gen_images(3, spec.input_shape, "normal", True, seed=2)).to(DEV)
    base = len(tile_configs())
    monkeypatch.setenv("RAFIKI_AUTOTUNE", "0")
    apart, _ = logits(spec, params, x, 3, "0", monkeypatch)
    for mode, tile in (("64", base + 1), ("32", base + 2), ("1", None), ("16", None), ("128", None)):
        z, recs = logits(spec, params, x, 3, mode, monkeypatch)
        fused = sorted(r["layer"] for r in recs if r["tile_cfg"] in (base + 1, base + 2))
        assert fused == ([2, 3, 4, 7, 8, 9, 10] if tile else []), mode
        assert all(r["tile_cfg"] == tile for r in recs if r["layer"] in fused)
        assert np.array_equal(z.view(np.uint32), apart.view(np.uint32)), mode
    monkeypatch.delenv("RAFIKI_AUTOTUNE")
    z, _ = logits(spec, params, x, 3, "128", monkeypatch)
    assert np.array_equal(z.view(np.uint32), apart.view(np.uint32))


def test_wider_maps_stay_apart(monkeypatch):
    """A map wider than the patch allows keeps its 3x3 apart; expansion and reduction still fuse."""
    spec = chain(256, (3, 30))
    params = wl.gen_params(spec, 6, True, "random")
    batch = wl.gen_images(2, spec.input_shape, "normal", True, seed=4)
    x = torch.from_numpy(batch).to(DEV)
    apart, _ = logits(spec, params, x, 2, "0", monkeypatch)
    z, recs = logits(spec, params, x, 2, "64", monkeypatch)
    tile = len(tile_configs()) + 1
    assert sorted(r["layer"] for r in recs if r["tile_cfg"] == tile) == [3, 4, 7, 8]
    assert np.array_equal(z.view(np.uint32), apart.view(np.uint32))


@pytest.mark.parametrize("mid, with_3x3", [(128, True), (256, False), (256, True), (64, True)])
def test_fused_blocks_nonfinite(mid, with_3x3, monkeypatch):
    """A positive NaN (of a layer's shift; arithmetic gives negative ones here) is kept by the ReLU of
    an unsplit layer, an integer maximum, and made 0 by that of a split layer's reduce launch: a
    unit does as the layers apart do.  The request holds an infinity and a NaN besides."""
    L = [conv(-1, 8, 4 * mid, 1),                   # 0: residual
         conv(-1, 8, mid, 1)]                       # 1: the unit's input
    if with_3x3:
        L.append(conv(1, mid, mid, 3))
    L.append(conv(len(L) - 1, mid, 4 * mid, 1, res=0))
    L.append(conv(len(L) - 1, 4 * mid, mid, 1))
    L.append(Layer(op=GLOBAL_AVGPOOL, input=len(L) - 1, c_in=mid, c_out=mid))
    L.append(Layer(op=FC, input=len(L) - 1, c_in=mid, c_out=24, bias=True))
    spec = ModelSpec("nonfinite", L, 24, (8, 6, 7))
    params = wl.gen_params(spec, 7, True, "random")
    P = params.layers
    batch = wl.gen_images(3, spec.input_shape, "normal", True, seed=mid).copy()
    batch[1, 3, 0, 0], batch[2, 3, 0, 0] = np.inf, np.nan
    x = torch.from_numpy(batch).to(DEV)
    for at in range(2, len(L) - 2):     # each of the unit's layers in turn
        P[at].bn_beta[5], beta = np.nan, P[at].bn_beta[5]
        apart, r0 = logits(spec, params, x, 3, "0", monkeypatch)
        splits = {r["layer"]: r["splits"] for r in r0 if r["kind"] == "conv_mfma"}
        # (a product with a NaN is a negative one: only the last layer's can reach the logits)
        assert np.isnan(apart[0]).any() == (at == len(L) - 3 and splits[at] == 1)
        for mode in ("64", "32"):
            z, _ = logits(spec, params, x, 3, mode, monkeypatch)
            ok = ~np.isnan(apart)
            assert np.array_equal(~np.isnan(z), ok), (at, mode)
            assert np.array_equal(z[ok].view(np.uint32), apart[ok].view(np.uint32)), (at, mode)
        P[at].bn_beta[5] = beta
