"""The patch kernel gives the tiled GEMM's bits.

RAFIKI_PATCH_TILES=1..3 runs every layer the kernel takes with one of its tiles (consecutive
pixels, rectangles 16 or 32 wide), 0 none.  The probes end in an average pool and a random FC, so
equal logits mean equal outputs.  Sizes: maps that rectangles do not divide, tiles across images,
the widest map of the consecutive form and one past it, one and several channel blocks and
channel tiles, 128-channel layers (two pixel groups), the fused max-pool.
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

# (c_in, c_out, (H, W), n, pool, relu, tiles that take it); at least 16,384 output positions x
# (c_out / 128) or under 12 K tiles, so that K is not split
CASES = {
    "flat_widest": (64, 256, (20, 63), 5, False, True, (1, 2, 3)),
    "one_past_widest": (64, 256, (18, 64), 4, False, True, (2, 3)),
    "odd_map_many_blocks": (256, 256, (13, 29), 27, False, True, (1, 2, 3)),
    "two_channel_tiles_no_relu": (128, 512, (9, 11), 50, False, False, (1, 2, 3)),
    "pool_ragged": (128, 256, (22, 38), 13, True, True, (2, 3)),
    "c128": (128, 128, (19, 37), 24, False, True, (2,)),
    "c128_pool": (64, 128, (34, 50), 3, True, False, (2,)),
    "tiny_map": (64, 256, (2, 2), 9, True, True, (2, 3)),
}


def run(spec, params, x, n, mode, monkeypatch):
    monkeypatch.setenv("RAFIKI_PATCH_TILES", mode)
    with Ensemble([spec], [params], precision="bf16", max_batch=n) as ens:
        out = torch.full((n, spec.n_classes), float("nan"), dtype=torch.float32, device=DEV)
        ens.model_logits(0, x, n, out)
        torch.cuda.synchronize()
        z = out.cpu().numpy().copy()
        ens.trace(True)
        ens.model_logits(0, x, n, out)
        recs = [r for r in ens.trace_read() if r["kind"] == "conv_mfma"]
    return z, recs


@pytest.mark.parametrize("name", sorted(CASES))
def test_patch_bitwise(name, monkeypatch):
    ci, co, hw, n, pool, relu, tiles = CASES[name]
    L = [Layer(op=CONV2D, input=-1, c_in=8, c_out=ci, kh=1, kw=1, stride=1, pad=0, relu=True, bn=True),
         Layer(op=CONV2D, input=0, c_in=ci, c_out=co, kh=3, kw=3, stride=1, pad=1, relu=relu, bn=True)]
    if pool:
        L.append(Layer(op=MAXPOOL2D, input=1, c_in=co, c_out=co, kh=2, kw=2, stride=2))
    L.append(Layer(op=GLOBAL_AVGPOOL, input=len(L) - 1, c_in=co, c_out=co))
    L.append(Layer(op=FC, input=len(L) - 1, c_in=co, c_out=10, bias=True))
    spec = ModelSpec("patch", L, 10, (8,) + hw)
    params = wl.gen_params(spec, 3, True, "random")
    batch = wl.gen_images(n, spec.input_shape, "normal", True, seed=2)
    x = torch.from_numpy(batch).to(DEV)
    z0, r0 = run(spec, params, x, n, "0", monkeypatch)
    assert np.isfinite(z0).all() and all(r["splits"] == 1 for r in r0[:2])
    first = len(tile_configs()) + 8
    for t in (1, 2, 3):
        z, recs = run(spec, params, x, n, str(t), monkeypatch)
        assert any(r["tile_cfg"] == first + t - 1 for r in recs) == (t in tiles), t
        assert np.array_equal(z.view(np.uint32), z0.view(np.uint32)), t
    ref = oracle.run_model(spec, params, batch[:2], act="bf16")
    assert np.abs(z0[:2] - ref).max() <= 1e-2 * np.abs(ref).max()
