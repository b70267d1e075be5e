"""Fused conv1d branches run from their table of per-tap products.

A vocabulary of at least 1024 rows and 192 channels takes the tap-table path when the
handle's batch allows the table; the features must then be the oracle's to one bf16 step and
agree with the separate convolutions (RAFIKI_FUSE_BRANCHES=0) to the same bound, whether one
workgroup takes a request or several share it.  Cases cover filter counts that are no
multiple of 4, 1 to 8 taps, a branch as wide as the sequence, batch-norm with negative
scales, no ReLU, ids outside the table and a grouped launch of two members.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads import Layer, ModelSpec, FC, EMBEDDING, CONV1D_MAXTIME, CONCAT
from paper_1804_06087_amd import Ensemble, RafikiError, RAFIKI_ERR_NOMEM

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def probe(vocab, dim, seq_len, filters, widths, relu=True, bn=False, seed=5):
    """The branches, their concatenation and an identity FC: the logits are the features."""
    L = [Layer(op=EMBEDDING, input=-1, c_in=vocab, c_out=dim)]
    for f, w in zip(filters, widths):
        L.append(Layer(op=CONV1D_MAXTIME, input=0, c_in=dim, c_out=f, kh=1, kw=w, relu=relu, bias=True, bn=bn))
    x, c = 1, filters[0]
    for i, f in enumerate(filters[1:]):
        L.append(Layer(op=CONCAT, input=x, input2=2 + i, c_in=c, c_out=c + f))
        x, c = len(L) - 1, c + f
    L.append(Layer(op=FC, input=x, c_in=c, c_out=c, bias=True))
    spec = ModelSpec("taps", L, c, (seq_len,), vocab=vocab)
    params = wl.gen_params(spec, seed, True, "random")
    params.layers[-1].weight = np.eye(c, dtype=np.float32)
    rng = np.random.default_rng(seed)
    for p, lay in zip(params.layers, L):
        if lay.op == CONV1D_MAXTIME:
            p.bias = rng.normal(0, 0.2, lay.c_out).astype(np.float32)
            if bn:
                p.bn_gamma = rng.normal(0, 1, lay.c_out).astype(np.float32)
    return spec, params


def run(specs, params, tok, max_batch):
    n = tok.shape[0]
    with Ensemble(specs, params, precision="bf16", max_batch=max_batch) as ens:
        x = torch.from_numpy(tok).to(DEV)
        out = torch.full((n, specs[0].n_classes), float("nan"), dtype=torch.float32, device=DEV)
        zs = []
        for m in range(len(specs)):
            for _ in range(2):      # the maxima's slots are reset as they are read
                ens.model_logits(m, x, n, out)
            torch.cuda.synchronize()
            zs.append(out.cpu().numpy().copy())
        ens.trace(True)
        ens.model_logits(0, x, n, out)
        kinds = [r["kind"] for r in ens.trace_read()]
        ens.trace(False)
        probs = torch.empty((n, specs[0].n_classes), dtype=torch.float32, device=DEV)
        labels = torch.empty((n,), dtype=torch.int32, device=DEV)
        both = []
        for call in (ens.infer, ens.infer_noalloc):
            call(x, n, (1 << len(specs)) - 1, probs, labels)
            torch.cuda.synchronize()
            both.append(probs.cpu().numpy().copy())
        assert np.array_equal(both[0], both[1])
    return zs, kinds, both[0]


def check(z, ref):
    """Within one bf16 step of the oracle's features, few of them different (fp32 against
    fp64 sums may round the other way)."""
    ref = np.asarray(ref, np.float64)
    d = np.abs(z - ref)
    assert (d <= np.abs(ref) * 2.0 ** -7 + 1e-6 * np.abs(ref).max()).all()
    assert (d > 0).mean() < 0.02


CASES = [
    # (n, max_batch, probe): one part per request at n >= 512, several below
    (3, 64, dict(vocab=2000, dim=300, seq_len=256, filters=(100, 100, 100), widths=(3, 4, 5))),
    (1, 64, dict(vocab=1024, dim=192, seq_len=40, filters=(5, 3), widths=(1, 8))),
    (512, 512, dict(vocab=1500, dim=200, seq_len=17, filters=(6, 33, 10), widths=(2, 7, 17 - 9))),
    (70, 70, dict(vocab=1100, dim=256, seq_len=8, filters=(8, 4), widths=(8, 2), relu=False)),
    (9, 64, dict(vocab=1300, dim=200, seq_len=61, filters=(30, 22), widths=(3, 6), relu=False, bn=True)),
    (600, 600, dict(vocab=1300, dim=200, seq_len=33, filters=(31,) * 2, widths=(5, 6), bn=True)),
]


@pytest.mark.parametrize("n, max_batch, case", CASES)
def test_tap_table_matches_oracle(n, max_batch, case, monkeypatch):
    spec, params = probe(**case)
    tok = wl.gen_tokens(n, case["seq_len"], case["vocab"], seed=n)
    zs, kinds, _ = run([spec], [params], tok, max_batch)
    assert kinds.count("tap_table") == 1 and "embed" not in kinds
    assert kinds.count("pool") == (0 if n >= 512 or case["seq_len"] < 32 else 1)
    rows = np.linspace(0, n - 1, min(n, 12)).astype(int)
    if not case.get("bn"):     # the oracle's conv1d has no batch-norm
        check(zs[0][rows], oracle.run_model(spec, params, tok[rows], act="bf16"))
    monkeypatch.setenv("RAFIKI_FUSE_BRANCHES", "0")
    apart, k2, _ = run([spec], [params], tok, max_batch)
    assert "tap_table" not in k2
    check(zs[0], apart[0])


def test_tap_table_invalid_ids_and_group():
    """Ids outside [0, vocab) add zero products; two members of one launch each match their
    own oracle."""
    case = dict(vocab=1200, dim=200, seq_len=50, filters=(12, 20), widths=(2, 5))
    models = [probe(seed=s, **case) for s in (5, 6)]
    tok = wl.gen_tokens(20, 50, 1200, seed=8)
    rng = np.random.default_rng(9)
    bad = rng.random(tok.shape) < 0.1
    tok[bad] = rng.choice(np.array([-1, 1200, 1207, 2**31 - 1, -2**31]), size=int(bad.sum())).astype(np.int32)
    zs, kinds, probs = run([m[0] for m in models], [m[1] for m in models], tok, 64)
    assert "tap_table" in kinds
    import copy
    soft = []
    for (spec, params), z in zip(models, zs):
        p2 = copy.deepcopy(params)
        p2.layers[0].weight = np.vstack([params.layers[0].weight, np.zeros((1, 200), np.float32)])
        check(z, oracle.run_model(spec, p2, np.where(bad, 1200, tok), act="bf16"))
        e = np.exp(z.astype(np.float64) - z.max(1, keepdims=True))
        soft.append(e / e.sum(1, keepdims=True))
    assert np.abs(probs - sum(soft) / 2).max() <= 1e-6     # the grouped launch: fp32 softmax of the same logits


@pytest.mark.parametrize("where", ["bias", "weight", "embedding"])
def test_nonfinite_parameters_keep_the_gemm(where, monkeypatch):
    """The table's maximum would pass a NaN over where the unsplit GEMM's ReLU keeps it."""
    spec, params = probe(vocab=1100, dim=200, seq_len=20, filters=(10, 6), widths=(2, 5))
    if where == "embedding":
        params.layers[0].weight[7, 3] = np.inf
    elif where == "weight":
        params.layers[1].weight.reshape(-1)[5] = np.nan
    else:
        params.layers[2].bias[3] = np.nan
    tok = wl.gen_tokens(64, 20, 1100, seed=3)
    out = []
    for mode in ("1", "0"):
        monkeypatch.setenv("RAFIKI_TAP_TABLE", mode)
        with Ensemble([spec], [params], precision="bf16", max_batch=64) as ens:
            x = torch.from_numpy(tok).to(DEV)
            z = torch.empty((64, spec.n_classes), dtype=torch.float32, device=DEV)
            ens.trace(True)
            ens.model_logits(0, x, 64, z)
            assert "tap_table" not in [r["kind"] for r in ens.trace_read()]
            ens.trace(False)
            out.append(z.cpu().numpy())
    assert np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32))


def test_small_vocabulary_and_small_handle_keep_the_gemm():
    for kw, mb in ((dict(vocab=1023, dim=300), 64), (dict(vocab=2000, dim=184), 64), (dict(vocab=30000, dim=192), 2)):
        spec, params = probe(seq_len=20, filters=(100, 100), widths=(3, 4), **kw)
        _, kinds, _ = run([spec], [params], wl.gen_tokens(2, 20, kw["vocab"], seed=1), mb)
        assert "tap_table" not in kinds, kw


def test_tap_table_switch(monkeypatch):
    """RAFIKI_TAP_TABLE fixes the choice that otherwise depends on max_batch: 1 builds the table for
    a handle of two requests, and the features are those of a larger handle's table bit for bit."""
    case = dict(vocab=30000, dim=192, seq_len=20, filters=(100, 100), widths=(3, 4))
    spec, params = probe(**case)
    tok = wl.gen_tokens(2, 20, 30000, seed=1)
    out = {}
    for mode, mb in (("1", 2), ("1", 64), ("0", 64)):
        monkeypatch.setenv("RAFIKI_TAP_TABLE", mode)
        zs, kinds, _ = run([spec], [params], tok, mb)
        assert ("tap_table" in kinds) == (mode == "1")
        out[mode, mb] = zs[0]
    assert np.array_equal(out["1", 2].view(np.uint32), out["1", 64].view(np.uint32))
    check(out["1", 2], out["0", 64])


def test_tables_never_cost_a_handle(monkeypatch):
    """A handle that fits in memory without tables is created whatever the tables would take: under
    every cap from the smallest that the GEMM alone needs, create succeeds."""
    # a table of 97 MB, more than the arena and workspace of a model without one
    case = dict(vocab=20000, dim=200, seq_len=256, filters=(100, 100, 100), widths=(3, 4, 5))
    models = [probe(seed=s, **case) for s in (5, 6)]
    specs, params = [m[0] for m in models], [m[1] for m in models]
    tok = wl.gen_tokens(3, 256, 20000, seed=1)

    def handle(cap, mode):
        monkeypatch.setenv("RAFIKI_DEVICE_MB", str(cap))
        if mode is None:
            monkeypatch.delenv("RAFIKI_TAP_TABLE", raising=False)
        else:
            monkeypatch.setenv("RAFIKI_TAP_TABLE", mode)
        return run(specs, params, tok, 64)

    need = 8
    while True:
        try:
            ref, kinds, _ = handle(need, "0")
            break
        except RafikiError as e:
            assert e.code == RAFIKI_ERR_NOMEM
            need += 2
            assert need < 400
    assert 8 < need < 140 and "tap_table" not in kinds
    seen = set()
    for cap in range(need, 260, 6):
        zs, kinds, _ = handle(cap, None)
        seen.add("tap_table" in kinds)
        for z, r in zip(zs, ref):
            check(z, r)
    assert seen == {False, True}
    with pytest.raises(RafikiError) as ei:
        handle(8, "1")
    assert ei.value.code == RAFIKI_ERR_NOMEM
