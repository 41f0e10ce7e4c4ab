"""The fused float32 layer on infinities, NaNs and numbers at the end of the float32 range, in weights, parameters,
features and embedding: infinite, NaN and finite results stand where the plain fp32 kernels have them."""
import numpy as np
import pytest
import torch

import ffsynth
import paper_2301_08739_amd as ff
from gpu_util import DEV, geoms, gpu_flatten, to_dev_feats, to_host

pytestmark = pytest.mark.gpu

HEADS = {64: 4, 128: 8, 256: 8}
INF, NAN, BIG = np.float32(np.inf), np.float32(np.nan), np.float32(3.4e38)   # BIG is finite and rounds to inf in bfloat16


def _put(p, key, at, value):
    p[key] = np.array(p[key], dtype=np.float32)
    p[key][at] = value


def _variants(C):
    """name -> what to do to (params, features, embedding)"""
    def weights(key, at, value):
        return lambda p, x, e: _put(p, key, at, value)

    def idle_unit(p, x, e):                  # hidden unit 5 is exactly zero, its weights at the end of the range
        _put(p, "w1", 5, 0)
        _put(p, "b1", 5, 0)
        _put(p, "w2", (slice(None), 5), BIG)

    def idle_feature(p, x, e):               # so is feature 2 of both LayerNorm outputs
        for key in ("ln1_g", "ln1_b", "ln2_g", "ln2_b"):
            _put(p, key, 2, 0)
        e[:, 2] = 0
        for key in ("w_qkv", "w1"):
            _put(p, key, (slice(None, None, 3), 2), BIG)

    def idle_columns(p, x, e):               # the embedding is at the end of the range where no projection looks
        _put(p, "w_qkv", (slice(None), 3), 0)
        e[::97, 3] = BIG

    def rows(which, value):
        def f(p, x, e):
            (x if which == "x" else e)[::97, 3] = value
        return f
    v = {"w1 inf": weights("w1", (9, 4), INF), "w1 -inf": weights("w1", (C + 3, 1), -INF), "w1 nan": weights("w1", (9, 4), NAN),
         "w1 big": weights("w1", (2, 7), BIG), "w2 inf": weights("w2", (3, 11), INF), "w2 nan": weights("w2", (3, 11), NAN),
         "w2 big": weights("w2", (3, 11), -BIG), "w2 big, unit idle": idle_unit, "w big, feature idle": idle_feature, "w_o inf": weights("w_o", (8, 2), INF),
         "w_o big": weights("w_o", (8, 2), BIG), "b1 inf": weights("b1", 7, INF), "b1 -inf": weights("b1", 7, -INF),
         "b1 big": weights("b1", 7, BIG), "b2 inf": weights("b2", 6, INF), "b2 nan": weights("b2", 6, NAN),
         "b_o inf": weights("b_o", 6, INF), "ln1_g inf": weights("ln1_g", 3, INF), "ln1_b nan": weights("ln1_b", 3, NAN),
         "ln2_g inf": weights("ln2_g", 3, -INF), "x inf": rows("x", INF), "x nan": rows("x", NAN), "x big": rows("x", BIG),
         "x 1e30": rows("x", np.float32(1e30)), "e inf": rows("e", INF), "e nan": rows("e", NAN),
         "e big, columns idle": idle_columns}
    for name, row in (("q", 1), ("k", C + 1), ("v", 2 * C + 1)):
        v[f"w_{name} inf"] = weights("w_qkv", (row, 2), INF)
        v[f"b_{name} inf"] = weights("b_qkv", row, INF)
        v[f"b_{name} nan"] = weights("b_qkv", row, NAN)
    return v


def _same(got, want, label):
    for what in (np.isnan, np.isposinf, np.isneginf):
        a, b = what(got), what(want)
        assert np.array_equal(a, b), f"{label}: {what.__name__} at {a.sum()} places, plain kernels at {b.sum()}"
    # finite results: float32 sums of the same terms in different order.  A weight or bias of 3.4e38 multiplies numbers
    # that are off by their own roundings, or is lost against others of that size: the terms are what counts there.
    f = np.isfinite(want)
    size = np.where(f, np.abs(want), 0).max(axis=1, keepdims=True) + 1
    if label.endswith(" big"):
        size = np.full_like(size, BIG)
    err = np.where(f, np.abs(np.where(f, got, 0) - np.where(f, want, 0)) / size, 0)
    assert err.max() <= 1e-5, f"{label}: {(err > 1e-5).sum()} of {f.sum()} finite results off, by up to {err.max():.2e} of the row"


@pytest.mark.parametrize("C,G", [(64, 20), (64, 64), (64, 100), (128, 31), (128, 64), (128, 69), (128, 100), (256, 20), (256, 64)])
def test_nonfinite_values_as_in_the_plain_kernels(cfg, C, G):
    c = cfg(2, 1)
    n = 1003 if G <= 64 else 9001            # (enough for the fused kernel)
    coords = np.ascontiguousarray(c["coords"][:n])
    dev = gpu_flatten(coords, geoms(c)[0], 0, 1, G, want_keys=False)[4]
    wrong = []
    for name, change in _variants(C).items():
        rng = np.random.default_rng(C + G)
        p = dict(ffsynth.layer_params(C, 2 * C, HEADS[C], seed=3))
        x, e = (rng.standard_normal((n, C)).astype(np.float32) for _ in range(2))
        change(p, x, e)
        lw = ff.LayerWeights(p, ff.FF_F32, DEV)
        for pe in ((e,) if name[0] == "e" else (None, e) if name[0] in "xw" else (None,)):
            got, want = (to_host(ff.ff_group_attention(
                to_dev_feats(x, ff.FF_F32), dev[0], dev[1], dev[2], -(-n // G), lw, G, ff.FF_F32, flags,
                pos_embed=None if pe is None else to_dev_feats(pe, ff.FF_F32))) for flags in (0, ff.FF_FLAG_FORCE_GENERIC))
            try:
                _same(got, want, name)
            except AssertionError as err:
                wrong.append(str(err).split("\n")[0] + (" (embedding)" if pe is not None else ""))
    print(*wrong, sep="\n")
    assert not wrong, len(wrong)


def test_nonfinite_values_through_a_block(cfg):
    """Features handed on in sorted order, rows starting over in some workgroups only."""
    c = cfg(2, 1)
    n, C, G = 4001, 128, 64
    coords = np.ascontiguousarray(c["coords"][:n])
    g = geoms(c)[0]
    params = [dict(ffsynth.layer_params(C, 2 * C, HEADS[C], seed=30 + i)) for i in range(3)]
    x = np.random.default_rng(1).standard_normal((n, C)).astype(np.float32)
    x[11, 5] = INF
    _put(params[2], "b2", 6, INF)
    layers = [ff.LayerWeights(p, ff.FF_F32, DEV) for p in params]
    ct = torch.from_numpy(coords).to(DEV)
    got = to_host(ff.ff_fwa_block(ct, g, G, layers, ff.FF_F32, to_dev_feats(x, ff.FF_F32)))
    cur = to_dev_feats(x, ff.FF_F32)
    for i, lw in enumerate(layers):
        perm, goff, ng, _ = ff.ff_flatten(ct, g, i % 2, i // 2 % 2, G)
        cur = ff.ff_group_attention(cur, perm, goff, ng, -(-n // G), lw, G, ff.FF_F32, ff.FF_FLAG_FORCE_GENERIC)
    want = to_host(cur)
    assert 0 < np.isnan(want).any(axis=1).sum() < n and np.isposinf(want[:, 6]).any()
    _same(got, want, "block")
