"""The fused 16-bit layer of 128 and 256 features (wavefronts that cut the features): at both sides of every block and half
block of group members, two frames (group starts that are no multiples of G), short last groups, and scores beyond what
2^score can stand for."""
import numpy as np
import pytest
import torch

import ffsynth
import oracle
import paper_2301_08739_amd as ff
from gpu_util import DEV, gpu_flatten, to_dev_feats, to_host

pytestmark = pytest.mark.gpu

HEADS = {64: 4, 128: 8, 256: 8}


@pytest.mark.parametrize("dt", [ff.FF_BF16, ff.FF_F16])
@pytest.mark.parametrize("C", [128, 256])
@pytest.mark.parametrize("G", [2, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113, 128])
def test_group_sizes(cfg, C, G, dt):
    n, bar = 3 * G + 101, 2e-2 if dt == ff.FF_BF16 else 2.5e-3
    c = cfg(2, 1)
    coords = c["coords"][:n].copy()
    coords[:, 0] = np.arange(n) % 3 == 0
    g = ff.Geometry(2, c["grid"], c["grid"], c["window"], c["window"])
    perm, off, ng, _, dev = gpu_flatten(coords, g, 0, 1, G, want_keys=False)
    rng = np.random.default_rng(C + G)
    x = to_dev_feats(rng.standard_normal((n, C)), dt)
    e = to_dev_feats(0.5 * rng.standard_normal((n, C)), dt)
    # as the layer holds them: the bar is for what the layer does to these numbers
    p = {k: to_host(to_dev_feats(v, dt)).astype(np.float32) if isinstance(v, np.ndarray) else v
         for k, v in ffsynth.layer_params(C, 2 * C, HEADS[C], seed=23).items()}
    # The probabilities of a row average the rounding errors of G value rows; those of the row's own LayerNorm output stay:
    # two independent errors, the first falling with sqrt(G), which the bar has room for from sixteen rows on.
    bar *= (1 + 1 / G) ** 0.5 if G < 16 else 1.0
    lw = ff.LayerWeights(p, dt, DEV)
    rounded = lambda t: to_host(t).astype(np.float32)
    for embed in (None, e):
        kw = {} if embed is None else dict(pos_embed=rounded(embed))
        want = oracle.layer(rounded(x), perm, off, p, **kw)
        wide = ff.ff_group_attention(x, dev[0], dev[1], dev[2], ng + 1, lw, G, dt, ff.FF_FLAG_OUT_F32, pos_embed=embed)
        narrow = ff.ff_group_attention(x, dev[0], dev[1], dev[2], ng + 1, lw, G, dt, pos_embed=embed)
        assert np.abs(to_host(wide) - want).max() <= bar
        assert torch.equal(wide.to(narrow.dtype), narrow)


@pytest.mark.parametrize("dt", [ff.FF_BF16, ff.FF_F16])
@pytest.mark.parametrize("C,G", [(128, 64), (128, 69), (256, 48)])
@pytest.mark.parametrize("score", [-300.0, 300.0])
def test_scores_beyond_the_exponents(C, G, dt, score):
    """All members of a group alike: every score of a row is the same number, so that the attention is the value row
    whatever the score is, also where 2^score is zero or infinite: the largest score has to go first."""
    n, d = 2 * G + 5, C // HEADS[C]
    rng = np.random.default_rng(3)
    p = ffsynth.layer_params(C, 2 * C, HEADS[C], seed=29)
    row = rng.standard_normal(C)
    x = to_dev_feats(np.repeat(row[None], n, 0), dt)
    z = (to_host(x)[0] - to_host(x)[0].mean()) / to_host(x)[0].std()
    # keys k = w z with k . k = d per head (first feature of the head alone), queries from the bias: q . k / sqrt(d) = score
    w = np.zeros((3 * C, C)); b = np.zeros(3 * C)
    for h in range(HEADS[C]):
        w[C + h * d] = z / C
        b[h * d] = score * np.sqrt(d)
    p = dict(p)
    half = lambda a: to_host(to_dev_feats(a, dt))
    p["w_qkv"] = half(np.concatenate([w[:2 * C], np.asarray(p["w_qkv"])[2 * C:]])).astype(np.float32)
    p["b_qkv"] = half(np.concatenate([b[:2 * C], np.asarray(p["b_qkv"])[2 * C:]])).astype(np.float32)
    p["ln1_g"], p["ln1_b"] = np.ones(C, np.float32), np.zeros(C, np.float32)
    lw = ff.LayerWeights(p, dt, DEV)
    off = np.array([0, G, 2 * G, n], np.int32)
    perm = np.arange(n, dtype=np.int32)
    dev = [torch.from_numpy(a).to(DEV) for a in (perm, off, np.array([3], np.int32))]
    got = to_host(ff.ff_group_attention(x, dev[0], dev[1], dev[2], 3, lw, G, dt, ff.FF_FLAG_OUT_F32))
    want = oracle.layer(to_host(x).astype(np.float32), perm, off, p)
    assert np.isfinite(got).all()
    # one value row reaches the output projection as it is (no averaging over keys): sqrt(2) of the bar, as for groups of one
    assert np.abs(got - want).max() <= (2e-2 if dt == ff.FF_BF16 else 2.5e-3) * 2 ** 0.5


@pytest.mark.parametrize("dt", [ff.FF_BF16, ff.FF_F16])
@pytest.mark.parametrize("C,G", [(64, 64), (128, 32), (128, 64), (128, 100), (256, 64), (256, 90)])
def test_infinite_output_biases(C, G, dt):
    """An infinite second FFN bias makes its feature infinite in every row, as in the plain kernels, and leaves the others as
    they are."""
    n = 2 * G + 5
    rng = np.random.default_rng(C)
    x = to_dev_feats(rng.standard_normal((n, C)), dt)
    dev = [torch.from_numpy(a).to(DEV) for a in (rng.permutation(n).astype(np.int32), np.array([0, G, 2 * G, n], np.int32),
                                                 np.array([3], np.int32))]
    run = lambda p, flags=0: to_host(ff.ff_group_attention(x, *dev, 3, ff.LayerWeights(p, dt, DEV), G, dt, ff.FF_FLAG_OUT_F32 | flags))
    p = dict(ffsynth.layer_params(C, 2 * C, HEADS[C], seed=41))
    want = run(p)
    p["b2"] = np.array(p["b2"], np.float32)
    p["b2"][[3, C - 7]] = np.inf, -np.inf
    got = run(p)
    assert np.isposinf(got[:, 3]).all() and np.isneginf(got[:, C - 7]).all()
    others = np.delete(np.arange(C), [3, C - 7])
    assert np.array_equal(got[:, others], want[:, others])
    assert np.array_equal(np.isposinf(got), np.isposinf(run(p, ff.FF_FLAG_FORCE_GENERIC)))


@pytest.mark.parametrize("dt", [ff.FF_BF16, ff.FF_F16])
@pytest.mark.parametrize("C,whole", [(128, 4), (256, 6)])
@pytest.mark.parametrize("G", [65, 66, 72, 79, 80])
def test_last_sixteen_rows(C, whole, G, dt):
    """Groups of 65 to 80: the last sixteen rows on products of their own give the bits of whole blocks of 32, in full groups, a
    last group of any length (rows below, across and in the last sixteen), with infinite biases and with an embedding."""
    rng = np.random.default_rng(C + G)
    p = dict(ffsynth.layer_params(C, 2 * C, HEADS[C], seed=43))
    q = {k: np.array(p[k], np.float32) for k in ("b1", "b2")}
    q["b1"][[1, C + 17]], q["b2"][[2, C - 9]] = np.inf, (np.inf, -np.inf)
    for last in (1, 63, 64, 65, G):
        n = 3 * G + last
        x, e = (to_dev_feats(rng.standard_normal((n, C)), dt) for _ in range(2))
        dev = [torch.from_numpy(a).to(DEV) for a in (rng.permutation(n).astype(np.int32),
                                                     np.array([0, G, 2 * G, 3 * G, n], np.int32), np.array([4], np.int32))]
        for params in (p, dict(p, **q)):
            lw = ff.LayerWeights(params, dt, DEV)
            for embed in (None, e):
                for fl in (0, ff.FF_FLAG_OUT_F32):
                    got, want = (ff.ff_group_attention(x, *dev, 4, lw, G, dt, fl | ff.FF_FLAG_VARIANT(v), pos_embed=embed)
                                 for v in (0, whole))
                    assert torch.equal(got.view(torch.int32 if fl else torch.int16), want.view(torch.int32 if fl else torch.int16))


@pytest.mark.parametrize("dt", [ff.FF_BF16, ff.FF_F16])
@pytest.mark.parametrize("G", [33, 48, 64, 97, 112, 128])
@pytest.mark.parametrize("groups", [1, 2, 128, 129, 513, 640, 641])
def test_groups_split_between_two_workgroups(G, groups, dt):
    """Up to 128 groups beyond whole rounds of 512 go to two workgroups each, 128 features: the same bits as with a bound on the number
    of groups (empty ones behind the list) at which none does; a short last group with members in one half only and in both, dropped
    tails, float32 results, an embedding.  (Beyond 512 groups of up to 64 the form that splits is asked for.)"""
    C = 128
    form = ff.FF_FLAG_VARIANT(7) if G <= 64 and groups > 512 else 0
    gen = torch.Generator(device=DEV).manual_seed(G + groups)
    lw = ff.LayerWeights(ffsynth.layer_params(C, 2 * C, HEADS[C], seed=47), dt, DEV).pack()
    bits = lambda t: t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)
    bound = groups + (300 - groups) % 512
    for last in (G // 2 - 1, G - 1):
        n = (groups - 1) * G + last
        x, e = (torch.randn(n, C, device=DEV, generator=gen).to(torch.bfloat16 if dt == ff.FF_BF16 else torch.float16) for _ in range(2))
        perm = torch.randperm(n, device=DEV, generator=gen).to(torch.int32)
        for fl, embed, k in ((0, None, groups), (ff.FF_FLAG_OUT_F32, e, groups), (ff.FF_FLAG_TAIL_DROP, None, groups - 1)):
            off = torch.arange(0, bound + 1, device=DEV, dtype=torch.int32).mul_(G).clamp_(max=n)
            off[k:] = n
            num = torch.full((1,), k, device=DEV, dtype=torch.int32)
            got, want = (ff.ff_group_attention(x, perm, off, num, most, lw, G, dt, fl | form, pos_embed=embed) for most in (groups, bound))
            assert torch.equal(bits(got), bits(want)), (last, fl)


@pytest.mark.parametrize("dt", [ff.FF_BF16, ff.FF_F16])
@pytest.mark.parametrize("C,G", [(128, 20), (128, 40), (128, 64), (128, 69), (128, 100), (128, 128), (256, 64), (256, 100)])
@pytest.mark.parametrize("groups", [3, 100, 640])
def test_results_over_the_embedding(C, G, groups, dt):
    """A caller may let the results overwrite the embedding: a group's rows of both belong to one workgroup, which reads before it
    writes.  Groups that two workgroups share would not have that, so none are shared then."""
    gen = torch.Generator(device=DEV).manual_seed(G + groups)
    tdt = torch.bfloat16 if dt == ff.FF_BF16 else torch.float16
    n = groups * G - G // 3
    lw = ff.LayerWeights(ffsynth.layer_params(C, 2 * C, HEADS[C], seed=53), dt, DEV).pack()
    x, e = (torch.randn(n, C, device=DEV, generator=gen).to(tdt) for _ in range(2))
    perm = torch.randperm(n, device=DEV, generator=gen).to(torch.int32)
    off = torch.arange(groups + 1, device=DEV, dtype=torch.int32).mul_(G).clamp_(max=n)
    num = torch.full((1,), groups, device=DEV, dtype=torch.int32)
    want = ff.ff_group_attention(x, perm, off, num, groups, lw, G, dt, pos_embed=e)
    both = e.clone()
    got = ff.ff_group_attention(x, perm, off, num, groups, lw, G, dt, pos_embed=both, out=both)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
