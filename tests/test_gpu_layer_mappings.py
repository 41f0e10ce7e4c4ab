"""Mappings of the fused 16-bit layer: at 64 features with five and six wavefronts per group, with two workgroups on a compute
unit and with more groups per workgroup; at 128 and 256 features with more row blocks than a group needs, with the last of them
computed whole or by half, and with the registers of two or of three workgroups on a SIMD.  At the edges of the group sizes they
serve, two frames (group starts that are no multiples of G), short last groups, wavefronts beyond the last group, dropped tails and
positional embedding.  Against the oracle, and bit for bit against another mapping: a mapping only says which wavefront
computes a row, the operations on it and their order are the same."""
import numpy as np
import pytest
import torch

import ffsynth
import oracle
import paper_2301_08739_amd as ff
from gpu_util import DEV, gpu_flatten, to_dev_feats, to_host

pytestmark = pytest.mark.gpu

HEADS = {64: 4, 128: 8, 256: 8}
# (C, mapping, the other mapping, takes a positional embedding, group sizes)
CASES = [(128, 3, 9, True, (65, 80)), (128, 13, 9, True, (65, 80)), (128, 14, 9, True, (81, 96)),
         (128, 8, 9, False, (97, 128)), (128, 15, 10, True, (1, 32)),
         (64, 3, 1, True, (17, 32)), (64, 8, 2, True, (33, 64)), (64, 5, 4, True, (65, 80)), (64, 6, 4, True, (81, 96)),
         (64, 7, 4, True, (97, 128)), (256, 7, 4, False, (81, 96)), (256, 8, 2, False, (33, 64))]


@pytest.mark.parametrize("dt", [ff.FF_BF16, ff.FF_F16])
@pytest.mark.parametrize("C,mapping,other,embeds,sizes", CASES)
def test_mapping(cfg, C, mapping, other, embeds, sizes, dt):
    n, bar = 613, 2e-2 if dt == ff.FF_BF16 else 2.5e-3
    c = cfg(2, 1)
    coords = c["coords"][:n].copy()
    coords[:, 0] = np.arange(n) % 5 == 0                     # two frames of unequal size
    g = ff.Geometry(2, c["grid"], c["grid"], c["window"], c["window"])
    rng = np.random.default_rng(C + mapping)
    x = to_dev_feats(rng.standard_normal((n, C)), dt)
    e = to_dev_feats(0.5 * rng.standard_normal((n, C)), dt)
    p = ffsynth.layer_params(C, 2 * C, HEADS[C], seed=17)
    lw = ff.LayerWeights(p, dt, DEV)
    for G in sizes:
        print(f"C={C} mapping {mapping} G={G}", flush=True)
        perm, off, ng, _, dev = gpu_flatten(coords, g, 1, 1, G, want_keys=False)
        dperm, doff, dng, _ = ff.ff_flatten(torch.from_numpy(coords).to(DEV), g, 1, 1, G, ff.FF_TAIL_DROP)
        drop = (dperm, doff, dng)

        def run(m, flags=0, lists=dev, embed=None):
            return to_host(ff.ff_group_attention(x, lists[0], lists[1], lists[2], -(-n // G) + 2, lw, G, dt,
                                                 flags | ff.FF_FLAG_VARIANT(m), pos_embed=embed))

        wide = run(mapping, ff.FF_FLAG_OUT_F32)
        # With one key per row the value row reaches the output projection as it is, where a group's probabilities
        # average the rounding errors of V away: independent errors of two operands (V, and LN1's output before it) in
        # the place of one, a factor of sqrt(2).
        assert np.abs(wide - oracle.layer(to_host(x).astype(np.float32), perm, off, p)).max() <= bar * (2 ** 0.5 if G == 1 else 1)
        for kw in [dict(flags=ff.FF_FLAG_OUT_F32), dict(), dict(flags=ff.FF_FLAG_TAIL_DROP, lists=drop)] + \
                ([dict(embed=e), dict(embed=e, flags=ff.FF_FLAG_OUT_F32)] if embeds else []):
            assert np.array_equal(run(mapping, **kw), run(other, **kw)), (G, kw.keys())
        if not embeds:
            with pytest.raises(Exception):
                run(mapping, embed=e)


@pytest.mark.parametrize("C", [64, 128, 256])
@pytest.mark.parametrize("G", [32, 64, 80, 96, 128])
def test_selected_mapping_at_its_bounds(C, G):
    """Launches of one, just under and just over a round of compute units per group of the workgroup: the mapping that
    is chosen agrees with the one that serves this size at any count."""
    other = {128: (10, 7, 9, 9, 9), 64: (1, 2, 4, 4, 4), 256: (1, 2, 4, 4, 4)}[C][[32, 64, 80, 96, 128].index(G)]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(C + G)
    lw = ff.LayerWeights(ffsynth.layer_params(C, 2 * C, HEADS[C], seed=5), ff.FF_BF16, DEV)
    for groups in (1, 255, 256, 257, 513, 1025):
        n = groups * G - G // 3
        perm = torch.randperm(n, device=DEV, generator=gen).to(torch.int32)
        goff = torch.arange(0, groups + 1, device=DEV, dtype=torch.int32).mul_(G).clamp_(max=n)
        num = torch.full((1,), groups, device=DEV, dtype=torch.int32)
        x = torch.randn(n, C, device=DEV, generator=gen).bfloat16()
        got = ff.ff_group_attention(x, perm, goff, num, groups, lw, G, ff.FF_BF16)
        want = ff.ff_group_attention(x, perm, goff, num, groups, lw, G, ff.FF_BF16, ff.FF_FLAG_VARIANT(other))
        assert torch.equal(got, want), groups
