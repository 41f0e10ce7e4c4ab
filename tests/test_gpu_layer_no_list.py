"""Group lists that do not cover the cloud: num_groups < 0 (a failed sort) computes and copies nothing, and a list that leaves
sorted positions uncovered, the first among them, gives its groups their rows and leaves the others alone."""
import numpy as np
import pytest
import torch

import ffsynth
import oracle
import paper_2301_08739_amd as ff
from gpu_util import DEV, to_dev_feats, to_host

pytestmark = pytest.mark.gpu

HEADS = {64: 4, 128: 8, 256: 8}
SHAPES = [(dt, C, G) for dt in (ff.FF_BF16, ff.FF_F16, ff.FF_F32) for C in (64, 128, 256) for G in (20, 64, 70, 128)
          if not (dt == ff.FF_F32 and C == 256 and G > 64)]


def _inputs(dt, C, n, seed):
    rng = np.random.default_rng(seed)
    p = ffsynth.layer_params(C, 2 * C, HEADS[C], seed=seed)
    return (rng, to_dev_feats(rng.standard_normal((n, C)), dt), to_dev_feats(0.5 * rng.standard_normal((n, C)), dt),
            p, ff.LayerWeights(p, dt, DEV))


@pytest.mark.parametrize("flags", [0, ff.FF_FLAG_FORCE_GENERIC])
@pytest.mark.parametrize("dt,C,G", SHAPES)
def test_no_list_computes_nothing(dt, C, G, flags):
    n = 9000 if dt == ff.FF_F32 and G > 64 else 700          # (enough rows for the fused float32 kernel)
    rng, x, e, p, lw = _inputs(dt, C, n, 31)
    groups = -(-n // G)
    perm = torch.from_numpy(rng.permutation(n).astype(np.int32)).to(DEV)
    goff = torch.arange(groups + 1, device=DEV, dtype=torch.int32).mul_(G).clamp_(max=n)
    num = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    for embed in (None, e):
        for more in (0, ff.FF_FLAG_OUT_F32, ff.FF_FLAG_TAIL_DROP, ff.FF_FLAG_OUT_F32 | ff.FF_FLAG_TAIL_DROP):
            for max_groups in (groups, 0):
                out = torch.full((n, C), 7.0, device=DEV, dtype=torch.float32 if more & ff.FF_FLAG_OUT_F32 else x.dtype)
                ff.ff_group_attention(x, perm, goff, num, max_groups, lw, G, dt, flags | more, out=out, pos_embed=embed)
                assert bool((out == 7.0).all()), (more, max_groups)


@pytest.mark.parametrize("dt,C,G", SHAPES)
def test_uncovered_positions(dt, C, G):
    n = 9000 if dt == ff.FF_F32 and G > 64 else 700
    rng, x, e, p, lw = _inputs(dt, C, n, 37)
    perm = rng.permutation(n).astype(np.int32)
    offs = np.concatenate([np.arange(5, n - 2 * G, G), [n - 11]]).astype(np.int32)   # ends short, begins at position 5
    k = len(offs) - 1
    last = offs[-2] + min(G, offs[-1] - offs[-2])
    goff = np.concatenate([offs, np.full(3, 1 << 30, np.int32)])      # what lies behind the list is nobody's
    dev = [torch.from_numpy(a).to(DEV) for a in (perm, goff, np.array([k], np.int32))]
    rounded = lambda t: to_host(t).astype(np.float32)
    out = torch.full((n, C), 7.0, device=DEV, dtype=torch.float32)
    ff.ff_group_attention(x, dev[0], dev[1], dev[2], k + 3, lw, G, dt, ff.FF_FLAG_OUT_F32, out=out, pos_embed=e)
    got = to_host(out)
    members = np.concatenate([perm[a:min(b, a + G)] for a, b in zip(offs[:-1], offs[1:])])
    rest = np.setdiff1d(perm, members)
    assert last - 5 == len(members) and (got[rest] == 7.0).all()
    held = {kk: to_host(to_dev_feats(v, dt)).astype(np.float32) if isinstance(v, np.ndarray) else v for kk, v in p.items()}
    want = oracle.layer(rounded(x), perm, np.concatenate([offs[:-1], [last]]), held, pos_embed=rounded(e))
    bar = {ff.FF_BF16: 2e-2, ff.FF_F16: 2.5e-3, ff.FF_F32: 1e-4}[dt]
    assert np.abs(got[members] - want[members]).max() <= bar
