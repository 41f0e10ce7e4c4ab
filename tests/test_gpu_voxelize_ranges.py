"""Points to pillars over grids of up to 1,983 ranges of 256 cells: edges of the tiles, of the ranges and of a range's list in
LDS, against the oracle, and bit for bit against the general path, which a grid with more frames takes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2301_08739_amd as ff
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _points(m, B, X, Y, seed, spread=1.0, out=0.05):
    """m points, the share `out` of them outside; spread < 1 crowds the others into the first cells of each axis."""
    rng = np.random.default_rng(seed)
    xy = ((rng.random((m, 2)) ** (1.0 / spread)) * [X, Y]).astype(np.float32)
    away = rng.random(m) < out
    xy[away] += np.float32(2 * max(X, Y))
    return xy, rng.integers(-1 if out else 0, B, m).astype(np.int32)


CASES = {  # m, frames, grid, spread, outside
    "one_point": (1, 1, (468, 468), 1.0, 0.0),
    "tile": (2048, 1, (468, 468), 1.0, 0.05),
    "tile_and_one": (2049, 1, (468, 468), 1.0, 0.05),
    "one_range": (256, 1, (16, 16), 1.0, 0.05),
    "one_cell_more": (257, 1, (1, 257), 1.0, 0.05),
    "odd_ranges": (3000, 3, (64, 33), 1.0, 0.05),
    "one_cell": (1, 1, (1, 1), 1.0, 0.0),
    "corner": (60000, 1, (468, 468), 0.1, 0.02),         # a range with several lists of points, cells with hundreds
    "into_one_cell": (9000, 1, (468, 468), 0.001, 0.1),
    "list": (4096, 1, (468, 468), 0.02, 0.0),
    "list_and_one": (4097, 1, (468, 468), 0.02, 0.0),
    "as_many_as_cells": (90000, 1, (300, 300), 0.5, 0.03),
    "one_point_more": (90001, 1, (300, 300), 0.5, 0.03),
    "most_points": (507648, 3, (1983, 85), 1.0, 0.01),
    "most_ranges": (30000, 3, (1983, 85), 1.0, 0.05),
    "one_range_more": (30000, 3, (1984, 86), 1.0, 0.05),
}


@pytest.mark.parametrize("name", list(CASES))
def test_against_the_oracle_and_the_general_path(name):
    m, B, (X, Y), spread, out = CASES[name]
    print(name, flush=True)
    xy, frame = _points(m, B, X, Y, 17 + m, spread, out)
    grid = ff.VoxelGrid(0.0, 0.0, 1.0, 1.0)
    many = 1983 * 256 // (X * Y) + 1
    for Cp in (3, 4):
        pf = np.random.default_rng(Cp).standard_normal((m, Cp)).astype(np.float32)
        dev = [torch.from_numpy(a).to(DEV) for a in (xy, frame, pf)]
        coords, feats, npil, p2p = ff.ff_voxelize(*dev, ff.Geometry(B, X, Y, 13, 13), grid)
        n = int(npil.item())
        wc, wf, wp = oracle.voxelize(xy, frame, pf, oracle.Geometry(B, X, Y, 13, 13), 0.0, 0.0, 1.0, 1.0)
        assert n == len(wc) and np.array_equal(coords[:n].cpu().numpy(), wc)
        assert np.array_equal(p2p.cpu().numpy(), wp)
        # float32 sums of k terms of size one: (k + 3) roundings of at most 2^-24 of the sum of magnitudes
        k = np.bincount(wp[wp >= 0], minlength=n).max(initial=1)
        size = np.zeros((n, Cp))
        np.add.at(size, wp[wp >= 0], np.abs(pf[wp >= 0]))
        size /= np.bincount(wp[wp >= 0], minlength=n)[:, None].clip(1)
        assert np.all(np.abs(feats[:n].cpu().numpy() - wf) <= (k + 3) * 2.0 ** -24 * size + 1e-30)
        if m <= 60000 and many > B and many <= 60000:
            other = [dev[0], torch.where(dev[1] < B, dev[1], -1), dev[2]]
            gc, gf, gn, gp = ff.ff_voxelize(*other, ff.Geometry(many, X, Y, 13, 13), grid)
            assert int(gn.item()) == n and torch.equal(gc[:n], coords[:n]) and torch.equal(gp, p2p)
            assert torch.equal(gf[:n], feats[:n])
