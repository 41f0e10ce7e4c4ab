"""Clouds sorted in one launch: where a workgroup's range of key values holds more pillars than its lists, where pillars share
cells, few or many of 32 key values, and on both sides of the limits of what is sorted this way (frames, grid, pillars, key values
of a range)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2301_08739_amd as ff
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _cells(B, X, Y, n, seed, each=1):
    """n pillars on distinct cells of a board, each cell `each` times, shuffled."""
    rng = np.random.default_rng(seed)
    k = np.repeat(rng.choice(B * X * Y, -(-n // each), replace=False), each)[:n]
    k = k[rng.permutation(n)]
    return np.stack([k // (X * Y), k // Y % X, k % Y], 1).astype(np.int32)


def _board(X, Y):  # every cell, in grid order: neighbours share a window
    k = np.arange(X * Y)
    return np.stack([0 * k, k // Y, k % Y], 1).astype(np.int32)


def _crowds(words, each, single, seed):
    """`words` runs of 32 cells of one window of 256 x 256 with `each` pillars, and `single` cells with one, shuffled."""
    rng = np.random.default_rng(seed)
    crowd = np.repeat(2 * np.arange(words), each) * 32 + rng.integers(0, 32, words * each)
    k = rng.permutation(np.concatenate([crowd, 65536 - 1 - 5 * np.arange(single)]))
    return np.stack([0 * k, k // 256, k % 256], 1).astype(np.int32)


CASES = {
    "most_of_one_cell": (lambda: np.tile(np.array([[0, 467, 467]], np.int32), (24576, 1)), 1, 468, 13),
    "ranked_words": (lambda: _crowds(90, 256, 0, 19), 1, 4096, 256),
    "crowded_word": (lambda: _crowds(1, 257, 0, 20), 1, 4096, 256),
    "most_crowded_words": (lambda: _crowds(95, 257, 150, 21), 1, 4096, 256),
    "crowded_and_single": (lambda: _crowds(3, 5000, 9000, 22), 1, 4096, 256),
    "a_window_twice": (lambda: _cells(1, 96, 128, 24576, 23, each=2), 1, 4096, 256),
    "a_window_once": (lambda: _cells(1, 256, 256, 24576, 24), 1, 4096, 256),
    "a_window_nearly_once": (lambda: np.concatenate([_cells(1, 256, 256, 24570, 25), np.zeros((6, 3), np.int32)]), 1, 4096, 256),
    "one_cell": (lambda: np.tile(np.array([[0, 300, 77]], np.int32), (20000, 1)), 1, 468, 13),
    "two_cells": (lambda: np.array([[0, 300, 77], [0, 300, 78]], np.int32)[np.arange(9001) % 3 // 2], 1, 468, 13),
    "one_pillar": (lambda: np.array([[0, 5, 9]], np.int32), 1, 468, 13),
    "board_in_grid_order": (lambda: _board(156, 156), 1, 468, 9),
    "dense_board": (lambda: _cells(1, 156, 156, 24336, 1), 1, 468, 13),
    "every_cell_twice": (lambda: _cells(1, 120, 120, 24000, 2, each=2), 1, 468, 13),
    "few_shared_cells": (lambda: np.concatenate([_cells(1, 468, 468, 12000, 3), _cells(1, 468, 468, 500, 4)]), 1, 468, 13),
    "few_cells": (lambda: np.random.default_rng(18).integers(0, 7, (5000, 3)).astype(np.int32) * [0, 1, 1], 1, 468, 13),
    "hundred_cells": (lambda: np.random.default_rng(13).integers(0, 10, (24000, 3)).astype(np.int32) * [0, 1, 1], 1, 468, 13),
    "half_in_one_cell": (lambda: np.concatenate([_cells(1, 468, 468, 6000, 14), np.tile(np.array([[0, 9, 9]], np.int32), (18000, 1))])
                         [np.random.default_rng(15).permutation(24000)], 1, 468, 13),
    "corner_cells_shared": (lambda: np.random.default_rng(16).integers(0, 120, (24576, 3)).astype(np.int32) * [0, 1, 1], 1, 468, 13),
    "many_shared_cells": (lambda: np.random.default_rng(17).integers(0, 200, (24576, 3)).astype(np.int32) * [0, 1, 1], 1, 468, 13),
    "sixteen_frames": (lambda: _cells(16, 60, 60, 5000, 5), 16, 60, 6),
    "seventeen_frames": (lambda: _cells(17, 60, 60, 5000, 6), 17, 60, 6),
    "grid_4096": (lambda: _cells(1, 4096, 4096, 7000, 7), 1, 4096, 256),
    "wide_keys": (lambda: _cells(2, 1500, 1500, 4000, 8), 2, 1500, 9),
    "window_of_one": (lambda: _cells(1, 468, 468, 9000, 9), 1, 468, 1),
    "most_pillars": (lambda: _cells(1, 468, 468, 24576, 10), 1, 468, 13),
    "one_more": (lambda: _cells(1, 468, 468, 24577, 11), 1, 468, 13),
    "eight_frames_two_rounds": (lambda: _cells(8, 468, 468, 24576, 12), 8, 468, 9),
}


@pytest.mark.parametrize("name", list(CASES))
def test_against_the_oracle(name):
    make, B, grid, w = CASES[name]
    coords = np.ascontiguousarray(make(), dtype=np.int32)
    g, og = ff.Geometry(B, grid, grid, w, w), oracle.Geometry(B, grid, grid, w, w)
    ct = torch.from_numpy(coords).to(DEV)
    pairs = [(0, 0), (1, 0), (0, 1), (1, 1)]
    for G, tail in ((64, ff.FF_TAIL_MASK), (7, ff.FF_TAIL_DROP)):
        print(name, G, flush=True)
        got = ff.ff_flatten_batch(ct, g, pairs, G, tail=tail)
        for (axis, shift), (perm, off, ng) in zip(pairs, got):
            if tail == ff.FF_TAIL_MASK:
                want_perm, want_off, want_keys = oracle.flatten(coords, og, axis, shift, G)
                k = int(ng.item())
                assert k == len(want_off) - 1 and np.array_equal(off.cpu().numpy()[:k + 1], want_off)
                assert np.array_equal(perm.cpu().numpy(), want_perm)
                one, one_off, one_ng, keys = ff.ff_flatten(ct, g, axis, shift, G, want_keys=True)
                assert torch.equal(one, perm) and int(one_ng.item()) == k
                assert np.array_equal(keys.cpu().numpy().view(np.uint64), want_keys)
            else:
                sizes = np.bincount(coords[:, 0], minlength=B)
                starts = np.concatenate([[0], np.cumsum(sizes)[:-1]])
                want = np.concatenate([starts[b] + G * np.arange(sizes[b] // G) for b in range(B)] + [[len(coords)]])
                assert int(ng.item()) == len(want) - 1
                assert np.array_equal(off.cpu().numpy()[:len(want)], want)
                assert np.array_equal(np.sort(perm.cpu().numpy()), np.arange(len(coords)))
