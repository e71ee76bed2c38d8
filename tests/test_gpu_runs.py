"""The runs of a tile's lists, from places in any order: the list kernels hand places out by LDS additions, whose lanes have always been
served in order but need not be, so a tile looks whether they were and sorts its runs if not."""
import ctypes
import os

import numpy as np
import pytest
import torch

from paper_2604_07144_amd import build

pytestmark = pytest.mark.gpu

TILE, WAVE, PADDING = 1024, 64, 1024 << 4


@pytest.fixture(scope="module")
def runs():
    if not os.path.exists(build.TEST_LIB_PATH):
        build.build_tests()
    return ctypes.CDLL(build.TEST_LIB_PATH)


def places_of(ids, M, order, rng):
    """Per request its place among its replica's: in request order, with the lanes of every 64 requests served the other way round, in any
    order, or in order but for the last two of one replica."""
    place = np.zeros(TILE, np.uint16)
    lanes = np.arange(TILE)
    key = {"in order": lanes, "lanes reversed": lanes // WAVE * WAVE + WAVE - 1 - lanes % WAVE, "any": rng.permutation(TILE), "two swapped": lanes}[order]
    for m in range(M):
        mine = np.flatnonzero(ids == m)
        place[mine[np.argsort(key[mine], kind="stable")]] = np.arange(mine.size)
    if order == "two swapped":
        longest = np.flatnonzero(ids == np.bincount(ids[ids < M], minlength=M).argmax())
        if longest.size >= 2:
            place[longest[-2:]] = place[longest[-2:]][::-1]
    return place


@pytest.mark.parametrize("order", ["in order", "lanes reversed", "any", "two swapped"])
@pytest.mark.parametrize("M", [1, 2, 63, 64, 65, 200, 1024])
def test_runs_come_out_in_order(runs, M, order):
    rng = np.random.default_rng(M)
    kinds = ["even", "one", "few", "some unlisted", "none", "a part"]
    ids = []
    for kind in kinds:
        t = rng.integers(0, M, TILE)
        if kind == "one":
            t[:] = M - 1
        elif kind == "few":
            t = rng.integers(0, min(M, 3), TILE)
        elif kind == "some unlisted":
            t = np.where(rng.random(TILE) < 0.5, M, t)
        elif kind == "none":
            t[:] = M
        elif kind == "a part":
            t[701:] = M
        ids.append(t)
    ids = np.stack(ids).astype(np.uint16)
    places = np.stack([places_of(t, M, order, rng) for t in ids])
    n, cap = len(kinds), int(runs.runs_tile_cap(ctypes.c_uint32(M)))
    dev = [torch.from_numpy(a.view(np.int16)).cuda() for a in (ids, places)]
    desc = torch.full((n, M), -1, dtype=torch.int32, device="cuda")
    lists = torch.full((n, cap), -1, dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    assert runs.runs_write(ctypes.c_void_p(dev[0].data_ptr()), ctypes.c_void_p(dev[1].data_ptr()), ctypes.c_uint32(M), ctypes.c_uint32(n),
                           ctypes.c_void_p(desc.data_ptr()), ctypes.c_void_p(lists.data_ptr())) == 0
    desc, lists = desc.cpu().numpy().view(np.uint32), lists.cpu().numpy().view(np.uint16)
    for j in range(n):
        at = 0
        for m in range(M):
            mine = np.flatnonzero(ids[j] == m)
            assert int(desc[j, m]) == (mine.size << 16 | at), (kinds[j], m)
            room = (mine.size + 7) // 8 * 8
            want = np.concatenate([mine << 4, np.full(room - mine.size, PADDING)])
            assert (lists[j, at:at + room] == want).all(), (kinds[j], m)
            at += room
        assert (lists[j, at:] == 0xFFFF).all(), kinds[j]                 # nothing is written beyond the runs
