"""The work lists of a batch, compiled for the host: every cell of every patch
once, items no longer than asked for, whatever the cells per item.  CPU only."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "hostbuild", "batch_items_host.cpp")
MAX = 2 ** 63 - 1
CUS, THREADS = 256, (256, 512)
ROOM = 1 << 20


@pytest.fixture(scope="module")
def bi(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("bi") / "libbi.so")
    # (an overflow wraps, and shows in the items)
    subprocess.run([gxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-fwrapv", "-o", out, SRC],
                   check=True, capture_output=True)
    L = C.CDLL(out)
    L.bi_cells.restype = L.bi_rounds.restype = C.c_int64
    return L


def _cut(L, patches, chunk, rounds):
    n = np.array([p[0] for p in patches], np.int64)
    ng = np.array([p[1] for p in patches], np.int32)
    out = np.zeros((ROOM, 3), np.int64)
    ptr = lambda a: a.ctypes.data_as(C.c_void_p)
    head = (ptr(n), ptr(ng), C.c_int32(len(patches)), C.c_int64(chunk))
    full, lanes = C.c_int64(-1), np.zeros(2, np.int32)
    if rounds:
        k = L.bi_rounds(*head, C.c_int64(CUS), C.c_int32(THREADS[0]), C.c_int32(THREADS[1]),
                        ptr(out), C.c_int64(ROOM), C.byref(full), ptr(lanes))
    else:
        k = L.bi_cells(*head, ptr(out), C.c_int64(ROOM))
    assert 0 <= k <= ROOM
    return out[:k], full.value, lanes


def _lanes(ng):
    lanes = 1
    while 2 * lanes < ng:
        lanes *= 2
    return lanes


PATCHES = {
    "uneven": [(700, 64), (300, 1), (513, 8), (0, 16), (70, 65), (1, 7), (33, 128), (2000, 3)],
    "wide": [(65536, 64), (4096, 33), (1, 2)],
    "none": [],
}


@pytest.mark.parametrize("chunk", [1, 9, 256, 1 << 20, 1 << 57, 1 << 58, 1 << 62, MAX])
@pytest.mark.parametrize("name", PATCHES)
@pytest.mark.parametrize("rounds", [False, True])
def test_every_cell_once(bi, name, chunk, rounds):
    patches = PATCHES[name]
    items, n_full, lanes = _cut(bi, patches, chunk, rounds)
    for p, (n, ng) in enumerate(patches):
        mine = items[items[:, 0] == p]
        assert (mine[:, 1:] == np.stack([np.append([0], mine[:-1, 2])[:len(mine)],
                                         mine[:, 2]], 1)).all()
        assert (len(mine) == 0) == (n == 0) and (n == 0 or mine[-1, 2] == n)
        most = max(chunk * 32 // _lanes(ng), 1) if rounds else chunk
        assert all(0 < c1 - c0 <= most for _, c0, c1 in mine.tolist())
        if chunk >= n and not rounds:
            assert len(mine) == (n > 0)
    ngs = [patches[p][1] for p in items[:, 0]]
    full = [2 * _lanes(g) == g for g in ngs]
    if rounds:
        assert n_full == sum(full) and all(full[:n_full])
        for f, at in ((0, slice(n_full, None)), (1, slice(0, n_full))):
            assert ngs[at] == sorted(ngs[at], reverse=True)
            assert lanes[f] == sum({_lanes(g) for g in ngs[at]})
    else:
        assert ngs == sorted(ngs, reverse=True)


@pytest.mark.parametrize("chunk", [1 << 40, 1 << 58, MAX])
def test_no_cap_cuts_by_rounds_alone(bi, chunk):
    """However large the cells per item, the items are those of the rounds: two
    of the cells that a workgroup has in flight at the least."""
    items, _, _ = _cut(bi, [(65536, 64), (4096, 33)], chunk, True)
    assert len(items) <= 65536 // 32 + 4096 // 16 + 2
