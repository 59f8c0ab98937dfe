"""A migration's work list, on a stand-in HIP runtime (CPU only; see
host_runtime.py): whatever the page size, the order of the free pages, partly
migrated samples and partial last pages, its pieces copy each moved page's rows
to its new frame once, no piece is longer than the kernel's steps for one, and
the list stays inside the staging buffer.
"""

import ctypes as C
import struct

import numpy as np
import pytest

import host_runtime as hr
from host_runtime import Pool

S1 = 0x51
STEP = 256                                   # 16-byte vectors a wave moves per step
STAGE = 1 << 20                              # the smallest staging buffer


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return hr.build(tmp_path_factory.mktemp("host"))


def work_list(lib):
    """(pieces as (source, destination, vectors), page lists as (slot, words), steps per piece, target tier)"""
    raw = C.string_at(lib.stub_migrate_args(), 48)
    stage, meta, desc, at, n, steps, lists, tier = struct.unpack("<QQQqIIii", raw)
    pieces = [struct.unpack("<QQIIQ", C.string_at(stage + at + 32 * k, 32))[:3] for k in range(n)]
    out = []
    for k in range(lists):
        words_at, meta_off, n_words, slot, _ = struct.unpack("<qqiiq", C.string_at(stage + 32 * k, 32))
        out.append((slot, list(struct.unpack(f"<{n_words}Q", C.string_at(stage + words_at, 8 * n_words)))))
        assert words_at % 16 == 0 and meta_off % 16 == 0 and words_at + 8 * n_words <= at
    return pieces, out, steps, tier, at + 32 * n


def expand(copies):
    """Copies of vectors as a dict from each vector's destination to its source; nothing is copied to twice."""
    d = {}
    for src, dst, vecs in copies:
        for v in range(vecs):
            assert dst + 16 * v not in d
            d[dst + 16 * v] = src + 16 * v
    return d


# hidden, rows a page: pages of 1, 3, 255, 256, 257, 600, 2047, 2048 and 2056 vectors
SIZES = [(8, 1), (8, 3), (8, 255), (8, 256), (8, 257), (16, 300), (8, 2047), (8, 2048), (64, 257)]


@pytest.mark.parametrize("hidden,page", SIZES)
@pytest.mark.parametrize("shuffle,chunk_pages", [(0, 0), (0, 5), (7, 3)])
def test_work_list_copies_what_moved(lib, hidden, page, shuffle, chunk_pages):
    rng = np.random.default_rng([hidden, page, shuffle])
    pool = Pool(lib, 64, 64, hidden, page, chunk_pages * 2 * hidden * page, shuffle)
    samples = []
    for _ in range(9):
        n = int(rng.integers(1, 5 * page + 1))
        tiers = [(0,), (1,), (0, 1), (0, 0, 1)][int(rng.integers(0, 4))]
        samples.append((pool.write(2, n, S1, tiers)[1], n))
    vpr = hidden // 8
    for round_ in range(8):
        tier = round_ % 2
        some = [samples[i] for i in rng.permutation(len(samples))[:int(rng.integers(1, len(samples) + 1))]]
        before = {i: pool.frames(i) for i, _ in some}
        lib.stub_clear()
        assert pool.migrate([i for i, _ in some], tier, S1) == 0
        log = pool.log()
        after = {i: pool.frames(i) for i, _ in some}
        want, moved = [], 0
        for i, n in some:
            for k, ((t0, a), (t1, b)) in enumerate(zip(before[i], after[i])):
                assert t1 == tier and (a == b) == (t0 == tier)
                if t0 != tier:
                    want.append((a, b, min(page, n - k * page) * vpr))
                    moved += 1
        if not moved:
            assert not any("launch" in l for l in log)
            continue
        pieces, lists, steps, to, used = work_list(lib)
        assert expand(pieces) == expand(want)
        assert all(0 < v <= steps * STEP for _, _, v in pieces) and to == tier
        assert len(pieces) <= sum(-(-v // (steps * STEP)) for _, _, v in want) and used <= STAGE
        if not shuffle and not chunk_pages and page * vpr < 8 * STEP:     # adjacent small pages: whole steps
            for (s, d, v), (s1, d1, _) in zip(pieces, pieces[1:]):
                assert v == STEP or (s + 16 * v, d + 16 * v) != (s1, d1)
        assert sorted(w for _, w in lists) == sorted(pool.pages(i) for i, _ in some
                                                     if any(t != tier for t, _ in before[i]))
    pool.destroy()
