"""A migration's work list, on a stand-in HIP runtime (CPU only; see
host_runtime.py): whatever the page size, the order of the free pages, partly
migrated samples and partial last pages, its pieces copy each moved page's rows
to its new frame once, no piece is longer than the kernel's steps for one, and
the list stays inside the staging buffer. Runs of 8 MiB of adjacent pages or
more, and only those, are copies by the runtime, none across two chunks of a
tier's backing.
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
        copies = pool.copies()
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
        assert not copies
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


def joined(copies):
    """Copies of vectors, by source, those that continue one another made one; nothing is copied to twice."""
    out = []
    for s, d, v in sorted(copies):
        if out and out[-1][0] + 16 * out[-1][2] == s and out[-1][1] + 16 * out[-1][2] == d:
            out[-1][2] += v
        else:
            out.append([s, d, v])
    ends = sorted((d, d + 16 * v) for _, d, v in out)
    assert all(a[1] <= b[0] for a, b in zip(ends, ends[1:]))
    return out


LONG = 8 << 20


@pytest.mark.parametrize("hidden,page", [(8192, 64), (8192, 16), (1024, 4096)])      # 1 MiB, 256 KiB and 8 MiB pages
@pytest.mark.parametrize("shuffle,chunk", [(0, 0), (0, 20 << 20), (3, 0)])
def test_long_runs_are_copies(lib, hidden, page, shuffle, chunk):
    rng = np.random.default_rng([hidden, page, shuffle, chunk])
    pb = 2 * hidden * page
    pages = (96 << 20) // pb
    chunk_pages = max(1, (chunk or 1 << 30) // pb)
    pool = Pool(lib, pages, pages, hidden, page, chunk, shuffle)
    samples, left, vpr = [], pages, hidden // 8
    while left > 0 and len(samples) < 8:
        n = min(left, int(rng.integers(1, max(2, (20 << 20) // pb))))
        rows = n * page - int(rng.integers(0, 2)) * int(rng.integers(0, page))
        samples.append((pool.write(2, rows, S1)[1], rows))
        left -= n
    seen = 0
    for round_ in range(6):
        tier = (round_ + 1) % 2
        some = samples if round_ < 2 else [samples[i] for i in rng.permutation(len(samples))[:4]]
        before = {i: pool.frames(i) for i, _ in some}
        lib.stub_clear()
        assert pool.migrate([i for i, _ in some], tier, S1) == 0
        want = [(a, b, min(page, n - k * page) * vpr) for i, n in some
                for k, ((t0, a), (_, b)) in enumerate(zip(before[i], pool.frames(i))) if t0 != tier]
        if not want:
            continue
        pieces, _, _, _, _ = work_list(lib)
        copies = [(s, d, n // 16) for s, d, n in pool.copies()]
        assert joined(pieces + copies) == joined(want)
        seen += len(copies)
        # the runs: pages in the order they are moved, each continuing the last on both sides
        starts = chunk_starts(pool, pages, chunk_pages)
        runs = []
        for s, d, v in want:
            if (runs and runs[-1][0] + 16 * runs[-1][2] == s and runs[-1][1] + 16 * runs[-1][2] == d
                    and s not in starts and d not in starts):
                runs[-1][2] += v
            else:
                runs.append([s, d, v])
        assert [tuple(r) for r in runs if 16 * r[2] >= LONG] == copies
        log = pool.log()
        assert log[-1].startswith("launch") and sum(l.startswith("launch") for l in log) == 1
        assert not any("malloc" in l for l in log)
    assert seen > 0 or shuffle
    pool.destroy()


def chunk_starts(pool, pages, chunk_pages):
    """Addresses of the first pages of the backing chunks (frames in order only where they are not shuffled)."""
    out = set()
    rs, ss, pb = (C.c_uint64 * 2)(), (C.c_uint64 * 2)(), C.c_int64()
    assert pool.lib.pool_layout(pool.p, rs, ss, pb) == 0
    for t in range(2):
        at = []
        for k in range(pages):
            tier, phys = C.c_int32(), C.c_uint64()
            assert pool.lib.pool_translate(pool.p, ss[t] + k * pb.value, tier, phys) == 0
            at.append(phys.value)
        if sorted(at) == at or chunk_pages < pages:
            out |= {at[k] for k in range(0, pages, chunk_pages)}
        else:
            out.add(min(at))
    return out


def test_the_work_list_takes_the_room_it_needs(lib):
    """The staging of 6000 pages of 28 KiB: 8 bytes each and 32 a piece, 7 pieces each in a random order; where they are
    adjacent they are copies by the runtime."""
    for shuffle, most in ((0, 0), (5, 6000 * (8 + 7 * 32) + 4096)):
        pool = Pool(lib, 6000, 6000, 1024, 14, 0, shuffle)
        ids = [pool.write(1, 14 * 1000, S1)[1] for _ in range(6)]
        pool.log()
        assert pool.migrate(ids, 1, S1) == 0
        taken = [int(l.split()[1]) for l in pool.log() if l.startswith("host_malloc")]
        assert sum(taken) <= most and len(taken) == (1 if shuffle else 0)
        pool.destroy()


def test_a_failed_copy_gives_the_pages_back_after_a_wait(lib):
    pool = Pool(lib, 24, 24, 8192, 64)
    i = pool.write(2, 20 * 64, S1)[1]
    pool.lib.pool_reclaim(pool.p, 1, None)
    before, frames = pool.stats(), pool.frames(i)
    lib.stub_copy(hr.INVALID_VALUE)
    pool.log()
    assert pool.migrate([i], 1, S1) == -6
    lib.stub_copy(0)
    log = pool.log()
    assert f"copy {S1}" in log and f"stream_sync {S1}" in log and not any("launch" in l for l in log)
    assert pool.stats() == before and pool.frames(i) == frames
    assert pool.migrate([i], 1, S1) == 0
    pool.destroy()
