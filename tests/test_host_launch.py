"""What the library makes of a launch's status, on a stand-in HIP runtime (CPU
only; see host_runtime.py).

An error that an earlier call of the thread left behind (of this library or of
the caller's own code) is not a launch's: writes, migrations, plans, packs and
the measurement aids enqueued with one pending succeed, keep their pages and
leave the error for whoever asks for it.
"""

import ctypes as C

import pytest

import host_runtime as hr
from paper_2606_23087_amd import flowpool as fp
from host_runtime import Pool

S1, S2 = 0x51, 0x52        # stream handles; the stand-in never looks into one


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return hr.build(tmp_path_factory.mktemp("host"))


@pytest.fixture()
def pool(lib):
    settings = (lib.stub_pending, lib.stub_launch, lib.stub_record, lib.stub_wait, lib.stub_busy, lib.stub_capturing)
    for f in settings:
        f(0)
    p = Pool(lib)
    p.log()
    yield p
    for f in settings:
        f(0)
    p.destroy()


MANY = 100                 # samples of a pack whose run table is copied to the device


def _call(pool, what, samples):
    """One call of a kind on stream S1, over resident samples."""
    if what == "write":
        return pool.write(3, 10, S1)[0]
    if what == "migrate":
        return pool.migrate(samples[:2], 1, S1)
    if what == "plan":
        return pool.plan(samples[:3], S1)
    if what == "copy":
        return pool.lib.fp_copy_bytes(C.c_void_p(1 << 20), C.c_void_p(1 << 21), 4096, 64, S1)
    if what == "gather":
        return pool.lib.fp_gather_rows(C.c_void_p(1 << 20), 8, 64, C.c_void_p(1 << 21), S1)
    ids = (samples * MANY)[:MANY] if "staged" in what else samples[:2]
    return pool.pack(ids, S1, "noalloc" in what)


CALLS = ["write", "migrate", "plan", "pack", "pack staged", "pack noalloc", "pack staged noalloc", "copy", "gather"]
KERNEL = dict(write="k_write", migrate="k_migrate", plan="k_cost", copy="k_copy", gather="k_gather")


@pytest.mark.parametrize("what", CALLS)
def test_an_earlier_error_is_not_the_launch_s(pool, what):
    samples = [pool.write(3, 10, S1)[1] for _ in range(4)]
    assert pool.lib.pool_reclaim(pool.p, 1, None) == 0
    hbm, host, n = pool.stats()
    pool.log()
    pool.lib.stub_pending(hr.INVALID_VALUE)
    assert _call(pool, what, samples) == 0, pool.lib.fp_last_error()
    assert pool.lib.stub_peek() == hr.INVALID_VALUE
    launches = [l for l in pool.log() if l.startswith("launch")]
    assert len(launches) == 1 and KERNEL.get(what, "k_pack") in launches[0]
    if what == "write":
        assert pool.stats() == (hbm - 3, host, n + 1)
    elif what == "migrate":
        # two samples' pages taken in the host tier; those they leave wait for the copies
        pool.lib.pool_reclaim(pool.p, 1, None)
        assert pool.stats() == (hbm + 6, host - 6, n)
    else:
        assert pool.stats() == (hbm, host, n)


@pytest.mark.parametrize("what", [c for c in CALLS if c not in ("copy", "gather")])
def test_a_failed_launch_waits_before_it_gives_back(pool, what):
    """A launch that reports a failure may still have queued its kernel, and a
    staged pack has queued the copy of its table: the call waits for the stream
    before what they use (pages, arena, staging buffer, event) can be used again."""
    samples = [pool.write(3, 10, S1)[1] for _ in range(4)]
    assert pool.lib.pool_reclaim(pool.p, 1, None) == 0
    before, pages = pool.stats(), [pool.pages(i) for i in samples]
    pool.log()
    pool.lib.stub_launch(hr.LAUNCH_FAILURE)
    assert _call(pool, what, samples) == -6          # EHIP
    pool.lib.stub_launch(0)
    log = pool.log()
    at = next(i for i, l in enumerate(log) if l.startswith("launch"))
    assert f"stream_sync {S1}" in log[at:], log
    assert pool.stats() == before and [pool.pages(i) for i in samples] == pages
    assert _call(pool, what, samples) == 0


@pytest.mark.parametrize("noalloc", [False, True])
def test_a_pack_that_fails_behind_its_table_s_copy_waits_for_it(pool, noalloc):
    samples = [pool.write(3, 10, S2)[1] for _ in range(4)]
    pool.lib.stub_busy(1)                            # the writes, on another stream, have not finished
    pool.lib.stub_wait(hr.INVALID_VALUE)
    pool.log()
    assert pool.pack((samples * MANY)[:MANY], S1, noalloc) == -6
    pool.lib.stub_wait(0)
    log = pool.log()
    assert f"copy {S1}" in log and f"stream_sync {S1}" in log[log.index(f"copy {S1}"):], log


def test_a_failed_launch_under_capture_does_not_wait(pool):
    samples = [pool.write(3, 10, S1)[1] for _ in range(2)]
    assert pool.lib.pool_reclaim(pool.p, 1, None) == 0
    pool.log()
    pool.lib.stub_capturing(1)
    pool.lib.stub_launch(hr.LAUNCH_FAILURE)
    assert pool.pack(samples, S1) == -6
    assert not any("sync" in l for l in pool.log())  # a wait would end the capture
    pool.lib.stub_launch(0)
    assert pool.pack(samples, S1) == 0
    assert pool.lib.pool_release_captured(pool.p, pool.ids(samples), 2) == 0
    pool.lib.stub_capturing(0)


def test_a_reported_hip_error_is_not_left_behind(pool):
    """A call that has returned EHIP has reported its error; the thread's next
    look at its last error (torch's after each of its launches, say) finds none."""
    lib = pool.lib
    cfg = fp.fp_pool_config()
    lib.fp_config_init(C.byref(cfg))
    cfg.hidden, cfg.page_tokens, cfg.hbm_pages, cfg.chunk_bytes = 1 << 20, 1 << 10, 1 << 19, 1 << 60
    out = C.c_void_p()
    assert lib.pool_create(C.byref(cfg), C.byref(out)) == -6 and not out.value      # 2^50 bytes
    assert lib.stub_peek() == 0
    i = pool.write(3, 10, S1)[1]
    lib.stub_busy(1)
    assert pool.pack([i], S2) == 0
    lib.stub_record(hr.INVALID_VALUE)
    assert lib.pool_free_sample(pool.p, i) == -6     # cannot record the reader's event
    assert lib.stub_peek() == 0
    lib.stub_launch(hr.LAUNCH_FAILURE)
    for what in CALLS:
        assert _call(pool, what, [i] * 4 if what not in ("migrate", "plan") else [i]) == -6
        assert lib.stub_peek() == 0, what
