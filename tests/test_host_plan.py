"""plan_microbatches refuses a bad list before it enqueues anything, on a
stand-in HIP runtime (CPU only; see host_runtime.py): no launch, no wait, no
allocation, whatever the list's length, and the first fault in the list is the
one reported.
"""

import pytest

import host_runtime as hr
from host_runtime import Pool

S1, S2 = 0x51, 0x52
EINVAL, ENOENT, ESTATE = -1, -3, -7


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return hr.build(tmp_path_factory.mktemp("host"))


@pytest.fixture()
def pool(lib):
    p = Pool(lib)
    yield p
    lib.stub_busy(0)
    lib.stub_capturing(0)
    p.destroy()


@pytest.mark.parametrize("bad,status", [
    (lambda i: [i[0], i[1], i[0]], EINVAL),
    (lambda i: [i[0], 999], ENOENT),
    (lambda i: [i[0], i[0], 999], EINVAL),
    (lambda i: [i[0], 999, i[0]], ENOENT),
    (lambda i: [999, 999], ENOENT),
    (lambda i: i * 60000, EINVAL),                   # longer than a staging buffer
])
@pytest.mark.parametrize("capturing", [0, 1])
def test_a_refused_list_enqueues_nothing(pool, bad, status, capturing):
    ids = [pool.write(3, 10, S2)[1] for _ in range(3)]
    pool.lib.stub_busy(1)                            # the writes have not finished
    pool.lib.stub_capturing(capturing)
    pool.log()
    assert pool.plan(bad(ids), S1) == status
    assert pool.log() == []
    if capturing:
        assert pool.plan(ids, S1) == ESTATE and pool.log() == []
        return
    for _ in range(2):                               # a list that is right is planned, also after a refusal
        assert pool.plan(ids, S1) == 0
        assert sum("k_cost" in l for l in pool.log()) == 1
    assert pool.plan(ids[:1], S1) == 0 and pool.plan([], S1) == 0
