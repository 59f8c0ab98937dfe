"""plan_microbatches around the sizes where its launch changes: the slots of up
to 960 samples travel in the kernel's arguments, more are read from pinned
memory, 256 samples fill a workgroup. Costs and assignment equal the oracle's,
and a list that is refused is refused with the same error as ever, whatever is
wrong with it further on.
"""

import numpy as np
import pytest

from gpu_common import say
from oracle.plan import cost_scaled, greedy_partition

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_23087_amd import flowpool
    return flowpool


@pytest.fixture(scope="module")
def pool(fp):
    """2100 samples of text rows alone, in an order of ids unlike their slots'."""
    p = fp.pool_create(hidden=8, page_tokens=1, hbm_pages=1, vocab=1)
    rng = np.random.default_rng(5)
    none = np.zeros(0, np.int32)
    lens = rng.integers(1, 3000, size=2100)
    ids = [fp.pool_write_sample(p, np.zeros(n, np.int32), none, none) for n in lens]
    order = rng.permutation(len(ids))
    yield p, [ids[i] for i in order], [int(lens[i]) for i in order]
    torch.cuda.synchronize()
    fp.pool_destroy(p)


@pytest.mark.parametrize("n", [0, 1, 63, 256, 257, 959, 960, 961, 1024, 2100])
@pytest.mark.parametrize("side", [False, True])
def test_plan_equals_the_oracle(fp, pool, n, side):
    say(f"case plan n {n} side {side}")
    p, ids, lens = pool
    k, cap, n_mb = 8192, 65536, 5
    stream = torch.cuda.Stream() if side else None
    got = fp.plan_microbatches(p, ids[:n], cap, n_mb, k, stream=stream)
    assign, tok, cost = greedy_partition(lens[:n], k, cap, n_mb)
    assert got["sample_cost_scaled"].tolist() == [cost_scaled(x, k) for x in lens[:n]]
    assert got["assign"].tolist() == list(assign)
    assert got["mb_tokens"].tolist() == list(tok) and got["mb_cost_scaled"].tolist() == list(cost)


@pytest.mark.parametrize("bad,code", [
    (lambda i: i[:5] + i[2:3], "EINVAL"),                       # a sample twice
    (lambda i: i[:5] + [999999], "ENOENT"),                     # an unknown one
    (lambda i: i[:5] + i[2:3] + [999999], "EINVAL"),            # the first fault is the one reported
    (lambda i: i[:5] + [999999] + i[2:3], "ENOENT"),
    (lambda i: [999999, 999999], "ENOENT"),
    (lambda i: i[:1000] + i[999:1000], "EINVAL"),
])
def test_refused_lists_and_the_plan_after_them(fp, pool, bad, code):
    p, ids, lens = pool
    with pytest.raises(fp.FlowPoolError) as e:
        fp.plan_microbatches(p, bad(list(ids)), 65536, 4, 8192)
    assert e.value.code == code
    got = fp.plan_microbatches(p, ids[:7], 65536, 4, 8192)
    assert got["assign"].tolist() == list(greedy_partition(lens[:7], 8192, 65536, 4)[0])


def test_refusals_on_a_capturing_stream(fp, pool):
    p, ids, _ = pool
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    x = torch.zeros(64, device="cuda")
    codes = []
    with torch.cuda.graph(g, stream=s):
        x += 1
        for lst in (ids[:3], ids[:3] + ids[:1], [999999]):
            with pytest.raises(fp.FlowPoolError) as e:
                fp.plan_microbatches(p, lst, 65536, 4, 8192, stream=s)
            codes.append(e.value.code)
    assert codes == ["ESTATE", "EINVAL", "ENOENT"]
    g.replay()
    torch.cuda.synchronize()
    assert float(x.sum()) == 64.0
