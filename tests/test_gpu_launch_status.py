"""Calls made while the thread holds an error of an earlier HIP call (here the
caller's own, a device that does not exist): writes, migrations in both
directions, plans and packs, with the run table in the kernel arguments and
copied to the device, are enqueued once, succeed and are right.
"""

import numpy as np
import pytest

from gpu_common import say, to_dev, to_host
from oracle.pack import definitional_pack
from oracle.plan import greedy_partition
from paper_2606_23087_amd.workloads import SampleSpec
from tagging import tagged_table, tagged_vis

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

H, P, VOCAB, N = 64, 4, 50, 90


@pytest.fixture(scope="module")
def fp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_23087_amd import flowpool
    return flowpool


def test_calls_with_an_error_pending(fp):
    say(f"case error pending: {N} samples written, migrated, planned and packed")
    hip = fp._lib                       # the HIP runtime the library is bound to, through its handle
    rng = np.random.default_rng(3)
    specs = [SampleSpec(rng.integers(0, VOCAB, size=5).astype(np.int32), np.array([2], np.int32),
                        np.array([int(rng.integers(1, 12))], np.int32)) for _ in range(N)]
    vis = [tagged_vis(i, s.n_vis, H, 2) for i, s in enumerate(specs)]
    dev = [to_dev(v) for v in vis]
    table = tagged_table(VOCAB, H, 2)
    t_dev = to_dev(table)
    pages = sum(-(-s.n_vis // P) for s in specs)
    pool = fp.pool_create(hidden=H, page_tokens=P, hbm_pages=pages, host_pages=pages, alloc="scatter", vocab=VOCAB)
    stream = torch.cuda.Stream()
    rows = sum(s.length for s in specs)

    def outs(n):
        return (torch.full((rows, H), 0x5A5A, dtype=torch.int16, device="cuda"),
                torch.full((n + 1,), -1, dtype=torch.int32, device="cuda"),
                torch.full((rows,), -1, dtype=torch.int32, device="cuda"))

    groups = [[3, 1, 2], list(range(N)), list(range(N - 1, 4, -1))]       # 9 runs; 270 and 255: copied to the device
    entries = [fp.pack_microbatch, fp.pack_microbatch, fp.pack_microbatch_noalloc]
    got = [outs(len(g)) for g in groups]
    torch.cuda.synchronize()
    try:
        assert hip.hipSetDevice(99) != 0 and hip.hipPeekAtLastError() != 0
        ids = [fp.pool_write_sample(pool, s.text_ids, s.img_pos, s.img_ntok, d, stream=stream)
               for s, d in zip(specs, dev)]
        assert hip.hipSetDevice(99) != 0
        assert fp.pool_migrate(pool, ids, fp.FP_TIER_HOST, stream=stream) == pages
        assert hip.hipSetDevice(99) != 0
        assert fp.pool_migrate(pool, ids[:40], fp.FP_TIER_HBM, stream=stream) > 40
        assert hip.hipSetDevice(99) != 0
        plan = fp.plan_microbatches(pool, ids, 4096, 3, 512, stream=stream)
        for g, o, entry in zip(groups, got, entries):
            assert hip.hipSetDevice(99) != 0
            entry(pool, [ids[i] for i in g], t_dev, VOCAB, o[0], rows, o[1], o[2], stream=stream)
        hip.hipGetLastError()           # cleared before torch's own calls look at it
        torch.cuda.synchronize()
        assert plan["assign"].tolist() == list(greedy_partition([s.length for s in specs], 512, 4096, 3)[0])
        for g, o in zip(groups, got):
            want, cu, pos, _ = definitional_pack([specs[i] for i in g], [vis[i] for i in g], table)
            n = len(want)
            assert np.array_equal(to_host(o[0][:n]), want) and bool((o[0][n:] == 0x5A5A).all())
            assert np.array_equal(o[1].cpu().numpy(), cu) and np.array_equal(o[2][:n].cpu().numpy(), pos)
        fp.pool_reclaim(pool, wait=True)
        assert fp.pool_stats(pool)["n_samples"] == N
    finally:
        hip.hipGetLastError()
        torch.cuda.synchronize()
        fp.pool_destroy(pool)
