"""The pages a migration leaves behind wait for the packs that read them, each
sample for its own reader streams, though the call looks at each stream once
for all samples: samples read by one of two streams, by both, by none, and by
the migration's own stream, with each stream's packs ending at its own time.
The packs queued before the migration read the old pages, which a write takes
over as soon as they are back.
"""

import numpy as np
import pytest

from gpu_common import say, to_dev, to_host
from oracle.pack import definitional_pack
from paper_2606_23087_amd.workloads import SampleSpec
from tagging import tagged_table, tagged_vis

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

H, P, VOCAB = 512, 16, 40
READERS = [(), ("a",), ("b",), ("a", "b"), ("m",), ("m", "b"), ("b",), ("a",)]


@pytest.fixture(scope="module")
def fp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_23087_amd import flowpool
    return flowpool


@pytest.mark.parametrize("to_host_tier", [True, False])
def test_each_sample_waits_for_its_own_readers(fp, to_host_tier):
    say(f"case migrate readers, to the host tier {to_host_tier}")
    rng = np.random.default_rng(8)
    rows = [P * (1 + i % 3) for i in range(len(READERS))]
    pages = [n // P for n in rows]
    total = sum(pages)
    pool = fp.pool_create(hidden=H, page_tokens=P, hbm_pages=2 * total, host_pages=2 * total, alloc="scatter",
                          vocab=VOCAB)
    streams = {k: torch.cuda.Stream() for k in "abm"}
    try:
        table = tagged_table(VOCAB, H, 8)
        t_dev = to_dev(table)
        specs, vis, ids = [], [], []
        for i, n in enumerate(rows):
            specs.append(SampleSpec(rng.integers(0, VOCAB, size=5).astype(np.int32), np.array([2], np.int32),
                                    np.array([n], np.int32)))
            vis.append(tagged_vis(i, n, H, 8))
            ids.append(fp.pool_write_sample(pool, specs[i].text_ids, specs[i].img_pos, specs[i].img_ntok,
                                            to_dev(vis[i]), np.full(pages[i], 0 if to_host_tier else 1, np.uint8)))
        big = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
        other = torch.empty_like(big)
        torch.cuda.synchronize()
        assert fp.pool_reclaim(pool) == 0
        outs = {}
        for k in streams:
            mine = [i for i, r in enumerate(READERS) if k in r]
            n = sum(specs[i].length for i in mine)
            outs[k] = (mine, torch.zeros((n, H), dtype=torch.int16, device="cuda"))
        torch.cuda.synchronize()
        # "b" stays busy for some 40 ms, "a" and the migration's own stream for a few.
        for k, copies in (("b", 100), ("a", 8), ("m", 4)):
            with torch.cuda.stream(streams[k]):
                for _ in range(copies):
                    other.copy_(big)
            mine, out = outs[k]
            fp.pack_microbatch(pool, [ids[i] for i in mine], t_dev, VOCAB, out, out.shape[0], stream=streams[k])
        moved = fp.pool_migrate(pool, ids, fp.FP_TIER_HOST if to_host_tier else fp.FP_TIER_HBM, stream=streams["m"])
        assert moved == total
        assert fp.pool_reclaim(pool) == total, "everything waits for the copies"
        streams["m"].synchronize()
        streams["a"].synchronize()
        held = sum(n for n, r in zip(pages, READERS) if "b" in r)
        assert not streams["b"].query() and fp.pool_reclaim(pool) == held
        # A write that takes the pages that are back, on the migration's stream.
        fresh = [fp.pool_write_sample(pool, specs[0].text_ids, specs[0].img_pos, np.array([P], np.int32),
                                      to_dev(tagged_vis(90, P, H, 9)),
                                      np.full(1, 0 if to_host_tier else 1, np.uint8), stream=streams["m"])
                 for _ in range(total - held)]
        streams["b"].synchronize()
        assert fp.pool_reclaim(pool) == 0
        torch.cuda.synchronize()
        for k, (mine, out) in outs.items():
            ref = definitional_pack([specs[i] for i in mine], [vis[i] for i in mine], table)[0]
            assert np.array_equal(to_host(out), ref), f"pack on stream {k}"
        out = torch.zeros((sum(s.length for s in specs), H), dtype=torch.int16, device="cuda")
        fp.pack_microbatch(pool, ids, t_dev, VOCAB, out, out.shape[0])
        torch.cuda.synchronize()
        assert np.array_equal(to_host(out), definitional_pack(specs, vis, table)[0])
        assert len(fresh) == total - held
    finally:
        torch.cuda.synchronize()
        fp.pool_destroy(pool)
