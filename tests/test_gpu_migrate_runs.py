"""Migrations of runs of adjacent pages around 8 MiB, from which on a run is one
copy by the DMA engines beside the kernel's pieces: runs just under, at and past
it, over several samples, with a partial last page, cut by the ends of the
backing's chunks, and pages of that size by themselves. Rows are checked in both
tiers' caller-owned memory, every byte of it, or, where the library allocates it
in chunks, through packs; packs on another stream read the pages before, during
and after.
"""

import numpy as np
import pytest

from gpu_common import say, to_dev, to_host
from oracle.pack import definitional_pack
from paper_2606_23087_amd.workloads import SampleSpec
from tagging import tagged_table, tagged_vis

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOCAB, FILL = 20, 0x5A5A


@pytest.fixture(scope="module")
def fp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_23087_amd import flowpool
    return flowpool


# hidden, page_tokens, visual rows of each sample, bytes of a chunk (0: the caller's memory)
CASES = [
    (4096, 64, [1024, 1023, 960, 30, 64, 1100], 0),      # 8 MiB, a row less, 7.5 MiB; some across two samples
    (4096, 64, [1024, 2048, 700], 3 << 20),              # 3 MiB chunks: no run as long as that
    (4096, 64, [1024, 2048, 700], 9 << 20),
    (256, 16, [16384 + 1600, 16383, 50], 0),             # 8 KiB pages
    (4096, 1024, [1024, 2500], 0),                       # pages of 8 MiB
]


@pytest.mark.parametrize("hidden,page,rows,chunk", CASES)
def test_long_runs(fp, hidden, page, rows, chunk):
    say(f"case migrate runs H {hidden} P {page} rows {rows} chunk {chunk}")
    pages = sum(-(-n // page) for n in rows) + 1
    back = {}
    if not chunk:
        back = {0: torch.full((pages * page, hidden), FILL, dtype=torch.int16, device="cuda"),
                1: torch.full((pages * page, hidden), FILL, dtype=torch.int16).pin_memory()}
    pool = fp.pool_create(hidden=hidden, page_tokens=page, hbm_pages=pages, host_pages=pages, alloc="scatter",
                          vocab=VOCAB, chunk_bytes=chunk, hbm_backing=back.get(0), host_backing=back.get(1))
    side = torch.cuda.Stream()
    try:
        specs = [SampleSpec(np.array([1, 2], np.int32), np.array([1], np.int32), np.array([n], np.int32)) for n in rows]
        vis = [tagged_vis(i, n, hidden, 3) for i, n in enumerate(rows)]
        ids = [fp.pool_write_sample(pool, s.text_ids, s.img_pos, s.img_ntok, to_dev(v)) for s, v in zip(specs, vis)]
        table = tagged_table(VOCAB, hidden, 3)
        t_dev = to_dev(table)
        ref = definitional_pack(specs, vis, table)[0]
        outs = [torch.zeros((len(ref), hidden), dtype=torch.int16, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        fp.pool_reclaim(pool, wait=True)

        def bytes_of(t):
            return to_host(back[t]) if back[t].is_cuda else back[t].numpy().view(np.uint16)

        for some, tier in ((ids, 1), (ids, 0), (ids[::2], 1), (ids, 1), (ids[:2], 0), (ids, 0)):
            want = {t: bytes_of(t).copy() for t in back}
            for o in outs:
                o.zero_()
            torch.cuda.synchronize()
            fp.pack_microbatch(pool, ids, t_dev, VOCAB, outs[0], len(ref), stream=side)
            fp.pool_migrate(pool, some, tier)
            fp.pack_microbatch(pool, ids, t_dev, VOCAB, outs[1], len(ref), stream=side)
            torch.cuda.synchronize()
            for o in outs:
                assert np.array_equal(to_host(o), ref), (some, tier)
            for sid in some if back else ():
                rows_of = vis[ids.index(sid)]
                for j, g in enumerate(fp.pool_sample_pages(pool, sid).tolist()):
                    t, phys = fp.pool_translate(pool, g)
                    assert t == tier
                    at = (phys - back[t].data_ptr()) // (2 * hidden)
                    part = rows_of[j * page:(j + 1) * page]
                    want[t][at:at + len(part)] = part
            for t in back:
                assert np.array_equal(bytes_of(t), want[t]), ("tier", t, "after migration to", tier)
            assert fp.pool_reclaim(pool, wait=True) == 0
    finally:
        torch.cuda.synchronize()
        fp.pool_forget_stream(pool, side)
        fp.pool_destroy(pool)
