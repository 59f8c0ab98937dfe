"""The migration kernel over page sizes of one vector to many steps (of 256
vectors), with and without a remainder, with the last page of a sample partial;
one page and more pages than workgroups; page lists longer than a step; both
directions, partly migrated samples among them, in shuffled frames. Every byte of both tiers' caller-owned memory is checked after each
migration: moved rows at their new frames, everything else as it was; then a
pack against the definitional pack checks the uploaded page lists.
"""

import numpy as np
import pytest

from gpu_common import say, to_dev, to_host
from oracle.pack import definitional_pack
from paper_2606_23087_amd.workloads import SampleSpec
from tagging import tagged_table, tagged_vis

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOCAB = 40
FILL = 0x5A5A


@pytest.fixture(scope="module")
def fp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_23087_amd import flowpool
    return flowpool


# hidden, page_tokens, visual rows of each sample
CASES = [
    (8, 1, [1]),
    (8, 1, [300, 2]),                # a page list of more than 256 words, one-vector pages
    (8, 1000, [2500, 1, 999]),       # pages of 1000 vectors
    (8, 1024, [3000]),               # four steps a page
    (8, 1025, [3076, 1025]),         # and one vector more
    (256, 16, [5, 64, 0, 33]),
    (3584, 37, [151, 37]),
    (4096, 64, [64, 130, 1, 200]),
    (8200, 3, [40]),
]


@pytest.mark.parametrize("hidden,page,rows", CASES)
def test_every_byte_of_a_migration(fp, hidden, page, rows):
    say(f"case migrate H {hidden} P {page} rows {rows}")
    rng = np.random.default_rng([hidden, page, len(rows)])
    need = sum(-(-n // page) for n in rows)
    pages = need + 2
    back = {fp.FP_TIER_HBM: torch.full((pages * page, hidden), FILL, dtype=torch.int16, device="cuda"),
            fp.FP_TIER_HOST: torch.full((pages * page, hidden), FILL, dtype=torch.int16).pin_memory()}
    pool = fp.pool_create(hidden=hidden, page_tokens=page, hbm_pages=pages, host_pages=pages, alloc="scatter",
                          vocab=VOCAB, frame_shuffle_seed=3, hbm_backing=back[0], host_backing=back[1])
    try:
        specs, vis, ids = [], [], []
        for i, n in enumerate(rows):
            t = int(rng.integers(1, 9))
            specs.append(SampleSpec(rng.integers(0, VOCAB, size=t).astype(np.int32),
                                    np.array([t // 2], np.int32), np.array([n], np.int32)))
            vis.append(tagged_vis(i, n, hidden, 3))
            wish = rng.integers(0, 2, size=-(-n // page)).astype(np.uint8)
            ids.append(fp.pool_write_sample(pool, specs[i].text_ids, specs[i].img_pos, specs[i].img_ntok,
                                            to_dev(vis[i]) if n else None, wish))
        table = tagged_table(VOCAB, hidden, 3)
        t_dev = to_dev(table)
        ref, _, _, _ = definitional_pack(specs, vis, table)
        torch.cuda.synchronize()

        def host(t):
            return to_host(back[t]) if back[t].is_cuda else back[t].numpy().view(np.uint16)

        for tier in (fp.FP_TIER_HOST, fp.FP_TIER_HBM, fp.FP_TIER_HOST):
            want = {t: host(t).copy() for t in back}
            before = [fp.pool_sample_pages(pool, i).tolist() if n else [] for i, n in zip(ids, rows)]
            on = [[fp.pool_translate(pool, g)[0] for g in b] for b in before]
            moved = fp.pool_migrate(pool, ids, tier)
            torch.cuda.synchronize()
            assert moved == sum(t != tier for o in on for t in o)
            for i, (sid, n) in enumerate(zip(ids, rows)):
                after = fp.pool_sample_pages(pool, sid).tolist() if n else []
                for j, g in enumerate(after):
                    t, phys = fp.pool_translate(pool, g)
                    assert t == tier and (g == before[i][j]) == (on[i][j] == tier)
                    at = (phys - back[t].data_ptr()) // (2 * hidden)
                    part = vis[i][j * page:(j + 1) * page]
                    want[t][at:at + len(part)] = part
            for t in back:
                assert np.array_equal(host(t), want[t]), ("tier", t, "after migration to", tier)
            out = torch.zeros((len(ref), hidden), dtype=torch.int16, device="cuda")
            fp.pack_microbatch(pool, ids, t_dev, VOCAB, out, len(ref))
            torch.cuda.synchronize()
            assert np.array_equal(to_host(out), ref)
            assert fp.pool_reclaim(pool, wait=True) == 0
    finally:
        torch.cuda.synchronize()
        fp.pool_destroy(pool)
