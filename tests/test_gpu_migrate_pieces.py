"""The migration kernel's pieces: adjacent pages smaller than 8 steps (of 256
vectors) taken together and cut into steps, larger pages a piece each, with
pages around both sizes, pages of one vector, more steps than waves, and tiers
whose free pages are in order, in a random order and in chunks. Every byte of
both tiers' caller-owned memory is checked after each migration, and a pack
against the definitional pack checks the uploaded page lists.
"""

import numpy as np
import pytest

from gpu_common import say, to_dev, to_host
from oracle.pack import definitional_pack
from paper_2606_23087_amd.workloads import SampleSpec
from tagging import tagged_table, tagged_vis

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOCAB, FILL = 40, 0x5A5A


@pytest.fixture(scope="module")
def fp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_23087_amd import flowpool
    return flowpool


# hidden, page_tokens, visual rows of each sample
CASES = [
    (8, 1, [1, 700, 2, 513]),            # one-vector pages
    (8, 255, [1000, 255, 1]),
    (8, 256, [2560, 257, 256]),          # pages of one step
    (8, 257, [2600, 1, 600]),
    (8, 2047, [9000, 2047]),             # pages just under 8 steps, cut where adjacent
    (8, 2048, [9000, 2048]),             # 8 steps: a piece a page
    (8, 2049, [9000, 2050]),             # a last step of one vector
    (256, 16, [3000, 5, 1601]),          # 8 KiB pages, more steps than waves
    (1000, 7, [200, 64]),
]


@pytest.mark.parametrize("hidden,page,rows", CASES)
@pytest.mark.parametrize("shuffle", [0, 5])
def test_every_byte_moves_once(fp, hidden, page, rows, shuffle):
    say(f"case migrate pieces H {hidden} P {page} rows {rows} shuffle {shuffle}")
    rng = np.random.default_rng([hidden, page, len(rows)])
    pages = sum(-(-n // page) for n in rows) + 2
    back = {fp.FP_TIER_HBM: torch.full((pages * page, hidden), FILL, dtype=torch.int16, device="cuda"),
            fp.FP_TIER_HOST: torch.full((pages * page, hidden), FILL, dtype=torch.int16).pin_memory()}
    pool = fp.pool_create(hidden=hidden, page_tokens=page, hbm_pages=pages, host_pages=pages, alloc="scatter",
                          vocab=VOCAB, frame_shuffle_seed=shuffle, hbm_backing=back[0], host_backing=back[1])
    try:
        specs = [SampleSpec(rng.integers(0, VOCAB, size=3).astype(np.int32), np.array([1], np.int32),
                            np.array([n], np.int32)) for n in rows]
        vis = [tagged_vis(i, n, hidden, 3) for i, n in enumerate(rows)]
        ids = [fp.pool_write_sample(pool, s.text_ids, s.img_pos, s.img_ntok, to_dev(v)) for s, v in zip(specs, vis)]
        table = tagged_table(VOCAB, hidden, 3)
        t_dev = to_dev(table)
        ref, _, _, _ = definitional_pack(specs, vis, table)
        torch.cuda.synchronize()

        def bytes_of(t):
            return to_host(back[t]) if back[t].is_cuda else back[t].numpy().view(np.uint16)

        def expect(want, sid, rows_of, tier):
            for j, g in enumerate(fp.pool_sample_pages(pool, sid).tolist()):
                t, phys = fp.pool_translate(pool, g)
                assert t == tier
                at = (phys - back[t].data_ptr()) // (2 * hidden)
                part = rows_of[j * page:(j + 1) * page]
                want[t][at:at + len(part)] = part

        def check_pack():
            out = torch.zeros((len(ref), hidden), dtype=torch.int16, device="cuda")
            fp.pack_microbatch(pool, ids, t_dev, VOCAB, out, len(ref))
            torch.cuda.synchronize()
            assert np.array_equal(to_host(out), ref)

        # all down, one up (its pages between the others'), all up, and twice round
        for some, tier in ((ids, 1), (ids[:1], 0), (ids, 0), (ids[1:], 1), (ids, 1), (ids, 0)):
            want = {t: bytes_of(t).copy() for t in back}
            fp.pool_migrate(pool, some, tier)
            torch.cuda.synchronize()
            for sid in some:
                expect(want, sid, vis[ids.index(sid)], tier)
            for t in back:
                assert np.array_equal(bytes_of(t), want[t]), ("tier", t, "after migration to", tier)
            check_pack()
            assert fp.pool_reclaim(pool, wait=True) == 0
    finally:
        torch.cuda.synchronize()
        fp.pool_destroy(pool)
