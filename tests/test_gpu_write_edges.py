"""The producer's write at the edges of its launch: chunk sizes and remainders,
rows shorter and longer than a chunk, page numbers passed as the first of
consecutive pages, inline (up to 192 scattered pages) and through the staging
buffer (more), metadata blocks on both sides of one workgroup's share.

Every byte of the caller-owned tier memory is checked: rows where the page
table says they belong, everything else untouched; then a pack of the sample
checks the uploaded metadata.
"""

import numpy as np
import pytest

from gpu_common import say, to_dev, to_host
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


# hidden, page_tokens, n_vis, n_text, scattered pages, pack_cus
CASES = [
    (8, 3, 1, 0, False, 0),            # one vector
    (8, 3, 767, 5, False, 1),          # 1 vector a row: a chunk of many rows, one per lane
    (8, 1, 193, 5, True, 0),           # 193 scattered pages: the list is read from the staging buffer
    (8, 1, 192, 5, True, 0),           # 192: the largest inline list
    (104, 7, 500, 9, True, 1),         # 13 vectors a row, 64 rows a chunk
    (256, 16, 64, 64, False, 0),       # 2048 vectors
    (256, 5, 173, 1000, True, 2),      # ragged pages, more than one chunk size
    (2560, 64, 100, 3, False, 1),
    (3584, 37, 151, 4096, True, 1),    # a metadata block of more than one workgroup (4096 ids)
    (3584, 64, 97, 4091, False, 1),
    (5120, 128, 130, 2, False, 1),     # 8 KiB chunks
    (8192, 32, 65, 30, True, 1),
    (8200, 3, 40, 1, True, 0),
    (256, 16, 0, 50, False, 0),        # text only: metadata and descriptor alone
]


@pytest.mark.parametrize("hidden,page,n_vis,n_text,scatter,cus", CASES)
def test_every_byte_of_a_write(fp, hidden, page, n_vis, n_text, scatter, cus):
    say(f"case write H {hidden} P {page} vis {n_vis} text {n_text} scatter {scatter} cus {cus}")
    rng = np.random.default_rng([hidden, page, n_vis])
    need = -(-n_vis // page)
    pages = 2 * need + 3
    back = torch.full((pages * page, hidden), FILL, dtype=torch.int16, device="cuda")
    pool = fp.pool_create(hidden=hidden, page_tokens=page, hbm_pages=pages, alloc="scatter" if scatter else "contig",
                          vocab=VOCAB, hbm_backing=back, pack_cus=cus)
    try:
        none = np.zeros(0, np.int32)
        if scatter:
            # Leave the free pages in an order with no two neighbours in a row.
            ones = [fp.pool_write_sample(pool, none, [0], [page]) for _ in range(pages)]
            for i in list(range(0, pages, 2)) + list(range(1, pages, 2)):
                fp.pool_free_sample(pool, ones[i])
        text = rng.integers(0, VOCAB, size=n_text).astype(np.int32)
        ntok = np.array([n_vis // 3, n_vis - n_vis // 3] if n_vis else [], np.int32)
        pos = np.array([n_text // 2, n_text] if n_vis else [], np.int32)
        vis = tagged_vis(1, n_vis, hidden, 3) if n_vis else np.zeros((0, hidden), np.uint16)
        sid = fp.pool_write_sample(pool, text, pos, ntok, to_dev(vis) if n_vis else None)
        gvas = fp.pool_sample_pages(pool, sid).tolist() if n_vis else []
        if scatter and need > 1:
            assert any(b - a != 2 * hidden * page for a, b in zip(gvas, gvas[1:]))
        torch.cuda.synchronize()
        want = np.full((pages * page, hidden), FILL, np.uint16)
        for j, g in enumerate(gvas):
            tier, phys = fp.pool_translate(pool, g)
            assert tier == fp.FP_TIER_HBM
            row = (phys - back.data_ptr()) // (2 * hidden)
            part = vis[j * page:(j + 1) * page]
            want[row:row + len(part)] = part
        got = to_host(back)
        assert np.array_equal(got, want), np.argwhere((got != want).any(axis=1))[:5].ravel().tolist()
        table = tagged_table(VOCAB, hidden, 3)
        n = n_vis + n_text
        out = torch.zeros((n, hidden), dtype=torch.int16, device="cuda")
        cu = torch.zeros(2, dtype=torch.int32, device="cuda")
        fp.pack_microbatch(pool, [sid], to_dev(table), VOCAB, out, n, cu)
        torch.cuda.synchronize()
        parts, t, v = [], 0, 0
        for p_, k in zip(pos.tolist(), ntok.tolist()):
            parts += [table[text[t:p_]], vis[v:v + k]]
            t, v = p_, v + k
        parts.append(table[text[t:]])
        assert np.array_equal(to_host(out), np.concatenate(parts))
        assert cu.tolist() == [0, n]
    finally:
        torch.cuda.synchronize()
        fp.pool_destroy(pool)
