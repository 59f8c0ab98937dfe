"""Where a pack's run table goes: the compact kernel arguments, the general
ones with 64 or as few as 16 buckets, or a device copy (4 bytes a sample, 16
a run, 18 a bucket, in 704 or 3840 bytes of arguments). Packs on both sides of
each limit, through both entry points, against the definitional pack; more
device-copied tables in flight than there are staging buffers, on two streams;
and what a HIP graph refuses to capture stays refused.
"""

import numpy as np
import pytest

from gpu_common import say, to_dev, to_host
from oracle.pack import definitional_pack
from paper_2606_23087_amd.workloads import SampleSpec
from tagging import tagged_table, tagged_vis

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

H, P, VOCAB = 64, 4, 50


@pytest.fixture(scope="module")
def fp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_23087_amd import flowpool
    return flowpool


class _Pool:
    """1-run samples (text only) 0..249, then 3-run samples (text, image, text) 250..349."""

    def __init__(self, fp):
        rng = np.random.default_rng(11)
        self.fp, self.specs, self.vis = fp, [], []
        self.pool = fp.pool_create(hidden=H, page_tokens=P, hbm_pages=400, vocab=VOCAB, pack_cus=1)
        self.table = tagged_table(VOCAB, H, 2)
        self.t_dev = to_dev(self.table)
        none = np.zeros(0, np.int32)
        self.ids = []
        for i in range(350):
            n_text = int(rng.integers(2, 30))
            text = rng.integers(0, VOCAB, size=n_text).astype(np.int32)
            img = i >= 250
            s = SampleSpec(text, np.array([1 + n_text // 3], np.int32) if img else none,
                           rng.integers(1, 12, size=1).astype(np.int32) if img else none)
            v = tagged_vis(i, s.n_vis, H, 2)
            self.specs.append(s)
            self.vis.append(v)
            self.ids.append(fp.pool_write_sample(self.pool, s.text_ids, s.img_pos, s.img_ntok,
                                                 to_dev(v) if s.n_vis else None))
        torch.cuda.synchronize()

    def outs(self, g):
        n = sum(self.specs[i].length for i in g)
        return (torch.full((n + 3, H), 0x5A5A, dtype=torch.int16, device="cuda"),
                torch.full((len(g) + 1,), -1, dtype=torch.int32, device="cuda"),
                torch.full((n + 3,), -1, dtype=torch.int32, device="cuda"))

    def pack(self, g, out, entry, stream=None):
        entry(self.pool, [self.ids[i] for i in g], self.t_dev, VOCAB, out[0], out[0].shape[0], out[1], out[2],
              stream=stream)

    def check(self, g, out):
        ref, cu, pos, _ = definitional_pack([self.specs[i] for i in g], [self.vis[i] for i in g], self.table)
        n = len(ref)
        assert np.array_equal(to_host(out[0][:n]), ref)
        assert bool((out[0][n:] == 0x5A5A).all()) and out[2][n:].tolist() == [-1] * 3
        assert np.array_equal(out[1].cpu().numpy(), cu) and np.array_equal(out[2][:n].cpu().numpy(), pos)


@pytest.fixture(scope="module")
def w(fp):
    p = _Pool(fp)
    yield p
    torch.cuda.synchronize()
    fp.pool_destroy(p.pool)


# text-only samples: 20 bytes each and 16 buckets: 20 n + 288 <= 704 (n <= 20, lengths padded to 16 bytes),
# 20 n + 1152 <= 3840 (n <= 134 with 64 buckets), 20 n + 288 <= 3840 (n <= 177)
TEXT = [1, 20, 21, 22, 33, 133, 134, 135, 176, 177, 178, 250]
# text-image-text samples: 52 bytes each: 8, 51, 68
IMAGE = [7, 8, 9, 50, 51, 52, 67, 68, 69, 100]


@pytest.mark.parametrize("first,n", [(0, k) for k in TEXT] + [(250, k) for k in IMAGE])
def test_run_table_limits(fp, w, first, n):
    say(f"case run table: {n} samples from {first}")
    g = list(range(first, first + n))
    for entry in (fp.pack_microbatch, fp.pack_microbatch_noalloc):
        out = w.outs(g)
        w.pack(g, out, entry)
        torch.cuda.synchronize()
        w.check(g, out)


def test_many_device_tables_in_flight(fp, w):
    say("case device-copied run tables: 24 packs in flight on two streams")
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    rng = np.random.default_rng(4)
    groups = [rng.permutation(350)[:int(rng.integers(180, 340))].tolist() for _ in range(24)]
    outs = [w.outs(g) for g in groups]
    torch.cuda.synchronize()
    for k, (g, o) in enumerate(zip(groups, outs)):
        w.pack(g, o, fp.pack_microbatch, streams[k % 2])
    torch.cuda.synchronize()
    for g, o in zip(groups, outs):
        w.check(g, o)
    outs = [w.outs(g) for g in groups]
    torch.cuda.synchronize()
    for g, o in zip(groups, outs):              # one stream: every call overwrites the shared scratch
        w.pack(g, o, fp.pack_microbatch_noalloc, streams[0])
    torch.cuda.synchronize()
    for g, o in zip(groups, outs):
        w.check(g, o)
    for s in streams:
        fp.pool_forget_stream(w.pool, s)


@pytest.mark.filterwarnings("ignore:The CUDA Graph is empty")     # a refused capture records nothing
def test_capture_limits_are_unchanged(fp, w):
    say("case capture: 33 samples, and 54 samples of 162 runs, are refused; 32 samples are captured")
    fp.pool_reclaim(w.pool, wait=True)
    stream = torch.cuda.Stream()
    for g, ok in ((list(range(32)), True), (list(range(33)), False), (list(range(250, 304)), False)):
        out = w.outs(g)
        w.pack(g, out, fp.pack_microbatch, stream)
        torch.cuda.synchronize()
        out[0].fill_(0x5A5A)
        graph = torch.cuda.CUDAGraph()
        if ok:
            with torch.cuda.graph(graph, stream=stream):
                w.pack(g, out, fp.pack_microbatch)
            for _ in range(3):
                out[0][:-3].zero_()
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                w.check(g, out)
            fp.pool_release_captured(w.pool, [w.ids[i] for i in g])
        else:
            with torch.cuda.graph(graph, stream=stream):
                with pytest.raises(fp.FlowPoolError) as e:
                    w.pack(g, out, fp.pack_microbatch)
            assert e.value.code == "ESTATE"
    torch.cuda.synchronize()
    fp.pool_forget_stream(w.pool, stream)
