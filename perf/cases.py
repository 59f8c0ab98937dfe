"""Performance cases of flowpool: what a training program has the library do,
through the public Python entry points (paper_2606_23087_amd.flowpool).

A training program on one GPU does five things with a pool, and each is a kind
of case here:

  pack      the backbone packs the microbatches of one plan, one call each;
  write     a producer (a frozen encoder) writes samples into the pool while
            the ones it wrote two batches ago are freed;
  plan      the resident samples' costs are evaluated and partitioned;
  step      a whole batch's life in one pass: write, plan, pack, free;
  prefetch  samples that live on the host tier are promoted to HBM, packed
            and demoted again.

All outputs are copied rows and whole numbers, so every tolerance is "exact".
"""

import math
import weakref

import numpy as np
import torch

from paper_2606_23087_amd import flowpool as fp

# Everything a case can state; listed() and draw() override the rest.
_DEFAULTS = dict(
    kind="pack", hidden=3584, page_tokens=64, alloc="contig", fragmented=False, host_share=0.0, vocab=152064,
    capacity=16384, n_mb=4, cost_k=8192, zigzag=False, noalloc=False, samples=0,
    images_lo=1, images_hi=4, image_rows_lo=256, image_rows_hi=1280, image_rows_step=4,
    text="lognormal", text_a=400.0, text_b=0.8, text_lo=16, text_hi=4096,
)


def _case(name=None, **kw):
    c = dict(_DEFAULTS, **kw)
    assert set(c) == set(_DEFAULTS)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest packs: 2 microbatches of 4 samples, hidden 256. Launch latency and host time.
        _case("pack_tiny", hidden=256, page_tokens=16, vocab=1000, capacity=512, n_mb=2, cost_k=4096, samples=8,
              images_hi=1, image_rows_lo=64, image_rows_hi=64, image_rows_step=1, text="uniform", text_a=32, text_b=128),
        # A small backbone with short microbatches: each pack moves a few tens of MB.
        _case("pack_mid", hidden=2560, capacity=4096, n_mb=8, image_rows_hi=1024, text_a=256.0),
        # The ordinary step of a VLM backbone of hidden size 3584 (the benchmark's headline workload).
        _case("pack_qwen"),
        # Many short samples (short questions, small or no images) in the same microbatch size: some 90 a pack.
        _case("pack_short", images_lo=0, images_hi=1, image_rows_lo=16, image_rows_hi=256, image_rows_step=1,
              text_a=96.0, text_lo=32, text_hi=512),
        # A 70B-class backbone over a pool whose pages are scattered by earlier writes and frees.
        _case("pack_frag70b", hidden=8192, page_tokens=32, alloc="scatter", fragmented=True, capacity=32768, n_mb=2,
              cost_k=4096, images_hi=6, image_rows_lo=196, image_rows_hi=1024, image_rows_step=1, text_a=600.0,
              text_b=1.0, text_hi=8192),
        # The largest packs: long videos, through the entry point for loops that must not allocate.
        _case("pack_video", hidden=5120, page_tokens=128, vocab=128256, capacity=65536, n_mb=2, cost_k=4096,
              noalloc=True, images_hi=1, image_rows_lo=2048, image_rows_hi=8192, image_rows_step=256, text="uniform",
              text_a=64, text_b=2048),
        # Half of the pages in pinned host memory, read by the pack over PCIe.
        _case("pack_tiered", hidden=4096, alloc="scatter", host_share=0.5, n_mb=1, image_rows_hi=1024,
              image_rows_step=1, text_a=512.0),
        # A producer writing small samples, 8 a batch: the latency of a write.
        _case("write_tiny", kind="write", hidden=256, page_tokens=16, vocab=1000, samples=8, images_hi=1,
              image_rows_lo=64, image_rows_hi=64, image_rows_step=1, text="uniform", text_a=32, text_b=128),
        # A producer writing a batch of ordinary samples (some 14 MB of image rows each).
        _case("write_qwen", kind="write", samples=16),
        # One plan of a step: some 430 resident samples into 64 microbatches.
        _case("plan_qwen", kind="plan", n_mb=64),
        # A batch from the encoder's output to the packed microbatches, and its samples' release.
        _case("step_qwen", kind="step", n_mb=4),
        # Host-tier samples brought into HBM ahead of their pack, and put back.
        _case("prefetch_tiered", kind="prefetch", hidden=4096, alloc="scatter", host_share=0.5, n_mb=1, samples=7,
              image_rows_hi=1024, image_rows_step=1, text_a=512.0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """A case of the same ranges: hidden 256 to 8192, pages of 16 to 128 rows, microbatches of 512 to 65536 rows."""
    kind = rng.choice(["pack"] * 5 + ["write"] * 2 + ["plan", "step", "prefetch"])
    hidden = 8 * int(_log(rng, 32, 1024.99))
    page_tokens = rng.choice([16, 32, 64, 128, rng.randint(16, 128)])
    c = dict(kind=kind, hidden=hidden, page_tokens=page_tokens, vocab=rng.choice([1000, 32003, 128256, 152064]))
    c["text_b"] = round(rng.uniform(0.5, 1.0), 2)
    c["image_rows_step"] = rng.choice([1, 1, 4])
    most = 335_000_000 // hidden                       # rows of one microbatch: at most 670 MB
    style = rng.choice(["short", "ordinary", "ordinary", "video"])
    if style == "short":
        c.update(images_lo=rng.randint(0, 1), images_hi=rng.randint(1, 2), image_rows_lo=rng.randint(1, 64),
                 image_rows_hi=rng.randint(64, 256), text_a=float(rng.randint(48, 200)), text_lo=24, text_hi=512)
        most = min(most, 16384)
    elif style == "ordinary":
        c.update(images_hi=rng.randint(1, 6), image_rows_lo=rng.randint(64, 256), image_rows_hi=rng.randint(600, 1280),
                 text_a=float(rng.randint(200, 700)))
    else:
        c.update(images_hi=1, image_rows_lo=2048, image_rows_hi=rng.randint(4096, 8192), text="uniform", text_a=64,
                 text_b=2048)
    c["capacity"] = int(_log(rng, 512 if style == "short" else 2048 if style == "ordinary" else 12288, most))
    if kind == "pack":
        c.update(alloc=rng.choice(["contig", "contig", "scatter"]), n_mb=rng.choice([1, 2, 2, 4]),
                 noalloc=rng.random() < 0.3)
        c["fragmented"] = c["alloc"] == "scatter"
        if c["n_mb"] == 4 and c["capacity"] * hidden > 64_000_000:
            c["n_mb"] = 2
        if c["alloc"] == "scatter" and rng.random() < 0.3:
            c.update(host_share=round(rng.uniform(0.1, 0.6), 2), n_mb=1, capacity=min(c["capacity"], 16384))
    elif kind == "write":
        c.update(samples=rng.randint(1, 16))
    elif kind == "plan":
        c.update(n_mb=rng.randint(8, 64), capacity=min(c["capacity"], 16384), zigzag=rng.random() < 0.5)
        if style == "video":
            c["capacity"] = 16384
    elif kind == "step":
        c.update(n_mb=rng.randint(1, 4), capacity=max(2048, min(c["capacity"], 60_000_000 // hidden)))
        if style == "video":
            c["capacity"] = 16384
    else:
        c.update(alloc="scatter", host_share=round(rng.uniform(0.2, 0.6), 2), n_mb=1, samples=rng.randint(2, 6))
    return _case(**c)


# ------------------------------------------------------------------ inputs

class _Sample:
    def __init__(self, text_ids, img_pos, img_ntok):
        self.text_ids, self.img_pos, self.img_ntok = text_ids, img_pos, img_ntok
        self.n_vis = int(img_ntok.sum())
        self.length = len(text_ids) + self.n_vis


def _samples(case, seed):
    """The samples in write order: case["samples"] of them, or as many as it takes to fill the plan's microbatches.
    Their sizes belong to the case, so every seed has the same work; their order, ids and image positions are the seed's."""
    rng, ids = np.random.default_rng(0x5A), np.random.default_rng([int(seed), 0x1D])
    out, total = [], 0
    want = case["capacity"] * case["n_mb"]
    while len(out) < case["samples"] if case["samples"] else total < want:
        if case["text"] == "uniform":
            n_text = int(rng.integers(int(case["text_a"]), int(case["text_b"]) + 1))
        else:
            n_text = int(case["text_a"] * math.exp(case["text_b"] * rng.standard_normal()) + 0.5)
            n_text = min(max(n_text, case["text_lo"]), case["text_hi"])
        k = int(rng.integers(case["images_lo"], case["images_hi"] + 1))
        step = case["image_rows_step"]
        steps = max(0, case["image_rows_hi"] - case["image_rows_lo"]) // step
        ntok = (case["image_rows_lo"] + step * rng.integers(0, steps + 1, size=k)).astype(np.int32)
        pos = np.sort(ids.integers(0, n_text + 1, size=k)).astype(np.int32)
        out.append(_Sample(ids.integers(0, case["vocab"], size=n_text).astype(np.int32), pos, ntok))
        total += out[-1].length
    return [out[i] for i in ids.permutation(len(out))]


def _generator(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 0x9E3779B1 + what) & ((1 << 62) - 1))
    return g


def _table(case, seed):
    t = torch.empty((case["vocab"], case["hidden"]), dtype=torch.bfloat16, device="cuda")
    return t.normal_(0.0, 0.02, generator=_generator(seed, 1))


def _vis(case, seed, i, n_vis):
    """The encoder's output for sample i."""
    v = torch.empty((n_vis, case["hidden"]), dtype=torch.bfloat16, device="cuda")
    return v.normal_(0.0, 1.0, generator=_generator(seed, 2 + i))


def _tiers(case, seed, i, n_pages):
    return (np.random.default_rng([int(seed), 0x71, i]).random(n_pages) < case["host_share"]).astype(np.uint8)


def _pages(case, s):
    return -(-s.n_vis // case["page_tokens"])


def _destroy(pool):
    torch.cuda.synchronize()
    fp.pool_destroy(pool)


class _Pool:
    """A pool handle that is destroyed with its state."""

    def __init__(self, case, hbm_pages, host_pages=0, **kw):
        self.handle = fp.pool_create(hidden=case["hidden"], page_tokens=case["page_tokens"], hbm_pages=hbm_pages,
                                     host_pages=host_pages, alloc=case["alloc"], vocab=case["vocab"], **kw)
        weakref.finalize(self, _destroy, self.handle)


def _scatter_free_pages(case, pool, pages, seed):
    """Leaves the pool's free pages in a random order, as a long run of writes and frees does."""
    rng = np.random.default_rng([int(seed), 0xF4])
    ids, none = [], np.zeros(0, np.int32)
    while pages > 0:
        k = min(pages, int(rng.integers(1, 9)))
        rows = np.array([k * case["page_tokens"]], np.int32)
        ids.append(fp.pool_write_sample(pool, none, np.zeros(1, np.int32), rows))
        pages -= k
    for i in rng.permutation(len(ids)):
        fp.pool_free_sample(pool, ids[i])


def _write(case, seed, pool, samples, vis):
    ids = []
    for i, s in enumerate(samples):
        wish = _tiers(case, seed, i, _pages(case, s)) if case["host_share"] else None
        ids.append(fp.pool_write_sample(pool, s.text_ids, s.img_pos, s.img_ntok, vis(i, s), wish))
    return ids


def _plan(case, pool, ids):
    return fp.plan_microbatches(pool, ids, case["capacity"], case["n_mb"], case["cost_k"],
                                policy=fp.FP_PLAN_ZIGZAG if case["zigzag"] else fp.FP_PLAN_LPT)


def _groups(ids, assign, n_mb):
    out = [[] for _ in range(n_mb)]
    for i, j in zip(ids, assign):
        if j >= 0:
            out[j].append(i)
    return out


def _outputs(case, samples):
    """Buffers of every microbatch: rows, cu_seqlens, position ids."""
    rows = case["capacity"] if case["kind"] != "prefetch" else sum(s.length for s in samples)
    return [(torch.zeros((rows, case["hidden"]), dtype=torch.bfloat16, device="cuda"),
             torch.zeros(len(samples) + 1, dtype=torch.int32, device="cuda"),
             torch.zeros(rows, dtype=torch.int32, device="cuda")) for _ in range(case["n_mb"])]


def prepare(case, seed):
    samples = _samples(case, seed)
    pages = sum(_pages(case, s) for s in samples)
    st = dict(case=case, samples=samples)
    kind = case["kind"]

    def encoder(i, s):
        return _vis(case, seed, i, s.n_vis) if s.n_vis else None

    if kind == "write":
        # Two batches are resident and a third is being written; the caller owns the memory behind the pages.
        total = 3 * max(pages, 1)
        backing = torch.zeros((total * case["page_tokens"], case["hidden"]), dtype=torch.bfloat16, device="cuda")
        st.update(pool=_Pool(case, total, hbm_backing=backing), backing=backing, batches=[],
                  vis=[encoder(i, s) for i, s in enumerate(samples)])
    elif kind == "step":
        st.update(pool=_Pool(case, 3 * max(pages, 1)), vis=[encoder(i, s) for i, s in enumerate(samples)],
                  table=_table(case, seed), outputs=_outputs(case, samples))
    elif kind == "plan":
        st["pool"] = _Pool(dict(case, hidden=8), max(pages, 1))      # the row size plays no part in a plan
        st["ids"] = [fp.pool_write_sample(st["pool"].handle, s.text_ids, s.img_pos, s.img_ntok) for s in samples]
    else:
        host = 2 * pages if case["host_share"] else 0
        hbm = (2 if case["fragmented"] or host else 1) * max(pages, 1)
        st["pool"] = _Pool(case, hbm, host)
        if case["fragmented"]:
            _scatter_free_pages(case, st["pool"].handle, hbm, seed)
        st["ids"] = _write(case, seed, st["pool"].handle, samples, encoder)
        st.update(table=_table(case, seed), outputs=_outputs(case, samples))
        if kind == "prefetch":
            st["groups"] = [st["ids"]]
            fp.pool_migrate(st["pool"].handle, st["ids"], fp.FP_TIER_HOST)
        else:
            plan = _plan(case, st["pool"].handle, st["ids"])
            st["groups"] = _groups(st["ids"], plan["assign"].tolist(), case["n_mb"])
    torch.cuda.synchronize()
    return st


# ------------------------------------------------------------------ one pass

def _pack_all(case, pool, st, groups):
    pack = fp.pack_microbatch_noalloc if case["noalloc"] else fp.pack_microbatch
    for ids, (rows, cu, pos) in zip(groups, st["outputs"]):
        pack(pool, ids, st["table"], case["vocab"], rows, rows.shape[0], cu, pos)
    return st["outputs"]


def _run_pack(case, pool, st):
    return _pack_all(case, pool, st, st["groups"])


def _run_write(case, pool, st):
    if len(st["batches"]) == 2:
        for i in st["batches"].pop(0):
            fp.pool_free_sample(pool, i)
    st["batches"].append([fp.pool_write_sample(pool, s.text_ids, s.img_pos, s.img_ntok, v)
                          for s, v in zip(st["samples"], st["vis"])])
    return st["backing"]


def _run_plan(case, pool, st):
    return _plan(case, pool, st["ids"])


def _run_step(case, pool, st):
    ids = [fp.pool_write_sample(pool, s.text_ids, s.img_pos, s.img_ntok, v)
           for s, v in zip(st["samples"], st["vis"])]
    plan = _plan(case, pool, ids)
    out = _pack_all(case, pool, st, _groups(ids, plan["assign"].tolist(), case["n_mb"]))
    for i in ids:
        fp.pool_free_sample(pool, i)
    return {"packed": out, "plan": plan}


def _run_prefetch(case, pool, st):
    fp.pool_migrate(pool, st["ids"], fp.FP_TIER_HBM)
    out = _pack_all(case, pool, st, st["groups"])
    fp.pool_migrate(pool, st["ids"], fp.FP_TIER_HOST)
    return out


_RUN = {"pack": _run_pack, "write": _run_write, "plan": _run_plan, "step": _run_step, "prefetch": _run_prefetch}


def run(st):
    return _RUN[st["case"]["kind"]](st["case"], st["pool"].handle, st)


# ------------------------------------------------------------------ what a pass cannot do without

def _partition(case, samples):
    """Plain greedy partition by decreasing cost (ties: the lower index)."""
    n_mb, cap = case["n_mb"], case["capacity"]
    length = np.array([s.length for s in samples], np.int64)
    cost = case["cost_k"] * length + length * length
    assign = np.full(len(samples), -1, np.int32)
    tok, acc, longest = np.zeros(n_mb, np.int32), np.zeros(n_mb, np.int64), np.zeros(n_mb, np.int32)
    for p, i in enumerate(np.lexsort((np.arange(len(samples)), -cost))):
        if case["zigzag"]:
            order = [(p + q) % (2 * n_mb) for q in range(2 * n_mb)]
            order = [r if r < n_mb else 2 * n_mb - 1 - r for r in order]
        else:
            order = np.argsort(acc, kind="stable").tolist()
        j = next((j for j in order if tok[j] + length[i] <= cap), None)
        if j is not None:
            assign[i] = j
            tok[j] += length[i]
            acc[j] += cost[i]
            longest[j] = max(longest[j], length[i])
    return dict(assign=assign, mb_tokens=tok, mb_cost_scaled=acc, mb_max_len=longest, sample_cost_scaled=cost)


def work(case):
    """Each row read once and written once, with the ids, position ids and cu_seqlens."""
    samples = _samples(case, 0)
    row = 2 * case["hidden"]
    vis = sum(s.n_vis for s in samples)
    text = 4 * sum(len(s.text_ids) for s in samples)
    if case["kind"] == "write":
        return {"bytes": 2 * vis * row + 2 * text, "flops": 0}
    if case["kind"] == "plan":
        # per sample its id, length, cost and assignment; per microbatch tokens, cost and longest
        return {"bytes": 24 * len(samples) + 16 * case["n_mb"], "flops": 0}
    if case["kind"] == "prefetch":
        packed = sum(s.length for s in samples)
        return {"bytes": 4 * vis * row + packed * (2 * row + 4) + text, "flops": 0}
    packed = int(_partition(case, samples)["mb_tokens"].sum())
    total = packed * (2 * row + 4) + text
    return {"bytes": total + (2 * vis * row + 2 * text if case["kind"] == "step" else 0), "flops": 0}


def tolerance(case):
    return "exact"


# ------------------------------------------------------------------ the same outputs from plain torch

def _packed(case, seed, samples, groups):
    table = _table(case, seed)
    out = _outputs(case, samples)
    for members, (rows, cu, pos) in zip(groups, out):
        at = 0
        for k, i in enumerate(members):
            s = samples[i]
            src = [table[torch.from_numpy(s.text_ids).cuda().long()]]
            start = at
            vis = _vis(case, seed, i, s.n_vis)
            t = v = 0
            for p, n in zip(s.img_pos.tolist(), s.img_ntok.tolist()):
                for piece in (src[0][t:p], vis[v:v + n]):
                    rows[at:at + len(piece)] = piece
                    at += len(piece)
                t, v = p, v + n
            rows[at:at + len(s.text_ids) - t] = src[0][t:]
            at = start + s.length
            pos[start:at] = torch.arange(s.length, dtype=torch.int32, device="cuda")
            cu[k + 1] = at
    return out


def exact(case, seed):
    samples = _samples(case, seed)
    kind = case["kind"]
    if kind == "write":
        total = 3 * max(sum(_pages(case, s) for s in samples), 1)
        backing = torch.zeros((total * case["page_tokens"], case["hidden"]), dtype=torch.bfloat16, device="cuda")
        page = 0
        for i, s in enumerate(samples):
            first = page * case["page_tokens"]
            backing[first:first + s.n_vis] = _vis(case, seed, i, s.n_vis)
            page += _pages(case, s)
        return backing
    if kind == "prefetch":
        return _packed(case, seed, samples, [list(range(len(samples)))])
    plan = _partition(case, samples)
    if kind == "plan":
        return plan
    out = _packed(case, seed, samples, _groups(range(len(samples)), plan["assign"].tolist(), case["n_mb"]))
    return {"packed": out, "plan": plan} if kind == "step" else out
