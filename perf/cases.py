"""Cases that time the engine's public calls over the range its users meet.

A case names one call (`form`), the shape of the device state it works on
(`state`, `allocs`, `total` bytes) and the options a caller chooses (`chunk`,
staging `budget`, share of rewritten chunks `dirty`). The states follow the
benchmark's workloads at sizes whose images are quick to make and compare:

  random      uniform bytes in a few allocations of log-uniform sizes (a small
              process: nothing zero, nothing compressible);
  training    the training state of a decoder, every tensor scaled: 292 bf16
              parameter tensors, three flat fp32 buffers, eight bf16
              activation buffers (303 allocations; the smallest are some
              hundred bytes, the largest a fifth of the state);
  hpc         fp64 / int32 arrays of log-uniform sizes with runs of zero
              64 KiB blocks (about 60 % zero);
  fragmented  many allocations of any byte length, log-uniform over five
              orders of magnitude, with zero 256 KiB blocks (30 %).

Forms:

  into          ckpt_dump_into: full dump into the caller's own buffer
  dump          ckpt_dump, full
  restore       ckpt_restore of a full image
  delta         ckpt_dump against an earlier image of the same state
  apply         ckpt_restore of a delta, in place over its base
  codec_dump    ckpt_dump with CKPT_OPT_CODEC
  codec_restore ckpt_restore of such an image
  graph_dump    ckpt_dump with CKPT_OPT_GRAPH (batched form)
  graph_restore ckpt_restore with CKPT_OPT_GRAPH
  serve         one burst of requests through the request loop: for eight
                tenants two full dumps, two delta dumps, four restores

All outputs are bytes (images, or the restored memory) and have to be equal
bit for bit. Where blocks are zero or rewritten is fixed by the case; the
values in them come from the seed, so an image's length does not depend on
the seed.
"""
import math
import zlib

import numpy as np
import torch

from paper_2502_16631_amd import mickpt as mk

BLOCK = 65536   # granule of zero runs and of rewritten runs
KIB, MIB, GIB = 1 << 10, 1 << 20, 1 << 30

# Smallest and largest total bytes of each form, the states it is used on and
# the chunk sizes: the default (64 KiB) and the autotuner's other two
# candidates; the codec takes up to 64 KiB, the request loop the default only.
ALL_CHUNKS = (16 * KIB, 64 * KIB, 256 * KIB)
FORMS = {
    "into": (256 * KIB, 64 * MIB, ("random", "hpc"), ALL_CHUNKS),
    "dump": (4 * MIB, GIB, ("random", "training", "hpc"), ALL_CHUNKS),
    "restore": (4 * MIB, GIB, ("random", "training", "hpc"), ALL_CHUNKS),
    "delta": (32 * MIB, 8 * 10**9, ("training", "hpc"), ALL_CHUNKS),
    "apply": (32 * MIB, 8 * 10**9, ("training", "hpc"), ALL_CHUNKS),
    "codec_dump": (64 * MIB, GIB, ("training",), (16 * KIB, 64 * KIB)),
    "codec_restore": (64 * MIB, GIB, ("training",), (16 * KIB, 64 * KIB)),
    "graph_dump": (64 * MIB, GIB, ("fragmented",), ALL_CHUNKS),
    "graph_restore": (64 * MIB, GIB, ("fragmented",), ALL_CHUNKS),
    "serve": (64 * MIB, GIB, ("training", "hpc"), (64 * KIB,)),
}


def _case(name, form, state, allocs, total, chunk=64 * KIB, dirty=0.0, budget=16 * GIB):
    return {"name": name, "form": form, "state": state, "allocs": allocs, "total": total, "chunk": chunk,
            "dirty": dirty, "budget": budget}


def listed():
    return [
        # a caller that may not allocate checkpoints a little state in a tight
        # loop: latency, launches and waits are all there is
        _case("into_small", "into", "random", 8, MIB),
        # a small process checkpointed and brought back: latency
        _case("dump_tiny", "dump", "random", 8, 16 * MIB),
        _case("restore_tiny", "restore", "random", 8, 16 * MIB),
        # periodic full checkpoint of a training job, and its restart
        _case("dump_training", "dump", "training", 303, GIB),
        _case("restore_training", "restore", "training", 303, GIB),
        # incremental checkpoint of a simulation, 5 % rewritten since the last
        # one, and the delta applied over its base
        _case("delta_hpc", "delta", "hpc", 512, 8 * 10**9, dirty=0.05),
        _case("apply_hpc", "apply", "hpc", 512, 8 * 10**9, dirty=0.05),
        # incremental checkpoint of a model most of which is frozen, in large
        # chunks, by a context with the default staging budget (4 GiB: the
        # state is larger, as on a nearly full device)
        _case("delta_frozen", "delta", "training", 303, 6 * 10**9, chunk=256 * KIB, dirty=0.01, budget=0),
        # checkpoint with the byte-plane codec, for fewer bytes on the link
        # and on disk, and its restore
        _case("codec_dump", "codec_dump", "training", 303, GIB),
        _case("codec_restore", "codec_restore", "training", 303, GIB),
        # a fragmented process, all its small allocations in one graph launch;
        # small chunks, as its allocations are small
        _case("graph_fragmented", "graph_dump", "fragmented", 2000, 10**9, chunk=16 * KIB),
        # many tenants on one device: a burst of dumps, deltas and restores
        _case("serve_burst", "serve", "training", 303, GIB, dirty=0.05),
    ]


def draw(rng):
    form = rng.choice(sorted(FORMS))
    lo, hi, states, chunks = FORMS[form]
    total = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    state = rng.choice(states)
    allocs = {"random": rng.randint(1, 24), "training": 303, "hpc": max(1, min(512, total // (8 * MIB))),
              "fragmented": rng.randint(200, 4000)}[state]
    dirty = rng.choice((0.005, 0.01, 0.05, 0.1)) if form in ("delta", "apply", "serve") else 0.0
    c = _case("", form, state, allocs, total, rng.choice(chunks), dirty, rng.choice((0, 16 * GIB)))
    del c["name"]
    return c


# ------------------------------------------------------------------ layout

def _loguniform(rng, n, lo, hi, total):
    s = np.exp(rng.uniform(math.log(lo), math.log(hi), n))
    for _ in range(200):
        s = np.clip(s * (total / s.sum()), lo, hi)
    return [max(1, int(x)) for x in s]


def _decoder_elements():
    """Elements of a 1.3B decoder's parameter tensors (24 layers, d 2048)."""
    d, ffn = 2048, 8192
    layer = [3 * d * d, 3 * d, d * d, d, ffn * d, ffn, ffn * d, d, d, d, d, d]
    return [50257 * d, 2048 * d] + layer * 24 + [d, d]


def _sizes(case, rng):
    """(size, kind) of every allocation; kind: "u8", "bf16", "f32", "f64", "i32"."""
    state, n, total = case["state"], case["allocs"], case["total"]
    if state == "training":
        el = _decoder_elements()
        k = total / (2 * sum(el) + 12 * sum(el) + 8 * GIB)
        out = [(2 * max(1, int(e * k)), "bf16") for e in el]
        return out + [(4 * max(1, int(sum(el) * k)), "f32")] * 3 + [(2 * max(1, int(GIB * k / 2)), "bf16")] * 8
    if state == "hpc":
        top = min(GIB, max(4 * MIB, total // 2)) if n > 1 else total
        sizes = _loguniform(rng, n, min(MIB, total), top, total)
        return [(max(8, s // 8 * 8), "f64" if rng.random() < 0.5 else "i32") for s in sizes]
    if state == "fragmented":
        return [(s, "u8") for s in _loguniform(rng, n, 256, 256 * MIB, total)]
    return [(s, "u8") for s in _loguniform(rng, n, total / (16 * n), total, total)]


class Layout:
    """Where the allocations lie in one arena and which of its parts are zero
    or rewritten: a function of the case alone."""

    def __init__(self, case):
        rng = np.random.default_rng(zlib.crc32(repr(sorted((k, v) for k, v in case.items() if k != "name")).encode()))
        self.sizes, self.kinds = zip(*_sizes(case, rng))
        align = 512 if case["state"] in ("random", "fragmented") else BLOCK
        self.off, at = [], 0
        for s in self.sizes:
            self.off.append(at)
            at += -(-s // align) * align
        self.bytes = -(-at // BLOCK) * BLOCK
        self.rows = self.bytes // BLOCK
        # (start, length) of zero parts (fragmented) or a mask of zero 64 KiB
        # rows (hpc); mask of rewritten rows
        self.zero_parts, self.zero_rows = [], np.zeros(self.rows, bool)
        if case["state"] == "fragmented":
            for o, s in zip(self.off, self.sizes):
                for b in range(0, s, 256 * KIB):
                    if rng.random() < 0.3:
                        self.zero_parts.append((o + b, min(256 * KIB, s - b)))
        if case["state"] == "hpc":
            self.zero_rows = self._runs(rng, 24, 16)
        self.dirty_rows = np.zeros(self.rows, bool)
        want = int(math.ceil(case["dirty"] * self.rows))
        while self.dirty_rows.sum() < want:
            s = int(rng.integers(0, self.rows))
            self.dirty_rows[s:s + int(rng.geometric(1 / 16))] = True

    def _runs(self, rng, mean_true, mean_false):
        m, at, on = np.zeros(self.rows, bool), 0, bool(rng.random() < 0.6)
        while at < self.rows:
            n = int(rng.geometric(1 / (mean_true if on else mean_false)))
            m[at:at + n] = on
            at, on = at + n, not on
        return m

    def payload(self, chunk, dirty_only):
        """Bytes of the chunks that hold data (or, of a delta, that changed)."""
        if self.zero_parts or not self.zero_rows.any() and not dirty_only:
            return sum(self.sizes) - sum(n for _, n in self.zero_parts)
        keep = self.dirty_rows if dirty_only else ~self.zero_rows
        total = 0
        for o, s in zip(self.off, self.sizes):
            r0, step = o // BLOCK, max(1, chunk // BLOCK)
            m = keep[r0:r0 + -(-s // BLOCK)]
            hit = np.logical_or.reduceat(m, np.arange(0, len(m), step))
            total += min(s, int(hit.sum()) * max(chunk, BLOCK))
        return total


# ------------------------------------------------------------------ states

def _fill(lay, case, seed):
    """The arena with the state's values."""
    gen = torch.Generator("cuda").manual_seed(seed)
    arena = torch.empty(lay.bytes, dtype=torch.uint8, device="cuda")
    if case["state"] == "training":
        split = lay.off[292], lay.off[295]
        arena[:split[0]].view(torch.bfloat16).normal_(0.0, 0.02, generator=gen)
        arena[split[0]:split[1]].view(torch.float32).normal_(0.0, 1e-3, generator=gen)
        lay_w = arena[lay.off[292]:lay.off[292] + lay.sizes[292]].view(torch.float32)
        lay_w.normal_(0.0, 0.02, generator=gen)   # master weights; the other two are Adam's moments
        arena[split[1]:].view(torch.bfloat16).normal_(0.0, 1.0, generator=gen)
    else:
        arena.view(torch.int32).random_(generator=gen)
        for o, s, k in zip(lay.off, lay.sizes, lay.kinds):
            if k == "f64":
                arena[o:o + s].view(torch.float64).normal_(0.0, 1.0, generator=gen)
    if lay.zero_rows.any():
        arena.view(-1, BLOCK)[torch.from_numpy(np.flatnonzero(lay.zero_rows)).cuda()] = 0
    for o, n in lay.zero_parts:
        arena[o:o + n].zero_()
    return arena


def _shuffled(lay, case, seed):
    """As _fill, but every seed holds the same values in another order within
    each chunk: a codec record's length depends on how often each byte value
    occurs, and images of several seeds are to have one length."""
    arena = _fill(lay, case, 20)
    c8 = case["chunk"] // 8
    perm = torch.randperm(c8, generator=torch.Generator().manual_seed(seed)).cuda()
    rows = arena.view(torch.int64).view(-1, c8)
    for i in range(0, rows.shape[0], 4096):
        rows[i:i + 4096] = rows[i:i + 4096, perm]
    return arena


def _rewrite(lay, arena, seed):
    """The case's rewritten rows get fresh bytes; returns what they held."""
    gen = torch.Generator("cuda").manual_seed(seed + 1)
    at = torch.from_numpy(np.flatnonzero(lay.dirty_rows)).cuda()
    rows = arena.view(-1, BLOCK)
    old = rows[at]
    rows[at] = torch.randint(0, 256, tuple(old.shape), dtype=torch.uint8, device="cuda", generator=gen)
    return at, old


def _table(lay, arena):
    return [(i, arena[o:o + s]) for i, (o, s) in enumerate(zip(lay.off, lay.sizes))]


_contexts, _served = {}, []


def _context(budget):
    """One context per staging budget, made once as a program does."""
    if budget not in _contexts:
        _contexts[budget] = mk.ckpt_ctx_create(0, budget)
    return _contexts[budget]


def _server():
    """(context, request loop over it), made once as a serving process does."""
    if not _served:
        ctx = mk.ckpt_ctx_create(0, 8 * GIB)
        _served.append((ctx, mk.ckpt_serve_create(ctx, 16, 16 * GIB)))
    return _served[0]


def _done(rc):
    if rc != mk.CKPT_OK:
        raise RuntimeError(mk.ckpt_strerror(rc))


def _dump(ctx, table, prev=None, opts=None):
    rc, img, _ = mk.ckpt_dump(ctx, table, prev=prev, opts=opts)
    _done(rc)
    return img


def prepare(case, seed):
    if case["form"] == "serve":
        return _prepare_serve(case, seed)
    lay, form = Layout(case), case["form"]
    ctx = _context(case["budget"])
    flags = {"codec": mk.OPT_CODEC, "graph": mk.OPT_GRAPH}.get(form.split("_")[0], 0)
    s = {"form": form, "ctx": ctx, "opts": mk.make_opts(chunk_size=case["chunk"], flags=flags)}
    plain = mk.make_opts(chunk_size=case["chunk"])
    arena = _shuffled(lay, case, seed) if form.startswith("codec") else _fill(lay, case, seed)
    table = _table(lay, arena)
    s["arena"], s["table"] = arena, table
    if form == "into":
        n = 4096 + 48 * len(table) + sum(x + 64 for x in lay.sizes) + 8 * (lay.bytes // case["chunk"] + len(table))
        s["out"] = torch.empty(n, dtype=torch.uint8, pin_memory=True).numpy()
    elif form in ("restore", "codec_restore", "graph_restore"):
        s["img"] = _dump(ctx, table, opts=s["opts"] if form == "codec_restore" else plain)
        arena.zero_()   # what the process that is brought back starts from
    elif form in ("delta", "apply"):
        s["base"] = _dump(ctx, table, opts=plain)
        at, old = _rewrite(lay, arena, seed)
        if form == "apply":
            s["img"] = _dump(ctx, table, prev=s["base"], opts=plain)
            arena.view(-1, BLOCK)[at] = old
    return s


def _prepare_serve(case, seed):
    (ctx, srv), jobs = _server(), []
    for t in range(8):
        one = dict(case, total=case["total"] // 8, dirty=case["dirty"])
        one["allocs"] = max(1, one["allocs"] // 8) if one["state"] == "hpc" else one["allocs"]
        lay = Layout(one)
        arena = _fill(lay, one, 8 * seed + t)
        table = _table(lay, arena)
        base = _dump(ctx, table) if t >= 2 else None
        if t in (2, 3):
            _rewrite(lay, arena, 8 * seed + t)
        if t >= 4:
            arena.zero_()
        jobs.append((t, table, base, arena))
    torch.cuda.synchronize()
    return {"form": "serve", "server": srv, "jobs": jobs}


# ------------------------------------------------------------------ passes

def run(s):
    form = s["form"]
    if form == "serve":
        return _run_serve(s)
    if form == "into":
        rc, n, _ = mk.ckpt_dump_into(s["ctx"], s["table"], s["out"], opts=s["opts"])
        _done(rc)
        return s["out"][:n]
    if form in ("dump", "delta", "codec_dump", "graph_dump"):
        return _dump(s["ctx"], s["table"], prev=s.get("base"), opts=s["opts"]).view()
    rc, _ = mk.ckpt_restore(s["ctx"], s["img"], s["table"], opts=s["opts"])
    _done(rc)
    return s["arena"]


def _run_serve(s):
    srv, tickets = s["server"], []
    for t, table, base, _ in s["jobs"]:
        kind = mk.REQ_RESTORE if t >= 4 else mk.REQ_DUMP
        rc, ticket = mk.ckpt_serve_submit(srv, kind, table, prev=base if t < 4 else None,
                                          img=base if t >= 4 else None, tenant=t)
        _done(rc)
        tickets.append(ticket)
    mk.ckpt_serve_drain(srv)
    out = []
    for (t, _, _, arena), ticket in zip(s["jobs"], tickets):
        done = False
        while not done:
            done, rc, img, _ = mk.ckpt_serve_poll(srv, ticket)
        _done(rc)
        out.append(arena if t >= 4 else img.view())
    return out


# ------------------------------------------------------------------ work

def work(case):
    """Bytes: the state read and the image written, or the image read and the
    memory written; a delta's dump reads all of the state, its apply reads the
    chunks that have to hold the base."""
    if case["form"] == "serve":
        one = dict(case, total=case["total"] // 8)
        one["allocs"] = max(1, one["allocs"] // 8) if one["state"] == "hpc" else one["allocs"]
        lay = Layout(one)
        full, delta, n = lay.payload(case["chunk"], False), lay.payload(case["chunk"], True), sum(lay.sizes)
        return {"bytes": 6 * (n + full) + 2 * (n + delta), "flops": 0}
    lay = Layout(case)
    n, form = sum(lay.sizes), case["form"]
    d = lay.payload(case["chunk"], form in ("delta", "apply"))
    if form.startswith("codec"):
        d = int(0.82 * d)   # what the codec stores of such a state
    if form == "apply":
        zero = int(lay.zero_rows.mean() * n)
        return {"bytes": (n - zero - d) + zero + 2 * d, "flops": 0}
    return {"bytes": n + d, "flops": 0}


def exact(case, seed):
    """No output is a computed number: images and restored memory are bytes,
    equal or wrong."""
    return None

