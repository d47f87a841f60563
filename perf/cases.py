"""The transfers this library is measured on, each through its public entry points.

A case names an operation, the pool's geometry, the layout and place of the
contiguous chunks, and how many contexts of how many tokens one pass moves:

  load      host chunks -> pool pages, one batched call
  offload   pool pages -> host chunks, one batched call
  swap      offload of one set of contexts, then load of another set into
            other pages, in turn on one stream (an eviction followed by a hit)
  both_ways the same two transfers at once on two streams: the load with the
            library's defaults, the offload with the background quota (16 workgroups of one wave, 4 KiB steps)
  layers    one call and one event per layer on a transfer stream; the
            compute stream waits for every layer's event
  noalloc   the load that takes a pool description instead of a handle

Every pass moves bytes and computes nothing, so outputs are compared bit for bit.
"""
import math
import random
import weakref

import numpy as np
import torch

import paper_2508_18572_amd as kv

LAYOUTS = {"token": kv.KVIO_HOST_TOKEN_MAJOR, "page": kv.KVIO_HOST_PAGE_FIRST, "head": kv.KVIO_HOST_HEAD_MAJOR}
FIELDS = ("op", "layout", "chunk", "staged", "L", "H", "D", "elem", "P", "spans", "tokens", "lengths")


def _case(op, L, H, D, elem, P, tokens, spans=1, layout="token", chunk="pinned", staged=False, lengths=0, name=None):
    c = dict(zip(FIELDS, (op, layout, chunk, staged, L, H, D, elem, P, spans, tokens, lengths)))
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # One page of the smallest pool: what a serving loop pays to bring in the last page of a hit.
        _case("noalloc", 2, 4, 64, 2, 16, 16, name="noalloc_page"),
        # The 2 MiB context of the smallest workload, and its backup.
        _case("load", 2, 4, 64, 2, 16, 1024, name="load_2mib"),
        _case("offload", 2, 4, 64, 2, 16, 1024, name="offload_2mib"),
        # Llama-3.1-8B KV at page size 1: every token row goes to (comes from) a slot of its own.
        _case("load", 32, 8, 128, 2, 1, 4096, name="load_8b_p1"),
        _case("offload", 32, 8, 128, 2, 1, 4096, name="offload_8b_p1"),
        # A batch of ragged partial hits evicted and another loaded, more of them than one launch carries.
        _case("swap", 32, 8, 128, 2, 16, 64, spans=80, lengths=4, name="swap_batch_8b"),
        # 70B GQA KV loaded layer by layer so that each layer can compute as soon as it is there.
        _case("layers", 80, 8, 128, 2, 16, 512, name="layers_70b"),
        # Qwen2.5-7B-1M KV at page size 1: a load beside the backup of other contexts.
        _case("both_ways", 28, 4, 128, 2, 1, 6144, name="both_ways_qwen"),
        # Head-major chunks (the head/token transpose), a context that ends inside a page.
        _case("swap", 32, 8, 128, 2, 16, 1000, layout="head", name="swap_head_major"),
        # Page-first chunks of an 8-bit cache: rows of 384 bytes, pages of 5 tokens, a ragged end.
        _case("swap", 40, 3, 128, 1, 5, 3001, layout="page", name="swap_page_first_fp8"),
        # A load through the copy engine and HBM staging, the mode meant for loads beside compute.
        _case("load", 32, 8, 128, 2, 16, 2048, staged=True, name="staged_load_8b"),
        # Chunks in device memory: a context received or kept contiguous in HBM, moved into pages and back.
        _case("swap", 32, 8, 128, 2, 16, 2048, chunk="device", name="swap_device_chunks"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A transfer of the same ranges: every operation, layout and place of the
    chunks; 1 to 32 KV heads of 64 to 256 dims in 8 and 16 bits; 2 to 80
    layers; pages of 1 to 256 tokens; 1 to 100 contexts; 32 KiB to 512 MiB in all
    (layer-wise and two-way transfers from 16 MiB, staged ones from the 64 MiB
    where staging begins, loads without a handle up to 64 MiB)."""
    op, layout, chunk, staged = rng.choice((
        ("load", "token", "pinned", False), ("offload", "token", "pinned", False),
        ("load", "head", "pinned", False), ("offload", "head", "pinned", False),
        ("load", "page", "pinned", False), ("offload", "page", "pinned", False),
        ("swap", "token", "pinned", False), ("layers", "token", "pinned", False),
        ("both_ways", "token", "pinned", False), ("noalloc", "token", "pinned", False),
        ("load", "token", "pinned", True), ("swap", "token", "device", False)))
    L, H = _log_uniform(rng, 2, 80), rng.choice((1, 2, 3, 4, 5, 8, 8, 16, 32))
    D, elem = rng.choice((64, 80, 96, 128, 128, 256)), rng.choice((1, 2, 2))
    P = rng.choice((1, 1, 2, 5, 16, 16, 24, 32, 64, 256))
    lo = 16 << 20 if op in ("layers", "both_ways") else 64 << 20 if staged else 32 << 10
    hi = 64 << 20 if op == "noalloc" else 256 << 20 if op in ("swap", "both_ways") else 512 << 20
    total = max(1, _log_uniform(rng, lo, hi) // (L * 2 * H * D * elem))     # tokens of all contexts
    spans = min(1 if rng.random() < 0.5 else _log_uniform(rng, 2, 100), max(1, total // max(8, P)),
                64 if op == "noalloc" else 100)
    tokens = max(1, total if spans == 1 else total // spans)
    return _case(op, L, H, D, elem, P, tokens, spans, layout, chunk, staged, lengths=rng.randrange(1 << 20))


def _lengths(case, which):
    """(tokens to move, tokens the chunk holds) of each context of set `which`:
    one full context, or partial hits of 50-100% of prefixes log-uniform in
    [tokens / 4, 4 tokens)."""
    T, P = case["tokens"], case["P"]
    pages = (lambda n: -(-n // P) * P) if case["spans"] > 1 or case["layout"] == "page" else (lambda n: n)
    if case["spans"] == 1:
        return [(T, pages(T))]
    rng = random.Random(case["lengths"] * 2 + which)
    out = []
    for _ in range(case["spans"]):
        prefix = max(1, int(T / 4 * 16 ** rng.random() / 1.35))       # the mean length is about T
        out.append((max(1, int(prefix * rng.uniform(0.5, 1.0))), pages(prefix)))
    return out


def _directions(case):
    """(sets loaded, sets offloaded); set 0 is loaded, set 1 offloaded."""
    return (case["op"] != "offload", case["op"] in ("offload", "swap", "both_ways"))


def work(case):
    """Every row that moves is read once and written once, its page index read once per layer call or transfer."""
    R, total = case["H"] * case["D"] * case["elem"], 0
    for which, used in enumerate(_directions(case)):
        if used:
            for t, _ in _lengths(case, which):
                total += 2 * case["L"] * 2 * R * t + 4 * -(-t // case["P"])
    return {"bytes": total, "flops": 0}


def tolerance(case):
    return "exact"


def _payload(gen, nbytes, elem):
    """KV bytes on the GPU: bf16 N(0, 1) elements, or 8-bit ones."""
    if elem == 2:
        return torch.randn(nbytes // 2, device="cuda", generator=gen, dtype=torch.bfloat16).view(torch.uint8)
    return torch.randint(0, 256, (nbytes,), device="cuda", generator=gen, dtype=torch.uint8)


class _Chunk:
    """One set's contiguous chunks, back to back in one allocation."""

    def __init__(self, case, sizes, src):
        self.offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        if case["chunk"] == "device":
            self.tensor, self.ptr = src, src.data_ptr()
            return
        buf = kv.HostBuffer(int(self.offsets[-1]))
        weakref.finalize(buf.array, kv.kvio_host_free, buf.ptr).atexit = False
        self.tensor, self.ptr = torch.from_numpy(buf.array), buf.ptr
        self.tensor.copy_(src)


class _State:
    pass


_streams = {}


def _stream(role):
    """The program's stream for this role, made once: a few streams, each with a hardware queue to itself."""
    if role not in _streams:
        _streams[role] = kv.Stream()
    return _streams[role].torch


def prepare(case, seed):
    L, H, D, elem, P = (case[k] for k in ("L", "H", "D", "elem", "P"))
    R = H * D * elem
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s = _State()
    s.op, s.L = case["op"], L
    sets = [_lengths(case, w) if used else [] for w, used in enumerate(_directions(case))]
    counts = [[-(-t // P) for t, _ in ctx] for ctx in sets]
    need = sum(sum(c) for c in counts)
    num_pages = need + need // 2 + 1                     # a pool that also holds other contexts
    S = num_pages * P
    pages = torch.randperm(num_pages, generator=gen, device="cuda")[:need].to(torch.int32)
    pool = _payload(gen, 2 * L * S * R, elem)
    s.pool = pool.view(torch.bfloat16 if elem == 2 else torch.uint8).view(2, L, S, H, D)
    s.spans, s.chunks, s.tables, at = [[], []], [None, None], [], 0
    for w, (ctx, cnt) in enumerate(zip(sets, counts)):
        if not ctx:
            continue
        sizes = [L * 2 * cap * R for _, cap in ctx]
        s.chunks[w] = _Chunk(case, sizes, _payload(gen, sum(sizes), elem))
        for i, ((t, cap), n) in enumerate(zip(ctx, cnt)):
            table = pages[at:at + n].clone()             # each context's own page table
            at += n
            s.tables.append(table)
            s.spans[w].append((s.chunks[w].ptr + int(s.chunks[w].offsets[i]), cap, t, table.data_ptr()))
    layout = LAYOUTS[case["layout"]]
    if case["op"] == "noalloc":
        s.desc, s.keep = kv.pool_desc(L, H, D, elem, P, S, [s.pool[0, l].data_ptr() for l in range(L)],
                                      [s.pool[1, l].data_ptr() for l in range(L)], host_layout=layout)
        return s
    mode = kv.launch(flags=kv.KVIO_LAUNCH_STAGED) if case["staged"] else None
    back = kv.launch(workgroups=16, threads=64, tile_kib=4) if case["op"] == "both_ways" else None
    s.handle = kv.KVPool(s.pool, P, load_launch=mode, offload_launch=back, host_layout=layout)
    if case["op"] == "layers":
        s.events = [torch.cuda.Event() for _ in range(L)]
        s.io = _stream("transfer")
    if case["op"] == "both_ways":
        s.io, s.background = _stream("transfer"), _stream("background")
    return s


def _words(x):
    """A whole buffer as 64-bit words (its own memory)."""
    return x.reshape(-1).view(torch.int64)


def run(s):
    if s.op == "noalloc":
        kv.kvio_load_noalloc(s.desc, s.spans[0], 0, s.L)
    elif s.op == "load":
        s.handle.load(s.spans[0])
    elif s.op == "offload":
        s.handle.offload(s.spans[1])
    elif s.op == "swap":
        s.handle.offload(s.spans[1])
        s.handle.load(s.spans[0])
    elif s.op == "layers":
        cur = torch.cuda.current_stream()
        s.io.wait_stream(cur)
        for l in range(s.L):
            s.handle.load_layer(s.spans[0], l, stream=s.io, done=s.events[l])
        for l in range(s.L):
            cur.wait_event(s.events[l])                  # a model would run layer l here
    else:
        cur = torch.cuda.current_stream()
        s.io.wait_stream(cur)
        s.background.wait_stream(cur)
        s.handle.load(s.spans[0], stream=s.io)
        s.handle.offload(s.spans[1], stream=s.background)
        cur.wait_stream(s.io)
        cur.wait_stream(s.background)
    out = {}
    if s.spans[0]:
        out["pool"] = _words(s.pool)
    if s.spans[1]:
        out["chunks"] = _words(s.chunks[1].tensor)
    return out
