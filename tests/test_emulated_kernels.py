"""The library's own sources, kernels included, built for the CPU (tests/c/emu:
the 64 lanes of a wave are coroutines that must meet at every cross-lane
operation, values taken as wave-uniform must be, and every buffer lies against
an inaccessible page), against the oracle: every form the entry points take --
host layouts, row widths, page sizes, ragged and empty spans, chunks at every
16-byte offset, spans and layer ranges beyond a launch's 32-bit counts, out-of-range pages,
launch shapes, staged transfers -- on kernels that count vectors rather than
rows."""
import ctypes
import importlib.util
import os
import random
import re
import shutil
import subprocess
import sys

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_18572_amd", "csrc")
CXX = "/opt/rocm/llvm/bin/clang++"
LAYOUT = {0: oracle.TOKEN_MAJOR, 1: oracle.PAGE_FIRST, 2: oracle.HEAD_MAJOR}

pytestmark = pytest.mark.skipif(not os.path.exists(CXX), reason="no clang++ (the sources use its vector types)")


def plain(text):
    """The source with its inline assembly as what it does: a store, or nothing."""
    text = re.sub(r'asm volatile\("[^;]*?" : : "v"\((\w+)\), "v"\((\w+)\), "s"\((\w+)\) : "memory"\);',
                  r"*(gvec *)((uintptr_t)\3 + \1) = \2;", text)
    text = re.sub(r'asm volatile\("[^;]*?" : : "v"\((\w+)\), "v"\((\w+)\) : "memory"\);', r"*\1 = \2;", text)
    text = re.sub(r'asm volatile\("" : [^;]*;', ";", text)
    assert "asm volatile" not in text
    return text


def build(out, extra=()):
    for f in os.listdir(CSRC):
        with open(os.path.join(CSRC, f)) as src, open(os.path.join(out, f), "w") as dst:
            dst.write(plain(src.read()))
    emu = os.path.join(ROOT, "tests", "c", "emu")
    sources = [os.path.join(out, f) for f in sorted(os.listdir(out)) if f.endswith((".cpp", ".hip"))]
    flags = ["-x", "c++", "-std=c++17", "-O1", "-fPIC", "-U_FORTIFY_SOURCE", "-I", emu, "-I",
             os.path.join(ROOT, "include"), "-I", out, *extra]
    objects = [s + ".o" for s in sources] + [os.path.join(out, "emu.o")]
    jobs = [subprocess.Popen([CXX, *flags, "-c", s, "-o", o])
            for s, o in zip(sources + [os.path.join(emu, "emu.cpp")], objects)]
    assert all([j.wait() == 0 for j in jobs])
    subprocess.run([CXX, "-shared", "-o", os.path.join(out, "libkvio.so"), *objects, "-pthread"], check=True)
    shutil.copy(os.path.join(ROOT, "paper_2508_18572_amd", "kvio.py"), out)


def load(out):
    spec = importlib.util.spec_from_file_location("kvio_emulated_" + os.path.basename(out), os.path.join(out, "kvio.py"))
    kv = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(kv)
    kv._lib.emu_alloc.restype = ctypes.c_void_p
    kv._lib.emu_alloc.argtypes = [ctypes.c_size_t, ctypes.c_int, ctypes.c_int]
    kv._lib.emu_free.argtypes = [ctypes.c_void_p]
    kv._lib.emu_launches.restype = kv._lib.emu_last_tiles.restype = kv._lib.emu_last_block.restype = ctypes.c_int64
    kv._lib.emu_last_pause.restype = kv._lib.emu_last_waves.restype = kv._lib.emu_default_load_kib.restype = ctypes.c_int64
    kv._lib.emu_default_load_kib.argtypes = [ctypes.c_int64, ctypes.c_int]
    return kv


class Memory:
    def __init__(self, kv, nbytes, device, at_end, skip=0):
        self.kv, self.base = kv, kv._lib.emu_alloc(nbytes + skip, device, at_end)
        self.ptr = self.base + skip
        self.array = np.ctypeslib.as_array((ctypes.c_uint8 * nbytes).from_address(self.ptr))

    def free(self):
        self.kv._lib.emu_free(self.base)


def one_case(kv, seed, bad_page=False):
    rng = random.Random(seed)
    layout, L, H, e = rng.choice([0, 1, 2]), rng.choice([1, 2, 3]), rng.choice([1, 2, 3, 5, 8]), rng.choice([1, 2])
    D = rng.choice([8, 16, 24, 40, 64, 80, 96, 128, 256, 320])
    D = 64 if D * e % 16 else D
    R, P = H * D * e, rng.choice([1, 1, 2, 3, 5, 7, 16, 64, 100])
    n = 1 if bad_page else rng.choice([1, 1, 2, 3, 5, 70])
    most = max(1, 60000 // (L * 2 * R) // min(n, 5) * 2)
    spans = []
    for _ in range(n):
        T = rng.randint(1 if bad_page else 0, most if n < 70 else max(1, most // 8))
        cap = T + rng.choice([0, 0, 1, 3, 17])
        spans.append((T, -(-cap // P) * P if layout == 1 else cap))
    need = sum(-(-t // P) for t, _ in spans)
    S = (need + rng.randint(1, 4)) * P
    nr = np.random.default_rng(seed)
    perm = nr.permutation(S // P).astype(np.int32)
    l0 = rng.randint(0, L - 1)
    l1 = rng.randint(l0 + 1, L)
    at_end, keep, local = rng.randint(0, 1), [], int(seed % 4 == 3)      # chunks in device memory

    def mem(nbytes, device, end=at_end, skip=0):
        keep.append(Memory(kv, nbytes, device, end, skip))
        return keep[-1]
    img = nr.integers(0, 256, size=(2, L, S, R), dtype=np.uint8)
    pool = [[mem(S * R, 1) for _ in range(L)] for _ in range(2)]
    for k in range(2):
        for l in range(L):
            pool[k][l].array[:] = img[k, l].reshape(-1)
    launch = kv.launch(rng.choice([0, 1, 2, 3]), rng.choice([0, 64, 128, 192]), rng.choice([0, 4, 8, 16]),
                       rng.choice([0, 0, 0, kv.KVIO_LAUNCH_CACHED, kv.KVIO_LAUNCH_NO_LDS]))
    staged = layout != 1 and rng.random() < 0.15 and not bad_page
    if staged:
        launch.flags |= kv.KVIO_LAUNCH_STAGED
    h = kv.kvio_pool_create(L, H, D, e, P, S, [m.ptr for m in pool[0]], [m.ptr for m in pool[1]], launch, launch, layout,
                            staging_bytes=8 * P * R * rng.choice([1, 2, 5]) if staged else 0)
    work, at = [], 0
    for T, cap in spans:
        nbytes, count = max(16, oracle.host_chunk_bytes(LAYOUT[layout], L, cap, R, P)), -(-T // P)
        src, dst = (mem(nbytes, local, skip=16 * rng.randint(0, 20)) for _ in range(2))
        src.array[:] = nr.integers(0, 256, nbytes, dtype=np.uint8)
        dst.array[:] = 0x55
        table = mem(max(16, -(-4 * count // 16) * 16), 1)
        pages = perm[at:at + count].copy()
        given = pages.copy()
        if bad_page:
            given[rng.randrange(count)] = rng.choice([-1, S // P, 2 ** 31 - 1, -2 ** 31])
        table.array[:4 * count] = given.view(np.uint8)
        work.append((T, cap, pages, given, src, dst, table))
        at += count
    kv.kvio_load(h, [(w[4].ptr, w[1], w[0], w[6].ptr) for w in work], l0, l1)
    got = np.stack([np.stack([m.array.reshape(S, R) for m in row]) for row in pool])
    exp = img.copy()
    oracle.load_layout(exp[0], exp[1], P, [(w[4].array, w[1], w[0], w[2]) for w in work], LAYOUT[layout], num_heads=H,
                       layer_begin=l0, layer_end=l1)
    if bad_page:
        for p in work[0][2][work[0][2] != work[0][3]]:
            exp[:, :, p * P:(p + 1) * P] = img[:, :, p * P:(p + 1) * P]
        with pytest.raises(kv.KvioError) as err:
            kv.kvio_check(h)
        assert err.value.status == kv.KVIO_ERANGE and f"context page {np.flatnonzero(work[0][2] != work[0][3])[0]}:" in err.value.detail
    assert np.array_equal(got, exp), f"load of case {seed}"
    kv.kvio_offload(h, [(w[5].ptr, w[1], w[0], w[6].ptr) for w in work], 0, L)
    for T, cap, pages, given, _, dst, _ in work:
        want = np.full(len(dst.array), 0x55, np.uint8)
        oracle.offload_layout(exp[0], exp[1], P, [(want, cap, T, pages)], LAYOUT[layout], num_heads=H)
        if bad_page:        # a chunk of fill bytes goes through the same pages: what the skipped one keeps
            fill, marks = np.full_like(exp, 0x55), np.full_like(want, 0)
            keep_pages = np.flatnonzero(pages == given)
            mark = np.zeros_like(exp)
            mark[:, :, (pages[keep_pages][:, None] * P + np.arange(P)).reshape(-1)] = 1
            oracle.offload_layout(mark[0], mark[1], P, [(marks, cap, T, pages)], LAYOUT[layout], num_heads=H)
            want[marks == 0] = 0x55
            del fill
        assert np.array_equal(dst.array, want), f"offload of case {seed}"
    if not bad_page:
        kv.kvio_check(h)
    kv.kvio_pool_destroy(h)
    for m in keep:
        m.free()


def run_cases(out, first, last, bad_page):
    kv = load(out)
    for seed in range(first, last):
        print("case", seed, "bad page" if bad_page else "", flush=True)      # a fault ends the process: the last line names it
        one_case(kv, seed, bad_page)


def beside_table(L):
    """Spans beside the layer table in a launch's arguments, as include/kvio.h states it."""
    header = open(os.path.join(ROOT, "include", "kvio.h")).read()
    num, den = re.search(r"64 - ceil\((\d+) \* L / (\d+)\) of them", header).groups()
    return 64 - -(-int(num) * L // int(den))


def noalloc_case(kv, L, n, layout, seed, split):
    """The load that takes a description: every layer's table entry is used, with n
    contexts of which the middle one is empty (the table lies behind the spans that
    remain) and the last one longer than a split build's launch takes."""
    H, D, e, P = 2, 16, 1, 3
    R, nr = H * D * e, np.random.default_rng(seed)
    tokens = [1 + (i * 5) % 7 for i in range(n)]
    if n > 2:
        tokens[n // 2] = 0
    tokens[-1] = 45
    caps = [-(-t // P) * P for t in tokens]
    perm, at = nr.permutation(sum(caps) // P + 2).astype(np.int32), 0
    S = len(perm) * P
    img = nr.integers(0, 256, size=(2, L, S, R), dtype=np.uint8)
    keep = [[Memory(kv, S * R, 1, seed & 1) for _ in range(L)] for _ in range(2)]
    for k in range(2):
        for l in range(L):
            keep[k][l].array[:] = img[k, l].reshape(-1)
    spans, ora, extra = [], [], []
    for t, cap in zip(tokens, caps):
        chunk, table = Memory(kv, max(16, L * 2 * cap * R), 0, seed & 1), Memory(kv, max(16, cap // P * 4), 1, 0)
        chunk.array[:] = nr.integers(0, 256, len(chunk.array), dtype=np.uint8)
        pages = perm[at:at + cap // P].copy()
        at += cap // P
        table.array[:4 * len(pages)] = pages.view(np.uint8)
        spans.append((chunk.ptr, cap, t, table.ptr))
        ora.append((chunk.array, cap, t, pages))
        extra += [chunk, table]
    desc, held = kv.pool_desc(L, H, D, e, P, S, [m.ptr for m in keep[0]], [m.ptr for m in keep[1]], host_layout=layout)
    l0, before = L // 3, kv._lib.emu_launches()
    kv.kvio_load_noalloc(desc, spans, l0, L)
    launches = kv._lib.emu_launches() - before
    got = np.stack([np.stack([m.array.reshape(S, R) for m in row]) for row in keep])
    oracle.load_layout(img[0], img[1], P, ora, LAYOUT[layout], num_heads=H, layer_begin=l0, layer_end=L)
    assert np.array_equal(got, img), f"noalloc load of {n} spans, {L} layers"
    if not split:       # the table in the one launch's arguments, or written by a kernel before it
        assert launches == (1 if n <= beside_table(L) else 2), (L, n, launches)
    for m in keep[0] + keep[1] + extra:
        m.free()


def run_noalloc(out, split):
    kv = load(out)
    for L in (1, 2, 3, 4, 5, 64, 80, 127, 128):  # the most spans beside the table, and one more
        beside = beside_table(L)
        for n in sorted({1, 2, beside - 1, beside, min(beside + 1, 64)}):
            print("noalloc", L, n, flush=True)
            noalloc_case(kv, L, n, (L + n) % 3, 1000 * L + n, split)


def run_staged_layers(out):
    """Staged transfers whose slots hold more layers than a launch counts planes of
    (4 in this build): the slot goes in several launches (the emulator refuses one
    with more)."""
    kv = load(out)
    for layout, L, H in ((0, 5, 1), (2, 5, 1), (2, 7, 2), (0, 1, 3)):
        D, e, P = 16, 1, 4
        R, nr, before = H * D * e, np.random.default_rng(L), kv._lib.emu_launches()
        img = nr.integers(0, 256, size=(2, L, 3 * P, R), dtype=np.uint8)
        keep = [[Memory(kv, 3 * P * R, 1, 1) for _ in range(L)] for _ in range(2)]
        for k in range(2):
            for l in range(L):
                keep[k][l].array[:] = img[k, l].reshape(-1)
        mode = kv.launch(flags=kv.KVIO_LAUNCH_STAGED)
        h = kv.kvio_pool_create(L, H, D, e, P, 3 * P, [m.ptr for m in keep[0]], [m.ptr for m in keep[1]], mode, mode,
                                layout, staging_bytes=4 * L * 2 * P * R)
        src, dst, table = Memory(kv, L * 2 * P * R, 0, 1), Memory(kv, L * 2 * P * R, 0, 1), Memory(kv, 16, 1, 1)
        src.array[:] = nr.integers(0, 256, len(src.array), dtype=np.uint8)
        dst.array[:] = 0x55
        pages = np.array([2], np.int32)
        table.array[:4] = pages.view(np.uint8)
        kv.kvio_load(h, [(src.ptr, P, P, table.ptr)], 0, L)
        kv.kvio_offload(h, [(dst.ptr, P, P, table.ptr)], 0, L)
        kv.kvio_check(h)
        oracle.load_layout(img[0], img[1], P, [(src.array, P, P, pages)], LAYOUT[layout], num_heads=H)
        assert np.array_equal(np.stack([np.stack([m.array.reshape(3 * P, R) for m in row]) for row in keep]), img)
        assert np.array_equal(src.array, dst.array)
        print("staged layers", layout, L, H, kv._lib.emu_launches() - before, "launches", flush=True)
        kv.kvio_pool_destroy(h)
        for m in keep[0] + keep[1] + [src, dst, table]:
            m.free()


def run_full_steps(out):
    """Narrow rows and head segments: a wave's step is as full as 64 rows (of all heads)
    can make it (a quarter may be lost to the tile's unit), in both directions, and
    loads of narrow rows with 16 KiB steps keep the workgroups of 256 threads that
    1024 are folded into, also where a smaller step would serve."""
    kv = load(out)
    for De, H, kib, layout in ((16, 8, 4, 2), (16, 8, 16, 2), (16, 3, 4, 2), (32, 8, 4, 2), (32, 4, 16, 2), (48, 5, 4, 2), (48, 5, 16, 2),
                               (48, 1, 4, 0), (48, 1, 4, 1), (112, 1, 16, 0), (112, 1, 16, 1), (80, 1, 16, 0), (96, 1, 8, 1)):
        L, P, T = 2, 16, 512
        R, nr = H * De, np.random.default_rng(De)
        keep = [[Memory(kv, T * R, 1, 1) for _ in range(L)] for _ in range(2)]
        mode = kv.launch(2, 1024 if kib == 16 else 64, kib)
        h = kv.kvio_pool_create(L, H, De, 1, P, T, [m.ptr for m in keep[0]], [m.ptr for m in keep[1]], mode, mode, layout)
        src, dst, table = Memory(kv, L * 2 * T * R, 0, 1), Memory(kv, L * 2 * T * R, 0, 1), Memory(kv, T // P * 4, 1, 1)
        src.array[:] = nr.integers(0, 256, len(src.array), dtype=np.uint8)
        pages = nr.permutation(T // P).astype(np.int32)
        table.array[:] = pages.view(np.uint8)
        step = min(kib * 1024, 64 * R)
        kv.kvio_load(h, [(src.ptr, T, T, table.ptr)], 0, L)
        load_tiles = kv._lib.emu_last_tiles()
        assert kv._lib.emu_last_block() <= 256, (De, H, kib)
        kv.kvio_offload(h, [(dst.ptr, T, T, table.ptr)], 0, L)
        assert np.array_equal(src.array, dst.array)
        for tiles in (load_tiles, kv._lib.emu_last_tiles()):
            assert tiles * step * 3 // 4 <= L * 2 * T * R, (De, H, kib, tiles)
        kv.kvio_pool_destroy(h)
        for m in keep[0] + keep[1] + [src, dst, table]:
            m.free()


def run_default_loads(out):
    """Default loads below 32 MiB keep 256 KiB in flight (two of them on two streams
    fill the link together), larger ones 192, and rows too narrow to fill a step take as many waves more."""
    kv = load(out)
    for layout in range(3):
        for shift in range(15, 25):
            assert kv._lib.emu_default_load_kib(1 << shift, layout) == 256, (layout, shift)
        for shift in range(25, 36):
            assert kv._lib.emu_default_load_kib(1 << shift, layout) == 192, (layout, shift)
    L, P = 1, 16
    for R, T, waves in ((16, 16384, 256), (32, 8192, 128), (48, 8192, 85), (512, 512, 64)):
        keep = [[Memory(kv, T * R, 1, 1) for _ in range(L)] for _ in range(2)]
        h = kv.kvio_pool_create(L, 1, R, 1, P, T, [m.ptr for m in keep[0]], [m.ptr for m in keep[1]])
        src, table = Memory(kv, L * 2 * T * R, 0, 1), Memory(kv, T // P * 4, 1, 1)
        src.array[:] = np.random.default_rng(R).integers(0, 256, len(src.array), dtype=np.uint8)
        pages = np.random.default_rng(R).permutation(T // P).astype(np.int32)
        table.array[:] = pages.view(np.uint8)
        kv.kvio_load(h, [(src.ptr, T, T, table.ptr)], 0, L)
        img = np.zeros((2, L, T, R), np.uint8)
        oracle.load(img[0], img[1], P, [(src.array, T, T, pages)])
        assert np.array_equal(np.stack([np.stack([m.array.reshape(T, R) for m in row]) for row in keep]), img)
        assert waves - 4 <= kv._lib.emu_last_waves() <= waves, (R, kv._lib.emu_last_waves())
        kv.kvio_pool_destroy(h)
        for m in keep[0] + keep[1] + [src, table]:
            m.free()


def run_pauses(out):
    """The pause of offloads on a small quota follows what they keep in flight: none
    where they do not reach the paced rate, longer the more they exceed it, the same
    for a byte whatever the row size, in every layout; none for large workgroups,
    quotas far above the rate, the default grid (also cached) and chunks in device memory."""
    kv = load(out)

    def pause(layout, De, H, quota, local=0, T=1024):
        L, P, R = 1, 16, H * De
        T = max(T, 131072 // R // 16 * 16)
        keep = [[Memory(kv, T * R, 1, 1) for _ in range(L)] for _ in range(2)]
        h = kv.kvio_pool_create(L, H, De, 1, P, T, [m.ptr for m in keep[0]], [m.ptr for m in keep[1]], None, kv.launch(*quota), layout)
        dst, table = Memory(kv, L * 2 * T * R, local, 1), Memory(kv, T // P * 4, 1, 1)
        for k in range(2):
            keep[k][0].array[:] = np.random.default_rng(k).integers(0, 256, T * R, dtype=np.uint8)
        pages = np.random.default_rng(R).permutation(T // P).astype(np.int32)
        table.array[:] = pages.view(np.uint8)
        kv.kvio_offload(h, [(dst.ptr, T, T, table.ptr)], 0, L)
        got, want = kv._lib.emu_last_pause(), np.zeros_like(dst.array)
        img = np.stack([np.stack([m.array.reshape(T, R) for m in row]) for row in keep])
        oracle.offload_layout(img[0], img[1], P, [(want, T, T, pages)], LAYOUT[layout], num_heads=H)
        assert np.array_equal(dst.array, want)
        kv.kvio_pool_destroy(h)
        for m in keep[0] + keep[1] + [dst, table]:
            m.free()
        return got

    for layout in range(3):
        at = {q: pause(layout, 256, 2, q) for q in ((8, 64, 4), (12, 64, 4), (16, 64, 4), (20, 64, 4), (4, 256, 4), (8, 256, 4), (32, 64, 4), (0, 0, 0),
                                                    (0, 0, 0, kv.KVIO_LAUNCH_CACHED), (16, 64, 4, kv.KVIO_LAUNCH_CACHED))}
        assert at[8, 64, 4] == at[12, 64, 4] == at[32, 64, 4] == at[8, 256, 4] == at[0, 0, 0] == at[0, 0, 0, 1] == 0, at
        assert 5 <= at[16, 64, 4] <= 9 and at[16, 64, 4, 1] == at[16, 64, 4] == at[4, 256, 4], at
        assert at[20, 64, 4] > 2 * at[16, 64, 4], at
        assert pause(layout, 256, 2, (16, 64, 4), local=1) == 0
    assert pause(0, 512, 1, (2, 1024, 4)) == 0
    for R in (128, 256, 512, 1024, 4096):
        assert 5 <= pause(0, R, 1, (16, 64, 4)) <= 9, R
    assert pause(0, 8192, 1, (16, 64, 4)) > 9                   # one table read for two steps
    assert pause(0, 16, 1, (8, 256, 4)) == pause(0, 2064, 1, (16, 64, 4)) == 0


def run_load_pauses(out):
    """Loads of a size (64 KiB in this build, 32 MiB otherwise) whose waves would queue on
    the link sleep behind each step, longer the more they would; none where they do
    not fill the link, with larger steps, with large workgroups and from device memory."""
    kv = load(out)

    def pause(layout, quota, T=2048, local=0, P=16, H=2, De=256):
        R = H * De
        keep = [Memory(kv, T * R, 1, 1) for _ in range(2)]
        h = kv.kvio_pool_create(1, H, De, 1, P, T, [keep[0].ptr], [keep[1].ptr], kv.launch(*quota), None, layout)
        src, table = Memory(kv, 2 * T * R, local, 1), Memory(kv, T // P * 4, 1, 1)
        src.array[:] = np.random.default_rng(T).integers(0, 256, len(src.array), dtype=np.uint8)
        pages = np.random.default_rng(R).permutation(T // P).astype(np.int32)
        table.array[:] = pages.view(np.uint8)
        kv.kvio_load(h, [(src.ptr, T, T, table.ptr)], 0, 1)
        img = np.zeros((2, 1, T, R), np.uint8)
        oracle.load_layout(img[0], img[1], P, [(src.array, T, T, pages)], LAYOUT[layout], num_heads=H)
        assert np.array_equal(np.stack([m.array.reshape(1, T, R) for m in keep]), img)
        got = kv._lib.emu_last_pause()
        kv.kvio_pool_destroy(h)
        for m in keep + [src, table]:
            m.free()
        return got

    for layout in range(3):
        at = {q: pause(layout, q) for q in ((8, 256, 4), (13, 192, 4), (7, 384, 4), (16, 192, 4), (16, 256, 4), (16, 192, 8), (16, 256, 16))}
        assert at[8, 256, 4] == at[16, 192, 8] == at[16, 256, 16] == 0, at
        assert at[13, 192, 4] <= at[7, 384, 4] < at[16, 192, 4] <= at[16, 256, 4] <= 40, at
        assert 20 <= at[16, 192, 4] and (8 <= at[13, 192, 4] <= 20 or layout == 1), at
        assert pause(layout, (16, 192, 4), local=1) == 0
        assert pause(layout, (16, 192, 4), T=48) == 0                # below the size
    assert pause(0, (4, 1024, 4)) == pause(0, (6, 512, 4)) == 0


def run_short_contexts(out):
    """Short head-major contexts on a fixed quota: a wave's step holds the rows of all
    heads (or of as many as fit), not one head's few vectors; long contexts, the
    default grid and KVIO_LAUNCH_NO_LDS go by address."""
    kv = load(out)
    P = 4
    for De, H, T, n, kib, most in ((256, 8, 1, 3, 4, 1.0), (256, 8, 3, 2, 4, 2.1), (128, 64, 1, 2, 4, 2.0), (128, 64, 2, 1, 4, 4.0),
                                   (64, 5, 4, 5, 16, 1.0), (160, 60, 1, 2, 8, 2.0), (16, 300, 7, 1, 4, None), (1040, 7, 1, 2, 4, None)):
        L, R, rng = 2, H * De, np.random.default_rng(H)
        S, cap = (n * -(-T // P) + 1) * P, T + 1
        img = rng.integers(0, 256, size=(2, L, S, R), dtype=np.uint8)
        perm, keep = rng.permutation(S // P).astype(np.int32), []
        for quota in ((2, 64, kib), (2, 64, kib, kv.KVIO_LAUNCH_NO_LDS), (0, 0, 0)):
            pool = [[Memory(kv, S * R, 1, 1) for _ in range(L)] for _ in range(2)]
            for k in range(2):
                for l in range(L):
                    pool[k][l].array[:] = img[k, l].reshape(-1)
            mode, spans, ora, outs = kv.launch(*quota), [], [], []
            h = kv.kvio_pool_create(L, H, De, 1, P, S, [m.ptr for m in pool[0]], [m.ptr for m in pool[1]], mode, mode, 2)
            for i in range(n):
                src, dst, table = Memory(kv, L * 2 * cap * R, 0, 1), Memory(kv, L * 2 * cap * R, 0, 0), Memory(kv, 16, 1, 1)
                src.array[:], dst.array[:] = rng.integers(0, 256, len(src.array), dtype=np.uint8), 0x55
                pages = perm[i * -(-T // P):(i + 1) * -(-T // P)].copy()
                table.array[:4 * len(pages)] = pages.view(np.uint8)
                spans.append((src.ptr, cap, T, table.ptr)), ora.append((src.array, cap, T, pages)), outs.append((dst, table))
                keep += [src, dst, table]
            kv.kvio_load(h, spans, 0, L)
            tiles, exp = kv._lib.emu_last_tiles(), img.copy()
            oracle.load_layout(exp[0], exp[1], P, ora, LAYOUT[2], num_heads=H)
            assert np.array_equal(np.stack([np.stack([m.array.reshape(S, R) for m in row]) for row in pool]), exp), (De, H, T, quota)
            kv.kvio_offload(h, [(o[0].ptr, cap, T, o[1].ptr) for o in outs], 0, L)
            for (dst, _), (_, _, _, pages) in zip(outs, ora):
                want = np.full(len(dst.array), 0x55, np.uint8)
                oracle.offload_layout(exp[0], exp[1], P, [(want, cap, T, pages)], LAYOUT[2], num_heads=H)
                assert np.array_equal(dst.array, want), (De, H, T, quota)
            if quota == (2, 64, kib) and most is not None:
                assert tiles <= most * L * 2 * n and kv._lib.emu_last_tiles() == tiles, (De, H, T, tiles)
            elif quota != (2, 64, kib) and De >= 64:
                assert tiles >= L * 2 * n * H, (De, H, T, quota, tiles)
            kv.kvio_pool_destroy(h)
            keep += pool[0] + pool[1]
        for m in keep:
            m.free()
    D = 64                                       # nothing to move: nothing launched
    pool = [Memory(kv, 4 * 2 * D, 1, 1) for _ in range(2)]
    h = kv.kvio_pool_create(1, 2, D, 1, 4, 4, [pool[0].ptr], [pool[1].ptr], kv.launch(1, 64, 4), kv.launch(1, 64, 4), 2)
    before = kv._lib.emu_launches()
    kv.kvio_load(h, [(0, 0, 0, 0)], 0, 1)
    assert kv._lib.emu_launches() == before
    kv.kvio_pool_destroy(h)


@pytest.fixture(scope="module")
def emulated(tmp_path_factory):
    out = {}
    for name, extra in (("whole", ()), ("split", ("-DKVIO_MAX_SPAN_VECS=40",)),
                        ("planes", ("-DKVIO_MAX_PLANES=4", "-DKVIO_PACED_LOAD_BYTES=65536"))):
        out[name] = str(tmp_path_factory.mktemp(name))
        build(out[name], extra)
    return out


@pytest.mark.parametrize("name,first,last,bad_page", [("whole", 0, 260, False), ("whole", 260, 320, True),
                                                      ("split", 320, 420, False), ("split", 420, 440, True),
                                                      ("planes", 440, 480, False)])
def test_library_on_emulated_waves(emulated, name, first, last, bad_page):
    """In a process of its own: an access out of bounds ends it."""
    code = (f"import sys; sys.path[:0] = [{ROOT!r}, {os.path.join(ROOT, 'tests')!r}]\n"
            f"import test_emulated_kernels as t\nt.run_cases({emulated[name]!r}, {first}, {last}, {bad_page})")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-200:] + r.stderr[-3000:]


@pytest.mark.parametrize("name", ["whole", "split"])
def test_noalloc_table_in_the_arguments(emulated, name):
    code = (f"import sys; sys.path[:0] = [{ROOT!r}, {os.path.join(ROOT, 'tests')!r}]\n"
            f"import test_emulated_kernels as t\nt.run_noalloc({emulated[name]!r}, {name == 'split'})")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-200:] + r.stderr[-3000:]


@pytest.mark.parametrize("name,run", [("planes", "run_staged_layers"), ("whole", "run_full_steps"),
                                      ("whole", "run_default_loads"), ("whole", "run_pauses"), ("planes", "run_load_pauses"),
                                      ("whole", "run_short_contexts")])
def test_launch_limits_and_steps(emulated, name, run):
    code = (f"import sys; sys.path[:0] = [{ROOT!r}, {os.path.join(ROOT, 'tests')!r}]\n"
            f"import test_emulated_kernels as t\nt.{run}({emulated[name]!r})")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-200:] + r.stderr[-3000:]
