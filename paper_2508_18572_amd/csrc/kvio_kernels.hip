// kvio_kernels.hip -- GPU-assisted paged-KV transfer kernels for gfx950 (CDNA4).
//
// Strata, Sec. 4.2: one kernel launch replaces many small DMA copies; each
// work item loads a small chunk of the source into registers and streams it
// to the destination, which may be pinned host memory read or written
// directly over the host link.  Sec. 4.2.1 / Fig. 6: the layout change between
// the contiguous host chunk and the layer-first paged pool is one extra
// offset computation per chunk.  Sec. 3.1 (Little's law, X = C * S / L): the
// host link is latency-bound for small transfers, so throughput comes from
// keeping many independent 16-byte requests in flight (C), not from larger
// pages (S).
//
// CDNA4 mapping
//   * A wavefront (64 lanes) owns one tile of 64 * U vectors of 16 bytes of one
//     plane (a contiguous run of a host chunk) of one context.  Tiles are cut
//     by vector and not by row, at 256-byte boundaries of the host address, so
//     that every row size fills its tiles and each wave-wide access covers 1 KiB
//     of consecutive host bytes.
//   * Page-offset expansion is wavefront-level: lane r resolves the pool slot of
//     the tile's row r with one coalesced page-table read and range-checks the
//     page; every vector then fetches its row's slot from the owning lane with a
//     cross-lane permute (ds_bpermute), so the page table is read once per row.
//   * A CU returns vector loads in order over all its waves: a page-table read
//     behind host reads takes a host round trip.  Loads therefore read a tile's
//     page-table entries one tile ahead, in front of the host reads.
//   * A step issues all U loads of a wave before any store (U KiB in flight per
//     wave); many waves over few workgroups keep the host link busy while
//     using a small part of the chip (Sec. 4.2: confine the I/O kernel to a
//     few compute units).
//   * Non-temporal loads and stores (Sec. 4.2: bypass the cache to limit
//     pollution of co-running kernels); stores into host memory also carry
//     the device-scope policy, which lets them fill the host link.
//   * Grid-stride over tiles in host-address order, so the waves of a launch
//     sweep a sliding window of consecutive host memory.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "kvio_internal.h"

namespace kvio {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Global address space: host-mapped and device memory are both reached with
// global_load / global_store (no flat-address aperture checks).
typedef __attribute__((address_space(1))) u32x4 gvec;

template <bool NT>
__device__ __forceinline__ u32x4 load16(const uint8_t *p) {
    const gvec *q = (const gvec *)(p);
    if constexpr (NT) {
        return __builtin_nontemporal_load(q);
    } else {
        return *q;
    }
}

template <bool NT>
__device__ __forceinline__ void store16(uint8_t *p, u32x4 v) {
    gvec *q = (gvec *)(p);
    if constexpr (NT) {
        __builtin_nontemporal_store(v, q);
    } else {
        *q = v;
    }
}

// The kernel arguments in the constant address space, where they lie: read
// through the scalar cache and known not to change, so that no store or atomic
// of a kernel makes the compiler read them again (or keep them, and with them
// the whole tile order, in vector registers).
#define KVIO_CONSTANT const __attribute__((address_space(4)))
typedef KVIO_CONSTANT CopyArgs Args;
typedef KVIO_CONSTANT SpanArg Span;

__device__ __forceinline__ Args &kernel_args() {
    return *reinterpret_cast<Args *>(reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()));
}

// A wave-uniform value, in scalar registers.
__device__ __forceinline__ int64_t scalar64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(static_cast<uint64_t>(v) >> 32));
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}

// Stores into pinned host memory (the offload's destination).  With the
// device-scope cache policy (SC1) a wave's 1 KiB stores reach the host link's
// full write rate, the copy engine's 57.0 GB/s, where the compiler's own
// stores (plain or non-temporal) top out 1-2.5% lower.  An SC1 store is
// acknowledged only once it has crossed the link, though, and a wave's next
// step waits for its earlier stores, so SC1 pays only when many bytes are in
// flight (the launcher decides, kSc1MinInflight).  No builtin selects SC1 for
// a global store, so that store is written out; "memory" keeps the compiler
// from moving other memory accesses across it, and the s_nop gives the two
// wait states CDNA3/4 require before a VALU may overwrite the data registers
// of a store wider than 64 bits (the compiler inserts them after its own
// stores but cannot see the store inside the asm).
template <bool NT, bool SC1>
__device__ __forceinline__ void store_host16(uint8_t *p, u32x4 v) {
    if constexpr (SC1) {
        gvec *q = (gvec *)(p);
        if constexpr (NT) {
            asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" : : "v"(q), "v"(v) : "memory");
        } else {
            asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(q), "v"(v) : "memory");
        }
    } else {
        store16<NT>(p, v);
    }
}

// The same store at an address in scalar registers (scalar64, taken where all
// lanes are active) plus a lane's 32-bit offset, which takes one address register for all stores of a step instead of two for each.
// The s_nop before it: a VMEM instruction may read a scalar register only five
// wait states after a VALU (v_readfirstlane) wrote it, which the compiler again
// cannot see to inside the asm.
template <bool NT, bool SC1>
__device__ __forceinline__ void store_host16(uint8_t *base, uint32_t off, u32x4 v) {
    if constexpr (SC1) {
        gvec *q = (gvec *)(base);
        if constexpr (NT) {
            asm volatile("s_nop 4\n\tglobal_store_dwordx4 %0, %1, %2 sc1 nt\n\ts_nop 1" : : "v"(off), "v"(v), "s"(q) : "memory");
        } else {
            asm volatile("s_nop 4\n\tglobal_store_dwordx4 %0, %1, %2 sc1\n\ts_nop 1" : : "v"(off), "v"(v), "s"(q) : "memory");
        }
    } else {
        store16<NT>(base + off, v);
    }
}

// n / d for n < 2^31 (see Divider).
__device__ __forceinline__ uint32_t div_small(uint32_t n, KVIO_CONSTANT Divider &d) {
    return static_cast<uint32_t>((static_cast<uint64_t>(n) * d.mul) >> d.shift);
}

// Largest span s >= lo with tile_prefix[s] <= w (binary search over the spans).
__device__ __forceinline__ int span_of(Args &a, int32_t w, int lo) {
    int hi = a.n_spans - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.tile_prefix[mid] <= w) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// A wave's position in the tile order: plane, tile inside the plane, the span
// that holds it and that span's last tile + 1.  The wave's tiles lie `waves`
// apart, so the next one is mostly in the same span of the same plane.
struct TileCursor {
    int32_t plane;
    int32_t w;
    int32_t end;
    int span;
};

__device__ __forceinline__ void cursor_to(Args &a, TileCursor &c, int from_span) {
    c.span = span_of(a, c.w, from_span);
    c.end = a.tile_prefix[c.span + 1];
}

__device__ __forceinline__ TileCursor cursor_at(Args &a, int32_t g) {
    TileCursor c;
    c.plane = static_cast<int32_t>(div_small(static_cast<uint32_t>(g), a.plane_div));
    c.w = g - c.plane * a.plane_tiles;
    cursor_to(a, c, 0);
    return c;
}

// Host layouts as the kernels see them: rows of one plane in one run (a token-
// major chunk's (layer, K|V), a head-major chunk's (layer, K|V, head)), or each
// row at an offset of its own (page-first).
constexpr int kHostTokenMajor = KVIO_HOST_TOKEN_MAJOR;
constexpr int kHostPageFirst = KVIO_HOST_PAGE_FIRST;
constexpr int kHostHeadMajor = KVIO_HOST_HEAD_MAJOR;

// A wave's tile: tile_vecs consecutive vectors of one plane of one span,
// counted from `first` to `end` (the vectors of the tile that exist).  All of
// it is wave-uniform and lives in scalar registers.  Tiles are cut by vector
// and not by row, so every lane of a step moves a vector whatever the row
// size, and the cuts lie at multiples of 256 host bytes, so that the reads and
// writes a wave sends over the link are whole.
struct Tile {
    uint8_t *host;     // address of the tile's vector 0 (page-first: of the chunk); may precede the span
    uint8_t *pool;     // the plane's pool layer (head-major: its head's column)
    int32_t left;      // vectors from vector 0 to the end of the span's plane
    int64_t safe;      // byte offset from `host` of a vector that exists
    const int32_t *table;   // the span's page table
    int32_t rows;           // and rows
    int32_t token0;         // context token of the span's row 0
    int32_t span;
    int32_t plane;     // page-first: (layer * 2 + K|V) of the chunk
    int32_t row0;      // first row (token) of the tile
    int32_t col0;      // column of vector 0 in row0; negative if vector 0 precedes the span
    int32_t first;
    int32_t end;
};

// The pool array of plane lkv = layer * 2 + K|V.
// The layer table is written before the launch and never during it, so it
// is read through the scalar cache: a vector load would wait its turn
// behind the compute unit's host reads.
// Without one it lies in the arguments, behind the spans.
__device__ __forceinline__ uint8_t *pool_layer(Args &a, int32_t lkv) {
    KVIO_CONSTANT uint64_t *layers = a.layers != nullptr
        ? reinterpret_cast<KVIO_CONSTANT uint64_t *>(reinterpret_cast<uintptr_t>(a.layers))
        : reinterpret_cast<KVIO_CONSTANT uint64_t *>(a.spans + a.n_spans);
    return reinterpret_cast<uint8_t *>(layers[(lkv & 1) * a.num_layers + (lkv >> 1)]);
}

template <int HL, bool WIDE>
__device__ __forceinline__ Tile locate(Args &a, const TileCursor &c) {
    Tile t;
    Span &sp = a.spans[c.span];
    int32_t lkv = c.plane, head = 0;
    if constexpr (HL == kHostHeadMajor) {
        lkv = static_cast<int32_t>(div_small(static_cast<uint32_t>(c.plane), a.head_div));
        head = c.plane - lkv * a.head_groups;
    }
    lkv += a.layer_begin * 2;
    t.span = c.span;
    t.table = sp.page_idx;
    t.rows = sp.num_tokens;
    t.token0 = sp.token0;
    t.plane = lkv;
    t.pool = pool_layer(a, lkv) + head * a.row_bytes;
    uint8_t *base = const_cast<uint8_t *>(sp.host);
    int32_t v0 = (c.w - a.tile_prefix[c.span]) * a.tile_vecs;
    if constexpr (HL != kHostPageFirst) {
        const int64_t plane = HL == kHostHeadMajor ? static_cast<int64_t>(lkv) * a.num_heads + head : lkv;
        base += plane * (sp.host_tokens * a.row_bytes);
        if constexpr (!WIDE) v0 -= static_cast<int32_t>(reinterpret_cast<uintptr_t>(base) >> 4) & a.cut_mask;
    }
    t.left = t.rows * a.vec_per_row - v0;
    t.row0 = static_cast<int32_t>(div_small(static_cast<uint32_t>(v0 > 0 ? v0 : 0), a.row_div));
    t.col0 = v0 - t.row0 * a.vec_per_row;
    t.first = v0 < 0 ? -v0 : 0;
    t.end = t.left < a.tile_vecs ? (t.left < 0 ? 0 : t.left) : a.tile_vecs;
    t.host = HL == kHostPageFirst ? base : base + static_cast<int64_t>(v0) * 16;
    t.safe = static_cast<int64_t>(t.left > 0 ? t.first : -v0) * 16;
    return t;
}

// The tile `waves` further on in the same span and plane, of one that begins
// inside the span: a dozen scalar instructions where locate takes over a
// hundred, which a wave would spend with none of its reads in flight.
template <int HL>
__device__ __forceinline__ void step_tile(Args &a, Tile &t) {
    if constexpr (HL != kHostPageFirst) t.host += static_cast<int64_t>(a.step_vecs) * 16;
    t.left -= a.step_vecs;
    t.end = t.left < a.tile_vecs ? (t.left < 0 ? 0 : t.left) : a.tile_vecs;
    t.row0 += a.step_rows;
    t.col0 += a.step_cols;
    if (t.col0 >= a.vec_per_row) {
        t.col0 -= a.vec_per_row;
        ++t.row0;
    }
}

// Lane r owns row row0 + r of the tile, if the tile can reach it and the span
// holds it.
__device__ __forceinline__ bool owns_row(Args &a, const Tile &t, int lane) {
    return lane < a.tile_rows && t.row0 < t.rows - lane;
}

// Lane r: the pool page that the page table gives row row0 + r (read only;
// checked by lane_slot).  Lanes without a row read the span's last entry, so
// the load carries no mask and the compiler counts it exactly.
__device__ __forceinline__ int32_t lane_page(Args &a, const Tile &t, int lane) {
    const uint32_t last = static_cast<uint32_t>(t.rows - 1);
    const uint32_t want = static_cast<uint32_t>(t.row0 + lane);
    return t.table[div_small(static_cast<uint32_t>(t.token0) + (want < last ? want : last), a.page_div)];
}

// Lane r: pool slot of row row0 + r given its page from lane_page, or -1 for
// lanes without a row and for an out-of-range page (recorded once in the error
// word, never dereferenced).
__device__ __forceinline__ int lane_slot(Args &a, const Tile &t, int lane, int32_t page) {
    const bool mine = owns_row(a, t, lane), valid = page >= 0 && page < a.num_pages;
    const uint32_t token = static_cast<uint32_t>(t.token0 + (mine ? t.row0 + lane : 0));
    const uint32_t cpage = div_small(token, a.page_div);
    const uint64_t bad = __ballot(mine && !valid);
    if (bad != 0) {                          // wave-uniform: every lane records the first bad row
        Span &sp = a.spans[t.span];
        const uint32_t at = __builtin_amdgcn_readlane(cpage, __builtin_ctzll(bad));
        const unsigned long long code = (static_cast<unsigned long long>(sp.origin + 1) << kErrSpanShift) |
                                        static_cast<unsigned long long>(sp.page_base + static_cast<int64_t>(at));
        atomicCAS(a.err, 0ull, code);
    }
    const uint32_t page_size = static_cast<uint32_t>(a.page_size);
    return mine && valid ? static_cast<int>(static_cast<uint32_t>(page) * page_size + (token - cpage * page_size)) : -1;
}

// Lane r, page-first host chunk (the layers of one context page stored
// together, Sec. 4.2.1 / Fig. 6): byte offset of row row0 + r of the tile's
// plane from the chunk start.  Rows of one page are contiguous; pages are
// L * 2 * P rows apart.  Lanes without a row get the span's last row.
__device__ __forceinline__ int64_t lane_host_row(Args &a, const Tile &t, int lane) {
    const uint32_t last = static_cast<uint32_t>(t.rows - 1);
    const uint32_t want = static_cast<uint32_t>(t.row0 + lane);
    const uint32_t token = static_cast<uint32_t>(t.token0) + (want < last ? want : last);
    const uint32_t cpage = div_small(token, a.page_div);
    const uint32_t off = token - cpage * static_cast<uint32_t>(a.page_size);
    return ((static_cast<int64_t>(cpage) * a.num_layers * 2 + t.plane) * a.page_size + off) * a.row_bytes;
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(v), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(static_cast<uint64_t>(v) >> 32), lane);
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}

// Row (from row0) and column of one lane's vectors, which lie 64 apart: from
// one vector to the next the row grows by 64 / V and the column by 64 % V (<
// V), with at most one carry, so only the first vector needs a division.  WIDE
// rows (V a multiple of 64) are walked by whole 64-vector chunks, on the
// scalar unit.
struct RowCol {
    int r, c;
};

template <bool WIDE>
__device__ __forceinline__ RowCol rowcol_of(Args &a, const Tile &t, int lane) {
    if constexpr (WIDE) return {0, t.col0};
    // cut_bias rows are added so that a vector before the span stays positive.
    const int j = t.col0 + lane + a.cut_bias * a.vec_per_row;
    const int r = static_cast<int>(div_small(static_cast<uint32_t>(j), a.row_div));
    return {r - a.cut_bias, j - r * a.vec_per_row};
}

__device__ __forceinline__ void advance64(Args &a, RowCol &p) {
    p.r += a.vec_step_rows;
    p.c += a.vec_step_cols;
    if (p.c >= a.vec_per_row) {
        p.c -= a.vec_per_row;
        ++p.r;
    }
}

// Vector k * 64 + lane of a tile exists (WIDE: the whole chunk k).
template <bool WIDE>
__device__ __forceinline__ bool exists(const Tile &t, int k, int lane) {
    if constexpr (WIDE) return k * 64 < t.end;
    return k * 64 + lane >= t.first && k * 64 + lane < t.end;
}

// Page-first: byte offset from the chunk of a lane's vector at p, given the
// lanes' row offsets.
template <bool WIDE>
__device__ __forceinline__ int64_t row_at(int64_t hoff, const RowCol &p, int lane) {
    const int64_t row = WIDE ? readlane64(hoff, p.r & 63)
                             : static_cast<int64_t>(__shfl(static_cast<long long>(hoff), p.r & 63));
    return row + p.c * 16 + (WIDE ? lane * 16 : 0);
}

// Slot of the row of a lane's vector at p, or -1.  WIDE rows take it with a
// readlane (scalar), others with a cross-lane permute.
template <bool WIDE>
__device__ __forceinline__ int slot_at(int slot, const RowCol &p) {
    return WIDE ? __builtin_amdgcn_readlane(slot, p.r & 63) : __shfl(slot, p.r & 63);
}

// Byte offset in the pool layer of a lane's vector at p, in slot s >= 0.
template <bool WIDE>
__device__ __forceinline__ int64_t pool_at(Args &a, int s, const RowCol &p, int lane) {
    return static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(s)) * static_cast<uint64_t>(a.pitch)) +
           p.c * 16 + (WIDE ? lane * 16 : 0);
}

// Host address of a lane's vector k of a tile.  Page-first rows lie apart: p is
// the vector's row and column and hoff the lanes' row offsets.  Elsewhere the
// tile is one run and both halves of its address are ready, the run's start in
// scalar registers.
template <bool WIDE, int HL>
__device__ __forceinline__ uint8_t *host_at(const Tile &t, int k, const RowCol &p, int64_t hoff, int lane) {
    if constexpr (HL == kHostPageFirst) return t.host + row_at<WIDE>(hoff, p, lane);
    return t.host + k * 1024 + lane * 16;
}

// Page-first: byte offsets from the chunk of a lane's U vectors of a tile.
// Elsewhere a tile is one run, and none are needed.
template <int U, bool WIDE, int HL>
__device__ __forceinline__ void host_rows(Args &a, const Tile &t, int lane, int64_t (&at)[U]) {
    if constexpr (HL == kHostPageFirst) {
        const int64_t hoff = lane_host_row(a, t, lane);
        RowCol p = rowcol_of<WIDE>(a, t, lane);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            at[k] = row_at<WIDE>(hoff, p, lane);
            advance64(a, p);
        }
    }
}

// The reads of a tile, all U behind one another; `at` from host_rows.  None
// carries a mask, so that the compiler counts them exactly (a precise wait for
// each).  A vector that does not move reads a place that exists and is
// discarded: the pool layer's first bytes, in device memory, or, in a wave's
// FIRST load tile, a host vector, so that the first reads of a launch wait for
// nothing but the kernel arguments.
template <int U, bool NT, bool WIDE, int HL, bool FIRST>
__device__ __forceinline__ void read_host(const Tile &t, const int64_t (&at)[U], int lane, u32x4 (&buf)[U]) {
    // Page-first: vector 0 of lane 0 is one of the tile's, or the span's last row's.
    const uint8_t *idle = !FIRST ? t.pool : t.host + (HL == kHostPageFirst ? readlane64(at[0], 0) : t.safe);
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const uint8_t *src = t.host + (HL == kHostPageFirst ? at[k] : static_cast<int64_t>(k * 1024 + lane * 16));
        buf[k] = load16<NT>(exists<WIDE>(t, k, lane) ? src : idle + (WIDE && !FIRST ? lane * 16 : 0));
    }
}

template <int U, bool NT, bool WIDE>
__device__ __forceinline__ void read_pool(Args &a, const Tile &t, int slot, int lane, u32x4 (&buf)[U]) {
    RowCol p = rowcol_of<WIDE>(a, t, lane);
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const int s = slot_at<WIDE>(slot, p);
        const int64_t off = pool_at<WIDE>(a, s, p, lane);
        buf[k] = load16<NT>(t.pool + (s >= 0 && exists<WIDE>(t, k, lane) ? off : 0));
        advance64(a, p);
    }
}

// Wait for the read of `v` and those before it; no access moves across.
__device__ __forceinline__ void arrive(u32x4 &v) { asm volatile("" : "+v"(v) : : "memory"); }

// The writes of a tile, each lane's behind its mask.  All reads have arrived
// before the first of them, on every path.  Left to itself the compiler waits
// inside each masked write, for the fewest operations that may be running
// there: its waits then take in the writes before, and where the paths around
// the last write meet, its read counts as still running and the next tile's
// reads wait for all of this tile's writes.
template <int DIR, int U, bool NT, bool SC1, bool WIDE, int HL>
__device__ __forceinline__ void write_tile(Args &a, const Tile &t, int slot, int lane, u32x4 (&buf)[U]) {
    const int64_t hoff = DIR == kOffload && HL == kHostPageFirst ? lane_host_row(a, t, lane) : 0;
    RowCol p = rowcol_of<WIDE>(a, t, lane);
#pragma unroll
    for (int k = 0; k < U; ++k) arrive(buf[k]);
#pragma unroll
    for (int k = 0; k < U; ++k) {
        // Every lane takes part in what the lanes exchange, also where some do
        // not store.
        const int s = slot_at<WIDE>(slot, p);
        const bool moves = s >= 0 && exists<WIDE>(t, k, lane);
        if constexpr (DIR == kLoad) {
            uint8_t *dst = t.pool + pool_at<WIDE>(a, s, p, lane);
            if (moves) store16<NT>(dst, buf[k]);
        } else {
            if constexpr (HL == kHostPageFirst) {
                uint8_t *dst = host_at<WIDE, HL>(t, k, p, hoff, lane);
                if (moves) store_host16<NT, SC1>(dst, buf[k]);
            } else {
                uint8_t *dst = reinterpret_cast<uint8_t *>(scalar64(reinterpret_cast<int64_t>(t.host + k * 1024)));
                if (moves) store_host16<NT, SC1>(dst, static_cast<uint32_t>(lane) * 16u, buf[k]);
            }
        }
        advance64(a, p);
    }
}

// Every argument that a launch's first reads depend on, in one batch of scalar
// loads: each batch is a round trip to memory, and left to itself the compiler
// spreads them over seven, one behind the other.
__device__ __forceinline__ void fetch_args(Args &a) {
    asm volatile("" : : "s"(a.total_tiles), "s"(a.waves_per_wg), "s"(a.layers), "s"(a.row_bytes), "s"(a.pitch), "s"(a.plane_tiles), "s"(a.planes), "s"(a.num_pages),
                 "s"(a.num_layers), "s"(a.layer_begin), "s"(a.page_size), "s"(a.vec_per_row), "s"(a.page_div.mul),
                 "s"(a.page_div.shift), "s"(a.row_div.mul), "s"(a.row_div.shift), "s"(a.tile_vecs), "s"(a.tile_rows),
                 "s"(a.cut_mask), "s"(a.n_spans), "s"(a.waves), "s"(a.tile_prefix[1]), "s"(a.spans[0].host),
                 "s"(a.spans[0].page_idx), "s"(a.spans[0].host_tokens), "s"(a.spans[0].num_tokens), "s"(a.spans[0].token0));
}

// What a paced wave sleeps behind a step that moved `vecs` vectors.
__device__ __forceinline__ void rest(Args &a, int vecs) {
    for (int i = static_cast<int>(static_cast<uint32_t>(a.pause) * static_cast<uint32_t>(vecs) >> 16); i > 0; --i) __builtin_amdgcn_s_sleep(1);
}

// The copy of one launch.  DIR: kLoad (host chunk -> pool) or kOffload (pool
// -> host chunk).  U: 16-byte vectors per lane per tile (one tile = up to U
// KiB per wave).  NT: non-temporal accesses.  SC1: offload host stores with
// the device-scope policy (store_host16).  WIDE: R is a multiple of 1 KiB.
// HL: host layout.
//
// A compute unit returns its vector loads in order, over all its waves.  A
// page-table read that a wave waits for before it issues its host reads
// therefore costs a whole host round trip (2-3 us) whenever a neighbour's host
// reads are ahead of it; waves in step (all reading the table, then all
// reading the host) hide this until one short tile puts a workgroup's waves
// out of step, which then ran at 65% of the other workgroups' rate and held
// the launch up (64 MiB of 384-byte rows: 47-50 GB/s with one short tile per
// plane, 57.2 without).  So the table entries of a wave's next tile are read
// right before the rows of the current one: they arrive, in order, before
// those do, and nothing else that a wave waits for stands behind a host read.
template <int DIR, int U, bool NT, bool SC1, bool WIDE, int HL>
__device__ __forceinline__ void copy_tiles(Args &a) {
    const int lane = threadIdx.x & 63;
    fetch_args(a);
    const int32_t g = static_cast<int32_t>(blockIdx.x) * a.waves_per_wg +
                      static_cast<int32_t>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
    if (g >= a.total_tiles) return;

    TileCursor cur = cursor_at(a, g);
    Tile t = locate<HL, WIDE>(a, cur);
    // The tile after x, and whether there is one; after the last it is x again, so
    // that every pass issues the same reads, in bounds.
    auto following = [&](const Tile &x, bool &there) {
        Tile n = x;
        int32_t w = cur.w + a.waves;
        if (w < cur.end && x.first == 0) {
            cur.w = w;
            step_tile<HL>(a, n);
            there = true;
            return n;
        }
        int32_t plane = cur.plane, from = cur.span;
        if (w >= a.plane_tiles) {                // into a later plane: its spans start over
            const int32_t planes = static_cast<int32_t>(div_small(static_cast<uint32_t>(w), a.plane_div));
            plane += planes;
            w -= planes * a.plane_tiles;
            from = 0;
        }
        there = plane < a.planes;
        if (there) {
            cur.plane = plane;
            cur.w = w;
            cursor_to(a, cur, from);
            n = locate<HL, WIDE>(a, cur);
        }
        return n;
    };
    u32x4 buf[U];
    bool more;
    if constexpr (DIR == kOffload) {
#pragma unroll 1
        do {
            const int slot = lane_slot(a, t, lane, lane_page(a, t, lane));
            read_pool<U, NT, WIDE>(a, t, slot, lane, buf);
            write_tile<DIR, U, NT, SC1, WIDE, HL>(a, t, slot, lane, buf);
            const int moved = t.end;
            t = following(t, more);
            if constexpr (!SC1) {
                if (more) rest(a, moved);
            }
        } while (more);
        return;
    }
    // The first tile, and the way to the third while its reads run.
    bool more_after;
    int64_t at[U];
    host_rows<U, WIDE, HL>(a, t, lane, at);
    read_host<U, NT, WIDE, HL, true>(t, at, lane, buf);
    int32_t page = lane_page(a, t, lane);
    Tile next = following(t, more);
    const int32_t next_page = lane_page(a, next, lane);
    int slot = lane_slot(a, t, lane, page);
    Tile after = following(next, more_after);
    int next_slot = lane_slot(a, next, lane, next_page);
    page = lane_page(a, after, lane);
    host_rows<U, WIDE, HL>(a, next, lane, at);
    write_tile<DIR, U, NT, SC1, WIDE, HL>(a, t, slot, lane, buf);
    if (!more) return;
    // The others: a tile's reads go out with its slots known, right behind the
    // writes of the one before; while they run, the wave takes the next tile's
    // slots from the entries it read a tile ago, finds the tile after that
    // and reads its entries.
#pragma unroll 1
    do {
        t = next;
        slot = next_slot;
        next = after;
        more = more_after;
        read_host<U, NT, WIDE, HL, false>(t, at, lane, buf);
        next_slot = lane_slot(a, next, lane, page);
        asm volatile("" : "+v"(next_slot));      // done with `page`, whose register the next read takes
        after = following(next, more_after);
        page = lane_page(a, after, lane);
        host_rows<U, WIDE, HL>(a, next, lane, at);
        if constexpr (HL == kHostPageFirst) {
            // worked out here, not when the tile's turn has come
#pragma unroll
            for (int k = 0; k < U; ++k) asm volatile("" : "+v"(at[k]));
        }
        write_tile<DIR, U, NT, SC1, WIDE, HL>(a, t, slot, lane, buf);
        if (a.pause != 0) {
            // In step, so that the pause leaves the compute unit's queue empty
            // (load_pause).  Waves that have ended are not waited for.
            __builtin_amdgcn_s_barrier();
            rest(a, t.end);
        }
    } while (more);
}

// Workgroup size bound of the kernels that need more than the 128 VGPRs per
// lane a 1024-thread workgroup leaves (page-first and head-major addressing,
// and loads of narrow token-major rows at 16 KiB steps); their launcher folds
// larger workgroups into more workgroups of this size.
constexpr int kNarrowBound = 256;

template <int DIR, int U, bool WIDE, int HL>
constexpr bool needs_narrow_bound() {
    return HL != KVIO_HOST_TOKEN_MAJOR || (DIR == kLoad && U == 16 && !WIDE);
}

template <int DIR, int U, bool NT, bool SC1, bool WIDE, int HL>
__global__ void __launch_bounds__((needs_narrow_bound<DIR, U, WIDE, HL>() ? kNarrowBound : 1024))
    kvio_copy_kernel(const CopyArgs) {
    copy_tiles<DIR, U, NT, SC1, WIDE, HL>(kernel_args());
}

// Head-major host chunk: one contiguous run per (layer, K|V, head).  A plane
// is one such run: its rows are the head's segments of De = R / H bytes, its
// pool rows lie R apart and start at the head's column.  So the head/token
// transpose of the layout conversion is the same address arithmetic as the
// paging, host accesses are whole runs whatever H, and nothing passes through
// LDS.  Against the transpose through LDS (below; host runs of 4 KiB / H), 64 MiB
// loads of segments of 64 bytes or more went from 35-57 to 56.6-57.2 GB/s over 1 to
// 32 heads.
template <int DIR, int U, bool NT, bool SC1>
__global__ void __launch_bounds__(kNarrowBound) kvio_head_major_kernel(const CopyArgs) {
    copy_tiles<DIR, U, NT, SC1, false, kHostHeadMajor>(kernel_args());
}

// ----------------------------------------------------------------------------
// Offloads on a small quota (below kSc1MinInflight: a background backup beside
// a load; also cached ones), from token-major and page-first chunks.  Their
// stores are the compiler's, acknowledged before they have crossed the link, so
// nothing tells a wave that the link is full, and what it sends too soon queues
// ahead of a co-running load's read requests (which PCIe lets pass no posted
// write).  These waves work in whole-row tiles, one step behind the other: slots,
// pool reads, host writes as the reads arrive, and a pause (pause_of).  At 16
// workgroups of one wave with 4 KiB steps, 336 MiB each way, beside a load, they
// led copy_tiles' offload, plain or overlapped, by 10 to 20 GB/s; with device-scope
// stores and overlap the load takes the whole link and the offload a third.
// Head-major offloads on such quotas run in copy_tiles, with the same pause.
// ----------------------------------------------------------------------------
// To the wave's next tile, if there is one.
__device__ __forceinline__ bool cursor_next(Args &a, TileCursor &cur) {
    int32_t from = cur.span;
    cur.w += a.waves;
    if (cur.w >= a.plane_tiles) {
        const int32_t planes = static_cast<int32_t>(div_small(static_cast<uint32_t>(cur.w), a.plane_div));
        cur.plane += planes;
        cur.w -= planes * a.plane_tiles;
        from = 0;
    }
    if (cur.plane >= a.planes) return false;
    if (from == 0 || cur.w >= cur.end) cursor_to(a, cur, from);
    return true;
}

struct RowTile {
    int span, layer, kv, group;              // group: of heads, where the launch transposes
    int t0, nrows;                           // first row in the span, and rows
};

__device__ __forceinline__ RowTile row_tile(Args &a, const TileCursor &c) {
    RowTile t;
    t.span = c.span;
    const int lkv = static_cast<int>(div_small(static_cast<uint32_t>(c.plane), a.head_div));
    t.group = c.plane - lkv * a.head_groups;
    t.layer = a.layer_begin + (lkv >> 1);
    t.kv = lkv & 1;
    t.t0 = (c.w - a.tile_prefix[c.span]) * a.tile_rows;
    const int left = a.spans[c.span].num_tokens - t.t0;
    t.nrows = left < a.tile_rows ? left : a.tile_rows;
    return t;
}

// Lane r: the pool page of the tile's row r (read only), of its last row where
// there is none, so that the load carries no mask.
__device__ __forceinline__ int32_t row_page(Args &a, Span &sp, const RowTile &t, int lane) {
    const int r = lane < t.nrows ? lane : t.nrows - 1;
    return sp.page_idx[div_small(static_cast<uint32_t>(sp.token0 + t.t0 + r), a.page_div)];
}

// And its pool slot, or -1 (see lane_slot).
__device__ __forceinline__ int row_slot(Args &a, Span &sp, const RowTile &t, int lane, int32_t page) {
    int slot = -1;
    if (lane < t.nrows) {
        const uint32_t token = static_cast<uint32_t>(sp.token0 + t.t0 + lane);
        const uint32_t cpage = div_small(token, a.page_div);
        if (page >= 0 && page < a.num_pages) {
            slot = static_cast<int>(static_cast<uint32_t>(page) * static_cast<uint32_t>(a.page_size) +
                                    (token - cpage * static_cast<uint32_t>(a.page_size)));
        } else {
            const unsigned long long code =
                (static_cast<unsigned long long>(sp.origin + 1) << kErrSpanShift) |
                static_cast<unsigned long long>(sp.page_base + static_cast<int64_t>(cpage));
            atomicCAS(a.err, 0ull, code);
        }
    }
    return slot;
}

template <int U, bool NT, bool WIDE, int HL>
__global__ void __launch_bounds__((HL != KVIO_HOST_TOKEN_MAJOR ? 256 : 1024)) kvio_copy_kernel_paced(const CopyArgs) {
    Args &a = kernel_args();
    const int lane = threadIdx.x & 63;
    const int32_t g = static_cast<int32_t>(blockIdx.x) * a.waves_per_wg +
                      static_cast<int32_t>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
    if (g >= a.total_tiles) return;
    TileCursor cur = cursor_at(a, g);
    int moved = 0;                           // vectors of the step before
#pragma unroll 1
    for (;;) {
        const RowTile t = row_tile(a, cur);
        Span &sp = a.spans[t.span];
        const uint8_t *pool = a.layers[t.kv * a.num_layers + t.layer];
        const int slot = row_slot(a, sp, t, lane, row_page(a, sp, t, lane));
        uint8_t *host = const_cast<uint8_t *>(sp.host);
        const int64_t plane = static_cast<int64_t>(t.layer) * 2 + t.kv;
        int64_t hoff = 0;                    // page-first: lane r's row r from the chunk
        if constexpr (HL == kHostPageFirst) {
            const uint32_t token = static_cast<uint32_t>(sp.token0 + t.t0 + (lane < t.nrows ? lane : 0));
            const uint32_t cpage = div_small(token, a.page_div);
            hoff = ((static_cast<int64_t>(cpage) * a.num_layers * 2 + plane) * a.page_size +
                    (token - cpage * static_cast<uint32_t>(a.page_size))) * a.row_bytes;
        } else {
            host += (plane * sp.host_tokens + t.t0) * a.row_bytes;
        }
        const int nvec = t.nrows * a.vec_per_row;
#pragma unroll 1
        for (int base = 0; base < nvec; base += 64 * U) {
            rest(a, moved);
            moved = nvec - base < 64 * U ? nvec - base : 64 * U;
            // Vector k: chunk base + k * 64 (WIDE, all lanes in one row) or this
            // lane's vector of it.
            const int j = base + (WIDE ? 0 : lane);
            const int r0 = static_cast<int>(div_small(static_cast<uint32_t>(j), a.row_div));
            RowCol p = {r0, j - r0 * a.vec_per_row};
            u32x4 buf[U];
            uint32_t moves = 0;
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int s = slot_at<WIDE>(slot, p);
                const bool ok = j + k * 64 < nvec && s >= 0;
                moves |= ok ? 1u << k : 0u;
                const int64_t off = pool_at<WIDE>(a, s, p, lane);
                buf[k] = load16<NT>(pool + (ok ? off : 0));
                advance64(a, p);
            }
            p = {r0, j - r0 * a.vec_per_row};
            auto at = [&](int k) -> uint8_t * {
                if constexpr (HL == kHostPageFirst) return host + row_at<WIDE>(hoff, p, lane);
                return host + static_cast<int64_t>(base + k * 64 + lane) * 16;
            };
            if (__all(moves == (1u << U) - 1u)) {
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    store16<NT>(at(k), buf[k]);
                    advance64(a, p);
                }
            } else {
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    uint8_t *dst = at(k);
                    if ((moves >> k) & 1u) store16<NT>(dst, buf[k]);
                    advance64(a, p);
                }
            }
        }
        if (!cursor_next(a, cur)) return;
    }
}

// ----------------------------------------------------------------------------
// Head-major chunks of narrow segments or few tokens, through LDS.  A wave owns a
// tile of n whole rows (of a row wider than a step, n is 1 and the tile a part of its
// heads) that fits its U KiB of LDS.  It reads the tile in
// host order (per head, n * De contiguous bytes), writes each vector to its
// place in pool order in its slice, and reads the slice back in pool order, so
// both sides are runs: host reads of n * De bytes, pool writes of whole rows.
// Offloads run the same two phases the other way round.  With Vd = De / 16 and V
// the vectors of a row of the tile:
//   pool order  p = r * V + h * Vd + c       (row r, head h, vector c)
//   host order  q = (h * n + r) * Vd + c
// A tile's page-table entries are read a tile ahead, as in copy_tiles.
// ----------------------------------------------------------------------------
template <int DIR, int U, bool NT, bool SC1>
__global__ void __launch_bounds__(kNarrowBound) kvio_head_transpose_kernel(const CopyArgs) {
    HIP_DYNAMIC_SHARED(u32x4, lds)           // U * 64 vectors per wave
    Args &a = kernel_args();
    const int lane = threadIdx.x & 63;
    const int wave_in_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t g = static_cast<int32_t>(blockIdx.x) * a.waves_per_wg + wave_in_wg;
    if (g >= a.total_tiles) return;
    u32x4 *slice = lds + wave_in_wg * (U * 64);
    const int Vd = a.vec_per_row;
    // The wave's lanes exchange data through its slice: what was written is there.
    auto exchange = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    TileCursor cur = cursor_at(a, g);
    RowTile t = row_tile(a, cur), next = t;
    int32_t page = row_page(a, a.spans[t.span], t, lane);
    asm volatile("" : : : "memory");         // ahead of the tile's reads
    bool more = true;
    auto look_ahead = [&] {
        asm volatile("" : "+v"(page) : : "memory");      // done with it
        more = cursor_next(a, cur);
        if (more) next = row_tile(a, cur);
        page = row_page(a, a.spans[next.span], next, lane);
        asm volatile("" : : : "memory");
    };
#pragma unroll 1
    for (;; t = next) {
        Span &sp = a.spans[t.span];
        const int32_t lkv = t.layer * 2 + t.kv;
        const int head0 = t.group * a.heads_per_tile;
        const int heads = a.num_heads - head0 < a.heads_per_tile ? a.num_heads - head0 : a.heads_per_tile;
        uint8_t *pool = pool_layer(a, lkv) + head0 * a.row_bytes;
        const int n = t.nrows, V = heads * Vd, nvec = n * V;      // the last group may be smaller; n is 1 where there are several
        const int64_t head_stride = sp.host_tokens * a.row_bytes;
        // The first head's run at the tile's first row.
        uint8_t *host = const_cast<uint8_t *>(sp.host) + (static_cast<int64_t>(lkv) * a.num_heads + head0) * head_stride + t.t0 * a.row_bytes;
        // Vector q of the tile in host order: its place in pool order, its row and
        // its byte offset from `host`.
        struct Host { int pool, r; int64_t off; };
        auto host_order = [&](int q) -> Host {
            const int hr = static_cast<int>(div_small(static_cast<uint32_t>(q), a.row_div));
            const int h = static_cast<int>(static_cast<unsigned>(hr) / static_cast<unsigned>(n)), r = hr - h * n, c = q - hr * Vd;
            return {r * V + h * Vd + c, r, h * head_stride + static_cast<int64_t>(r * Vd + c) * 16};
        };
        u32x4 buf[U];
        if constexpr (DIR == kLoad) {
            int pos[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int q = k * 64 + lane;
                const Host x = host_order(q);
                pos[k] = q < nvec ? x.pool : -1;
                buf[k] = load16<NT>(q < nvec ? host + x.off : pool);
            }
            const int slot = row_slot(a, sp, t, lane, page);
            look_ahead();
#pragma unroll
            for (int k = 0; k < U; ++k) arrive(buf[k]);
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (pos[k] >= 0) slice[pos[k]] = buf[k];
            exchange();
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int p = k * 64 + lane;
                const int r = static_cast<int>(div_small(static_cast<uint32_t>(p), a.part_div));
                const int s = __shfl(slot, r & 63);
                if (p < nvec && s >= 0) store16<NT>(pool + s * a.pitch + (p - r * V) * 16, slice[p]);
            }
        } else {
            const int slot = row_slot(a, sp, t, lane, page);
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int p = k * 64 + lane;
                const int r = static_cast<int>(div_small(static_cast<uint32_t>(p), a.part_div));
                const int s = __shfl(slot, r & 63);
                buf[k] = load16<NT>(pool + (p < nvec && s >= 0 ? s * a.pitch + (p - r * V) * 16 : 0));
            }
            look_ahead();
#pragma unroll
            for (int k = 0; k < U; ++k) arrive(buf[k]);
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (k * 64 + lane < nvec) slice[k * 64 + lane] = buf[k];
            exchange();
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int q = k * 64 + lane;
                const Host x = host_order(q);
                const int s = __shfl(slot, x.r & 63);
                if (q < nvec && s >= 0) store_host16<NT, SC1>(host + x.off, slice[x.pool]);
            }
        }
        exchange();                          // the next tile takes the slice
        if (!more) return;
    }
}

template <int DIR, int U, bool NT, bool SC1, int HL>
static void launch_layout(const CopyArgs &a, dim3 grid, dim3 block, hipStream_t stream) {
    if constexpr (HL == kHostHeadMajor) {
        if (a.transpose)
            hipLaunchKernelGGL((kvio_head_transpose_kernel<DIR, U, NT, SC1>), grid, block,
                               static_cast<size_t>(block.x / 64) * U * 1024, stream, a);
        else
            hipLaunchKernelGGL((kvio_head_major_kernel<DIR, U, NT, SC1>), grid, block, 0, stream, a);
    } else {
        const bool wide = a.vec_per_row % 64 == 0;
        if constexpr (DIR == kOffload && !SC1) {
            if (a.whole_rows) {
                if (wide)
                    hipLaunchKernelGGL((kvio_copy_kernel_paced<U, NT, true, HL>), grid, block, 0, stream, a);
                else
                    hipLaunchKernelGGL((kvio_copy_kernel_paced<U, NT, false, HL>), grid, block, 0, stream, a);
                return;
            }
        }
        if (wide)
            hipLaunchKernelGGL((kvio_copy_kernel<DIR, U, NT, SC1, true, HL>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((kvio_copy_kernel<DIR, U, NT, SC1, false, HL>), grid, block, 0, stream, a);
    }
}

// Offloads on a small quota move kPacedMBps and no more: a wave sleeps behind each
// step for what the step's share of that rate leaves (above some 48 GB/s the
// link's write side fills, a load's read requests stand behind it, and both ways
// together fall to 60-75 GB/s).  `takes` is a step's time where few waves run, in ns,
// taken from steps of 4 to 16 KiB over row sizes: the table's read once a tile, and
// the rows' way through the wave, longer where rows fill no step or lie apart
// (head-major).  No sleep where the quota does not reach the rate, none of more than
// kPacedSleep ns (the waves of such quotas wait for one another long before: 8
// workgroups of 4 waves x 4 KiB moved 2 MiB in 80 us, without in 56), and none with more
// than four waves in a workgroup (2 x 1024 threads are bound by their compute units:
// 53.7 GB/s alone, 33 if they slept too).
// 192 MiB each way, GB/s until both are done | offload alone, with a constant 0.16 us
// behind each tile and as now:
//   16 waves x 4 KiB, rows of 1 KiB 91|46.7, 93|47.2; 2 KiB 83|48.7, 90|48.9; 512 bytes
//     83|50.8, 94|48.7; 8 KiB 71|45.0, 92|46.9; head-major (which had no sleep) 70|54.8, 90|46.1
//   rows of 1 KiB: 8 waves x 4 KiB 47|23.4, 55|27.4; 12 x 8 KiB 69|54.6, 90|45.3; 8 x 16 75|52.8,
//     91|46.4; no sleep: 16 x 8 77|40.2, 79|43.9, 8 workgroups of 4 x 4 KiB 83|45.5, 78|48.8
constexpr int64_t kPacedMBps = 46500;
constexpr int64_t kPacedSleep = 700;
constexpr int kPacedWavesPerWg = 4;
// Of loads: ns of an unhindered step of 4 KiB, longer where rows lie apart, and the
// longest sleep.
constexpr int64_t kLoadMBps = 57400;
constexpr int64_t kLoadTrip = 2360;
constexpr int64_t kLoadTripPageFirst = 2760;
constexpr int64_t kLongestRest = 1000;
constexpr int kLoadWavesPerWg = 6;

static int32_t pause_of(const CopyArgs &a, int U) {
    const int64_t tile = a.whole_rows ? int64_t(a.tile_rows) * a.vec_per_row : a.tile_vecs;
    const int64_t steps = (tile + 64 * U - 1) / (64 * U), step = std::min<int64_t>(tile, 64 * U);
    if (a.waves_per_wg > kPacedWavesPerWg) return 0;
    const int64_t takes = a.host_layout == kHostHeadMajor ? 610 + step * 16 * 153 / 1024
                                                          : 410 + step * 16 * (step < 64 * U ? 100 : 80) / 1024 + 480 / steps;
    const int64_t spare = a.waves * step * 16 * 1000 / kPacedMBps - takes;
    return spare <= 0 || spare > kPacedSleep ? 0 : static_cast<int32_t>((spare << 16) / 26 / step + 1);      // 26 ns: 64 cycles
}

// Loads of kPacedLoadBytes or more: the waves of a workgroup wait for one another
// behind a step and then sleep for what the step would otherwise queue for on the
// link, its share of the link's rate less the way of an unhindered step.  A compute
// unit returns its vector loads in order, so while its waves keep host reads in
// flight without a gap, every load of a kernel that shares it takes a host round
// trip.  And reads that queue on the link slow an offload beside them.
// A decode step of 7.3 ms beside loads (ms | the load's GB/s), a load alone, and
// with a background offload beside (both together), 39 waves; 48 waves:
//   neither          21.6 | 56.2   57.5    98.8;  26.6 | 56.8   57.5    94.9
//   in step          11.9 | 56.7   57.5    97.8;  19.6 | 57.2   57.5    94.0
//   slept, 0.4 us    17.0 | 55.2   57.3   102.3;  20.6 | 56.0   57.3    94.7
//   as now           11.3 | 55.8   57.4   102.6;  10.5 | 56.5   57.5   102.5
// Alone, 48 MiB of 2 KiB rows: 16 x 192 879 us without, 881 as now, 8 x 384 894, 880, 16 x 256
// 884, 879.  Not for larger steps, whose way is longer (16 x 192 of 8 KiB 881, 929), nor
// workgroups bound by their compute units (4 x 1024 1156, 1213).
static int32_t load_pause(const CopyArgs &a) {
    if (a.tile_vecs > 256 || a.waves_per_wg > kLoadWavesPerWg) return 0;
    int64_t rows = 0;
    for (int32_t i = 0; i < a.n_spans; ++i) rows += a.spans[i].num_tokens;
    const int64_t plane = rows * a.vec_per_row * a.heads_per_tile;          // vectors
    if (plane < kPacedLoadBytes / 16 / a.planes) return 0;
    const int64_t step = std::max<int64_t>(plane / a.plane_tiles, 1);
    const int64_t trip = a.host_layout == KVIO_HOST_PAGE_FIRST ? kLoadTripPageFirst : kLoadTrip;
    const int64_t spare = std::min(a.waves * step * 16 * 1000 / kLoadMBps - trip, kLongestRest);
    return spare <= 0 ? 0 : static_cast<int32_t>((spare << 16) / 26 / step + 1);
}

template <int DIR, int U, bool NT, bool SC1>
static hipError_t launch_u(CopyArgs &a, const Shape &s, hipStream_t stream) {
    dim3 grid(s.workgroups), block(s.threads);
    // The bound goes by the step asked for, also where a smaller one serves (small
    // tiles of narrow rows).  2 x 1024 threads with 16 KiB steps would otherwise read
    // the link from two compute units, at 21 GB/s (rows of 112 bytes; 56.2 folded).
    const bool narrow_bound = a.host_layout != KVIO_HOST_TOKEN_MAJOR ||
                              (DIR == kLoad && s.tile_kib == 16 && a.vec_per_row % 64 != 0);
    if (narrow_bound && s.threads > kNarrowBound) {
        grid = dim3(static_cast<unsigned>(int64_t(s.workgroups) * s.threads / kNarrowBound));
        block = dim3(kNarrowBound);
    }
    a.waves_per_wg = static_cast<int32_t>(block.x / 64);
    a.waves = static_cast<int32_t>(grid.x) * a.waves_per_wg;
    a.step_vecs = a.waves * a.tile_vecs;         // used where it stays inside a span
    a.step_rows = a.step_vecs / a.vec_per_row;
    a.step_cols = a.step_vecs % a.vec_per_row;
    a.pause = s.local || a.transpose ? 0 : DIR == kLoad ? load_pause(a) : SC1 ? 0 : pause_of(a, U);
    switch (a.host_layout) {
        case kHostPageFirst: launch_layout<DIR, U, NT, SC1, kHostPageFirst>(a, grid, block, stream); break;
        case kHostHeadMajor: launch_layout<DIR, U, NT, SC1, kHostHeadMajor>(a, grid, block, stream); break;
        default: launch_layout<DIR, U, NT, SC1, kHostTokenMajor>(a, grid, block, stream);
    }
    return hipGetLastError();
}

template <int DIR, bool NT, bool SC1>
static hipError_t launch_step(CopyArgs &a, const Shape &s, hipStream_t stream) {
    // The smallest step that holds a tile (rows below 64 bytes make small ones).
    if (a.tile_vecs <= 256) return launch_u<DIR, 4, NT, SC1>(a, s, stream);
    if (a.tile_vecs <= 512) return launch_u<DIR, 8, NT, SC1>(a, s, stream);
    return launch_u<DIR, 16, NT, SC1>(a, s, stream);
}

hipError_t launch_copy(CopyArgs &a, Direction dir, const Shape &s, hipStream_t stream) {
    if (dir == kLoad)
        return s.nontemporal ? launch_step<kLoad, true, false>(a, s, stream) : launch_step<kLoad, false, false>(a, s, stream);
    if (s.device_scope) return launch_step<kOffload, true, true>(a, s, stream);
    return s.nontemporal ? launch_step<kOffload, true, false>(a, s, stream)
                         : launch_step<kOffload, false, false>(a, s, stream);
}

}  // namespace kvio
