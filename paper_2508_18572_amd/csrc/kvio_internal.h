// kvio_internal.h -- what the C ABI layer hands to the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kvio.h"

namespace kvio {

// One cached context as the kernel sees it: the device-visible address of its
// host chunk, its page table and its sizes.
struct SpanArg {
    const uint8_t *host;       // device-visible address of the chunk
    const int32_t *page_idx;   // device page table
    int64_t host_tokens;       // per-(layer, K|V) token stride of the chunk
    int32_t num_tokens;        // tokens to move; num_tokens * vec_per_row <= kMaxSpanVecs
    int32_t origin;            // index of the caller's span (error records)
    int32_t page_base;         // context page of page_idx[0] (error records)
    int32_t token0;            // context token of row 0, counted from page_idx[0] (page-first: and from `host`)
};

// Division of n < 2^31 by a fixed d in [1, 2^31): (n * mul) >> shift with shift
// = 31 + ceil(log2 d) and mul = ceil(2^shift / d) < 2^32.  mul * d exceeds
// 2^shift by less than d, so the quotient is exact for n < 2^31.
struct Divider {
    uint32_t mul;
    uint32_t shift;
};

inline Divider divider(int64_t d) {
    uint32_t s = 0;
    while ((int64_t(1) << s) < d) ++s;
    return {static_cast<uint32_t>(((uint64_t(1) << (31 + s)) + uint64_t(d) - 1) / uint64_t(d)), 31 + s};
}

// Kernel arguments of one launch.  Passed by value (kernarg segment), so every
// launch carries its own span table and no device staging buffer is shared
// between calls on different streams.
//
// Work decomposition: a "plane" is one run of host rows of the launch's layer
// range -- a (layer, K|V), or for head-major chunks a (layer, K|V, head), where the
// launch transposes a (layer, K|V) and all its heads or a group of them --
// planes ordered layer-major; a "tile" is tile_vecs consecutive 16-byte vectors
// of one span in one plane.  tile_prefix[s] is the first tile of span s inside
// a plane, so a plane holds plane_tiles = tile_prefix[n_spans] tiles and the
// launch total_tiles = planes * plane_tiles.
//
// Tiles of narrow rows are cut where (host address / 16) & cut_mask is 0 (the
// first tile of a plane is shorter by what precedes the plane's first vector).
struct CopyArgs {
    // Device table: layers[kv * num_layers + l].  Null: the table lies behind the
    // last span, in the place of spans that the launch does not have (loads, and
    // offloads that are not paced).
    uint8_t *const *layers;
    unsigned long long *err;       // device error record (0 = none)
    int64_t row_bytes;             // bytes of a host row: R, or De for head-major chunks
    int64_t pitch;                 // bytes from one pool row to the next: R
    int64_t num_pages;             // S / P
    int64_t total_tiles;           // planes * plane_tiles
    int32_t planes;
    int32_t plane_tiles;
    int32_t num_layers;            // L, stride of the layer table
    int32_t layer_begin;
    int32_t page_size;             // P
    int32_t vec_per_row;           // V = row_bytes / 16
    Divider page_div;              // by P
    Divider row_div;               // by V
    Divider head_div;              // by head_groups
    Divider part_div;              // by heads_per_tile * V
    Divider plane_div;             // by plane_tiles
    int32_t vec_step_rows;         // 64 / V: rows a lane's vector index advances per 64 vectors
    int32_t vec_step_cols;         // 64 % V: and columns (carried into the row at V)
    int32_t tile_vecs;             // vectors per tile, a multiple of 64
    int32_t tile_rows;             // rows a tile can touch, 1 .. 64
    int32_t cut_mask;
    int32_t cut_bias;              // rows that cover cut_mask vectors
    int32_t whole_rows;            // tiles are tile_rows whole rows
    int32_t n_spans;               // spans in this launch, 1 .. KVIO_MAX_SPANS_PER_LAUNCH
    int32_t host_layout;           // KVIO_HOST_*
    int32_t num_heads;             // H (head-major chunks)
    int32_t transpose;             // head-major: tiles are tile_rows rows of heads_per_tile heads
    int32_t heads_per_tile;        // 1, or where the launch transposes: all heads, or of a row wider than a step, as many as fit
    int32_t head_groups;           // planes of a (layer, K|V): ceil(H / heads_per_tile) for head-major chunks, else 1
    // Set by launch_copy: waves of a workgroup and of the launch, and the vectors,
    // rows and columns from a wave's tile to its next one.
    int32_t waves_per_wg;
    int32_t waves;
    int32_t step_vecs;
    int32_t step_rows;
    int32_t step_cols;
    int32_t pause;                 // sleep behind a step, in 64 cycles / 2^16 for each vector it moved
    int32_t tile_prefix[KVIO_MAX_SPANS_PER_LAUNCH + 1];
    SpanArg spans[KVIO_MAX_SPANS_PER_LAUNCH];
};

// Spans a launch may hold beside a layer table of its own: 64 - ceil(2 L / 5).
static_assert(sizeof(SpanArg) == 40, "kvio.h states how many spans go beside the layer table");
inline int32_t spans_beside_table(int32_t num_layers) {
    return KVIO_MAX_SPANS_PER_LAUNCH - static_cast<int32_t>((2 * int64_t(num_layers) * sizeof(uint8_t *) + sizeof(SpanArg) - 1) / sizeof(SpanArg));
}

// Most vectors of a span in one plane and most planes of a launch: what lies in
// a plane is counted in 32 bits.  Larger transfers are split by the host (a
// build may lower them to have small ones split).
#ifndef KVIO_MAX_SPAN_VECS
#define KVIO_MAX_SPAN_VECS (int64_t(1) << 30)
#endif
#ifndef KVIO_MAX_PLANES
#define KVIO_MAX_PLANES (int64_t(1) << 30)
#endif
constexpr int64_t kMaxSpanVecs = KVIO_MAX_SPAN_VECS;
constexpr int64_t kMaxPlanes = KVIO_MAX_PLANES;
constexpr int64_t kMaxWaves = int64_t(1) << 20;

enum Direction { kLoad = 0, kOffload = 1 };

// Resolved launch shape (every field valid).
struct Shape {
    int workgroups;
    int threads;
    int tile_kib;      // 4, 8 or 16: vectors of 16 B per lane per step
    bool nontemporal;
    bool device_scope;  // offload host stores with the device-scope (SC1) policy
    bool grows;         // the grid is the library's: it may grow for short spans
    bool local;         // the chunks lie in the memory of the pool's own GPU
    int lds_below;      // head-major chunks: segments of fewer 16-byte vectors go through LDS
};

// Library defaults for the launch shape, chosen by measurement on MI355X
// (PCIe Gen5 x16 host link), on 16 of the 256 CUs for large loads.
//   Load of 32 MiB or more: 16 workgroups x 3 waves, 4 KiB steps (192 KiB in
//   flight), which pause between steps (load_pause): 57.5 GB/s alone, beside a
//   background offload 102.5 both ways.  39 waves reach 57.2-57.4 and 102.6.
//   Loads below that: 64 waves, 16 x 4 below 4 MiB and 32 x 2 above.  48 waves take
//   as long alone (2 MiB of 512-byte rows 40.1 against 40.4 us), but on two streams,
//   each with contexts of its own, 1.5 to 3% longer at every size (8 MiB: 155 against
//   151 us).  Four waves on a CU lead two on small loads (256 KiB 8.3 against 8.6 us,
//   on two streams 6.5 against 7.2) and are 0.5% behind from 8 MiB on; page-first,
//   whose waves also work out row offsets, 2% behind from 1 MiB on.
//   Offload: 32 workgroups x 4 waves with 16 KiB steps (57.0 GB/s with the
//   device-scope host stores).  Page-first offloads take 64 x 4 waves with 8 KiB
//   steps: 56.6-57.1 GB/s against 56.0-57.0 with 128 waves of 16 KiB (the same
//   2 MiB in flight), ahead at every row width (2-4 GiB, page sizes 1 and 16).
// A default grid grows until as many bytes are in flight where tiles are mostly
// empty, because spans are short, up to kMostGrowth times (64 head-major contexts of 1 to 7
// tokens, rows of 512 bytes: 2.4 times faster than without, token-major 1.2; no
// effect on a background offload beside: 91.4 against 91.3 GB/s both ways), and for
// loads where rows are too narrow to fill a step (a tile's 64 rows of 16 bytes are 1 KiB).
constexpr int kDefaultThreads = 256;
constexpr Shape kDefaultLoad = {16, 192, 4, true, false, false, false, 0};
constexpr Shape kDefaultLoadMiddle = {32, 128, 4, true, false, false, false, 0};
constexpr Shape kDefaultLoadSmall = {16, kDefaultThreads, 4, true, false, false, false, 0};
constexpr int64_t kMiddleLoadBytes = int64_t(32) << 20;
#ifndef KVIO_PACED_LOAD_BYTES
#define KVIO_PACED_LOAD_BYTES kMiddleLoadBytes
#endif
constexpr int64_t kPacedLoadBytes = KVIO_PACED_LOAD_BYTES;      // a build may have small loads paced
constexpr int64_t kSmallLoadBytes = int64_t(4) << 20;
constexpr int64_t kSmallLoadBytesPageFirst = int64_t(512) << 10;
constexpr Shape kDefaultOffload = {32, kDefaultThreads, 16, true, false, false, false, 0};
constexpr Shape kDefaultOffloadPageFirst = {64, kDefaultThreads, 8, true, false, false, false, 0};
constexpr int64_t kMostGrowth = 8;
// Head-major chunks whose segments are narrower than this many 16-byte vectors go
// through LDS.  By address (a tile is one head's run of up to 64 rows) a step of
// 16-byte segments holds 1 KiB, and its pool accesses are 16 bytes each; through
// LDS a tile holds whole rows of all heads, and host runs and pool rows are both
// long.  64 MiB, by address and through LDS, GB/s:
//   loads     8 heads of 16 bytes 30.0, 57.3; 32 of 32 54.3, 57.2; 16 of 48 54.0, 50.1
//   offloads  8 heads of 16 bytes 56.0, 56.5; 32 of 32 53.8, 56.3; 16 of 48 53.6, 54.2
//   2 MiB     8 of 16: load 28.4, 50.7, offload 53.0, 50.3; 16 of 48: 49.7, 45.1, 50.5, 46.1
//   quota of 8 x 256, 4 KiB steps: load 8 of 16 19.6, 42.6, offload 24.8, 43.4
//   chunks in device memory: load 8 of 16 392, 2640, offload 1115, 2650
// At 64 bytes the direct path leads (loads 57.2 against 56.7).  Loads take 32 waves
// of 8 KiB steps at every size: 48 are 5% slower, 4 KiB steps 45% (the host runs of
// a tile are its step divided by the heads).
constexpr int kTransposeBelow = 4;
constexpr Shape kDefaultLoadTranspose = {16, 128, 8, true, false, false, false, 0};
inline bool transposes(int host_layout, int lds_below, int num_heads, int64_t seg_bytes, int tile_kib) {
    return host_layout == KVIO_HOST_HEAD_MAJOR && num_heads > 1 && seg_bytes < int64_t(lds_below) * 16 &&
           (lds_below > kTransposeBelow || num_heads * seg_bytes <= int64_t(tile_kib) * 1024);
}
// Chunks in the memory of the pool's own GPU (a copy between two caches, a gather
// for a consumer there): nothing crosses the host link, so the whole chip copies,
// with the compiler's stores.  256 MiB of 2 KiB rows in 90-93 us each way (5.9 TB/s
// read and written) where the shapes and stores for host memory took 2039 and 587;
// 256 to 2048 workgroups and steps of 4 to 16 KiB differ by 5%.
constexpr Shape kDefaultLocal = {1024, kDefaultThreads, 4, true, false, false, true, 0};

// The default shape of a call that moves `bytes` in direction `dir` between
// the pool and host chunks of layout `host_layout` (KVIO_HOST_*), head-major ones
// with `num_heads` segments of `seg_bytes`.
inline Shape default_shape(int dir, int64_t bytes, int host_layout, int lds_below, int num_heads, int64_t seg_bytes) {
    if (dir != 0) return host_layout == KVIO_HOST_PAGE_FIRST ? kDefaultOffloadPageFirst : kDefaultOffload;
    if (transposes(host_layout, lds_below, num_heads, seg_bytes, kDefaultLoadTranspose.tile_kib)) return kDefaultLoadTranspose;
    const int64_t small = host_layout == KVIO_HOST_PAGE_FIRST ? kSmallLoadBytesPageFirst : kSmallLoadBytes;
    return bytes < small ? kDefaultLoadSmall : bytes < kMiddleLoadBytes ? kDefaultLoadMiddle : kDefaultLoad;
}
// Offloads whose quota keeps at least this many bytes in flight (waves x step)
// store into host memory with the SC1 policy: enough to cover the longer
// acknowledgement of those stores, so the link runs at its full write rate (57.0
// against 55.7 GB/s at the default 128 waves x 16 KiB).  Smaller quotas (16 waves
// x 4 KiB: 27 against 44 GB/s) keep the plain policy.  The quota decides and not what
// a short call leaves of it: default offloads of 32 to 512 KiB take 4.0-12.5 us with
// SC1 and 4.6-13.1 with plain stores (page-first of 2 MiB alone 41.3 and 40.2).  A build may move the
// threshold (-DKVIO_SC1_MIN_INFLIGHT=0 stores every offload with SC1; a huge value
// never does), which is how both policies were measured over launch shapes.
#ifndef KVIO_SC1_MIN_INFLIGHT
#define KVIO_SC1_MIN_INFLIGHT (int64_t(512) << 10)
#endif
constexpr int64_t kSc1MinInflight = KVIO_SC1_MIN_INFLIGHT;

// Staged transfers: the scatter / gather between the HBM staging buffer and
// the pool is HBM-bound, so it takes the whole chip (4 GiB of 2 KiB rows at
// page size 1 in 1.75 ms, 2.4 TB/s of payload).
constexpr Shape kDefaultStaged = {1024, kDefaultThreads, 16, true, false, false, true, 0};

// Fill in how the vectors of a plane are cut into tiles, from row_bytes and
// host_layout: tiles of up to tile_kib KiB that touch at most 64 rows (a lane
// of the wave resolves each row's slot).
// Offloads into host memory without the SC1 policy, token-major and page-first, take
// tiles of up to 64 whole rows instead (tile_rows of them, counted by
// whole_rows).
void cut_tiles(CopyArgs *a, const Shape &shape, Direction dir);
// Take spans[n_spans], which is filled in, into the launch.
void add_span(CopyArgs *a);

// Enqueue one copy kernel.  `a` must be populated but for what this sets.
hipError_t launch_copy(CopyArgs &a, Direction dir, const Shape &shape, hipStream_t stream);

// Error record layout: bits 40..63 = span index + 1, bits 0..39 = context page.
constexpr int kErrSpanShift = 40;

}  // namespace kvio
