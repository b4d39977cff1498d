// Internal declarations shared by the planner and the runtime.
#pragma once

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <memory>
#include <string>
#include <vector>

#include "ii.h"
#include "scatter_math.h"
#include "scatter_types.h"

namespace ii {

constexpr uint32_t kDefaultTile = 4u << 10;  // segment bytes per workgroup (<= kMaxTile)
constexpr uint32_t kMaxLanes = 4;             // streams a ring's chunks alternate between
constexpr uint64_t kIoAlign = 4096;           // block alignment of direct-I/O file reads
constexpr uint64_t kCopyAlign = 256;          // host-to-device copies start and end on these
constexpr uint32_t kMaxDmaGroups = 2;         // most copies a pinned chunk is moved with

// How a load from a pinned blob moves one chunk of a plan with gaps.
enum PinnedMove : uint8_t {
    kPinnedInPlace = 0,  // one copy of the used range, gaps included, at chunk offsets
    kPinnedGroups = 1,   // one 1-D or 2-D copy per run group, into the packed layout
    kPinnedGather = 2,   // host gather into the pinned slot, then one copy
};

// Runs of a chunk that share one length and one source distance between
// consecutive starts: count rows of len bytes, the first at chunk offset
// off, every stride bytes, landing back to back at packed offset poff --
// what one 2-D host-to-device copy moves (a single run has count 1).
struct DmaGroup {
    uint32_t off;
    uint32_t poff;
    uint32_t len;
    uint32_t count;
    uint32_t stride;
};

// A destination range [b, e) of tensor i (the destination checks).
struct DstRange {
    uint64_t b, e;
    size_t i;
};

// Largest payload for which the image kernel runs its variant with more loads
// in flight whatever the table: where the two measured the same. Small loads
// are bounded by latency (the least of them lie in the 256 MiB memory-side
// cache, image and destinations), large ones by the rate of the stream, which
// more loads in flight hold up. Back-to-back loads, dense against mixed:
// transformer tables of 37 MB 11.3 and 10.2 us, 73 MB 19.8 and 18.8, 168 MB
// 40.8 and 40.1, 293 MB 89.8 and 87.0, 335 MB 105.7 and 108.1, 566 MB 175 and
// 184; one rank of four of 252 MB 79.7 and 73.4, 311 MB 94.8 and 92.0, 370 MB
// 117.4 and 118.9. Below 20 MB a load takes the host longer than the device.
constexpr uint64_t kMixedBytes = 300ull << 20;

// Largest payload of a dense table whose pinned blob is read over the link
// (reads_over_link, runtime.hip, says why the line lies here).
constexpr uint64_t kLinkBytes = 64ull << 20;

// Static device workspace of ii_load_device_noalloc (runtime.hip): the
// kernel's tables, and after them what the segments' rows are formed from
// (28 bytes for each 32-byte row).
constexpr uint64_t kScratchBytes = 64ull << 20;
constexpr uint64_t kStageBytes = kScratchBytes / 32 * 28;

struct Runtime;  // device-side state (runtime.hip)

void set_error(const char* fmt, ...);
int fail(int code, const char* fmt, ...);

}  // namespace ii

struct ii_plan_s {
    // table as given
    std::vector<std::string> names;
    std::vector<int32_t> dtype;
    std::vector<int32_t> ndim;
    std::vector<int64_t> shape_flat;
    std::vector<uint64_t> shape_start;
    std::vector<uint64_t> src_offset;
    std::vector<uint64_t> dst_align;
    std::vector<uint64_t> row_stride;  // 0 for contiguous tensors
    // derived
    std::vector<uint64_t> nbytes;
    std::vector<uint64_t> rows;        // 1 for contiguous tensors, 0 for empty ones
    std::vector<uint64_t> dst_offset;
    uint64_t payload = 0, arena_bytes = 0, max_align = 1;
    uint64_t lo = 0, hi = 0;
    uint64_t copy_bytes = 0;  // host-to-device bytes of a load from a pinned blob
    // of those, the payload of chunks moved row by row: by 2-D copies or
    // gathered on the host
    uint64_t row_bytes = 0;
    uint64_t chunk_bytes = 0;
    size_t num_chunks = 0;
    std::vector<uint64_t> chunk_seg_begin;  // num_chunks + 1
    // segments in chunk order, then by offset inside the chunk
    std::vector<uint32_t> seg_chunk, seg_off, seg_tensor, seg_len;
    std::vector<uint64_t> seg_toff;
    // Packed staging: when the host stage copies a chunk anyway (pageable
    // blob, file), it gathers only the segments' bytes, back to back in
    // segment order, so the link carries payload only. Segment s then sits
    // at seg_poff[s] of its slot; chunk k's slot holds chunk_plen[k] bytes.
    // A run is a maximal group of consecutive segments that are also
    // adjacent in the chunk (one memcpy): chunk offset run_off, slot offset
    // run_poff, run_len.
    bool packed_distinct = false;  // false: packed layout == chunk layout for every chunk
    // per chunk: how a load from a pinned blob moves it (PinnedMove) --
    // by copies of its run groups when it has at most kMaxDmaGroups of them,
    // else gathered on the host when more than a quarter of its used range
    // is gaps, else its used range in place
    std::vector<uint8_t> chunk_pinned;
    // per chunk: whether its groups' rows are whole 4-byte words. The copy
    // engine moves other rows one by one (218 MB in rows of 1659 and 3473
    // bytes: 219 ms, 4.1 gathered on the host), so those are gathered.
    std::vector<uint8_t> chunk_words;
    std::vector<uint64_t> chunk_group_begin;  // num_chunks + 1 (plans with gaps)
    std::vector<ii::DmaGroup> groups;
    std::vector<uint32_t> seg_poff;
    std::vector<uint64_t> chunk_plen;
    std::vector<uint64_t> chunk_run_begin;  // num_chunks + 1
    std::vector<uint32_t> run_off, run_poff, run_len;
    // ring tiles (see TileDev), chunk by chunk: what the scatter of one
    // staged or in-place chunk runs over. Only their number is kept: which
    // segments meet a tile, and its window, follow from the segments
    // (ring_tiles, ring_window)
    uint32_t tile_bytes = ii::kDefaultTile;
    std::vector<uint64_t> chunk_tile_begin;  // num_chunks + 1
    // layout tiles (the resident-image kernel): the segments in destination
    // layout order -- lseg[j] is the j-th segment by layout position
    // dst_offset[tensor] + tensor offset -- and tiles of tile_bytes of
    // layout positions: tile g takes the window of layout positions
    // [w * tile_bytes, (w + 1) * tile_bytes) with w = lwin[g] (w = g when
    // lwin is empty: every window holds segment bytes) and the layout-order
    // segments [ltiles[g].first, ltiles[g].last) that meet it
    std::vector<uint32_t> lseg;
    // what the device forms the kernel's rows from, in the order it is
    // uploaded in, so that one copy takes all: a destination per segment
    // (written by ii_load_device_noalloc, which allocates nothing, and by
    // loads whose destinations go as kernel arguments), a LayoutRow and a
    // length
    std::vector<uint64_t> lstage;
    uint64_t* ldst() { return lstage.data(); }
    const uint64_t* ldst() const { return lstage.data(); }
    const ii::LayoutRow* lrows() const {
        return reinterpret_cast<const ii::LayoutRow*>(lstage.data() + lseg.size());
    }
    const uint32_t* llen() const {
        return reinterpret_cast<const uint32_t*>(lstage.data() + 3 * lseg.size());
    }
    uint64_t nltiles = 0;
    // bytes of the 128-byte source lines a kernel reads that walks the
    // layout: lines that neighbouring segments share count once
    uint64_t line_bytes = 0;
    // kept only for layouts with padding-only windows; otherwise tile g is
    // window g, and the ranges follow from the segments (row_tiles)
    std::vector<ii::TileDev> ltiles;
    std::vector<uint32_t> lwin;
    // whether the image kernel runs its variant for tables of many small
    // tensors (more loads in flight; see the planner's rule)
    bool layout_mixed = false;
    // whether an image load runs it for its size (see kMixedBytes)
    bool layout_small = false;
    // whether an untraced load reads a pinned blob over the link
    bool pinned_link = false;
    // for the destination checks: the first non-empty tensor (n if none),
    // whether there are empty ones, the end of the last non-empty tensor in
    // the layout and the largest alignment of a non-empty one
    size_t first_live = 0;
    bool has_empty = false;
    uint64_t layout_end = 0, live_align = 1;
    // the destination ranges ii_load_device_noalloc's checks sort, sized when
    // the plan is made so that the call itself allocates nothing
    std::vector<ii::DstRange> na_ranges;
    // runtime configuration
    uint32_t ring_depth = 3;
    uint32_t host_threads = 8;
    uint32_t copy_streams = 2;
    bool trace = false;
    // device state, created by the first load
    ii::Runtime* rt = nullptr;
    std::atomic<int> busy{0};

    uint64_t chunk_len(size_t k) const {
        return k + 1 < num_chunks ? chunk_bytes : (hi - lo) - chunk_bytes * (num_chunks - 1);
    }
    // The bytes of chunk k a load moves: from its first segment's start to
    // its last segment's end, rounded out to kCopyAlign inside the chunk;
    // empty if the chunk holds no segment (a gap between the tensors of a
    // sharded table).
    void chunk_used(size_t k, uint64_t* b, uint64_t* e) const {
        const uint64_t s0 = chunk_seg_begin[k], s1 = chunk_seg_begin[k + 1];
        if (s0 == s1) {
            *b = *e = 0;
            return;
        }
        const uint64_t a = ii::kCopyAlign;
        const uint64_t end = (uint64_t)seg_off[s1 - 1] + seg_len[s1 - 1];
        *b = seg_off[s0] & ~(a - 1);
        *e = std::min<uint64_t>(chunk_len(k), (end + a - 1) & ~(a - 1));
    }
};

namespace ii {
void runtime_destroy(ii_plan_t* p);
}
