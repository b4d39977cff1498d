// The launches of scatter.hip, as the runtime calls them.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

#include "scatter_types.h"

namespace ii {

// The tables of one resident-image launch, in device memory.
struct LayoutTable {
    const TileDev* tiles;
    const uint32_t* win;  // null: tile g is window g
    uint64_t ntiles;
    const LayoutSeg* rows;
    uint64_t nrows;
};

enum class ImageKernel { kDense, kMixed, kLink };

hipError_t launch_scatter_slot(const uint8_t* slot, const TileDev* tiles, const TileWin* wins,
                               uint32_t ntiles, const SegDev* segs, uint64_t base, bool implicit,
                               uint32_t tile_bytes, uint64_t plen, hipStream_t stream);
hipError_t launch_scatter_layout(const uint8_t* span, const LayoutTable& table, uint64_t base,
                                 uint32_t tile_bytes, ImageKernel which, hipStream_t stream);
// Form the ring's tiles and, unless wins is null, their windows of chunk
// offsets, from n segments.
hipError_t launch_ring_tables(const RingSeg* segs, uint32_t n, uint32_t tile_bytes, TileDev* tiles,
                              TileWin* wins, uint64_t ntiles, hipStream_t stream);

// Form the layout rows of n segments (dst null: rows of the plan's layout)
// and, unless tiles is null, the layout tiles' segment ranges.
hipError_t launch_layout_tables(const LayoutRow* from, const uint32_t* len, const uint64_t* dst,
                                uint32_t n, uint32_t tile_bytes, LayoutSeg* rows, TileDev* tiles,
                                uint64_t ntiles, hipStream_t stream);

// The same for n segments from s0 on, what the rows are formed from in the
// kernel's arguments: n destinations if has_dst, n LayoutRows, n lengths.
// before: where segment s0 - 1 ends (0: none); after: where segment s0 + n
// starts (all ones: none). tiles: of the whole layout, rows likewise.
struct LayoutArgs {
    uint64_t words[448];  // 3.5 KiB: 179 segments, 128 with destinations
};
constexpr uint32_t kByValueLaunches = 4;
hipError_t launch_layout_tables_by_value(const LayoutArgs& args, bool has_dst, uint32_t n,
                                         uint32_t s0, uint64_t before, uint64_t after,
                                         uint32_t tile_bytes, LayoutSeg* rows, TileDev* tiles,
                                         hipStream_t stream);
hipError_t launch_zero(const RangeDev* ranges, uint32_t n, hipStream_t stream);

}  // namespace ii
