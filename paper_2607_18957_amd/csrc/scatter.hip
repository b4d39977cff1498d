// Chunk -> tensor scatter for gfx950 (CDNA4), and the zero-fill used by the
// arena switch.
//
// The scatter is the device half of the refined tensor materialisation in
// InstantInfer (arXiv 2607.18957, Sec. 4.2): once a chunk is resident in
// device memory, every tensor piece it holds is copied into the tensor's own
// buffer ((C_i,InGPU)->(T_j,Alloc) moves T_j to Loaded). It is pure data
// movement, bound by HBM bandwidth: per payload byte one read of the chunk
// and one write of the tensor.
//
// Work split. One 128-thread workgroup (two wavefronts) owns one tile of
// tile_bytes (4 KiB by default), two 16-byte units per lane. Measured on a
// Llama-8B-shaped set against 256 threads x 8 KiB, 64 x 2 KiB, 8 and 16 KiB
// tiles, four or eight units per lane and persistent grids of 8 or 16
// workgroups per CU: two units per lane in small workgroups, one tile each,
// is fastest. Per tile a table holds the range of segment rows whose bytes
// meet it (layout_tables, ring_tables), so a workgroup reads only its own
// rows.
//   Ring (scatter_slot): a staged chunk's segment bytes are cut in segment
// order, gaps between segments skipped, so no workgroup exists for bytes no
// tensor needs (the gaps a sharded table leaves in the file). In a packed
// staging slot, and in a chunk without gaps, a tile's window is simply its
// share of the slot or chunk.
//   Resident image (scatter_layout): the tiles are windows of the plan's
// destination layout instead, the segments of all chunks in layout order.
// Each workgroup then writes one aligned 4 KiB block of destination memory
// (less any padding) and reads wherever its bytes lie. Writes that start or
// end inside a 128-byte line cost HBM bandwidth (a plain copy into a
// destination 48 bytes off a line runs 7% slower than an aligned one) while
// misaligned reads cost nothing measurable, so cutting by destination wins
// wherever source and destination offsets are not congruent modulo the
// tile (the 100,000-tensor set: 5.43 against 5.09 TB/s) and ties where
// they are (the Llama sets). An image in pinned host memory is read over the
// link by few workgroups that walk the same tiles (scatter_layout_link).
//
// Units. Destination memory is written in 16-byte blocks aligned to 16
// bytes, so every store of a block that a segment covers completely is one
// dwordx4 store. A unit is one (segment, destination block) pair. A unit
// belongs to the tile whose window holds its anchor: the coordinate of the
// first destination byte it covers -- its source offset in the chunk for
// the ring, its layout position for the resident image. Within a segment
// both coordinates grow with the destination address, so every unit has
// exactly one owner even when the source and destination phases (address
// mod 16) differ, and the units a tile owns are contiguous within each
// segment.
//
// Lanes to units. The workgroup stages its segment rows in LDS, counts each
// segment's units in the tile, and forms an exclusive prefix sum. Lane u of
// the tile's unit range then finds its segment by binary search over the
// prefix sums in LDS. Consecutive lanes get consecutive units, so a large
// segment is copied with fully coalesced 16-byte accesses, and many
// segments smaller than a wavefront (64 lanes x 16 B = 1 KiB) are served by
// one wavefront in the same pass. (The resident-image kernel's variant for
// tables of many small tensors skips this staging for tiles that one
// segment meets: every lane forms that one row itself.)
//
// Phase shift. The 16 source bytes of a destination block start at any
// address a. The lane loads the aligned 16-byte words at a & ~15 and
// (a & ~15) + 16 -- each only if it holds a byte the unit needs, so no load
// touches a 16-byte word outside the source data -- and assembles the block
// with funnel shifts (v_alignbit_b32). Blocks a segment covers only partly
// (its first and last block, or a segment shorter than 16 bytes) are
// written with 8/4/2/1-byte stores of exactly the covered bytes: padding and
// neighbouring tensors are never read-modify-written.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "scatter_launch.h"
#include "scatter_math.h"
#include "scatter_types.h"

namespace ii {

static_assert((uint64_t)kMaxGridBlocks * kBlock <= 0xffffffffull,
              "one launch must stay within 2^32 - 1 work-items");
// scatter_slot launches the tiles of one chunk: at most 2^32 / 1024
static_assert((1ull << 32) / 1024 <= kMaxGridBlocks, "a chunk's tiles fit one launch");

namespace {

constexpr uint32_t kLinkRun = 4;  // consecutive tiles a link workgroup takes at a time

// Global-address-space accesses: plain pointers made from integer addresses
// would be generic (flat) accesses, which also count against the LDS wait
// counter.
#define II_GLOBAL __attribute__((address_space(1)))
typedef uint32_t v4u32 __attribute__((ext_vector_type(4)));
typedef II_GLOBAL v4u32 g_v4;
typedef II_GLOBAL uint64_t g_u64;
typedef II_GLOBAL uint32_t g_u32;
typedef II_GLOBAL uint16_t g_u16;
typedef II_GLOBAL uint8_t g_u8;

struct DevMem {
    __device__ __forceinline__ U4 ld16(uint64_t a) const {
        const v4u32 x = *reinterpret_cast<const g_v4*>(a);
        return U4{x.x, x.y, x.z, x.w};
    }
    // Whole destination blocks are streamed out with non-temporal stores: the
    // kernel never reads them back, and keeping them out of the caches leaves
    // room for the source stream (measured ~3% faster on large tables).
    __device__ __forceinline__ void st16(uint64_t a, U4 v) {
        v4u32 x = {v.x, v.y, v.z, v.w};
        __builtin_nontemporal_store(x, reinterpret_cast<g_v4*>(a));
    }
    __device__ __forceinline__ void st8(uint64_t a, uint32_t lo, uint32_t hi) {
        *reinterpret_cast<g_u64*>(a) = ((uint64_t)hi << 32) | lo;
    }
    __device__ __forceinline__ void st4(uint64_t a, uint32_t v) { *reinterpret_cast<g_u32*>(a) = v; }
    __device__ __forceinline__ void st2(uint64_t a, uint16_t v) { *reinterpret_cast<g_u16*>(a) = v; }
    __device__ __forceinline__ void st1(uint64_t a, uint8_t v) { *reinterpret_cast<g_u8*>(a) = v; }
};

// Inclusive prefix sum across the 64 lanes of a wavefront.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    return v;
}

}  // namespace

// Lane units base + j * kBlock + threadIdx.x (j < kUnroll) below total,
// row_at(u) giving the row of unit u; all stores follow all loads. Two issue
// orders:
//   kOverlap = false: each unit's phase shift follows its own loads, so the
//     wait for unit j's words comes before unit j + 1's loads issue -- at
//     most one unit's loads in flight per lane;
//   kOverlap = true: every unit's loads issue before any loaded word is
//     used, and all shifts precede the first store (a wait for loads issued
//     before a store would also wait for that store; the empty asm pins each
//     shifted block there, or the compiler sinks a unit's shift into its
//     store branch, after the previous unit's store).
// Measured: on tables of large tensors, where a tile is one unbroken 4 KiB
// stream, the first is faster (83.4% against 77.2% of HBM peak on a
// Llama-8B-shaped set); more loads in flight only lengthen the queues. On
// the 100,000-tensor set, a tenth of whose tiles meet three segments or more
// and spend longer forming rows, the second is for those (all tiles one unit
// at a time 326.0 us, only tiles of one segment 322.0).
template <bool kOverlap, class RowAt>
__device__ __forceinline__ void move_units(DevMem& mem, uint32_t base, uint32_t total,
                                           RowAt row_at) {
    UnitIO io[kUnroll];
    U4 v[kUnroll];
    if (kOverlap) {
        U4 x0[kUnroll], x1[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            const uint32_t u = base + (uint32_t)j * kBlock + threadIdx.x;
            io[j].c0 = io[j].c1 = io[j].p = 0;  // every unit is shifted below
            x0[j] = x1[j] = U4{0, 0, 0, 0};
            if (u < total) {
                io[j] = unit_io(row_at(u), u);
                if (io[j].need0) x0[j] = mem.ld16(io[j].A);
                if (io[j].need1) x1[j] = mem.ld16(io[j].A + 16);
            }
        }
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            v[j] = funnel16(x0[j], x1[j], io[j].p);
            asm volatile("" : "+v"(v[j].x), "+v"(v[j].y), "+v"(v[j].z), "+v"(v[j].w));
        }
    } else {
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            const uint32_t u = base + (uint32_t)j * kBlock + threadIdx.x;
            io[j].c0 = io[j].c1 = 0;
            if (u < total) {
                io[j] = unit_io(row_at(u), u);
                U4 x0{0, 0, 0, 0}, x1{0, 0, 0, 0};
                if (io[j].need0) x0 = mem.ld16(io[j].A);
                if (io[j].need1) x1 = mem.ld16(io[j].A + 16);
                v[j] = funnel16(x0, x1, io[j].p);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kUnroll; ++j)
        if (io[j].c1 > io[j].c0) store_unit(mem, io[j].d, v[j], io[j].c0, io[j].c1);
}

// One workgroup's share of the scatter: the units anchored in its window,
// among segment rows [s_first, s_last). row(s, &cnt) returns the row of
// segment s seen from the window and its count of units anchored there.
// Every tile holds segment bytes, so s_first < s_last (the planner
// guarantees it); the batch loop runs at least once with no guard, which
// lets the argument loads issue together with the tile's own.
template <bool kOverlap, class RowOf>
__device__ __forceinline__ void scatter_tile(uint32_t s_first, uint32_t s_last, RowOf row) {
    __shared__ SegRow rows[kMaxSegBatch];
    __shared__ uint32_t pre[kMaxSegBatch];
    __shared__ uint32_t wsum[kBlock / 64];

    const uint32_t tid = threadIdx.x;
    DevMem mem;

    uint32_t s0 = s_first;
    do {
        const uint32_t ns = min((uint32_t)kMaxSegBatch, s_last - s0);
        uint32_t cnt = 0;
        if (tid < ns) rows[tid] = row(s0 + tid, &cnt);
        const uint32_t inc = wave_scan(cnt);
        if ((tid & 63u) == 63u) wsum[tid >> 6] = inc;
        __syncthreads();
        uint32_t before_wave = 0, total = 0;
#pragma unroll
        for (uint32_t w = 0; w < kBlock / 64; ++w) {
            const uint32_t x = wsum[w];
            before_wave += (w < (tid >> 6)) ? x : 0u;
            total += x;
        }
        if (tid < ns) {
            const uint32_t ex = before_wave + inc - cnt;
            pre[tid] = ex;
            rows[tid].ubase -= ex;
        }
        __syncthreads();

        for (uint32_t base = 0; base < total; base += kBlock * kUnroll)
            move_units<kOverlap>(mem, base, total,
                                 [&](uint32_t u) { return rows[find_row(pre, ns, u)]; });
        __syncthreads();  // rows/pre are rewritten by the next batch
        s0 += kMaxSegBatch;
    } while (s0 < s_last);
}

// Ring path: one chunk, staged in a device slot that starts at `slot`; one
// workgroup per tile of the chunk (`tiles` points at the chunk's first).
// A segment goes to base + its row's dst (rows of the plan's own layout and
// the arena's address, or resolved addresses and 0).
// implicit: tile m takes slot offsets [m * tile_bytes, ...) up to plen -- a
// packed slot, or a chunk without gaps at its own offsets; otherwise the
// slot holds a chunk with gaps at its own offsets and the tile's window of
// chunk offsets (`wins`, the chunk's first) applies.
__global__ __launch_bounds__(kBlock) void scatter_slot(
    const uint8_t* __restrict__ slot, const TileDev* __restrict__ tiles,
    const TileWin* __restrict__ wins, const SegDev* __restrict__ segs, uint64_t base,
    uint32_t implicit, uint32_t tile_bytes, uint64_t plen) {
    const uint32_t g = blockIdx.x;
    const TileDev td = tiles[g];
    uint64_t w0, w1;
    if (implicit) {
        w0 = (uint64_t)g * tile_bytes;
        w1 = min(plen, w0 + tile_bytes);
    } else {
        const TileWin tw = wins[g];
        w0 = tw.w0;
        w1 = tw.w1;
    }
    const uint64_t cbase = reinterpret_cast<uint64_t>(slot);
    scatter_tile<false>(td.first, td.last, [&](uint32_t s, uint32_t* cnt) {
        const SegDev sd = segs[s];
        return make_row(base + sd.dst, sd.off, sd.len, cbase, w0, w1, cnt);
    });
}

// A tile that one segment meets, without LDS or barriers: every lane forms
// the row itself (its prefix is 0, so unit u is unit u of the row) -- the
// arithmetic of scatter_tile with a single row. One unit's loads at a time:
// such a tile is one unbroken stream, and issuing both units' loads first
// lengthens the queues as it does in a table of large tensors (100,000
// tensors 327.9 -> 322.0 us, 40,000 130.7 -> 128.9; tables of large tensors
// of 37 to 168 MB level). Tiles of several segments spend longer forming
// rows and keep all their loads in flight (one at a time: 326 us).
__device__ __forceinline__ void scatter_one_row(const SegRow& row, uint32_t total) {
    DevMem mem;
    for (uint32_t base = 0; base < total; base += kBlock * kUnroll)
        move_units<false>(mem, base, total, [&](uint32_t) { return row; });
}

// Resident-image path: the whole table in one dispatch (a grid of gy rows of
// gx workgroups, see grid_shape; tile g = y * gx + x, none past ntiles).
// `span` is the device address of the blob's span byte lo; segment rows are
// in layout order. Tile g takes the layout window w = win[g] (w = g when win
// is null: no window of the layout is all padding).
//   A segment goes to base + its row's dst. Tensors that fill the plan's
// layout in one arena take rows whose dst is their layout position, uploaded
// once, and the arena's address: a table of 40,000 tensors loaded into two
// arenas in turn spent 384 us a call forming and uploading rows with
// resolved addresses, for a kernel of 130 us; it now takes 132 us.
//   kMixed, chosen per plan (the planner's rule: enough tiles meet three or
// more segments, or the load fits the memory-side cache): tiles that one
// segment meets skip the LDS staging and its barriers (scatter_one_row), and
// the others issue all their loads before using any (move_units). Both put
// loads in flight sooner, which pays where tiles spend long forming rows and
// costs on large tables of large tensors (measured, dense and mixed:
// 100,000-tensor set 330.1 and 322.0 us; a Llama-8B set 83.4% and 77.2% of
// HBM peak; its rank-1-of-4 shard, whose tiles meet at most two segments,
// 80.0% and 76.2%).
template <bool kMixed>
__global__ __launch_bounds__(kBlock) void scatter_layout(
    const uint8_t* __restrict__ span, const TileDev* __restrict__ tiles,
    const uint32_t* __restrict__ win, const LayoutSeg* __restrict__ segs, uint64_t base,
    uint32_t tile_bytes, uint32_t ntiles) {
    const uint32_t g = blockIdx.y * gridDim.x + blockIdx.x;
    if (g >= ntiles) return;
    const TileDev td = tiles[g];
    const uint64_t w0 = (uint64_t)(win ? win[g] : g) * tile_bytes;
    const uint64_t w1 = w0 + tile_bytes;
    const uint64_t sb = reinterpret_cast<uint64_t>(span);
    // source address of layout position x is sb + ls.src + (x - ls.pos)
    auto row_of = [&](uint32_t s, uint32_t* cnt) {
        const LayoutSeg ls = segs[s];
        return make_row(base + ls.dst, ls.pos, ls.len, sb + ls.src - ls.pos, w0, w1, cnt);
    };
    if (kMixed && td.last - td.first == 1) {
        uint32_t total;
        const SegRow row = row_of(td.first, &total);
        scatter_one_row(row, total);
        return;
    }
    scatter_tile<kMixed>(td.first, td.last, row_of);
}

// The same table read over the host link: `span` is pinned host memory. What
// bounds it is the link (57.3 GB/s for a 1 GiB copy-engine copy), and how
// many reads are in flight decides how close it gets. With one workgroup per
// tile the whole chip's worth of reads queues at the link at once, in an
// order that spreads over 33 MB of the blob: a launch then costs ~55 us on
// top of its bytes (16.8 MB in 354 us, 3.0 GB at 55.6 GB/s). 256 workgroups
// (one per compute unit, two wavefronts each) that walk the tiles front to
// back keep ~1 MB in flight and read a compact moving window: 16.8 MB in 302
// us, 3.0 GB at 57.5 GB/s. Swept from 32 to 512 workgroups: 192 and more are
// level, 64 nearly, 96 to 144 lose 4-7%, 32 loses 20%.
//   Other kernels run slower meanwhile, for as long as the load takes: beside
// 256 workgroups bf16 products of 4096 x 4096 matrices took 1.9 to 5 times
// as long, beside 64 of them 1.5 to 1.6 times. So large tables go with 64
// (link_blocks): a 749 MB shard 13.05 -> 13.08 ms alone and 13.6 -> 13.4 beside
// those products, 948 MB of permuted tensors 16.95 -> 17.04 ms.
//   Each workgroup takes kLinkRun consecutive tiles at a time: where source
// and destination are not congruent, neighbouring tiles share a 128-byte
// source line, and the one L2 that both now go through fetches it over the
// link once (100,000 tensors in a permuted file: 54.8 GB/s with runs of 1,
// 55.5 with 2, 56.0 with 4, 56.1 with 8; a run of 4 leaves small tables
// spread over more workgroups).
//   All of a tile's loads are issued before any is used: a link read takes
// microseconds, and waits between units would double them.
__global__ __launch_bounds__(kBlock) void scatter_layout_link(
    const uint8_t* __restrict__ span, const TileDev* __restrict__ tiles,
    const uint32_t* __restrict__ win, const LayoutSeg* __restrict__ segs, uint64_t base,
    uint32_t tile_bytes, uint32_t ntiles) {
    const uint64_t sb = reinterpret_cast<uint64_t>(span);
    // ntiles < 2^31 and a step is at most 256 * kLinkRun: no wrap
    for (uint32_t g0 = blockIdx.x * kLinkRun; g0 < ntiles; g0 += gridDim.x * kLinkRun) {
        const uint32_t g1 = min(ntiles, g0 + kLinkRun);
        for (uint32_t g = g0; g < g1; ++g) {
            const TileDev td = tiles[g];
            const uint64_t w0 = (uint64_t)(win ? win[g] : g) * tile_bytes;
            const uint64_t w1 = w0 + tile_bytes;
            scatter_tile<true>(td.first, td.last, [&](uint32_t s, uint32_t* cnt) {
                const LayoutSeg ls = segs[s];
                return make_row(base + ls.dst, ls.pos, ls.len, sb + ls.src - ls.pos, w0, w1, cnt);
            });
        }
    }
}

// The image kernel's tables from what the host knows of each segment (20
// bytes, 28 with a destination of its own): its 32-byte row, and its share
// of the tiles' segment ranges, 8 bytes per 4 KiB of the layout.
//   What it replaces is the host: building the ranges there and uploading
// them was 31 MB for a Llama-8B-shaped table and most of a first load, and
// ii_load_device_noalloc uploaded them on every call.
//   kWave: one wavefront per segment fills its ranges, shared between
// gridDim.y of them; without, one thread per segment, and only segments of
// more than kFewTiles tiles are filled by their whole wavefront. A segment
// of a few tiles keeps one lane of a wavefront busy, one of many needs them
// all: 5,000 segments of 12 tiles on average take 4.6 us with a
// wavefront each and 11 us with a thread each; 150,000 of 0.7 tiles take 5.8
// us with a thread each.
constexpr uint32_t kTableBlock = 256;
constexpr uint64_t kFewTiles = 8;

// put(t, j, m) for each tile m of segment j's range t, by whichever lanes:
// every lane of a wavefront calls this with its own segment (kWave: all with
// the same).
template <bool kWave, class Put>
__device__ __forceinline__ void fill_tiles(const RowTiles& t, bool valid, uint32_t j, Put put) {
    const uint32_t lane = threadIdx.x & 63u;
    auto fill = [&](const RowTiles& rt, uint32_t s) {
        for (uint64_t m = rt.m0 + blockIdx.y * 64u + lane; m <= rt.m1; m += gridDim.y * 64u)
            put(rt, s, m);
    };
    if (kWave) {
        if (valid) fill(t, j);
        return;
    }
    const bool wide = valid && t.m1 - t.m0 >= kFewTiles;
    if (valid && !wide && blockIdx.y == 0)
        for (uint64_t m = t.m0; m <= t.m1; ++m) put(t, j, m);
    for (uint64_t todo = __ballot(wide); todo; todo &= todo - 1) {
        const int src = __ffsll((unsigned long long)todo) - 1;
        RowTiles w;
        w.m0 = __shfl(t.m0, src, 64);
        w.m1 = __shfl(t.m1, src, 64);
        w.first0 = __shfl((int)t.first0, src, 64) != 0;
        w.last1 = __shfl((int)t.last1, src, 64) != 0;
        fill(w, j - lane + (uint32_t)src);
    }
}

// The segment of a lane of the tables kernels.
template <bool kWave>
__device__ __forceinline__ uint32_t table_segment() {
    return kWave ? blockIdx.x * (kTableBlock / 64) + (threadIdx.x >> 6)
                 : blockIdx.x * kTableBlock + threadIdx.x;
}

// from, len and dst hold segments s0 .. s0 + n - 1 of the layout; `before`:
// where the segment before them ends (0: none), `after`: where the one
// behind them starts (all ones: none).
template <bool kWave>
__device__ __forceinline__ void form_tables(const LayoutRow* __restrict__ from,
                                            const uint32_t* __restrict__ len,
                                            const uint64_t* __restrict__ dst, uint32_t n,
                                            uint32_t s0, uint64_t before, uint64_t after,
                                            uint32_t tile_bytes, uint32_t shift,
                                            LayoutSeg* __restrict__ rows,
                                            TileDev* __restrict__ tiles) {
    const uint32_t j = table_segment<kWave>();
    RowTiles t{1, 0, false, false};  // no tiles
    rows += s0;
    if (j < n) {
        const LayoutRow r = from[j];
        const uint32_t l = len[j];
        const uint64_t prev_end = j ? from[j - 1].pos + len[j - 1] : before;
        const uint64_t next_pos = j + 1 < n ? from[j + 1].pos : after;
        t = row_tiles(r.pos, l, prev_end, next_pos, tile_bytes, shift);
        if (blockIdx.y == 0 && (!kWave || (threadIdx.x & 63u) == 0))
            rows[j] = LayoutSeg{r.src, dst ? dst[j] : r.pos, r.pos, l, 0};
    }
    if (!tiles) return;
    fill_tiles<kWave>(t, j < n, s0 + j, [&](const RowTiles& rt, uint32_t s, uint64_t m) {
        if (m > rt.m0 || rt.first0) tiles[m].first = s;
        if (m < rt.m1 || rt.last1) tiles[m].last = s + 1;
    });
}

template <bool kWave>
__global__ __launch_bounds__(kTableBlock) void layout_tables(
    const LayoutRow* __restrict__ from, const uint32_t* __restrict__ len,
    const uint64_t* __restrict__ dst, uint32_t n, uint32_t tile_bytes, uint32_t shift,
    LayoutSeg* __restrict__ rows, TileDev* __restrict__ tiles) {
    form_tables<kWave>(from, len, dst, n, 0, 0, ~0ull, tile_bytes, shift, rows, tiles);
}

// The ring's tables the same way: a tile's segments, and for plans with gaps
// its window of chunk offsets, which the segment it starts in knows, as it
// knows the end of the window before. (Listed on the host and uploaded they
// were 8 or 16 bytes per 4 KiB of the model: most of ii_plan, 17 ms for a
// Llama-8B-shaped table, and 31 MB of the ring's set-up.)
template <bool kWave>
__global__ __launch_bounds__(kTableBlock) void ring_tables(const RingSeg* __restrict__ segs,
                                                           uint32_t n, uint32_t tile_bytes,
                                                           uint32_t shift,
                                                           TileDev* __restrict__ tiles,
                                                           TileWin* __restrict__ wins) {
    const uint32_t j = table_segment<kWave>();
    RowTiles t{1, 0, false, false};  // no tiles
    if (j < n) {
        const RingSeg r = segs[j];
        const bool ends = j + 1 == n || segs[j + 1].tile0 != r.tile0;
        t = ring_tiles(r.poff, r.len, ends, tile_bytes, shift);
        if (wins && ends) wins[r.tile0 + t.m1].w1 = r.off + r.len;
    }
    fill_tiles<kWave>(t, j < n, j, [&](const RowTiles& rt, uint32_t s, uint64_t m) {
        const RingSeg r = segs[s];
        const uint64_t g = r.tile0 + m;
        if (m < rt.m1 || rt.last1) tiles[g].last = s + 1;
        if (!(m > rt.m0 || rt.first0)) return;
        tiles[g].first = s;
        if (!wins) return;
        const uint32_t w = ring_window(r.off, r.poff, m, tile_bytes);
        wins[g].w0 = w;
        if (m) wins[g - 1].w1 = w;
    });
}

// The layout tables with what the rows are formed from passed by value, in
// the order destinations (if any), rows, lengths: a small table needs no
// upload. A copy from pageable memory of more than 16 KiB crosses to a copy
// engine and back, ~25 us between two kernels, and a smaller one takes the
// host 2.7 us for 512 bytes and 8.8 us for 16 KiB; a launch with 3.5 KiB of
// arguments takes the host 3.3 us, so up to kByValueLaunches of them go, one
// behind the other, each with its share of the segments.
__global__ __launch_bounds__(kTableBlock) void layout_tables_by_value(
    LayoutArgs, uint32_t has_dst, uint32_t n, uint32_t s0, uint64_t before, uint64_t after,
    uint32_t tile_bytes, uint32_t shift, LayoutSeg* __restrict__ rows,
    TileDev* __restrict__ tiles) {
    // the first argument where it lies, at the start of the kernel's argument
    // segment: indexed as a variable it would be copied to scratch, 3.5 KiB a
    // lane (253 us)
    const uint64_t* const words = (const uint64_t*)__builtin_amdgcn_kernarg_segment_ptr();
    const uint64_t* const w = words + (has_dst ? n : 0);
    form_tables<true>(reinterpret_cast<const LayoutRow*>(w),
                      reinterpret_cast<const uint32_t*>(w + 2 * n),
                      has_dst ? words : nullptr, n, s0, before, after, tile_bytes, shift, rows,
                      tiles);
}

// Zero the byte ranges [r.begin, r.end) (device addresses). One workgroup per
// range; 16-byte stores for whole aligned blocks, exact narrow stores at the
// edges.
__global__ __launch_bounds__(kBlock) void zero_ranges(const RangeDev* __restrict__ ranges,
                                                       uint32_t n) {
    if (blockIdx.x >= n) return;
    const RangeDev r = ranges[blockIdx.x];
    if (r.end <= r.begin) return;
    DevMem mem;
    const uint64_t b0 = r.begin >> 4, b1 = (r.end - 1) >> 4;
    const U4 z{0, 0, 0, 0};
    for (uint64_t b = b0 + threadIdx.x; b <= b1; b += kBlock) {
        const uint64_t d = b << 4;
        const uint64_t ds = d > r.begin ? d : r.begin;
        const uint64_t de = (d + 16) < r.end ? d + 16 : r.end;
        store_unit(mem, d, z, (uint32_t)(ds - d), (uint32_t)(de - d));
    }
}

hipError_t launch_scatter_slot(const uint8_t* slot, const TileDev* tiles, const TileWin* wins,
                               uint32_t ntiles, const SegDev* segs, uint64_t base, bool implicit,
                               uint32_t tile_bytes, uint64_t plen, hipStream_t stream) {
    if (ntiles == 0) return hipSuccess;
    if (!implicit && !wins) return hipErrorInvalidValue;
    hipLaunchKernelGGL(scatter_slot, dim3(ntiles), dim3(kBlock), 0, stream, slot, tiles, wins,
                       segs, base, implicit ? 1u : 0u, tile_bytes, plen);
    return hipGetLastError();
}

hipError_t launch_scatter_layout(const uint8_t* span, const LayoutTable& t, uint64_t base,
                                 uint32_t tile_bytes, ImageKernel which, hipStream_t stream) {
    if (t.ntiles == 0) return hipSuccess;
    if (t.ntiles > 0x7fffffffull) return hipErrorInvalidConfiguration;
    const uint32_t n = (uint32_t)t.ntiles;
    uint32_t gx, gy;
    grid_shape(n, &gx, &gy);
    switch (which) {
    case ImageKernel::kDense:
        hipLaunchKernelGGL(scatter_layout<false>, dim3(gx, gy), dim3(kBlock), 0, stream, span,
                           t.tiles, t.win, t.rows, base, tile_bytes, n);
        break;
    case ImageKernel::kMixed:
        hipLaunchKernelGGL(scatter_layout<true>, dim3(gx, gy), dim3(kBlock), 0, stream, span,
                           t.tiles, t.win, t.rows, base, tile_bytes, n);
        break;
    case ImageKernel::kLink:
        gx = std::min((n + kLinkRun - 1) / kLinkRun, link_blocks(n, t.nrows));
        hipLaunchKernelGGL(scatter_layout_link, dim3(gx), dim3(kBlock), 0, stream, span, t.tiles,
                           t.win, t.rows, base, tile_bytes, n);
        break;
    }
    return hipGetLastError();
}

// Workgroups that share the ranges of long segments: enough in all to fill
// the chip.
static uint32_t table_slices(uint32_t gx, const TileDev* tiles) {
    return tiles ? std::max(1u, std::min(256u, 1024u / gx)) : 1u;
}

hipError_t launch_layout_tables(const LayoutRow* from, const uint32_t* len, const uint64_t* dst,
                                uint32_t n, uint32_t tile_bytes, LayoutSeg* rows, TileDev* tiles,
                                uint64_t ntiles, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const uint32_t shift = tile_shift(tile_bytes);
    if (tiles && ntiles >= 4ull * n) {
        const uint32_t gx = (uint32_t)(((uint64_t)n + 3) / 4);
        hipLaunchKernelGGL(layout_tables<true>, dim3(gx, table_slices(gx, tiles)),
                           dim3(kTableBlock), 0, stream, from, len, dst, n, tile_bytes, shift,
                           rows, tiles);
    } else {
        const uint32_t gx = (uint32_t)(((uint64_t)n + kTableBlock - 1) / kTableBlock);
        hipLaunchKernelGGL(layout_tables<false>, dim3(gx, table_slices(gx, tiles)),
                           dim3(kTableBlock), 0, stream, from, len, dst, n, tile_bytes, shift,
                           rows, tiles);
    }
    return hipGetLastError();
}

hipError_t launch_ring_tables(const RingSeg* segs, uint32_t n, uint32_t tile_bytes, TileDev* tiles,
                              TileWin* wins, uint64_t ntiles, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const uint32_t shift = tile_shift(tile_bytes);
    if (ntiles >= 4ull * n) {
        const uint32_t gx = (uint32_t)(((uint64_t)n + 3) / 4);
        hipLaunchKernelGGL(ring_tables<true>, dim3(gx, table_slices(gx, tiles)), dim3(kTableBlock),
                           0, stream, segs, n, tile_bytes, shift, tiles, wins);
    } else {
        const uint32_t gx = (uint32_t)(((uint64_t)n + kTableBlock - 1) / kTableBlock);
        hipLaunchKernelGGL(ring_tables<false>, dim3(gx, table_slices(gx, tiles)),
                           dim3(kTableBlock), 0, stream, segs, n, tile_bytes, shift, tiles, wins);
    }
    return hipGetLastError();
}

hipError_t launch_layout_tables_by_value(const LayoutArgs& a, bool has_dst, uint32_t n,
                                         uint32_t s0, uint64_t before, uint64_t after,
                                         uint32_t tile_bytes, LayoutSeg* rows, TileDev* tiles,
                                         hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if ((has_dst ? 28ull : 20ull) * n > sizeof a) return hipErrorInvalidValue;
    const uint32_t gx = (n + 3) / 4;
    hipLaunchKernelGGL(layout_tables_by_value, dim3(gx, table_slices(gx, tiles)),
                       dim3(kTableBlock), 0, stream, a, has_dst ? 1u : 0u, n, s0, before, after,
                       tile_bytes, tile_shift(tile_bytes), rows, tiles);
    return hipGetLastError();
}

hipError_t launch_zero(const RangeDev* ranges, uint32_t n, hipStream_t stream) {
    for (uint32_t r0 = 0; r0 < n; r0 += kMaxGridBlocks) {
        const uint32_t m = std::min<uint32_t>(kMaxGridBlocks, n - r0);
        hipLaunchKernelGGL(zero_ranges, dim3(m), dim3(kBlock), 0, stream, ranges + r0, m);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ii
