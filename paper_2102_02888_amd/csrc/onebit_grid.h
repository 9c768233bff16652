// Launch shapes of the tile kernels and the order in which their waves take
// work.  Integer arithmetic only, with no HIP dependency, so that a host
// program can enumerate a whole launch and check that every tile or item is
// taken by exactly one wave.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define ONEBIT_HD __host__ __device__
#else
#define ONEBIT_HD
#endif

namespace onebit {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kBlock = kWave * kWavesPerBlock;

// The first compression step's row walk runs 16-wave workgroups and gives two
// waves to each 1024-element block (half a block each): 8 blocks per
// workgroup.
constexpr int kWorkerWavesPerBlock = 2;
constexpr int kRowWaves = 16;
constexpr int kRowBlock = kWave * kRowWaves;
constexpr int kWorkerRowTiles = kRowWaves / kWorkerWavesPerBlock;

// Workgroups are dispatched to the chip's 8 XCDs round-robin (block b runs on
// XCD (b + c) % 8 for a fixed c), and each XCD has its own L2.  Grids are
// launched as multiples of 8 blocks and renumbered so that each XCD takes one
// contiguous eighth of the work: every XCD then streams its own address range
// instead of all eight interleaving pieces of the same streams.
constexpr int kXcds = 8;

// Plans keep the tile count below 2^25, so a grid of one wave per tile stays
// far below the 2^32 work-item limit.  The finalize kernel caps its grid at
// kMaxGridBlocks and strides.  All others launch one workgroup (or wave) for each
// piece of work, in as many launches as it takes: at most kMaxLaunchTiles
// blocks, tiles or table-sharing workgroups of up to 256 threads at a time (2^30
// work-items), and at most kMaxPassItems (row, block) items of the worker pass
// and the explicit errors, one workgroup of up to 256 threads each, so that a
// BERT-Large-sized pass (n = 32) is one launch.
constexpr int64_t kMaxGridBlocks = (int64_t)1 << 22;
constexpr int64_t kMaxPassItems = (int64_t)3 << 22;
static_assert(kMaxPassItems * kBlock < ((int64_t)1 << 32), "work-items of one launch");
constexpr int64_t kMaxLaunchTiles = (int64_t)1 << 22;

// Tiles (or workgroups) of the launch that starts at base, of total.
ONEBIT_HD inline int64_t launch_piece(int64_t total, int64_t base)
{
    return total - base < kMaxLaunchTiles ? total - base : kMaxLaunchTiles;
}

// Blocks for one wave per item at waves_per_block waves per block, rounded up
// to a multiple of kXcds (0 for no items).
ONEBIT_HD inline int64_t xcd_grid(int64_t waves, int waves_per_block)
{
    const int64_t blocks = (waves + waves_per_block - 1) / waves_per_block;
    return (blocks + kXcds - 1) / kXcds * kXcds;
}

// Logical block of physical block b in a grid of `grid` blocks (a multiple of
// kXcds): the blocks of XCD x are logical blocks [x, x + 1) * grid / kXcds.
ONEBIT_HD inline int64_t xcd_block_of(int64_t b, int64_t grid)
{
    return (b % kXcds) * (grid / kXcds) + b / kXcds;
}

// Chunk owners' workgroups that share one segment's lookup tables: each takes
// up to kWavesPerBlock consecutive tiles of one segment in the chunk-major
// tile list, one per wave.  A segment whose tiles sit at list positions
// [pos, pos + count) gets server_blocks_of(count) workgroups; entry i is
// server_block_entry(pos, count, i), from which the kernel reads the first
// position and the number of tiles.  Positions stay below 2^25 (the plans'
// tile limit), so an entry fits an int32.
ONEBIT_HD inline int64_t server_blocks_of(int64_t count)
{
    return (count + kWavesPerBlock - 1) / kWavesPerBlock;
}

ONEBIT_HD inline int32_t server_block_entry(int64_t pos, int64_t count, int64_t i)
{
    const int64_t first = pos + i * kWavesPerBlock;
    const int64_t left = pos + count - first;
    return (int32_t)(first * 8 + (left < kWavesPerBlock ? left : kWavesPerBlock));
}

ONEBIT_HD inline int64_t server_block_first(int32_t entry) { return entry >> 3; }
ONEBIT_HD inline int server_block_tiles(int32_t entry) { return entry & 7; }

// Exact quotient of an item number below 2^31 by a fixed divisor d < 2^31:
// (item * mul) >> shift with mul = ceil(2^(31+s) / d), s = ceil(log2 d),
// shift = 31 + s.  mul * d exceeds 2^(31+s) by less than d <= 2^s, so the
// error item * (mul * d - 2^(31+s)) / (d * 2^(31+s)) stays below 1/d.
struct FastDiv {
    uint64_t mul;
    uint32_t shift;
};

ONEBIT_HD inline FastDiv fast_div(int64_t d)
{
    uint32_t s = 0;
    while (((int64_t)1 << s) < d) ++s;
    const uint64_t one = (uint64_t)1 << (31 + s);
    return {(one + (uint64_t)d - 1) / (uint64_t)d, 31 + s};
}

// Quotient of x (below 2^31) by the divisor f was made for.
ONEBIT_HD inline int64_t fast_quotient(int64_t x, FastDiv f)
{
    return (int64_t)(((uint64_t)x * f.mul) >> f.shift);
}

}  // namespace onebit
