// Internal interface between the C-ABI layer and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "onebit_grid.h"

namespace onebit {

// A unit of work: up to kTileElems consecutive elements of one segment,
// starting on a 64-element (one sign word) boundary.  Partial sums are kept per
// tile, and the chunk owners' passes with lookup tables walk tiles.
struct Tile {
    int64_t start;  // first flat element (multiple of 64)
    int32_t len;    // elements in the tile, 1..kTileElems
    int32_t seg;    // segment q = k*n + j
};

constexpr int kSubBlocks = 4;                       // float4 loads per lane per array
constexpr int kTileElems = kWave * 4 * kSubBlocks;  // 1024 elements = 16 sign words
constexpr int kTileWords = kTileElems / 64;
constexpr int kServerRowBatch = 32;                 // worker rows staged in LDS at a time

// The streaming passes walk the flat buffer in blocks: block b is elements
// [b * kTileElems, (b + 1) * kTileElems) of the padded length (only the last
// one can be short).  Tiles are cut at block boundaries, so a block holds
// whole tiles: one full tile (`whole`), or up to 16 short ones whose sign
// words fill it from its first word on.  Word w of a block belongs to tile
// `tile` + (number of bits of `starts` at or below w) - 1.
struct Block {
    int32_t tile;     // the block's first tile
    int32_t seg;      // that tile's segment
    uint32_t starts;  // bit w: a tile starts at the block's word w
    int32_t whole;    // 1: one tile of kTileElems elements
};

// A segment's range of the tile list and its length.
struct alignas(16) Segment {
    int64_t len;
    int32_t tile;   // its first tile
    int32_t tiles;  // 0 for an empty segment
    int32_t next;   // the next segment that is not empty (num_segments: none)
    int32_t pad[3];
};

// Plans whose segments all have at most this many tiles add a segment's partial
// sums in the order of a wave (see segment_sum), others in a workgroup's.
constexpr int kWaveSegTiles = 256;

// Device-side layout tables owned by a plan.
struct DeviceTables {
    const Tile *tiles;             // [T], in address (segment) order
    const Block *blocks;           // [num_blocks], every block of the padded length
    int64_t num_blocks;            // ceil(D / kTileElems)
    int64_t padded_len;            // D
    const int32_t *chunk_tiles;    // [T], tile ids in chunk-major order
    const Segment *segs;           // [S]
    int64_t num_segments;          // S
    const int32_t *server_blocks;  // chunk owners' shared-table workgroups, chunk-major
                                   // (entries of onebit_grid.h's server_block_entry)
};

// Gradient element types (the values of the ONEBIT_GRAD_* constants).
constexpr int kGradF32 = 0;
constexpr int kGradBF16 = 1;
constexpr int kGradF16 = 2;

hipError_t launch_warmup(const DeviceTables &tb, float *x, float *m,
                         float *v, const void *g, int grad_dtype, int64_t g_ld, int n_grads,
                         float lr, float beta1, float beta2, float eps, int use_bc, float bc1,
                         float bc2, hipStream_t s);

// m != NULL: fp32 momentum; m == NULL: momentum decoded from (m_bits, m_scales).
hipError_t launch_worker_pass(const DeviceTables &tb, int64_t num_tiles, const float *m,
                              const uint64_t *m_bits, const float *m_scales, const void *g,
                              int grad_dtype, int64_t g_ld, float *err, int64_t err_ld,
                              const float *scales, int64_t scales_ld, uint64_t *bits,
                              int64_t bits_ld, double *partial, int n_local, float beta1,
                              hipStream_t s);

hipError_t launch_adam_message(const DeviceTables &tb, const uint64_t *bits, const float *scales,
                               float *x, float *m, float *v, float lr, float beta1, float beta2,
                               float eps, int use_bc, float bc1, float bc2, hipStream_t s);

hipError_t launch_uncompressed(const DeviceTables &tb, float *x, float *m,
                               const float *v, const void *g, int grad_dtype, int64_t g_ld,
                               int n, float lr, float beta1, float eps, hipStream_t s);

// out[0] = sum of |v| over the real elements (fp64, fixed order); partial
// holds at least min(2048, num_blocks / 4 + 8) values.
hipError_t launch_l1_norm(const DeviceTables &tb, const float *v, double *partial, double *out,
                          hipStream_t s);

// zero_padding (here and below): padding elements are written as 0.
hipError_t launch_decode(const DeviceTables &tb, const uint64_t *bits, const float *scales,
                         float *out, int zero_padding, hipStream_t s);

// Segment scales from per-tile partial sums.  Worker form (cnt = 0): all
// num_segments segments of each of `rows` rows, scale[i*scales_ld + q] from
// partial[i*part_ld + tiles of q].  Server form: segments k*n + j for
// j in [jb, jb + cnt) and every tensor k, one row.  max_seg_tiles picks the
// lanes per segment.
hipError_t launch_finalize(const DeviceTables &tb, int64_t max_seg_tiles, int64_t num_segments,
                           int64_t rows, int n, int jb, int cnt, const double *partial,
                           int64_t part_ld, float *scales, int64_t scales_ld, hipStream_t s);

// Bytes of the chunk owners' lookup tables for `segments` owned segments.
size_t server_table_bytes(int n, int64_t segments);

// The chunk owners' pass over tiles [tile_begin, tile_begin + tile_count) of
// the chunk-major tile list, for chunks [cb, cb + nown) of num_tensors
// tensors.  tables != NULL (at least server_table_bytes(n, num_tensors *
// nown) bytes, 256-byte aligned) and flags (num_tensors * nown int32): the
// owned segments' tables are built there first and copied by the pass, which
// for n <= 32 runs the num_blocks shared-table workgroups of server_blocks
// (the call's range of DeviceTables::server_blocks); tables == NULL: the
// pass builds them per tile.  wpartial != NULL (only with every chunk owned,
// tables == NULL, n <= kServerRowBatch and both bases 0): wscales is written
// instead of read, from the workers' per-tile partial sums (rows of wpart_ld),
// as in launch_update.  direct (every chunk owned, both bases 0, any n): the
// pass that adds the workers one by one, over blocks.
hipError_t launch_server_pass(const DeviceTables &tb, int64_t tile_begin, int64_t tile_count,
                              int n, const uint64_t *wbits, int64_t bits_ld,
                              int64_t bits_word_base, float *wscales, int64_t scales_ld,
                              int64_t scales_seg_base, float *serr, float *sscales,
                              uint64_t *sbits, double *partial, const double *wpartial,
                              int64_t wpart_ld, int num_tensors, int cb,
                              int nown, double *tables, int32_t *flags,
                              const int32_t *server_blocks, int64_t num_blocks, bool direct,
                              hipStream_t s);

// partial != NULL: sscales is written instead of read, each segment's scale
// being formed from the chunk owners' per-tile partial sums (launch_finalize's
// work, in the pass that needs the scales).
hipError_t launch_update(const DeviceTables &tb, const uint64_t *sbits, float *sscales,
                         const double *partial, float *x, float *m_out, const float *v, float lr,
                         float eps, hipStream_t s);

// The library's own scratch memory, for callers that cannot allocate: a
// static device array of kScratchBytes on every device the library runs on,
// held until the process ends.  scratch_address() returns its device address
// on `device` (looked up once per device, with that device made current for
// the lookup and restored afterwards), or an error for a device index at or
// above kMaxScratchDevices or a failed lookup.  Every call on one device
// shares the array.
constexpr size_t kScratchBytes = (size_t)96 << 20;
constexpr int kMaxScratchDevices = 64;
hipError_t scratch_address(int device, void **ptr);

hipError_t launch_materialize(const DeviceTables &tb, int rows, const float *err, int64_t err_ld,
                              const float *scales, int64_t scales_ld, float *out, int64_t out_ld,
                              int zero_padding, hipStream_t s);

}  // namespace onebit
