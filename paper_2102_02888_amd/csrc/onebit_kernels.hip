// gfx950 kernels of the 1-bit Adam hot path (arXiv 2102.02888).
//
// Every kernel streams over the flat parameter buffer and, except for the
// chunk owners' decode-and-average (bound by vector ALU issue), is bound by
// HBM bandwidth; no MFMA (nothing here is a dense contraction).  The streaming
// passes walk blocks of 1024 elements (onebit_internal.h), each wave (64 lanes)
// holding one or more sub-blocks of 256 elements, a float4 per lane, so every
// global load/store is a 128-bit access and a wave moves 1 KiB per instruction.
// The chunk owners' passes with lookup tables walk tiles, up to 1024 elements
// that never cross a segment, as lists of one owner's tiles.  A sub-block spans
// four 16-lane DPP rows, and each row's 64 elements form one LSB-first uint64
// sign word (bit b of word w of a block or tile <=> element 64w+b), assembled
// with a row-wide OR of the lanes' 4-bit nibbles.
//
// Arithmetic contract (shared with the layout/format description in
// onebit.h): fp32 values, one rounding per operation (built with
// -ffp-contract=off), correctly rounded sqrt and division, fp64 reductions
// rounded once to fp32.  Reductions over a segment are deterministic:
// per-tile partial sums (a fixed lane reduction order) are written to a
// workspace and summed in a fixed order by a finalize kernel, or by the pass
// that needs the scale; no atomics.
#include "onebit_internal.h"
#include <algorithm>
#include <mutex>

namespace onebit {
namespace {

// Four consecutive floats.  The native vector type lets the non-temporal
// builtins take it; every stream here is touched once per launch, so loads
// and stores are non-temporal (they do not displace other data in the caches
// on the way to HBM).
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u32 __attribute__((ext_vector_type(4)));
typedef uint32_t v2u32 __attribute__((ext_vector_type(2)));

// Full tiles move through raw buffer instructions: the base sits in scalar
// registers and each lane adds a 32-bit byte offset, and the cache policy is
// an operand.  Loads are non-temporal (nt); stores are non-temporal at device
// scope (nt and sc1), which drains the streams of written state to HBM faster
// than nt alone.  The resource covers 2 GiB from the base, far more than a
// block; its fourth word is the gfx9-family buffer format word.
constexpr int kStreamLoad = 2;        // nt
constexpr int kStreamStore = 2 | 16;  // nt, sc1
// Small plans, whose rows can stay in the caches (row_caching): stores, and of
// the smallest ones gradient loads, without nt.
constexpr int kCachedLoad = 0;
constexpr int kCachedStore = 16;      // sc1

// Resource for a wave-uniform base p (a tile's start in some row: every
// caller's p is the same in all lanes).  p is read from the first active lane,
// so the base stays in scalar registers even where the compiler holds it in
// vector registers, with no per-access loop over distinct lane values.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t stream_rsrc(const void *p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)hi << 32) | lo), (short)0,
                                             0x7FFFFFFF, 0x00020000);
}

// Loads elements li..li+3 of p; FULL means the whole tile is in range (a
// wave-uniform fact), otherwise lanes past len read zeros.
template <bool FULL>
__device__ __forceinline__ v4f ld4(const float *__restrict__ p, int li, int len)
{
    if (FULL)
        return __builtin_bit_cast(
            v4f, __builtin_amdgcn_raw_buffer_load_b128(stream_rsrc(p), li * 4, 0, kStreamLoad));
    if (li + 4 <= len) return __builtin_nontemporal_load((const v4f *)(p + li));
    v4f r = {0.f, 0.f, 0.f, 0.f};
    if (li < len) r.x = p[li];
    if (li + 1 < len) r.y = p[li + 1];
    if (li + 2 < len) r.z = p[li + 2];
    return r;
}

// Stores elements li..li+3 of p.  Full tiles store non-temporally; partial
// tiles store plainly (lanes past len store nothing), because their waves
// may still load after storing.
template <bool FULL>
__device__ __forceinline__ void st4(float *__restrict__ p, int li, int len, v4f v)
{
    if (FULL) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u32, v), stream_rsrc(p),
                                               li * 4, 0, kStreamStore);
        return;
    }
    if (li + 4 <= len) {
        *(v4f *)(p + li) = v;
        return;
    }
    if (li < len) p[li] = v.x;
    if (li + 1 < len) p[li + 1] = v.y;
    if (li + 2 < len) p[li + 2] = v.z;
}

// Gradient element types.  16-bit gradients are widened to fp32 exactly
// (bf16 by a 16-bit shift, fp16 by the hardware conversion), so the method's
// arithmetic is the same as for fp32 gradients of those values.
struct GradF32 {
    using T = float;
};
struct GradBF16 {
    using T = uint16_t;
};
struct GradF16 {
    using T = _Float16;
};

__device__ __forceinline__ float widen(uint16_t a) { return __uint_as_float((uint32_t)a << 16); }
__device__ __forceinline__ float widen(_Float16 a) { return (float)a; }

typedef uint16_t v4u16 __attribute__((ext_vector_type(4)));
typedef _Float16 v4f16 __attribute__((ext_vector_type(4)));

// 16-bit gradient elements li..li+3 as fp32.
template <class G, int POLICY>
__device__ __forceinline__ v4f ldg4(const typename G::T *__restrict__ p, int li)
{
    const v2u32 w = __builtin_amdgcn_raw_buffer_load_b64(stream_rsrc(p), li * 2, 0, POLICY);
    v4f r;
    if constexpr (__is_same(typename G::T, uint16_t)) {
        const v4u16 h = __builtin_bit_cast(v4u16, w);
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = widen((uint16_t)h[c]);
    } else {
        const v4f16 h = __builtin_bit_cast(v4f16, w);
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = widen((_Float16)h[c]);
    }
    return r;
}

// OR of a 32-bit value over the 16 lanes of each DPP row (every lane of the
// row receives the result).  xor-1 and xor-2 quad permutes OR each quad; the
// row rotations by 4 and by 8 then OR the four quads, whichever way the
// rotation turns.
__device__ __forceinline__ uint32_t row_or16(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);   // quad_perm 2,3,0,1
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, false);  // row_ror 4
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);  // row_ror 8
    return v;
}

// Sign word of 64 consecutive elements held by one 16-lane row, 4 per lane:
// lane L of the row contributes its 4 sign bits (nib, element 4L+c at bit c)
// at bit positions 4L..4L+3.  Every lane of the row receives the word.
__device__ __forceinline__ uint64_t row_sign_word(uint32_t nib, int lane)
{
    const int r = lane & 15;
    const uint32_t lo = r < 8 ? nib << (4 * r) : 0u;
    const uint32_t hi = r >= 8 ? nib << (4 * (r - 8)) : 0u;
    return ((uint64_t)row_or16(hi) << 32) | (uint64_t)row_or16(lo);
}

// DPP move of an fp64 value (both 32-bit halves); lanes the pattern does not
// reach get 0.0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Deterministic wave-wide fp64 sums (every lane gets the same value).
// wave_sum: xor butterfly through lane shuffles (cross-lane traffic goes
// through the LDS crossbar, off the vector ALU).
__device__ __forceinline__ double wave_sum(double a)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) a += __shfl_xor(a, off, kWave);
    return a;
}

// wave_sum_dpp: a fixed tree of DPP row shifts and row broadcasts read from
// lane 63; fewer instructions, but six dependent vector steps.  The worker
// pass (short waves, bound by memory latency) measured ~0.6% slower with it,
// the ALU-bound chunk-owner pass faster.
__device__ __forceinline__ double wave_sum_dpp(double a)
{
    a += dpp_f64<0x111, 0xF>(a);  // row_shr 1
    a += dpp_f64<0x112, 0xF>(a);  // row_shr 2
    a += dpp_f64<0x114, 0xF>(a);  // row_shr 4
    a += dpp_f64<0x118, 0xF>(a);  // row_shr 8
    a += dpp_f64<0x142, 0xA>(a);  // row_bcast 15
    a += dpp_f64<0x143, 0xC>(a);  // row_bcast 31
    const int lo = __builtin_amdgcn_readlane(__double2loint(a), kWave - 1);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(a), kWave - 1);
    return __hiloint2double(hi, lo);
}

// This block's logical number in a grid launched by xcd_grid (one contiguous
// eighth of the logical blocks per XCD).
__device__ __forceinline__ int64_t xcd_block() { return xcd_block_of(blockIdx.x, gridDim.x); }

// This wave's number within its workgroup, as a wave-uniform (scalar) value,
// so that tile indices, tile descriptors and the addresses derived from them
// stay in scalar registers.  Kernels whose waves take different tiles or blocks
// use it; where a workgroup has one block, the block's number already is
// scalar.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Error from the compensated form: z - C[z] given z and its segment scale s.
__device__ __forceinline__ float error_of(float z, float s) { return z >= 0.f ? z - s : z + s; }

// ---------------------------------------------------------------------------
// Blocks (the streaming passes).  A wave's loads of a block need its number
// only, so they are issued before the block's record, and the scales that
// hang on it, have arrived.  A whole block is one full tile of one segment.
// A mixed block (short tiles, several segments, padding) is streamed the same
// way; each 16-lane row holds one sign word, which lies in one tile, so the
// lanes look up their row's tile and store only their real elements.
// ---------------------------------------------------------------------------

// The record of block b (wave-uniform), in one 128-bit load.
__device__ __forceinline__ Block load_block(const Block *__restrict__ blocks, int64_t b)
{
    const int4 r = ((const int4 *)blocks)[b];
    return Block{r.x, r.y, (uint32_t)r.z, r.w};
}

// Loads elements li..li+3 of the block at p; lim = elements of the block
// inside the padded length (a multiple of 64).  INSIDE: the whole block is.
template <bool INSIDE, int POLICY = kStreamLoad>
__device__ __forceinline__ v4f ldb4(const float *__restrict__ p, int li, int lim)
{
    if (INSIDE || li < lim)
        return __builtin_bit_cast(
            v4f, __builtin_amdgcn_raw_buffer_load_b128(stream_rsrc(p), li * 4, 0, POLICY));
    return v4f{0.f, 0.f, 0.f, 0.f};
}

template <bool INSIDE, class G, int POLICY = kStreamLoad>
__device__ __forceinline__ v4f ldgb4(const typename G::T *__restrict__ p, int li, int lim)
{
    if constexpr (sizeof(typename G::T) == 4) {
        return ldb4<INSIDE, POLICY>((const float *)p, li, lim);
    } else {
        if (INSIDE || li < lim) return ldg4<G, POLICY>(p, li);
        return v4f{0.f, 0.f, 0.f, 0.f};
    }
}

// The tile of word w of a mixed block (w inside the padded length).
__device__ __forceinline__ Tile block_word_tile(const Tile *__restrict__ tiles, const Block &rec,
                                                int w)
{
    return tiles[rec.tile + __popc(rec.starts & ((2u << w) - 1u)) - 1];
}

// How many of the 4 elements at flat index e the tile holds (0..4).
__device__ __forceinline__ int tile_valid4(const Tile &t, int64_t e)
{
    const int64_t left = t.start + t.len - e;
    return left >= 4 ? 4 : left > 0 ? (int)left : 0;
}

// Stores elements li..li+3 of the block at p, the first `valid` of them.
template <bool WHOLE, bool CACHED = false>
__device__ __forceinline__ void stb4(float *__restrict__ p, int li, int valid, v4f v)
{
    if (WHOLE || valid == 4) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u32, v), stream_rsrc(p),
                                               li * 4, 0, CACHED ? kCachedStore : kStreamStore);
        return;
    }
    if (valid > 0) p[li] = v.x;
    if (valid > 1) p[li + 1] = v.y;
    if (valid > 2) p[li + 2] = v.z;
}

// Sum over the 16 lanes of each row (every lane of the row gets it).
__device__ __forceinline__ double row_sum(double a)
{
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) a += __shfl_xor(a, off, kWave);
    return a;
}

// Sum of tile j's words of a mixed block from the words' sums, in word order.
__device__ __forceinline__ double block_tile_sum(const double *__restrict__ words, uint32_t starts,
                                                 int j)
{
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kTileWords; ++w)
        if (__popc(starts & ((2u << w) - 1u)) - 1 == j) s += words[w];
    return s;
}

// The sign bit of +-a (bit set: +a), exact for any a.
__device__ __forceinline__ float with_sign(float a, uint32_t nib, int c)
{
    return __uint_as_float(__float_as_uint(a) ^ (((~nib >> c) & 1u) << 31));
}

// ---------------------------------------------------------------------------
// Warm-up Adam (eq. (alg:v)) on the average of n_grads gradient rows.
//
// The row-summing kernels (this one and the 32-bit comparison step) come in
// three shapes (launch_row_sum picks one): SB sub-blocks of a block per wave,
// WAVES waves per workgroup, the loads of BATCH rows issued together.  With
// BATCH = 1 the waves of a workgroup read each gradient row together, with a
// workgroup barrier after every row, so that a row is streamed in runs of
// WAVES * SB KB (fp32); waves past the last block keep the pace, so every wave
// reaches every barrier.
// ---------------------------------------------------------------------------
template <int SB_, int WAVES_, int BATCH_>
struct RowShape {
    static constexpr int SB = SB_, WAVES = WAVES_, BATCH = BATCH_;
    static constexpr int PARTS = kSubBlocks / SB_;  // waves per block
};

// This wave's part of a block in the row-summing kernels.
struct RowPart {
    int64_t blk, base;
    int lim, sb0;
    bool active;
};

template <class Sh>
__device__ __forceinline__ RowPart row_part(int64_t block_base, int64_t num_blocks,
                                            int64_t padded_len)
{
    const int64_t u = xcd_block() * Sh::WAVES + wave_id();
    RowPart r;
    r.blk = block_base + u / Sh::PARTS;
    r.sb0 = (int)(u % Sh::PARTS) * Sh::SB;
    r.active = r.blk < num_blocks;
    r.base = r.blk * kTileElems;
    const int64_t room = padded_len - r.base;
    r.lim = room < kTileElems ? (int)room : kTileElems;
    return r;
}

template <bool INSIDE, class G, int SB>
__device__ __forceinline__ void load_grad_row(v4f (&gv)[SB], const typename G::T *__restrict__ row,
                                              int sb0, int lane, int lim)
{
#pragma unroll
    for (int b = 0; b < SB; ++b)
        gv[b] = ldgb4<INSIDE, G>(row, (sb0 + b) * (kWave * 4) + 4 * lane, lim);
}

// sum += one loaded gradient row (fp64, rows added in row order)
template <int SB>
__device__ __forceinline__ void add_grad_row(double (&sum)[SB][4], const v4f (&gv)[SB], bool in)
{
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[b][c] += in ? (double)gv[b][c] : 0.0;
}

// sum += worker i's momentum beta1 m + (1 - beta1) g_i (fp32, then fp64 sum)
template <int SB>
__device__ __forceinline__ void add_momentum_row(double (&sum)[SB][4], const v4f (&bm)[SB],
                                                 const v4f (&gv)[SB], bool in, float omb1)
{
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float mi = omb1 * gv[b][c];
            mi = bm[b][c] + mi;
            sum[b][c] += in ? (double)mi : 0.0;
        }
}

// Reads the n rows of this wave's part in row order, BATCH rows' loads at a
// time, and hands each to use(gv, last), last telling that it is a row past
// the end (the last row again, to be left out).  With BATCH = 1 the waves of
// the workgroup read each row together (a barrier after every row).
template <bool INSIDE, class G, int SB, int BATCH, class Use>
__device__ __forceinline__ void walk_rows(const RowPart &p, const typename G::T *__restrict__ row,
                                          int64_t g_ld, int n, int lane, Use use)
{
    for (int i = 0; i < n; i += BATCH) {
        if (p.active) {
            v4f gv[BATCH][SB];
#pragma unroll
            for (int k = 0; k < BATCH; ++k)
                load_grad_row<INSIDE, G, SB>(gv[k], row + (int64_t)min(i + k, n - 1) * g_ld, p.sb0,
                                             lane, p.lim);
#pragma unroll
            for (int k = 0; k < BATCH; ++k) use(gv[k], i + k < n);
        }
        if (BATCH == 1) __builtin_amdgcn_s_barrier();
    }
}

// How many of the lane's 4 elements of each sub-block are real.
template <int SB>
__device__ __forceinline__ void part_valid(int (&valid)[SB], const Tile *__restrict__ tiles,
                                           const Block &rec, const RowPart &p, int lane)
{
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        const int li = (p.sb0 + b) * (kWave * 4) + 4 * lane;
        valid[b] = 4;
        if (!rec.whole)
            valid[b] = li < p.lim
                           ? tile_valid4(block_word_tile(tiles, rec, li >> 6), p.base + li)
                           : 0;
    }
}

template <class G, class Sh>
__global__ __launch_bounds__(Sh::WAVES *kWave) void k_warmup(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t block_base,
    int64_t num_blocks,
    int64_t padded_len, float *__restrict__ x, float *__restrict__ m, float *__restrict__ v,
    const typename G::T *__restrict__ g, int64_t g_ld, int n_grads, float lr, float beta1,
    float omb1, float beta2, float omb2, float eps, int use_bc, float bc1, float bc2)
{
    constexpr int SB = Sh::SB;
    const int lane = threadIdx.x & (kWave - 1);
    const RowPart p = row_part<Sh>(block_base, num_blocks, padded_len);
    double sum[SB][4];
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[b][c] = 0.0;
    const typename G::T *row = g + p.base;
    const auto use = [&](const v4f(&gv)[SB], bool in) { add_grad_row<SB>(sum, gv, in); };
    if (p.lim == kTileElems)
        walk_rows<true, G, SB, Sh::BATCH>(p, row, g_ld, n_grads, lane, use);
    else
        walk_rows<false, G, SB, Sh::BATCH>(p, row, g_ld, n_grads, lane, use);
    if (!p.active) return;
    const Block rec = load_block(blocks, p.blk);
    x += p.base;
    m += p.base;
    v += p.base;
    v4f xv[SB], mv[SB], vv[SB];
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        const int li = (p.sb0 + b) * (kWave * 4) + 4 * lane;
        xv[b] = ldb4<false>(x, li, p.lim);
        mv[b] = ldb4<false>(m, li, p.lim);
        vv[b] = ldb4<false>(v, li, p.lim);
    }
    int valid[SB];
    part_valid<SB>(valid, tiles, rec, p, lane);
    const double dn = (double)n_grads;
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        const int li = (p.sb0 + b) * (kWave * 4) + 4 * lane;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float gbar = (float)(sum[b][c] / dn);
            float mn = beta1 * mv[b][c];
            mn = mn + omb1 * gbar;
            const float gsq = gbar * gbar;
            float vn = beta2 * vv[b][c];
            vn = vn + omb2 * gsq;
            float mh = mn, vh = vn;
            if (use_bc) {
                mh = mn / bc1;
                vh = vn / bc2;
            }
            const float denom = __builtin_sqrtf(vh) + eps;
            const float ratio = mh / denom;
            const float step = lr * ratio;
            xv[b][c] = xv[b][c] - step;
            mv[b][c] = mn;
            vv[b][c] = vn;
        }
        stb4<false>(x, li, valid[b], xv[b]);
        stb4<false>(m, li, valid[b], mv[b]);
        stb4<false>(v, li, valid[b], vv[b]);
    }
}

// ---------------------------------------------------------------------------
// "1-bit Adam (32-bits)" comparison variant (Section 7.2): the compression
// stage with the identity compressor -- variance frozen, momenta averaged
// uncompressed.  m_i = beta1 m + (1-beta1) g_i per worker, m = mean_i m_i
// (fp64 sum in worker order, one rounding), x -= lr m / sqrt(v + eps).
// ---------------------------------------------------------------------------
template <class G, class Sh>
__global__ __launch_bounds__(Sh::WAVES *kWave) void k_uncompressed(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t block_base,
    int64_t num_blocks,
    int64_t padded_len, float *__restrict__ x, float *__restrict__ m, const float *__restrict__ v,
    const typename G::T *__restrict__ g, int64_t g_ld, int n, float lr, float beta1, float omb1,
    float eps)
{
    constexpr int SB = Sh::SB;
    const int lane = threadIdx.x & (kWave - 1);
    const RowPart p = row_part<Sh>(block_base, num_blocks, padded_len);
    double sum[SB][4];
    v4f bm[SB], xv[SB], vv[SB];
    // whole-block waves load x and v ahead of the rows, with m (BERT-Base, 16
    // rows: 1.450 ms against 1.517 after them)
    constexpr bool kEarly = SB == kSubBlocks;
    x += p.base;
    v += p.base;
    if (p.active) {
        m += p.base;
#pragma unroll
        for (int b = 0; b < SB; ++b) {
            const int li = (p.sb0 + b) * (kWave * 4) + 4 * lane;
            bm[b] = beta1 * ldb4<false>(m, li, p.lim);
            if (kEarly) {
                xv[b] = ldb4<false>(x, li, p.lim);
                vv[b] = ldb4<false>(v, li, p.lim);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[b][c] = 0.0;
        }
    }
    const typename G::T *row = g + p.base;
    const auto use = [&](const v4f(&gv)[SB], bool in) { add_momentum_row<SB>(sum, bm, gv, in, omb1); };
    if (p.lim == kTileElems)
        walk_rows<true, G, SB, Sh::BATCH>(p, row, g_ld, n, lane, use);
    else
        walk_rows<false, G, SB, Sh::BATCH>(p, row, g_ld, n, lane, use);
    if (!p.active) return;
    const Block rec = load_block(blocks, p.blk);
    if (!kEarly) {
#pragma unroll
        for (int b = 0; b < SB; ++b) {
            const int li = (p.sb0 + b) * (kWave * 4) + 4 * lane;
            xv[b] = ldb4<false>(x, li, p.lim);
            vv[b] = ldb4<false>(v, li, p.lim);
        }
    }
    int valid[SB];
    part_valid<SB>(valid, tiles, rec, p, lane);
    const double dn = (double)n;
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        const int li = (p.sb0 + b) * (kWave * 4) + 4 * lane;
        v4f mv;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float mbar = (float)(sum[b][c] / dn);
            const float denom = __builtin_sqrtf(vv[b][c] + eps);
            const float ratio = mbar / denom;
            const float step = lr * ratio;
            xv[b][c] = xv[b][c] - step;
            mv[c] = mbar;
        }
        stb4<false>(x, li, valid[b], xv[b]);
        stb4<false>(m, li, valid[b], mv);
    }
}

// ---------------------------------------------------------------------------
// The sum of a segment's per-tile partial sums, in one order for every plan
// whose segments have at most 256 tiles, whichever pass or number of lanes adds
// them: 64 strided sums, v's being (p[v] + p[v + 64]) + (p[v + 128] + p[v +
// 192]), then v and v + 32, then v and v + 16, and so on down to v and v + 1.
// LANES lanes (a power of two) each hold 64 / LANES of the strided sums; MAX is
// the most tiles there can be, and all loads are issued together.  Every lane
// gets the sum.  (Absent tiles add 0, which changes no sum of squares.)
// ---------------------------------------------------------------------------
template <int LANES, int MAX>
__device__ __forceinline__ double segment_sum(const double *__restrict__ part, int tiles, int lane)
{
    constexpr int J = MAX < kWave ? (MAX + LANES - 1) / LANES : kWave / LANES;
    constexpr int R = (MAX + kWave - 1) / kWave;
    static_assert((J & (J - 1)) == 0 && (R == 1 || R == 4), "whole rounds");
    double p[R][J];
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int t = lane + LANES * j + kWave * k;
            p[k][j] = t < tiles ? part[t] : 0.0;
        }
    double s[J];
#pragma unroll
    for (int j = 0; j < J; ++j)
        s[j] = R == 1 ? p[0][j] : (p[0][j] + p[R > 1][j]) + (p[R / 2][j] + p[R - 1][j]);
#pragma unroll
    for (int h = J / 2; h >= 1; h /= 2)
#pragma unroll
        for (int j = 0; j < h; ++j) s[j] += s[j + h];
#pragma unroll
    for (int off = LANES / 2; off >= 1; off >>= 1) s[0] += __shfl_xor(s[0], off, kWave);
    return s[0];
}

// ---------------------------------------------------------------------------
// Scales formed where they are needed (the fused step on plans whose segments
// have few tiles): the pass that reads a scale sums its segment's partial sums
// itself, and the part that holds the segment's first word writes the scale
// out, with the zeros of the empty segments around it.  Every reader sums in
// the same order, so all get the same value.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float scale_of(double sum, int64_t len)
{
    return (float)__builtin_sqrt(sum / (double)len);
}

// Zeros for the empty segments after segment q (and before it, when q is the
// first that is not empty), by `lanes` lanes.
__device__ __forceinline__ void zero_empty(float *__restrict__ scales, int q, const Segment &sg,
                                           int lane, int lanes)
{
    for (int e = q + 1 + lane; e < sg.next; e += lanes) scales[e] = 0.f;
    if (sg.tile == 0)
        for (int e = lane; e < q; e += lanes) scales[e] = 0.f;
}

// The scale of segment sg (at most kWaveSegTiles tiles), in the finalize
// kernel's order, by a whole wave or by each 16-lane row for a segment of its
// own.
__device__ __forceinline__ float wave_scale(const Segment &sg, const double *__restrict__ partial,
                                            int lane)
{
    return scale_of(segment_sum<kWave, kWaveSegTiles>(partial + sg.tile, sg.tiles, lane),
                    sg.len);
}

__device__ __forceinline__ float row_scale(const Segment &sg, const double *__restrict__ partial,
                                           int lane)
{
    return scale_of(segment_sum<16, kWaveSegTiles>(partial + sg.tile, sg.tiles, lane & 15),
                    sg.len);
}

// ---------------------------------------------------------------------------
// One sub-block of a block as a wave of the update-like passes sees it: which
// elements are real, and the sign word and scale of each lane's segment.  The
// caller issues its own loads first; INSIDE as in ldb4.
// ---------------------------------------------------------------------------
struct Lane4 {
    float s;       // the scale of the lane's segment
    uint32_t nib;  // the lane's 4 sign bits (bits above are undefined)
    int valid;     // how many of its 4 elements are real
};

template <bool WHOLE>
__device__ __forceinline__ Lane4 lane_message(const Tile *__restrict__ tiles, const Block &rec,
                                              int64_t base, int li, int lim, uint64_t word, float s0,
                                              const float *__restrict__ scales)
{
    Lane4 r{s0, (uint32_t)(word >> (li & 63)), 4};
    if (!WHOLE) {
        r.valid = 0;
        if (li < lim) {
            const Tile t = block_word_tile(tiles, rec, li >> 6);
            r.valid = tile_valid4(t, base + li);
            r.s = scales[t.seg];
        }
    }
    return r;
}

// ---------------------------------------------------------------------------
// Adam step whose gradient is a decoded message (g = bit ? scale : -scale);
// the "Adam(1-bit Naive)" comparison variant of Section 7.2 updates m and v
// from the compressed gradient this way.  A workgroup takes one block, one
// 256-element sub-block per wave, as in the update.  Loads first, then stores.
// Five workgroups per CU, held by unused LDS (3 KB of loads per wave, 15 KB per
// SIMD): the naive step on 200 fp16 tensors 371.6 us at eight, 367.8 at five.
// ---------------------------------------------------------------------------
template <bool WHOLE>
__device__ __forceinline__ void adam_message_sub(const Lane4 &l, int li, v4f xv, v4f mv, v4f vv,
                                                 float *__restrict__ x, float *__restrict__ m,
                                                 float *__restrict__ v, float lr, float beta1,
                                                 float omb1, float beta2, float omb2, float eps,
                                                 int use_bc, float bc1, float bc2)
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float gbar = with_sign(l.s, l.nib, c);
        float mn = beta1 * mv[c];
        mn = mn + omb1 * gbar;
        const float gsq = gbar * gbar;
        float vn = beta2 * vv[c];
        vn = vn + omb2 * gsq;
        float mh = mn, vh = vn;
        if (use_bc) {
            mh = mn / bc1;
            vh = vn / bc2;
        }
        const float denom = __builtin_sqrtf(vh) + eps;
        const float ratio = mh / denom;
        const float step = lr * ratio;
        xv[c] = xv[c] - step;
        mv[c] = mn;
        vv[c] = vn;
    }
    stb4<WHOLE>(x, li, l.valid, xv);
    stb4<WHOLE>(m, li, l.valid, mv);
    stb4<WHOLE>(v, li, l.valid, vv);
}

__global__ __launch_bounds__(kBlock) void k_adam_message(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t block_base,
    int64_t num_blocks, int64_t padded_len, const uint64_t *__restrict__ bits,
    const float *__restrict__ scales, float *__restrict__ x, float *__restrict__ m,
    float *__restrict__ v, float lr, float beta1, float omb1, float beta2, float omb2, float eps,
    int use_bc, float bc1, float bc2)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t blk = block_base + xcd_block();
    if (blk >= num_blocks) return;
    const int64_t base = blk * kTileElems;
    const int64_t room = padded_len - base;
    const int lim = room < kTileElems ? (int)room : kTileElems;
    const int li = (threadIdx.x >> 6) * (kWave * 4) + 4 * lane;
    x += base;
    m += base;
    v += base;
    uint64_t word = 0;
    v4f xv, mv, vv;
    if (lim == kTileElems || li < lim) word = bits[(base + li) >> 6];
    if (lim == kTileElems) {
        xv = ldb4<true>(x, li, lim);
        mv = ldb4<true>(m, li, lim);
        vv = ldb4<true>(v, li, lim);
    } else {
        xv = ldb4<false>(x, li, lim);
        mv = ldb4<false>(m, li, lim);
        vv = ldb4<false>(v, li, lim);
    }
    const Block rec = load_block(blocks, blk);
    const float s0 = scales[rec.seg];
    if (rec.whole)
        adam_message_sub<true>(lane_message<true>(tiles, rec, base, li, lim, word, s0, scales), li,
                               xv, mv, vv, x, m, v, lr, beta1, omb1, beta2, omb2, eps, use_bc, bc1,
                               bc2);
    else
        adam_message_sub<false>(lane_message<false>(tiles, rec, base, li, lim, word, s0, scales),
                                li, xv, mv, vv, x, m, v, lr, beta1, omb1, beta2, omb2, eps, use_bc,
                                bc1, bc2);
}

// ---------------------------------------------------------------------------
// Worker pass: for each local worker i, z_i = (beta1 m + (1-beta1) g_i) + delta_i,
// sign words of z_i, per-tile partial sum of z_i^2, and z_i written back as the
// new compensated error state.
//
// Packed momentum (every step after the first): a workgroup takes one item,
// one block of one worker's row, and the items run row by row, split into one
// contiguous eighth per XCD: the waves in flight on an XCD stream the same two
// rows (g_i and the error state of worker i).  The momentum of a block is
// re-derived by every worker, 1/8 byte per element per worker from a sign
// array small enough to stay in the last-level cache.
//
// What bounds it is HBM, and how close it comes depends on the bytes of loads
// that each SIMD keeps in flight: about 15 KB is best (fewer leave the memory
// idle, more make its read and write streams interfere).  With every load
// issued before the block's record arrives, a wave has its loads in flight
// nearly all its life, so the parts of a block are sized for that: fp32
// gradients take one sub-block per wave (2 KB of loads, 8 waves per SIMD),
// 16-bit ones two (3 KB) at 5 waves per SIMD, held there by unused LDS.  Step
// of the BERT-Base shape, n = 16, one process, same buffers, fp32 / bf16
// gradients, in ms (two dependent loads before the rows' loads, before:
// 3.641 / 3.124): one sub-block per wave at 8, 7, 6, 5 waves 3.531, 3.540,
// 3.774, 4.663 / 3.171, 3.401, 3.717, 4.908; two at 8, 7, 6, 5, 4, 3 waves
// 3.666, 3.645, 3.589, 3.556, 3.542, 3.781 / 3.128, 3.097, 3.041, 3.033,
// 3.095, 3.704; four at 8, 3, 2 waves 3.727, 3.574, 3.541 / 3.222, 3.038,
// 3.218.
//
// An fp32 momentum (the first compression step) is read once per block for all
// local workers instead, by k_worker_rows, where that pays (packed_grid).
// ---------------------------------------------------------------------------
// Unused dynamic LDS that lets `groups` workgroups of a kernel onto a CU at
// once (160 KB of LDS, allocated in steps of 512 bytes or less).
constexpr int idle_lds(int groups) { return 160 * 1024 / groups / 512 * 512; }

// The packed pass: sub-blocks per wave, waves per workgroup (one block), and
// the unused LDS that holds the occupancy at 5 waves per SIMD (160 KB of LDS
// for 10 workgroups of two waves on a CU's four SIMDs), see above.
template <class G>
constexpr int kPassSubBlocks = sizeof(typename G::T) == 2 ? 2 : 1;
template <class G>
constexpr int kPassWaves = kSubBlocks / kPassSubBlocks<G>;
template <class G>
constexpr int kPassIdleLds = sizeof(typename G::T) == 2 ? idle_lds(10) - 512 : 0;

// A wave's loads of its part of one block: the gradient row, the compensated
// row and the momentum (sign words, or fp32 values).
template <bool INSIDE, bool PACKED, class G, int SB, int CACHE>
__device__ __forceinline__ void worker_load(v4f (&gv)[SB], v4f (&cv)[SB], v4f (&mv)[SB],
                                            uint64_t (&word)[SB],
                                            const typename G::T *__restrict__ gi,
                                            const float *__restrict__ ei,
                                            const float *__restrict__ m,
                                            const uint64_t *__restrict__ m_bits, int sb0, int lane,
                                            int lim)
{
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        const int li = (sb0 + b) * (kWave * 4) + 4 * lane;
        word[b] = 0;
        if (PACKED) {
            if (INSIDE || li < lim) word[b] = m_bits[li >> 6];
        } else {
            mv[b] = ldb4<INSIDE>(m, li, lim);
        }
        gv[b] = ldgb4<INSIDE, G, CACHE == 2 ? kCachedLoad : kStreamLoad>(gi, li, lim);
        cv[b] = ldb4<INSIDE>(ei, li, lim);
    }
}

// The wave's sum (wave_sum's) of each of SB values per lane, to sums[0 .. SB).
// Two values share the exchanges: the first one leaves each half of the wave
// with one value to go on with.
template <int SB>
__device__ __forceinline__ void store_wave_sums(const double (&a)[SB], double *sums, int lane)
{
    static_assert(SB == 1 || SB == 2, "");
    if (SB == 1) {
        const double s = wave_sum(a[0]);
        if (lane == 0) sums[0] = s;
        return;
    }
    const bool upper = lane >= kWave / 2;
    double s = (upper ? a[SB - 1] : a[0]) + __shfl_xor(upper ? a[0] : a[SB - 1], kWave / 2, kWave);
#pragma unroll
    for (int off = kWave / 4; off >= 1; off >>= 1) s += __shfl_xor(s, off, kWave);
    if ((lane & (kWave / 2 - 1)) == 0) sums[lane / (kWave / 2)] = s;
}

// The arithmetic and stores of this wave's sub-blocks of one block of a
// worker's row: z = (beta1 m + (1 - beta1) g) + delta from the momentum term
// bm = beta1 m, the gradient and the previous compensated value with its scale
// sp; the new compensated value and the sign words are stored.  sums (the
// block's area in LDS) gets this wave's part of the sums of z^2: one per
// sub-block (WHOLE) or one per word, so that the tiles' sums do not depend on
// how many sub-blocks a wave takes.
template <bool WHOLE, int SB, bool CACHED = false>
__device__ __forceinline__ void worker_compute(const float (&sp)[SB], const int (&valid)[SB],
                                                 const v4f (&bm)[SB], const v4f (&gv)[SB],
                                                 const v4f (&cv)[SB], float *__restrict__ ei,
                                                 uint64_t *__restrict__ bi, int sb0, int lane,
                                                 int lim, float omb1, double *sums)
{
    double acc[SB];
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        const int li = (sb0 + b) * (kWave * 4) + 4 * lane;
        v4f zv;
        uint32_t nib = 0;
        acc[b] = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float d = error_of(cv[b][c], sp[b]);
            float mi = omb1 * gv[b][c];
            mi = bm[b][c] + mi;
            const float z = mi + d;
            zv[c] = z;
            const bool in = WHOLE || c < valid[b];
            const double zd = in ? (double)z : 0.0;
            acc[b] += zd * zd;
            nib |= (in && z >= 0.f) ? (1u << c) : 0u;
        }
        stb4<WHOLE, CACHED>(ei, li, valid[b], zv);
        const uint64_t out = row_sign_word(nib, lane);
        const int w = 4 * (sb0 + b) + (lane >> 4);
        if ((lane & 15) == 0 && (WHOLE || li < lim)) bi[w] = out;
        if (!WHOLE) {
            const double row = row_sum(acc[b]);
            if ((lane & 15) == 0) sums[w] = row;
        }
    }
    if (WHOLE) store_wave_sums(acc, sums + sb0, lane);
}

// The block's partial sums (one per tile) from its sub-blocks' sums (WHOLE) or
// its words' sums, by the lanes of one wave.
template <bool WHOLE>
__device__ __forceinline__ void block_partials(double *__restrict__ partial, const Block &rec,
                                               const double *sums, int lane)
{
    if (WHOLE) {
        if (lane == 0) partial[rec.tile] = ((sums[0] + sums[1]) + sums[2]) + sums[3];
    } else if (lane < __popc(rec.starts)) {
        partial[rec.tile + lane] = block_tile_sum(sums, rec.starts, lane);
    }
}

// One block of a worker's row (this wave's sub-blocks) from its loaded values.
// Every wave of the workgroup has the same block, so all reach the barrier.
template <bool WHOLE, bool PACKED, int SB, bool CACHED>
__device__ __forceinline__ void worker_block(
    double (&red)[kTileWords], const Tile *__restrict__ tiles, const Block &rec, int64_t base,
    int lim, int lane, int wv, const v4f (&mv)[SB], const uint64_t (&word)[SB], float s0,
    float ms0, const float *__restrict__ m_scales, const v4f (&gv)[SB], const v4f (&cv)[SB],
    const float *__restrict__ scales, float *__restrict__ ei, uint64_t *__restrict__ bi,
    double *__restrict__ partial, float beta1, float omb1)
{
    const int sb0 = wv * SB;
    // the scales of each sub-block's elements, one segment for a whole block
    float sp[SB];
    v4f bm[SB];
    int valid[SB];
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        float bs = PACKED ? beta1 * ms0 : 0.f;
        sp[b] = s0;
        valid[b] = 4;
        if (!WHOLE) {
            const int li = (sb0 + b) * (kWave * 4) + 4 * lane;
            valid[b] = 0;
            if (li < lim) {
                const Tile t = block_word_tile(tiles, rec, li >> 6);
                valid[b] = tile_valid4(t, base + li);
                sp[b] = scales[t.seg];
                if (PACKED) bs = beta1 * m_scales[t.seg];
            }
        }
        const uint32_t mnib = (uint32_t)(word[b] >> (4 * (lane & 15)));
#pragma unroll
        for (int c = 0; c < 4; ++c) bm[b][c] = PACKED ? with_sign(bs, mnib, c) : beta1 * mv[b][c];
    }
    worker_compute<WHOLE, SB, CACHED>(sp, valid, bm, gv, cv, ei, bi, sb0, lane, lim, omb1, red);
    __syncthreads();
    if (wv == 0) block_partials<WHOLE>(partial, rec, red, lane);
}

// PACKED: m_{t-1} is the previous step's gathered server message, decoded
// from its sign words and segment scale (+-scale, exactly the fp32 value the
// update would have stored), so no fp32 momentum buffer is read.  CACHE: see
// row_caching.
template <bool PACKED, class G, int CACHE>
__global__ __launch_bounds__(kWave *kPassWaves<G>) void k_worker_pass(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t num_blocks,
    FastDiv by_blocks, int64_t padded_len, int64_t num_tiles, const float *__restrict__ m,
    const uint64_t *__restrict__ m_bits, const float *__restrict__ m_scales,
    const typename G::T *__restrict__ g, int64_t g_ld, float *__restrict__ err, int64_t err_ld,
    const float *__restrict__ scales, int64_t scales_ld, uint64_t *__restrict__ bits,
    int64_t bits_ld, double *__restrict__ partial, int64_t item_base, int64_t num_items,
    float beta1, float omb1)
{
    constexpr int SB = kPassSubBlocks<G>;
    __shared__ double red[kTileWords];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x >> 6;
    // each XCD takes one contiguous eighth of the launch's items, one per workgroup
    const int64_t at = xcd_block();
    if (at >= num_items) return;  // the whole workgroup
    const int64_t item = item_base + at;
    const int64_t i = fast_quotient(item, by_blocks);
    const int64_t blk = item - i * num_blocks;
    const int64_t base = blk * kTileElems;
    const int64_t room = padded_len - base;
    const int lim = room < kTileElems ? (int)room : kTileElems;
    const typename G::T *gi = g + i * g_ld + base;
    float *ei = err + i * err_ld + base;
    v4f gv[SB], cv[SB], mv[SB];
    uint64_t word[SB];
    if (lim == kTileElems)
        worker_load<true, PACKED, G, SB, CACHE>(gv, cv, mv, word, gi, ei, m + base,
                                                m_bits + (base >> 6), wv * SB, lane, lim);
    else
        worker_load<false, PACKED, G, SB, CACHE>(gv, cv, mv, word, gi, ei, m + base,
                                                 m_bits + (base >> 6), wv * SB, lane, lim);
    const Block rec = load_block(blocks, blk);
    scales += i * scales_ld;
    // read here, before the branch, so that they travel with the rows
    const float s0 = scales[rec.seg];
    const float ms0 = PACKED ? m_scales[rec.seg] : 0.f;
    uint64_t *bi = bits + i * bits_ld + (base >> 6);
    if (rec.whole)
        worker_block<true, PACKED, SB, (CACHE > 0)>(red, tiles, rec, base, lim, lane, wv, mv, word,
                                                    s0, ms0, m_scales, gv, cv, scales, ei, bi,
                                                    partial + i * num_tiles, beta1, omb1);
    else
        worker_block<false, PACKED, SB, (CACHE > 0)>(red, tiles, rec, base, lim, lane, wv, mv, word,
                                                     s0, ms0, m_scales, gv, cv, scales, ei, bi,
                                                     partial + i * num_tiles, beta1, omb1);
}

// ---------------------------------------------------------------------------
// The worker pass with an fp32 momentum (the first compression step): m is
// read once per block for all local workers, and the 16 waves of a workgroup
// walk the worker rows together (one barrier per row), as in the warm-up.
// The waves of a block leave their sums of row i in red[i & 1]; after the
// barrier its first wave adds them and writes the partial sums.  red[i & 1] is
// written again only after the next barrier, by which time that read is done.
//
// Two sub-blocks per wave and one workgroup per CU keep 16 KB of loads in
// flight per SIMD, in runs of 32 KB per row.  Step with an fp32 momentum of the
// BERT-Base shape, n = 16, one process, same buffers: 4.37 ms with each row's
// loads issued before the previous row's stores (two rows in flight), 4.21 ms
// without; one sub-block per wave 4.35, four 4.32, workgroups of 8 waves
// 4.54, of 4 (one sub-block) 4.68, two workgroups per CU 4.45, the packed pass
// reading m for every worker 4.80.  The kernel's attribute allocates enough
// registers that a second workgroup does not fit, whatever the code needs.
// ---------------------------------------------------------------------------
constexpr int kWalkParts = kWorkerWavesPerBlock;          // waves per block
constexpr int kWalkSubBlocks = kSubBlocks / kWalkParts;   // sub-blocks per wave
constexpr int kWalkWaves = kRowWaves;
constexpr int kWalkBlocks = kWorkerRowTiles;              // blocks per workgroup
static_assert(kWalkBlocks * kWalkParts == kWalkWaves, "whole blocks");

template <bool WHOLE, class G>
__device__ __forceinline__ void worker_rows_walk(
    double (&red)[2][kWalkBlocks][kTileWords], const Tile *__restrict__ tiles, const Block &rec,
    int64_t base, int lim, int sb0, int lane, int wb, bool active,
    const v4f (&bm)[kWalkSubBlocks], const typename G::T *__restrict__ g, int64_t g_ld,
    float *__restrict__ err, int64_t err_ld, const float *__restrict__ scales, int64_t scales_ld,
    uint64_t *__restrict__ bits, int64_t bits_ld, double *__restrict__ partial, int64_t num_tiles,
    int n_local, float omb1)
{
    constexpr int SB = kWalkSubBlocks;
    int seg[SB], valid[SB];
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        seg[b] = rec.seg;
        valid[b] = 4;
        if (!WHOLE) {
            const int li = (sb0 + b) * (kWave * 4) + 4 * lane;
            valid[b] = 0;
            if (active && li < lim) {
                const Tile t = block_word_tile(tiles, rec, li >> 6);
                seg[b] = t.seg;
                valid[b] = tile_valid4(t, base + li);
            }
        }
    }
    g += base;
    err += base;
    bits += base >> 6;
    const auto load = [&](int64_t i, v4f(&gv)[SB], v4f(&cv)[SB], float(&sp)[SB]) {
        if (!active) return;
#pragma unroll
        for (int b = 0; b < SB; ++b) {
            const int li = (sb0 + b) * (kWave * 4) + 4 * lane;
            gv[b] = ldgb4<WHOLE, G>(g + i * g_ld, li, lim);
            cv[b] = ldb4<WHOLE>(err + i * err_ld, li, lim);
            sp[b] = scales[i * scales_ld + seg[b]];
        }
    };
    const auto finish = [&](int64_t i, const v4f(&gv)[SB], const v4f(&cv)[SB],
                            const float(&sp)[SB]) {
        double *sums = red[i & 1][wb];
        if (active)
            worker_compute<WHOLE, SB>(sp, valid, bm, gv, cv, err + i * err_ld, bits + i * bits_ld,
                                      sb0, lane, lim, omb1, sums);
        __syncthreads();  // and the workgroup moves to the next row together
        if (active && sb0 == 0)
            block_partials<WHOLE>(partial + i * num_tiles, rec, sums, lane);
    };
    for (int i = 0; i < n_local; ++i) {
        v4f ga[SB], ca[SB];
        float sa[SB];
        load(i, ga, ca, sa);
        finish(i, ga, ca, sa);
    }
}

template <class G>
__global__ __launch_bounds__(kWalkWaves *kWave)
    __attribute__((amdgpu_waves_per_eu(kWalkWaves / 4, kWalkWaves / 4))) void k_worker_rows(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t block_base,
    int64_t num_blocks, int64_t padded_len, int64_t num_tiles, const float *__restrict__ m,
    const typename G::T *__restrict__ g, int64_t g_ld, float *__restrict__ err, int64_t err_ld,
    const float *__restrict__ scales, int64_t scales_ld, uint64_t *__restrict__ bits,
    int64_t bits_ld, double *__restrict__ partial, int n_local, float beta1, float omb1)
{
    constexpr int SB = kWalkSubBlocks;
    __shared__ double red[2][kWalkBlocks][kTileWords];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_id();
    const int wb = wv / kWalkParts;
    const int sb0 = wv % kWalkParts * SB;
    const int64_t blk = block_base + xcd_block() * kWalkBlocks + wb;
    const bool active = blk < num_blocks;
    const int64_t base = blk * kTileElems;
    const int64_t room = padded_len - base;
    const int lim = room < kTileElems ? (int)room : kTileElems;
    Block rec{0, 0, 0, 0};
    v4f bm[SB];
    if (active) {
        rec = load_block(blocks, blk);
#pragma unroll
        for (int b = 0; b < SB; ++b)
            bm[b] = beta1 * ldb4<false>(m + base, (sb0 + b) * (kWave * 4) + 4 * lane, lim);
    }
    if (rec.whole)
        worker_rows_walk<true, G>(red, tiles, rec, base, lim, sb0, lane, wb, true, bm, g, g_ld,
                                  err, err_ld, scales, scales_ld, bits, bits_ld, partial,
                                  num_tiles, n_local, omb1);
    else
        worker_rows_walk<false, G>(red, tiles, rec, base, lim, sb0, lane, wb, active, bm, g, g_ld,
                                   err, err_ld, scales, scales_ld, bits, bits_ld, partial,
                                   num_tiles, n_local, omb1);
}

// ---------------------------------------------------------------------------
// Scale finalize: scale = fp32(sqrt(sum over the segment's tiles / len)); empty
// segments get 0.  The order of the sum is the plan's (segment_sum's, or a
// workgroup's where a segment has more than 256 tiles), so a scale depends
// neither on scheduling nor on the rows or owners of a call.  LANES lanes
// cooperate on one segment of one row, fewer for
// segments of few tiles (launch_finalize): with a wave for each, the 2 million
// (row, segment) pairs of 2,000 tensors of 64 to 8192 elements with n = 32
// took 470 us of a 900 us step, which is 422 us with a lane for each; the
// 5,000-tensor workload's step went from 10.05 to 9.98 ms with 16 lanes.
// ---------------------------------------------------------------------------
// The sum by a whole workgroup.
__device__ __forceinline__ double block_segment_sum(const double *__restrict__ part, int tiles,
                                                    double *red)
{
    const int tid = threadIdx.x;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int t = tid;
    for (; t + 3 * kBlock < tiles; t += 4 * kBlock) {
        s0 += part[t];
        s1 += part[t + kBlock];
        s2 += part[t + 2 * kBlock];
        s3 += part[t + 3 * kBlock];
    }
    for (; t < tiles; t += kBlock) s0 += part[t];
    const double s = wave_sum((s0 + s1) + (s2 + s3));
    if ((tid & (kWave - 1)) == 0) red[tid / kWave] = s;
    __syncthreads();
    return ((red[0] + red[1]) + red[2]) + red[3];
}

template <int LANES, int MAX>
__device__ __forceinline__ float finalize_one(const double *__restrict__ part, const Segment &seg,
                                              double *red)
{
    double s;
    if constexpr (LANES > kWave)
        s = block_segment_sum(part + seg.tile, seg.tiles, red);
    else
        s = segment_sum<LANES, MAX>(part + seg.tile, seg.tiles, threadIdx.x % LANES);
    return seg.len > 0 ? scale_of(s, seg.len) : 0.0f;
}

// count segments per row; cnt = 0: segment p is the p-th, else (server form)
// segments k*n + j for j in [jb, jb + cnt) and every tensor k, in that order.
// No segment has more than MAX tiles (if LANES is at most a wave).
template <int LANES, int MAX>
__global__ __launch_bounds__(kBlock) void k_finalize(const Segment *__restrict__ segs,
                                                     uint32_t count, int64_t rows, int n, int jb,
                                                     int cnt, const double *__restrict__ partial,
                                                     int64_t part_ld, float *__restrict__ scales,
                                                     int64_t scales_ld)
{
    __shared__ double red[kBlock / kWave];
    // LANES lanes per segment; the grid may be smaller than the rows or the
    // segments, so each group of lanes strides over both (uniform per block
    // or per wave where it has to be)
    constexpr uint32_t kPer = kBlock / LANES;
    for (int64_t i = blockIdx.y; i < rows; i += gridDim.y) {
        for (uint32_t p = blockIdx.x * kPer + threadIdx.x / LANES; p < count;
             p += gridDim.x * kPer) {
            const uint32_t q = cnt == 0 || cnt == n
                                   ? p
                                   : p / (uint32_t)cnt * (uint32_t)n + jb + p % (uint32_t)cnt;
            const float s = finalize_one<LANES, MAX>(partial + i * part_ld, segs[q], red);
            if (threadIdx.x % LANES == 0) scales[i * scales_ld + q] = s;
            if (LANES > kWave) __syncthreads();  // red is reused by the next segment
        }
    }
}

// ---------------------------------------------------------------------------
// Server pass over the tiles of the owned chunks: decode and average the n
// incoming messages, add the server error, write the sign words and the new
// compensated server state, and the tile's sum of squares.
//
// Each wave owns its own LDS region, so it synchronises only with itself (no
// workgroup barrier); a tile's error-state loads are issued first so that
// they overlap the sign-word traffic.  Incoming sign words are
// staged in LDS 32 worker rows at a time (coalesced 128-byte row reads),
// transposed so that the words of consecutive workers for one 32-element
// half-word are adjacent.  For the table lookups each group of 8 workers is
// then regrouped in place, four 8x8 bit transposes per (half-word, group):
// afterwards each LDS byte holds the 8 workers' bits of one element, the
// element's table index.
//
// The average is an fp64 sum of +-scale over the workers in worker order.
// When every partial sum of the segment's scales is exactly representable in
// fp64 (the scales' exponents span at most 29 - ceil(log2 n) binades; true
// for any realistic message set) the sum is exact, so it may be formed in any
// grouping: then each group of 8 workers is one lookup in a 256-entry table
// of its signed scale sums, indexed by the 8 workers' bits of the element.
// The 256-entry tables are sums of two 16-entry tables, each built from 4
// scales; they depend on the segment's scales only.  Otherwise every worker
// is added one by one.  Both give the oracle's sum.
// ---------------------------------------------------------------------------
// Wave-wide max of an int through DPP: shifts within each 16-lane row, then
// row broadcasts carry the row maxima up to lane 63, which every lane reads.
__device__ __forceinline__ int wave_max(int v)
{
    constexpr int lo = INT32_MIN;
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x111, 0xF, 0xF, false));  // row_shr 1
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x112, 0xF, 0xF, false));  // row_shr 2
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x114, 0xF, 0xF, false));  // row_shr 4
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x118, 0xF, 0xF, false));  // row_shr 8
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x142, 0xA, 0xF, false));  // row_bcast 15
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x143, 0xC, 0xF, false));  // row_bcast 31
    return __builtin_amdgcn_readlane(v, kWave - 1);
}

__device__ __forceinline__ int wave_min(int v) { return -wave_max(-v); }

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One sub-block (256 elements) of the server pass's last part: average, add
// the server error, store the new compensated error state and the sign words;
// returns this wave's fp64 sum of squares of the sub-block (every lane gets
// it).  sum[c] and cv[c] are the lane's elements b*256 + 4*lane + c.
template <bool FULL, bool POW2>
__device__ __forceinline__ double server_epilogue_sub(const double (&sum)[4], v4f cv,
                                                      float sprev, int n, int lane,
                                                      const Tile &tile, int b,
                                                      float *__restrict__ serr,
                                                      uint64_t *__restrict__ sbits)
{
    const int len = tile.len;
    const int64_t base = tile.start;
    const int nwords = (len + 63) >> 6;
    const double dn = (double)n;
    const double inv_n = 1.0 / dn;
    const int li = b * (kWave * 4) + 4 * lane;
    double acc = 0.0;
    v4f zv;
    uint32_t nib = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        // avg = sum / n rounded to fp32 (for a power-of-two n, sum * (1/n) is
        // the same exact scaling), then the compensated value and its square
        const float avg = (float)(POW2 ? sum[c] * inv_n : sum[c] / dn);
        const float z = avg + error_of(cv[c], sprev);
        zv[c] = z;
        const bool valid = FULL || li + c < len;
        const double zd = valid ? (double)z : 0.0;
        // zd * zd is exact in fp64 (a 24-bit significand squared), so the
        // fused form rounds exactly as the separate multiply and add would
        acc = __builtin_fma(zd, zd, acc);
        nib |= (valid && z >= 0.f) ? (1u << c) : 0u;
    }
    st4<FULL>(serr + base, li, len, zv);
    const uint64_t word = row_sign_word(nib, lane);
    const int w = 4 * b + (lane >> 4);
    if ((lane & 15) == 0 && (FULL || w < nwords)) sbits[(base >> 6) + w] = word;
    return acc;
}

// LDS row stride (in 32-bit words) of the sign staging: a multiple of 4 keeps
// 128-bit accesses aligned, and 40 puts the 64 words a wave reads at once in
// the accumulation on 64 different banks.
constexpr int kBitsStride = kServerRowBatch + 8;

// One wave's LDS working set for a batch of up to kServerRowBatch incoming
// rows of one tile: the sign words, transposed ([half-word h][row r]), the
// rows' scales, and the lookup tables built from them (the 256-entry tables
// of two groups of 8 rows at a time).
struct ServerBatchLds {
    uint32_t bits[2 * kTileWords][kBitsStride];
    double lut4[kServerRowBatch / 4][16];
    double lut8[2][256];
    float scale[kServerRowBatch];
};

// One wave's LDS working set in the one-wave-per-tile pass (n <= 8 G8 <=
// kServerRowBatch): the 256-entry tables of all G8 groups of 8 rows, held at
// once, are built from the 16-entry tables before the tile's words are staged
// (so those share the staging area).  G8 follows n, so that smaller n leave
// room for more workgroups per CU.
template <int G8>
struct ServerTileLds {
    union {
        uint32_t bits[2 * kTileWords][kBitsStride];
        double lut4[kServerRowBatch / 4][16];
    };
    double lut8[G8][256];
    float scale[kServerRowBatch];
};

// 8x8 bit transposes of the four byte columns of 8 words: bit j of byte b of
// a[k] moves to bit k of byte b of a[j] (three rounds of block swaps: 4x4,
// 2x2, 1x1 bits, each on all four bytes at once).
__device__ __forceinline__ void transpose_bits8x8(uint32_t (&a)[8])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t t = ((a[k] >> 4) ^ a[k + 4]) & 0x0F0F0F0Fu;
        a[k] ^= t << 4;
        a[k + 4] ^= t;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = (i & 1) + 4 * (i >> 1);  // 0, 1, 4, 5
        const uint32_t t = ((a[k] >> 2) ^ a[k + 2]) & 0x33333333u;
        a[k] ^= t << 2;
        a[k + 2] ^= t;
    }
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
        const uint32_t t = ((a[k] >> 1) ^ a[k + 1]) & 0x55555555u;
        a[k] ^= t << 1;
        a[k + 1] ^= t;
    }
}

// The incoming sign words and scales of one tile as the chunk owner reads
// them: row i's word for tile word wi is at words[i * bits_ld + wi], its
// scale at scales[i * scales_ld].
struct ServerRows {
    const uint64_t *words;   // the tile's first word in row 0
    int64_t bits_ld;
    const float *scales;     // the segment's scale in row 0
    int64_t scales_ld;
    int nwords;              // words of the tile
    bool full;               // a full tile
};

// Loads the words of rows [r0, r0 + rows) of the tile (rows <=
// kServerRowBatch): lane L takes word wi = L % 16 of rows r0 + L/16 + 4k.
__device__ __forceinline__ void server_load_words(const ServerRows &in, int r0, int rows,
                                                  int lane, uint64_t (&stg)[kServerRowBatch / 4])
{
    const int wi = lane & (kTileWords - 1);
    const uint64_t *p = in.words + (int64_t)(r0 + (lane >> 4)) * in.bits_ld + wi;
    const int64_t step = 4 * in.bits_ld;
    if (in.full && rows == kServerRowBatch) {  // wave-uniform: every load in range
#pragma unroll
        for (int k = 0; k < kServerRowBatch / 4; ++k) stg[k] = __builtin_nontemporal_load(p + k * step);
    } else {
#pragma unroll
        for (int k = 0; k < kServerRowBatch / 4; ++k) {
            const int r = (lane >> 4) + 4 * k;
            stg[k] = (r < rows && wi < in.nwords) ? __builtin_nontemporal_load(p + k * step) : 0ull;
        }
    }
}

// The words of rows [r0, r0 + rows) and the scale of row r0 + lane.
__device__ __forceinline__ void server_load_batch(const ServerRows &in, int r0, int rows,
                                                  int lane, uint64_t (&stg)[kServerRowBatch / 4],
                                                  float &scl)
{
    server_load_words(in, r0, rows, lane, stg);
    scl = lane < rows ? in.scales[(int64_t)(r0 + lane) * in.scales_ld] : 0.f;
}

// Writes loaded words into the wave's staging area (rows past the batch's
// last row, up to the next multiple of 8, get zero words).
template <class Lds>
__device__ __forceinline__ void server_stage_words(Lds &L, const ServerRows &in, int rows,
                                                   int lane,
                                                   const uint64_t (&stg)[kServerRowBatch / 4])
{
    const int wi = lane & (kTileWords - 1);
    const int rows8 = (rows + 7) & ~7;
    if (in.full && rows == kServerRowBatch) {  // wave-uniform
#pragma unroll
        for (int k = 0; k < kServerRowBatch / 4; ++k) {
            const int r = (lane >> 4) + 4 * k;
            L.bits[2 * wi][r] = (uint32_t)stg[k];
            L.bits[2 * wi + 1][r] = (uint32_t)(stg[k] >> 32);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kServerRowBatch / 4; ++k) {
            const int r = (lane >> 4) + 4 * k;
            if (r < rows8 && wi < in.nwords) {
                L.bits[2 * wi][r] = (uint32_t)stg[k];
                L.bits[2 * wi + 1][r] = (uint32_t)(stg[k] >> 32);
            }
        }
    }
}

// Stages a loaded batch: its words, and the scale of row `lane`.
template <class Lds>
__device__ __forceinline__ void server_stage_batch(Lds &L, const ServerRows &in,
                                                   int rows, int lane,
                                                   const uint64_t (&stg)[kServerRowBatch / 4],
                                                   float scl)
{
    server_stage_words(L, in, rows, lane, stg);
    if (lane < rows) L.scale[lane] = scl;
}

// The 16-entry tables of 4 rows, two per group of 8 (rows past the last row
// add 0): lut4[q][idx] is the sum over k < 4 of +-scale[4q + k], + where bit
// k of idx is set.
template <class Lds>
__device__ __forceinline__ void server_build_lut4(Lds &L, int rows, int lane)
{
    const int groups8 = (rows + 7) >> 3;
    for (int e = lane; e < 32 * groups8; e += kWave) {
        const int q = e >> 4, idx = e & 15;
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int r = 4 * q + k;
            if (r < rows) {
                const double sc = (double)L.scale[r];
                v += ((idx >> k) & 1) ? sc : -sc;
            }
        }
        L.lut4[q][idx] = v;
    }
}

// Regroups each staged (half-word, group of 8 rows) block in place by four
// 8x8 bit transposes, after which byte e>>3 of word r8 + (e&7) of the block is
// element e's table index (the 8 rows' bits of e).
template <class Lds>
__device__ __forceinline__ void server_regroup_bits(Lds &L, int rows, int lane)
{
    const int groups8 = (rows + 7) >> 3;
#pragma unroll 1
    for (int k = 0; k < (2 * kTileWords) * (kServerRowBatch / 8) / kWave; ++k) {
        const int blk = lane + kWave * k;
        const int hwb = blk & (2 * kTileWords - 1), gb = blk / (2 * kTileWords);
        if (gb < groups8) {
            uint32_t *p = &L.bits[hwb][8 * gb];
            const uint4 u0 = *(const uint4 *)p;
            const uint4 u1 = *(const uint4 *)(p + 4);
            uint32_t a[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
            transpose_bits8x8(a);
            *(uint4 *)p = make_uint4(a[0], a[1], a[2], a[3]);
            *(uint4 *)(p + 4) = make_uint4(a[4], a[5], a[6], a[7]);
        }
    }
}

// sum += the group of 8 rows starting at row r8, one lookup per element in
// its 256-entry table lut (regrouped words).  Two sub-blocks at a time: their
// 8 table indices first, then the 8 lookups, then the adds, so that the LDS
// round trips overlap.
template <class Lds>
__device__ __forceinline__ void server_lookup_group(double (&sum)[kSubBlocks][4], const Lds &L,
                                                    int r8, const double *lut, int lane)
{
    const int half = (lane >> 3) & 1;
#pragma unroll
    for (int bh = 0; bh < kSubBlocks; bh += 2) {
        uint32_t idx[2][4];
#pragma unroll
        for (int bb = 0; bb < 2; ++bb) {
            const int hw = 2 * (4 * (bh + bb) + (lane >> 4)) + half;
            // the lane's elements e = 4 (lane & 7) + c of the half-word:
            // byte e >> 3 of word e & 7 holds the 8 rows' bits of e
            const uint8_t *blk = (const uint8_t *)&L.bits[hw][r8];
            const int o = 16 * (lane & 1) + ((lane & 7) >> 1);
#pragma unroll
            for (int c = 0; c < 4; ++c) idx[bb][c] = blk[o + 4 * c];
        }
        double val[2][4];
#pragma unroll
        for (int bb = 0; bb < 2; ++bb)
#pragma unroll
            for (int c = 0; c < 4; ++c) val[bb][c] = lut[idx[bb][c]];
#pragma unroll
        for (int bb = 0; bb < 2; ++bb)
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[bh + bb][c] += val[bb][c];
    }
}

// sum += the staged batch's decoded messages, grouped: each group of 8 rows is
// one lookup in a 256-entry table of its signed scale sums (exact, so any
// grouping gives the worker-order sum).  The 16-entry tables of 4 rows are
// built first, then the staged words are regrouped; the 256-entry tables are
// built two groups at a time.
__device__ __forceinline__ void server_batch_grouped(double (&sum)[kSubBlocks][4],
                                                     ServerBatchLds &L, int rows, int lane)
{
    const int groups8 = (rows + 7) >> 3;
    server_build_lut4(L, rows, lane);
    server_regroup_bits(L, rows, lane);
    wave_sync();
    for (int g0 = 0; 8 * g0 < rows; g0 += 2) {
        const int gcnt = min(2, groups8 - g0);
#pragma unroll
        for (int k = 0; k < 512 / kWave; ++k) {
            const int e = lane + kWave * k;
            const int g = e >> 8, idx = e & 255;  // g = k / 4: uniform
            if (g < gcnt) {
                const int q = 2 * (g0 + g);
                L.lut8[g][idx] = L.lut4[q][idx & 15] + L.lut4[q + 1][idx >> 4];
            }
        }
        wave_sync();
        for (int g = 0; g < gcnt; ++g) server_lookup_group(sum, L, 8 * (g0 + g), L.lut8[g], lane);
        wave_sync();
    }
}

// sum += the staged batch's decoded messages one worker at a time, in row
// order (the path for scale sets whose partial sums may round).
template <class Lds>
__device__ __forceinline__ void server_batch_one_by_one(double (&sum)[kSubBlocks][4],
                                                        const Lds &L, int rows, int lane)
{
    const int half = (lane >> 3) & 1;
    const int shift = 4 * (lane & 7);
    for (int r = 0; r < rows; ++r) {
        const double sp = (double)L.scale[r];
        const double sn = -sp;
#pragma unroll
        for (int b = 0; b < kSubBlocks; ++b) {
            const uint32_t nib = (L.bits[2 * (4 * b + (lane >> 4)) + half][r] >> shift) & 0xFu;
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[b][c] += ((nib >> c) & 1u) ? sp : sn;
        }
    }
}

// Whether the segment's incoming scales allow the grouped sum: every partial
// sum of +-scales is exact in fp64 when the nonzero scales' exponents span at
// most grouping_limit = 29 - ceil(log2 n) binades (and none is Inf or NaN).
// `first` holds the scale of row `lane` when n <= kServerRowBatch (already
// loaded); otherwise all n scales are read.  Every lane gets the answer.
__device__ __forceinline__ bool server_grouped(const ServerRows &in, int n, int grouping_limit,
                                               int lane, float first)
{
    int emax = 0, emin = 1 << 20;
    auto widen = [&](float sc) {
        const uint32_t u = __float_as_uint(sc) & 0x7FFFFFFFu;
        if (u == 0) return;
        const int e = max((int)(u >> 23), 1);
        emax = max(emax, e);
        emin = min(emin, e);
    };
    if (n <= kServerRowBatch)
        widen(first);
    else
        for (int r = lane; r < n; r += kWave) widen(in.scales[(int64_t)r * in.scales_ld]);
    emax = wave_max(emax);
    emin = wave_min(emin);
    return emax < 255 && (emax == 0 || emax - emin <= grouping_limit);
}

// The last part of a tile for every sub-block: average, add the server error,
// store the new compensated error state and the sign words; returns the
// wave's fp64 sum of squares of the tile (every lane gets it).  FULL and POW2
// are wave-uniform, so each wave runs one variant.
__device__ __forceinline__ double server_epilogue(const double (&sum)[kSubBlocks][4],
                                                  const v4f (&cv)[kSubBlocks], float sprev, int n,
                                                  int lane, const Tile &tile, bool full,
                                                  float *__restrict__ serr,
                                                  uint64_t *__restrict__ sbits)
{
    const bool pow2 = (n & (n - 1)) == 0;
    double acc = 0.0;
#pragma unroll
    for (int b = 0; b < kSubBlocks; ++b) {
        if (full && pow2)
            acc += server_epilogue_sub<true, true>(sum[b], cv[b], sprev, n, lane, tile, b, serr, sbits);
        else if (full)
            acc += server_epilogue_sub<true, false>(sum[b], cv[b], sprev, n, lane, tile, b, serr, sbits);
        else if (pow2)
            acc += server_epilogue_sub<false, true>(sum[b], cv[b], sprev, n, lane, tile, b, serr, sbits);
        else
            acc += server_epilogue_sub<false, false>(sum[b], cv[b], sprev, n, lane, tile, b, serr, sbits);
    }
    return wave_sum_dpp(acc);
}

// ---------------------------------------------------------------------------
// Tables of the owned segments, built once per call when the caller's
// workspace holds them: for owned segment u (segment q = k*n + j of chunk j
// in [cb, cb + nown), u = k*nown + j - cb) flags[u] says whether the grouped
// sum applies, and if so tables[(u*groups8 + g)*256 + idx] is the signed sum
// of the scales of rows 8g .. 8g+7 (+ where bit k of idx is set; rows past n
// add nothing).  One workgroup per (owned segment, group); each decides on
// the segment's flag by itself, and group 0's writes it.  Every entry is an
// exact fp64 sum when the flag is set, so it equals the in-kernel tables'.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_server_tables(
    int n, int cb, int nown, int grouping_limit, const float *__restrict__ wscales,
    int64_t scales_ld, int64_t scales_seg_base, double *__restrict__ tables,
    int32_t *__restrict__ flags)
{
    const int groups8 = (n + 7) >> 3;
    const int64_t u = blockIdx.x / groups8;
    const int g = blockIdx.x - u * groups8;
    const int64_t q = (u / nown) * n + cb + (u % nown);
    const float *sc = wscales + (q - scales_seg_base);
    const int lane = threadIdx.x & (kWave - 1);
    const ServerRows in{nullptr, 0, sc, scales_ld, 0, false};
    // every wave reads the n scales and reaches the same decision
    const float first = (n <= kServerRowBatch && lane < n) ? sc[(int64_t)lane * scales_ld] : 0.f;
    const bool ok = server_grouped(in, n, grouping_limit, lane, first);
    if (g == 0 && threadIdx.x == 0) flags[u] = ok ? 1 : 0;
    if (!ok) return;
    static_assert(kBlock == 256, "one table entry per thread");
    const int idx = threadIdx.x;
    double v = 0.0;
    for (int k = 0; k < 8 && 8 * g + k < n; ++k) {
        const double s = (double)sc[(int64_t)(8 * g + k) * scales_ld];
        v += ((idx >> k) & 1) ? s : -s;
    }
    tables[((u * groups8) + g) * 256 + idx] = v;
}

// Where a call's owned-segment tables and flags are, for the passes that copy
// them (passed by value as a kernel argument).
struct ServerTables {
    const double *tables;
    const int32_t *flags;
    int cb;    // first owned chunk
    int nown;  // owned chunks
};

// Copies the 256-entry tables of groups [g0, g0 + gcnt) of owned segment u
// into lut (gcnt 2 KB tables) with direct global-to-LDS loads, 1 KB per
// instruction: lane L's 16 bytes land at byte 16 L of each kilobyte.  The
// caller waits for them (vmcnt) before reading lut.
__device__ __forceinline__ void server_fetch_tables(double *lut, const ServerTables &st,
                                                    int64_t u, int groups8, int g0, int gcnt,
                                                    int lane)
{
    const char *src = (const char *)(st.tables + (u * groups8 + g0) * 256) + 16 * lane;
    for (int k = 0; k < 2 * gcnt; ++k)
        __builtin_amdgcn_global_load_lds((const void *)(src + 1024 * k),
                                         (__attribute__((address_space(3))) void *)((char *)lut +
                                                                                    1024 * k),
                                         16, 0, 0);
}

// Owned segment index of segment q.
__device__ __forceinline__ int64_t owned_segment(int64_t q, int n, const ServerTables &st)
{
    const int64_t k = q / n;
    return k * st.nown + (q - k * n) - st.cb;
}

// Waits for every vector memory operation of the wave, the direct-to-LDS
// table loads included (the compiler does not track those): s_waitcnt with
// vmcnt 0 (bits 3:0 and 15:14) and the expcnt (6:4) and lgkmcnt (11:8) fields
// at their maxima, which wait for nothing.
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// ---------------------------------------------------------------------------
// Chunk owners' pass over blocks, every chunk owned: a workgroup takes one
// block, one sub-block per wave, and each lane adds the n decoded values of its
// 4 elements one by one in worker order (the oracle's sum whatever the scales),
// reading the byte that holds its 4 sign bits from each worker's row.  No LDS
// tables, no regrouping and no exactness check, so a short tile costs what its
// elements do, where a wave per tile builds its tables for 64 elements as for
// 1,024 (the caller's rule says from where on this pays).
// ---------------------------------------------------------------------------
constexpr int kDirectBatch = 8;  // workers whose sign bits are loaded together

// sum[c] += +-s by the lane's bit c of nib.
__device__ __forceinline__ void add_decoded(double (&sum)[4], float s, uint32_t nib)
{
    const double d = (double)s;
    const int lo = __double2loint(d);
    const uint32_t hi = (uint32_t)__double2hiint(d);
#pragma unroll
    for (int c = 0; c < 4; ++c)
        sum[c] += __hiloint2double((int)(hi ^ ((~nib << (31 - c)) & 0x80000000u)), lo);
}

// The sums of squares of the block's tiles from its lanes' sums (red[t]: thread
// t's 4 elements), in the order of the passes over tiles, so that a scale does
// not depend on which pass a call takes.  There lane L of a wave has the
// elements 4L .. 4L + 3 of each sub-block of its tile: for n <= kServerRowBatch
// it adds the sub-blocks' sums and the wave adds the lanes'; for more workers
// each sub-block's wave adds its lanes' and the four sums are added in pairs.
template <bool WHOLE>
__device__ __forceinline__ void server_direct_partials(const double (&red)[kBlock],
                                                       const Block &rec, int lim, int lane, int wv,
                                                       bool split, double *__restrict__ partial)
{
    uint32_t rest = WHOLE ? 1u : rec.starts;
    for (int j = 0; rest != 0; ++j) {
        const int w0 = __ffs(rest) - 1;
        rest &= rest - 1;
        if ((j & (kWavesPerBlock - 1)) != wv) continue;  // the waves take turns
        const int words = (WHOLE ? kTileWords : rest ? __ffs(rest) - 1 : lim >> 6) - w0;
        double a[kSubBlocks];
#pragma unroll
        for (int b = 0; b < kSubBlocks; ++b)
            a[b] = 4 * b + (lane >> 4) < words ? red[16 * (w0 + 4 * b) + lane] : 0.0;
        double s;
        if (split && words > 4) {
#pragma unroll
            for (int b = 0; b < kSubBlocks; ++b) a[b] = wave_sum_dpp(a[b]);
            s = (a[0] + a[1]) + (a[2] + a[3]);
        } else {
            s = wave_sum_dpp(((a[0] + a[1]) + a[2]) + a[3]);
        }
        if (lane == 0) partial[rec.tile + j] = s;
    }
}

template <bool WHOLE>
__device__ __forceinline__ void server_direct_block(
    double (&red)[kBlock], const Tile *__restrict__ tiles, const Block &rec, int64_t base,
    int lim, int lane, int wv, v4f cv, int n, const uint8_t *__restrict__ bytes,
    int64_t bytes_ld, uint32_t (&first)[kDirectBatch], const float *__restrict__ wscales,
    int64_t scales_ld, float *__restrict__ serr, float sprev,
    const float *__restrict__ sscales, uint64_t *__restrict__ sbits,
    double *__restrict__ partial)
{
    const int li = wv * (kWave * 4) + 4 * lane;
    const bool in = WHOLE || li < lim;
    int seg = rec.seg, valid = 4;
    if (!WHOLE) {
        valid = 0;
        if (in) {
            const Tile tile = block_word_tile(tiles, rec, li >> 6);
            seg = tile.seg;
            valid = tile_valid4(tile, base + li);
            sprev = sscales[seg];
        }
    }
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i0 = 0; i0 < n; i0 += kDirectBatch) {
        uint32_t cur[kDirectBatch];
#pragma unroll
        for (int k = 0; k < kDirectBatch; ++k) {
            cur[k] = first[k];
            const int i = i0 + kDirectBatch + k;
            if (i < n && in) first[k] = bytes[(int64_t)i * bytes_ld];
        }
#pragma unroll
        for (int k = 0; k < kDirectBatch; ++k) {
            const int i = i0 + k;
            if (i >= n) break;
            const float s = wscales[(int64_t)i * scales_ld + seg];
            add_decoded(sum, s, cur[k] >> (lane & 1 ? 4 : 0));
        }
    }
    const double dn = (double)n;
    const bool pow2 = (n & (n - 1)) == 0;
    const double inv_n = 1.0 / dn;
    double acc = 0.0;
    v4f zv;
    uint32_t nib = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        // for a power-of-two n, sum * (1/n) is the same exact scaling
        const float avg = (float)(pow2 ? sum[c] * inv_n : sum[c] / dn);
        const float z = avg + error_of(cv[c], sprev);
        zv[c] = z;
        const bool real = WHOLE || c < valid;
        const double zd = real ? (double)z : 0.0;
        acc = __builtin_fma(zd, zd, acc);  // zd * zd is exact in fp64
        nib |= (real && z >= 0.f) ? (1u << c) : 0u;
    }
    stb4<WHOLE>(serr, li, valid, zv);
    const uint64_t word = row_sign_word(nib, lane);
    if ((lane & 15) == 0 && in) sbits[li >> 6] = word;
    red[threadIdx.x] = acc;
    __syncthreads();
    server_direct_partials<WHOLE>(red, rec, lim, lane, wv, n > kServerRowBatch, partial);
}

__global__ __launch_bounds__(kBlock) void k_server_direct(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t block_base,
    int64_t num_blocks, int64_t padded_len, int n, const uint64_t *__restrict__ wbits,
    int64_t bits_ld, const float *__restrict__ wscales, int64_t scales_ld, float *__restrict__ serr, const float *__restrict__ sscales,
    uint64_t *__restrict__ sbits, double *__restrict__ partial)
{
    __shared__ double red[kBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_id();
    const int64_t blk = block_base + xcd_block();
    if (blk >= num_blocks) return;  // the whole workgroup
    const int64_t base = blk * kTileElems;
    const int64_t room = padded_len - base;
    const int lim = room < kTileElems ? (int)room : kTileElems;
    const int li = wv * (kWave * 4) + 4 * lane;
    serr += base;
    sbits += base >> 6;
    const uint8_t *bytes = (const uint8_t *)wbits + ((base + li) >> 3);
    const int64_t bytes_ld = bits_ld * 8;
    const v4f cv = lim == kTileElems ? ldb4<true>(serr, li, lim) : ldb4<false>(serr, li, lim);
    uint32_t first[kDirectBatch];
#pragma unroll
    for (int k = 0; k < kDirectBatch; ++k) {
        first[k] = 0;
        if (k < n && li < lim) first[k] = bytes[k * bytes_ld];
    }
    const Block rec = load_block(blocks, blk);
    const float sprev = sscales[rec.seg];
    if (rec.whole)
        server_direct_block<true>(red, tiles, rec, base, lim, lane, wv, cv, n, bytes, bytes_ld,
                                  first, wscales, scales_ld, serr, sprev, sscales, sbits, partial);
    else
        server_direct_block<false>(red, tiles, rec, base, lim, lane, wv, cv, n, bytes, bytes_ld,
                                   first, wscales, scales_ld, serr, sprev, sscales, sbits,
                                   partial);
}

// The sums of a segment's partial sums of n workers, n <= N (rows of part_ld),
// by one wave, in segment_sum's order: lane L gets worker L / (64 / N)'s (any
// value where that is n or more).  Up to 64 tiles the lanes of a worker add its
// tiles, in one, four or more loads each.  Beyond (at most kWaveSegTiles) the
// wave takes four workers at a time, every lane its strided sum of each; the
// first two exchanges also leave each 16 lanes with one worker to go on with.
template <int N>
__device__ __forceinline__ double worker_segment_sums(const double *__restrict__ part,
                                                      int64_t part_ld, int n, int tiles, int lane)
{
    constexpr int kPer = kWave / N;
    const int mine = lane / kPer;
    if (tiles <= kWave) {
        const double *row = part + min(mine, n - 1) * part_ld;
        if (tiles <= kPer) return segment_sum<kPer, kPer>(row, tiles, lane % kPer);
        if (4 * kPer < kWave && tiles <= 4 * kPer)
            return segment_sum<kPer, 4 * kPer>(row, tiles, lane % kPer);
        return segment_sum<kPer, kWave>(row, tiles, lane % kPer);
    }
    double sum = 0.0;
#pragma unroll 1
    for (int r0 = 0; r0 < n; r0 += 4) {
        double p[4][4], s[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int t = lane + kWave * k;
                p[r][k] = t < tiles ? part[min(r0 + r, n - 1) * part_ld + t] : 0.0;
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = (p[r][0] + p[r][1]) + (p[r][2] + p[r][3]);
#pragma unroll
        for (int keep = 2, off = kWave / 2; keep >= 1; keep /= 2, off /= 2) {
            const bool upper = (lane & off) != 0;
#pragma unroll
            for (int j = 0; j < keep; ++j) {
                const double give = upper ? s[j] : s[j + keep];
                s[j] = (upper ? s[j + keep] : s[j]) + __shfl_xor(give, off, kWave);
            }
        }
        const double four = row_sum(s[0]);  // worker r0 + lane / 16's
        const double v = N == 4 ? four : __shfl(four, 16 * (mine & 3), kWave);
        if (mine - r0 >= 0 && mine - r0 < 4) sum = v;
    }
    return sum;
}

// ---------------------------------------------------------------------------
// Chunk owners' pass for n <= kServerRowBatch, one wave per tile, building
// the tables itself.  The tile's error-state and sign-word loads are issued
// first; the wave then reads the segment's scales, decides between the
// grouped and the one-by-one sum, and builds the 256-entry tables of every
// group of 8 workers (the 16-entry tables first, in the staging area, before
// the words are staged).  The words are then staged and regrouped, every
// group is looked up, and the tile is finished.  Each wave owns its LDS area,
// so it synchronises only with itself.
// ---------------------------------------------------------------------------
// With one group of 8 workers (n <= 8) the tables leave LDS for five
// workgroups per CU; asking for five waves per SIMD keeps the registers
// there too (95 instead of 126 VGPRs, no spills): 0.90 -> 0.86 ms on the
// stress workload.  Larger G8 is limited by its LDS.
//
// FORM (every chunk owned): the tiles are taken in address order, and the
// workers' scales are formed here from their partial sums, which saves the
// finalize kernel's launch.
template <int G8, bool FORM>  // groups of 8 workers the LDS tables hold: n <= 8 G8
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(G8 == 1 ? 5 : 1))) void k_server_pass(
    const Tile *__restrict__ tiles, const int32_t *__restrict__ chunk_tiles, int64_t tile_begin,
    int64_t tile_count, int n,
    int grouping_limit, const uint64_t *__restrict__ wbits, int64_t bits_ld,
    int64_t bits_word_base, float *__restrict__ wscales, int64_t scales_ld,
    int64_t scales_seg_base, float *__restrict__ serr, const float *__restrict__ sscales,
    uint64_t *__restrict__ sbits, double *__restrict__ partial, const Segment *__restrict__ segs,
    const double *__restrict__ wpartial, int64_t wpart_ld)
{
    __shared__ __align__(16) ServerTileLds<G8> s_lds[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    // wave-uniform: the tile and its fields live in scalar registers
    const int wv = wave_id();
    const int64_t rel = xcd_block() * kWavesPerBlock + wv;
    if (rel >= tile_count) return;
    ServerTileLds<G8> &L = s_lds[wv];
    const int groups8 = (n + 7) >> 3;
    const int64_t t = FORM ? tile_begin + rel : (int64_t)chunk_tiles[tile_begin + rel];
    const Tile tile = tiles[t];
    const int len = tile.len;
    const int64_t base = tile.start;
    const ServerRows in{wbits + ((base >> 6) - bits_word_base), bits_ld,
                        wscales + ((int64_t)tile.seg - scales_seg_base), scales_ld,
                        (len + 63) >> 6, len == kTileElems};
    const float sprev = sscales[tile.seg];
    v4f cv[kSubBlocks];
#pragma unroll
    for (int b = 0; b < kSubBlocks; ++b) {
        const int li = b * (kWave * 4) + 4 * lane;
        cv[b] = in.full ? ld4<true>(serr + base, li, len) : ld4<false>(serr + base, li, len);
    }
    uint64_t stg[kServerRowBatch / 4];
    server_load_words(in, 0, n, lane, stg);
    float scl;
    if (FORM) {
        const Segment sg = segs[tile.seg];
        const bool four = G8 == 1 && n <= 4;
        const int per = four ? kWave / 4 : kWave / (8 * G8);  // lanes per worker
        const int r = lane / per;
        const double *src = wpartial + sg.tile;
        const double s = four ? worker_segment_sums<4>(src, wpart_ld, n, sg.tiles, lane)
                              : worker_segment_sums<8 * G8>(src, wpart_ld, n, sg.tiles, lane);
        const float sr = scale_of(s, sg.len);
        const bool first = sg.tile == t;
        if (r < n && lane % per == 0) {
            L.scale[r] = sr;
            if (first) wscales[(int64_t)r * scales_ld + tile.seg] = sr;
        }
        if (first)
            for (int i = 0; i < n; ++i)
                zero_empty(wscales + (int64_t)i * scales_ld, tile.seg, sg, lane, kWave);
        wave_sync();
        scl = lane < n ? L.scale[lane] : 0.f;
    } else {
        scl = lane < n ? in.scales[(int64_t)lane * in.scales_ld] : 0.f;
        if (lane < n) L.scale[lane] = scl;
    }
    const bool grouped = server_grouped(in, n, grouping_limit, lane, scl);
    if (grouped) {
        wave_sync();
        server_build_lut4(L, n, lane);
        wave_sync();
#pragma unroll
        for (int k = 0; k < G8 * 256 / kWave; ++k) {
            const int e = lane + kWave * k;
            const int g = e >> 8, idx = e & 255;  // g = k / 4: uniform
            if (g < groups8)
                L.lut8[g][idx] = L.lut4[2 * g][idx & 15] + L.lut4[2 * g + 1][idx >> 4];
        }
        wave_sync();  // lut4 shares the staging area
    }
    server_stage_words(L, in, n, lane, stg);
    wave_sync();
    double sum[kSubBlocks][4];
#pragma unroll
    for (int b = 0; b < kSubBlocks; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[b][c] = 0.0;
    if (grouped) {
        server_regroup_bits(L, n, lane);
        wave_sync();
        for (int g = 0; g < groups8; ++g) server_lookup_group(sum, L, 8 * g, L.lut8[g], lane);
    } else {
        server_batch_one_by_one(sum, L, n, lane);
    }
    const double acc = server_epilogue(sum, cv, sprev, n, lane, tile, in.full, serr, sbits);
    if (lane == 0) partial[t] = acc;
}

// ---------------------------------------------------------------------------
// Chunk owners' pass for n <= kServerRowBatch with the tables in the
// workspace: each workgroup takes up to kWavesPerBlock consecutive tiles of
// one segment (entry b of `blocks`, one tile per wave) and shares one copy of
// the segment's tables, wave g copying group g's.  The tile loads are issued
// first; after one workgroup barrier (tables and staged words in place) each
// wave regroups its own words, looks every group up and finishes its tile.
// One shared table set instead of one per wave leaves room in LDS for five
// workgroups per CU.
// ---------------------------------------------------------------------------
struct ServerSharedLds {
    uint32_t bits[kWavesPerBlock][2 * kTileWords][kBitsStride];
    double lut8[kServerRowBatch / 8][256];
    float scale[kServerRowBatch];
};

// One wave's part of it, in the form the staging and summing helpers take.
struct ServerWaveLds {
    uint32_t (&bits)[2 * kTileWords][kBitsStride];
    float (&scale)[kServerRowBatch];
};

// Five waves per SIMD (90 instead of 122 VGPRs, no spills; the 28.8 KB of
// LDS per workgroup allows five per CU): 0.71 -> 0.69 ms on the BERT-Large
// shape, 0.21 -> 0.19 ms on BERT-Base.
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_server_shared(
    const Tile *__restrict__ tiles, const int32_t *__restrict__ chunk_tiles,
    const int32_t *__restrict__ blocks, int64_t num_blocks, int n,
    const uint64_t *__restrict__ wbits, int64_t bits_ld, int64_t bits_word_base,
    const float *__restrict__ wscales, int64_t scales_ld, int64_t scales_seg_base,
    float *__restrict__ serr, const float *__restrict__ sscales, uint64_t *__restrict__ sbits,
    double *__restrict__ partial, ServerTables st)
{
    __shared__ __align__(16) ServerSharedLds S;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_id();
    const int64_t b = xcd_block();
    if (b >= num_blocks) return;  // the whole workgroup
    const int32_t entry = blocks[b];
    const int64_t first = server_block_first(entry);
    const bool has = wv < server_block_tiles(entry);
    const int groups8 = (n + 7) >> 3;
    // every tile of the workgroup is in this segment
    const int seg = tiles[chunk_tiles[first]].seg;
    const int64_t u = owned_segment(seg, n, st);
    const bool grouped = st.flags[u] != 0;
    const int64_t t = chunk_tiles[first + (has ? wv : 0)];
    const Tile tile = tiles[t];
    const int len = tile.len;
    const int64_t base = tile.start;
    const ServerRows in{wbits + ((base >> 6) - bits_word_base), bits_ld,
                        wscales + ((int64_t)seg - scales_seg_base), scales_ld,
                        (len + 63) >> 6, len == kTileElems};
    const float sprev = sscales[seg];
    v4f cv[kSubBlocks];
    uint64_t stg[kServerRowBatch / 4];
    if (has) {
#pragma unroll
        for (int k = 0; k < kSubBlocks; ++k) {
            const int li = k * (kWave * 4) + 4 * lane;
            cv[k] = in.full ? ld4<true>(serr + base, li, len) : ld4<false>(serr + base, li, len);
        }
        server_load_words(in, 0, n, lane, stg);
    }
    if (grouped) {
        if (wv < groups8) server_fetch_tables(&S.lut8[wv][0], st, u, groups8, wv, 1, lane);
    } else if (wv == 0 && lane < n) {
        S.scale[lane] = in.scales[(int64_t)lane * in.scales_ld];
    }
    ServerWaveLds L{S.bits[wv], S.scale};
    if (has) server_stage_words(L, in, n, lane, stg);
    wait_vmem();
    __syncthreads();
    if (!has) return;
    double sum[kSubBlocks][4];
#pragma unroll
    for (int k = 0; k < kSubBlocks; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[k][c] = 0.0;
    if (grouped) {
        server_regroup_bits(L, n, lane);
        wave_sync();
        for (int g = 0; g < groups8; ++g) server_lookup_group(sum, L, 8 * g, S.lut8[g], lane);
    } else {
        server_batch_one_by_one(sum, L, n, lane);
    }
    const double acc = server_epilogue(sum, cv, sprev, n, lane, tile, in.full, serr, sbits);
    if (lane == 0) partial[t] = acc;
}

// ---------------------------------------------------------------------------
// Chunk owners' pass for many workers (n > kServerRowBatch) with the tables in
// the workspace: one workgroup per tile, wave w owning sub-block w of it (256
// elements: words 4w .. 4w+3).  The waves walk the incoming rows together in
// batches of kServerRowBatch: each loads and stages its own sub-block's words
// of the batch (4 words of each of 32 rows), the four share the batch's
// tables (wave g copies group g's), and the next batch's words and tables are
// on their way while a batch is looked up (two table buffers, one workgroup
// barrier per batch).  No partial sums are exchanged: each wave finishes its
// own sub-block, and the tile's sum of squares adds the four waves' in a
// fixed order.
// ---------------------------------------------------------------------------
struct ServerSubLds {
    uint32_t bits[kSubBlocks][2 * kTileWords / kSubBlocks][kBitsStride];  // each wave's 8 half-words
    double lut8[2][kServerRowBatch / 8][256];  // batch b's tables in lut8[b & 1]
    float scale[2][kServerRowBatch];           // batch b's scales (one-by-one sum)
    double red[kSubBlocks];
};

// Loads the words of sub-block w of rows [r0, r0 + rows) of the tile (rows <=
// kServerRowBatch): lane L takes word 4w + L % 4 of rows r0 + L/4 and
// r0 + L/4 + 16 (zero past the batch's rows and the tile's words).
__device__ __forceinline__ void server_load_sub_words(const ServerRows &in, int w, int r0,
                                                      int rows, int lane, uint64_t (&stg)[2])
{
    const int wi = 4 * w + (lane & 3);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int r = (lane >> 2) + 16 * k;
        stg[k] = (r < rows && wi < in.nwords)
                     ? __builtin_nontemporal_load(in.words + (int64_t)(r0 + r) * in.bits_ld + wi)
                     : 0ull;
    }
}

// Writes them into the wave's staging area ([local half-word][row]; the
// rows past the batch's last row, up to the next multiple of 8, get zero
// words).
__device__ __forceinline__ void server_stage_sub_words(uint32_t (&bits)[2 * kTileWords /
                                                                          kSubBlocks][kBitsStride],
                                                       int rows, int lane,
                                                       const uint64_t (&stg)[2])
{
    const int j = lane & 3;
    const int rows8 = (rows + 7) & ~7;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int r = (lane >> 2) + 16 * k;
        if (r < rows8) {
            bits[2 * j][r] = (uint32_t)stg[k];
            bits[2 * j + 1][r] = (uint32_t)(stg[k] >> 32);
        }
    }
}

__global__ __launch_bounds__(kSubBlocks * kWave) void k_server_subblocks(
    const Tile *__restrict__ tiles, const int32_t *__restrict__ chunk_tiles, int64_t tile_begin,
    int64_t tile_count, int n, const uint64_t *__restrict__ wbits, int64_t bits_ld,
    int64_t bits_word_base, const float *__restrict__ wscales, int64_t scales_ld,
    int64_t scales_seg_base, float *__restrict__ serr, const float *__restrict__ sscales,
    uint64_t *__restrict__ sbits, double *__restrict__ partial, ServerTables st)
{
    __shared__ __align__(16) ServerSubLds S;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_id();
    const int64_t rel = xcd_block();
    if (rel >= tile_count) return;  // the whole workgroup
    const int64_t t = chunk_tiles[tile_begin + rel];
    const Tile tile = tiles[t];
    const int len = tile.len;
    const int64_t base = tile.start;
    const ServerRows in{wbits + ((base >> 6) - bits_word_base), bits_ld,
                        wscales + ((int64_t)tile.seg - scales_seg_base), scales_ld,
                        (len + 63) >> 6, len == kTileElems};
    const int groups8 = (n + 7) >> 3;
    const int64_t u = owned_segment(tile.seg, n, st);
    const bool grouped = st.flags[u] != 0;
    const float sprev = sscales[tile.seg];
    const int li = wv * (kWave * 4) + 4 * lane;  // this wave's sub-block
    const v4f cv = in.full ? ld4<true>(serr + base, li, len) : ld4<false>(serr + base, li, len);
    uint64_t stg[2];
    const int rows0 = min(kServerRowBatch, n);
    server_load_sub_words(in, wv, 0, rows0, lane, stg);
    if (grouped && wv < ((rows0 + 7) >> 3))
        server_fetch_tables(&S.lut8[0][wv][0], st, u, groups8, wv, 1, lane);
    auto &bits = S.bits[wv];
    const int hw = lane >> 3;  // the lane's half-word of the sub-block
    const int o = 16 * (lane & 1) + ((lane & 7) >> 1);
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int r0 = 0; r0 < n; r0 += kServerRowBatch) {  // workgroup-uniform
        const int cur = (r0 / kServerRowBatch) & 1;
        const int rows = min(kServerRowBatch, n - r0);
        const int g8 = (rows + 7) >> 3;
        if (!grouped && wv == 0 && lane < rows)
            S.scale[cur][lane] = in.scales[(int64_t)(r0 + lane) * in.scales_ld];
        server_stage_sub_words(bits, rows, lane, stg);
        wait_vmem();
        // this batch's tables, scales and words are in place, and every wave
        // is done with the previous batch (whose buffers come next)
        __syncthreads();
        const int r1 = r0 + kServerRowBatch;
        if (r1 < n) {
            const int rows1 = min(kServerRowBatch, n - r1);
            if (grouped && wv < ((rows1 + 7) >> 3))
                server_fetch_tables(&S.lut8[cur ^ 1][wv][0], st, u, groups8, (r1 >> 3) + wv, 1,
                                    lane);
            server_load_sub_words(in, wv, r1, rows1, lane, stg);
        }
        if (grouped) {
            // regroup the sub-block's (half-word, group of 8 rows) blocks
            if (lane < 8 * g8) {
                uint32_t *p = &bits[lane & 7][8 * (lane >> 3)];
                const uint4 u0 = *(const uint4 *)p;
                const uint4 u1 = *(const uint4 *)(p + 4);
                uint32_t a[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
                transpose_bits8x8(a);
                *(uint4 *)p = make_uint4(a[0], a[1], a[2], a[3]);
                *(uint4 *)(p + 4) = make_uint4(a[4], a[5], a[6], a[7]);
            }
            wave_sync();
            for (int g = 0; g < g8; ++g) {
                const uint8_t *blk = (const uint8_t *)&bits[hw][8 * g];
                uint32_t idx[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) idx[c] = blk[o + 4 * c];
                double val[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) val[c] = S.lut8[cur][g][idx[c]];
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[c] += val[c];
            }
        } else {
            const int shift = 4 * (lane & 7);
            for (int r = 0; r < rows; ++r) {
                const double sp = (double)S.scale[cur][r];
                const uint32_t nib = (bits[hw][r] >> shift) & 0xFu;
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[c] += ((nib >> c) & 1u) ? sp : -sp;
            }
        }
        wave_sync();  // before this wave's staging area takes the next batch
    }
    const bool pow2 = (n & (n - 1)) == 0;
    double acc;
    if (in.full && pow2)
        acc = server_epilogue_sub<true, true>(sum, cv, sprev, n, lane, tile, wv, serr, sbits);
    else if (in.full)
        acc = server_epilogue_sub<true, false>(sum, cv, sprev, n, lane, tile, wv, serr, sbits);
    else if (pow2)
        acc = server_epilogue_sub<false, true>(sum, cv, sprev, n, lane, tile, wv, serr, sbits);
    else
        acc = server_epilogue_sub<false, false>(sum, cv, sprev, n, lane, tile, wv, serr, sbits);
    acc = wave_sum_dpp(acc);
    if (lane == 0) S.red[wv] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[t] = (S.red[0] + S.red[1]) + (S.red[2] + S.red[3]);
}

// ---------------------------------------------------------------------------
// Chunk owners' pass for many workers (n > kServerRowBatch): the
// kSplitWaves waves of a workgroup share one tile.  When the grouped sum
// applies, wave w takes row batches w, w + kSplitWaves, ...; the waves' exact
// partial sums are then added through LDS (exact, so in any order), and wave
// w finishes sub-block w of the tile.  Otherwise wave 0 adds every row one by
// one in worker order and hands the other waves their sub-blocks.  Every wave
// reads the n scales and builds each batch's tables itself (the pass with the
// tables in the workspace is k_server_subblocks).
// ---------------------------------------------------------------------------
constexpr int kSplitWaves = kSubBlocks;

__global__ __launch_bounds__(kSplitWaves * kWave) void k_server_split(
    const Tile *__restrict__ tiles, const int32_t *__restrict__ chunk_tiles, int64_t tile_begin,
    int64_t tile_count, int n, int grouping_limit, const uint64_t *__restrict__ wbits,
    int64_t bits_ld, int64_t bits_word_base, const float *__restrict__ wscales,
    int64_t scales_ld, int64_t scales_seg_base, float *__restrict__ serr,
    const float *__restrict__ sscales, uint64_t *__restrict__ sbits, double *__restrict__ partial)
{
    // the staging areas while rows are summed, then the exchange of partial
    // sums: xch[sub-block][source wave][element of the sub-block]
    union SplitLds {
        ServerBatchLds batch[kSplitWaves];
        double xch[kSubBlocks][kSplitWaves][kWave * 4];
    };
    __shared__ __align__(16) SplitLds s_lds;
    __shared__ double s_red[kSplitWaves];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_id();
    const int64_t rel = xcd_block();
    if (rel >= tile_count) return;  // the whole workgroup
    const int64_t t = chunk_tiles[tile_begin + rel];
    const Tile tile = tiles[t];
    const int len = tile.len;
    const int64_t base = tile.start;
    const ServerRows in{wbits + ((base >> 6) - bits_word_base), bits_ld,
                        wscales + ((int64_t)tile.seg - scales_seg_base), scales_ld,
                        (len + 63) >> 6, len == kTileElems};
    ServerBatchLds &L = s_lds.batch[wv];

    const float sprev = sscales[tile.seg];
    const int li = wv * (kWave * 4) + 4 * lane;  // this wave's sub-block
    const v4f cv = in.full ? ld4<true>(serr + base, li, len) : ld4<false>(serr + base, li, len);
    uint64_t stg[kServerRowBatch / 4];
    float scl = 0.f;
    const int rfirst = kServerRowBatch * wv;  // may be past n when n <= 96: no rows then
    server_load_batch(in, rfirst, max(0, min(kServerRowBatch, n - rfirst)), lane, stg, scl);
    // every wave reads all n scales and reaches the same decision
    const bool grouped = server_grouped(in, n, grouping_limit, lane, 0.f);
    double sum[kSubBlocks][4];
#pragma unroll
    for (int b = 0; b < kSubBlocks; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[b][c] = 0.0;
    if (grouped) {
        constexpr int kStep = kServerRowBatch * kSplitWaves;
        for (int r0 = rfirst; r0 < n; r0 += kStep) {
            const int rows = min(kServerRowBatch, n - r0);
            server_stage_batch(L, in, rows, lane, stg, scl);
            // the next batch's words travel while this one is summed
            if (r0 + kStep < n)
                server_load_batch(in, r0 + kStep, min(kServerRowBatch, n - r0 - kStep), lane, stg,
                                  scl);
            wave_sync();
            server_batch_grouped(sum, L, rows, lane);
            wave_sync();
        }
    } else if (wv == 0) {
        for (int r0 = 0; r0 < n; r0 += kServerRowBatch) {
            const int rows = min(kServerRowBatch, n - r0);
            if (r0 > 0) server_load_batch(in, r0, rows, lane, stg, scl);
            server_stage_batch(L, in, rows, lane, stg, scl);
            wave_sync();
            server_batch_one_by_one(sum, L, rows, lane);
            wave_sync();
        }
    }
    __syncthreads();  // every wave is done with its staging area
#pragma unroll
    for (int b = 0; b < kSubBlocks; ++b) {
        if (b == wv) continue;
        double2 *dst = (double2 *)&s_lds.xch[b][wv][4 * lane];
        dst[0] = make_double2(sum[b][0], sum[b][1]);
        dst[1] = make_double2(sum[b][2], sum[b][3]);
    }
    __syncthreads();
    double s4[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) s4[c] = sum[wv][c];
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
        if (w == wv) continue;
        const double2 *src = (const double2 *)&s_lds.xch[wv][w][4 * lane];
        const double2 a = src[0], b = src[1];
        s4[0] += a.x;
        s4[1] += a.y;
        s4[2] += b.x;
        s4[3] += b.y;
    }
    const bool pow2 = (n & (n - 1)) == 0;
    double acc;
    if (in.full && pow2)
        acc = server_epilogue_sub<true, true>(s4, cv, sprev, n, lane, tile, wv, serr, sbits);
    else if (in.full)
        acc = server_epilogue_sub<true, false>(s4, cv, sprev, n, lane, tile, wv, serr, sbits);
    else if (pow2)
        acc = server_epilogue_sub<false, true>(s4, cv, sprev, n, lane, tile, wv, serr, sbits);
    else
        acc = server_epilogue_sub<false, false>(s4, cv, sprev, n, lane, tile, wv, serr, sbits);
    acc = wave_sum_dpp(acc);
    if (lane == 0) s_red[wv] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[t] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
}


// ---------------------------------------------------------------------------
// Decompress + preconditioned update: x -= lr * (+-scale) / sqrt(v + eps).
// ---------------------------------------------------------------------------
// Every load of a wave's part of a block is issued before its first store.
// Kernels here keep that order wherever a wave would otherwise re-read data
// after storing: on
// this hardware a variant that interleaved the sign-word loads with the
// stores returned wrong words for about 1% of the elements of a 334M-element
// launch (exact on small grids), and the loads-first form is exact.
template <bool WHOLE>
__device__ __forceinline__ void update_sub(const Lane4 &l, int li, v4f xv, v4f vv,
                                           float *__restrict__ x, float *__restrict__ m_out,
                                           float lr, float eps)
{
    v4f mv;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float mbar = with_sign(l.s, l.nib, c);
        const float denom = __builtin_sqrtf(vv[c] + eps);
        const float ratio = mbar / denom;
        const float step = lr * ratio;
        xv[c] = xv[c] - step;
        mv[c] = mbar;
    }
    stb4<WHOLE>(x, li, l.valid, xv);
    if (m_out) stb4<WHOLE>(m_out, li, l.valid, mv);
}

// A workgroup takes one block, one 256-element sub-block per wave: each wave
// keeps 2 KB of loads in flight instead of 8 KB (a whole block), which the mix
// of two read streams and one written stream favours: 0.667 -> 0.619 ms on the
// BERT-Large shape, 1.112 -> 1.033 ms on the 5,000-tensor stress workload
// (half a tile per wave: 0.640 and 1.070 ms), in one A/B process each.  Large
// plans run seven workgroups per CU, held by unused LDS (launch_update).
//
// FORM: the scales are formed here from the chunk owners' partial sums (see
// wave_scale), which saves the finalize kernel's launch.
template <bool FORM>
__global__ __launch_bounds__(kBlock) void k_update(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t block_base,
    int64_t num_blocks, int64_t padded_len, const Segment *__restrict__ segs,
    const double *__restrict__ partial, const uint64_t *__restrict__ sbits,
    float *__restrict__ sscales, float *__restrict__ x, float *__restrict__ m_out,
    const float *__restrict__ v, float lr, float eps)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t blk = block_base + xcd_block();
    if (blk >= num_blocks) return;
    const int64_t base = blk * kTileElems;
    const int64_t room = padded_len - base;
    const int lim = room < kTileElems ? (int)room : kTileElems;
    const int li = (threadIdx.x >> 6) * (kWave * 4) + 4 * lane;
    x += base;
    if (m_out) m_out += base;
    uint64_t word = 0;
    v4f xv, vv;
    if (lim == kTileElems || li < lim) word = sbits[(base + li) >> 6];
    if (lim == kTileElems) {
        xv = ldb4<true>(x, li, lim);
        vv = ldb4<true>(v + base, li, lim);
    } else {
        xv = ldb4<false>(x, li, lim);
        vv = ldb4<false>(v + base, li, lim);
    }
    const Block rec = load_block(blocks, blk);
    if (FORM) {
        if (rec.whole) {
            const Segment sg = segs[rec.seg];
            const float s = wave_scale(sg, partial, lane);
            if (threadIdx.x < kWave && sg.tile == rec.tile) {
                if (lane == 0) sscales[rec.seg] = s;
                zero_empty(sscales, rec.seg, sg, lane, kWave);
            }
            update_sub<true>(Lane4{s, (uint32_t)(word >> (li & 63)), 4}, li, xv, vv, x, m_out, lr,
                             eps);
        } else if (li < lim) {
            const int w = li >> 6;
            const int t = rec.tile + __popc(rec.starts & ((2u << w) - 1u)) - 1;
            const Tile tile = tiles[t];
            const Segment sg = segs[tile.seg];
            const float s = row_scale(sg, partial, lane);
            if (sg.tile == t && ((rec.starts >> w) & 1u)) {  // the segment's first word
                if ((lane & 15) == 0) sscales[tile.seg] = s;
                zero_empty(sscales, tile.seg, sg, lane & 15, 16);
            }
            update_sub<false>(Lane4{s, (uint32_t)(word >> (li & 63)), tile_valid4(tile, base + li)},
                              li, xv, vv, x, m_out, lr, eps);
        }
        return;
    }
    const float s0 = sscales[rec.seg];
    if (rec.whole)
        update_sub<true>(lane_message<true>(tiles, rec, base, li, lim, word, s0, sscales), li, xv,
                         vv, x, m_out, lr, eps);
    else
        update_sub<false>(lane_message<false>(tiles, rec, base, li, lim, word, s0, sscales), li,
                          xv, vv, x, m_out, lr, eps);
}

// ---------------------------------------------------------------------------
// Explicit values: the error from the compensated form, and the decoded
// message (+-scale of each element's segment).  A workgroup takes one block of
// one row, one sub-block per wave, every load before its stores (a wave that
// walked the rows of its tile lane by lane took 362 us for 8 rows of 30 million
// elements, 284 us now).  zero_padding: padding elements are written
// as 0 (the caller then need not clear the buffer first); else they are left.
// ---------------------------------------------------------------------------
// Zeros past the first `valid` elements; returns how many to store.
__device__ __forceinline__ int pad_zeros(v4f &v, int valid, int li, int lim, int zero_padding)
{
    if (!zero_padding) return valid;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (c >= valid) v[c] = 0.f;
    return li < lim ? 4 : 0;
}

__global__ __launch_bounds__(kBlock) void k_materialize(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t num_blocks,
    FastDiv by_blocks, int64_t padded_len, const float *err, int64_t err_ld,
    const float *__restrict__ scales, int64_t scales_ld, float *out, int64_t out_ld,
    int zero_padding, int64_t item_base, int64_t num_items)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t at = xcd_block();
    if (at >= num_items) return;
    const int64_t item = item_base + at;
    const int64_t r = fast_quotient(item, by_blocks);
    const int64_t blk = item - r * num_blocks;
    const int64_t base = blk * kTileElems;
    const int64_t room = padded_len - base;
    const int lim = room < kTileElems ? (int)room : kTileElems;
    const int li = (threadIdx.x >> 6) * (kWave * 4) + 4 * lane;
    const float *src = err + r * err_ld + base;
    v4f zv = lim == kTileElems ? ldb4<true>(src, li, lim) : ldb4<false>(src, li, lim);
    const Block rec = load_block(blocks, blk);
    scales += r * scales_ld;
    float s = scales[rec.seg];
    int valid = 4;
    if (!rec.whole) {
        valid = 0;
        if (li < lim) {
            const Tile t = block_word_tile(tiles, rec, li >> 6);
            valid = tile_valid4(t, base + li);
            s = scales[t.seg];
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) zv[c] = error_of(zv[c], s);
    valid = pad_zeros(zv, valid, li, lim, zero_padding);
    stb4<false>(out + r * out_ld + base, li, valid, zv);
}

__global__ __launch_bounds__(kBlock) void k_decode(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t block_base,
    int64_t num_blocks, int64_t padded_len, const uint64_t *__restrict__ bits,
    const float *__restrict__ scales, float *__restrict__ out, int zero_padding)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t blk = block_base + xcd_block();
    if (blk >= num_blocks) return;
    const int64_t base = blk * kTileElems;
    const int64_t room = padded_len - base;
    const int lim = room < kTileElems ? (int)room : kTileElems;
    const int li = (threadIdx.x >> 6) * (kWave * 4) + 4 * lane;
    const uint64_t word = li < lim ? bits[(base + li) >> 6] : 0;
    const Block rec = load_block(blocks, blk);
    const float s0 = scales[rec.seg];
    const Lane4 l = rec.whole ? lane_message<true>(tiles, rec, base, li, lim, word, s0, scales)
                              : lane_message<false>(tiles, rec, base, li, lim, word, s0, scales);
    v4f v;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = with_sign(l.s, l.nib, c);
    const int valid = pad_zeros(v, l.valid, li, lim, zero_padding);
    stb4<false>(out + base, li, valid, v);
}

// ---------------------------------------------------------------------------
// l1 norm of a buffer over the real elements (the variance-stability
// indicator of Section 7.1): fp64 partial sums of |v| over up to kL1Groups
// workgroups (each a run of blocks, its waves taking turns), then one
// workgroup sums those in a fixed order.  With a partial sum per tile that last
// workgroup read 326,000 of them for the BERT-Large shape: 187 + 306 us, now
// 204 + 6 us.
// ---------------------------------------------------------------------------
constexpr int64_t kL1Groups = 2048;  // 8 waves on every SIMD

__global__ __launch_bounds__(kBlock) void k_l1_partial(
    const Tile *__restrict__ tiles, const Block *__restrict__ blocks, int64_t num_blocks,
    int64_t padded_len, const float *__restrict__ v, double *__restrict__ partial)
{
    __shared__ double red[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x >> 6;
    const int64_t per = (num_blocks + gridDim.x - 1) / gridDim.x;
    const int64_t group = xcd_block();
    const int64_t end = min(num_blocks, (group + 1) * per);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t blk = group * per + wv; blk < end; blk += kWavesPerBlock) {
        const int64_t base = blk * kTileElems;
        const int64_t room = padded_len - base;
        const int lim = room < kTileElems ? (int)room : kTileElems;
        v4f vv[kSubBlocks];
#pragma unroll
        for (int b = 0; b < kSubBlocks; ++b) {
            const int li = b * (kWave * 4) + 4 * lane;
            vv[b] = lim == kTileElems ? ldb4<true>(v + base, li, lim) : ldb4<false>(v + base, li, lim);
        }
        const Block rec = load_block(blocks, blk);
        if (rec.whole) {
#pragma unroll
            for (int b = 0; b < kSubBlocks; ++b)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] += (double)__builtin_fabsf(vv[b][c]);
        } else {
#pragma unroll
            for (int b = 0; b < kSubBlocks; ++b) {
                const int li = b * (kWave * 4) + 4 * lane;
                if (li >= lim) continue;
                const int valid = tile_valid4(block_word_tile(tiles, rec, li >> 6), base + li);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c < valid) acc[c] += (double)__builtin_fabsf(vv[b][c]);
            }
        }
    }
    const double s = wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
    if (lane == 0) red[wv] = s;
    __syncthreads();
    if (threadIdx.x == 0) partial[group] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(kBlock) void k_l1_final(const double *__restrict__ partial,
                                                     int64_t count, double *__restrict__ out)
{
    __shared__ double red[kWavesPerBlock];
    double s = 0.0;
#pragma unroll 8
    for (int64_t t = threadIdx.x; t < count; t += kBlock) s += partial[t];
    s = wave_sum(s);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = ((red[0] + red[1]) + red[2]) + red[3];
}

// Rows of a two-dimensional grid (kernels stride beyond it).
constexpr int64_t kMaxGridRows = 65535;

// Workgroups (of kWavesPerBlock waves) for one wave per item.
inline int64_t blocks_for(int64_t waves) { return xcd_grid(waves, kWavesPerBlock); }

}  // namespace

// The shape of a row-summing launch over num_blocks blocks and n rows.
// - Small plans (2^21 elements of fp32, 2^22 of 16-bit gradients, whose waves
//   are all on the chip at once): four rows' loads at a time and no barrier,
//   since one row after another is a chain of n round trips (10^6 elements, 16
//   fp32 rows: 13.6 us against 16.8, 18.4 and 35.6 in the shapes (1, 4, 1),
//   (1, 16, 1) and (4, 16, 1); 10^5 elements, 32 rows 12.6 against 14.2, 20.5
//   and 45.6; but 4x10^6 elements, 16 rows 59.8 against 51.1 in (1, 16, 1)).
// - Few rows, or a plan that does not fill the chip with whole blocks: one
//   sub-block per wave (BERT-Large, fp32 rows: n = 4 2.19 ms against 2.26 with
//   a whole block, n = 8 with the norm 3.46 against 3.53; fp16 n = 4 1.73
//   against 1.78 with two; 6x10^6 elements, 16 fp32 rows 82 us against 98).
// - Many rows: the longer runs of a whole block (fp32; BERT-Base, n = 32: 2.72
//   against 2.84 ms) or two sub-blocks (16-bit; 12 million elements, n = 16:
//   114 us against 123 with one and 137 with four).
template <class G>
using ManyRows = RowShape<sizeof(typename G::T) == 4 ? 4 : 2, 16, 1>;
using FewRows = RowShape<1, 16, 1>;
using SmallPlan = RowShape<1, 4, 4>;

template <class G, class F>
static void launch_row_sum(const DeviceTables &tb, int n, F launch)
{
    constexpr bool f32 = sizeof(typename G::T) == 4;
    if (tb.num_blocks <= (f32 ? 2048 : 4096))
        launch(SmallPlan{});
    else if (n <= (f32 ? 12 : 4) || (f32 && tb.num_blocks <= 8192))
        launch(FewRows{});
    else
        launch(ManyRows<G>{});
}

template <class G>
static void launch_warmup_t(const DeviceTables &tb, float *x, float *m, float *v, const void *g,
                            int64_t g_ld, int n_grads, float lr, float beta1, float beta2,
                            float eps, int use_bc, float bc1, float bc2, hipStream_t s)
{
    const float omb1 = 1.0f - beta1, omb2 = 1.0f - beta2;
    launch_row_sum<G>(tb, n_grads, [&](auto shape) {
        using Sh = decltype(shape);
        for (int64_t base = 0; base < tb.num_blocks; base += kMaxLaunchTiles) {
            const int64_t count = launch_piece(tb.num_blocks, base);
            hipLaunchKernelGGL((k_warmup<G, Sh>),
                               dim3((unsigned)xcd_grid(count * Sh::PARTS, Sh::WAVES)),
                               dim3(Sh::WAVES * kWave), 0, s, tb.tiles, tb.blocks, base,
                               base + count, tb.padded_len, x, m, v, (const typename G::T *)g, g_ld,
                               n_grads, lr, beta1, omb1, beta2, omb2, eps, use_bc, bc1, bc2);
        }
    });
}

hipError_t launch_warmup(const DeviceTables &tb, float *x, float *m, float *v, const void *g,
                         int grad_dtype, int64_t g_ld, int n_grads, float lr, float beta1,
                         float beta2, float eps, int use_bc, float bc1, float bc2, hipStream_t s)
{
    const auto launch = grad_dtype == kGradBF16  ? launch_warmup_t<GradBF16>
                        : grad_dtype == kGradF16 ? launch_warmup_t<GradF16>
                                                 : launch_warmup_t<GradF32>;
    launch(tb, x, m, v, g, g_ld, n_grads, lr, beta1, beta2, eps, use_bc, bc1, bc2, s);
    return hipGetLastError();
}

// What a call keeps in the caches.  1: its gradient and error rows fit a quarter
// of the 256 MB last-level cache, so the error rows that it writes can still be
// there in the next step and are stored without nt.  2: the gradient rows also
// fit half of the XCDs' 32 MB of L2 and are loaded without nt.  The error loads
// keep nt, and larger gradients too: loads without it lose where other work
// between two steps has filled the cache.
// Step, us, 0 / 1 / 2 / error loads without nt too, (a) back to back, (b) after
// 128 MB of other writes and new gradients, (c) after 1 GB of other writes and
// new gradients, (d) the same with old gradients: 2^20 elements n = 4 (16 MB of
// gradients) (a) 20.6 / 19.2 / 19.1 / 19.2, (b) 24.4 / 23.4 / 23.6 / 23.2, (c) 25.1
// / 25.6 / 25.6 / 26.2, (d) 25.9 / 26.3 / 28.9 / 30.3, stepping five states in turn
// 24.7 / 24.0 / 23.3 / 23.3; 5x10^5 n = 16 (32 MB) (a) 27.3 / 26.2 / 27.7 / 27.7,
// (b) 31.3 / 30.3 / 30.5 / 30.7, (c) 32.2 / 31.7 / 32.4 / 32.8, (d) 33.3 / 33.6 /
// 38.9 / 40.3, in turn 32.4 / 31.4 / 33.4 / 31.8; 2x10^6 n = 4 (32 MB) (a) 35.5 /
// 34.1 / 36.3 / 35.9, (b) 39.2 / 37.9 / 38.0 / 38.2, (d) 42.0 / 42.3 / 47.6 / 49.2.
// Up to 24 MB of gradients 2 is within 3% of 1 with new gradients, and 3 to 5%
// ahead in turn; at 32 MB it is 6% behind there.
static int row_caching(int64_t items, size_t grad_bytes)
{
    const int64_t elems = items * kTileElems;
    if (elems * (int64_t)(grad_bytes + 4) > (int64_t)64 << 20) return 0;
    return elems * (int64_t)grad_bytes <= (int64_t)16 << 20 ? 2 : 1;
}

template <bool PACKED, class G>
static void launch_worker_items(const DeviceTables &tb, int64_t num_tiles, const float *m,
                                const uint64_t *m_bits, const float *m_scales, const void *g,
                                int64_t g_ld, float *err, int64_t err_ld, const float *scales,
                                int64_t scales_ld, uint64_t *bits, int64_t bits_ld,
                                double *partial, int n_local, float beta1, hipStream_t s)
{
    const int64_t items = (int64_t)n_local * tb.num_blocks;
    const int cache = row_caching(items, sizeof(typename G::T));
    const auto kernel = cache == 2   ? k_worker_pass<PACKED, G, 2>
                        : cache == 1 ? k_worker_pass<PACKED, G, 1>
                                     : k_worker_pass<PACKED, G, 0>;
    for (int64_t base = 0; base < items; base += kMaxPassItems) {
        const int64_t count = std::min(items - base, kMaxPassItems);
        hipLaunchKernelGGL(kernel, dim3((unsigned)xcd_grid(count, 1)),
                           dim3(kWave * kPassWaves<G>), kPassIdleLds<G>, s, tb.tiles, tb.blocks,
                           tb.num_blocks, fast_div(tb.num_blocks), tb.padded_len, num_tiles, m,
                           m_bits, m_scales, (const typename G::T *)g, g_ld, err, err_ld, scales,
                           scales_ld, bits, bits_ld, partial, base, count, beta1, 1.0f - beta1);
    }
}

// Whether a call with an fp32 momentum takes the packed pass's grid, which reads
// m again for every worker (from the caches, on plans of this size), instead of
// the row walk.  The walk's workgroups of 8 blocks run one to a CU, 2,048 blocks
// at a time, and step over the rows together, so a last round that is far from
// full costs as much as a full one: the packed grid wins there in the first two
// rounds.  Call, us, walk / packed, fp32 gradients unless said: 10^5 elements,
// 32 rows (a step) 103 / 32; 1,030 blocks n = 8 32.2 / 25.4, bf16 33.0 / 25.0, n = 32
// 112.9 / 88.0; 1,300 n = 8 34.0 / 31.2; 1,500 n = 8 34.6 / 37.1, bf16 35.5 / 34.3;
// 2,000 n = 8 40.0 / 48.0; 2,100 n = 8 62.0 / 50.0, n = 32 221 / 179; 2,500 n = 8 63.9 /
// 58.6; 2,900 n = 8 66.6 / 69.6; 4,000 n = 8 73.6 / 89.5; 4,340 n = 8 95.9 / 97.7, n =
// 16 181.7 / 186.1.  Two or three rows share m too little for the
// walk to pay before it runs several rounds: n = 2 2,100 blocks 17.3 / 14.0, 3,500
// 22.7 / 20.3, 4,500 29.6 / 27.2; n = 3 2,000 19.0 / 17.4, 3,100 28.2 / 28.2, 4,000
// 32.7 / 35.7.
static bool packed_grid(int64_t num_blocks, int n_local)
{
    constexpr int64_t round = 256 * kWalkBlocks;  // blocks on the chip at once
    if (n_local == 1) return true;                // no other row to share m with
    if (n_local == 2 && num_blocks <= 2 * round + round / 4) return true;
    if (n_local == 3 && num_blocks <= round + round / 2) return true;
    return num_blocks <= round * 11 / 16 ||
           (num_blocks > round && num_blocks <= round + round * 3 / 8);
}

template <class G>
static void launch_worker_g(const DeviceTables &tb, int64_t num_tiles, const float *m,
                            const uint64_t *m_bits, const float *m_scales, const void *g,
                            int64_t g_ld, float *err, int64_t err_ld, const float *scales,
                            int64_t scales_ld, uint64_t *bits, int64_t bits_ld, double *partial,
                            int n_local, float beta1, hipStream_t s)
{
    if (!m) {
        launch_worker_items<true, G>(tb, num_tiles, m, m_bits, m_scales, g, g_ld, err, err_ld,
                                     scales, scales_ld, bits, bits_ld, partial, n_local, beta1, s);
        return;
    }
    if (packed_grid(tb.num_blocks, n_local)) {
        launch_worker_items<false, G>(tb, num_tiles, m, m_bits, m_scales, g, g_ld, err, err_ld,
                                      scales, scales_ld, bits, bits_ld, partial, n_local, beta1,
                                      s);
        return;
    }
    for (int64_t base = 0; base < tb.num_blocks; base += kMaxLaunchTiles) {
        const int64_t count = launch_piece(tb.num_blocks, base);
        hipLaunchKernelGGL(k_worker_rows<G>, dim3((unsigned)xcd_grid(count, kWalkBlocks)),
                           dim3(kWalkWaves * kWave), 0, s, tb.tiles, tb.blocks, base, base + count,
                           tb.padded_len, num_tiles, m, (const typename G::T *)g, g_ld, err,
                           err_ld, scales, scales_ld, bits, bits_ld, partial, n_local, beta1,
                           1.0f - beta1);
    }
}

hipError_t launch_worker_pass(const DeviceTables &tb, int64_t num_tiles, const float *m,
                              const uint64_t *m_bits, const float *m_scales, const void *g,
                              int grad_dtype, int64_t g_ld, float *err, int64_t err_ld,
                              const float *scales, int64_t scales_ld, uint64_t *bits,
                              int64_t bits_ld, double *partial, int n_local, float beta1,
                              hipStream_t s)
{
    const auto launch = grad_dtype == kGradBF16  ? launch_worker_g<GradBF16>
                        : grad_dtype == kGradF16 ? launch_worker_g<GradF16>
                                                 : launch_worker_g<GradF32>;
    launch(tb, num_tiles, m, m_bits, m_scales, g, g_ld, err, err_ld, scales, scales_ld, bits,
           bits_ld, partial, n_local, beta1, s);
    return hipGetLastError();
}

hipError_t launch_adam_message(const DeviceTables &tb, const uint64_t *bits, const float *scales,
                               float *x, float *m, float *v, float lr, float beta1, float beta2,
                               float eps, int use_bc, float bc1, float bc2, hipStream_t s)
{
    const float omb1 = 1.0f - beta1, omb2 = 1.0f - beta2;
    for (int64_t base = 0; base < tb.num_blocks; base += kMaxLaunchTiles) {
        const int64_t count = launch_piece(tb.num_blocks, base);
        hipLaunchKernelGGL(k_adam_message, dim3((unsigned)xcd_grid(count, 1)), dim3(kBlock),
                           idle_lds(5), s, tb.tiles, tb.blocks, base, base + count, tb.padded_len,
                           bits, scales, x, m, v, lr, beta1, omb1, beta2, omb2, eps, use_bc, bc1, bc2);
    }
    return hipGetLastError();
}

template <class G>
static void launch_uncompressed_t(const DeviceTables &tb, float *x, float *m, const float *v,
                                  const void *g, int64_t g_ld, int n, float lr, float beta1,
                                  float eps, hipStream_t s)
{
    const float omb1 = 1.0f - beta1;
    launch_row_sum<G>(tb, n, [&](auto shape) {
        using Sh = decltype(shape);
        for (int64_t base = 0; base < tb.num_blocks; base += kMaxLaunchTiles) {
            const int64_t count = launch_piece(tb.num_blocks, base);
            hipLaunchKernelGGL((k_uncompressed<G, Sh>),
                               dim3((unsigned)xcd_grid(count * Sh::PARTS, Sh::WAVES)),
                               dim3(Sh::WAVES * kWave), 0, s, tb.tiles, tb.blocks, base,
                               base + count, tb.padded_len, x, m, v, (const typename G::T *)g, g_ld,
                               n, lr, beta1, omb1, eps);
        }
    });
}

hipError_t launch_uncompressed(const DeviceTables &tb, float *x, float *m, const float *v,
                               const void *g, int grad_dtype, int64_t g_ld, int n, float lr,
                               float beta1, float eps, hipStream_t s)
{
    const auto launch = grad_dtype == kGradBF16  ? launch_uncompressed_t<GradBF16>
                        : grad_dtype == kGradF16 ? launch_uncompressed_t<GradF16>
                                                 : launch_uncompressed_t<GradF32>;
    launch(tb, x, m, v, g, g_ld, n, lr, beta1, eps, s);
    return hipGetLastError();
}

hipError_t launch_l1_norm(const DeviceTables &tb, const float *v, double *partial, double *out,
                          hipStream_t s)
{
    const int64_t groups =
        std::min(kL1Groups, xcd_grid(tb.num_blocks, kWavesPerBlock));  // multiples of kXcds
    if (groups > 0)
        hipLaunchKernelGGL(k_l1_partial, dim3((unsigned)groups), dim3(kBlock), 0, s, tb.tiles,
                           tb.blocks, tb.num_blocks, tb.padded_len, v, partial);
    hipLaunchKernelGGL(k_l1_final, dim3(1), dim3(kBlock), 0, s, partial, groups, out);
    return hipGetLastError();
}

hipError_t launch_decode(const DeviceTables &tb, const uint64_t *bits, const float *scales,
                         float *out, int zero_padding, hipStream_t s)
{
    for (int64_t base = 0; base < tb.num_blocks; base += kMaxLaunchTiles) {
        const int64_t count = launch_piece(tb.num_blocks, base);
        hipLaunchKernelGGL(k_decode, dim3((unsigned)xcd_grid(count, 1)), dim3(kBlock), 0, s,
                           tb.tiles, tb.blocks, base, base + count, tb.padded_len, bits, scales,
                           out, zero_padding);
    }
    return hipGetLastError();
}

template <int LANES, int MAX>
static void launch_finalize_t(const DeviceTables &tb, int64_t num_segments, int64_t rows, int n,
                              int jb, int cnt, const double *partial, int64_t part_ld,
                              float *scales, int64_t scales_ld, hipStream_t s)
{
    const int64_t per = kBlock / LANES;
    const dim3 grid((unsigned)std::min((num_segments + per - 1) / per, kMaxGridBlocks),
                    (unsigned)std::min(rows, kMaxGridRows));
    hipLaunchKernelGGL((k_finalize<LANES, MAX>), grid, dim3(kBlock), 0, s, tb.segs,
                       (uint32_t)num_segments, rows, n, jb, cnt, partial, part_ld, scales,
                       scales_ld);
}

hipError_t launch_finalize(const DeviceTables &tb, int64_t max_seg_tiles, int64_t num_segments,
                           int64_t rows, int n, int jb, int cnt, const double *partial,
                           int64_t part_ld, float *scales, int64_t scales_ld, hipStream_t s)
{
    if (num_segments <= 0 || rows <= 0) return hipSuccess;
    // A workgroup for segments above 256 tiles (there are few of them, and
    // their latency counts), which is the plan's order of summation too.  Below
    // that the lanes share one order: as many as leave a lane at most 16
    // partial sums, but a whole wave, with fewer dependent steps, while all the
    // pairs' waves are on the chip at once anyway.
    const bool few = num_segments * rows <= 4096;
    const auto launch = max_seg_tiles > kWaveSegTiles ? launch_finalize_t<kBlock, kWaveSegTiles>
                        : max_seg_tiles > 4 && few       ? launch_finalize_t<kWave, kWaveSegTiles>
                        : max_seg_tiles > kWave          ? launch_finalize_t<16, kWaveSegTiles>
                        : max_seg_tiles > 4              ? launch_finalize_t<8, kWave>
                                                         : launch_finalize_t<1, 4>;
    launch(tb, num_segments, rows, n, jb, cnt, partial, part_ld, scales, scales_ld, s);
    return hipGetLastError();
}

size_t server_table_bytes(int n, int64_t segments)
{
    return (size_t)segments * (size_t)((n + 7) / 8) * 256 * sizeof(double);
}

hipError_t launch_server_pass(const DeviceTables &tb, int64_t tile_begin, int64_t tile_count,
                              int n, const uint64_t *wbits, int64_t bits_ld,
                              int64_t bits_word_base, float *wscales, int64_t scales_ld,
                              int64_t scales_seg_base, float *serr, float *sscales,
                              uint64_t *sbits, double *partial, const double *wpartial,
                              int64_t wpart_ld, int num_tensors, int cb, int nown, double *tables, int32_t *flags,
                              const int32_t *server_blocks, int64_t num_blocks, bool direct,
                              hipStream_t s)
{
    if (direct) {
        for (int64_t base = 0; base < tb.num_blocks; base += kMaxLaunchTiles) {
            const int64_t count = launch_piece(tb.num_blocks, base);
            hipLaunchKernelGGL(k_server_direct, dim3((unsigned)xcd_grid(count, 1)), dim3(kBlock),
                               0, s, tb.tiles, tb.blocks, base, base + count, tb.padded_len, n,
                               wbits, bits_ld, wscales, scales_ld, serr, sscales, sbits, partial);
        }
        return hipGetLastError();
    }
    int log2n = 0;
    while ((1 << log2n) < n) ++log2n;
    const int grouping_limit = 29 - log2n;
    const ServerTables st{tables, flags, cb, nown};
    const bool use_tables = tables != nullptr;
    if (use_tables)
        hipLaunchKernelGGL(k_server_tables,
                           dim3((unsigned)((int64_t)num_tensors * nown * ((n + 7) / 8))),
                           dim3(kBlock), 0, s, n, cb, nown, grouping_limit, wscales, scales_ld,
                           scales_seg_base, tables, flags);
    // more than one batch of rows: the waves of a workgroup share each tile
    // (one workgroup per tile, launched kMaxLaunchTiles tiles at a time)
    if (n > kServerRowBatch) {
        for (int64_t off = 0; off < tile_count; off += kMaxLaunchTiles) {
            const int64_t count = launch_piece(tile_count, off);
            const dim3 grid((unsigned)xcd_grid(count, 1));
            if (use_tables)
                hipLaunchKernelGGL(k_server_subblocks, grid, dim3(kSubBlocks * kWave), 0, s,
                                   tb.tiles, tb.chunk_tiles, tile_begin + off, count, n, wbits,
                                   bits_ld, bits_word_base, wscales, scales_ld, scales_seg_base,
                                   serr, sscales, sbits, partial, st);
            else
                hipLaunchKernelGGL(k_server_split, grid, dim3(kSplitWaves * kWave), 0, s,
                                   tb.tiles, tb.chunk_tiles, tile_begin + off, count, n,
                                   grouping_limit, wbits, bits_ld, bits_word_base, wscales,
                                   scales_ld, scales_seg_base, serr, sscales, sbits, partial);
        }
    } else if (use_tables) {
        // a workgroup per entry of the block list (up to one per tile)
        for (int64_t off = 0; off < num_blocks; off += kMaxLaunchTiles) {
            const int64_t count = launch_piece(num_blocks, off);
            hipLaunchKernelGGL(k_server_shared, dim3((unsigned)xcd_grid(count, 1)), dim3(kBlock),
                               0, s, tb.tiles, tb.chunk_tiles, server_blocks + off, count, n,
                               wbits, bits_ld, bits_word_base, wscales, scales_ld,
                               scales_seg_base, serr, sscales, sbits, partial, st);
        }
    } else {
        // tables for as many groups of 8 as n needs: more workgroups per CU
        // for small n
        const auto kernel = n <= 8    ? (wpartial ? k_server_pass<1, true> : k_server_pass<1, false>)
                            : n <= 16 ? (wpartial ? k_server_pass<2, true> : k_server_pass<2, false>)
                                      : (wpartial ? k_server_pass<4, true> : k_server_pass<4, false>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks_for(tile_count)), dim3(kBlock), 0, s,
                           tb.tiles, tb.chunk_tiles, tile_begin, tile_count, n, grouping_limit,
                           wbits, bits_ld, bits_word_base, wscales, scales_ld, scales_seg_base,
                           serr, sscales, sbits, partial, tb.segs, wpartial, wpart_ld);
    }
    return hipGetLastError();
}

hipError_t launch_update(const DeviceTables &tb, const uint64_t *sbits, float *sscales,
                         const double *partial, float *x, float *m_out, const float *v, float lr,
                         float eps, hipStream_t s)
{
    // Seven workgroups per CU above 2^24 elements, where memory bounds the pass
    // and a little less in flight suits its read and write streams; below, x and
    // v are mostly in the last-level cache and every wave helps.  Update, us, at
    // eight / seven / six, in one process on the same buffers: 3x10^6 elements
    // 6.9 / 6.9 / 7.5, 6x10^6 10.5 / 10.8 / 11.8, 10^7 18.4 / 18.7 / 19.4, 1.4x10^7
    // 26.2 / 26.5 / 27.0, 1.8x10^7 34.5 / 34.0 / 34.0, BERT-Large 606.4 / 602.5 /
    // 603.4, 5,000 tensors 1002 / 995 / 1007.
    const size_t lds = tb.num_blocks > 16384 ? idle_lds(7) : 0;
    const auto kernel = partial ? k_update<true> : k_update<false>;
    for (int64_t base = 0; base < tb.num_blocks; base += kMaxLaunchTiles) {
        const int64_t count = launch_piece(tb.num_blocks, base);
        hipLaunchKernelGGL(kernel, dim3((unsigned)xcd_grid(count, 1)), dim3(kBlock), lds,
                           s, tb.tiles, tb.blocks, base, base + count, tb.padded_len, tb.segs,
                           partial, sbits, sscales, x, m_out, v, lr, eps);
    }
    return hipGetLastError();
}

hipError_t launch_materialize(const DeviceTables &tb, int rows, const float *err, int64_t err_ld,
                              const float *scales, int64_t scales_ld, float *out, int64_t out_ld,
                              int zero_padding, hipStream_t s)
{
    const int64_t items = (int64_t)rows * tb.num_blocks;
    for (int64_t base = 0; base < items; base += kMaxPassItems) {
        const int64_t count = std::min(items - base, kMaxPassItems);
        hipLaunchKernelGGL(k_materialize, dim3((unsigned)xcd_grid(count, 1)),
                           dim3(kBlock), 0, s, tb.tiles, tb.blocks, tb.num_blocks,
                           fast_div(tb.num_blocks), tb.padded_len, err, err_ld, scales, scales_ld,
                           out, out_ld, zero_padding, base, count);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scratch memory of the entry point that allocates nothing: the per-tile
// fp64 partial sums that the caller's workspace holds otherwise.  Host code
// never uses the array's name as an address (on the host it is only a
// handle for the symbol lookup); it uses the per-device address that
// hipGetSymbolAddress returns.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];

namespace {
std::once_flag g_scratch_once[kMaxScratchDevices];
void *g_scratch_ptr[kMaxScratchDevices];
hipError_t g_scratch_err[kMaxScratchDevices];
}  // namespace

hipError_t scratch_address(int device, void **ptr)
{
    *ptr = nullptr;
    if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::call_once(g_scratch_once[device], [device] {
        int prev = -1;
        hipError_t e = hipGetDevice(&prev);
        if (e == hipSuccess && prev != device) e = hipSetDevice(device);
        void *p = nullptr;
        if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (prev >= 0 && prev != device) {
            const hipError_t r = hipSetDevice(prev);
            if (e == hipSuccess) e = r;
        }
        g_scratch_err[device] = e;
        g_scratch_ptr[device] = e == hipSuccess ? p : nullptr;
    });
    *ptr = g_scratch_ptr[device];
    return g_scratch_err[device];
}

}  // namespace onebit
