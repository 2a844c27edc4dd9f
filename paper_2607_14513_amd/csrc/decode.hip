// decode.hip -- random-access decode and SH evaluation on gfx950.
//
//   decode       every block of every band back to 8-bit RGBA texels;
//   decode_eval  for each listed slot (one per lane): find its 16 band blocks
//                by index x block size (random access, Sec. I), decode its
//                texel from each, dequantise (vmin + q * delta); then
//                c = sum_k Hhat_k Y_k(d) (Sec. II colour equation) for every
//                direction, computed as a K = 16 matrix product on the
//                matrix cores.
#include "gsbc_internal.h"
#include "bc_format.h"

namespace gsbc {
namespace {

constexpr int kEvalBlock = 256;

__device__ __forceinline__ uint32_t zigzag_texel(uint32_t j)
{
    uint32_t x = (j & 1u) | (((j >> 2) & 1u) << 1);
    uint32_t y = ((j >> 1) & 1u) | (((j >> 3) & 1u) << 1);
    return 4 * y + x;
}

template <class Lut = Bc7ConstLut>
__device__ __forceinline__ uint32_t band_texel(const uint8_t *blocks, const BandArgs &b, int k,
                                               uint64_t blk, int texel, const Lut &lut = Lut{})
{
    if (b.format[k] == GSBC_FMT_NONE) return 0u;   // a stream given 0 bits stores no blocks
    const uint8_t *base = blocks + b.offset[k];
    if (b.format[k] == 1) {
        uint2 w = *reinterpret_cast<const uint2 *>(base + blk * 8);
        return bc1_texel(w.x, w.y, texel);
    }
    ulonglong2 w = *reinterpret_cast<const ulonglong2 *>(base + blk * 16);
    Blk128 q{w.x, w.y};
    return bc7_texel(q, texel, lut);
}

// The band texels of slot s, each found through the arrangement:
// 0: stream k, block s/16, zigzag texel of s%16 (only the n_streams kept
// bands of a lower-degree scene; px[k] = 0 past them); 1: stream 0, block s,
// texel k; 2: stream k/4, block s/4, texel 4 (s%4) + k%4 (only the bands of
// the n_streams streams: one stream is Fig. SetupC, bands 0..3).
// One load per block, each decoded as it arrives (the fewest memory
// instructions, for gathers that issue little else):
template <int ARR, class Lut>
__device__ __forceinline__ void slot_texels_arr(const uint8_t *blocks, const BandArgs &b, uint32_t s, uint32_t px[16],
                                                const Lut &lut)
{
#pragma unroll
    for (int k = 0; k < 16; k++) {
        if (ARR == 1) px[k] = band_texel(blocks, b, 0, s, k, lut);
        else if (ARR == 2) px[k] = (uint32_t)(k >> 2) < b.n_streams
                                       ? band_texel(blocks, b, k >> 2, s >> 2, 4 * (int)(s & 3u) + (k & 3), lut) : 0u;
        else px[k] = (uint32_t)k < b.n_streams ? band_texel(blocks, b, k, s >> 4, (int)zigzag_texel(s & 15u), lut)
                                               : 0u;
    }
}

// or every block loaded before any is decoded, as two 8-byte halves (an
// 8-byte BC1 block loads its one half twice), so that the loads share one
// wait, and the BC7 partition table read through `lut`:
template <int ARR, class Lut>
__device__ __forceinline__ void slot_texels_arr_batched(const uint8_t *blocks, const BandArgs &b, uint32_t s,
                                                        uint32_t px[16], const Lut &lut)
{
    uint2 lo[16], hi[16];
#pragma unroll
    for (int k = 0; k < 16; k++) {
        // stream of band k (a dropped band reads stream 0's block and ignores it)
        const int sk = ARR == 1 ? 0
                     : ARR == 2 ? ((uint32_t)(k >> 2) < b.n_streams ? (k >> 2) : 0)
                                : ((uint32_t)k < b.n_streams ? k : 0);
        const uint64_t blk = ARR == 1 ? s : ARR == 2 ? (s >> 2) : (s >> 4);
        const bool wide = b.format[sk] != 1;
        const uint8_t *q = blocks + b.offset[sk] + blk * (wide ? 16 : 8);
        // a stream given 0 bits stores no blocks: nothing to load
        const bool stored = b.format[sk] != GSBC_FMT_NONE;
        lo[k] = stored ? *reinterpret_cast<const uint2 *>(q) : make_uint2(0u, 0u);
        hi[k] = stored ? *reinterpret_cast<const uint2 *>(q + (wide ? 8 : 0)) : make_uint2(0u, 0u);
    }
#pragma unroll
    for (int k = 0; k < 16; k++) {
        const int sk = ARR == 1 ? 0 : ARR == 2 ? (k >> 2) : k;
        const int texel = ARR == 1 ? k : ARR == 2 ? 4 * (int)(s & 3u) + (k & 3) : (int)zigzag_texel(s & 15u);
        if ((ARR == 0 && (uint32_t)k >= b.n_streams) || (ARR == 2 && (uint32_t)(k >> 2) >= b.n_streams) ||
            b.format[sk] == GSBC_FMT_NONE)
            px[k] = 0u;
        else if (b.format[sk] == 1) px[k] = bc1_texel(lo[k].x, lo[k].y, texel);
        else px[k] = bc7_texel(Blk128{lo[k].x | (uint64_t)lo[k].y << 32, hi[k].x | (uint64_t)hi[k].y << 32}, texel, lut);
    }
}

// Dequantised coefficient of code q (low byte) in band k: vmin + q delta with
// the FP64 step delta = dhi + dlo (to 2^-48).  Each fused step rounds once,
// relative to its own result: vmin + q dhi, then + q dlo, so the value
// carries about one FP32 rounding of itself.  With delta rounded to FP32
// the step's error (2^-24 of the whole band range) would dominate whenever
// vmin and q delta nearly cancel.
__device__ __forceinline__ float dequant(uint32_t q, const BandArgs &b, int k)
{
    const float qf = (float)(q & 255u);
    return fmaf(qf, b.dlo[k], fmaf(qf, b.dhi[k], b.vmin[k]));
}

// Bands present in the scene: all 16, or the lowest n_streams (band
// arrangement) or 4 n_streams (quad arrangement, Fig. SetupC with one
// stream) of a lower-degree scene; the rest are exactly zero.
__device__ __forceinline__ uint32_t kept_bands(const BandArgs &b)
{
    return b.arrangement == 0 ? b.n_streams : b.arrangement == 2 ? 4u * b.n_streams : 16u;
}

// Band k has coded values: it is one of the scene's bands and its stream
// was not given 0 bits (band arrangement only); otherwise it is zero.
__device__ __forceinline__ bool band_coded(const BandArgs &b, int k)
{
    return (uint32_t)k < kept_bands(b) && !(b.arrangement == 0 && b.format[k] == GSBC_FMT_NONE);
}

// The BC7 partition table comes through lut: Bc7ConstLut (constant memory) or
// Bc7LdsLut (the workgroup's LDS copy, whose lookups wait on LDS
// instead of on a second memory round trip after the block's).
template <class Lut>
__device__ __forceinline__ void slot_texels(const uint8_t *blocks, const BandArgs &b, uint32_t s, uint32_t px[16],
                                            const Lut &lut)
{
    if (b.arrangement == 1) slot_texels_arr<1>(blocks, b, s, px, lut);
    else if (b.arrangement == 2) slot_texels_arr<2>(blocks, b, s, px, lut);
    else slot_texels_arr<0>(blocks, b, s, px, lut);
}

template <class Lut>
__device__ __forceinline__ void slot_texels_batched(const uint8_t *blocks, const BandArgs &b, uint32_t s,
                                                    uint32_t px[16], const Lut &lut)
{
    if (b.arrangement == 1) slot_texels_arr_batched<1>(blocks, b, s, px, lut);
    else if (b.arrangement == 2) slot_texels_arr_batched<2>(blocks, b, s, px, lut);
    else slot_texels_arr_batched<0>(blocks, b, s, px, lut);
}

// All 16 texels of the block whose halves are lo and hi (BC1: lo alone), zero
// without stored blocks.
template <class Lut>
__device__ __forceinline__ void block_texels(uint32_t format, uint2 lo, uint2 hi, uint32_t (&px)[16], const Lut &lut)
{
    if (format == 1) bc1_block(lo.x, lo.y, px);
    else if (format != GSBC_FMT_NONE)
        bc7_block(Blk128{lo.x | (uint64_t)lo.y << 32, hi.x | (uint64_t)hi.y << 32}, px, lut);
    else
#pragma unroll
        for (int i = 0; i < 16; i++) px[i] = 0u;
}

// Block blk of a stream, as two halves (a BC1 block's one half twice).
__device__ __forceinline__ void load_block(const uint8_t *base, uint32_t format, uint64_t blk, uint2 &lo, uint2 &hi)
{
    lo = hi = make_uint2(0u, 0u);
    if (format == GSBC_FMT_NONE) return;   // a stream given 0 bits stores no blocks
    const bool wide = format != 1;
    const uint8_t *q = base + blk * (wide ? 16 : 8);
    lo = *reinterpret_cast<const uint2 *>(q);
    hi = *reinterpret_cast<const uint2 *>(q + (wide ? 8 : 0));
}

// A workgroup's copy of the partition table; the caller synchronises.
__device__ __forceinline__ Bc7LdsLut stage_parts(Bc7Part *rows)
{
    for (uint32_t e = threadIdx.x; e < (uint32_t)kBc7PartRows; e += 256) rows[e] = kBc7Parts.row[e];
    return Bc7LdsLut{rows};
}

// The band texels of slot s0 + t for each thread t of 256, s0 a multiple of
// 256 and all 256 slots in the scene.  Their texels are those of 256 whole
// blocks (64 in the quad arrangement's one-stream form), so each thread
// decodes one block for all its texels, about a quarter of the instructions
// of 16 texels found one by one, and hands them over in LDS: row `band`, slot
// t at t + 4 (t / 16) (16-byte pieces, spread over the banks).  1,048,576
// slots x 64 directions 182 -> 145 us, all of a 3,145,728-slot scene from one
// view position 0.26 -> 0.09 ms (part of each gain is the texel decoder's).
// wanted(i, k): whether any of the k slots from s0 + i on is asked for; the
// blocks of others are not read.
constexpr int kTileRow = 320;
constexpr int kTileWords = 16 * kTileRow;

template <class Lut, class Wanted>
__device__ __forceinline__ void slot_texels_tile(const uint8_t *blocks, const BandArgs &b, uint64_t s0, uint32_t *tile,
                                                 uint32_t (&px)[16], const Lut &lut, Wanted wanted)
{
    const uint32_t t = threadIdx.x, lane = t & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
    uint2 lo, hi;
    if (b.arrangement == 1) {         // block s holds slot s's bands
        if (!wanted(t, 1)) return;
        load_block(blocks + b.offset[0], b.format[0], s0 + t, lo, hi);
        block_texels(b.format[0], lo, hi, px, lut);
        return;
    }
    if (b.arrangement == 2) {         // a wave's 64 blocks of stream `wave`: 4 slots x 4 bands each
        if (wave < b.n_streams && wanted(4 * lane, 4)) {
            load_block(blocks + b.offset[wave], b.format[wave], (s0 >> 2) + lane, lo, hi);
            block_texels(b.format[wave], lo, hi, px, lut);
#pragma unroll
            for (int q = 0; q < 4; q++)
                *reinterpret_cast<uint4 *>(&tile[(4 * wave + q) * kTileRow + 20 * (lane >> 2) + 4 * (lane & 3u)]) =
                    make_uint4(px[q], px[4 + q], px[8 + q], px[12 + q]);
        }
    } else {                          // a wave's 16 blocks of each of 4 bands
        const uint32_t band = t >> 4;
        uint32_t format = GSBC_FMT_NONE;
        uint64_t offset = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; q++)
            if ((lane >> 4) == q && 4 * wave + q < b.n_streams && wanted(16 * (lane & 15u), 16)) {
                format = b.format[4 * wave + q];
                offset = b.offset[4 * wave + q];
            }
        load_block(blocks + offset, format, (s0 >> 4) + (lane & 15u), lo, hi);
        block_texels(format, lo, hi, px, lut);
#pragma unroll
        for (int q = 0; q < 4; q++)   // slot j of the block is its texel zigzag_texel(j): 4 q's quadrant
            *reinterpret_cast<uint4 *>(&tile[band * kTileRow + 20 * (lane & 15u) + 4 * q]) =
                make_uint4(px[zigzag_texel(4 * q)], px[zigzag_texel(4 * q + 1)], px[zigzag_texel(4 * q + 2)],
                           px[zigzag_texel(4 * q + 3)]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; k++) px[k] = tile[k * kTileRow + t + 4 * (t >> 4)];   // (bands without values: not used)
}

// One block per thread; a wave's 64 blocks leave through LDS as 4 KB in a
// row.  The stream is the grid's second index, so its format is one branch
// for the whole workgroup.  Bound by the stores (25.6 MB of texels at 400,009
// slots: 8.2 us, 28.6 with the block's fields found for every texel).
__global__ __launch_bounds__(256) void k_decode(const uint8_t *blocks, BandArgs b, uint64_t nblk, uint32_t *tex)
{
    __shared__ __align__(16) uint32_t s_px[256 * 20];
    __shared__ __align__(8) Bc7Part s_rows[kBc7PartRows];
    const uint32_t t = threadIdx.x, k = blockIdx.y;
    const uint64_t b0 = (uint64_t)blockIdx.x * 256, blk = b0 + t;
    const Bc7LdsLut lut = stage_parts(s_rows);
    uint2 lo, hi;
    load_block(blocks + b.offset[k], b.format[k], blk < nblk ? blk : nblk - 1, lo, hi);
    __syncthreads();
    uint32_t px[16];
    block_texels(b.format[k], lo, hi, px, lut);
#pragma unroll
    for (int q = 0; q < 4; q++)
        *reinterpret_cast<uint4 *>(&s_px[20 * t + 4 * q]) = make_uint4(px[4 * q], px[4 * q + 1], px[4 * q + 2], px[4 * q + 3]);
    __syncthreads();
    uint4 *dst = reinterpret_cast<uint4 *>(tex + (k * nblk + b0) * 16);
    const uint32_t quarters = 4 * (uint32_t)min((uint64_t)256, nblk - b0);
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const uint32_t e = 256 * q + t;
        if (e < quarters) dst[e] = *reinterpret_cast<const uint4 *>(&s_px[20 * (e >> 2) + 4 * (e & 3u)]);
    }
}

// Real SH basis of degree <= 3 in FP32 (3DGS sign convention, k = l^2+l+m).
__device__ __forceinline__ void sh_basis(float x, float y, float z, float (&Y)[16])
{
    const float c0 = 0.28209479177387814f, c1 = 0.4886025119029199f;
    const float c2a = 1.0925484305920792f, c2b = 0.31539156525252005f, c2c = 0.5462742152960396f;
    const float c3a = 0.5900435899266435f, c3b = 2.890611442640554f, c3c = 0.4570457994644658f;
    const float c3d = 0.3731763325901154f, c3e = 1.445305721320277f;
    const float xx = x * x, yy = y * y, zz = z * z;
    Y[0] = c0;
    Y[1] = -c1 * y;
    Y[2] = c1 * z;
    Y[3] = -c1 * x;
    Y[4] = c2a * x * y;
    Y[5] = -c2a * y * z;
    Y[6] = c2b * (2.0f * zz - xx - yy);
    Y[7] = -c2a * x * z;
    Y[8] = c2c * (xx - yy);
    Y[9] = -c3a * y * (3.0f * xx - yy);
    Y[10] = c3b * x * y * z;
    Y[11] = -c3c * y * (4.0f * zz - xx - yy);
    Y[12] = c3d * z * (2.0f * zz - 3.0f * xx - 3.0f * yy);
    Y[13] = -c3c * x * (4.0f * zz - xx - yy);
    Y[14] = c3e * z * (xx - yy);
    Y[15] = -c3a * x * (xx - 3.0f * yy);
}

// decode_eval as a contraction: out[v][3j+c] = sum_k Y[v][k] * H[j][k][c], a
// (directions x 16) by (16 x 3m) product with K = 16.  A workgroup decodes 256
// slots once (one lane each) into an LDS matrix Hm[k][3*slot + c], then its
// four waves compute 16 x 16 output tiles with v_mfma_f32_16x16x4f32 (four
// K-steps each), holding their B operands in registers across the direction
// tiles.  Lane layout of that instruction: lane l supplies A[l%16][l/16] and
// B[l/16][l%16] and receives D[4*(l/16) + r][l%16], r = 0..3.
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kSlots = 256;                 // slots per workgroup
constexpr int kCols = 3 * kSlots;           // output floats per direction
constexpr int kDirChunk = 256;              // directions per workgroup (grid.y), one per thread; their basis rows sit in LDS
static_assert(kDirChunk == kEvalBlock, "a thread makes one direction's basis row");
constexpr int kBasStride = 17;              // padded basis row in LDS
constexpr int kStageStride = 196;           // padded staging row (192 columns per wave)
// SR staging rows per wave: 16 (all rows of a 16-direction tile at once;
// two workgroups per CU) or 8 (the tile in two halves; 49.7 KB of LDS and at
// most 168 VGPRs, so three workgroups per CU).  Three hide the decode
// prologue better and win when a workgroup has few directions to write; at
// hundreds of directions the two-workgroup form writes faster.
template <int SR>
constexpr int lds_floats()
{
    return kDirChunk * kBasStride + 4 * SR * kStageStride > 16 * kCols + 2 * kBc7PartRows
               ? kDirChunk * kBasStride + 4 * SR * kStageStride
               : 16 * kCols + 2 * kBc7PartRows;
}

template <int SR>
__device__ __forceinline__ void decode_eval_body(const uint8_t *blocks, const BandArgs &b, const uint32_t *prim_idx,
                                                 uint64_t m, uint64_t n_prims, const float *dirs, uint32_t n_dirs,
                                                 float *out)
{
    __shared__ __align__(16) float lds[lds_floats<SR>()];
    float(*Hm)[kCols] = reinterpret_cast<float(*)[kCols]>(lds);
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);   // wave-uniform: row addresses stay scalar
    const uint64_t j0 = (uint64_t)blockIdx.x * kSlots;
    const uint32_t vc0 = blockIdx.y * kDirChunk;
    const uint32_t v_end = min(n_dirs, vc0 + kDirChunk);
    // this thread's direction, loaded with the slot's index (each workgroup
    // makes its basis rows: with a launch of their own and their read-back,
    // 1,003 slots x 9 directions took 11.8 us instead of 9.2, 1,048,576 x 64
    // 189 instead of 182)
    const uint32_t vd = min(vc0 + (uint32_t)t, n_dirs - 1);
    const float dir[3] = {dirs[3 * (uint64_t)vd], dirs[3 * (uint64_t)vd + 1], dirs[3 * (uint64_t)vd + 2]};
    // ---- decode: lane t -> slot j0 + t
    {
        const uint64_t j = j0 + t;
        const uint32_t s = j < m ? (prim_idx ? prim_idx[j] : (uint32_t)j) : 0u;
        // BC7 partition table for the decode, in the LDS past Hm (its loads
        // issued with the slot's index load)
        const Bc7LdsLut lut = stage_parts(reinterpret_cast<Bc7Part *>(lds + 16 * kCols));
        __syncthreads();
        // 256 slots in a row: whole blocks, handed over where Hm goes next
        const bool whole = !prim_idx && j0 + kSlots <= min(m, n_prims);
        uint32_t px[16];
        if (whole) {
            slot_texels_tile(blocks, b, j0, reinterpret_cast<uint32_t *>(lds), px, lut, [](uint32_t, int) { return true; });
            __syncthreads();
        }
        float h[16][3];
        if (j < m) {
            if (s < n_prims) {
                if (!whole) slot_texels_batched(blocks, b, s, px, lut);
#pragma unroll
                for (int k = 0; k < 16; k++) {
                    const bool kept = band_coded(b, k);
#pragma unroll
                    for (int c = 0; c < 3; c++) h[k][c] = kept ? dequant(px[k] >> (8 * c), b, k) : 0.0f;
                }
            } else {   // not a slot of this scene: NaN colours, no block access
#pragma unroll
                for (int k = 0; k < 16; k++) h[k][0] = h[k][1] = h[k][2] = __builtin_nanf("");
            }
        } else {
#pragma unroll
            for (int k = 0; k < 16; k++) h[k][0] = h[k][1] = h[k][2] = 0.0f;
        }
#pragma unroll
        for (int k = 0; k < 16; k++) {
            Hm[k][3 * t] = h[k][0];
            Hm[k][3 * t + 1] = h[k][1];
            Hm[k][3 * t + 2] = h[k][2];
        }
    }
    __syncthreads();
    // ---- B operands of this wave's 12 column tiles, held across directions
    const int row = lane >> 4, col = lane & 15;
    float bop[12][4];
#pragma unroll
    for (int q = 0; q < 12; q++) {
        const int c0 = 16 * (wave * 12 + q);
#pragma unroll
        for (int s = 0; s < 4; s++) bop[q][s] = Hm[4 * s + row][c0 + col];
    }
    const uint64_t cols_valid = (m - j0 < (uint64_t)kSlots ? m - j0 : (uint64_t)kSlots) * 3;
    const uint64_t row_stride = 3 * m;
    // rows start 16-byte aligned (output base aligned, row length a multiple of 4 floats)
    const bool rows16 = (row_stride & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    const uint32_t wcol0 = 16 * 12 * wave;                  // this wave's first column
    float *obase = out + 3 * j0 + wcol0;
    // Hm is dead once every wave holds its B operands.  It then holds this
    // workgroup's basis rows (the A operands) and each wave's staging tile,
    // so the direction loop issues no vector-memory loads: on this ISA one
    // counter tracks loads and stores together, and waiting for a load would
    // also wait for every store issued before it.
    float *bas = lds;                                                  // [kDirChunk][kBasStride]
    float(*stage)[kStageStride] = reinterpret_cast<float(*)[kStageStride]>(lds + kDirChunk * kBasStride) + SR * wave;
    float Y[16];
    sh_basis(dir[0], dir[1], dir[2], Y);
    __syncthreads();           // every wave holds its B operands
#pragma unroll
    for (int k = 0; k < 16; k++) bas[t * kBasStride + k] = vc0 + t < v_end ? Y[k] : 0.0f;
    __syncthreads();
    if constexpr (SR == 16) {
        for (uint32_t v0 = vc0; v0 < v_end; v0 += 16) {
            // A operand: Y[v0 + col][4s + row]
            float aop[4];
    #pragma unroll
            for (int s = 0; s < 4; s++) aop[s] = bas[(v0 - vc0 + col) * kBasStride + 4 * s + row];
            // all 12 tiles staged (16 rows x 192 columns), then each row leaves as
            // three back-to-back stores of 64 floats: 768 contiguous bytes
    #pragma unroll
            for (int q = 0; q < 12; q++) {
                floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    #pragma unroll
                for (int s = 0; s < 4; s++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[s], bop[q][s], acc, 0, 0, 0);
    #pragma unroll
                for (int r = 0; r < 4; r++) stage[4 * row + r][16 * q + col] = acc[r];
            }
            bool cok[3];
    #pragma unroll
            for (int h = 0; h < 3; h++) cok[h] = wcol0 + 64 * h + lane < cols_valid;
            float *o = obase + v0 * row_stride + lane;
            if (v0 + 16 <= v_end && wcol0 + 192 <= cols_valid && rows16) {
                // whole rows, every column valid, 16-byte aligned: lanes 0..47
                // store 4 consecutive columns each, one instruction per row
                if (lane < 48) {
                    floatx4 *o4 = reinterpret_cast<floatx4 *>(obase + v0 * row_stride) + lane;
    #pragma unroll
                    for (int half = 0; half < 2; half++) {
                        floatx4 x[8];
    #pragma unroll
                        for (int rr = 0; rr < 8; rr++)
                            x[rr] = *reinterpret_cast<const floatx4 *>(&stage[8 * half + rr][4 * lane]);
    #pragma unroll
                        for (int rr = 0; rr < 8; rr++)
                            __builtin_nontemporal_store(x[rr], o4 + (8 * half + rr) * (row_stride / 4));
                    }
                }
            } else if (v0 + 16 <= v_end) {
    #pragma unroll
                for (int half = 0; half < 2; half++) {
                    float x[8][3];
    #pragma unroll
                    for (int rr = 0; rr < 8; rr++)
    #pragma unroll
                        for (int h = 0; h < 3; h++) x[rr][h] = stage[8 * half + rr][64 * h + lane];
    #pragma unroll
                    for (int rr = 0; rr < 8; rr++)
    #pragma unroll
                        for (int h = 0; h < 3; h++)
                            if (cok[h]) __builtin_nontemporal_store(x[rr][h], o + (8 * half + rr) * row_stride + 64 * h);
                }
            } else {
                for (uint32_t rr = 0; v0 + rr < v_end; rr++)
    #pragma unroll
                    for (int h = 0; h < 3; h++)
                        if (cok[h]) __builtin_nontemporal_store(stage[rr][64 * h + lane], o + rr * row_stride + 64 * h);
            }
            // The four waves start each direction tile together, so their
            // 768-byte pieces of a row leave close in time (one 3 KB stretch
            // of it): a bare s_barrier, which waits on no memory counter.
            // Every wave runs the same iterations (v0 and v_end are uniform
            // over the workgroup); 7.27 -> 7.14 ms at 3,145,728 x 1,024.
            __builtin_amdgcn_s_barrier();
        }
    } else {
        for (uint32_t v0 = vc0; v0 < v_end; v0 += 16) {
            float aop[4];
    #pragma unroll
            for (int s = 0; s < 4; s++) aop[s] = bas[(v0 - vc0 + col) * kBasStride + 4 * s + row];
            floatx4 acc[12];
    #pragma unroll
            for (int q = 0; q < 12; q++) {
                acc[q] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    #pragma unroll
                for (int s = 0; s < 4; s++) acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[s], bop[q][s], acc[q], 0, 0, 0);
            }
            bool cok[3];
    #pragma unroll
            for (int h = 0; h < 3; h++) cok[h] = wcol0 + 64 * h + lane < cols_valid;
            const bool fast = v0 + 16 <= v_end && wcol0 + 192 <= cols_valid && rows16;
            // half hr stages rows 4 i + 2 hr + e (i = 0..3, e = 0, 1) at staging row 2 i + e
    #pragma unroll
            for (int hr = 0; hr < 2; hr++) {
    #pragma unroll
                for (int q = 0; q < 12; q++)
    #pragma unroll
                    for (int e = 0; e < 2; e++) stage[2 * row + e][16 * q + col] = acc[q][2 * hr + e];
                if (fast) {
                    if (lane < 48) {
                        floatx4 *o4 = reinterpret_cast<floatx4 *>(obase + (v0 + 2 * hr) * row_stride) + lane;
    #pragma unroll
                        for (int g = 0; g < 8; g += 4) {
                            floatx4 x[4];
    #pragma unroll
                            for (int e = 0; e < 4; e++) x[e] = *reinterpret_cast<const floatx4 *>(&stage[g + e][4 * lane]);
    #pragma unroll
                            for (int e = 0; e < 4; e++)
                                __builtin_nontemporal_store(x[e], o4 + (4 * ((g + e) >> 1) + ((g + e) & 1)) * (row_stride / 4));
                        }
                    }
                } else {
                    float *o = obase + v0 * row_stride + lane;
                    for (int sr = 0; sr < 8; sr++) {
                        const uint32_t dv = 4 * (sr >> 1) + 2 * hr + (sr & 1);
                        if (v0 + dv < v_end)
    #pragma unroll
                            for (int h = 0; h < 3; h++)
                                if (cok[h]) __builtin_nontemporal_store(stage[sr][64 * h + lane], o + dv * row_stride + 64 * h);
                    }
                }
            }
        }
    }
}

__global__ __launch_bounds__(kEvalBlock) void k_decode_eval(const uint8_t *blocks, BandArgs b,
                                                            const uint32_t *prim_idx, uint64_t m,
                                                            uint64_t n_prims, const float *dirs,
                                                            uint32_t n_dirs, float *out)
{
    decode_eval_body<16>(blocks, b, prim_idx, m, n_prims, dirs, n_dirs, out);
}

__global__ __launch_bounds__(kEvalBlock) __attribute__((amdgpu_waves_per_eu(3))) void k_decode_eval_small(
    const uint8_t *blocks, BandArgs b, const uint32_t *prim_idx, uint64_t m, uint64_t n_prims, const float *dirs,
    uint32_t n_dirs, float *out)
{
    decode_eval_body<8>(blocks, b, prim_idx, m, n_prims, dirs, n_dirs, out);
}

// The 16 basis functions at the direction from slot s's primitive (through
// perm) towards view position f.
__device__ __forceinline__ void view_basis(uint32_t s, const float *pos, const uint32_t *perm, float fx, float fy,
                                           float fz, float (&Y)[16])
{
    const uint64_t pi = perm[s];
    float x = fx - pos[3 * pi], y = fy - pos[3 * pi + 1], z = fz - pos[3 * pi + 2];
    const float r = sqrtf(x * x + y * y + z * z);
    const float inv = r > 0.0f ? 1.0f / r : 0.0f;
    x *= inv;
    y *= inv;
    z *= inv;
    sh_basis(x, y, z, Y);
}

// The decoded, dequantised texels dotted with the basis functions (FP32, k order).
__device__ __forceinline__ void colour_sum(const BandArgs &b, const uint32_t (&px)[16], const float (&Y)[16],
                                           float c[3])
{
    c[0] = c[1] = c[2] = 0.0f;
#pragma unroll
    for (int k = 0; k < 16; k++) {
        if (band_coded(b, k)) {
#pragma unroll
            for (int ch = 0; ch < 3; ch++) c[ch] = fmaf(dequant(px[k] >> (8 * ch), b, k), Y[k], c[ch]);
        }
    }
}

// Colour of slot s seen from view position f (Sec. II, c(f) = H w(f - p)):
// its primitive's position through perm, d = (f - p)/|f - p| (zero when
// f = p), the 16 basis functions dotted with the decoded, dequantised texels
// (FP32, k order).  s must be below the scene's n_prims.
template <class Lut>
__device__ __forceinline__ void view_colour(const uint8_t *blocks, const BandArgs &b, uint32_t s, const float *pos,
                                            const uint32_t *perm, float fx, float fy, float fz, float c[3],
                                            const Lut &lut)
{
    float Y[16];
    view_basis(s, pos, perm, fx, fy, fz, Y);
    uint32_t px[16];
    slot_texels(blocks, b, s, px, lut);
    colour_sum(b, px, Y, c);
}

// The blend's colours first: all slots or the marked ones only (a byte each).
// All are decoded where most will be read and each slot's primitive is known to
// be one of pos (perm below n_prims, which pos holds at least); else only marked
// ones, of which alone the caller answers for perm: lists with less than an entry
// a slot in use (786,432 slots, 0.27 entries each: 59 us against 69), and scenes
// that hold a part of pos's primitives.  From there on marks cost more than
// unlisted slots (3.6 entries each: 319 us against 309; 16.6 M entries of
// 3,145,728 slots 1,525 against 1,393).
__device__ __forceinline__ bool all_slots(const uint32_t *tile_start, uint32_t tiles, uint64_t list_len, uint64_t n_prims,
                                          const uint32_t *odd)
{
    return *odd == 0 && min((uint64_t)tile_start[tiles], list_len) >= n_prims;
}

// Marks (n_marks bytes, a multiple of 16) cleared; *odd is set where a perm entry
// is no number below n_prims.
__global__ __launch_bounds__(256) void k_clear_marks(uint4 *mark, uint64_t n_marks, const uint32_t *perm, uint64_t n_prims,
                                                     uint32_t *odd)
{
    const uint64_t e0 = (uint64_t)blockIdx.x * 256;
    if (e0 + threadIdx.x < n_marks / 16) mark[e0 + threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
    bool bad = false;
#pragma unroll
    for (uint32_t q = 0; q < 16; q++) {
        const uint64_t s = 16 * e0 + 256 * q + threadIdx.x;
        bad |= s < n_prims && perm[min(s, n_prims - 1)] >= n_prims;
    }
    if (bad) *odd = 1;
}

// One lane per listed slot; out-of-range slot ids give NaN.  MARKED: all slots,
// or those with a mark (see all_slots): then nothing of the others is read,
// neither their blocks nor their perm entries and positions, and their colours
// are left as they are or NaN.
template <bool MARKED>
__global__ __launch_bounds__(256) void k_decode_eval_view(const uint8_t *blocks, BandArgs b, const uint32_t *prim_idx,
                                                          const uint8_t *mark, const uint32_t *odd,
                                                          const uint32_t *tile_start, uint32_t tiles, uint64_t list_len,
                                                          uint64_t m, uint64_t n_prims, const float *pos,
                                                          const uint32_t *perm, float fx, float fy, float fz,
                                                          float *out)
{
    __shared__ __align__(16) uint32_t s_tile[kTileWords];
    __shared__ __align__(8) Bc7Part s_rows[kBc7PartRows];
    __shared__ uint64_t s_marks[4];
    const uint64_t j0 = (uint64_t)blockIdx.x * 256, j = j0 + threadIdx.x;
    bool mine = j < m;
    if (MARKED) {
        mine = mine && (all_slots(tile_start, tiles, list_len, n_prims, odd) || mark[j] != 0);
        const uint64_t marks = __ballot(mine);
        if ((threadIdx.x & 63u) == 0) s_marks[threadIdx.x >> 6] = marks;
        if (!__syncthreads_or(mine)) return;
    }
    const Bc7LdsLut lut = stage_parts(s_rows);
    __syncthreads();
    float c[3] = {__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf("")};
    if (!prim_idx && j0 + 256 <= min(m, n_prims)) {   // 256 slots in a row: whole blocks
        float Y[16];
        if (mine) view_basis((uint32_t)j, pos, perm, fx, fy, fz, Y);
        uint32_t px[16];
        slot_texels_tile(blocks, b, j0, s_tile, px, lut, [&](uint32_t i, int k) {
            return !MARKED || ((s_marks[i >> 6] >> (i & 63u)) & ((1ull << k) - 1u)) != 0;
        });
        if (mine) colour_sum(b, px, Y, c);
    } else if (mine) {
        const uint32_t s = prim_idx ? prim_idx[j] : (uint32_t)j;
        if (s < n_prims) view_colour(blocks, b, s, pos, perm, fx, fy, fz, c, lut);
    }
    if (j >= m || (MARKED && __ballot(mine) == 0)) return;
    out[3 * j] = c[0];
    out[3 * j + 1] = c[1];
    out[3 * j + 2] = c[2];
}

// Tiles by decreasing list length (bucketed by floor(log2 L), empty tiles
// last): one workgroup counts, scans and scatters.  The blend takes tiles
// in this order so that the longest lists start first instead of ending
// the launch alone; the order within a bucket does not matter (each tile is
// computed on its own).  Workgroup 0 does that.  The others, where there are
// any, set a mark on every slot that their tile's list names (ids past the scene
// have none) unless all slots' colours are wanted.  Bound by the marks' scattered
// byte stores (16.6 M entries 121 us with eight loads of the list in flight per
// lane, 180 with one and 256 lanes a tile).
__global__ __launch_bounds__(1024) void k_tile_order(const uint32_t *tile_start, const uint32_t *list, uint64_t list_len,
                                                    uint32_t tiles, uint32_t *order, uint64_t n_prims, uint8_t *mark,
                                                    const uint32_t *odd)
{
    __shared__ uint32_t cnt[33];
    const uint32_t t = threadIdx.x;
    if (blockIdx.x) {
        if (all_slots(tile_start, tiles, list_len, n_prims, odd)) return;
        const uint32_t tile = blockIdx.x - 1;
        const uint64_t b1 = min((uint64_t)tile_start[tile + 1], list_len);
        const uint64_t b0 = min((uint64_t)tile_start[tile], b1);
        constexpr int kLoads = 8;   // in flight per lane
        for (uint64_t base = b0 + t; base < b1; base += 1024 * kLoads) {
            uint32_t s[kLoads];
#pragma unroll
            for (int q = 0; q < kLoads; q++) s[q] = list[min(base + 1024 * q, b1 - 1)];
#pragma unroll
            for (int q = 0; q < kLoads; q++)
                if (s[q] < n_prims) mark[s[q]] = 1;
        }
        return;
    }
    if (t < 33) cnt[t] = 0u;
    __syncthreads();
    auto key = [&](uint32_t i) {
        const uint64_t e = min((uint64_t)tile_start[i + 1], list_len), s0 = min((uint64_t)tile_start[i], e);
        const uint64_t L = e - s0;
        return L == 0 ? 32u : (uint32_t)__clzll(L) - 32u;   // 31 - floor(log2 L) for L below 2^32
    };
    for (uint32_t i = t; i < tiles; i += 1024) atomicAdd(&cnt[key(i)], 1u);
    __syncthreads();
    if (t == 0) {
        uint32_t run = 0;
        for (int k = 0; k < 33; k++) {
            const uint32_t c = cnt[k];
            cnt[k] = run;
            run += c;
        }
    }
    __syncthreads();
    for (uint32_t i = t; i < tiles; i += 1024) order[atomicAdd(&cnt[key(i)], 1u)] = i;
}

// Colour stage of a tile rasteriser (Sec. II, eq. preblend with the
// premultiplied coefficients of eq. premult), one workgroup per 16x16 tile,
// one lane per pixel.  The tile's list is taken 256 entries at a time: lane t
// stages entry t in LDS with its colour c~ = Htilde w(f - p) (read where it
// was computed beforehand, else decoded here from the bitstreams), the
// primitive's footprint and opacity mu, the conic turned into base-2 exponent
// coefficients (A, B, C) = -log2(e) (a/2, b, c/2); then every pixel walks the
// staged entries front to back: g = 2^(A dx^2 + B dx dy + C dy^2) at its
// centre, w = g T, a += w c~, T -= mu w.  A list entry past n_prims gives NaN
// colour.  Once every pixel of a wave (or of the tile) has T exactly 0, the
// remaining entries change nothing (w = 0 and T stays 0 for finite colours)
// and are skipped.
// Bound by the issue of the walk's instructions.  Apart from the decode's
// registers and with T mu not formed by itself, colours and blend of a
// 1920 x 1088 frame (16.5 M entries) 1,293 -> 1,270 us.  Two and four pixels
// per lane, which share dx and the LDS reads, took 1,326 and 1,545: a tile's
// waves are then fewer and its walk longer.  The decoding kernel takes short
// lists only: blocks decoded as they arrive and the partition table in constant
// memory start sooner than 16 loads ahead and a copy in LDS (lists of 0.02
// entries a slot, 786,432 slots: 28 against 42 us).
template <bool COLOURS>
__global__ __launch_bounds__(256) void k_blend_tiles(const uint8_t *blocks, BandArgs b, uint64_t n_prims,
                                                     const float *pos, const uint32_t *perm, float fx, float fy,
                                                     float fz, const float *mu, const float *foot,
                                                     const uint32_t *tile_start, const uint32_t *list,
                                                     uint64_t list_len, const uint32_t *order, uint32_t tiles_x,
                                                     const float *colours, uint32_t *odd, float *image, float *trans)
{
    if (COLOURS && odd && blockIdx.x == 0 && threadIdx.x == 0) *odd = 0;   // for the next call
    // per staged entry: mean x, mean y, A, B | C, mu, colour r, g | colour b
    // (rows of 12 floats: three 16-byte LDS reads per entry, all lanes
    // reading the same row)
    __shared__ __align__(16) float s_par[256][12];
    const uint32_t t = threadIdx.x, tile = order[blockIdx.x];
    const uint32_t tx = tile % tiles_x, ty = tile / tiles_x;
    const float x = (float)(16 * tx + (t & 15u)) + 0.5f, y = (float)(16 * ty + (t >> 4)) + 0.5f;
    const uint64_t b1 = min((uint64_t)tile_start[tile + 1], list_len);
    const uint64_t b0 = min((uint64_t)tile_start[tile], b1);
    constexpr float kLog2e = 1.4426950408889634f;
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, T = 1.0f;
    for (uint64_t base = b0; base < b1; base += 256) {
        const uint64_t e = base + t;
        if (e < b1) {
            const uint32_t s = list[e];
            float c[3] = {__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf("")};
            uint64_t i = 0;
            if (s < n_prims) {
                if constexpr (COLOURS) {   // the colour computed beforehand, once per primitive
                    c[0] = colours[3 * (uint64_t)s];
                    c[1] = colours[3 * (uint64_t)s + 1];
                    c[2] = colours[3 * (uint64_t)s + 2];
                } else {
                    view_colour(blocks, b, s, pos, perm, fx, fy, fz, c, Bc7ConstLut{});
                }
                i = perm[s];
            }
            s_par[t][0] = foot[5 * i];
            s_par[t][1] = foot[5 * i + 1];
            s_par[t][2] = -0.5f * kLog2e * foot[5 * i + 2];
            s_par[t][3] = -kLog2e * foot[5 * i + 3];
            s_par[t][4] = -0.5f * kLog2e * foot[5 * i + 4];
            s_par[t][5] = mu[i];
            s_par[t][6] = c[0];
            s_par[t][7] = c[1];
            s_par[t][8] = c[2];
        }
        __syncthreads();
        const uint32_t cnt = (uint32_t)(b1 - base < 256 ? b1 - base : 256);
        for (uint32_t j0 = 0; j0 < cnt; j0 += 32) {
            if (__all(T == 0.0f)) break;   // this wave is done for the chunk
            const uint32_t j1 = j0 + 32 < cnt ? j0 + 32 : cnt;
            // four entries' reads in flight at once
#pragma unroll 4
            for (uint32_t j = j0; j < j1; j++) {
                const float4 pa = *reinterpret_cast<const float4 *>(&s_par[j][0]);
                const float4 pb = *reinterpret_cast<const float4 *>(&s_par[j][4]);
                const float blue = s_par[j][8];
                const float dx = x - pa.x, dy = y - pa.y;
                const float ex = fmaf(dx, fmaf(pa.z, dx, pa.w * dy), pb.x * dy * dy);
                const float g = __builtin_amdgcn_exp2f(ex);
                const float w = g * T;
                a0 = fmaf(w, pb.z, a0);
                a1 = fmaf(w, pb.w, a1);
                a2 = fmaf(w, blue, a2);
                T = fmaf(-pb.y, w, T);
            }
        }
        if (__syncthreads_and(T == 0.0f)) break;   // every pixel of the tile is covered
    }
    const uint64_t W = 16 * (uint64_t)tiles_x;
    const uint64_t o = (16 * (uint64_t)ty + (t >> 4)) * W + 16 * tx + (t & 15u);
    image[3 * o] = a0;
    image[3 * o + 1] = a1;
    image[3 * o + 2] = a2;
    if (trans) trans[o] = T;
}

}  // namespace

hipError_t launch_blend_tiles(const uint8_t *blocks, const BandArgs &b, uint64_t n_prims, const float *pos,
                              const uint32_t *perm, const float view[3], const float *mu, const float *foot,
                              const uint32_t *tile_start, const uint32_t *list, uint64_t list_len, uint32_t tiles_x,
                              uint32_t tiles_y, const float *colours, float *image, float *trans, uint32_t *order,
                              float *fill_colours, uint8_t *marks, uint32_t *odd, hipStream_t st)
{
    const uint64_t tiles = (uint64_t)tiles_x * tiles_y;
    if (tiles == 0) return hipSuccess;
    const uint64_t n_marks = (n_prims + 15) / 16 * 16;
    if (fill_colours)
        GSBC_LAUNCH("clear_marks", k_clear_marks, dim3((uint32_t)((n_marks / 16 + 255) / 256)), dim3(256), 0, st,
                    reinterpret_cast<uint4 *>(marks), n_marks, perm, n_prims, odd);
    GSBC_LAUNCH("tile_order", k_tile_order, dim3(fill_colours ? 1 + (uint32_t)tiles : 1), dim3(1024), 0, st, tile_start, list,
                list_len, (uint32_t)tiles, order, n_prims, marks, odd);
    if (fill_colours) {
        GSBC_LAUNCH("decode_eval_view", k_decode_eval_view<true>, dim3((uint32_t)((n_prims + 255) / 256)), dim3(256), 0, st,
                    blocks, b, nullptr, marks, odd, tile_start, (uint32_t)tiles, list_len, n_prims, n_prims, pos, perm, view[0],
                    view[1], view[2], fill_colours);
        colours = fill_colours;
    }
    GSBC_LAUNCH("blend_tiles", colours ? k_blend_tiles<true> : k_blend_tiles<false>, dim3((uint32_t)tiles), dim3(256), 0,
                st, blocks, b, n_prims, pos, perm, view[0], view[1], view[2], mu, foot, tile_start, list, list_len, order,
                tiles_x, colours, fill_colours ? odd : nullptr, image, trans);
    return hipGetLastError();
}

hipError_t launch_decode_eval_view(const uint8_t *blocks, const BandArgs &b, uint64_t n_prims, const float *pos,
                                   const uint32_t *perm, const float view[3], const uint32_t *prim_idx, uint64_t m,
                                   float *out, hipStream_t st)
{
    if (m == 0) return hipSuccess;
    GSBC_LAUNCH("decode_eval_view", k_decode_eval_view<false>, dim3((uint32_t)((m + 255) / 256)), dim3(256), 0, st, blocks, b,
                prim_idx, nullptr, nullptr, nullptr, 0u, 0ull, m, n_prims, pos, perm, view[0], view[1], view[2], out);
    return hipGetLastError();
}

hipError_t launch_decode(const uint8_t *blocks, const BandArgs &b, uint64_t nblk, uint8_t *textures,
                         hipStream_t st)
{
    if (nblk == 0 || b.n_streams == 0) return hipSuccess;
    GSBC_LAUNCH("decode", k_decode, dim3((uint32_t)((nblk + 255) / 256), b.n_streams), dim3(256), 0, st, blocks, b,
                nblk, reinterpret_cast<uint32_t *>(textures));
    return hipGetLastError();
}

hipError_t launch_decode_eval(const uint8_t *blocks, const BandArgs &b, uint64_t n_prims, const float *dirs,
                              uint32_t n_dirs, const uint32_t *prim_idx, uint64_t m, float *out, hipStream_t st)
{
    if (m == 0 || n_dirs == 0) return hipSuccess;
    dim3 grid((uint32_t)((m + kSlots - 1) / kSlots), (n_dirs + kDirChunk - 1) / kDirChunk);
    if (n_dirs <= (uint32_t)kDirChunk)   // one direction chunk per workgroup: three workgroups per CU
        GSBC_LAUNCH("decode_eval", k_decode_eval_small, grid, dim3(kEvalBlock), 0, st, blocks, b, prim_idx, m,
                    n_prims, dirs, n_dirs, out);
    else
        GSBC_LAUNCH("decode_eval", k_decode_eval, grid, dim3(kEvalBlock), 0, st, blocks, b, prim_idx, m, n_prims,
                    dirs, n_dirs, out);
    return hipGetLastError();
}

}  // namespace gsbc
