// bc_format.h -- BC1 / BC7 format constants and texel decoders for the
// gfx950 kernels (D3D11 BC1 and BC7 block formats, the fixed-rate BTC
// schemes of Sec. III-A/B of Said & Rauwendaal).
//
// The BC7 partition maps and anchor texels are transcribed from the public
// BC7/BPTC format specification.  2-subset maps are 16-bit masks (bit i =
// subset of texel i); 3-subset maps are packed at compile time from their
// row strings into 2 bits per texel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gsbc {

// ------------------------------------------------------------------ BC7 modes
struct Bc7Mode {
    int ns;        // subsets
    int partbits;  // partition field width
    int rotbits;   // rotation field width
    int selbits;   // index-selection field width
    int cb;        // colour endpoint bits per channel
    int ab;        // alpha endpoint bits (0: none)
    int pb;        // p-bits: 0 none, 1 one per subset, 2 one per endpoint
    int ib;        // primary index bits
    int ib2;       // secondary index bits (0: none)
};

__host__ __device__ constexpr Bc7Mode bc7_mode(int m)
{
    return m == 0 ? Bc7Mode{3, 4, 0, 0, 4, 0, 2, 3, 0}
         : m == 1 ? Bc7Mode{2, 6, 0, 0, 6, 0, 1, 3, 0}
         : m == 2 ? Bc7Mode{3, 6, 0, 0, 5, 0, 0, 2, 0}
         : m == 3 ? Bc7Mode{2, 6, 0, 0, 7, 0, 2, 2, 0}
         : m == 4 ? Bc7Mode{1, 0, 2, 1, 5, 6, 0, 2, 3}
         : m == 5 ? Bc7Mode{1, 0, 2, 0, 7, 8, 0, 2, 2}
         : m == 6 ? Bc7Mode{1, 0, 0, 0, 7, 7, 2, 4, 0}
                  : Bc7Mode{2, 6, 0, 0, 5, 5, 2, 2, 0};
}

// Interpolation weight of index i with n index bits: round(64 i / (2^n - 1)).
__host__ __device__ constexpr int bc7_weight(int n, int i)
{
    return (128 * i + ((1 << n) - 1)) / (2 * ((1 << n) - 1));
}

// The same weights for n and i known only at run time (the decoders), by one
// multiply-add and a shift: (i * bc7_weight_step(n) + 128) >> 8.
__host__ __device__ constexpr uint32_t bc7_weight_step(int n) { return n == 2 ? 5461u : n == 3 ? 2341u : 1092u; }

__host__ __device__ constexpr bool bc7_weight_steps_ok()
{
    for (int n = 2; n <= 4; n++)
        for (uint32_t i = 0; i < (1u << n); i++)
            if ((int)((i * bc7_weight_step(n) + 128u) >> 8) != bc7_weight(n, (int)i)) return false;
    return true;
}
static_assert(bc7_weight_steps_ok(), "BC7 weights by one multiply-add");

__host__ __device__ constexpr int interp64(int e0, int e1, int w)
{
    return ((64 - w) * e0 + w * e1 + 32) >> 6;
}

// Expand an n-bit value (5 <= n <= 8) to 8 bits by replicating its top bits.
__host__ __device__ constexpr int expand_bits(int v, int n)
{
    return n >= 8 ? v : (v << (8 - n)) | (v >> (2 * n - 8));
}

// ------------------------------------------------------------ partition maps
constexpr uint16_t kPart2[64] = {
    0xCCCC, 0x8888, 0xEEEE, 0xECC8, 0xC880, 0xFEEC, 0xFEC8, 0xEC80,
    0xC800, 0xFFEC, 0xFE80, 0xE800, 0xFFE8, 0xFF00, 0xFFF0, 0xF000,
    0xF710, 0x008E, 0x7100, 0x08CE, 0x008C, 0x7310, 0x3100, 0x8CCE,
    0x088C, 0x3110, 0x6666, 0x366C, 0x17E8, 0x0FF0, 0x718E, 0x399C,
    0xAAAA, 0xF0F0, 0x5A5A, 0x33CC, 0x3C3C, 0x55AA, 0x9696, 0xA55A,
    0x73CE, 0x13C8, 0x324C, 0x3BDC, 0x6996, 0xC33C, 0x9966, 0x0660,
    0x0272, 0x04E4, 0x4E40, 0x2720, 0xC936, 0x936C, 0x39C6, 0x639C,
    0x9336, 0x9CC6, 0x817E, 0xE718, 0xCCF0, 0x0FCC, 0x7744, 0xEE22,
};

__host__ __device__ constexpr uint32_t pack_row3(const char *r)
{
    uint32_t v = 0;
    for (int i = 0; i < 16; i++) v |= (uint32_t)(r[i] - '0') << (2 * i);
    return v;
}

// (constexpr: the encoder plans its visiting order from it at compile time)
constexpr uint32_t kPart3[64] = {
    pack_row3("0011001102212222"), pack_row3("0001001122112221"), pack_row3("0000200122112211"),
    pack_row3("0222002200110111"), pack_row3("0000000011221122"), pack_row3("0011001100220022"),
    pack_row3("0022002211111111"), pack_row3("0011001122112211"), pack_row3("0000000011112222"),
    pack_row3("0000111111112222"), pack_row3("0000111122222222"), pack_row3("0012001200120012"),
    pack_row3("0112011201120112"), pack_row3("0122012201220122"), pack_row3("0011011211221222"),
    pack_row3("0011200122002220"), pack_row3("0001001101121122"), pack_row3("0111001120012200"),
    pack_row3("0000112211221122"), pack_row3("0022002200221111"), pack_row3("0111011102220222"),
    pack_row3("0001000122212221"), pack_row3("0000001101220122"), pack_row3("0000110022102210"),
    pack_row3("0122012200110000"), pack_row3("0012001211222222"), pack_row3("0110122112210110"),
    pack_row3("0000011012211221"), pack_row3("0022110211020022"), pack_row3("0110011020022222"),
    pack_row3("0011012201220011"), pack_row3("0000200022112221"), pack_row3("0000000211221222"),
    pack_row3("0222002200120011"), pack_row3("0011001200220222"), pack_row3("0120012001200120"),
    pack_row3("0000111122220000"), pack_row3("0120120120120120"), pack_row3("0120201212010120"),
    pack_row3("0011220011220011"), pack_row3("0011112222000011"), pack_row3("0101010122222222"),
    pack_row3("0000000021212121"), pack_row3("0022112200221122"), pack_row3("0022001100220011"),
    pack_row3("0220122102201221"), pack_row3("0101222222220101"), pack_row3("0000212121212121"),
    pack_row3("0101010101012222"), pack_row3("0222011102220111"), pack_row3("0002111200021112"),
    pack_row3("0000211221122112"), pack_row3("0222011101110222"), pack_row3("0002111211120002"),
    pack_row3("0110011001102222"), pack_row3("0000000021122112"), pack_row3("0110011022222222"),
    pack_row3("0022001100110022"), pack_row3("0022112211220022"), pack_row3("0000000000002112"),
    pack_row3("0002000100020001"), pack_row3("0222122202221222"), pack_row3("0101222222222222"),
    pack_row3("0111201122012220"),
};

// Anchor texel of the second subset (2-subset partitions), and of the second
// and third subsets (3-subset partitions).  Subset 0's anchor is texel 0.
constexpr uint8_t kAnchor2[64] = {
    15, 15, 15, 15, 15, 15, 15, 15, 15, 15, 15, 15, 15, 15, 15, 15,
    15, 2, 8, 2, 2, 8, 8, 15, 2, 8, 2, 2, 8, 8, 2, 2,
    15, 15, 6, 8, 2, 8, 15, 15, 2, 8, 2, 2, 2, 15, 15, 6,
    6, 2, 6, 8, 15, 15, 2, 2, 15, 15, 15, 15, 15, 2, 2, 15,
};
constexpr uint8_t kAnchor3b[64] = {
    3, 3, 15, 15, 8, 3, 15, 15, 8, 8, 6, 6, 6, 5, 3, 3,
    3, 3, 8, 15, 3, 3, 6, 10, 5, 8, 8, 6, 8, 5, 15, 15,
    8, 15, 3, 5, 6, 10, 8, 15, 15, 3, 15, 5, 15, 15, 15, 15,
    3, 15, 5, 5, 5, 8, 5, 10, 5, 10, 8, 13, 15, 12, 3, 3,
};
constexpr uint8_t kAnchor3c[64] = {
    15, 8, 8, 3, 15, 15, 3, 8, 15, 15, 15, 15, 15, 15, 15, 8,
    15, 8, 15, 3, 15, 8, 15, 8, 3, 15, 6, 10, 15, 15, 10, 8,
    15, 3, 15, 10, 10, 8, 9, 10, 6, 15, 8, 15, 3, 6, 6, 8,
    15, 3, 15, 15, 15, 15, 15, 15, 15, 15, 15, 15, 3, 15, 15, 8,
};

// One row of the decoders' partition table: the subset of each texel at 2
// bits a texel and a bit for each anchor texel.  Rows 0..63 are the 2-subset
// partitions, 64..127 the 3-subset ones, 128 the single subset.
struct Bc7Part {
    uint32_t map, anchors;
};
constexpr int kBc7PartRows = 129;
struct Bc7PartTable {
    Bc7Part row[kBc7PartRows];
};

constexpr Bc7PartTable bc7_part_table()
{
    Bc7PartTable t{};
    for (int p = 0; p < 64; p++) {
        for (int i = 0; i < 16; i++) t.row[p].map |= (uint32_t)((kPart2[p] >> i) & 1) << (2 * i);
        t.row[p].anchors = 1u | 1u << kAnchor2[p];
        t.row[64 + p] = Bc7Part{kPart3[p], 1u | 1u << kAnchor3b[p] | 1u << kAnchor3c[p]};
    }
    t.row[128] = Bc7Part{0u, 1u};
    return t;
}
static __constant__ __align__(8) Bc7PartTable kBc7Parts = bc7_part_table();

// Access to the table for the decoders: in constant memory, or a workgroup's
// copy in LDS (Bc7LdsLut), whose per-lane lookups wait on LDS instead of on
// the vector-memory counter that loads and stores share.
struct Bc7ConstLut {
    __device__ Bc7Part row(uint32_t e) const { return kBc7Parts.row[e]; }
};

struct Bc7LdsLut {
    const Bc7Part *rows;   // kBc7PartRows of them
    __device__ Bc7Part row(uint32_t e) const { return rows[e]; }
};

// Anchor texel of subset s.
__device__ inline int bc7_anchor(int ns, int p, int s)
{
    if (s == 0) return 0;
    if (ns == 2) return kAnchor2[p];
    return s == 1 ? kAnchor3b[p] : kAnchor3c[p];
}

// A 128-bit block held as two little-endian 64-bit halves.
struct Blk128 {
    uint64_t lo, hi;
};

// ------------------------------------------------------------- BC1 decode
__device__ inline void bc1_expand(uint32_t c, int e[3])
{
    int r5 = (c >> 11) & 31, g6 = (c >> 5) & 63, b5 = c & 31;
    e[0] = (r5 << 3) | (r5 >> 2);
    e[1] = (g6 << 2) | (g6 >> 4);
    e[2] = (b5 << 3) | (b5 >> 2);
}

// The decoders' arithmetic is bound by instruction issue (a colour of one
// primitive takes 16 texels), so it is written for the instructions that do
// several steps at once: a byte permute looks up a per-mode constant or packs
// channels, a funnel shift cuts a field at a position that differs from lane
// to lane, and a two-way 16-bit dot product interpolates a channel.  The
// gathers of 1,003 listed slots and of the fused colour stage took 26 and 1,248
// us by shifts and masks of 64 bits, by these 19 and 909.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Low word of (hi:lo) >> n, 0 <= n < 32.
__device__ inline uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t n) { return __builtin_amdgcn_alignbit(hi, lo, n); }

// n bits of x from bit `at` (both below 32).
__device__ inline uint32_t bits(uint32_t x, uint32_t at, uint32_t n) { return __builtin_amdgcn_ubfe(x, at, n); }

// Halves of e times halves of w, summed, plus c.
__device__ inline uint32_t dot2(uint32_t e, uint32_t w, uint32_t c)
{
    return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, e), __builtin_bit_cast(u16x2, w), c, false);
}

// Four bytes of (hi:lo), one per selector byte: 0..3 of lo, 4..7 of hi, 0x0C zero.
__device__ inline uint32_t bytes(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

// ------------------------------------------------------------- BC1 palette
// A block's endpoints as pairs (first | second << 16) per channel, and the
// weights of its four colours: colour = (pair . weights + 1) mult >> 16, with
// mult 1/3 or 1/2 (exact for the sums that occur, below 767; the pure
// endpoints come out as (3 e + 1) / 3 and (2 e + 1) / 2, rounded down).
struct Bc1Head {
    uint32_t r, g, b, first, second, mult;
    bool three;
};

__device__ inline Bc1Head bc1_head(uint32_t w0)
{
    Bc1Head h;
    const uint32_t r5 = (w0 >> 11) & 0x001F001Fu, g6 = (w0 >> 5) & 0x003F003Fu, b5 = w0 & 0x001F001Fu;
    h.r = r5 << 3 | ((r5 >> 2) & 0x00070007u);
    h.g = g6 << 2 | ((g6 >> 4) & 0x00030003u);
    h.b = b5 << 3 | ((b5 >> 2) & 0x00070007u);
    h.three = (w0 & 0xFFFFu) <= (w0 >> 16);   // two endpoints, their mean and transparent black
    h.first = h.three ? 0x00010002u : 0x01020003u;    // byte k: weight of the first endpoint in colour k
    h.second = h.three ? 0x00010200u : 0x02010300u;
    h.mult = h.three ? 32768u : 21846u;
    return h;
}

__device__ inline uint32_t bc1_colour(const Bc1Head &h, uint32_t k)
{
    const uint32_t w = bytes(h.second, h.first, __umul24(k, 0x00010001u) + 0x0C040C00u);
    const uint32_t r = __umul24(dot2(h.r, w, 1u), h.mult), g = __umul24(dot2(h.g, w, 1u), h.mult),
                   b = __umul24(dot2(h.b, w, 1u), h.mult);
    // each channel in byte 2 of its product; alpha 255, or 0 for transparent black
    const uint32_t alpha = h.three && k == 3u ? 0u : 0xFF000000u;
    return bytes(g, r, 0x0C0C0602u) | (b & 0x00FF0000u) | alpha;
}

// Texel i of a BC1 block given as two 32-bit words; RGBA packed in a uint32
// (R in the low byte).
__device__ inline uint32_t bc1_texel(uint32_t w0, uint32_t w1, int i)
{
    return bc1_colour(bc1_head(w0), (w1 >> (2 * i)) & 3u);
}

// All 16 texels.
__device__ inline void bc1_block(uint32_t w0, uint32_t w1, uint32_t (&px)[16])
{
    const Bc1Head h = bc1_head(w0);
    uint32_t pal[4];
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) pal[k] = bc1_colour(h, k);
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const bool b0 = (w1 >> (2 * i)) & 1u, b1 = (w1 >> (2 * i + 1)) & 1u;
        const uint32_t lo = b0 ? pal[1] : pal[0], hi = b0 ? pal[3] : pal[2];
        px[i] = b1 ? hi : lo;
    }
}

// ------------------------------------------------------------- BC7 decode
// Bit positions of a mode's fields: colour endpoints (channel by channel,
// each all its endpoints in order), alpha endpoints, p-bits, first and second
// index.
struct Bc7Layout {
    int colour, alpha, pbits, index, index2;
};

constexpr Bc7Layout bc7_layout(int m)
{
    const Bc7Mode d = bc7_mode(m);
    const int colour = m + 1 + d.partbits + d.rotbits + d.selbits;
    const int alpha = colour + 6 * d.ns * d.cb;
    const int pbits = alpha + 2 * d.ns * d.ab;
    const int index = pbits + d.pb * d.ns;
    return Bc7Layout{colour, alpha, pbits, index, index + 16 * d.ib - d.ns};
}

// One constant per mode, mode m in byte m.
template <class F>
constexpr uint64_t bc7_by_mode(F f)
{
    uint64_t v = 0;
    for (int m = 0; m < 8; m++) v |= (uint64_t)(uint8_t)f(m) << (8 * m);
    return v;
}

// What the decoders below rely on.
constexpr bool bc7_layout_ok()
{
    for (int m = 0; m < 8; m++) {
        const Bc7Mode d = bc7_mode(m);
        const Bc7Layout l = bc7_layout(m);
        // the first channel of any subset starts in the first word, a channel's endpoints span at most 30 bits
        if (l.colour + 2 * (d.ns - 1) * d.cb >= 32 || 2 * d.ns * d.cb > 30) return false;
        // alpha endpoints: within words 1 and 2, in mode 7 within words 2 and 3
        if (d.ab && (l.alpha < (m == 7 ? 64 : 32) || l.alpha >= (m == 7 ? 96 : 64) || 2 * d.ns * d.ab > 20)) return false;
        // p-bits within words 2 and 3, in mode 6 the last bit of word 1 and the first of word 2
        if (d.pb && (m == 6 ? l.pbits != 63 : (l.pbits < 64 || l.pbits >= 96))) return false;
        // indices within the upper half, in mode 4 the first within words 1 and 2
        if (m == 4 ? (l.index < 32 || l.index2 > 96) : l.index < 64) return false;
        if (d.ib2 && (l.index2 < 64 || l.index2 + 16 * d.ib2 - 1 != 128)) return false;
        if (!d.ib2 && l.index2 != 128) return false;
    }
    return true;
}
static_assert(bc7_layout_ok(), "BC7 field positions");

// A block's mode and the fields that all its texels share.
struct Bc7Head {
    uint32_t sel;              // byte-permute selector of the mode: m in the low byte, the others zero
    uint32_t m;
    uint32_t cb, ab, hp;       // endpoint bits; 1 with p-bits
    uint32_t up, down, aup, adown;   // an n-bit code's expansion to 8 bits: << 8 - n, | >> 2 n - 8
    uint32_t amask;            // 255 in both halves without stored alpha
    uint32_t rot;              // the last permute: (B, A):(R, G) to the rotated texel, all zero in the reserved mode
    uint32_t ib, ib2, step, step2;   // index bits and weight steps
    uint32_t ibase, ibase2;    // first bit of the indices in iw:iv and w3:w2
    uint32_t iv, iw;
    bool swap, second;         // colour takes the second index; alpha takes the second index
    Bc7Part part;
};

#define GSBC_BY_MODE(expr) [&] { constexpr uint64_t t = bc7_by_mode([](int m) { \
        [[maybe_unused]] const Bc7Mode d = bc7_mode(m); \
        [[maybe_unused]] const Bc7Layout l = bc7_layout(m); \
        return (expr); }); \
        return bytes((uint32_t)(t >> 32), (uint32_t)t, h.sel); }()

template <class Lut>
__device__ inline Bc7Head bc7_head(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, const Lut &lut)
{
    Bc7Head h;
    const bool reserved = (w0 & 255u) == 0u;   // no mode bit: every texel zero (the fields are read as mode 7's)
    h.m = (uint32_t)__builtin_ctz(w0 | 0x80u);
    h.sel = h.m | 0x0C0C0C00u;
    const uint32_t after = w0 >> (h.m + 1u);
    // row of the partition table
    const uint32_t row = GSBC_BY_MODE(d.ns == 1 ? 128 : d.ns == 3 ? 64 : 0) + (after & GSBC_BY_MODE((1 << d.partbits) - 1));
    h.part = lut.row(row);
    const uint32_t rot = after & GSBC_BY_MODE(d.rotbits ? 3 : 0);
    h.rot = rot == 0u ? 0x05040100u : rot == 1u ? 0x00040105u : rot == 2u ? 0x01040500u : 0x04050100u;
    if (reserved) h.rot = 0x0C0C0C0Cu;
    h.cb = GSBC_BY_MODE(d.cb);
    h.ab = GSBC_BY_MODE(d.ab);
    h.hp = GSBC_BY_MODE(d.pb ? 1 : 0);
    const uint32_t n = h.cb + h.hp, an = h.ab + h.hp;
    h.up = 8u - n;
    h.down = 2u * n - 8u;
    h.amask = h.ab ? 0u : 0x00FF00FFu;
    h.aup = h.ab ? 8u - an : 0u;
    h.adown = h.ab ? 2u * an - 8u : 0u;
    const bool four = h.m == 4u;
    h.ib = GSBC_BY_MODE(d.ib);
    h.ib2 = GSBC_BY_MODE(d.ib2);
    h.step = h.m == 6u ? bc7_weight_step(4) : h.m < 2u ? bc7_weight_step(3) : bc7_weight_step(2);
    h.step2 = four ? bc7_weight_step(3) : bc7_weight_step(2);
    h.ibase = GSBC_BY_MODE(m == 4 ? l.index - 32 : l.index - 64);
    h.ibase2 = GSBC_BY_MODE(d.ib2 ? l.index2 - 64 : 0);
    h.iv = four ? w1 : w2;
    h.iw = four ? w2 : w3;
    h.swap = four && (w0 & 0x80u);             // mode 4's index selection bit
    h.second = h.ib2 != 0u && !h.swap;
    return h;
}

// Two stored codes of n bits, the first in the low bits, as endpoints of 8
// bits in the halves of a word; pp holds their p-bits.
__device__ inline uint32_t bc7_endpoints(uint32_t code0, uint32_t code1, uint32_t pp, uint32_t hp, uint32_t up,
                                         uint32_t down)
{
    const uint32_t v = (code0 | code1 << 16) << hp | pp;
    return v << up | ((v >> down) & 0x00FF00FFu);
}

// p-bits of the block: word whose low bits are the first subset's.
__device__ inline uint32_t bc7_pbits(const Bc7Head &h, uint32_t w1, uint32_t w2, uint32_t w3)
{
    const bool six = h.m == 6u;
    const uint32_t w = funnel(six ? w2 : w3, six ? w1 : w2, GSBC_BY_MODE(l.pbits & 31));
    return h.hp ? w : 0u;
}

// p-bits of a subset whose bits start at q's low bit, in the halves of a word.
__device__ inline uint32_t bc7_pair(const Bc7Head &h, uint32_t q)
{
    return (q & 1u) | ((q << GSBC_BY_MODE(d.pb == 1 ? 16 : 15)) & 0x00010000u);
}

// The texel of endpoints (pairs of r, g, b, a) at indices i1 and i2:
// interp64 of each channel, as weights times 4 and >> 8.
__device__ inline uint32_t bc7_mix(const Bc7Head &h, uint32_t r, uint32_t g, uint32_t b, uint32_t a, uint32_t i1,
                                   uint32_t i2)
{
    const uint32_t ci = h.swap ? i2 : i1, cs = h.swap ? h.step2 : h.step;
    const uint32_t ai = h.second ? i2 : i1, as = h.second ? h.step2 : h.step;
    // (256 - 4 w) | 4 w << 16
    const uint32_t wc = __umul24((__umul24(ci, cs) + 128u) >> 8, 0x3FFFCu) + 256u;
    const uint32_t wa = __umul24((__umul24(ai, as) + 128u) >> 8, 0x3FFFCu) + 256u;
    const uint32_t rg = bytes(dot2(g, wc, 128u), dot2(r, wc, 128u), 0x0C0C0501u);
    const uint32_t ba = bytes(dot2(a, wa, 128u), dot2(b, wc, 128u), 0x0C0C0501u);
    return bytes(ba, rg, h.rot);
}

// Texel i of a BC7 block, RGBA packed in a uint32 (R in the low byte).
template <class Lut>
__device__ inline uint32_t bc7_texel(const Blk128 &b, int i, const Lut &lut)
{
    const uint32_t w0 = (uint32_t)b.lo, w1 = (uint32_t)(b.lo >> 32), w2 = (uint32_t)b.hi, w3 = (uint32_t)(b.hi >> 32);
    const Bc7Head h = bc7_head(w0, w1, w2, w3, lut);
    const uint32_t s = bits(h.part.map, 2u * i, 2u);
    // the subset's red at the low end of S, green and blue one stride up each
    const uint32_t at = GSBC_BY_MODE(l.colour) + 2u * s * h.cb, stride = GSBC_BY_MODE(2 * d.ns * d.cb);
    const uint32_t S0 = funnel(w1, w0, at), S1 = funnel(w2, w1, at), S2 = funnel(w3, w2, at);
    const uint32_t T0 = funnel(S1, S0, stride), T1 = funnel(S2, S1, stride), U0 = funnel(T1, T0, stride);
    const uint32_t pp = bc7_pair(h, bc7_pbits(h, w1, w2, w3) >> (s * GSBC_BY_MODE(d.pb)));
    const uint32_t r = bc7_endpoints(bits(S0, 0u, h.cb), bits(S0, h.cb, h.cb), pp, h.hp, h.up, h.down);
    const uint32_t g = bc7_endpoints(bits(T0, 0u, h.cb), bits(T0, h.cb, h.cb), pp, h.hp, h.up, h.down);
    const uint32_t bl = bc7_endpoints(bits(U0, 0u, h.cb), bits(U0, h.cb, h.cb), pp, h.hp, h.up, h.down);
    const bool seven = h.m == 7u;
    const uint32_t A = funnel(seven ? w3 : w2, seven ? w2 : w1, GSBC_BY_MODE(l.alpha & 31) + 2u * s * h.ab);
    const uint32_t a = bc7_endpoints(bits(A, 0u, h.ab), bits(A, h.ab, h.ab), pp, h.hp, h.aup, h.adown) | h.amask;
    // indices: one bit less for each anchor texel before i and for i itself
    const uint32_t before = (uint32_t)__popc(h.part.anchors & ((1u << i) - 1u)), own = (h.part.anchors >> i) & 1u;
    const uint64_t iw = (uint64_t)h.iw << 32 | h.iv, jw = (uint64_t)w3 << 32 | w2;
    const uint32_t i1 = bits((uint32_t)(iw >> (h.ibase + i * h.ib - before)), 0u, h.ib - own);
    const uint32_t i2 = bits((uint32_t)(jw >> ((h.ibase2 + i * h.ib2 - (i > 0)) & 63u)), 0u, h.ib2 - (i == 0));
    return bc7_mix(h, r, g, bl, a, i1, i2);
}
__device__ inline uint32_t bc7_texel(const Blk128 &b, int i) { return bc7_texel(b, i, Bc7ConstLut{}); }

// All 16 texels: the fields and endpoints are taken once, the index bits are
// given their anchors' missing top bits so that every texel's are h.ib wide.
template <class Lut>
__device__ inline void bc7_block(const Blk128 &b, uint32_t (&px)[16], const Lut &lut)
{
    const uint32_t w0 = (uint32_t)b.lo, w1 = (uint32_t)(b.lo >> 32), w2 = (uint32_t)b.hi, w3 = (uint32_t)(b.hi >> 32);
    const Bc7Head h = bc7_head(w0, w1, w2, w3, lut);
    const uint32_t at = GSBC_BY_MODE(l.colour), stride = GSBC_BY_MODE(2 * d.ns * d.cb);
    const uint32_t S0 = funnel(w1, w0, at), S1 = funnel(w2, w1, at), S2 = funnel(w3, w2, at);
    const uint32_t T0 = funnel(S1, S0, stride), T1 = funnel(S2, S1, stride), U0 = funnel(T1, T0, stride);
    const bool seven = h.m == 7u;
    const uint32_t A = funnel(seven ? w3 : w2, seven ? w2 : w1, GSBC_BY_MODE(l.alpha & 31));
    const uint32_t P = bc7_pbits(h, w1, w2, w3), pstep = GSBC_BY_MODE(d.pb);
    uint32_t r[3], g[3], bl[3], a[3];
#pragma unroll
    for (uint32_t s = 0; s < 3; s++) {   // (a subset that the mode has not is never chosen below)
        const uint32_t c0 = 2u * s * h.cb, c1 = c0 + h.cb, a0 = 2u * s * h.ab, a1 = a0 + h.ab;
        const uint32_t pp = bc7_pair(h, P >> (s * pstep));
        r[s] = bc7_endpoints(bits(S0, c0, h.cb), bits(S0, c1, h.cb), pp, h.hp, h.up, h.down);
        g[s] = bc7_endpoints(bits(T0, c0, h.cb), bits(T0, c1, h.cb), pp, h.hp, h.up, h.down);
        bl[s] = bc7_endpoints(bits(U0, c0, h.cb), bits(U0, c1, h.cb), pp, h.hp, h.up, h.down);
        a[s] = bc7_endpoints(bits(A, a0, h.ab), bits(A, a1, h.ab), pp, h.hp, h.aup, h.adown) | h.amask;
    }
    uint64_t iw = ((uint64_t)h.iw << 32 | h.iv) >> h.ibase, jw = ((uint64_t)w3 << 32 | w2) >> h.ibase2;
    uint32_t left = h.part.anchors;
#pragma unroll
    for (int s = 0; s < 3; s++) {        // anchors in texel order: bit p and what is above move up by one
        const uint32_t p = ((uint32_t)__builtin_ctz(left | 0x10000u) + 1u) * h.ib - 1u;
        iw += left ? iw & (~0ull << (p & 63u)) : 0ull;
        left &= left - 1u;
    }
    jw += jw & (~0ull << ((h.ib2 - 1u) & 63u));
    const uint32_t ilo = (uint32_t)iw, ihi = (uint32_t)(iw >> (8u * h.ib));
    const uint32_t jlo = (uint32_t)jw, jhi = (uint32_t)(jw >> (8u * h.ib2));
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const uint32_t s = bits(h.part.map, 2u * i, 2u);
        const bool s1 = s == 1u, s2 = s == 2u;
        const uint32_t i1 = bits(i < 8 ? ilo : ihi, (i & 7) * h.ib, h.ib);
        const uint32_t i2 = bits(i < 8 ? jlo : jhi, (i & 7) * h.ib2, h.ib2);
        px[i] = bc7_mix(h, s2 ? r[2] : s1 ? r[1] : r[0], s2 ? g[2] : s1 ? g[1] : g[0], s2 ? bl[2] : s1 ? bl[1] : bl[0],
                        s2 ? a[2] : s1 ? a[1] : a[0], i1, i2);
    }
}

#undef GSBC_BY_MODE

}  // namespace gsbc
