// bc7_encode.hip -- BC7 encoder for gfx950 (BTC with 1-3 reference-colour
// pairs per block, Sec. III-B; the paper codes 4x4 band blocks this way,
// Sec. V).
//
// Search: 285 candidates in a fixed order (mode 0 partitions 0..15; modes
// 1, 2, 3 partitions 0..63; mode 4 rotation x index-selection; mode 5
// rotation; mode 6; mode 7 partitions 0..63).  Each subset is fitted on its
// own: identical texels use precomputed single-value endpoint tables;
// otherwise the endpoints are the texels of least and greatest projection on
// the principal axis (integer power iteration), quantised for every p-bit
// choice, texels take their least-SSE palette entry, and one least-squares
// refit is kept if it lowers the SSE.  The winner minimises
// (SSE << 9) | candidate, a total order, so the result is independent of how
// candidates are spread over lanes.
//
// Layout on the GPU: one lane per block, all lanes of a wave work on the same
// candidate, so partition masks, anchors and mode parameters are wave-uniform
// (scalar registers) and only the texel arithmetic is per lane.  Pass 1 keeps
// only the best key, and fits a block's candidate only if a lower bound of
// its SSE leaves it a chance; pass 2 re-fits each lane's winner (identical
// arithmetic) to emit its bits.
#include "gsbc_internal.h"
#include "bc_format.h"

#include <mutex>
#include <vector>

namespace gsbc {

// Zero, read from memory (external linkage, so it is not folded): see
// entry_const.
__constant__ uint32_t g_bc7_opaque_zero = 0u;

namespace {

// ---- tables (device global memory, built on the host at first use)
// nearest[cls][p][t]: code c minimising |value(c, p) - t| (lowest on ties)
// in the low byte, value(c, p) in the high byte; cls = (cb - 4) * 2 + has_pbit.
// near64[cls][p][t]: 64 value(c, p) of the same code (the search reads only
// values, in the scale its palette entries use).
// sv[cls][p0 + 2 p1][slot][v]: single-value pair (c0 | c1 << 8 | err << 16)
// whose interpolation at weight(nb, K) is nearest v; slot = nb offset + K.
struct Tables {
    const uint16_t *nearest;
    const uint16_t *near64;
    const uint32_t *sv;
};
constexpr int kSlots = 28;
__host__ __device__ constexpr int slot_of(int nb, int k) { return (nb == 2 ? 0 : nb == 3 ? 4 : 12) + k; }
__host__ __device__ constexpr int cls_of(int cb, int pb) { return (cb - 4) * 2 + (pb ? 1 : 0); }

__host__ __device__ constexpr int ep_value(int code, int p, int cb, int pb)
{
    return pb ? expand_bits((code << 1) | p, cb + 1) : expand_bits(code, cb);
}

__device__ __forceinline__ int bitlen(int x) { return 32 - __clz(x); }

// ---- candidate geometry
// Members of subset s of 3-subset partition p: the 2-bit map's low bits (1),
// high bits (2) or neither (0), brought together from every second bit.
__host__ __device__ constexpr uint32_t mask3_of(uint32_t map, int s)
{
    uint32_t x = (s == 0 ? ~(map | map >> 1) : s == 1 ? map : map >> 1) & 0x55555555u;
    x = (x | x >> 1) & 0x33333333u;
    x = (x | x >> 2) & 0x0F0F0F0Fu;
    x = (x | x >> 4) & 0x00FF00FFu;
    return (x | x >> 8) & 0xFFFFu;
}
__device__ __forceinline__ uint32_t mask3(int p, int s) { return mask3_of(kPart3[p], s); }
__device__ __forceinline__ uint32_t mask2(int p, int s)
{
    uint32_t w = kPart2[p];
    return s ? w : (~w & 0xFFFFu);
}

// Candidate index -> (mode, partition, rotation, index selection)
__device__ __forceinline__ void candidate(int ci, int &m, int &p, int &r, int &s)
{
    p = r = s = 0;
    if (ci < 16) { m = 0; p = ci; }
    else if (ci < 80) { m = 1; p = ci - 16; }
    else if (ci < 144) { m = 2; p = ci - 80; }
    else if (ci < 208) { m = 3; p = ci - 144; }
    else if (ci < 216) { m = 4; r = (ci - 208) >> 1; s = (ci - 208) & 1; }
    else if (ci < 220) { m = 5; r = ci - 216; }
    else if (ci < 221) { m = 6; }
    else { m = 7; p = ci - 221; }
}

// ---- texels in LDS
//
// Texels sit in LDS, one column per lane, scaled by -8: rg holds -8 R and
// -8 G as 16-bit halves, bx holds -8 B (16 bits).  Because |x|^2 is the same for every
// palette entry, the least-SSE entry is the least 256 (|p|^2 - 2 x.p) + k.
// Each entry is held as E = (64 pR, 64 pG) in 16-bit halves, Eb = 64 pB and
// C = 256 |p|^2 + k, so one texel x entry evaluation is
//   t = (-8 B) * Eb + C                    (v_mad_i32_i24)
//   t = (-8 R, -8 G) . E + t               (v_dot2c_i32_i16)
//   best = min(best, t)                    (half a v_min3_i32)
// and the members' minima plus 256 sum |x|^2 (taken once per subset from
// its sums) give 256 SSE + sum k exactly (all terms stay within int32:
// |t| < 2^27).  Summed over at most 16 members the k terms stay below 256,
// so the subset SSE is the sum shifted right by 8.  The 64-scaled entries
// are what the interpolation (64 - w) e0 + w e1 + 32 yields once its low six
// bits are masked off, which keeps palette construction short.
// In the search the subset masks are wave-uniform, so texel loops walk the
// set bits of a mask with scalar control.
constexpr int kWG = 256;
constexpr int kQEntries = 10 * 2 * 256;
constexpr int kScaleNeg = -8;          // texel scale in LDS

struct TexLds {
    uint32_t rg[16][kWG];
    int16_t bx[16][kWG];
    uint16_t q[kQEntries];        // search: near64; emit: nearest
};

typedef short short2_t __attribute__((ext_vector_type(2)));

// -8 times the value 255 (a rotated-out channel's replacement)
constexpr int kNeg255 = kScaleNeg * 255;

// Texel i of this lane in the LDS layout; rotation r puts 255 in channel r-1.
__device__ __forceinline__ void texel(const TexLds &S, int i, int rot, uint32_t &rg, int &b)
{
    rg = S.rg[i][threadIdx.x];
    b = S.bx[i][threadIdx.x];
    if (rot) {
        if (rot == 1) rg = (rg & 0xFFFF0000u) | ((uint32_t)kNeg255 & 0xFFFFu);
        else if (rot == 2) rg = (rg & 0xFFFFu) | ((uint32_t)kNeg255 << 16);
        else b = kNeg255;
    }
}

// The texel's channels, negated: (-R, -G, -B) (exact: the stored values are
// multiples of 8).
__device__ __forceinline__ void unpack_neg(uint32_t rg, int b, int (&x)[3])
{
    x[0] = __builtin_amdgcn_sbfe((int)rg, 3, 13);
    x[1] = (int)rg >> 19;
    x[2] = b >> 3;
}

__device__ __forceinline__ void unpack(uint32_t rg, int b, int (&x)[3])
{
    unpack_neg(rg, b, x);
    x[0] = -x[0];
    x[1] = -x[1];
    x[2] = -x[2];
}

// Per-subset data shared across modes: whether every member is the same
// colour, and the two endpoint colours (texels of least and greatest
// projection on the principal axis, or the common colour).
struct Prep {
    bool same;
    int lo[3], hi[3];
    int nSx[3];  // negated member sums per channel (for the least-squares refit)
    int xx;      // sum of |x|^2 over the members
};

// Member sums of a subset: count, negated per-channel sums and the six
// distinct products (RR, RG, RB, GG, GB, BB; the same for negated values).
// Integer, so the sums of disjoint subsets add up exactly: the last subset
// of a partition is the block total minus the others.
struct Sums {
    int n;
    int nSx[3];
    int XX[6];
};

__device__ __forceinline__ Sums subset_sums(const TexLds &S, uint32_t mask, int rot)
{
    Sums m;
    m.n = __popc(mask);
    m.nSx[0] = m.nSx[1] = m.nSx[2] = 0;
#pragma unroll
    for (int q = 0; q < 6; q++) m.XX[q] = 0;
    // -8 R and -8 G summed in the 16-bit halves of one word (at most 16
    // members: |sum| <= 32640)
    short2_t srg = {0, 0};
    for (uint32_t mm = mask; mm; mm &= mm - 1) {
        uint32_t rg;
        int b;
        texel(S, __ffs(mm) - 1, rot, rg, b);
        int x[3];
        unpack_neg(rg, b, x);
        srg += __builtin_bit_cast(short2_t, rg);
        m.nSx[2] += x[2];
        m.XX[0] += mul_i24(x[0], x[0]); m.XX[1] += mul_i24(x[0], x[1]); m.XX[2] += mul_i24(x[0], x[2]);
        m.XX[3] += mul_i24(x[1], x[1]); m.XX[4] += mul_i24(x[1], x[2]); m.XX[5] += mul_i24(x[2], x[2]);
    }
    m.nSx[0] = (int)srg.x >> 3;
    m.nSx[1] = (int)srg.y >> 3;
    return m;
}

__device__ __forceinline__ Sums sums_minus(const Sums &t, const Sums &a)
{
    Sums m;
    m.n = t.n - a.n;
#pragma unroll
    for (int c = 0; c < 3; c++) m.nSx[c] = t.nSx[c] - a.nSx[c];
#pragma unroll
    for (int q = 0; q < 6; q++) m.XX[q] = t.XX[q] - a.XX[q];
    return m;
}

// Principal axis and endpoint texels of a subset from its sums.  The exact
// covariance C = n XX - Sx Sx^T (the same from negated sums) is zero exactly
// when every member has the same colour.
__device__ __forceinline__ Prep prep_subset(const TexLds &S, uint32_t mask, int rot, const Sums &m)
{
    Prep P;
    // n <= 16, XX < 2^21 and |Sx| < 2^12: 24-bit multiplies with exact products
    const int n = m.n;
    int C[3][3];
    C[0][0] = __mul24(n, m.XX[0]) - __mul24(m.nSx[0], m.nSx[0]);
    C[0][1] = C[1][0] = __mul24(n, m.XX[1]) - __mul24(m.nSx[0], m.nSx[1]);
    C[0][2] = C[2][0] = __mul24(n, m.XX[2]) - __mul24(m.nSx[0], m.nSx[2]);
    C[1][1] = __mul24(n, m.XX[3]) - __mul24(m.nSx[1], m.nSx[1]);
    C[1][2] = C[2][1] = __mul24(n, m.XX[4]) - __mul24(m.nSx[1], m.nSx[2]);
    C[2][2] = __mul24(n, m.XX[5]) - __mul24(m.nSx[2], m.nSx[2]);
    P.same = (C[0][0] | C[1][1] | C[2][2]) == 0;
    P.nSx[0] = m.nSx[0]; P.nSx[1] = m.nSx[1]; P.nSx[2] = m.nSx[2];
    P.xx = m.XX[0] + m.XX[3] + m.XX[5];
    if (P.same) {
        uint32_t rg;
        int b;
        texel(S, __ffs(mask) - 1, rot, rg, b);
        unpack(rg, b, P.lo);
        P.hi[0] = P.lo[0]; P.hi[1] = P.lo[1]; P.hi[2] = P.lo[2];
        return P;
    }
    // principal axis: integer power iteration on the exact covariance
    // row of the largest diagonal entry (lowest index on ties), by selects
    const int j = (C[1][1] > C[0][0]) ? ((C[2][2] > C[1][1]) ? 2 : 1) : ((C[2][2] > C[0][0]) ? 2 : 0);
    const int tsh = max(0, bitlen(j == 0 ? C[0][0] : (j == 1 ? C[1][1] : C[2][2])) - 14);
    int Cs[3][3];
#pragma unroll
    for (int a = 0; a < 3; a++)
#pragma unroll
        for (int c = 0; c < 3; c++) Cs[a][c] = C[a][c] >> tsh;
    int v[3];
#pragma unroll
    for (int c = 0; c < 3; c++) v[c] = j == 0 ? Cs[0][c] : (j == 1 ? Cs[1][c] : Cs[2][c]);
    // |Cs| <= 2^14 (the largest diagonal is below 2^14 and bounds every entry
    // of the positive semi-definite C) and |v| <= 2^15, so the products are
    // 16-bit dot products with exact 32-bit sums (|u| < 3 * 2^29).
    short2_t c01[3];
#pragma unroll
    for (int a = 0; a < 3; a++) c01[a] = short2_t{(short)Cs[a][0], (short)Cs[a][1]};
#pragma unroll
    for (int it = 0; it < 8; it++) {
        const short2_t v01 = {(short)v[0], (short)v[1]};
        int u[3];
        // the third term as a 24-bit product (|Cs| <= 2^14, |v| <= 2^15)
        // accumulated into by the dot product of the first two
#pragma unroll
        for (int a = 0; a < 3; a++) u[a] = __builtin_amdgcn_sdot2(c01[a], v01, __mul24(Cs[a][2], v[2]), false);
        // max(max |u_a|, 1) as max(max u, -min u, 1): its bit length minus 15,
        // at least 0, is the shift that brings max |v| below 2^15
        const int mx = max(max(u[0], max(u[1], u[2])), max(-min(u[0], min(u[1], u[2])), 1));
        const uint32_t sh = __builtin_elementwise_sub_sat(17u, (uint32_t)__builtin_clz((uint32_t)mx));
#pragma unroll
        for (int a = 0; a < 3; a++) v[a] = u[a] >> sh;
    }
    if (v[0] == 0 && v[1] == 0 && v[2] == 0) v[0] = v[1] = v[2] = 1;
    // members of least and greatest projection p, the first of each on ties.
    // The stored texels give q = -8 p in one dot product and one multiply-add
    // (|q| < 2^28); 2 q = -16 p leaves four low bits for the member index:
    // the largest 2q + 15 - i is the least p (first i), the least 2q + i is
    // the greatest p (first i).
    const short2_t v01 = {(short)v[0], (short)v[1]};
    int klo = (int)0x80000000, khi = 0x7FFFFFFF;
    for (uint32_t mm = mask; mm; mm &= mm - 1) {
        const int i = __ffs(mm) - 1;
        uint32_t rg;
        int b;
        texel(S, i, rot, rg, b);
        const int q = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, rg), v01, mul_i24(b, v[2]), false);
        klo = max(klo, 2 * q + (15 - i));
        khi = min(khi, 2 * q + i);
    }
    uint32_t rg;
    int b;
    texel(S, 15 - (klo & 15), rot, rg, b);
    unpack(rg, b, P.lo);
    texel(S, khi & 15, rot, rg, b);
    unpack(rg, b, P.hi);
    return P;
}

__device__ __forceinline__ Prep prep_subset(const TexLds &S, uint32_t mask, int rot)
{
    return prep_subset(S, mask, rot, subset_sums(S, mask, rot));
}

// Result of fitting one endpoint pair to a subset.  eval_pair leaves idx in
// member order (IW bits per member, first member lowest; IW = 2 for 2-bit
// indices, else 4); fit_colour returns it by texel position (4 bits at 4 i
// for member i).
struct PairFit {
    uint32_t sse;
    uint64_t idx;
    uint32_t c0, c1;   // endpoint codes, 8 bits per channel, R lowest
    int p0, p1;
};

template <int NB>
constexpr int idx_width() { return NB == 2 ? 2 : 4; }

// Palette entry constant C = 256 |p|^2 + k from the 64-scaled entry:
// (64 p) . (64 p) + 16 k = 16 C, exactly.  The opaque zero keeps 16 k an
// addition (its bits are provably clear of the product's, which would turn
// it into an or), so product and sum fuse into one v_mad_u32_u24.
__device__ __forceinline__ int entry_const(uint32_t e, int eb, int k)
{
    const short2_t es = __builtin_bit_cast(short2_t, e);
    const uint32_t b2k = mul_u24((uint32_t)eb, (uint32_t)eb) + (16u * (uint32_t)k + g_bc7_opaque_zero);
    return __builtin_amdgcn_sdot2(es, es, (int)b2k, false) >> 4;
}

// (c) for one endpoint pair: quantise for every p-bit combination, index
// every member by least SSE; keep the best combination (lowest on ties).
// Up to 32 palette entries are held at once, so each member is read once
// for all combinations (once per combination for 16-entry palettes).  Per
// member and combination the running sum takes 256 SSE + k in one add and
// the index enters a shift register (newest member at the top; it holds the
// n indices in its top IW n bits).  IDX = false: the SSE only.  CODES: the
// LDS table holds code | value << 8 (the emit pass, which needs the codes);
// otherwise it holds 64 value (the search).
template <int CB, int PB, int NB, bool IDX, bool CODES>
__device__ __forceinline__ PairFit eval_pair(const TexLds &S, uint32_t mask, int rot, const int (&lo)[3],
                                             const int (&hi)[3], int xx)
{
    constexpr int NPC = PB == 2 ? 4 : PB == 1 ? 2 : 1;
    constexpr int NE = 1 << NB;
    constexpr int CPV = NPC * NE <= 32 ? NPC : 1;   // combinations per member visit
    constexpr int NP = PB ? 2 : 1;                  // p-bit values of an endpoint
    constexpr int IW = idx_width<NB>();
    constexpr bool WIDE = IW * 16 > 32;             // the indices need two words
    constexpr int cls = cls_of(CB, PB);
    const int n = __popc(mask);
    // each endpoint quantised for each p-bit value: E = (64 v_R, 64 v_G),
    // Eb = 64 v_B, and the codes (emit)
    uint32_t E[2][NP], code[2][NP];
    int Eb[2][NP];
#pragma unroll
    for (int end = 0; end < 2; end++)
#pragma unroll
        for (int p = 0; p < NP; p++) {
            const uint16_t *t = S.q + (cls * 2 + p) * 256;
            const int *v = end ? hi : lo;
            uint32_t e[3];
#pragma unroll
            for (int c = 0; c < 3; c++) e[c] = t[v[c]];
            if (CODES) {
                code[end][p] = (e[0] & 255u) | (e[1] & 255u) << 8 | (e[2] & 255u) << 16;
#pragma unroll
                for (int c = 0; c < 3; c++) e[c] = (e[c] >> 8) << 6;
            } else {
                code[end][p] = 0;
            }
            E[end][p] = e[0] | (e[1] << 16);
            Eb[end][p] = (int)e[2];
        }
    PairFit best;
    best.sse = 0xFFFFFFFFu;
    best.idx = 0;
    best.c0 = best.c1 = 0;
    best.p0 = best.p1 = 0;
#pragma unroll
    for (int pc0 = 0; pc0 < NPC; pc0 += CPV) {
        // Interpolation (64 - w) e0 + w e1 + 32 = (64 e0 + 32) + w (e1 - e0)
        // stays within [32, 16352], so R and G are interpolated together in
        // 16-bit lanes; masking its low six bits gives the 64-scaled entry.
        uint32_t prg[CPV][NE];
        int pb[CPV][NE], pk[CPV][NE];
#pragma unroll
        for (int j = 0; j < CPV; j++) {
            const int pc = pc0 + j;
            const int p0 = PB == 2 ? (pc & 1) : PB == 1 ? pc : 0;
            const int p1 = PB == 2 ? (pc >> 1) : PB == 1 ? pc : 0;
            const uint32_t E0 = E[0][p0], E1 = E[1][p1];
            const int B0 = Eb[0][p0], B1 = Eb[1][p1];
            const short2_t a_rg = __builtin_bit_cast(short2_t, E0 | 0x00200020u);
            const short2_t s_rg = (__builtin_bit_cast(short2_t, E1) - __builtin_bit_cast(short2_t, E0)) >> (short)6;
            const int a_b = B0 | 32, s_b = (B1 - B0) >> 6;
#pragma unroll
            for (int k = 0; k < NE; k++) {
                // entries 0 and NE-1 are the endpoints themselves (weights 0 and 64)
                const short w = (short)bc7_weight(NB, k);
                const uint32_t e = k == 0 ? E0 : k == NE - 1 ? E1
                                 : __builtin_bit_cast(uint32_t, a_rg + s_rg * w) & 0xFFC0FFC0u;
                const int eb = k == 0 ? B0 : k == NE - 1 ? B1 : (a_b + mul_i24(s_b, w)) & ~63;
                prg[j][k] = e;
                pb[j][k] = eb;
                pk[j][k] = entry_const(e, eb, k);
            }
        }
        // 256 SSE + k summed over members: 256 |x|^2 added once per subset
        uint32_t acc[CPV], rlo[CPV], rhi[CPV];
#pragma unroll
        for (int j = 0; j < CPV; j++) {
            acc[j] = 256u * (uint32_t)xx;
            rlo[j] = rhi[j] = 0;
        }
        // least key of one member against combination j's entries
        auto least = [&](uint32_t rg, int b, int j) {
            int kb = 0x7FFFFFFF;
#pragma unroll
            for (int k = 0; k < NE; k++) {
                // with a p-bit per endpoint, entry 0 depends only on p0 and
                // entry NE-1 only on p1: combinations share those keys
                const int js = (PB == 2 && CPV == 4) ? (k == 0 ? (j & 1) : k == NE - 1 ? (j & 2) : j) : j;
                const int key = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, rg),
                                                       __builtin_bit_cast(short2_t, prg[js][k]),
                                                       mul_i24(b, pb[js][k]) + pk[js][k], false);
                kb = min(kb, key);
            }
            return (uint32_t)kb;   // 256 (SSE - |x|^2) + k of this member
        };
        auto push_index = [&](int j, uint32_t kb) {
            if (IDX) {
                if (WIDE) {
                    rlo[j] = __builtin_amdgcn_alignbit(rhi[j], rlo[j], IW);
                    rhi[j] = __builtin_amdgcn_alignbit(kb, rhi[j], IW);
                } else {
                    rlo[j] = __builtin_amdgcn_alignbit(kb, rlo[j], IW);
                }
            }
        };
        // members two at a time (their keys join the sums in one three-way
        // add), then the odd one
        uint32_t m = mask;
        for (; m & (m - 1); m &= m - 1, m &= m - 1) {
            uint32_t rg0, rg1;
            int b0, b1;
            texel(S, __ffs(m) - 1, rot, rg0, b0);
            texel(S, __ffs(m & (m - 1)) - 1, rot, rg1, b1);
#pragma unroll
            for (int j = 0; j < CPV; j++) {
                const uint32_t k0 = least(rg0, b0, j), k1 = least(rg1, b1, j);
                acc[j] += k0 + k1;
                push_index(j, k0);
                push_index(j, k1);
            }
        }
        if (m) {
            uint32_t rg;
            int b;
            texel(S, __ffs(m) - 1, rot, rg, b);
#pragma unroll
            for (int j = 0; j < CPV; j++) {
                const uint32_t kb = least(rg, b, j);
                acc[j] += kb;
                push_index(j, kb);
            }
        }
#pragma unroll
        for (int j = 0; j < CPV; j++) {
            const uint32_t sse = acc[j] >> 8;
            if (sse < best.sse) {
                const int pc = pc0 + j;
                const int p0 = PB == 2 ? (pc & 1) : PB == 1 ? pc : 0;
                const int p1 = PB == 2 ? (pc >> 1) : PB == 1 ? pc : 0;
                best.sse = sse;
                best.idx = !IDX ? 0
                         : WIDE ? (((uint64_t)rhi[j] << 32) | rlo[j]) >> (64 - IW * n)
                                : (uint64_t)(rlo[j] >> (32 - IW * n));
                best.c0 = code[0][p0];
                best.c1 = code[1][p1];
                best.p0 = p0;
                best.p1 = p1;
            }
        }
    }
    return best;
}

// Index weight of NB-bit index k from the weight table packed in bytes
// (v_perm_b32 picks byte k; selector 0x0C gives zero bytes).
__host__ __device__ constexpr uint32_t pack_weights(int nb, int first)
{
    return (uint32_t)bc7_weight(nb, first) | ((uint32_t)bc7_weight(nb, first + 1) << 8) |
           ((uint32_t)bc7_weight(nb, first + 2) << 16) | ((uint32_t)bc7_weight(nb, first + 3) << 24);
}
static_assert(pack_weights(2, 0) == 0x402B1500u && pack_weights(3, 0) == 0x1B120900u &&
              pack_weights(3, 4) == 0x40372E25u, "BC7 weight tables");

// Weight of the index in the low bits of f (the bits above are ignored).
template <int NB>
__device__ __forceinline__ int weight_of(uint32_t f)
{
    const uint32_t sel = (f & (NB == 2 ? 3u : 7u)) | 0x0C0C0C00u;
    if (NB == 2) return (int)__builtin_amdgcn_perm(0u, pack_weights(2, 0), sel);
    if (NB == 3) return (int)__builtin_amdgcn_perm(pack_weights(3, 4), pack_weights(3, 0), sel);
    return bc7_weight(NB, (int)(f & 15u));
}

// (d) least-squares endpoints for the chosen indices; false if singular.
// With weights (64 - w, w) the normal-equation sums follow from the member
// count n, sum(w), sum(w^2), the channel sums Sx and sum(w x):
//   A = 4096 n - 128 sum(w) + sum(w^2), B = sum(w^2), AB = 64 sum(w) - sum(w^2),
//   SA = 64 Sx - SB.
// The sums of w x are taken on the stored texels, -8 x, by 16-bit dot
// products with (w, 0) and (0, w), so every channel sum carries the factor
// -8; the right-hand sides are formed at that scale and the factor is taken
// out exactly (a power of two) with the reciprocal.
template <int NB>
__device__ __forceinline__ bool ls_endpoints(const TexLds &S, uint32_t mask, int rot, uint64_t idx, const int (&nSx)[3],
                                             int (&lo)[3], int (&hi)[3])
{
    constexpr int IW = idx_width<NB>();
    int W1 = 0, W2 = 0, SB8[3] = {0, 0, 0};   // SB8 = -8 sum(w x)
    uint32_t cur = (uint32_t)idx;
    int j = 0;
    for (uint32_t m = mask; m; m &= m - 1, j++) {
        if (IW == 4 && j == 8) cur = (uint32_t)(idx >> 32);
        uint32_t rg;
        int b;
        texel(S, __ffs(m) - 1, rot, rg, b);
        const int w = weight_of<NB>(cur);   // member order
        cur >>= IW;
        W1 += w;
        W2 += (int)mul_u24((uint32_t)w, (uint32_t)w);
        SB8[0] = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, rg), __builtin_bit_cast(short2_t, (uint32_t)w),
                                        SB8[0], false);
        SB8[1] = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, rg),
                                        __builtin_bit_cast(short2_t, (uint32_t)w << 16), SB8[1], false);
        SB8[2] += mul_i24(b, w);
    }
    const int n = __popc(mask);
    const int A = 4096 * n - 128 * W1 + W2, B = W2, AB = 64 * W1 - W2;
    const double det = fma((double)A, (double)B, -((double)AB * (double)AB));
    if (det == 0.0) return false;
    // 1/det in FP64 from the FP32 reciprocal and two Newton steps (within
    // 2^-50), times 64 (exact) for the numerators' common factor and -1/8
    // (exact) for the texel scale
    double inv = (double)__builtin_amdgcn_rcpf((float)det);
    inv = fma(fma(-det, inv, 1.0), inv, inv);
    inv = -8.0 * fma(fma(-det, inv, 1.0), inv, inv);
#pragma unroll
    for (int c = 0; c < 3; c++) {
        // Exact numerators n = 64 m (|m| < 2^36), here formed as -8 m
        // (|8 m| < 2^39, products and differences exact in FP64).
        // floor(n/det + 1/2) is taken as floor(m * 64 inv + 1/2 + 2^-37):
        // (2 n + det) / (2 det) is a multiple of 1/(2 det) >= 2^-33, and for
        // |n/det| <= 512 the FP64 error is below 2^-40, so the margin never
        // moves the floor; larger quotients clamp to 0 or 255 either way.
        const double SA8 = (double)(512 * nSx[c] - SB8[c]);
        const double m0 = fma((double)B, SA8, -((double)AB * (double)SB8[c]));
        const double m1 = fma((double)A, (double)SB8[c], -((double)AB * SA8));
        // floor then clamp to [0, 255] equals clamp then truncate
        const double q0 = fma(m0, inv, 0.5 + 0x1p-37), q1 = fma(m1, inv, 0.5 + 0x1p-37);
        lo[c] = (int)fmin(fmax(q0, 0.0), 255.0);
        hi[c] = (int)fmin(fmax(q1, 0.0), 255.0);
    }
    return true;
}

// Fit one colour subset with endpoint precision (CB, PB) and NB-bit indices.
// SEARCH: only the SSE is wanted (the search pass, whose LDS table holds 64-
// scaled values); the refit's indices and the positional index layout are
// skipped.
template <int CB, int PB, int NB, bool SEARCH = false>
__device__ __forceinline__ PairFit fit_colour(const TexLds &S, uint32_t mask, int rot, const Prep &P,
                                              const uint32_t *sv)
{
    constexpr int NPC = PB == 2 ? 4 : PB == 1 ? 2 : 1;
    constexpr int cls = cls_of(CB, PB);
    constexpr int IW = idx_width<NB>();
    if (P.same) {
        // (a) single value: best (p-bits, index) from the per-channel tables
        PairFit f;
        f.sse = 0xFFFFFFFFu;
        f.idx = 0;
        f.c0 = f.c1 = 0;
        f.p0 = f.p1 = 0;
        // (rolled: unrolled, the rows' addresses fill the scalar registers)
#pragma unroll 1
        for (int pc = 0; pc < NPC; pc++) {
            const int p0 = PB == 2 ? (pc & 1) : PB == 1 ? pc : 0;
            const int p1 = PB == 2 ? (pc >> 1) : PB == 1 ? pc : 0;
#pragma unroll 1
            for (int k = 0; k < (1 << NB); k++) {
                const uint32_t *row = sv + ((uint64_t)(cls * 4 + p0 + 2 * p1) * kSlots + slot_of(NB, k)) * 256;
                uint32_t e = 0, c0 = 0, c1 = 0;
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    const uint32_t ent = row[P.lo[c]];
                    const uint32_t er = ent >> 16;
                    e += er * er;
                    c0 |= (ent & 255u) << (8 * c);
                    c1 |= ((ent >> 8) & 255u) << (8 * c);
                }
                if (e < f.sse) {
                    f.sse = e;
                    f.idx = (uint64_t)k * 0x1111111111111111ull;
                    f.c0 = c0;
                    f.c1 = c1;
                    f.p0 = p0;
                    f.p1 = p1;
                }
            }
        }
        f.sse *= (uint32_t)__popc(mask);
        return f;
    }
    // (b) endpoints from the principal axis, (c) quantise and index,
    // (d) one least-squares refit kept only if strictly better
    PairFit f = eval_pair<CB, PB, NB, true, !SEARCH>(S, mask, rot, P.lo, P.hi, P.xx);
    int rlo[3], rhi[3];
    if (ls_endpoints<NB>(S, mask, rot, f.idx, P.nSx, rlo, rhi)) {
        PairFit g = eval_pair<CB, PB, NB, !SEARCH, !SEARCH>(S, mask, rot, rlo, rhi, P.xx);
        if (g.sse < f.sse) f = g;
    }
    if (SEARCH) return f;
    // member order -> texel positions
    uint64_t pos = 0, c = f.idx;
    for (uint32_t m = mask; m; m &= m - 1) {
        pos |= (c & ((1u << IW) - 1)) << (4 * (__ffs(m) - 1));
        c >>= IW;
    }
    f.idx = pos;
    return f;
}

// Scalar channel of modes 4 and 5: the 16 values of channel r-1 (rotation
// r > 0) or the constant 255 (r = 0); precision AB bits, NB-bit indices.
// The values are taken negated from the stored texels; every sum below is
// negated with them and the keys are unchanged.
template <int AB, int NB, bool CODES>
__device__ __forceinline__ PairFit fit_scalar(const TexLds &S, int rot, const uint32_t *sv)
{
    constexpr int cls = cls_of(AB, 0);
    auto nvalue = [&](int i) {
        const uint32_t rg = S.rg[i][threadIdx.x];
        const int b = S.bx[i][threadIdx.x];
        return rot == 0 ? -255 : rot == 1 ? __builtin_amdgcn_sbfe((int)rg, 3, 13) : rot == 2 ? (int)rg >> 19 : b >> 3;
    };
    const int v0 = nvalue(0);
    int nlo = v0, nhi = v0;
    bool same = true;
    // (member loops partly rolled: unrolled, the 16 values stay in registers
    // from pass to pass, which spills in the search)
#pragma unroll 3
    for (int i = 1; i < 16; i++) {
        int v = nvalue(i);
        same &= v == v0;
        nlo = min(nlo, v);
        nhi = max(nhi, v);
    }
    PairFit best;
    best.sse = 0xFFFFFFFFu;
    best.idx = 0;
    best.c0 = best.c1 = 0;
    best.p0 = best.p1 = 0;
    if (same) {
#pragma unroll 1
        for (int k = 0; k < (1 << NB); k++) {
            const uint32_t ent = sv[((uint64_t)(cls * 4) * kSlots + slot_of(NB, k)) * 256 + (-v0)];
            const uint32_t er = ent >> 16;
            if (er * er < best.sse) {
                best.sse = er * er;
                best.idx = (uint64_t)k * 0x1111111111111111ull;
                best.c0 = ent & 255u;
                best.c1 = (ent >> 8) & 255u;
            }
        }
        best.sse *= 16u;
        return best;
    }
    int elo = -nhi, ehi = -nlo;   // least and greatest value
    for (int pass = 0; pass < 2; pass++) {
        const uint32_t e0 = S.q[cls * 2 * 256 + elo], e1 = S.q[cls * 2 * 256 + ehi];
        const int d0 = CODES ? (int)(e0 >> 8) : (int)(e0 >> 6), d1 = CODES ? (int)(e1 >> 8) : (int)(e1 >> 6);
        // entry k as 32 p (against the negated value) and 16 p^2 + k
        int pal[1 << NB], pk[1 << NB];
#pragma unroll
        for (int k = 0; k < (1 << NB); k++) {
            const int pv = interp64(d0, d1, bc7_weight(NB, k));
            pal[k] = 32 * pv;
            pk[k] = 16 * (int)__builtin_amdgcn_udot4((uint32_t)pv, (uint32_t)pv, 0u, false) + k;
        }
        uint32_t sse = 0;
        uint64_t idx = 0;
        int A = 0, B = 0, AB2 = 0, nSA = 0, nSB = 0;
#pragma unroll 2
        for (int i = 0; i < 16; i++) {
            const int x = nvalue(i);
            int kmin = 0x7FFFFFFF;
#pragma unroll
            for (int k = 0; k < (1 << NB); k++) kmin = min(kmin, mul_i24(x, pal[k]) + pk[k]);
            const uint32_t kb = (uint32_t)(kmin + 16 * x * x);   // 16 SSE + k
            sse += kb >> 4;
            idx |= (uint64_t)(kb & 15u) << (4 * i);
            const int w = bc7_weight(NB, (int)(kb & 15u)), a = 64 - w;
            A += a * a; B += w * w; AB2 += a * w; nSA += a * x; nSB += w * x;
        }
        if (sse < best.sse) {
            best.sse = sse;
            best.idx = idx;
            best.c0 = CODES ? e0 & 255u : 0u;
            best.c1 = CODES ? e1 & 255u : 0u;
        }
        if (pass == 1) break;
        const double det = (double)A * (double)B - (double)AB2 * (double)AB2;
        if (det == 0.0) break;
        // numerators of the positive values (the negated sums flip their sign)
        double n0 = -64.0 * ((double)B * (double)nSA - (double)AB2 * (double)nSB);
        double n1 = -64.0 * ((double)A * (double)nSB - (double)AB2 * (double)nSA);
        double q0 = floor(n0 / det + 0.5), q1 = floor(n1 / det + 0.5);
        elo = q0 < 0.0 ? 0 : (q0 > 255.0 ? 255 : (int)q0);
        ehi = q1 < 0.0 ? 0 : (q1 > 255.0 ? 255 : (int)q1);
    }
    return best;
}

// (e) the anchor texel's index must have its top bit clear; otherwise swap
// the endpoints (and p-bits) and mirror every member's index.
template <int NB>
__device__ __forceinline__ void anchor_fix(PairFit &f, uint32_t mask, int anchor)
{
    if (!((f.idx >> (4 * anchor + NB - 1)) & 1)) return;
    uint32_t t = f.c0; f.c0 = f.c1; f.c1 = t;
    int u = f.p0; f.p0 = f.p1; f.p1 = u;
    uint64_t spread = 0;
    for (uint32_t m = mask; m; m &= m - 1) spread |= (uint64_t)((1u << NB) - 1) << (4 * (__ffs(m) - 1));
    f.idx ^= spread;   // k -> (2^NB - 1) - k on the members
}

// ---- the candidates of one partition shape
//
// The principal axis and the extreme texels of a subset depend only on its
// members, so they are found once and shared by the modes with that
// partition.  A wave's lanes hold different blocks; the masks are
// wave-uniform in the search (scalar member loops) and per lane in the seed
// pass.
__device__ __forceinline__ void consider(uint32_t sse, int ci, uint32_t &best)
{
    best = min(best, (sse << 9) | (uint32_t)ci);
}

// Candidate types of the search: 2-subset partitions (modes 1, 3, 7),
// 3-subset ones in mode 0 and in mode 2, rotations (modes 4, 5), mode 6.
enum { kTwo = 0, kThree0 = 1, kThree2 = 2, kRot = 3, kSix = 4, kTypes = 5 };
constexpr uint32_t kGone = 0xFFFFFFFFu;   // a mode that is out of the race

// Add the subset's SSE to each of the type's modes still in the race (e[0]
// only, except for modes 1, 3, 7).
template <int TYPE>
__device__ __forceinline__ void add_subset(const TexLds &S, uint32_t m, const Sums &sums, const uint32_t *sv, uint32_t (&e)[3])
{
    const Prep P = prep_subset(S, m, 0, sums);
    auto add = [&](int q, auto fit) {
        if (__any(e[q] != kGone)) {
            const uint32_t v = fit();
            e[q] = e[q] == kGone ? kGone : e[q] + v;
        }
    };
    if (TYPE == kTwo) {
        add(0, [&] { return fit_colour<6, 1, 3, true>(S, m, 0, P, sv).sse; });
        add(1, [&] { return fit_colour<7, 2, 2, true>(S, m, 0, P, sv).sse; });
        add(2, [&] { return fit_colour<5, 2, 2, true>(S, m, 0, P, sv).sse; });
    } else if (TYPE == kThree0) {
        e[0] += fit_colour<4, 2, 3, true>(S, m, 0, P, sv).sse;
    } else {
        e[0] += fit_colour<5, 0, 2, true>(S, m, 0, P, sv).sse;
    }
}

// Key of a partition whose subsets are all added.
template <int TYPE>
__device__ __forceinline__ uint32_t partition_key(int p, const uint32_t (&e)[3])
{
    if (TYPE == kThree0) return (e[0] << 9) | (uint32_t)p;
    if (TYPE == kThree2) return (e[0] << 9) | (uint32_t)(80 + p);
    uint32_t best = 0xFFFFFFFFu;
    if (e[0] != kGone) consider(e[0], 16 + p, best);
    if (e[1] != kGone) consider(e[1], 144 + p, best);
    if (e[2] != kGone) consider(e[2], 221 + p, best);
    return best;
}

// The full mask, not a constant to the compiler: with one it unrolls the
// member loops and keeps all texels in registers, which spill.
__device__ __forceinline__ uint32_t all_texels() { return 0xFFFFu + g_bc7_opaque_zero; }

// ---- visiting order of the 3-subset partitions, where every one is fitted
//
// Of the 192 subset masks of the 64 three-subset partitions only 140 differ
// (36 of the 48 of partitions 0..15, the ones mode 0 also uses).  They are
// visited in the order below; a mask that recurs is fitted once and its SSE
// kept in an LDS slot of its lane until its last use.  This order (found
// offline by a local search) needs at most kSlots2 slots for mode 2 and kSlots0
// for mode 0; a static check below recomputes both.
constexpr int kOrder3[64] = {62, 9,  2,  0,  60, 42, 61, 27, 38, 18, 46, 33, 51, 47, 55, 41,
                             31, 17, 63, 15, 23, 10, 36, 22, 8,  56, 29, 4,  3,  24, 6,  32,
                             25, 19, 14, 37, 34, 7,  26, 43, 52, 5,  54, 50, 20, 48, 1,  39,
                             58, 13, 35, 57, 53, 30, 21, 59, 49, 40, 28, 45, 16, 11, 44, 12};
constexpr int kSlots2 = 6, kSlots0 = 4;

// What is done at visit t (partition kOrder3[t]), subset s, per mode:
//   kFit           fit the subset
//   kKeep | slot   fit it and keep the SSE in the slot (the mask recurs)
//   kTake | slot   take the SSE from the slot (fitted at an earlier visit)
constexpr uint8_t kFit = 0, kKeep = 0x40, kTake = 0x80;
struct Plan3 {
    uint8_t act[2][64][3];   // [0]: mode 2 (all partitions), [1]: mode 0 (partitions 0..15)
    int slots[2];            // slots each mode needs
};

constexpr Plan3 make_plan3()
{
    Plan3 P{};
    for (int mode = 0; mode < 2; mode++) {
        // each visit's mask, then its last visit
        uint32_t mk[192] = {};
        int pos[192] = {}, n = 0;
        for (int t = 0; t < 64; t++)
            for (int s = 0; s < 3; s++)
                if (mode == 0 || kOrder3[t] < 16) { mk[n] = mask3_of(kPart3[kOrder3[t]], s); pos[n] = t * 3 + s; n++; }
        bool used[8] = {};
        uint32_t held[8] = {};
        int most = 0;
        for (int q = 0; q < n; q++) {
            int later = -1, slot = -1;
            for (int r = q + 1; r < n; r++)
                if (mk[r] == mk[q]) { later = r; break; }
            for (int z = 0; z < 8; z++)
                if (used[z] && held[z] == mk[q]) slot = z;
            uint8_t a = kFit;
            if (slot >= 0) {
                a = (uint8_t)(kTake | slot);
                if (later < 0) used[slot] = false;   // last use
            } else if (later >= 0) {
                int z = 0;
                while (used[z]) z++;
                used[z] = true;
                held[z] = mk[q];
                a = (uint8_t)(kKeep | z);
                int live = 0;
                for (int y = 0; y < 8; y++) live += used[y] ? 1 : 0;
                most = live > most ? live : most;
            }
            P.act[mode][pos[q] / 3][pos[q] % 3] = a;
        }
        P.slots[mode] = most;
    }
    return P;
}
constexpr Plan3 kPlan3 = make_plan3();
static_assert(kPlan3.slots[0] <= kSlots2 && kPlan3.slots[1] <= kSlots0, "3-subset visiting order needs more slots");

// Per-lane SSE slots (kSlots2 for mode 2, then kSlots0 for mode 0), one column
// per lane.
typedef uint32_t Cache3[kSlots2 + kSlots0][kWG];

// The best key over every 2-subset partition (THREE: 3-subset partition).
template <bool THREE>
__device__ __forceinline__ uint32_t search_every(const TexLds &S, Cache3 &cache, uint32_t mode_mask, const uint32_t *sv)
{
    uint32_t best = 0xFFFFFFFFu;
    if (!THREE) {
        const Sums tot = subset_sums(S, all_texels(), 0);
        for (int p = 0; p < 64; p++) {
            const uint32_t m0 = mask2(p, 0), m1 = mask2(p, 1);
            const Sums s0 = subset_sums(S, m0, 0);
            const Prep P0 = prep_subset(S, m0, 0, s0), P1 = prep_subset(S, m1, 0, sums_minus(tot, s0));
            if (mode_mask & 0x02)
                consider(fit_colour<6, 1, 3, true>(S, m0, 0, P0, sv).sse + fit_colour<6, 1, 3, true>(S, m1, 0, P1, sv).sse,
                         16 + p, best);
            if (mode_mask & 0x08)
                consider(fit_colour<7, 2, 2, true>(S, m0, 0, P0, sv).sse + fit_colour<7, 2, 2, true>(S, m1, 0, P1, sv).sse,
                         144 + p, best);
            if (mode_mask & 0x80)
                consider(fit_colour<5, 2, 2, true>(S, m0, 0, P0, sv).sse + fit_colour<5, 2, 2, true>(S, m1, 0, P1, sv).sse,
                         221 + p, best);
        }
    } else {
        const bool on2 = mode_mask & 0x04, on0 = mode_mask & 0x01;
        for (int t = 0; t < 64; t++) {
            const int p = kOrder3[t];
            if (!on2 && p >= 16) continue;
            const bool with0 = on0 && p < 16;
            uint32_t e2 = 0, e0 = 0;
#pragma unroll 1
            for (int s = 0; s < 3; s++) {
                const uint32_t msk = mask3(p, s);
                const int a2 = kPlan3.act[0][t][s], a0 = kPlan3.act[1][t][s];
                const bool fit2 = on2 && !(a2 & kTake), fit0 = with0 && !(a0 & kTake);
                uint32_t v2 = 0, v0 = 0;
                if (on2 && (a2 & kTake)) v2 = cache[a2 & 15][threadIdx.x];
                if (with0 && (a0 & kTake)) v0 = cache[kSlots2 + (a0 & 15)][threadIdx.x];
                if (fit2 || fit0) {
                    const Prep P = prep_subset(S, msk, 0);
                    if (fit2) {
                        v2 = fit_colour<5, 0, 2, true>(S, msk, 0, P, sv).sse;
                        if (a2 & kKeep) cache[a2 & 15][threadIdx.x] = v2;
                    }
                    if (fit0) {
                        v0 = fit_colour<4, 2, 3, true>(S, msk, 0, P, sv).sse;
                        if (a0 & kKeep) cache[kSlots2 + (a0 & 15)][threadIdx.x] = v0;
                    }
                }
                e2 += v2;
                e0 += v0;
            }
            if (on2) consider(e2, 80 + p, best);
            if (with0) consider(e0, p, best);
        }
    }
    return best;
}

// rotation r: modes 4 (both index selections) and 5
__device__ __forceinline__ uint32_t search_rotation(const TexLds &S, int r, uint32_t mode_mask, const uint32_t *sv)
{
    uint32_t best = 0xFFFFFFFFu;
    const uint32_t full = all_texels();
    const Prep P = prep_subset(S, full, r);
    if (mode_mask & 0x10) {
        uint32_t s0 = fit_colour<5, 0, 2, true>(S, full, r, P, sv).sse;
        uint32_t s1 = fit_colour<5, 0, 3, true>(S, full, r, P, sv).sse;
        if (r) { s0 += fit_scalar<6, 3, false>(S, r, sv).sse; s1 += fit_scalar<6, 2, false>(S, r, sv).sse; }
        consider(s0, 208 + 2 * r, best);
        consider(s1, 209 + 2 * r, best);
    }
    if (mode_mask & 0x20) {
        uint32_t s5 = fit_colour<7, 0, 2, true>(S, full, r, P, sv).sse;
        if (r) s5 += fit_scalar<8, 2, false>(S, r, sv).sse;
        consider(s5, 216 + r, best);
    }
    return best;
}

// mode 6
__device__ __forceinline__ uint32_t search_mode6(const TexLds &S, const uint32_t *sv)
{
    const uint32_t full = all_texels();
    const Prep P = prep_subset(S, full, 0);
    return (fit_colour<7, 2, 4, true>(S, full, 0, P, sv).sse << 9) | 220u;
}

// ---- pass 2: re-fit the winner (same arithmetic) and lay out its bits
struct Writer {
    uint64_t lo = 0, hi = 0;
    int pos = 0;
    __device__ void put(uint32_t v, int n)
    {
        uint64_t x = (uint64_t)v & ((1ull << n) - 1);
        if (pos >= 64) hi |= x << (pos - 64);
        else {
            lo |= x << pos;
            if (pos + n > 64) hi |= x >> (64 - pos);
        }
        pos += n;
    }
};

template <int M, int CB, int PB, int NB>
__device__ void emit_partitioned(const TexLds &S, int p, const uint32_t *sv, Writer &w)
{
    constexpr Bc7Mode md = bc7_mode(M);
    constexpr int NS = md.ns;
    PairFit f[NS];
    uint32_t msk[NS];
    int anc[NS];
#pragma unroll
    for (int s = 0; s < NS; s++) {
        msk[s] = NS == 3 ? mask3(p, s) : mask2(p, s);
        anc[s] = bc7_anchor(NS, p, s);
        const Prep P = prep_subset(S, msk[s], 0);
        f[s] = fit_colour<CB, PB, NB>(S, msk[s], 0, P, sv);
        anchor_fix<NB>(f[s], msk[s], anc[s]);
    }
    w.put(1u << M, M + 1);
    w.put((uint32_t)p, md.partbits);
#pragma unroll
    for (int c = 0; c < 3; c++)
#pragma unroll
        for (int s = 0; s < NS; s++) { w.put(f[s].c0 >> (8 * c), CB); w.put(f[s].c1 >> (8 * c), CB); }
    if (md.ab)   // alpha is not coded for these colour blocks: all-ones fields
#pragma unroll
        for (int s = 0; s < NS; s++) { w.put((1u << md.ab) - 1, md.ab); w.put((1u << md.ab) - 1, md.ab); }
    if (PB == 2)
#pragma unroll
        for (int s = 0; s < NS; s++) { w.put(f[s].p0, 1); w.put(f[s].p1, 1); }
    else if (PB == 1)
#pragma unroll
        for (int s = 0; s < NS; s++) w.put(f[s].p0, 1);
    // members' indices live in their own subset's fit: merge them
    uint64_t idx = 0;
#pragma unroll
    for (int s = 0; s < NS; s++) {
        uint64_t sel = 0;
        for (uint32_t m = msk[s]; m; m &= m - 1) sel |= (uint64_t)15 << (4 * (__ffs(m) - 1));
        idx |= f[s].idx & sel;
    }
#pragma unroll
    for (int i = 0; i < 16; i++) {
        bool anchored = false;
#pragma unroll
        for (int q = 0; q < NS; q++) anchored |= anc[q] == i;
        w.put((uint32_t)((idx >> (4 * i)) & 15), NB - (anchored ? 1 : 0));
    }
}

// Modes 4 and 5: one colour pair plus a scalar pair, rotation r.
template <int M, int CB, int AB, int CNB, int SNB>
__device__ void emit_rotated(const TexLds &S, int r, int sel, const uint32_t *sv, Writer &w)
{
    const uint32_t full = all_texels();
    const Prep P = prep_subset(S, full, r);
    PairFit fc = fit_colour<CB, 0, CNB>(S, full, r, P, sv);
    anchor_fix<CNB>(fc, 0xFFFFu, 0);
    PairFit fs = fit_scalar<AB, SNB, true>(S, r, sv);
    anchor_fix<SNB>(fs, 0xFFFFu, 0);
    w.put(1u << M, M + 1);
    w.put((uint32_t)r, 2);
    if (M == 4) w.put((uint32_t)sel, 1);
#pragma unroll
    for (int c = 0; c < 3; c++) { w.put(fc.c0 >> (8 * c), CB); w.put(fc.c1 >> (8 * c), CB); }
    w.put(fs.c0, AB);
    w.put(fs.c1, AB);
    // primary index set (2 bits) first, then the secondary set; index
    // selection 1 stores the scalar indices in the primary set
    const uint64_t first = (M == 4 && sel) ? fs.idx : fc.idx;
    const uint64_t second = (M == 4 && sel) ? fc.idx : fs.idx;
    constexpr int NB1 = 2, NB2 = (M == 4) ? 3 : 2;
#pragma unroll
    for (int i = 0; i < 16; i++) w.put((uint32_t)((first >> (4 * i)) & 15), NB1 - (i == 0));
#pragma unroll
    for (int i = 0; i < 16; i++) w.put((uint32_t)((second >> (4 * i)) & 15), NB2 - (i == 0));
}

// Bits of a winning candidate of mode M.
template <int M>
__device__ __forceinline__ void emit(const TexLds &S, int ci, const uint32_t *sv, uint64_t &lo, uint64_t &hi)
{
    int m, p, r, s;
    candidate(ci, m, p, r, s);
    Writer w;
    if (M == 0) emit_partitioned<0, 4, 2, 3>(S, p, sv, w);
    else if (M == 1) emit_partitioned<1, 6, 1, 3>(S, p, sv, w);
    else if (M == 2) emit_partitioned<2, 5, 0, 2>(S, p, sv, w);
    else if (M == 3) emit_partitioned<3, 7, 2, 2>(S, p, sv, w);
    else if (M == 4) {
        if (s == 0) emit_rotated<4, 5, 6, 2, 3>(S, r, 0, sv, w);
        else emit_rotated<4, 5, 6, 3, 2>(S, r, 1, sv, w);
    } else if (M == 5) emit_rotated<5, 7, 8, 2, 2>(S, r, 0, sv, w);
    else if (M == 6) {
        const uint32_t full = all_texels();
        const Prep P = prep_subset(S, full, 0);
        PairFit f = fit_colour<7, 2, 4>(S, full, 0, P, sv);
        anchor_fix<4>(f, 0xFFFFu, 0);
        w.put(1u << 6, 7);
#pragma unroll
        for (int c = 0; c < 3; c++) { w.put(f.c0 >> (8 * c), 7); w.put(f.c1 >> (8 * c), 7); }
        w.put(127, 7); w.put(127, 7);   // alpha not coded: all-ones fields
        w.put(f.p0, 1); w.put(f.p1, 1);
#pragma unroll
        for (int i = 0; i < 16; i++) w.put((uint32_t)((f.idx >> (4 * i)) & 15), 4 - (i == 0));
    } else emit_partitioned<7, 5, 2, 2>(S, p, sv, w);
    lo = w.lo;
    hi = w.hi;
}

struct Bc7Launch {
    EncodeArgs a;
    Tables T;
};

// The nearest-code table into LDS: 64-scaled values for the search,
// code | value << 8 for the emit pass.
__device__ __forceinline__ void stage_table(TexLds &S, const uint16_t *table)
{
    for (int q = threadIdx.x; q < kQEntries / 2; q += kWG)
        reinterpret_cast<uint32_t *>(S.q)[q] = reinterpret_cast<const uint32_t *>(table)[q];
}

// This lane's block (zeros when not live) into its LDS column in the -8
// scaled layout.  The caller brackets it with barriers.
__device__ __forceinline__ void stage_texels(TexLds &S, const uint8_t *src, bool live)
{
    uint32_t t[16];
#pragma unroll
    for (int i = 0; i < 16; i++) t[i] = 0;
    if (live) {
        const uint4 *p = reinterpret_cast<const uint4 *>(src);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            uint4 v = p[q];
            t[4 * q] = v.x; t[4 * q + 1] = v.y; t[4 * q + 2] = v.z; t[4 * q + 3] = v.w;
        }
    }
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const int r = (int)(t[i] & 255u), g = (int)((t[i] >> 8) & 255u), bb = (int)((t[i] >> 16) & 255u);
        S.rg[i][threadIdx.x] = ((uint32_t)(kScaleNeg * r) & 0xFFFFu) | ((uint32_t)(kScaleNeg * g) << 16);
        S.bx[i][threadIdx.x] = (int16_t)(kScaleNeg * bb);
    }
}

// Items handled by this workgroup: one (its own index) without a queue,
// else popped from the queue until exhausted.  Every workgroup leaves the
// loop once the counter passes the last item.
struct ItemLoop {
    uint32_t item, n_items;
    __device__ __forceinline__ ItemLoop(const WorkSplit &w, uint32_t items, uint32_t *s_item)
    {
        n_items = items;
        item = blockIdx.x;
        if (w.queue) {
            if (threadIdx.x == 0) *s_item = atomicAdd(w.queue, 1u);
            __syncthreads();
            item = *s_item;
        }
    }
    __device__ __forceinline__ bool next(const WorkSplit &w, uint32_t *s_item)
    {
        if (!w.queue) return false;
        __syncthreads();   // every thread has read *s_item
        if (threadIdx.x == 0) *s_item = atomicAdd(w.queue, 1u);
        __syncthreads();
        item = *s_item;
        return item < n_items;
    }
};

// ---- pass 1: search
//
// Almost all of the 285 candidates of a block can be ruled out without being
// fitted.  A palette lies near a line: whatever the endpoints, its entries
// are within kCheb of some straight line in every channel (the line through
// the rounded interpolants, see kCheb), so a subset of n texels whose summed
// squared distance to its own best line is R has
//     SSE >= (max(0, sqrt(R) - sqrt(3 kCheb^2 n)))^2
// (the triangle inequality on the members' distances).
// R is the trace of the subset's scatter matrix less its largest eigenvalue.
// A candidate whose bound is above the SSE of a candidate already fitted
// cannot win (nor tie), so it is left out; the others are fitted exactly as
// before, and the winner is the same.  Three kernels:
//   bounds  the member sums of every subset of the 64 + 64 partitions as
//           matrix products (0/1 masks times texel features) on the matrix
//           cores, from them each candidate's bound (16 bits, rounded down),
//           and the least bound of the 3-subset partitions and rotations;
//   seed    fits those two per block (they win or come within 2 % of the
//           winner on most blocks) and compares every bound with their SSE:
//           one 64-bit word per (64 blocks, candidate) says which blocks are left;
//   search  one wave per (candidate, window of blocks): the blocks left are
//           taken 64 at a time, one per lane, whatever their places in the
//           window, so the fits run on full waves with wave-uniform masks.
//           Each is tested again against the block's best so far, and once
//           more when the partition's largest subset is fitted (its SSE and
//           the bounds of the others); the blocks still left are gathered to
//           full waves again for the other subsets.
// On 1,048,576 primitives of synthetic SH bands 2-3 of 64 2-subset
// partitions, 20 of 64 3-subset ones (mode 2), 6 of 16 (mode 0) and 2 of 4
// rotations are left in bands 1-15, twice to eight times as many in the
// smooth band 0; half to 85 % of those stop at their largest subset.  VALU
// instructions per 64 blocks: bounds 28 k, seeds 13 k, search 79 k (735 k for
// an exhaustive search); 1,048,576 blocks: 16.5 ms exhaustive, 4.2 ms now.

// Largest deviation, in one channel, of a rounded palette from the straight
// line nearest to it: entry k is e0 + floor((w_k D + 32)/64) with D = e1 - e0,
// so the deviations depend on D mod 64 only; the minimax line fit over all
// 64 residues gives 0.3605 (2-bit indices), 0.4474 (3) and 0.4706 (4).
// sqrt(3) times that, rounded up, is the slack of a member of three channels
// (sqrt(2): one channel constant, as rotations leave it; modes 1, 3, 7 and
// modes 4, 5 share the larger slack of 3-bit indices):
constexpr float kSlack2 = 0.6245f, kSlack3 = 0.7750f, kSlack4 = 0.8152f;
constexpr float kSlackRot = 0.6328f;

// sqrt of 16 R of a block whose texels lie so near a line (R up to 12) that its
// bounds come out below 1 (coded as 0) or little above: sixteen such blocks go
// without.  What bounds and gathers do not have to do on blocks of two adjacent
// levels: 1,048,576 of them 18.97 -> 17.84 ms (17.19 exhaustive).
constexpr float kFlatRoot = 13.86f;

// Candidate words of a slice (64 blocks), per type.
constexpr int kWordAt[kTypes + 1] = {0, 64, 80, 144, 148, 149};
constexpr int kWords = 149;
constexpr int kTiles = 13;   // 16-row mask tiles: 4 of 2-subset masks, 8 of 3-subset masks, all ones

// Bounds of a chunk of blocks (nc of them: the scratch of a large encode stays
// at 167 MB), 16 bits each:
//   b2[16][nc] 4 partitions, b3[32][nc] 2 partitions, b0[8][nc] 2, br[nc] 4 rotations,
//   seed[nc]: least 3-subset partition | least rotation << 8 | mode 6's bound << 16
struct Bounds {
    uint2 *b2;
    uint32_t *b3, *b0;
    uint2 *br;
    uint32_t *seed;
    uint64_t nc;
};

struct Bc7Search {
    EncodeArgs a;
    Tables T;
    WorkSplit w;
    uint64_t first;             // first block of the chunk
    uint32_t slices;            // slices of the chunk
    Bounds B;
    uint64_t *words;            // [slice][kWords]
    uint32_t *dense;            // slices that k_bc7_every takes: their number, then a list; or null
    const uint8_t **src;        // [slice] texels of the slice's first block
    uint32_t win[kTypes];       // search: slices per window, per type
    uint32_t types;             // search: candidate types of this launch, bit per type
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// A bound v >= 0 as 16 bits (5 of exponent, 11 of fraction), rounded down;
// below 1 it is 0.  Monotone, so a candidate is left out only if its bound
// exceeds the SSE coded the same way.
__device__ __forceinline__ uint32_t bound16(float v)
{
    return (uint32_t)max(__float_as_int(v) - (127 << 23), 0) >> 12;
}
__device__ __forceinline__ float bound_value(uint32_t b) { return b ? __int_as_float((int)(b << 12) + (127 << 23)) : 0.0f; }

// sqrt of n R for a subset of n members with sums S = (x, y, z, xx, xy, xz,
// yy, yz, zz), from below.  n XX - Sx Sx^T is exact in FP32 (integers below
// 2^24).  Its largest eigenvalue is q + 2 p f with f the largest root of
// 4 f^3 - 3 f = hr (the trigonometric solution), found by one Newton step
// from a fit within 0.004; the step lands above the root (the cubic is
// convex there), and the margins cover the rounding of hr, whose effect on f
// grows to sqrt(rounding) where the two largest eigenvalues meet.
__device__ __forceinline__ float residual_root(float n, const float (&S)[9])
{
    const float cxx = fmaf(n, S[3], -S[0] * S[0]), cxy = fmaf(n, S[4], -S[0] * S[1]), cxz = fmaf(n, S[5], -S[0] * S[2]);
    const float cyy = fmaf(n, S[6], -S[1] * S[1]), cyz = fmaf(n, S[7], -S[1] * S[2]), czz = fmaf(n, S[8], -S[2] * S[2]);
    const float tr = cxx + cyy + czz, q = tr * (1.0f / 3.0f);
    const float a = cxx - q, b = cyy - q, c = czz - q;
    const float off = fmaf(cxy, cxy, fmaf(cxz, cxz, cyz * cyz));
    const float p2 = fmaxf(fmaf(2.0f, off, fmaf(a, a, fmaf(b, b, c * c))) * (1.0f / 6.0f), 1e-3f);
    const float det = fmaf(a, fmaf(b, c, -cyz * cyz),
                           fmaf(-cxy, fmaf(cxy, c, -cyz * cxz), cxz * fmaf(cxy, cyz, -b * cxz)));
    const float ip = __builtin_amdgcn_rsqf(p2), p = p2 * ip;
    const float hr = fminf(fmaxf(0.5f * det * ip * ip * ip, -1.0f), 1.0f);
    const float s = __builtin_amdgcn_sqrtf(fmaf(0.5f, hr, 0.5f));
    const float f0 = fmaf(s, fmaf(s, -0.0774f, 0.5774f), 0.5f);
    const float f2 = f0 * f0;
    const float num = fmaf(f0, fmaf(4.0f, f2, -3.0f), -hr), den = fmaxf(fmaf(12.0f, f2, -3.0f), 1e-3f);
    const float f = fmaf(-num, __builtin_amdgcn_rcpf(den), f0) + 5e-4f;
    const float lam = fmaf(2.0f * p, f, q * 1.0001f);
    return __builtin_amdgcn_sqrtf(fmaxf(tr - lam, 0.0f));
}

// (max(0, sqrt(R) - c sqrt(n)))^2 from root = sqrt(n R)
__device__ __forceinline__ float bound_term(float root, float n, float rn, float c)
{
    const float d = fmaxf(fmaf(-c, n, root), 0.0f);
    return d * d * rn;
}

// Row i of mask tile t (see kTiles): 2-subset partition 16 t + i; or of the
// 3-subset tile t - 4, partition 8 (t - 4) + i/2, subset 1 + i%2 (subset 0 is
// what the block's total leaves); or all texels.
__device__ __forceinline__ uint32_t tile_mask(int t, int i)
{
    if (t < 4) return kPart2[16 * t + i];
    if (t < 12) return mask3(8 * (t - 4) + (i >> 1), 1 + (i & 1));
    return 0xFFFFu;
}

// Where a block's first fits come from, by the modes that are on.  Usually the
// best-bounded 3-subset partition in mode 2 and the best-bounded rotation.
// Without modes 2, 4 and 5 the best-bounded 2-subset partition, or mode 0's.
// With one-subset modes only, every candidate is fitted and nothing bounded:
// 13 at most, and the bounds cost as much as a few (1,048,576 blocks in mode 6
// alone: 1,999 us bounded and gathered, 544 fitted; without a first fit that
// rules others out mode 0 alone takes 4,390 us, with one 1,117; mode 1 8,650 and
// 1,141; exhaustive 2,213 and 5,408).
enum { kSeedUsual, kSeedOther, kSeedEvery };
__host__ __device__ inline int seed_kind(uint32_t mode_mask)
{
    return !(mode_mask & 0x8F) ? kSeedEvery : mode_mask & 0x34 ? kSeedUsual : kSeedOther;
}

// With partitions of one shape only, slices whose blocks keep this share (%) of
// the candidates after the first fits have them all fitted in order instead: the
// gathers and the masks fitted more than once cost more than the little that is
// ruled out saves (1,048,576 blocks along gradients in mode 2 5.6 -> 4.1 ms, in
// mode 1 7.7 -> 6.3; exhaustive 3.2 and 5.4).  With both shapes the second test
// rules out more than that (all modes 16.6 -> 18.7 ms).
constexpr uint32_t kDense = 85;

// Bounds of every candidate of the modes that are on.  A wave takes 16 blocks
// at a time: with v_mfma_f32_16x16x32_bf16, lane l supplies row l%16 of A (a mask) and
// column l%16 of B (a block's texel feature) for k = 8 (l/16) .. + 7, and
// receives rows 4 (l/16) .. + 3 of column l%16: four subsets of one block,
// every feature of them in the same lane.  k < 16 are the texels' values or
// their products' low bytes, k >= 16 the products' high bytes against masks
// scaled by 256 (8-bit integers are exact in bf16, the sums in FP32).
// A workgroup takes `per` blocks, 256 or, when they are few, 64 (one step of
// 16 blocks a wave instead of four: 4,112 blocks 68 -> 22 us).
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(3))) void k_bc7_bounds(Bc7Search L, uint32_t per)
{
    __shared__ uint4 tile[kTiles][64];
    __shared__ uint32_t count[12][4];      // members of rows 4 g .. 4 g + 3, one byte each
    for (int e = threadIdx.x; e < kTiles * 64; e += kWG) {
        const int l = e & 63;
        const uint32_t m = tile_mask(e >> 6, l & 15) >> (8 * ((l >> 4) & 1)), one = l < 32 ? 0x3F80u : 0x4380u;
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; j++) w[j] = ((m >> (2 * j)) & 1u ? one : 0u) | ((m >> (2 * j + 1)) & 1u ? one << 16 : 0u);
        tile[e >> 6][l] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    if (threadIdx.x < 48) {
        uint32_t c = 0;
        for (int r = 0; r < 4; r++) c |= (uint32_t)__popc(tile_mask(threadIdx.x >> 2, 4 * (threadIdx.x & 3) + r)) << (8 * r);
        count[threadIdx.x >> 2][threadIdx.x & 3] = c;
    }
    __syncthreads();
    const EncodeArgs &a = L.a;
    const bool on2 = a.mode_mask & 0x8A, other = seed_kind(a.mode_mask) == kSeedOther;
    const int tiles3 = a.mode_mask & 0x04 ? 8 : a.mode_mask & 0x01 ? 2 : 0;   // mode 0 has 16 partitions
    const int lane = threadIdx.x & 63, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t c0 = (uint64_t)blockIdx.x * per, g0 = L.first + c0;   // a workgroup lies in one run
    const BlockRun run = a.run[find_run(a.run, a.nrun, g0)];
    const uint64_t b0 = g0 - run.gbase;
    if (threadIdx.x < per / 64) L.src[(c0 >> 6) + threadIdx.x] = run.src + (b0 + 64 * threadIdx.x) * 64;
    if (L.dense && blockIdx.x == 0 && threadIdx.x == 0) L.dense[0] = 0;
    const uint32_t sh = lane < 32 ? 0u : 8u, lin = lane < 32 ? 0xFFu : 0u;
    for (uint32_t sb = wave; sb < per / 16; sb += kWG / 64) {
        const uint64_t b = b0 + 16 * sb + (lane & 15), c = c0 + 16 * sb + (lane & 15);
        // eight texels of the lane's block (the run's last block stands in past its end)
        const uint4 *src = reinterpret_cast<const uint4 *>(run.src + min(b, run.nblk - 1) * 64 + 32 * (grp & 1));
        const uint4 v0 = src[0], v1 = src[1];
        const uint32_t px[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        bf16x8 B[9];
        {
            uint32_t w[9][4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                uint32_t f[2][9];
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    const uint32_t t = px[2 * j + h], r = t & 255u, g = (t >> 8) & 255u, bl = (t >> 16) & 255u;
                    const uint32_t pr[6] = {mul_u24(r, r), mul_u24(r, g), mul_u24(r, bl), mul_u24(g, g), mul_u24(g, bl), mul_u24(bl, bl)};
                    f[h][0] = __float_as_uint((float)(r & lin));
                    f[h][1] = __float_as_uint((float)(g & lin));
                    f[h][2] = __float_as_uint((float)(bl & lin));
#pragma unroll
                    for (int q = 0; q < 6; q++) f[h][3 + q] = __float_as_uint((float)((pr[q] >> sh) & 255u));
                }
                // the top halves of two FP32 values (exact: 8-bit integers)
#pragma unroll
                for (int q = 0; q < 9; q++) w[q][j] = __builtin_amdgcn_perm(f[1][q], f[0][q], 0x07060302u);
            }
#pragma unroll
            for (int q = 0; q < 9; q++) B[q] = __builtin_bit_cast(bf16x8, make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]));
        }
        auto sums = [&](int t, floatx4 (&D)[9]) {
            const bf16x8 A = __builtin_bit_cast(bf16x8, tile[t][lane]);
#pragma unroll
            for (int q = 0; q < 9; q++)
                D[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B[q], floatx4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
        };
        floatx4 D[9];
        sums(12, D);
        float tot[9];
#pragma unroll
        for (int q = 0; q < 9; q++) tot[q] = D[q][0];
        // one subset: lane group r takes rotation r (its channel is constant)
        bool flat;
        {
            float m[9];
            const float kr = grp == 1 ? 0.0f : 1.0f, kg = grp == 2 ? 0.0f : 1.0f, kb = grp == 3 ? 0.0f : 1.0f;
            m[0] = tot[0] * kr; m[1] = tot[1] * kg; m[2] = tot[2] * kb;
            m[3] = tot[3] * kr; m[4] = tot[4] * (kr * kg); m[5] = tot[5] * (kr * kb);
            m[6] = tot[6] * kg; m[7] = tot[7] * (kg * kb); m[8] = tot[8] * kb;
            const float root = residual_root(16.0f, m);
            const uint32_t lb = bound16(bound_term(root, 16.0f, 1.0f / 16.0f, grp ? kSlackRot : kSlack3));
            reinterpret_cast<uint16_t *>(L.B.br)[4 * c + grp] = (uint16_t)lb;
            uint32_t least = lb << 8 | (uint32_t)grp;
            least = min(least, (uint32_t)__shfl_xor((int)least, 16));
            least = min(least, (uint32_t)__shfl_xor((int)least, 32));
            // (mode 6 is rotation 0's subset: lane group 0)
            const uint32_t lb6 = bound16(bound_term(root, 16.0f, 1.0f / 16.0f, kSlack4));
            if (grp == 0) L.B.seed[c] = (least & 255u) << 8 | lb6 << 16;
            flat = __all(grp || root <= kFlatRoot);
        }
        if (flat) {   // every bound 0: sixteen blocks that no bound would rule anything out of
            for (int t = 0; t < (on2 ? 4 : 0); t++) L.B.b2[(uint64_t)(4 * t + grp) * L.B.nc + c] = make_uint2(0u, 0u);
            for (int t = 0; t < tiles3; t++) {
                L.B.b3[(uint64_t)(4 * t + grp) * L.B.nc + c] = 0u;
                if (t < 2) L.B.b0[(uint64_t)(4 * t + grp) * L.B.nc + c] = 0u;
            }
            continue;   // (the seed's partition is 0)
        }
        // 2-subset partitions: rows are subset 1, the total less them subset 0
        uint32_t least = ~0u;
#pragma unroll 1
        for (int t = 0; t < (on2 ? 4 : 0); t++) {
            sums(t, D);
            const uint32_t cnt = count[t][grp];
            uint32_t lb[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float n1 = (float)((cnt >> (8 * r)) & 255u), n0 = 16.0f - n1;
                float s1[9], s0[9];
#pragma unroll
                for (int q = 0; q < 9; q++) { s1[q] = D[q][r]; s0[q] = tot[q] - s1[q]; }
                lb[r] = bound16(bound_term(residual_root(n1, s1), n1, __builtin_amdgcn_rcpf(n1), kSlack3) +
                                bound_term(residual_root(n0, s0), n0, __builtin_amdgcn_rcpf(n0), kSlack3));
            }
            L.B.b2[(uint64_t)(4 * t + grp) * L.B.nc + c] = make_uint2(lb[0] | lb[1] << 16, lb[2] | lb[3] << 16);
            if (other)
#pragma unroll
                for (int r = 0; r < 4; r++) least = min(least, lb[r] << 8 | (uint32_t)(16 * t + 4 * grp + r));
        }
        // 3-subset partitions: two rows each
#pragma unroll 1
        for (int t = 0; t < tiles3; t++) {
            sums(4 + t, D);
            const uint32_t cnt = count[4 + t][grp];
            uint32_t lb[2], lb0[2];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const float n1 = (float)((cnt >> (16 * h)) & 255u), n2 = (float)((cnt >> (16 * h + 8)) & 255u);
                const float n0 = 16.0f - n1 - n2;
                float s0[9], s1[9], s2[9];
#pragma unroll
                for (int q = 0; q < 9; q++) { s1[q] = D[q][2 * h]; s2[q] = D[q][2 * h + 1]; s0[q] = tot[q] - s1[q] - s2[q]; }
                const float r0 = residual_root(n0, s0), r1 = residual_root(n1, s1), r2 = residual_root(n2, s2);
                const float q0 = __builtin_amdgcn_rcpf(n0), q1 = __builtin_amdgcn_rcpf(n1), q2 = __builtin_amdgcn_rcpf(n2);
                lb[h] = bound16(bound_term(r0, n0, q0, kSlack2) + bound_term(r1, n1, q1, kSlack2) + bound_term(r2, n2, q2, kSlack2));
                lb0[h] = bound16(bound_term(r0, n0, q0, kSlack3) + bound_term(r1, n1, q1, kSlack3) + bound_term(r2, n2, q2, kSlack3));
                if (!(other && on2)) least = min(least, (other ? lb0[h] : lb[h]) << 8 | (uint32_t)(8 * t + 2 * grp + h));
            }
            L.B.b3[(uint64_t)(4 * t + grp) * L.B.nc + c] = lb[0] | lb[1] << 16;
            if (t < 2) L.B.b0[(uint64_t)(4 * t + grp) * L.B.nc + c] = lb0[0] | lb0[1] << 16;
        }
        least = min(least, (uint32_t)__shfl_xor((int)least, 16));
        least = min(least, (uint32_t)__shfl_xor((int)least, 32));
        if (grp == 0) L.B.seed[c] |= least & 255u;
    }
}

// Seeds, and the words of the blocks each candidate is left with: lane =
// block.  Where blocks are few (`pairs`), two waves share 64 blocks: one
// fits the 3-subset seed and writes the words of the 3-subset partitions, the
// other the rotation seed and the other words (4,112 blocks: 76 -> 57 us;
// 524,288 blocks: 205 -> 250 us, where a wave does both).  The seeds' own bits
// are cleared (they are fitted here).  SEEDS: see seed_kind.  DENSE: slices to be
// fitted in order are listed.
template <int SEEDS, bool DENSE>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(SEEDS == kSeedUsual ? 4 : 3))) void k_bc7_seed(Bc7Search L, bool pairs)
{
    __shared__ TexLds S;
    __shared__ uint32_t s_key[4][64];
    const EncodeArgs &a = L.a;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool parts = !pairs || (wave & 1), others = !pairs || !(wave & 1);
    const uint64_t c0 = (uint64_t)blockIdx.x * (pairs ? kWG / 2 : kWG), g0 = L.first + c0;
    const uint64_t c = c0 + 64 * (pairs ? wave >> 1 : wave) + lane, g = L.first + c;
    const BlockRun run = a.run[find_run(a.run, a.nrun, g0)];
    const uint64_t b = g - run.gbase;
    const bool live = b < run.nblk;
    stage_table(S, L.T.near64);
    stage_texels(S, run.src + b * 64, live);
    __syncthreads();
    // a block of one colour has the same SSE in every partition of a mode
    bool one = live;
#pragma unroll
    for (int i = 1; i < 16; i++) one &= S.rg[i][threadIdx.x] == S.rg[0][threadIdx.x] && S.bx[i][threadIdx.x] == S.bx[0][threadIdx.x];
    const bool on2 = a.mode_mask & 0x8A;
    const uint32_t seed = SEEDS == kSeedEvery ? 0u : L.B.seed[c];
    // the seeds: a 3-subset partition, a 2-subset partition, a rotation (-1: none)
    const int p = one ? 0 : (int)(seed & 255u);
    const int p3 = SEEDS == kSeedUsual || !on2 ? p : -1, p2 = SEEDS == kSeedOther && on2 ? p : -1;
    const int rot = SEEDS == kSeedUsual ? (int)((seed >> 8) & 255u) : -1;
    uint32_t key = ~0u;
    if (SEEDS == kSeedEvery && live) {
        if (a.mode_mask & 0x30)
#pragma unroll 1
            for (int r = parts ? 0 : 2; r < (others ? 4 : 2); r++) key = min(key, search_rotation(S, r, a.mode_mask, L.T.sv));
        if (others && (a.mode_mask & 0x40)) key = min(key, search_mode6(S, L.T.sv));
    }
    if (SEEDS == kSeedOther && live) {
        uint32_t e[3] = {a.mode_mask & 0x02 ? 0u : kGone, a.mode_mask & 0x08 ? 0u : kGone, a.mode_mask & 0x80 ? 0u : kGone};
        if (on2 && others) {
#pragma unroll 1
            for (int s = 0; s < 2; s++) {
                const uint32_t m = mask2(p2, s);
                add_subset<kTwo>(S, m, subset_sums(S, m, 0), L.T.sv, e);
            }
            key = partition_key<kTwo>(p2, e);
        }
        if (!on2 && parts) {
            e[0] = 0;
#pragma unroll 1
            for (int s = 0; s < 3; s++) {
                const uint32_t m = mask3(p3, s);
                add_subset<kThree0>(S, m, subset_sums(S, m, 0), L.T.sv, e);
            }
            key = partition_key<kThree0>(p3, e);
        }
    }
    if (SEEDS == kSeedUsual && live) {
        if (parts) {
            if (a.mode_mask & 0x04) {
                uint32_t e[3] = {0, 0, 0};
#pragma unroll 1
                for (int s = 0; s < 3; s++) {
                    const uint32_t m = mask3(p3, s);
                    add_subset<kThree2>(S, m, subset_sums(S, m, 0), L.T.sv, e);
                }
                key = partition_key<kThree2>(p3, e);
            }
        }
        if (others && (a.mode_mask & 0x30)) key = min(key, search_rotation(S, rot, a.mode_mask, L.T.sv));
    }
    if (pairs) {
        s_key[wave][lane] = key;
        __syncthreads();
        key = min(key, s_key[wave ^ 1][lane]);
    }
    if (parts) a.keys[g] = key;
    if (SEEDS == kSeedEvery) return;
    // 0 .. thr: bounds that may still win (with no seed, all of them; past the
    // run, none; only partition 0 of a block of one colour)
    const int thr = !live ? -1 : key == ~0u ? 0xFFFF : (int)bound16((float)(key >> 9));
    const int thrp = one ? -1 : thr;   // of partitions from 1
    uint64_t w0 = 0, w1 = 0;           // lane p's words
    auto put = [&](uint64_t &w, int at, bool keep) {
        const uint64_t m = __ballot(keep);
        if (lane == at) w = m;
    };
    uint64_t *words = L.words + (c >> 6) * kWords;
    // (only the words of modes that are on: their bounds are there, and the search reads no others)
    const int p0 = SEEDS == kSeedOther ? p3 : -1;   // mode 0's seed
    if (SEEDS == kSeedUsual && parts && (a.mode_mask & 0x04)) {
#pragma unroll 4
        for (int q = 0; q < 32; q++) {
            const uint32_t v = L.B.b3[q * L.B.nc + c];
            put(w0, 2 * q, (int)(v & 0xFFFFu) <= (q ? thrp : thr) && p3 != 2 * q);
            put(w0, 2 * q + 1, (int)(v >> 16) <= thrp && p3 != 2 * q + 1);
        }
    }
    if (parts && (a.mode_mask & 0x01)) {
#pragma unroll 4
        for (int q = 0; q < 8; q++) {
            const uint32_t v = L.B.b0[q * L.B.nc + c];
            put(w1, 2 * q, (int)(v & 0xFFFFu) <= (q ? thrp : thr) && (SEEDS == kSeedUsual || p0 != 2 * q));
            put(w1, 2 * q + 1, (int)(v >> 16) <= thrp && (SEEDS == kSeedUsual || p0 != 2 * q + 1));
        }
    }
    // slices most of whose blocks keep most partitions go to k_bc7_every
    auto is_dense = [&](uint64_t u, uint64_t v, uint32_t cands) {
        if (!DENSE) return false;
        uint32_t n = (uint32_t)__popcll(u) + (uint32_t)__popcll(v);
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) n += (uint32_t)__shfl_xor((int)n, d);
        if (n * 100u < 64u * cands * kDense) return false;
        if (lane == 0) L.dense[4 + atomicAdd(L.dense, 1u)] = (uint32_t)(c >> 6);
        return true;
    };
    if (parts && (a.mode_mask & 0x05)) {
        const uint32_t cands = (a.mode_mask & 0x04 ? 64u : 0u) + (a.mode_mask & 0x01 ? 16u : 0u);
        if (is_dense(w0, w1, cands)) w0 = w1 = 0;
        if (SEEDS == kSeedUsual && (a.mode_mask & 0x04)) words[kWordAt[kThree2] + lane] = w0;
        if ((a.mode_mask & 0x01) && lane < 16) words[kWordAt[kThree0] + lane] = w1;
    }
    if (others) {
        if (on2) {
#pragma unroll 4
            for (int q = 0; q < 16; q++) {
                const uint2 v = L.B.b2[q * L.B.nc + c];
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const uint32_t lb = ((r < 2 ? v.x : v.y) >> (16 * (r & 1))) & 0xFFFFu;
                    put(w0, 4 * q + r, (int)lb <= (q + r ? thrp : thr) && (SEEDS == kSeedUsual || p2 != 4 * q + r));
                }
            }
            if (is_dense(w0, 0, 64)) w0 = 0;
            words[kWordAt[kTwo] + lane] = w0;
        }
        const uint2 vr = L.B.br[c];
#pragma unroll
        for (int r = 0; r < 4; r++)
            put(w1, r, (int)(((r < 2 ? vr.x : vr.y) >> (16 * (r & 1))) & 0xFFFFu) <= thr && rot != r);
        put(w1, 4, (int)(seed >> 16) <= thr);
        if (lane < 5) words[kWordAt[kRot] + lane] = w1;
    }
}

// Slices that the seeds found dense, where one shape of partition is on: every
// partition, one lane per block, the texels staged once.
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(3))) void k_bc7_every(Bc7Search L)
{
    __shared__ TexLds S;
    __shared__ Cache3 cache;
    const uint32_t n = L.dense[0], at = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.x * 4 >= n) return;
    stage_table(S, L.T.near64);
    const uint32_t slice = L.dense[4 + min(at, n - 1)];
    const uint64_t g0 = L.first + (uint64_t)slice * 64, g = g0 + (threadIdx.x & 63u);
    const BlockRun run = L.a.run[find_run(L.a.run, L.a.nrun, g0)];
    const uint64_t b = g - run.gbase;
    const bool live = at < n && b < run.nblk;
    stage_texels(S, run.src + b * 64, live);
    __syncthreads();
    if (live)
        atomicMin(L.a.keys + g, L.a.mode_mask & 0x8A ? search_every<false>(S, cache, L.a.mode_mask, L.T.sv)
                                                     : search_every<true>(S, cache, L.a.mode_mask, L.T.sv));
}

// Bit k (from 0) among the set bits of w.
__device__ __forceinline__ int nth_bit(uint64_t w, int k)
{
    uint32_t x = (uint32_t)w;
    int at = 0, n = __popc(x);
    if (k >= n) { k -= n; x = (uint32_t)(w >> 32); at = 32; }
#pragma unroll
    for (int s = 16; s; s >>= 1) {
        n = __popc(x & ((1u << s) - 1u));
        if (k >= n) { k -= n; x >>= s; at += s; }
    }
    return at;
}

// Items of a search launch, type after type: (window, candidate) pairs, a
// window's candidates next to each other (its texels stay in L2).  The
// longest items come early: with mode 2 first, which lowers most blocks' best
// for the types after it, the launch ended on the 2-subset items of a dense
// window (5.41 ms at 1,048,576 blocks against 4.52).  Before them only mode 6,
// which few blocks keep unless their colours lie along a line, where it
// lowers the best at once (1,048,576 such blocks 19.6 -> 15.4 ms).
struct Items {
    uint32_t n[kTypes];
    uint32_t total;
};
template <int T>
struct Type { static constexpr int value = T; };
__host__ __device__ constexpr uint32_t per_window(int type) { return (uint32_t)(kWordAt[type + 1] - kWordAt[type]); }
// Workgroups go to the chip's eight XCDs in turn, each with an L2 of its own.
// From 131,072 blocks on, window w's items are those of XCD w % 8 (windows
// padded to eights), so that its texels are fetched into one L2 instead of
// all (BC7 of 1,048,576 blocks 4.51 -> 4.46 ms, a batch of 16 scenes 7.39 ->
// 7.11); with fewer windows the padding leaves XCDs idle (4,112 blocks 238 ->
// 242 us).
__host__ __device__ inline bool by_xcd(const Bc7Search &L) { return L.slices >= (1u << 17) / 64; }

__host__ __device__ inline Items search_items(const Bc7Search &L)
{
    constexpr uint32_t modes[kTypes] = {0x8A, 0x01, 0x04, 0x30, 0x40};
    Items I;
    I.total = 0;
    for (int t = 0; t < kTypes; t++) {
        const bool on = (L.types >> t & 1) && (L.a.mode_mask & modes[t]);
        const uint32_t windows = (L.slices + L.win[t] - 1) / L.win[t];
        const uint32_t whole = !by_xcd(L) ? 1u : per_window(t) < 4 ? 32u : 8u;   // whole eights of workgroups
        I.n[t] = on ? per_window(t) * ((windows + whole - 1) / whole * whole) : 0u;
        I.total += I.n[t];
    }
    return I;
}

constexpr int kMaxWin = 128;   // slices per window, at most

// One wave's LDS.  Blocks are held by their place in the window.
struct WaveLds {
    uint64_t word[kMaxWin];    // the candidate's words
    uint16_t end[kMaxWin];     // running count of their bits
    uint16_t q1[128];          // blocks to fit
    uint16_t q2[128];          // blocks whose largest subset is fitted ...
    uint32_t e[3][128];        // ... and its SSEs
};

// Orders a wave's LDS writes before its reads of other lanes' data.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The candidates left of one window, for one candidate p of the type.
template <int TYPE>
__device__ __forceinline__ void search_item(const Bc7Search &L, TexLds &S, WaveLds &W, uint32_t s0, uint32_t ns, int p)
{
    const EncodeArgs &a = L.a;
    const int lane = threadIdx.x & 63;
    constexpr bool kParts = TYPE == kTwo || TYPE == kThree0 || TYPE == kThree2;
    constexpr int NS = TYPE == kTwo ? 2 : 3;
    // the candidate's bound of chunk block c
    const uint64_t nc = L.B.nc;
    const uint16_t *lb = TYPE == kTwo ? reinterpret_cast<const uint16_t *>(L.B.b2) + (p >> 2) * nc * 4 + (p & 3)
                       : TYPE == kThree2 ? reinterpret_cast<const uint16_t *>(L.B.b3) + (p >> 1) * nc * 2 + (p & 1)
                       : TYPE == kThree0 ? reinterpret_cast<const uint16_t *>(L.B.b0) + (p >> 1) * nc * 2 + (p & 1)
                       : TYPE == kRot ? reinterpret_cast<const uint16_t *>(L.B.br) + p
                                      : reinterpret_cast<const uint16_t *>(L.B.seed) + 1;
    constexpr int kStep = TYPE == kTwo || TYPE == kRot ? 4 : 2;
    uint32_t *const keys = a.keys + L.first + (uint64_t)s0 * 64;   // of the window
    lb += (uint64_t)s0 * 64 * kStep;
    // the window's words and the running count of their bits
    uint32_t n = 0;
    for (uint32_t h = 0; h < ns; h += 64) {
        const uint32_t i = h + lane;
        const uint64_t x = i < ns ? L.words[(uint64_t)(s0 + i) * kWords + kWordAt[TYPE] + p] : 0ull;
        uint32_t e = (uint32_t)__popcll(x);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)e, d);
            if (lane >= d) e += o;
        }
        if (i < ns) {
            W.word[i] = x;
            W.end[i] = (uint16_t)(n + e);
        }
        n += (uint32_t)__builtin_amdgcn_readlane((int)e, 63);
    }
    if (n == 0) return;
    wave_lds_fence();
    // partitions: the largest subset first (one stage for the other types)
    uint32_t first = 0xFFFFu;
    int s_first = 0;
    if (kParts) {
        const uint32_t m0 = NS == 2 ? mask2(p, 0) : mask3(p, 0), m1 = NS == 2 ? mask2(p, 1) : mask3(p, 1);
        const uint32_t m2 = NS == 2 ? 0u : mask3(p, 2);
        const int c0 = __popc(m0), c1 = __popc(m1), c2 = __popc(m2);
        s_first = c0 >= c1 && c0 >= c2 ? 0 : c1 >= c2 ? 1 : 2;
        first = s_first == 0 ? m0 : s_first == 1 ? m1 : m2;
    }
    constexpr float kSlack = TYPE == kThree2 ? kSlack2 : kSlack3;
    const float members = (float)__popc(first), inv = __builtin_amdgcn_rcpf(members);
    auto stage = [&](uint32_t at, bool live) { stage_texels(S, live ? L.src[s0 + (at >> 6)] + 64 * (at & 63u) : nullptr, live); };
    // the other subsets of `count` blocks at the top of q2
    auto finish = [&](uint32_t q2, uint32_t count) {
        wave_lds_fence();
        const bool live = (uint32_t)lane < count;
        const uint32_t at = live ? W.q2[q2 + lane] : 0u;
        stage(at, live);
        if (live) {
            uint32_t e[3];
            e[0] = W.e[0][q2 + lane];
            if (TYPE == kTwo) { e[1] = W.e[1][q2 + lane]; e[2] = W.e[2][q2 + lane]; }
#pragma unroll 1
            for (int s = 0; s < NS; s++) {
                if (s == s_first) continue;
                const uint32_t m = NS == 2 ? mask2(p, s) : mask3(p, s);
                add_subset<TYPE>(S, m, subset_sums(S, m, 0), L.T.sv, e);
            }
            atomicMin(keys + at, partition_key<TYPE>(p, e));
        }
        wave_lds_fence();
    };
    uint32_t t = 0, q1 = 0, q2 = 0;
    while (true) {
        // gather 64 blocks whose best so far still leaves the candidate a chance
        while (q1 < 64 && t < n) {
            const uint32_t i = t + lane;
            uint32_t lo = 0, hi = n == 64 * ns ? 0 : ns - 1;   // (all of the window's blocks: i itself)
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (W.end[mid] > i) hi = mid;
                else lo = mid + 1;
            }
            bool keep = i < n;
            uint32_t at = i;
            if (keep && n != 64 * ns) {
                const uint64_t x = W.word[lo];
                at = lo * 64 + (uint32_t)nth_bit(x, (int)(i - ((uint32_t)W.end[lo] - (uint32_t)__popcll(x))));
            }
            if (keep) {
                const uint32_t key = keys[at];
                keep = key == ~0u || (uint32_t)lb[(uint64_t)at * kStep] <= bound16((float)(key >> 9));
            }
            const uint64_t m = __ballot(keep);
            if (keep) W.q1[q1 + lanes_below(m)] = (uint16_t)at;
            q1 += (uint32_t)__popcll(m);
            t += 64;
        }
        if (q1 == 0) break;
        wave_lds_fence();
        const uint32_t count = q1 < 64 ? q1 : 64;
        q1 -= count;
        const bool live = (uint32_t)lane < count;
        const uint32_t at = live ? W.q1[q1 + lane] : 0u;
        stage(at, live);
        uint32_t key = ~0u, e[3] = {kGone, kGone, kGone};
        if (live) {
            if (TYPE == kRot) key = search_rotation(S, p, a.mode_mask, L.T.sv);
            if (TYPE == kSix) key = search_mode6(S, L.T.sv);
            if (kParts) {
                const Sums sums = subset_sums(S, first, 0);
                const float f[9] = {(float)sums.nSx[0], (float)sums.nSx[1], (float)sums.nSx[2], (float)sums.XX[0], (float)sums.XX[1],
                                    (float)sums.XX[2], (float)sums.XX[3], (float)sums.XX[4], (float)sums.XX[5]};
                // what the bounds leave for the other subsets (the same arithmetic as the bounds')
                const float rest = fmaf(bound_value(lb[(uint64_t)at * kStep]), 1.0f - 2e-6f,
                                        -bound_term(residual_root(members, f), members, inv, kSlack));
                if (TYPE == kTwo) {
                    if (a.mode_mask & 0x02) e[0] = 0;
                    if (a.mode_mask & 0x08) e[1] = 0;
                    if (a.mode_mask & 0x80) e[2] = 0;
                } else e[0] = 0;
                add_subset<TYPE>(S, first, sums, L.T.sv, e);
                const uint32_t best = keys[at];
                const float room = best == ~0u ? 1e9f : (float)(best >> 9) * (1.0f + 2e-6f) - fmaxf(rest, 0.0f);
#pragma unroll
                for (int q = 0; q < (TYPE == kTwo ? 3 : 1); q++)
                    if ((float)e[q] > room) e[q] = kGone;
            } else atomicMin(keys + at, key);
        }
        if (kParts) {
            const bool keep = live && (e[0] & e[1] & e[2]) != kGone;
            const uint64_t m = __ballot(keep);
            if (keep) {
                const uint32_t to = q2 + lanes_below(m);
                W.q2[to] = (uint16_t)at;
                W.e[0][to] = e[0];
                if (TYPE == kTwo) { W.e[1][to] = e[1]; W.e[2][to] = e[2]; }
            }
            q2 += (uint32_t)__popcll(m);
            if (q2 >= 64) { q2 -= 64; finish(q2, 64); }
        }
    }
    if (kParts && q2) finish(0, q2);
    wave_lds_fence();
}

// One item per wave (the workgroup shares the code table only, so its waves
// run apart between the barriers of the queue).
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(3))) void k_bc7_search(Bc7Search L)
{
    __shared__ TexLds S;
    __shared__ WaveLds W[4];
    __shared__ uint32_t s_item;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Items I = search_items(L);
    stage_table(S, L.T.near64);
    ItemLoop it(L.w, (I.total + 3) / 4, &s_item);
    __syncthreads();
    if (it.item >= it.n_items) return;
    do {
        uint32_t q = it.item * 4 + wave;
        if (q >= I.total) continue;
        // the item's type (the first whose items reach past q), its window and candidate
        auto item = [&](auto type) {
            constexpr int T = decltype(type)::value;
            if (q >= I.n[T]) { q -= I.n[T]; return false; }
            uint32_t window = q / per_window(T), p = q % per_window(T);
            if constexpr (per_window(T) >= 4) {
                if (by_xcd(L)) {   // (every type starts at a multiple of eight workgroups)
                    constexpr uint32_t groups = per_window(T) / 4;   // workgroups per window
                    const uint32_t g = q >> 2, i = g >> 3;
                    window = i / groups * 8 + (g & 7u);
                    p = i % groups * 4 + (q & 3u);
                }
            }
            const uint32_t s0 = window * L.win[T];
            if (s0 < L.slices) search_item<T>(L, S, W[wave], s0, min(L.win[T], L.slices - s0), (int)p);
            return true;
        };
        if (!item(Type<kSix>()) && !item(Type<kTwo>()) && !item(Type<kThree0>()) && !item(Type<kRot>()))
            item(Type<kThree2>());
    } while (it.next(L.w, &s_item));
}

// ---- pass 2: the winners' bits
__device__ __forceinline__ int mode_of_candidate(int ci)
{
    return ci < 16 ? 0 : ci < 80 ? 1 : ci < 144 ? 2 : ci < 208 ? 3 : ci < 216 ? 4 : ci < 220 ? 5 : ci < 221 ? 6 : 7;
}

// Re-fit each block's winning candidate and write its bits.  A workgroup
// takes `per` consecutive indices (512, or 256 when they are few), lists
// them by the mode of their winner in LDS, and its waves take 64 of one mode
// at a time, so that a wave runs one mode's code; the costlier modes first.
// Padding indices (key all-ones) join no list.  Each 256 indices lie in one
// run: their SSEs (key >> 9) are summed and reach the run's sum as one atomic.
// One launch, bound by the spread of the batches' lengths over the waves:
// separate count, scan, fill and eight emit launches took 0.43 ms at 1,048,576
// blocks and 0.18 ms at 4,112, this 0.39 and 0.055 ms.
constexpr int kEmitMost = 512;
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(3))) void k_bc7_emit(Bc7Launch L, uint32_t per)
{
    __shared__ TexLds S;
    __shared__ uint16_t s_list[kEmitMost];
    __shared__ uint32_t s_count[8], s_at[8], s_next;
    __shared__ BlockRun s_run[kEmitMost / kWG];
    const EncodeArgs &a = L.a;
    const int lane = threadIdx.x & 63;
    const uint64_t g0 = (uint64_t)blockIdx.x * per;
    const uint32_t rounds = (uint32_t)min((uint64_t)per, a.total - g0) / kWG;
    if (threadIdx.x < 8) s_count[threadIdx.x] = 0;
    if (threadIdx.x == 0) s_next = 0;
    if (threadIdx.x < rounds) s_run[threadIdx.x] = a.run[find_run(a.run, a.nrun, g0 + threadIdx.x * kWG)];
    stage_table(S, L.T.nearest);
    __syncthreads();
    uint32_t key[kEmitMost / kWG], rank[kEmitMost / kWG];
#pragma unroll
    for (uint32_t r = 0; r < kEmitMost / kWG; r++) {
        key[r] = r < rounds ? a.keys[g0 + r * kWG + threadIdx.x] : ~0u;
        if (key[r] != ~0u) rank[r] = atomicAdd(&s_count[mode_of_candidate((int)(key[r] & 511u))], 1u);
        if (r < rounds && s_run[r].sse) {
            unsigned long long x = key[r] != ~0u ? (unsigned long long)(key[r] >> 9) : 0ull;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
            if (lane == 0 && x) atomicAdd(s_run[r].sse, x);
        }
    }
    __syncthreads();
    constexpr int kOrder[8] = {4, 0, 5, 6, 1, 2, 3, 7};
    if (threadIdx.x == 0) {
        uint32_t at = 0;
        for (int q = 0; q < 8; q++) { s_at[kOrder[q]] = at; at += s_count[kOrder[q]]; }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kEmitMost / kWG; r++)
        if (key[r] != ~0u) s_list[s_at[mode_of_candidate((int)(key[r] & 511u))] + rank[r]] = (uint16_t)(r * kWG + threadIdx.x);
    __syncthreads();
    // batches of up to 64 of one mode, taken by the waves as they come free
    auto take = [&] {
        uint32_t b = 0;
        if (lane == 0) b = atomicAdd(&s_next, 1u);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
    };
    uint32_t batch = take(), base = 0;   // base: batches of the modes before
    auto run_mode = [&](auto mode) {
        constexpr int M = decltype(mode)::value;
        const uint32_t n = s_count[M], first = s_at[M], batches = (n + 63) / 64;
        for (; batch < base + batches; batch = take()) {
            const uint32_t e0 = (batch - base) * 64;
            const uint32_t e = e0 + lane;
            const bool live = e < n;
            const uint32_t at = live ? s_list[first + e] : 0u;
            const BlockRun &run = s_run[at / kWG];
            const uint64_t b = g0 + at - run.gbase;
            stage_texels(S, run.src + b * 64, live);   // lanes past the list stage zeros
            if (live) {
                uint64_t lo, hi;
                emit<M>(S, (int)(a.keys[g0 + at] & 511u), L.T.sv, lo, hi);
                *reinterpret_cast<ulonglong2 *>(run.dst + b * 16) = make_ulonglong2(lo, hi);
            }
        }
        base += batches;
    };
    run_mode(Type<4>());
    run_mode(Type<0>());
    run_mode(Type<5>());
    run_mode(Type<6>());
    run_mode(Type<1>());
    run_mode(Type<2>());
    run_mode(Type<3>());
    run_mode(Type<7>());
}

// ---- host-side table construction
struct HostTables {
    std::vector<uint16_t> nearest;  // [10][2][256]
    std::vector<uint16_t> near64;   // [10][2][256]
    std::vector<uint32_t> sv;       // [10][4][kSlots][256]
};

void build_nearest(HostTables &H)
{
    H.nearest.assign(10 * 2 * 256, 0);
    for (int cb = 4; cb <= 8; cb++)
        for (int pb = 0; pb < 2; pb++)
            for (int p = 0; p < 2; p++) {
                if (!pb && p) continue;
                const int nc = 1 << cb;
                uint16_t *row = &H.nearest[(cls_of(cb, pb) * 2 + p) * 256];
                for (int t = 0; t < 256; t++) {
                    int bc = 0, bd = 1 << 30;
                    for (int c = 0; c < nc; c++) {
                        int d = ep_value(c, p, cb, pb) - t;
                        d = d < 0 ? -d : d;
                        if (d < bd) { bd = d; bc = c; }
                    }
                    row[t] = (uint16_t)(bc | (ep_value(bc, p, cb, pb) << 8));
                }
            }
    H.near64.resize(H.nearest.size());
    for (size_t q = 0; q < H.nearest.size(); q++) H.near64[q] = (uint16_t)((H.nearest[q] >> 8) << 6);
}

// Best pair per target value v for one (class, p-bits, weight): first the
// best pair (by |c0-c1|, c0, c1) reaching each interpolated value u, then for
// each v the nearest reachable u (both sides of v compared by the same key).
void build_sv_entry(uint32_t *row, int cb, int pb, int p0, int p1, int wgt)
{
    const int nc = 1 << cb;
    int bestpair[256];
    for (int u = 0; u < 256; u++) bestpair[u] = -1;
    auto better = [&](int a0, int a1, int b0, int b1) {   // is (a0,a1) ahead of (b0,b1)?
        int da = a0 > a1 ? a0 - a1 : a1 - a0, db = b0 > b1 ? b0 - b1 : b1 - b0;
        if (da != db) return da < db;
        if (a0 != b0) return a0 < b0;
        return a1 < b1;
    };
    for (int a = 0; a < nc; a++)
        for (int b = 0; b < nc; b++) {
            int u = interp64(ep_value(a, p0, cb, pb), ep_value(b, p1, cb, pb), wgt);
            int cur = bestpair[u];
            if (cur < 0 || better(a, b, cur >> 8, cur & 255)) bestpair[u] = (a << 8) | b;
        }
    for (int v = 0; v < 256; v++) {
        for (int d = 0; d < 256; d++) {
            int pick = -1;
            for (int side = 0; side < 2; side++) {
                int u = side ? v + d : v - d;
                if (u < 0 || u > 255 || bestpair[u] < 0) continue;
                int pr = bestpair[u];
                if (pick < 0 || better(pr >> 8, pr & 255, pick >> 8, pick & 255)) pick = pr;
            }
            if (pick >= 0) {
                row[v] = (uint32_t)(pick >> 8) | ((uint32_t)(pick & 255) << 8) | ((uint32_t)d << 16);
                break;
            }
        }
    }
}

void build_sv(HostTables &H)
{
    H.sv.assign((size_t)10 * 4 * kSlots * 256, 0);
    struct Use { int cb, pb, nb; };
    const Use uses[] = {{4, 2, 3}, {6, 1, 3}, {5, 0, 2}, {7, 2, 2}, {5, 0, 3}, {6, 0, 3}, {6, 0, 2},
                        {7, 0, 2}, {8, 0, 2}, {7, 2, 4}, {5, 2, 2}};
    for (const Use &u : uses) {
        const int npc = u.pb == 2 ? 4 : u.pb == 1 ? 2 : 1;
        for (int pc = 0; pc < npc; pc++) {
            int p0 = u.pb == 2 ? (pc & 1) : u.pb == 1 ? pc : 0;
            int p1 = u.pb == 2 ? (pc >> 1) : u.pb == 1 ? pc : 0;
            for (int k = 0; k < (1 << u.nb); k++) {
                uint32_t *row = &H.sv[(((size_t)cls_of(u.cb, u.pb) * 4 + p0 + 2 * p1) * kSlots + slot_of(u.nb, k)) * 256];
                build_sv_entry(row, u.cb, u.pb, p0, p1, bc7_weight(u.nb, k));
            }
        }
    }
}

}  // namespace

// Device copies of the tables, one set per device, made once per device
// (under a lock: contexts may be created from several threads).
static void *g_tab[kMaxDevices];
static std::mutex g_tab_lock;

hipError_t upload_bc7_tables(int device, hipStream_t st)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(g_tab_lock);
    if (g_tab[device]) return hipSuccess;
    static HostTables H;
    if (H.nearest.empty()) { build_nearest(H); build_sv(H); }
    size_t nb = H.nearest.size() * 2, sb = H.sv.size() * 4;
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, 2 * nb + sb);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(p, H.nearest.data(), nb, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync((char *)p + nb, H.near64.data(), nb, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync((char *)p + 2 * nb, H.sv.data(), sb, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) { (void)hipFree(p); return e; }
    g_tab[device] = p;
    return hipSuccess;
}

hipError_t launch_bc7_encode(const EncodeArgs &a, const WorkSplit *w3, uint32_t split, hipStream_t st,
                             hipEvent_t alone)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (!g_tab[dev]) return hipErrorNotInitialized;
    if (a.total == 0) return hipSuccess;
    if (split > 3 || a.chunk == 0 || a.chunk % kRunAlign) return hipErrorInvalidValue;
    Bc7Launch L;
    L.a = a;
    L.T.nearest = static_cast<const uint16_t *>(g_tab[dev]);
    L.T.near64 = L.T.nearest + kQEntries;
    L.T.sv = reinterpret_cast<const uint32_t *>(L.T.near64 + kQEntries);
    // scratch: keys[total], then for one chunk: slice texels | candidate words | bounds
    Bc7Search Q;
    Q.a = a;
    Q.T = L.T;
    uint8_t *s = reinterpret_cast<uint8_t *>(a.keys) + 4 * a.total;
    auto take = [&](size_t bytes) { uint8_t *r = s; s += (bytes + 15) & ~(size_t)15; return r; };
    const uint64_t nc = a.total < a.chunk ? a.total : a.chunk;
    Q.src = reinterpret_cast<const uint8_t **>(take(8 * (nc / 64)));
    Q.words = reinterpret_cast<uint64_t *>(take(8 * kWords * (nc / 64)));
    uint32_t *const dense = reinterpret_cast<uint32_t *>(take(4 * (nc / 64) + 16));
    Q.B.nc = nc;
    Q.B.b2 = reinterpret_cast<uint2 *>(take(16 * 8 * nc));
    Q.B.b3 = reinterpret_cast<uint32_t *>(take(32 * 4 * nc));
    Q.B.b0 = reinterpret_cast<uint32_t *>(take(8 * 4 * nc));
    Q.B.br = reinterpret_cast<uint2 *>(take(8 * nc));
    Q.B.seed = reinterpret_cast<uint32_t *>(take(4 * nc));
    auto launch = [&](int q, uint32_t types, const char *name) -> hipError_t {
        Q.w = w3[q];
        Q.types = types;
        // Windows: long enough that a candidate's blocks fill waves (about 1
        // in 20 blocks is left of a 2-subset partition, 1 in 3 of a 3-subset
        // one or a rotation), short enough that a small scene spreads over
        // the chip.
        auto window = [&](uint32_t split, uint32_t most) {
            uint32_t n = Q.slices / split;
            n = n < 4 ? 4 : n > most ? most : n;
            n *= Q.w.item_rounds;
            return n > (uint32_t)kMaxWin ? (uint32_t)kMaxWin : n;
        };
        Q.win[kTwo] = window(32, kMaxWin);
        Q.win[kThree0] = Q.win[kThree2] = window(64, 64);
        Q.win[kRot] = Q.win[kSix] = window(512, 16);
        const Items I = search_items(Q);
        if (I.total == 0) return hipSuccess;
        if (Q.w.queue) {
            hipError_t f = launch_fill_u64(reinterpret_cast<unsigned long long *>(Q.w.queue), 1, 0, st);
            if (f != hipSuccess) return f;
        }
        GSBC_LAUNCH(name, k_bc7_search, dim3(Q.w.queue ? Q.w.grid : (I.total + 3) / 4), dim3(kWG), 0, st, Q);
        return hipGetLastError();
    };
    constexpr uint32_t kType2 = 1u << kTwo, kType3 = 1u << kThree0 | 1u << kThree2, kType1 = 1u << kRot | 1u << kSix;
    // Up to which kernel the (first chunk's) launches want the chip to
    // themselves: the bounds fill it from few blocks on, the seeds from about
    // 196,608 (both formats, other work after the bounds / after the seeds:
    // 131,072 primitives 923 / 972 us, 200,003 1,466 / 1,436, 262,144 1,995 /
    // 1,760, 524,288 3,262 / 3,180, 1,048,576 6,139 / 6,140).
    const bool seeds_fill = a.total >= (3u << 16);
    for (uint64_t first = 0; first < a.total; first += nc) {
        const uint64_t left = a.total - first < nc ? a.total - first : nc;
        Q.first = first;
        Q.slices = (uint32_t)(left / 64);
        const uint32_t per = left >= (1u << 17) ? kWG : 64;
        const bool pairs = left < (1u << 17);
        // (one shape of partition only: with both, what the other one reaches rules more out)
        Q.dense = !pairs && !(a.mode_mask & 0x8A) != !(a.mode_mask & 0x05) ? dense : nullptr;
        const int seeds = seed_kind(a.mode_mask);
        if (seeds != kSeedEvery) GSBC_LAUNCH("bc7_bounds", k_bc7_bounds, dim3((uint32_t)(left / per)), dim3(kWG), 0, st, Q, per);
        if (alone && !seeds_fill && first == 0 && (e = hipEventRecord(alone, st)) != hipSuccess) return e;
        auto seed = seeds == kSeedUsual ? (Q.dense ? k_bc7_seed<kSeedUsual, true> : k_bc7_seed<kSeedUsual, false>)
                  : seeds == kSeedOther ? (Q.dense ? k_bc7_seed<kSeedOther, true> : k_bc7_seed<kSeedOther, false>)
                                        : k_bc7_seed<kSeedEvery, false>;
        GSBC_LAUNCH("bc7_seed", seed, dim3((uint32_t)(left / (pairs ? kWG / 2 : kWG))), dim3(kWG), 0, st, Q, pairs);
        if (alone && seeds_fill && first == 0 && (e = hipEventRecord(alone, st)) != hipSuccess) return e;
        if (seeds == kSeedEvery) continue;
        if (Q.dense) GSBC_LAUNCH("bc7_every", k_bc7_every, dim3((uint32_t)(left / kWG)), dim3(kWG), 0, st, Q);
        if (split == 0) {
            if ((e = launch(0, kType3, "bc7_search_3subset")) != hipSuccess) return e;
            if ((e = launch(1, kType1, "bc7_search_1subset")) != hipSuccess) return e;
            if ((e = launch(2, kType2, "bc7_search_2subset")) != hipSuccess) return e;
        } else if (split == 1) {
            if ((e = launch(0, kType3 | kType1, "bc7_search_3subset_1subset")) != hipSuccess) return e;
            if ((e = launch(1, kType2, "bc7_search_2subset")) != hipSuccess) return e;
        } else {
            if ((e = launch(0, kType3 | kType1 | kType2, "bc7_search_items")) != hipSuccess) return e;
        }
    }
    // 512 indices fill a mode's last batch better, 256 spread further (BC7 of
    // 65,536 blocks 0.43 against 0.47 ms, of 200,003 1.21 against 1.20 ms)
    const uint32_t per = a.total >= (1u << 17) ? kEmitMost : kWG;
    // (timed under the name its bucketing has always had)
    GSBC_LAUNCH("bc7_bucket", k_bc7_emit, dim3((uint32_t)((a.total + per - 1) / per)), dim3(kWG), 0, st, L, per);
    return hipGetLastError();
}

}  // namespace gsbc
