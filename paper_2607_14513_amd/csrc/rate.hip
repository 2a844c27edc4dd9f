// rate.hip -- per-band format choice at an exact bit rate (Sec. IV-B: each
// bitstream keeps a fixed block size, so random access survives, while the
// number of bits per primitive is set by which bands use which format).
//
// Band 0 is BC7.  AUTO: of bands 1..S-1, the k with the largest
// coefficient-domain gain (SSE_BC1 - SSE_BC7) * delta^2 are BC7 and the
// rest BC1 (the lower band wins ties); every upgrade costs the same bits,
// so the k largest gains minimise the total error at that budget.
// AUTO_ZERO: each band 1..S-1 is BC7, BC1 or not stored at all (0 bits; its
// coefficients decode to zero), at an exact number of four-bit units, with
// the least total distortion, found by dynamic programming over bands and
// units (the costs 2, 1, 0 are not uniform, so no greedy order is exact).
// Selection and the stream copy run on the device (no host round trip).
#include "gsbc_internal.h"

namespace gsbc {
namespace {

// The selection from each band's format (lane q < S holds band q's), and the
// SSE sums (16 of BC1, 16 of BC7), to the device record and, for the host, to
// pinned memory (a copy engine's two small copies cost more than the wait).
__device__ void write_selection(uint32_t fmt, uint32_t S, uint64_t nblk, const unsigned long long *sse, RateSel *sel,
                                RateSel *host_sel, unsigned long long *host_sse)
{
    const uint32_t t = threadIdx.x;   // one wave
    if (t >= S) fmt = 0u;
    // streams are padded to 16 bytes (bands past S hold nothing)
    uint64_t bytes = t >= S || fmt == GSBC_FMT_NONE ? 0 : nblk * (fmt == GSBC_FMT_BC1 ? 8 : 16);
    bytes = (bytes + 15) & ~(uint64_t)15;
    uint64_t end = bytes;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        const uint64_t o = __shfl_up(end, d);
        if (t >= (uint32_t)d) end += o;
    }
    if (t < 16) {
        sel->format[t] = host_sel->format[t] = fmt;
        sel->offset[t] = host_sel->offset[t] = t < S ? end - bytes : 0u;
        if (t == 15) sel->payload_bytes = host_sel->payload_bytes = end;
    }
    if (t < 32) host_sse[t] = sse[t];
}

// One wave, lane q = band q.  A band is BC7 if fewer than k bands come before
// it (larger gain, the lower band on ties).  Gains are ranked by their bits
// (ordered as the values are), so exactly k bands are BC7 whatever they hold.
// A gain that is no number (a band whose range is infinite or NaN) has no rank:
// then the bands are picked one by one, the first one left against the others,
// as the rule is written (a NaN is passed by nothing and passes nothing).
__global__ __launch_bounds__(64) void k_rate_select(const unsigned long long *sse, BandArgs b, uint32_t S, uint32_t k,
                                                    uint64_t nblk, RateSel *sel, RateSel *host_sel,
                                                    unsigned long long *host_sse)
{
    const uint32_t t = threadIdx.x, q = t & 15u;
    const double d = (double)b.delta[q];
    const double gain = (double)((long long)sse[q] - (long long)sse[16 + q]) * (d * d) + 0.0;   // -0 as 0
    const uint64_t u = (uint64_t)__double_as_longlong(gain);
    const uint64_t key = u >> 63 ? ~u : u | 1ull << 63;
    uint32_t before = 0;
    for (uint32_t o = 1; o < S; o++) {
        const uint64_t other = __shfl(key, (int)o);
        before += o != q && (other > key || (other == key && o < q)) ? 1u : 0u;
    }
    bool wide = q == 0 || before < k;
    if (__any(q >= 1 && q < S && gain != gain)) {
        wide = q == 0;
        for (uint32_t pick = 0; pick < k; pick++) {
            const uint32_t left = ~(uint32_t)__ballot(wide) & ((1u << S) - 1u);   // (lanes 0..15 hold the bands)
            uint32_t best = (uint32_t)__ffs(left) - 1;
            for (uint32_t rest = left & (left - 1); rest; rest &= rest - 1) {
                const uint32_t o = (uint32_t)__ffs(rest) - 1;
                if (__shfl(gain, (int)o) > __shfl(gain, (int)best)) best = o;
            }
            wide |= q == best;
        }
    }
    write_selection(wide ? GSBC_FMT_BC7 : GSBC_FMT_BC1, S, nblk, sse, sel, host_sel, host_sse);
}

// Code histogram of every band's R, G and B texel channels: one workgroup
// per (band, slice of blocks), counts in LDS, then added to hist[band][256].
__global__ __launch_bounds__(256) void k_band_hist(const uint8_t *tex, uint64_t nblk,
                                                   unsigned long long *hist)
{
    __shared__ uint32_t h[256];
    const uint32_t band = blockIdx.y;
    h[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t *t = reinterpret_cast<const uint32_t *>(tex + (uint64_t)band * nblk * 64);
    const uint64_t words = nblk * 16;   // one RGBA texel per word
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (uint64_t)gridDim.x * 256) {
        const uint32_t w = t[i];
        atomicAdd(&h[w & 255u], 1u);
        atomicAdd(&h[(w >> 8) & 255u], 1u);
        atomicAdd(&h[(w >> 16) & 255u], 1u);
    }
    __syncthreads();
    if (h[threadIdx.x]) atomicAdd(&hist[band * 256 + threadIdx.x], (unsigned long long)h[threadIdx.x]);
}

// AUTO_ZERO choice for U units over bands 1..S-1 (BC7 2, BC1 1, none 0).
// Band distortions: SSE * delta^2 for the coded formats; for none, the sum
// over codes q (ascending) of count_q * (vmin + q delta)^2.  least[b][u] is
// the least total of bands b..S-1 with u units, each band's distortion
// added to the total of the later bands (rounded addition is monotone, so
// the least total splits over the choice at band b); the choice then walks
// the bands upward taking, at each, the first of BC7, BC1, none that keeps
// the least total.
// One workgroup: every band's 256 terms at once into LDS, one lane per band
// adds them in order, one lane per unit count takes a band's three choices at
// a time, and the walk reads what they left.  (One thread over scratch memory
// took 211 us, a fifth of a 65,536-primitive encode; this 15.)
__global__ __launch_bounds__(1024) void k_rate_select_zero(const unsigned long long *sse, const unsigned long long *hist,
                                                           BandArgs b, uint32_t S, uint32_t U, uint64_t nblk, RateSel *sel,
                                                           RateSel *host_sel, unsigned long long *host_sse)
{
    __shared__ double term[16][256 + 1];
    __shared__ double dist[16][3], least[17][31];
    __shared__ uint8_t ok[17][31], code[16];
    const uint32_t t = threadIdx.x;
    for (uint32_t e = t; e < S * 256; e += 1024) {
        const uint32_t band = e >> 8, q = e & 255u;
        const double d = (double)b.delta[band], v = (double)b.vmin[band] + (double)(int)q * d;
        term[band][q] = (double)hist[e] * (v * v);
    }
    __syncthreads();
    if (t >= 64) return;   // the rest is one wave's
    if (t >= 1 && t < S) {
        const double d = (double)b.delta[t];
        dist[t][0] = (double)sse[16 + t] * (d * d);
        dist[t][1] = (double)sse[t] * (d * d);
        double z = 0.0;
#pragma unroll 16
        for (int q = 0; q < 256; q++) z += term[t][q];
        dist[t][2] = z;
    }
    constexpr int kUnits[3] = {2, 1, 0};
    constexpr uint32_t kCode[3] = {GSBC_FMT_BC7, GSBC_FMT_BC1, GSBC_FMT_NONE};
    const int u = (int)t;
    if (u <= 30) {
        ok[S][u] = u == 0;
        least[S][u] = 0.0;
    }
    for (int band = (int)S - 1; band >= 1; band--) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (u <= 30) {
            bool have = false;
            double best = 0.0;
#pragma unroll
            for (int o = 0; o < 3; o++) {
                const int r = u - kUnits[o];
                if (r < 0 || !ok[band + 1][r]) continue;
                const double v = dist[band][o] + least[band + 1][r];
                if (!have || v < best) {
                    best = v;
                    have = true;
                }
            }
            ok[band][u] = have;
            least[band][u] = best;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (t == 0) {
        int left = (int)U;
        code[0] = GSBC_FMT_BC7;
        for (uint32_t band = 1; band < S; band++) {
            code[band] = GSBC_FMT_BC1;
            for (int o = 0; o < 3; o++) {
                const int r = left - kUnits[o];
                if (r < 0 || !ok[band + 1][r] || dist[band][o] + least[band + 1][r] != least[band][left]) continue;
                code[band] = (uint8_t)kCode[o];
                left = r;
                break;
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    write_selection(t < S ? code[t] : 0u, S, nblk, sse, sel, host_sel, host_sse);
}

// blockIdx.y = band; 8-byte words.  A stream with no bits copies nothing.
__global__ __launch_bounds__(256) void k_copy_streams(const uint8_t *src1, const uint8_t *src7, const RateSel *sel,
                                                      uint64_t nblk, uint8_t *out)
{
    const int q = blockIdx.y;
    if (sel->format[q] == GSBC_FMT_NONE) return;
    const bool bc1 = sel->format[q] == GSBC_FMT_BC1;
    const uint64_t words = nblk * (bc1 ? 1 : 2);
    const uint64_t padded = (words + 1) & ~(uint64_t)1;   // streams are 16-byte aligned
    const uint64_t *src = reinterpret_cast<const uint64_t *>(bc1 ? src1 + q * ((8 * nblk + 15) & ~(uint64_t)15) : src7 + q * 16 * nblk);
    uint64_t *dst = reinterpret_cast<uint64_t *>(out + sel->offset[q]);
    for (uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; w < padded; w += (uint64_t)gridDim.x * blockDim.x)
        dst[w] = w < words ? src[w] : 0ull;
}

__global__ void k_fill_u64(unsigned long long *p, uint64_t n, unsigned long long v)
{
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

}  // namespace

hipError_t launch_rate_select(const unsigned long long *sse, const BandArgs &b, uint32_t S, uint32_t k, uint64_t nblk,
                              RateSel *sel, RateSel *host_sel, unsigned long long *host_sse, hipStream_t st)
{
    GSBC_LAUNCH("rate_select", k_rate_select, dim3(1), dim3(64), 0, st, sse, b, S, k, nblk, sel, host_sel, host_sse);
    return hipGetLastError();
}

// The encode's run tables, handed over as kernel arguments, into device
// memory, and its SSE sums to zero: one launch for two copies and a clear.
__global__ __launch_bounds__(64) void k_encode_setup(RunTables t, BlockRun *runs, unsigned long long *sse)
{
    const uint32_t *src = reinterpret_cast<const uint32_t *>(&t);
    for (uint32_t e = threadIdx.x; e < sizeof(RunTables) / 4; e += 64) reinterpret_cast<uint32_t *>(runs)[e] = src[e];
    if (threadIdx.x < 32) sse[threadIdx.x] = 0;
}

hipError_t launch_encode_setup(const RunTables &t, BlockRun *runs, unsigned long long *sse, hipStream_t st)
{
    GSBC_LAUNCH("fill", k_encode_setup, dim3(1), dim3(64), 0, st, t, runs, sse);
    return hipGetLastError();
}

hipError_t launch_band_hist(const uint8_t *tex, uint32_t S, uint64_t nblk, unsigned long long *hist, hipStream_t st)
{
    uint64_t gx = (nblk * 16 + 255) / 256;
    gx = gx > 256 ? 256 : (gx == 0 ? 1 : gx);
    GSBC_LAUNCH("band_hist", k_band_hist, dim3((uint32_t)gx, S), dim3(256), 0, st, tex, nblk, hist);
    return hipGetLastError();
}

hipError_t launch_rate_select_zero(const unsigned long long *sse, const unsigned long long *hist, const BandArgs &b,
                                   uint32_t S, uint32_t U, uint64_t nblk, RateSel *sel, RateSel *host_sel,
                                   unsigned long long *host_sse, hipStream_t st)
{
    GSBC_LAUNCH("rate_select", k_rate_select_zero, dim3(1), dim3(1024), 0, st, sse, hist, b, S, U, nblk, sel, host_sel,
                host_sse);
    return hipGetLastError();
}

hipError_t launch_copy_streams(const uint8_t *src1, const uint8_t *src7, const RateSel *sel, uint32_t S, uint64_t nblk,
                               uint8_t *out, hipStream_t st)
{
    uint64_t words = nblk * 2;
    uint32_t gx = (uint32_t)((words + 255) / 256);
    gx = gx > 1024 ? 1024 : (gx == 0 ? 1 : gx);
    GSBC_LAUNCH("copy_streams", k_copy_streams, dim3(gx, S), dim3(256), 0, st, src1, src7, sel, nblk, out);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, uint64_t n, unsigned long long v, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    GSBC_LAUNCH("fill", k_fill_u64, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

}  // namespace gsbc
