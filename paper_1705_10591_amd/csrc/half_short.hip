// Short launches of the general case for short data types (fp16, bf16, int8): layers whose tiles do not fill
// the chip.
//
// general_half_kernel gives such a layer one round of its 64 x 256 tiles on a part of the CUs, each a long chain
// of chunks, two barriers of latency apart.  Here a workgroup has a small tile, 16 A filters x 16 B pixels, and
// its S waves share the reduction: each takes a stretch of it in the order in which the weights lie, and the
// waves' sums meet in LDS.  With channels innermost sixteen bytes of a pixel or of a filter are an operand of
// v_mfma_*_16x16x32 (16x16x64 for int8) as they lie in memory, so operands come straight from there (the L2, at
// these sizes) into the matrix-core registers, kAhead steps ahead: no staging, no barrier before the end.
//  * A unit is 32 bytes of channels at one tap.  Units are numbered as a filter's lie in memory: taps, then channel
//    groups (channels last), or channel groups, then taps (channel-blocked).  A step takes two units; lane (g, l)
//    brings piece g % 2 of unit g / 2 of filter l and of pixel l.
//  * A unit's offset from its pixel is the same for all pixels: every wave makes a table of its stretch in LDS.
//  * Pixels are numbered along (image, y, x); the last ones of a tile may be none.
// What bounds it is the latency of a wave's steps, and the vector memory path once the waves fill the SIMDs: a
// step of a 64 x 64 tile takes 8 KB through it for 256 cycles of products.
//
// Measured (general_half_kernel -> this one, kernels replayed from a graph): three images of 320 x 8 x 8 with 106
// 3x3 filters, bf16, blocked 22.0 -> 6.0 us; two of 384 x 17 x 18 with 229 5x5, int8 49.7 -> 19.6;
// one of 352 x 25 x 25 with 25 3x3, bf16 28.2 -> 6.1; eleven of 112 x 11 x 11 with 227 7x7, bf16 52.9 -> 14.1; one of 256 x
// 14 x 14 with 256 3x3, fp16 21.3 -> 6.6.
// Sums are a half or a quarter as long: errors against 64 bits halve (3.2e-7 -> 1.6e-7 in the first of these).
#include <algorithm>
#include "half_kernel.h"

namespace dconv {

namespace {

struct HalfShortParams {
    const char* in;
    const char* filt;
    float* out;              // (int32 bit patterns for 8-bit inputs)
    int N, H, W, K, F, Ho, Wo;
    int image, row;          // bytes of an image and of a filter
    int ps, gs;              // bytes from pixel to pixel, from channel group to channel group
    int units, steps;
    int blocked;
    int px, ptiles, ftiles, total;
    int by_filter;           // workgroups next to each other share filters, not pixels
    FastDiv d_wo, d_ho, d_inner, d_f, d_tiles;       // d_inner: taps (blocked) or channel groups
};

template <int DT>
__device__ __forceinline__ v4f mfma_step(v4f a, v4f b, v4f acc) {
    if (DT == kI8)
        return __builtin_bit_cast(v4f, __builtin_amdgcn_mfma_i32_16x16x64_i8(
            __builtin_bit_cast(v4i, a), __builtin_bit_cast(v4i, b), __builtin_bit_cast(v4i, acc), 0, 0, 0));
    if (DT == kBF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), acc, 0, 0, 0);
}

template <int DT>
__device__ __forceinline__ float add(float a, float b) {
    if (DT == kI8) return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a) + __builtin_bit_cast(uint32_t, b));
    return a + b;
}

template <int DT, int A, int B, int S>
__global__ void __launch_bounds__(64 * S)
short_half_kernel(HalfShortParams p)
{
    constexpr int kAhead = 4, THREADS = 64 * S, TM = 16 * A, TN = 16 * B;
    constexpr uint32_t kNowhere = 0xC0000000u;
    constexpr int kRsrcFlags = 0x00020000;

    extern __shared__ __attribute__((aligned(16))) uint32_t short_lds[];
    // offsets of units: all waves' stretches one after the other; then [wave][filter][pixel] sums
    uint32_t* const table = short_lds;
    float* const sums = (float*)(short_lds + 2 * p.steps);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, l16 = lane & 15;
    const int wg = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    if (wg >= p.total) return;                                  // uniform: before any barrier
    const int major = fdiv(wg, p.d_tiles), minor = wg - major * p.d_tiles.d;
    const int ft = p.by_filter ? major : minor, pt = p.by_filter ? minor : major;
    const int s0 = range_start(wave, p.steps, S), s1 = range_start(wave + 1, p.steps, S);

    // ---- this wave's stretch of the table (a unit beyond the last is nowhere)
    for (int u = 2 * s0 + lane; u < 2 * s1; u += 64) {
        const int outer = fdiv(u, p.d_inner), inner = u - outer * p.d_inner.d;
        const int tap = p.blocked ? inner : outer, group = p.blocked ? outer : inner, i = fdiv(tap, p.d_f);
        table[u] = u < p.units ? (uint32_t)(group * p.gs + (i * p.W + tap - i * p.F) * p.ps) : kNowhere;
    }

    // ---- what a lane loads
    const auto irs = __builtin_amdgcn_make_buffer_rsrc((void*)p.in, 0, p.N * p.image, kRsrcFlags);
    const auto wrs = __builtin_amdgcn_make_buffer_rsrc((void*)p.filt, 0, p.K * p.row, kRsrcFlags);
    uint32_t pix[B], row[A];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int pp = pt * TN + b * 16 + l16, Q = fdiv(pp, p.d_wo), x = pp - Q * p.Wo, n = fdiv(Q, p.d_ho), y = Q - n * p.Ho;
        pix[b] = pp < p.px ? (uint32_t)(n * p.image + (y * p.W + x) * p.ps + (g & 1) * 16) : kNowhere;
    }
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int k = ft * TM + a * 16 + l16;
        row[a] = k < p.K ? (uint32_t)(k * p.row + g * 16) : kNowhere;
    }
    v4f w[kAhead][A], x[kAhead][B];
    auto fetch = [&](int s, v4f (&w)[A], v4f (&x)[B]) __attribute__((always_inline)) {
        const uint32_t off = table[2 * min(s, s1 - 1) + (g >> 1)];
        // beyond the stretch nothing is read, and beyond the last unit neither operand is (what lies there
        // is another filter's); no sum of two offsets is below an extent unless both are there
        const bool there = s < s1 && 2 * s + (g >> 1) < p.units;
#pragma unroll
        for (int a = 0; a < A; ++a)
            w[a] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(wrs, there ? row[a] + s * 64 : kNowhere, 0, 0));
#pragma unroll
        for (int b = 0; b < B; ++b)
            x[b] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(irs, there ? pix[b] + off : kNowhere, 0, 0));
    };
    v4f acc[A][B];
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b) acc[a][b] = v4f{};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the wave's table is in LDS
    if (s0 < s1) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d) fetch(s0 + d, w[d], x[d]);
        for (int s = s0; s < s1; s += kAhead)
#pragma unroll
            for (int d = 0; d < kAhead; ++d) {                  // (steps beyond the stretch add products of zeros)
#pragma unroll
                for (int a = 0; a < A; ++a)
#pragma unroll
                    for (int b = 0; b < B; ++b) acc[a][b] = mfma_step<DT>(w[d][a], x[d][b], acc[a][b]);
                fetch(s + d + kAhead, w[d], x[d]);
            }
    }

    // ---- the waves' sums meet
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) sums[(wave * TM + a * 16 + 4 * g + r) * TN + b * 16 + l16] = acc[a][b][r];
    __syncthreads();
    const int64_t plane = (int64_t)p.Ho * p.Wo;
#pragma unroll
    for (int e0 = 0; e0 < TM * TN; e0 += THREADS) {
        const int e = e0 + tid, f = e / TN, pp = pt * TN + e % TN, k = ft * TM + f;
        if (e >= TM * TN || pp >= p.px || k >= p.K) continue;
        float v[2] = {sums[e], sums[TM * TN + e]};
#pragma unroll
        for (int s = 2; s < S; ++s) v[s & 1] = add<DT>(v[s & 1], sums[s * TM * TN + e]);
        const int Q = fdiv(pp, p.d_wo), xx = pp - Q * p.Wo, n = fdiv(Q, p.d_ho), y = Q - n * p.Ho;
        p.out[((int64_t)n * p.K + k) * plane + (int64_t)y * p.Wo + xx] = add<DT>(v[0], v[1]);
    }
}

template <int DT, int A, int B, int S>
int short_half_launch(const void* in, const void* filt, float* out, const Shape& s, hipStream_t st, bool blocked)
{
    const int run = s.C * elem_bytes(DT), groups = run / kHalfChunkBytes;
    HalfShortParams p{(const char*)in, (const char*)filt, out, s.N, s.H, s.W, s.K, s.F, s.Ho, s.Wo,
                      s.H * s.W * run, s.F * s.F * run, blocked ? kHalfChunkBytes : run,
                      blocked ? s.H * s.W * kHalfChunkBytes : kHalfChunkBytes, groups * s.F * s.F, 0, blocked ? 1 : 0,
                      s.N * s.Ho * s.Wo, 0, 0, 0, 0, make_fastdiv(s.Wo), make_fastdiv(s.Ho),
                      make_fastdiv(blocked ? s.F * s.F : groups), make_fastdiv(s.F), {}};
    p.steps = (p.units + 1) / 2;
    p.ptiles = (p.px + 16 * B - 1) / (16 * B);
    p.ftiles = (s.K + 16 * A - 1) / (16 * A);
    p.total = p.ptiles * p.ftiles;
    p.by_filter = (int64_t)s.K * p.row > (int64_t)s.N * p.image;
    p.d_tiles = make_fastdiv(p.by_filter ? p.ptiles : p.ftiles);
    const int lds = p.steps * 8 + S * A * B * 1024;
    auto kern = short_half_kernel<DT, A, B, S>;
    static std::atomic<uint64_t> lds_limit_raised{0};
    // (64 KB need no raised limit: a call of a few microseconds is spared the look at the device)
    if (lds > 65536 && !raise_lds_limit((const void*)kern, kGenLdsLimit, lds_limit_raised)) return DCONV_LAUNCH_FAILED;
    begin_launch();
    hipLaunchKernelGGL(kern, dim3((unsigned)((p.total + 7) / 8 * 8)), dim3(64 * S), (size_t)lds, st, p);
    return launch_status();
}

template <int DT>
int short_half_dtype(const void* in, const void* filt, float* out, const Shape& s, hipStream_t st, bool blocked, int cfg)
{
    switch (cfg) {
    case 0: return short_half_launch<DT, 1, 1, 4>(in, filt, out, s, st, blocked);
    case 1: return short_half_launch<DT, 2, 2, 4>(in, filt, out, s, st, blocked);
    case 2: return short_half_launch<DT, 4, 2, 4>(in, filt, out, s, st, blocked);
    case 3: return short_half_launch<DT, 4, 4, 2>(in, filt, out, s, st, blocked);
    case 4: return short_half_launch<DT, 4, 4, 4>(in, filt, out, s, st, blocked);
    default: return DCONV_UNSUPPORTED;
    }
}

bool short_half_supports(const Shape& s, int dtype)
{
    // whole units, their offsets in a table in LDS, 32-bit byte offsets into every tensor
    const int64_t run = (int64_t)s.C * elem_bytes(dtype), lim = 1LL << 30;
    return run % kHalfChunkBytes == 0 && run / kHalfChunkBytes * s.F * s.F <= 16384 && s.K * s.F * s.F * run < lim &&
           (int64_t)s.N * s.H * s.W * run < lim && (int64_t)s.N * s.Ho * s.Wo * s.K < lim;
}

}  // namespace

// Kernel times of the configurations in microseconds, fitted to 947 layers drawn at random and measured from
// replayed graphs (16 to 512 channels and filters of 1x1 to 7x7, 7 x 7 to 128 x 128 maps, 1 to 64 images, 8 and 16
// bits, both layouts, up to 12 GFLOP; rms 15 %): launch, steps of a wave (their latency), steps of the waves of
// a SIMD beyond its first, waves, memory and output.  The configuration picked is 2.5 % above the fastest on average.
double short_half_time(const Shape& s, int dtype, int* cfg)
{
    // (filters and pixels of a tile and waves as powers of two: whole arithmetic, as the smallest calls take no
    // longer on the GPU than on the host)
    static const struct { int m, n, s; double launch, chain, more, wave, mb, out; } kCfg[] = {
        {4, 4, 2, 3.185, 0.127, 0.129, 0.025, 0.308, 0.313}, {5, 5, 2, 3.739, 0.244, 0.254, 0.057, 0.158, 0.253},
        {6, 5, 2, 4.219, 0.352, 0.340, 0.000, 0.188, 0.384}, {6, 6, 1, 6.045, 0.266, 0.415, 0.000, 0.196, 0.240},
        {6, 6, 2, 5.404, 0.444, 0.411, 0.234, 0.098, 0.429}};
    if (!short_half_supports(s, dtype)) return 1e300;
    const int64_t px = (int64_t)s.N * s.Ho * s.Wo, run = (int64_t)s.C * elem_bytes(dtype);
    const int64_t steps = (run / kHalfChunkBytes * s.F * s.F + 1) / 2;
    const double out = 4e-6 * px * s.K, mb = 1e-6 * run * ((double)s.N * s.H * s.W + (double)s.K * s.F * s.F) + out;
    auto up = [](int64_t n, int log2) { return (n + (1 << log2) - 1) >> log2; };
    double best = 1e300;
    for (int c = 0; c < 5; ++c) {
        const auto& k = kCfg[c];
        const double chain = (double)up(steps, k.s);
        const double waves = (double)((up(px, k.n) * up(s.K, k.m)) << k.s) * (1.0 / 1024);     // per SIMD
        const double t = k.launch + k.chain * chain + k.more * std::max(0.0, waves - 1) * chain + k.wave * waves + k.mb * mb + k.out * out;
        if (t < best) { best = t; *cfg = c; }
    }
    return best;
}

int launch_short_half(const void* in, const void* filt, float* out, const Shape& s, hipStream_t st, int dtype, bool blocked, int cfg)
{
    if (!short_half_supports(s, dtype) || (((uintptr_t)in) & 15) != 0 || (((uintptr_t)filt) & 15) != 0) return DCONV_UNSUPPORTED;
    switch (dtype) {
    case kF16: return short_half_dtype<kF16>(in, filt, out, s, st, blocked, cfg);
    case kBF16: return short_half_dtype<kBF16>(in, filt, out, s, st, blocked, cfg);
    case kI8: return short_half_dtype<kI8>(in, filt, out, s, st, blocked, cfg);
    default: return DCONV_UNSUPPORTED;
    }
}

}  // namespace dconv
