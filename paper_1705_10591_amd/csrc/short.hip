// The general case for SHORT launches: layers whose tiles do not fill the chip, fp32 matrix cores, one kernel.
//
// A layer of a few hundred MFLOP takes the tiled kernel one round of large tiles on part of the chip, or tiles
// cut over channels whose parts a second kernel adds.  Here a workgroup has a small tile, 16 A filters x 16 B
// pixels, and its S waves share the reduction: each takes a stretch of the C * F * F taps, in the order in which
// the weights lie, and the waves' sums meet in LDS.  Operands come straight from memory (the L2, at these
// sizes) into the registers that v_mfma_f32_16x16x4_f32 reads, kAhead steps of sixteen taps ahead: no staging, no
// barrier before the end, nothing but the launch and one round of latencies in front of the first product.
//  * Lane (g, l) of a step loads weights 4 g .. 4 g + 3 of filter l, 16 bytes; product q takes word q of them, so
//    its reduction index g is tap 4 g + q, of which lane (g, l) loads pixel l: sixteen pixels next to each other.
//  * A tap's offset from its pixel is the same for all pixels: every wave makes a table of its stretch in LDS, one
//    16-byte read a step.
//  * Pixels are numbered along (image, y, x); the last ones of a tile may be none.
//  * Sixteen taps are summed by themselves, every other one of 32, before they join a wave's sum.
#include <algorithm>
#include <cmath>
#include "general_kernel.h"

namespace dconv {

namespace {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

struct ShortParams {
    const float* in;
    const float* filt;
    float* out;
    int N, C, H, W, K, F, Ho, Wo;
    int T, steps;            // taps; steps of sixteen
    int px, ptiles, ftiles, total;
    int by_filter;           // workgroups next to each other share filters, not pixels
    FastDiv d_wo, d_ho, d_ff, d_f, d_tiles;
};

template <int A, int B, int S>
__global__ void __launch_bounds__(64 * S)
short_kernel(ShortParams p)
{
    constexpr int kAhead = 4, THREADS = 64 * S, TM = 16 * A, TN = 16 * B;
    constexpr uint32_t kNowhere = 0xC0000000u;
    constexpr int kRsrcFlags = 0x00020000;

    extern __shared__ __attribute__((aligned(16))) v4u lds_words[];
    // offsets of taps: all waves' stretches one after the other, whole steps; then [wave][filter][pixel] sums
    uint32_t* const table = (uint32_t*)lds_words;
    float* const sums = (float*)(lds_words + (p.steps + S) * 4);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, l16 = lane & 15;
    const int G = gridDim.x;
    const int wg = (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8);
    if (wg >= p.total) return;                                  // uniform: before any barrier
    const int major = fdiv(wg, p.d_tiles), minor = wg - major * p.d_tiles.d;
    const int ft = p.by_filter ? major : minor, pt = p.by_filter ? minor : major;

    const int HW = p.H * p.W;
    const int s0 = range_start(wave, p.steps, S), s1 = range_start(wave + 1, p.steps, S);

    // ---- this wave's stretch of the table (taps beyond the last are nowhere)
    for (int e = s0 * 16 + lane; e < s1 * 16; e += 64) {
        const int c = fdiv(e, p.d_ff), ij = e - c * p.F * p.F, i = fdiv(ij, p.d_f);
        table[e] = e < p.T ? (uint32_t)(c * HW + i * p.W + ij - i * p.F) * 4u : kNowhere;
    }

    // ---- what a lane loads
    const auto irs = __builtin_amdgcn_make_buffer_rsrc((void*)p.in, 0, p.N * p.C * HW * 4, kRsrcFlags);
    const auto wrs = __builtin_amdgcn_make_buffer_rsrc((void*)p.filt, 0, p.K * p.T * 4, kRsrcFlags);
    uint32_t pix[B], row[A];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int pp = pt * TN + b * 16 + l16, Q = fdiv(pp, p.d_wo), x = pp - Q * p.Wo, n = fdiv(Q, p.d_ho), y = Q - n * p.Ho;
        pix[b] = pp < p.px ? (uint32_t)(n * p.C * HW + y * p.W + x) * 4u : kNowhere;
    }
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int k = ft * TM + a * 16 + l16;
        row[a] = k < p.K ? (uint32_t)(k * p.T + 4 * g) * 4u : kNowhere;
    }
    v4f w[kAhead][A], x[kAhead][B];
    auto fetch = [&](int s, v4f (&w)[A], v4f (&x)[B]) __attribute__((always_inline)) {
        const v4u off = *(const v4u*)(table + min(s, s1 - 1) * 16 + 4 * g);
        const bool there = s < s1;                              // uniform; beyond the stretch nothing is read
#pragma unroll
        for (int a = 0; a < A; ++a)
            w[a] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(wrs, there ? row[a] : kNowhere, s * 64, 0));
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // (no sum of the two is below the extent unless both are there)
                const uint32_t o = there ? pix[b] + off[q] : kNowhere;
                x[b][q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(irs, o, 0, 0));
            }
    };
    v4f acc[A][B], part[A][B][2];
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b) { acc[a][b] = v4f{}; part[a][b][0] = v4f{}; part[a][b][1] = v4f{}; }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the wave's table is in LDS
    if (s0 < s1) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d) fetch(s0 + d, w[d], x[d]);
        for (int s = s0; s < s1; s += kAhead)
#pragma unroll
            for (int d = 0; d < kAhead; ++d) {
                if (s + d < s1) {                               // uniform
                    // (the last step: weights beyond the last tap are another filter's, against pixels that are zero)
                    if ((s + d + 1) * 16 > p.T) {
#pragma unroll
                        for (int a = 0; a < A; ++a)
#pragma unroll
                            for (int q = 0; q < 4; ++q) w[d][a][q] = (s + d) * 16 + 4 * g + q < p.T ? w[d][a][q] : 0.f;
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int a = 0; a < A; ++a)
#pragma unroll
                            for (int b = 0; b < B; ++b)
                                part[a][b][q & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[d][a][q], x[d][b][q], part[a][b][q & 1], 0, 0, 0);
                    if ((s + d - s0) & 1) {
#pragma unroll
                        for (int a = 0; a < A; ++a)
#pragma unroll
                            for (int b = 0; b < B; ++b) {
                                acc[a][b] += part[a][b][0] + part[a][b][1];
                                part[a][b][0] = v4f{};
                                part[a][b][1] = v4f{};
                            }
                    }
                }
                fetch(s + d + kAhead, w[d], x[d]);
            }
    }

    // ---- the waves' sums meet
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) sums[(wave * TM + a * 16 + 4 * g + r) * TN + b * 16 + l16] = acc[a][b][r] + (part[a][b][0][r] + part[a][b][1][r]);
    __syncthreads();
    const int64_t plane = (int64_t)p.Ho * p.Wo;
#pragma unroll
    for (int e0 = 0; e0 < TM * TN; e0 += THREADS) {
        const int e = e0 + tid, f = e / TN, pp = pt * TN + e % TN, k = ft * TM + f;
        if (e >= TM * TN || pp >= p.px || k >= p.K) continue;
        float v[4] = {};
#pragma unroll
        for (int s = 0; s < S; ++s) v[s & 3] += sums[s * TM * TN + e];
        const int Q = fdiv(pp, p.d_wo), xx = pp - Q * p.Wo, n = fdiv(Q, p.d_ho), y = Q - n * p.Ho;
        p.out[((int64_t)n * p.K + k) * plane + (int64_t)y * p.Wo + xx] = (v[0] + v[1]) + (v[2] + v[3]);
    }
}

template <int A, int B, int S>
int short_launch(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st)
{
    ShortParams p{in, filt, out, s.N, s.C, s.H, s.W, s.K, s.F, s.Ho, s.Wo, s.C * s.F * s.F, 0, s.N * s.Ho * s.Wo, 0, 0, 0, 0,
                  make_fastdiv(s.Wo), make_fastdiv(s.Ho), make_fastdiv(s.F * s.F), make_fastdiv(s.F), {}};
    p.steps = (p.T + 15) / 16;
    p.ptiles = (p.px + 16 * B - 1) / (16 * B);
    p.ftiles = (s.K + 16 * A - 1) / (16 * A);
    p.total = p.ptiles * p.ftiles;
    p.by_filter = (int64_t)s.K * p.T > (int64_t)s.N * s.C * s.H * s.W;
    p.d_tiles = make_fastdiv(p.by_filter ? p.ptiles : p.ftiles);
    const int lds = (p.steps + S) * 64 + S * A * B * 1024;
    auto kern = short_kernel<A, B, S>;
    static std::atomic<uint64_t> lds_limit_raised{0};
    // (64 KB need no raised limit: a call of a few microseconds is spared the look at the device)
    if (lds > 65536 && !raise_lds_limit((const void*)kern, kGenLdsLimit, lds_limit_raised)) return DCONV_LAUNCH_FAILED;
    begin_launch();
    hipLaunchKernelGGL(kern, dim3((unsigned)((p.total + 7) / 8 * 8)), dim3(64 * S), (size_t)lds, st, p);
    return launch_status();
}

bool short_supports(const Shape& s)
{
    // taps in a table in LDS, 32-bit byte offsets into every tensor
    const int64_t T = (int64_t)s.C * s.F * s.F, lim = 1LL << 28;
    return T <= 16384 && s.K * T < lim && (int64_t)s.N * s.C * s.H * s.W < lim && (int64_t)s.N * s.Ho * s.Wo < lim / 64;
}

}  // namespace

// Kernel times of the configurations and the general kernels, in microseconds, fitted to 1000 layers drawn at
// random and measured from replayed graphs (1 to 512 channels, 9 to 512 filters of 1x1 to 11x11, 7 x 7 to 128 x 256
// maps, 1 to 64 images, up to 6 GFLOP; rms 8 to 15 % and 18 %): launch, steps of a wave (their latency), steps of
// the waves of a SIMD beyond its first, waves, memory and output.  The configuration picked is 2 % above the
// fastest on average.
static double short_time(const Shape& s, int* cfg)
{
    static const struct { int a, b, waves; double launch, chain, more, wave, mb, out; } kCfg[] = {
        {1, 1, 4, 3.72, 0.253, 0.154, 0.000, 0.073, 0.565}, {1, 1, 8, 3.70, 0.400, 0.158, 0.000, 0.083, 0.882},
        {2, 2, 2, 4.66, 0.540, 0.372, 0.112, 0.070, 0.356}, {2, 2, 4, 4.33, 0.580, 0.363, 0.195, 0.041, 0.402},
        {2, 1, 8, 3.65, 0.566, 0.225, 0.173, 0.051, 0.509}};
    const double px = (double)s.N * s.Ho * s.Wo, T = (double)s.C * s.F * s.F, steps = std::ceil(T / 16);
    const double out = 4e-6 * px * s.K, mb = 4e-6 * ((double)s.N * s.C * s.H * s.W + s.K * T) + out;
    double best = 1e300;
    for (int c = 0; c < 5; ++c) {
        const auto& k = kCfg[c];
        const double chain = std::ceil(steps / k.waves);
        const double waves = std::ceil(px / (16 * k.b)) * std::ceil(s.K / (16.0 * k.a)) * k.waves / 1024;      // per SIMD
        const double t = k.launch + k.chain * chain + k.more * std::max(0.0, waves - 1) * chain + k.wave * waves + k.mb * mb + k.out * out;
        if (t < best) { best = t; *cfg = c; }
    }
    return best;
}

// The general kernel, by the tiles of the shape's own choice: 5.4, whole tiles one after the other on the CUs at
// 150 TFLOP/s or, if that is less, what sharing them takes, the root of the products' time, memory at 7 TB/s
// beside it and 0.25 per thousand taps; rms 15.5 %.  It has to promise a tenth: of 4531 layers that the fit did
// not see (both kernels' times within 19 % rms of their estimates) 2889 are chosen, 1.86 times faster on average (1 x 256 x 14 x 14
// with 256 3x3 filters 16.3 -> 8.7 us, 8 x 50 x 30 x 30 with 90 24.9 -> 14.1, 4 x 64 x 28 x 28 with 64 12.9 -> 9.6, 16 x 32 x
// 14 x 14 with 96 1x1 filters 8.3 -> 4.3), 94 of them 3 % or more slower, 57 by more than a tenth (7 to 40 us; few filters on few
// channels and large maps among them, the worst 13.6 -> 23.6).  With 15 % 52 would be, and 233 layers fewer be chosen, most of
// them faster here and all of them closer to the exact sums.  A list of slower ones:
// profiles/rule_short_launches.txt.  Errors against 64 bits: 1.85e-7 -> 1.09e-7 with 256 channels.
struct GeneralTiles { double even, whole; };
static GeneralTiles general_tiles(const Shape& s)
{
    const int shape = general_auto_shape(s), mt = shape == 2 ? 32 : 64, nt = shape == 0 ? 128 : 256;
    const double tiles = std::ceil((double)s.N * s.Ho * s.Wo / nt) * ((s.K + mt - 1) / mt);
    const double one = mt * nt * (double)s.C * s.F * s.F * 3.4e-6, even = tiles * one / 256;            // us of a CU
    return {even, tiles <= 256 * (shape == 1 ? 2 : 3) ? std::ceil(tiles / 256) * one : even};
}

ShortChoice short_choice(const Shape& s)
{
    ShortChoice r{1e300, 0};
    if (!short_supports(s)) return r;
    const double here = short_time(s, &r.cfg);
    if (s.N == 1 && s.C == 1) return r;
    const double px = (double)s.N * s.Ho * s.Wo, T = (double)s.C * s.F * s.F;
    const double mb = 4e-6 * ((double)s.N * s.C * s.H * s.W + s.K * T + px * s.K);
    const GeneralTiles t = general_tiles(s);
    const double there = 5.44 + 1.067 * std::min(t.whole, 1.2 * t.even + 4) + 0.016 * t.even + 0.139 * mb + 2.1 * std::sqrt(t.even) + 0.25e-3 * T;
    if (here < 0.9 * there) r.time = here;
    return r;
}

bool general_would_share_tiles(const Shape& s)
{
    const GeneralTiles t = general_tiles(s);
    return t.whole > 1.2 * t.even + 4;
}

int launch_short(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, int cfg)
{
    if (!short_supports(s)) return DCONV_UNSUPPORTED;
    switch (cfg) {
    case 0: return short_launch<1, 1, 4>(in, filt, out, s, st);
    case 1: return short_launch<1, 1, 8>(in, filt, out, s, st);
    case 2: return short_launch<2, 2, 2>(in, filt, out, s, st);
    case 3: return short_launch<2, 2, 4>(in, filt, out, s, st);
    case 4: return short_launch<2, 1, 8>(in, filt, out, s, st);
    default: return DCONV_UNSUPPORTED;
    }
}

}  // namespace dconv
