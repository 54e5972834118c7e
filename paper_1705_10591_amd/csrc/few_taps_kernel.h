// The general case with few filters, on the fp32 matrix cores: the TAPS of all filters are the rows of a
// product.
//
// A block of 32 filters would be nearly empty with three.  Instead every input row is multiplied by the
// K * F * F x C matrix of all weights, which gives for every pixel what it adds to the outputs around
// it, P[k, i, j][x] = sum_c w[k, c, i, j] in[c][y][x]; the sums out[k][y - i][x - j] += P[k, i, j][x] are then
// shifted additions, one per tap and pixel whatever the number of channels.  Three 3x3 filters fill 27 of 32
// rows, every pixel is loaded once (per band of rows), straight into the registers that the product reads.
//
//  * A wave holds 64 pixels of a row: lane (g, l) loads four pixels of channel 4 q + g, 16 bytes, and the four are
//    the columns of four products (pixel 4 l + b in product b), so a lane ends with four pixels of a tap row next to
//    each other.  Loads run kAhead * 16 channels ahead, across rows.
//  * A phase is four waves' rows: one row of up to 256 columns, two of 128, four of 64.  Their P goes to LDS; behind
//    a barrier a thread takes a column and some filters, adds the F x F taps up and keeps the F - 1 rows of
//    outputs that are not complete yet in LDS, its own.  Two sets of P where they fit, so that the next phase's
//    products begin meanwhile.
//  * A workgroup, of four or eight waves, has a band of rows of a column strip of an image.
//
// Errors: sixteen channels are summed by themselves, the groups then, the taps last: 0.97e-7 of the norm with 64
// channels of 3x3 and values in -1 .. 1, 1.2e-7 with activations (the vector-ALU kernel, one chain of 576, 4.3e-7 and 4.6e-7).
//
// What bounds it: 8 x 64 x 224 x 224, three 3x3 filters: 50 -> 36 us by the call, 33.5 the kernel.  10 rows of products a CU take
// 17.6 us on the fp32 matrix cores (27 rows of 32, 224 columns of 256, 9 rows for 7 of output), their input 21 us
// at 5 TB/s; the additions and barriers between phases cost 0.7 us a phase (with four waves a workgroup, one
// row a phase: 2 us more).  16 x 256 x 64 x 64, three 3x3 filters (on the general kernel before): 93 -> 28 us;
// 4 x 128 x 56 x 56: 26 -> 11.3; 8 x 64 x 224 x 224, twelve 1x1 filters: 43 -> 26 (kernels replayed from a graph).
#pragma once
#include <algorithm>
#include <cmath>
#include "general_kernel.h"

namespace dconv {

constexpr int kFtMostBlocks = 7;                // blocks of sixteen tap rows
constexpr int kFtLds = 81920;                   // half of a CU's

struct FewTapsParams {
    const float* in;
    const float* filt;
    float* out;
    int N, C, H, W, K, Ho, Wo;
    int cb, nstrips, so;     // column blocks of 64 per row, strips, output columns per strip
    int rb, nbands;          // output rows per band
    int cgs;                 // groups of sixteen channels
    int bufs;                // sets of P
    int total;               // workgroups
    FastDiv d_strips, d_bands, d_c, d_ff;
};

template <int F, int MB, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
few_taps_kernel(FewTapsParams p)
{
    constexpr int FF = F * F, THREADS = 64 * NW, PW = THREADS + 16;      // (a tap's columns of all rows of a phase, and what the last ones read past them)
    constexpr int kAhead = MB <= 2 ? 4 : MB <= 4 ? 3 : 2;
    constexpr uint32_t kNowhere = 0xC0000000u;
    constexpr int kRsrcFlags = 0x00020000;

    extern __shared__ __attribute__((aligned(16))) v4f lds_quads[];
    const int R = p.K * FF;
    v4f* const wts = lds_quads;                                 // [group of channels][block][lane]: channels 4 q + g, q = 0..3
    float* const P0 = (float*)(wts + p.cgs * MB * 64);          // [set][tap][column]
    float* const S = P0 + p.bufs * R * PW;                      // [filter][row to come][column], a thread's own

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, l16 = lane & 15;
    const int G = gridDim.x;
    const int wg = (G % 8 == 0) ? (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
    if (wg >= p.total) return;                                  // uniform: before any barrier

    const int up = fdiv(wg, p.d_strips), strip = wg - up * p.nstrips;
    const int n = fdiv(up, p.d_bands), y0 = (up - n * p.nbands) * p.rb;
    const int x0 = strip * p.so;
    const int rows = min(p.rb, p.Ho - y0) + F - 1;              // input rows of the band
    const int rp = NW / p.cb, cols = p.cb * 64;
    const int phases = (rows + rp - 1) / rp;
    const int HW = p.H * p.W;

    // ---- what a wave loads: row `wave / cb` of a phase, columns from (wave % cb) * 64 on
    const int wrow = wave / p.cb, wcol = (wave % p.cb) * 64;
    const int64_t image = (int64_t)n * p.C * HW * 4, left = (int64_t)p.N * p.C * HW * 4 - image;
    const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.in + image), 0, (int)min(left, (int64_t)0x7FFFFFFF), kRsrcFlags);
    const bool inside = x0 + wcol + 4 * l16 < p.W;
    const uint32_t vfirst = (uint32_t)(g * HW + y0 * p.W + x0 + wcol + 4 * l16) * 4u;
    v4f x[kAhead][4];
    auto fetch = [&](int phase, int cg, v4f (&x)[4]) __attribute__((always_inline)) {
        const int row = phase * rp + wrow;
        const uint32_t v = inside && row < rows && cg < p.cgs ? vfirst + (uint32_t)(row * p.W) * 4u : kNowhere;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = cg * 16 + q * 4;
            const uint32_t vq = c + 4 <= p.C || c + g < p.C ? v : kNowhere;      // (channels beyond C are zero)
            x[q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rs, vq, c * HW * 4, 0));
        }
    };
#pragma unroll
    for (int d = 0; d < kAhead; ++d) fetch(0, d, x[d]);

    // ---- weights: read as they lie, written where the products read them
    for (int e = tid; e < p.cgs * MB * 64; e += THREADS) wts[e] = v4f{};
    __syncthreads();
    {
        const int words = p.K * p.C * FF;
#pragma unroll 4
        for (int e = tid; e < words; e += THREADS) {
            const int kc = fdiv(e, p.d_ff), t = e - kc * FF, k = fdiv(kc, p.d_c), c = kc - k * p.C;
            const int row = k * FF + t, cg = c >> 4, q = (c >> 2) & 3;
            ((float*)&wts[(cg * MB + (row >> 4)) * 64 + (c & 3) * 16 + (row & 15)])[q] = p.filt[e];
        }
    }
    for (int e = tid; e < p.K * (F - 1) * cols; e += THREADS) S[e] = 0.f;
    __syncthreads();

    const int64_t plane = (int64_t)p.Ho * p.Wo;
    const int mycol = tid & (cols - 1), mygroup = tid / cols;    // this thread's column; filters mygroup, mygroup + rp, ...
    const bool writes = mycol < p.so && x0 + mycol < p.Wo;
    float* const dst = p.out + (int64_t)n * p.K * plane + (int64_t)y0 * p.Wo + x0 + mycol;

    auto meet = []() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // (sixteen channels are summed by themselves before they join the total where registers allow it)
    constexpr bool kApart = MB <= 4;
    v4f acc[MB][4], part[kApart ? MB : 1][4];
    for (int phase = 0; phase < phases; ++phase) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[m][b] = v4f{};
        for (int c0 = 0; c0 < p.cgs; c0 += kAhead)
#pragma unroll
            for (int d = 0; d < kAhead; ++d) {
                const int cg = c0 + d;
                if (cg < p.cgs) {                               // uniform
                    auto& sum = [&]() -> auto& { if constexpr (kApart) return part; else return acc; }();
                    v4f a[MB];
#pragma unroll
                    for (int m = 0; m < MB; ++m) a[m] = wts[(cg * MB + m) * 64 + lane];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int m = 0; m < MB; ++m)
#pragma unroll
                            for (int b = 0; b < 4; ++b)
                                sum[m][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m][q], x[d][q][b], kApart && q == 0 ? v4f{} : sum[m][b], 0, 0, 0);
                    if (kApart) {
#pragma unroll
                        for (int m = 0; m < MB; ++m)
#pragma unroll
                            for (int b = 0; b < 4; ++b) acc[m][b] += sum[m][b];
                    }
                }
                // what takes this place next: kAhead groups on, or the next row's (always the same number of loads, so
                // that the compiler can count the ones under way: where there is nothing to bring they read nothing)
                const bool wraps = c0 + kAhead >= p.cgs;
                fetch(wraps ? phase + 1 : phase, wraps ? d : cg + kAhead, x[d]);
                __builtin_amdgcn_sched_barrier(0);
            }
        float* const P = P0 + (phase % p.bufs) * R * PW;
#pragma unroll
        for (int m = 0; m < MB; ++m) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m * 16 + 4 * g + r;
                if (row < R) *(v4f*)(P + row * PW + wave * 64 + 4 * l16) = v4f{acc[m][0][r], acc[m][1][r], acc[m][2][r], acc[m][3][r]};
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        meet();
        for (int s = 0; s < rp; ++s) {
            const int row = phase * rp + s;
            if (row >= rows) break;                             // uniform
            for (int k = mygroup; k < p.K; k += rp) {
                const float* src = P + k * FF * PW + s * cols + mycol;
                float* const sk = S + k * (F - 1) * cols + mycol;
                float next = 0.f;                               // what the rows above have left for the output row at hand
#pragma unroll
                for (int i = F - 1; i >= 0; --i) {
                    float sum = src[i * F * PW];
#pragma unroll
                    for (int j = 1; j < F; ++j) sum += src[(i * F + j) * PW + j];
                    if (i > 0) sum += sk[(i - 1) * cols];
                    if (i == F - 1) next = sum;
                    else sk[i * cols] = sum;
                }
                if (writes && row >= F - 1) dst[k * plane + (int64_t)(row - (F - 1)) * p.Wo] = next;
            }
        }
        if (p.bufs == 1) meet();
    }
}

// ---- host side -----------------------------------------------------------------------------------

// Waves and rows of a workgroup, by an estimate of what one costs a CU: the products of its rows, the additions
// behind them, which another workgroup of the CU covers in part.
inline FewTapsPlan few_taps_plan(const Shape& s)
{
    FewTapsPlan pl{};
    const int R = s.K * s.F * s.F;
    if (s.F > 7 || s.K > 16 || R > 16 * kFtMostBlocks) return pl;
    pl.mb = (R + 15) / 16;
    pl.cb = s.W <= 64 ? 1 : s.W <= 128 ? 2 : 4;
    pl.so = (pl.cb * 64 - (s.F - 1)) & ~3;
    if (s.W <= pl.cb * 64) pl.so = pl.cb * 64;                   // (one strip: no columns shared)
    pl.nstrips = (s.Wo + pl.so - 1) / pl.so;
    pl.cgs = (s.C + 15) / 16;
    const double product = pl.cgs * 16 * pl.mb * 33 / 2300.0;    // us of a SIMD's matrix cores for a wave's row
    double least = 1e300;
    for (int nw : {4, 8}) {
        const int rp = nw / pl.cb;
        const int fixed = pl.cgs * pl.mb * 1024 + s.K * (s.F - 1) * pl.cb * 256, set = R * (64 * nw + 16) * 4;
        const int bufs = fixed + 2 * set <= (nw == 4 ? kFtLds : kGenLdsLimit) ? 2 : 1, lds = fixed + bufs * set;
        if (lds > kGenLdsLimit || (nw == 8 && pl.mb > 4)) continue;
        const bool two = lds <= kFtLds;                          // workgroups per CU
        const double add = 0.4 + 0.25 * s.K;           // us of a phase that is not products
        for (int want : {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 56, 64, 80, 96, 128}) {
            const int rb = std::min(want, s.Ho);
            const int nbands = (s.Ho + rb - 1) / rb;
            const double wgs = (double)s.N * nbands * pl.nstrips, phases = (rb + s.F - 1 + rp - 1) / rp;
            if (wgs > 2e9) continue;
            const double per_cu = std::ceil(wgs / 256);
            const double one = nw / 4 * product + add, both = 2 * product * nw / 4 + 0.3 * add;
            const double cost = (two ? std::floor(per_cu / 2) * std::max(one, both) + std::fmod(per_cu, 2.0) * one : per_cu * one) * phases + 1.0 * per_cu;
            if (cost >= least) continue;
            least = cost;
            pl.nw = nw; pl.rb = rb; pl.nbands = nbands; pl.bufs = bufs; pl.lds = lds;
            pl.total = (int)wgs;
            pl.cost = cost;
            pl.ok = true;
            if (want >= s.Ho) break;
        }
    }
    if ((int64_t)(s.C + 16) * s.H * s.W >= 1LL << 29) pl.ok = false;      // lanes address an image with 32-bit byte offsets
    return pl;
}

template <int F, int MB, int NW>
int few_taps_launch(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, const FewTapsPlan& pl)
{
    auto kern = few_taps_kernel<F, MB, NW>;
    static std::atomic<uint64_t> lds_limit_raised{0};
    if (!raise_lds_limit((const void*)kern, kGenLdsLimit, lds_limit_raised)) return DCONV_LAUNCH_FAILED;
    FewTapsParams p{in, filt, out, s.N, s.C, s.H, s.W, s.K, s.Ho, s.Wo, pl.cb, pl.nstrips, pl.so, pl.rb, pl.nbands, pl.cgs, pl.bufs, pl.total,
                    make_fastdiv(pl.nstrips), make_fastdiv(pl.nbands), make_fastdiv(s.C), make_fastdiv(F * F)};
    begin_launch();
    hipLaunchKernelGGL(kern, dim3((unsigned)((pl.total + 7) / 8 * 8)), dim3(64 * NW), (size_t)pl.lds, st, p);
    return launch_status();
}

// Implemented once per filter side, each in its own translation unit.
template <int F>
int few_taps_for_F(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, const FewTapsPlan& pl);

}  // namespace dconv
