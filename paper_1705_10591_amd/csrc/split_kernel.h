// General-case direct convolution in fp32 on the bf16 matrix cores of gfx950.
//
// v_mfma_f32_32x32x2_f32 forms 32 multiply-adds per lane in 64 cycles, v_mfma_f32_32x32x16_bf16
// 256 in 32: sixteen times the rate.  A 24-bit fp32 value is the exact sum of three bf16 values,
// x = x_h + x_m + x_l (each the rest rounded to the eight bits of bf16), so
//   x * w = h h' + (h m' + m h') + (m m' + h l' + l h') + (m l' + l m' + l l')
// with |m| <= 2^-8 |x| and |l| <= 2^-17 |x|.  The last three are left out, 2^-24 |x w| at most together,
// and six bf16 instructions do the work of eight fp32 ones of twice the length: the matrix-core
// time of a layer falls to 6/16.  Products of parts are exact and the sums stay in fp32.
// Errors of dense sums against 64 bits are smaller than those of the fp32 instructions (fewer
// additions per sum: an instruction adds eight products at a time, large and small products are
// summed apart, and every block of sixteen channels is summed by itself before it joins the
// total): 7.6e-7 -> 1.0e-7 with 256 channels of 3x3, 2.7e-7 -> 0.7e-7 with 64.  A sum of one term,
// which the fp32 instructions round once, may be off by 1 ulp.
//
// What is kept from general_tiled_kernel: Algorithm 2's (filter block) x (pixel block) tiles,
// pixels numbered along (n, y, x) of a column strip, channel chunks staged in LDS with the next
// ones on their way, a persistent launch over (tile, chunk) units whose ranges may end inside a
// tile.  What differs:
//  * tile: 64 filters x 256 pixels, eight waves of 64 x 32, two per SIMD, which take turns at the
//    matrix cores (see the main loop);
//  * chunk: sixteen channels; a matrix-core step is one tap of sixteen channels, a lane's operand
//    eight channels of one pixel or filter in bf16: 16 bytes, one LDS read;
//  * images are split on the way to LDS: a thread loads the sixteen channels of one pixel (sixteen
//    planes, each load contiguous over the lanes), two at a time, splits them in registers and
//    writes 16-byte pieces.  Filters, which every pixel tile would split again, are split once
//    by a small kernel in front (split_filters_kernel) and copied to LDS as they lie.
//
// What bounds it: the chip's power (a bare loop of these instructions on random bits runs at 1.75
// of the published 2.5 PFLOP/s, i.e. 290 TFLOP/s of fp32 products), then the turns: 32 x 256 x
// 28 x 28 with 512 3x3 filters 420 -> 249 us = 205 TFLOP/s (122 on the fp32 instructions; 205 us
// with the staging left out), 64 x 128 x 56 x 56 with 128 459 -> 285 us.
//
// Values a bf16 triple cannot carry are found and their outputs computed again in fp32:
//  * infinities, NaN and values above the largest bf16: their splits make NaN, so every output
//    they reach is not finite; such outputs are formed again (redo_block);
//  * values below 2^-103, whose last parts may fall below the smallest bf16 (2^-133): each loses
//    at most 2^-134; where a tile has staged one, outputs below 2^-60 are formed again (all of
//    the tile's where values above 2^40 occur beside them).
// What that costs: a wave that has such an output computes its block of 64 filters x 32 pixels again
// behind the main loop, at the rate of its SIMD's fp32 matrix cores.  32 x 256 x 28 x 28 with 512 3x3
// filters, by events around a call: 278 us, one NaN pixel 596, a filter of values near 2^-110 502,
// nothing but NaN 967 (the fp32 kernel 460-490 for any data; with a lane for each such output, one after
// the other, 5500, 372 and 7560); 32 x 64 x 56 x 56 with 64: 62, 91, 200, 199 (fp32 83); few
// tiles of many taps, 8 x 97 x 25 x 25 with 250 7x7 filters: 75, 399, 420, 423 (fp32 100).
#pragma once
#include "general_kernel.h"

namespace dconv {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

struct SplitParams {
    const float* in;
    const float* filt;
    float* out;
    const v4u* wsplit;   // workspace: the filter bank split (split_filters_kernel)
    const int* wflags;   // workspace: one word per filter block of a phase, what its values are like
    float* part;     // workspace: partial tiles, [workgroup][2][MT * NT]
    int* cnt;        // workspace: arrivals per shared tile, indexed by its first workgroup; all 0
    int N, C, H, W, K, Ho, Wo;
    int bw, nstrips, LS, RS, pt_full, KB;      // as in HalfParams
    int nun;         // units per tile: channel chunks x row groups
    int tiles, G, split;
    int Hc;          // image-block rows set aside per image: Ho + IR - 1
    FastDiv d_strip, d_kb, d_wsf, d_wsl, d_ho, d_hc, d_ls, d_nun;
};

// A unit is sixteen channels x IR filter rows and has an image block of its own; it is consumed in
// phases of RG filter rows, each with a filter block of its own.  Both blocks have two slots in
// LDS.  Up to 4x4 an image block serves all filter rows; beyond, the LDS holds the rows that one
// filter row touches.
constexpr int split_image_rows(int F) { return F <= 4 ? F : 1; }
constexpr int split_phase_rows(int F) { return F <= 2 ? F : 1; }
constexpr int split_filter_block(int F) { return split_phase_rows(F) * F * 6 * 64; }     // 16-byte pieces
// pixels of an image block: a thread stages one
constexpr int split_most_pixels(int F)
{
    const int fit = ((kGenLdsLimit / 32 - split_filter_block(F)) / 3 - 1) / 2;
    return fit < 512 ? fit : 512;
}
template <int F, int IR_, int RG_>
struct SplitGeom {
    static constexpr int IR = IR_, RG = RG_;
    static_assert(F % IR == 0 && IR % RG == 0, "row groups of one size");
    static constexpr int NG = F / IR, NP = IR / RG;
    static constexpr int S = RG * F;                  // matrix-core steps per phase
    static constexpr int THREADS = 512, MT = 64, NT = 256, CK = 16;
    static constexpr int FB = split_filter_block(F);  // 16-byte pieces of a filter block: [tap][half][part][filter]
    static_assert(FB == S * 6 * MT, "filter block");
    static constexpr int NFI = (FB / 64 + 7) / 8;     // loads of 64 pieces per wave
    static constexpr int MOST = split_most_pixels(F);
    static constexpr int PS = 2 * MOST + 1;           // LDS pieces per part: [half][pixel], a spare one
    static constexpr int IB = 3 * PS;                 // LDS pieces of an image block
};

// A wave's block of 64 filters x 32 pixels in fp32, on the fp32 matrix cores, for the outputs that the
// split cannot form: those in `again` (bit 16 mt + r: accumulator r of block mt) are written.
// The two reduction indices of an instruction are two channels.  Operands come straight from memory,
// a filter row of two channels a time, kAhead rows ahead: a lane brings its pixel's words and the
// row of two filters, so the filter loads gather.
template <int F>
__device__ __forceinline__ void redo_block(const char* ibase, int64_t ileft, uint32_t ipix, const float* w, int wbytes, char* out,
                                           uint32_t again, int C, int W, int HW, int64_t plane)
{
    constexpr int FF = F * F, NA = (F + 3) / 4, kAhead = F <= 4 ? 4 : 2;
    constexpr uint32_t kNowhere = 0xC0000000u;
    constexpr int kRsrcFlags = 0x00020000;
    const int lane = threadIdx.x & 63, h = lane >> 5, l32 = lane & 31;
    const int rows = (C + 1) / 2 * F;
    v4f a[kAhead][2][NA];
    float b[kAhead][F];
    // (a channel beyond C and filters beyond K read zero)
    auto fetch = [&](int u, v4f (&a)[2][NA], float (&b)[F]) __attribute__((always_inline)) {
        u = min(u, rows - 1);
        const int c0 = u / F * 2, i = u % F;
        const bool there = c0 + h < C;
        const int64_t ioff = ((int64_t)c0 * HW + (int64_t)i * W) * 4;
        const int woff = (c0 * FF + i * F) * 4;
        const auto irs = __builtin_amdgcn_make_buffer_rsrc((void*)(ibase + ioff), 0, (int)min(ileft - ioff, (int64_t)0x7FFFFFFF), kRsrcFlags);
        const auto wrs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)w + woff), 0, wbytes - woff, kRsrcFlags);
        const uint32_t iv = there ? ipix + (uint32_t)(h * HW) * 4u : kNowhere;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const uint32_t wv = there ? (uint32_t)((mt * 32 + l32) * C + h) * (FF * 4u) : kNowhere;
#pragma unroll
            for (int q = 0; q < NA; ++q)
                a[mt][q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(wrs, wv + 16u * q, 0, 0));
        }
#pragma unroll
        for (int jj = 0; jj < F; ++jj) b[jj] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(irs, iv + 4u * jj, 0, 0));
    };
    v16f acc[2] = {};
#pragma unroll
    for (int d = 0; d < kAhead; ++d) fetch(d, a[d], b[d]);
    for (int u0 = 0; u0 < rows; u0 += kAhead)
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {
            if (u0 + d < rows) {                             // uniform
#pragma unroll
                for (int jj = 0; jj < F; ++jj)
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt) acc[mt] = mfma_32x32x2(a[d][mt][jj / 4][jj % 4], b[d][jj], acc[mt]);
            }
            fetch(u0 + d + kAhead, a[d], b[d]);
        }
#pragma unroll
    for (int r = 0; r < 32; ++r)
        if (again >> r & 1) *reinterpret_cast<float*>(out + (int64_t)((r >> 4) * 32 + mfma_row(r & 15, 0)) * plane * 4) = acc[r >> 4][r & 15];
}

// What a set of split values is like: the smallest last remainder that is not zero (its bits, less one,
// without the sign; below kSplitTiny it is subnormal and bf16 may have lost part of it) and the
// largest magnitude.
struct SplitRange {
    uint32_t least = 0xFFFFFFFFu;
    float most = 0.f;
    __device__ bool tiny() const { return least < 0x00FFFFFFu; }
    __device__ bool huge() const { return most > 0x1p40f; }
};

// Two values as three bf16 parts each, packed.
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& hb, uint32_t& mb, uint32_t& lb, SplitRange& range)
{
    hb = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){x0, x1}, v2bf));
    const float r0 = x0 - __builtin_bit_cast(float, hb << 16);
    const float r1 = x1 - __builtin_bit_cast(float, hb & 0xFFFF0000u);
    mb = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){r0, r1}, v2bf));
    const float s0 = r0 - __builtin_bit_cast(float, mb << 16);
    const float s1 = r1 - __builtin_bit_cast(float, mb & 0xFFFF0000u);
    lb = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){s0, s1}, v2bf));
    const uint32_t t0 = (__builtin_bit_cast(uint32_t, s0) << 1) - 1u, t1 = (__builtin_bit_cast(uint32_t, s1) << 1) - 1u;
    range.least = min(range.least, min(t0, t1));
    range.most = fmaxf(fmaxf(range.most, fabsf(x0)), fabsf(x1));
}

// The filter bank in the order in which general_split_kernel's phases take it to LDS: block
// (filter tile, channel chunk, row group) of [tap][half][part][64 filters] pieces of eight channels,
// zeros for filters beyond K and channels beyond C.  One workgroup per block.  The bank is small
// beside the images (a few MB at most, read once), so this costs a launch of some 3 us and saves
// every workgroup of the main kernel the splitting of its filters in every chunk.
template <int F, int RG>
__global__ void __launch_bounds__(256)
split_filters_kernel(const float* filt, v4u* wsplit, int* wflags, int K, int C, int chunks)
{
    constexpr int MT = 64, S = RG * F, NGR = F / RG, FF = F * F;
    const int block = blockIdx.x;
    const int g = block % NGR, cidx = block / NGR % chunks, kb = block / NGR / chunks;
    SplitRange range;
    // (taps fastest: they lie together in memory)
    for (int e = threadIdx.x; e < S * 2 * MT; e += 256) {
        const int t = e % S, hf = (e / S) & 1, k = e / (2 * S);
        float x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int c = cidx * 16 + hf * 8 + q;
            x[q] = kb * MT + k < K && c < C ? filt[((int64_t)(kb * MT + k) * C + c) * FF + g * S + t] : 0.f;
        }
        v4u part[3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t hb, mb, lb;
            split_pair(x[2 * q], x[2 * q + 1], hb, mb, lb, range);
            part[0][q] = hb;
            part[1][q] = mb;
            part[2][q] = lb;
        }
        v4u* d = wsplit + (int64_t)block * (S * 6 * MT) + (t * 2 + hf) * 3 * MT + k;
#pragma unroll
        for (int q = 0; q < 3; ++q) d[q * MT] = part[q];
    }
    const int flags = __syncthreads_or((range.tiny() ? 1 : 0) | (range.huge() ? 2 : 0));
    if (threadIdx.x == 0) wflags[block] = flags;
}

template <int F, int IR, int RG>
__global__ void __launch_bounds__(512, 2)
general_split_kernel(SplitParams p)
{
    using Gm = SplitGeom<F, IR, RG>;
    constexpr int S = Gm::S, NG = Gm::NG, NP = Gm::NP, THREADS = Gm::THREADS, MT = Gm::MT, NT = Gm::NT, CK = Gm::CK;
    constexpr int NFI = Gm::NFI, FB = Gm::FB;
    constexpr int MOST = Gm::MOST, PS = Gm::PS, IB = Gm::IB;
    constexpr int FF = F * F, MW = 2;
    constexpr uint32_t kNowhere = 0xC0000000u;
    constexpr int kRsrcFlags = 0x00020000;

    extern __shared__ __attribute__((aligned(16))) v4u lds_pieces[];
    v4u* const fslots = lds_pieces;                 // two filter blocks, then two image blocks
    v4u* const islots = lds_pieces + 2 * FB;
    __shared__ int s_old;
    __shared__ int s_tiny[4], s_huge[4];     // by tile & 3: a value below 2^-103 / above 2^40 was staged

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l32 = lane & 31;

    const int LS = p.LS;
    const int G = p.G;
    const int j = (G % 8 == 0) ? (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
    const int nun = p.nun;
    const int U = p.split ? p.tiles * nun : p.tiles;
    const int unit_scale = p.split ? 1 : nun;
    const int u0 = range_start(j, U, G) * unit_scale;
    const int u1 = range_start(j + 1, U, G) * unit_scale;
    if (u0 >= u1) return;                           // uniform: before any barrier

    const int HW = p.H * p.W;
    const int64_t plane = (int64_t)p.Ho * p.Wo;
    const int CFF = p.C * FF;
    const int per_strip = p.pt_full * p.KB;

    if (tid < 4) { s_tiny[tid] = 0; s_huge[tid] = 0; }

    // ---- staging.  Image: thread tid brings pixel tid of the block, eight channels at a time.
    // Loads are range-checked as in general_tiled_kernel: lanes with nothing to bring read zero;
    // channels beyond C read zero by a scalar offset beyond the extent.  Filters: the split
    // block is copied as it lies.
    uint32_t ig;             // byte offset from in[n_first][c0][first row][0]
    const int ipix = tid < p.RS * LS ? tid : -1;
    const int ipos0 = ipix >= 0 ? ipix : 2 * MOST, ipos1 = ipix >= 0 ? MOST + ipix : 2 * MOST;
    const char* ibase = (const char*)p.in;
    int64_t ileft = 0;
    const int64_t in_bytes = (int64_t)p.N * p.C * HW * 4;
    auto setup_fetch = [&](int tile) __attribute__((always_inline)) {
        const int strip = min(fdiv(tile, p.d_strip), p.nstrips - 1);
        const int rem = tile - strip * per_strip;
        const int ptile = fdiv(rem, p.d_kb);
        const int x0 = strip * p.bw;
        const int ws = min(p.bw, p.Wo - x0);
        const bool last_strip = strip == p.nstrips - 1;
        const FastDiv d_ws{last_strip ? p.d_wsl.m : p.d_wsf.m, last_strip ? p.d_wsl.sh : p.d_wsf.sh, ws};
        const int total_p = p.N * p.Ho * ws;
        const int p0 = ptile * NT;
        const int Q0 = fdiv(p0, d_ws);
        const int n_first = fdiv(Q0, p.d_ho);
        const int y_first = Q0 - n_first * p.Ho;
        const int Ql = fdiv(min(p0 + NT, total_p) - 1, d_ws);
        const int nl = fdiv(Ql, p.d_ho);
        const int nslots = (nl - n_first) * p.Hc + (Ql - nl * p.Ho) - y_first + IR;
        const int row = fdiv(tid, p.d_ls), col = tid - row * LS;
        const int dn = fdiv(y_first + row, p.d_hc);
        const int yy = y_first + row - dn * p.Hc;
        const bool there = ipix >= 0 && row < nslots && n_first + dn < p.N && x0 + col < p.W;
        ig = there ? (uint32_t)(dn * p.C * HW + yy * p.W + x0 + col) * 4u : kNowhere;
        const int64_t ifirst = (int64_t)n_first * p.C * HW * 4;
        ibase = (const char*)p.in + ifirst;
        ileft = in_bytes - ifirst;
    };
    float ireg[CK];
    // channels 2i and 2i + 1 of the thread's pixel, unit `unit` of the tile set up
    auto fetch_pair = [&](int i, int unit) __attribute__((always_inline)) {
        const int cidx = unit / NG, c0 = cidx * CK;
        const int64_t off = ((int64_t)c0 * HW + (int64_t)(unit - cidx * NG) * IR * p.W) * 4;
        const int64_t left = max(min(ileft - off, (int64_t)0x7FFFFFFF), (int64_t)0);
        auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)(ibase + off), 0, (int)left, kRsrcFlags);
        int hw4 = HW * 4;
        asm volatile("" : "+s"(hw4));              // (the offsets are formed here and not kept across the loop)
#pragma unroll
        for (int e = 2 * i; e < 2 * i + 2; ++e) {
            const int so = c0 + e < p.C ? e * hw4 : 0x7FFFFFFF;
            ireg[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, ig, so, 0));
        }
    };
    // first filter block of unit v
    const int chunks = nun / NG;
    auto block_of = [&](int v) __attribute__((always_inline)) {
        const int t = fdiv(v, p.d_nun), un = v - t * nun;
        const int strip = min(fdiv(t, p.d_strip), p.nstrips - 1);
        const int rem = t - strip * per_strip;
        const int kb = rem - fdiv(rem, p.d_kb) * p.KB;
        return (kb * chunks * NG + un) * NP;
    };
    const auto wrs = __builtin_amdgcn_make_buffer_rsrc((void*)p.wsplit, 0, p.KB * chunks * NG * NP * FB * 16, kRsrcFlags);
    // straight into LDS, 64 pieces a load: lane l of the wave brings piece l
    typedef __attribute__((address_space(3))) void* lds_ptr;
    auto fetch_filter = [&](int k, int block, v4u* fs) __attribute__((always_inline)) {
        const int g = k * 8 + wave;
        if ((k + 1) * 8 <= FB / 64 || g < FB / 64)                  // uniform
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lds_ptr)(fs + g * 64), 16, lane * 16, block * (FB * 16) + g * 1024, 0, 0);
    };
    SplitRange range;
    // Split a pair of values; after four pairs a half's three pieces go to LDS.
    v4u being[3];
    auto commit_pair = [&](int i, v4u* is) __attribute__((always_inline)) {
        const int q = i % 4;
        uint32_t hb, mb, lb;
        split_pair(ireg[2 * i], ireg[2 * i + 1], hb, mb, lb, range);
        asm volatile("" : "+v"(hb), "+v"(mb), "+v"(lb), "+v"(range.least), "+v"(range.most));      // (here, and not gathered before the write)
        being[0][q] = hb;
        being[1][q] = mb;
        being[2][q] = lb;
        if (q == 3) {
            v4u* d = is + (i < 4 ? ipos0 : ipos1);
            d[0] = being[0];
            d[PS] = being[1];
            d[2 * PS] = being[2];
        }
    };
    // What the values staged so far are like, noted for a tile when it ends and for the next one (whose
    // first image block is staged by then); `wf`: the flags of the tile's filter blocks.
    const auto* flags = (const __attribute__((address_space(4))) int*)p.wflags;      // (scalar loads)
    int wf = 0;
    auto note_range = [&](int t) __attribute__((always_inline)) {
        if (range.tiny()) { s_tiny[t & 3] = 1; s_tiny[(t + 1) & 3] = 1; }
        if (range.huge()) { s_huge[t & 3] = 1; s_huge[(t + 1) & 3] = 1; }
        if (wf & 1) s_tiny[t & 3] = 1;
        if (wf & 2) s_huge[t & 3] = 1;
        range = SplitRange();
        wf = 0;
    };

    // ---- the compute side ----------------------------------------------------------------------
    int base = 0;            // piece (within an image block) of the lane's pixel at tap (0, 0), part 0
    uint32_t oofs = 0;       // byte offset of out[n][k0 + 4*h][y][x] from out[n_first][k0][0][0]
    bool valid = false;
    int kleft = 0;
    int n_first_c = 0, ck0 = 0;
    float* obase_t = p.out;
    auto setup_compute = [&](int tile) __attribute__((always_inline)) {
        const int strip = min(fdiv(tile, p.d_strip), p.nstrips - 1);
        const int rem = tile - strip * per_strip;
        const int ptile = fdiv(rem, p.d_kb), kb = rem - ptile * p.KB;
        const int x0 = strip * p.bw;
        const int ws = min(p.bw, p.Wo - x0);
        const bool last_strip = strip == p.nstrips - 1;
        const FastDiv d_ws{last_strip ? p.d_wsl.m : p.d_wsf.m, last_strip ? p.d_wsl.sh : p.d_wsf.sh, ws};
        const int total_p = p.N * p.Ho * ws;
        const int p0 = ptile * NT;
        const int Q0 = fdiv(p0, d_ws);
        const int n_first = fdiv(Q0, p.d_ho);
        const int y_first = Q0 - n_first * p.Ho;
        ck0 = kb * MT;
        n_first_c = n_first;
        kleft = p.K - ck0 - 4 * h;
        obase_t = p.out + ((int64_t)n_first * p.K + ck0) * plane;
        const uint32_t kplane = (uint32_t)p.K * (uint32_t)plane;
        const int pp = p0 + wave * 32 + l32;
        valid = pp < total_p;
        const int pc = valid ? pp : total_p - 1;
        const int Q = fdiv(pc, d_ws), xl = pc - Q * ws;
        const int n = fdiv(Q, p.d_ho), y = Q - n * p.Ho;
        base = h * MOST + ((n - n_first) * p.Hc + y - y_first) * LS + xl;
        oofs = ((uint32_t)(n - n_first) * kplane + (uint32_t)(4 * h * (int)plane + y * p.Wo + x0 + xl)) * 4u;
    };
    const int wb = h * 3 * MT + l32;
    // part q of the operands of step s of a phase whose first filter row within the unit is i0
    auto load_a = [&](int q, int s, const v4u* fs, v4u (&a)[MW][3]) __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MW; ++mt) a[mt][q] = fs[wb + s * 6 * MT + q * MT + mt * 32];
    };
    auto load_b = [&](int q, int s, int i0, const v4u* is, v4u (&b)[3]) __attribute__((always_inline)) {
        b[q] = is[base + q * PS + (i0 + s / F) * LS + s % F];
    };
    auto mfma = [](v4u a, v4u b, v16f c) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    };

    // sums of the current unit (products of leading parts; all others), and the total
    v16f hi[MW], lo[MW], acc[MW];
    auto zero = [&](v16f (&v)[MW]) __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MW; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) v[mt][r] = 0.f;
    };

    auto add_unit = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MW; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mt][r] += hi[mt][r] + lo[mt][r];
    };

    // Tiles with outputs to be formed again, noted per wave for the pass behind the main loop: one bit for the
    // workgroup's first tile, one for its last (which another workgroup may have to write), the others
    // share 62.
    const int tfirst = fdiv(u0, p.d_nun), tlast = fdiv(u1 - 1, p.d_nun);
    uint64_t redo = 0;
    int redo_kind = 0;
    auto redo_bit = [&](int t) __attribute__((always_inline)) {
        return 1ull << (t == tfirst ? 0 : t == tlast ? 1 : 2 + (t - tfirst) % 62);
    };
    // kind of tile: 0 no tiny values, 1 tiny ones, 2 tiny and huge ones; finite outputs below
    // redo_below(kind) are formed again
    auto redo_below = [](int kind) __attribute__((always_inline)) { return kind == 0 ? -1.f : kind == 1 ? 0x1p-60f : __builtin_inff(); };
    auto emit = [&](int t, bool any_tiny, bool any_huge) __attribute__((always_inline)) {
        const int kind = any_tiny ? (any_huge ? 2 : 1) : 0;
        const float least = redo_below(kind);
        bool again = false;
#pragma unroll
        for (int mt = 0; mt < MW; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kk = mt * 32 + mfma_row(r, 0);
                char* ob = (char*)(obase_t + kk * plane);
                const float v = acc[mt][r];
                again |= !(fabsf(v) < __builtin_inff()) | (fabsf(v) < least);
                if (valid && kk < kleft) *reinterpret_cast<float*>(ob + oofs) = v;
            }
        if (__any(again && valid)) {
            redo |= redo_bit(t);
            redo_kind = max(redo_kind, kind);
        }
    };
    auto part_ptr = [&](int wgi, int which) __attribute__((always_inline)) {
        char* b = (char*)(p.part + ((int64_t)(2 * wgi + which)) * (MT * NT) + wave * (MW * 16 * kWave));
        return reinterpret_cast<float*>(b + (uint32_t)lane * 4u);
    };
    // (see general_tiled_kernel; an arrival also carries what the workgroup staged: arrivals in
    // the low ten bits, then those with tiny and with huge values)
    auto finish_tile = [&](int tile, bool whole) __attribute__((always_inline)) {
        const bool any_tiny = s_tiny[tile & 3] != 0, any_huge = s_huge[tile & 3] != 0;
        if (tid == 0) { s_tiny[(tile + 3) & 3] = 0; s_huge[(tile + 3) & 3] = 0; }
        if (whole) { emit(tile, any_tiny, any_huge); return; }
        const int t0u = tile * nun;
        const int first = unit_owner(t0u, U, G), last = unit_owner(t0u + nun - 1, U, G);
        const int m = last - first + 1;
        float* mine = part_ptr(j, u0 >= t0u ? 0 : 1);
#pragma unroll
        for (int mt = 0; mt < MW; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                __hip_atomic_store(mine + (mt * 16 + r) * kWave, acc[mt][r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0x0F70);        // every wave's stores are performed before the arrival counts
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __syncthreads();
        const int arrival = 1 + (any_tiny ? 1 << 10 : 0) + (any_huge ? 1 << 20 : 0);
        if (tid == 0)
            s_old = __hip_atomic_fetch_add(&p.cnt[first], arrival, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + arrival;
        __syncthreads();
        const int now = s_old;
        if ((now & 1023) != m) return;
        if (tid == 0) __hip_atomic_store(&p.cnt[first], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (m > 2) zero(acc);
        for (int i = first; i <= last; ++i) {
            if (m == 2 && i == j) continue;
            const float* src = part_ptr(i, range_start(i, U, G) >= t0u ? 0 : 1);
#pragma unroll
            for (int mt = 0; mt < MW; ++mt) {
                float v[16];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    v[r] = __hip_atomic_load(src + (mt * 16 + r) * kWave, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mt][r] += v[r];
            }
        }
        emit(tile, ((now >> 10) & 1023) != 0, (now >> 20) != 0);
    };

    // ---- prologue: the first unit's image block and first filter block go to LDS, the next ones
    // into registers
    int tile = fdiv(u0, p.d_nun), unit = u0 - tile * nun;       // the unit being consumed
    int ftile = tile, funit = unit;                             // the unit whose image block is requested
    auto advance_fetch = [&]() __attribute__((always_inline)) {
        if (++funit == nun) { funit = 0; ++ftile; setup_fetch(ftile); }
    };
    setup_fetch(ftile);
    // first filter blocks of the unit being consumed and of the next one
    int b_of[2] = {block_of(u0), block_of(min(u0 + 1, u1 - 1))};
#pragma unroll
    for (int i = 0; i < 8; ++i) fetch_pair(i, funit);
#pragma unroll
    for (int k = 0; k < NFI; ++k) fetch_filter(k, b_of[0], fslots);
    bool from_first = unit == 0;
    setup_compute(tile);
    zero(acc);
#pragma unroll
    for (int i = 0; i < 8; ++i) commit_pair(i, islots);
    __builtin_amdgcn_s_waitcnt(0x0F70);                         // vmcnt(0): this wave's filter pieces are in LDS
    if (u0 + 1 < u1) advance_fetch();
#pragma unroll
    for (int i = 0; i < 8; ++i) fetch_pair(i, funit);
    __syncthreads();
    v4u a[MW][3], b[3];

    // ---- main loop: one (tile, unit) per trip ----------------------------------------------------
    // The workgroup's two halves (waves 0-3 and 4-7, one wave of each per SIMD) take turns.  A step
    // has two parts, each ended by a barrier: bringing its operands from LDS, with a share of the
    // staging and of the unit's vector arithmetic, and its twelve matrix-core instructions.  The
    // second half runs one part behind the first (`fork`, until `join`), so that a SIMD's matrix
    // cores work for one wave while the other wave issues everything else.  Every part waits for
    // its LDS accesses before its barrier, so a block written during the parts of phase P is
    // complete, and the block it replaces is no longer read, when phase P + 1 begins.
    const bool second = wave >= 4;
    auto meet = []() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int T = NP * S;                                   // steps of a unit
    // the step at which pair i of the next unit's image block is split and the pair of the unit
    // after it requested; loads issued in phase ph between its filter block and its last step
    auto pair_step = [](int i) constexpr { return 1 + i * (T - 1) / 8; };
    auto later_loads = [&](int ph) constexpr {
        int n = 0;
        for (int i = 0; i < 8; ++i) n += pair_step(i) / S == ph && pair_step(i) % S < S - 1 ? 2 : 0;
        return n;
    };
    // (that count holds in the order written: the compiler moves no load across this)
    auto in_order = []() __attribute__((always_inline)) { asm volatile("" ::: "memory"); };
    auto wait_filter = [](int later) __attribute__((always_inline)) {      // vmcnt(later), other counters left alone
        switch (later) {
        case 0: __builtin_amdgcn_s_waitcnt(0x0F70); break;
        case 2: __builtin_amdgcn_s_waitcnt(0x0F72); break;
        case 4: __builtin_amdgcn_s_waitcnt(0x0F74); break;
        case 6: __builtin_amdgcn_s_waitcnt(0x0F76); break;
        case 8: __builtin_amdgcn_s_waitcnt(0x0F78); break;
        case 10: __builtin_amdgcn_s_waitcnt(0x0F7A); break;
        case 12: __builtin_amdgcn_s_waitcnt(0x0F7C); break;
        case 14: __builtin_amdgcn_s_waitcnt(0x0F7E); break;
        default: __builtin_amdgcn_s_waitcnt(0x0F70); break;
        }
    };
    int fpar = 0, ipar = 0;                 // slots of the filter block and image block being consumed
    bool pending = false;                   // the previous unit's sums have not joined the total yet
    if (second) meet();
    for (int u = u0; u < u1; ++u) {
        const bool has1 = u + 1 < u1;
        const bool tile_ends = unit == nun - 1 || !has1;
        if (u + 2 < u1) advance_fetch();
        const v4u* is = islots + ipar * IB;
        v4u* inext = islots + (ipar ^ 1) * IB;
#pragma unroll
        for (int ph = 0; ph < NP; ++ph) {
            const v4u* fs = fslots + fpar * FB;
            v4u* fnext = fslots + (fpar ^ 1) * FB;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int t = ph * S + s;
#pragma unroll
                for (int q = 0; q < 3; ++q) { load_b(q, s, ph * RG, is, b); load_a(q, s, fs, a); }
                __builtin_amdgcn_sched_barrier(0);              // the operands first
                // the next phase's filter block is requested as the phase begins and has landed by
                // its last step; later loads (of the image block) may still be on their way
                if (s == 0) {
                    wf |= flags[b_of[0] + ph];
#pragma unroll
                    for (int k = 0; k < NFI; ++k) fetch_filter(k, b_of[(ph + 1) / NP] + (ph + 1) % NP, fnext);
                    in_order();
                }
                if (s == S - 1) {
                    in_order();
                    wait_filter(later_loads(ph));
                    in_order();
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (pair_step(i) == t) {
                        commit_pair(i, inext);
                        fetch_pair(i, funit);
                    }
                if (t == 0) {
                    if (pending) add_unit();
                    pending = true;
                }
                meet();
                const bool fresh = t == 0;                      // the unit's first products: sums from zero
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) lo[mt] = mfma(a[mt][0], b[2], fresh ? (v16f){} : lo[mt]);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) lo[mt] = mfma(a[mt][2], b[0], lo[mt]);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) lo[mt] = mfma(a[mt][1], b[1], lo[mt]);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) lo[mt] = mfma(a[mt][0], b[1], lo[mt]);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) lo[mt] = mfma(a[mt][1], b[0], lo[mt]);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) hi[mt] = mfma(a[mt][0], b[0], fresh ? (v16f){} : hi[mt]);
                __builtin_amdgcn_s_setprio(0);
                meet();
            }
            fpar ^= 1;
        }
        ipar ^= 1;
        b_of[0] = b_of[1];
        b_of[1] = block_of(min(u + 2, u1 - 1));
        if (tile_ends) {
            if (!second) meet();
            add_unit();
            pending = false;
            note_range(tile);
            __syncthreads();
            finish_tile(tile, from_first && unit == nun - 1);
            if (has1) {
                ++tile; unit = 0; from_first = true;
                setup_compute(tile);
                zero(acc);
                if (second) meet();
            }
        } else {
            ++unit;
        }
    }

    // ---- outputs that the split cannot form: a wave's blocks again, in fp32 (nothing else is
    // kept in registers here, as it would be if the main loop called this)
    if (redo == 0) return;
    __builtin_amdgcn_s_waitcnt(0x0F70);                         // this wave's outputs are in memory
    const float least = redo_below(redo_kind);
    for (int t = tfirst; t <= tlast; ++t) {
        if ((redo & redo_bit(t)) == 0) continue;                // uniform
        setup_compute(t);
        uint32_t which = 0;
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            const int kk = (r >> 4) * 32 + mfma_row(r & 15, 0);
            if (valid && kk < kleft) {
                const float v = __hip_atomic_load(reinterpret_cast<float*>((char*)(obase_t + kk * plane) + oofs), __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
                if (!(fabsf(v) < __builtin_inff()) | (fabsf(v) < least)) which |= 1u << r;
            }
        }
        if (!__any(which != 0)) continue;
        const uint32_t o0 = oofs / 4u - (uint32_t)(4 * h) * (uint32_t)plane;     // (n - n_first, 0, y, x)
        const int dn = (int)((int64_t)o0 / ((int64_t)p.K * plane));
        const int yx = (int)((int64_t)o0 - (int64_t)dn * p.K * plane);
        const int y = yx / p.Wo, x = yx - y * p.Wo;
        const int64_t ifirst = (int64_t)n_first_c * p.C * HW * 4;
        redo_block<F>((const char*)p.in + ifirst, in_bytes - ifirst, (uint32_t)(dn * p.C * HW + y * p.W + x) * 4u,
                      p.filt + (int64_t)ck0 * CFF, (p.K - ck0) * CFF * 4, (char*)obase_t + oofs, which, p.C, p.W, HW, plane);
    }
}

// ---- host side -----------------------------------------------------------------------------------

struct SplitPlan {
    int bw, nstrips, LS, RS, pt_full, pt_last;
    bool ok;
};

// The widest column strips (at most 128 columns) whose image block of rg filter rows the workgroup
// can stage and hold: `most` pixels.
inline SplitPlan make_split_plan(const Shape& s, int rg, int NT, int most)
{
    SplitPlan pl{};
    for (int nstrips = (s.Wo + 127) / 128; nstrips <= s.Wo; ++nstrips) {
        pl.bw = (s.Wo + nstrips - 1) / nstrips;
        pl.nstrips = (s.Wo + pl.bw - 1) / pl.bw;
        pl.LS = pl.bw + s.F - 1;
        const int wmin = s.Wo - (pl.nstrips - 1) * pl.bw;
        const int64_t all_rows = (int64_t)s.N * s.Ho;
        const int rows = (int)std::min<int64_t>((NT - 2) / wmin + 2, all_rows);
        const int cross = std::min(rows >= 2 ? (rows - 2) / s.Ho + 1 : 0, s.N - 1);
        pl.RS = rows + (rg - 1) * (cross + 1);
        pl.pt_full = (int)(((int64_t)s.N * s.Ho * pl.bw + NT - 1) / NT);
        pl.pt_last = (int)(((int64_t)s.N * s.Ho * wmin + NT - 1) / NT);
        if ((int64_t)pl.RS * pl.LS <= most) { pl.ok = true; return pl; }
    }
    pl.ok = false;
    return pl;
}

template <int F, int IR, int RG>
int split_try_launch(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st,
                     const GenSched& sched)
{
    using Gm = SplitGeom<F, IR, RG>;
    constexpr int MT = Gm::MT, NT = Gm::NT, THREADS = Gm::THREADS;
    const SplitPlan pl = make_split_plan(s, IR, NT, Gm::MOST);
    if (!pl.ok) return DCONV_UNSUPPORTED;
    const int64_t lds_bytes = 2LL * 16 * (Gm::FB + Gm::IB);
    const int KB = (s.K + MT - 1) / MT;
    const int nun = (s.C + Gm::CK - 1) / Gm::CK * Gm::NG;
    const int64_t tiles = ((int64_t)(pl.nstrips - 1) * pl.pt_full + pl.pt_last) * KB;
    if (tiles * nun > 2147483647LL || (int64_t)s.N * s.Ho * s.Wo > 2147483647LL) return DCONV_UNSUPPORTED;
    // Lanes address HBM with 32-bit byte offsets from per-tile bases (the tile's first image and
    // the unit's first channel; its first filter): what a lane adds must stay below 2 GiB.
    {
        const int wmin = s.Wo - (pl.nstrips - 1) * pl.bw;
        const int64_t span = std::min<int64_t>(NT / ((int64_t)s.Ho * wmin) + 2, s.N);
        const int64_t plane = (int64_t)s.Ho * s.Wo;
        const int64_t lim = 1LL << 29;                                // floats: 2 GiB
        if (((span - 1) * s.C + Gm::CK + 1) * s.H * s.W >= lim || (span - 1) * s.K * plane + 6 * plane >= lim)
            return DCONV_UNSUPPORTED;
    }
    const int cus = gen_cus();
    if (cus <= 0) return DCONV_LAUNCH_FAILED;
    const int split = sched.mode == 2 ? 1 : 0;
    const int64_t U = split ? tiles * nun : tiles;
    int G = sched.force_G > 0 ? sched.force_G : cus;
    if (G > U) G = (int)U;

    // the split filter bank, one flag word per block, partial tiles: in what the workspace has for
    // partial tiles alone, so that no call needs a larger one than before
    const int chunks = (s.C + Gm::CK - 1) / Gm::CK;
    const int64_t blocks = (int64_t)KB * chunks * (F / RG);
    const int64_t bank_floats = blocks * Gm::FB * 4, flag_floats = (blocks + 3) / 4 * 4;
    const int64_t part_floats = split ? (int64_t)G * 2 * MT * NT : 0;
    const size_t floats = (size_t)(bank_floats + flag_floats + part_floats);
    if (floats > kGenWorkspaceFloats) return DCONV_UNSUPPORTED;
    auto kern = general_split_kernel<F, IR, RG>;
    static std::atomic<uint64_t> lds_limit_raised{0};
    if (!raise_lds_limit((const void*)kern, kGenLdsLimit, lds_limit_raised)) return DCONV_LAUNCH_FAILED;
    GenWorkspace ws;
    if (sched.static_ws) {
        if (gen_static_workspace(st, floats, split ? (size_t)G : 0, &ws) != DCONV_OK) return DCONV_UNSUPPORTED;
    } else {
        ws = gen_workspace(st, floats, split ? (size_t)G : 0);
        if (!ws.part || (split && !ws.cnt)) return DCONV_UNSUPPORTED;
    }
    v4u* bank = (v4u*)ws.part;
    int* flags = (int*)(ws.part + bank_floats);
    float* part = ws.part + bank_floats + flag_floats;
    begin_launch();
    hipLaunchKernelGGL((split_filters_kernel<F, RG>), dim3((unsigned)blocks), dim3(256), 0, st, filt, bank, flags, s.K, s.C,
                       chunks);
    if (const int rc = launch_status(); rc != DCONV_OK) return rc;
    SplitParams p{in, filt, out, bank, flags, part, ws.cnt, s.N, s.C, s.H, s.W, s.K, s.Ho, s.Wo,
                  pl.bw, pl.nstrips, pl.LS, pl.RS, pl.pt_full, KB, nun, (int)tiles, G, split, s.Ho + IR - 1,
                  make_fastdiv(pl.pt_full * KB), make_fastdiv(KB), make_fastdiv(pl.bw),
                  make_fastdiv(s.Wo - (pl.nstrips - 1) * pl.bw), make_fastdiv(s.Ho), make_fastdiv(s.Ho + IR - 1),
                  make_fastdiv(pl.LS), make_fastdiv(nun)};
    begin_launch();
    hipLaunchKernelGGL(kern, dim3((unsigned)G), dim3(THREADS), (size_t)lds_bytes, st, p);
    return launch_status();
}

// Implemented once per filter side, each in its own translation unit.
template <int F>
int split_launch_for_F(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st,
                       const GenSched& sched);

}  // namespace dconv
