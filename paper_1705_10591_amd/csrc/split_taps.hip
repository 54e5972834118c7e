// fp32 direct convolution of FEW CHANNELS on the bf16 matrix cores of gfx950: one large image, or the first
// layer of a network.
//
// v_mfma_f32_16x16x32_bf16 runs at sixteen times the rate of the fp32 instructions.  As in split_kernel.h a value is
// the exact sum of three bf16 parts, and of the nine products of parts the six largest are formed: what is left out,
// m l' + l m' + l l', is 2^-24 |x w| at most.  Products of parts are exact; h h' and the five small ones are summed
// apart, in fp32, until the end.  Whole numbers whose sums the fp32 instructions form exactly come out the same.
// Against 64 bits a sum of 81 random products is off by 0.51e-7 of its norm (1.63e-7), one of 363 by 0.98e-7 (3.3e-7), one of
// 25 by 0.35e-7 (0.91e-7): in brackets the fp32 instructions, which round after every two products, these after eight.
// Filters of 2, 3, 6 and 12 weights among zeros: 0.26e-7, 0.26e-7, 0.27e-7, 0.30e-7 (0.31e-7, 0.35e-7, 0.48e-7, 0.65e-7); the
// furthest single sum of two terms 2.3 times 2^-24 of its terms' magnitudes (1.9).
// (Two fp16 parts under a scale and three products hold 23 of a value's 24 bits and were 485 and 112 us in the cases
// below: products of two whole numbers of 12 bits came out wrong in the last digit.)
// What parts cannot give is formed again:
//  * sums that are not finite (infinities and NaN make NaN of the parts), and, where an operand has values below 2^-103,
//    whose last part may fall below the smallest bf16, sums below 2^-60 (all of them beside values above 2^40):
//    the wave's 64 pixels, behind the main loop, on the fp32 matrix cores;
//  * filters of one weight give their pixels rounded once: read again as the tile ends.
// Measured, on layers of 81 to 363 taps: all outputs formed again 1.6 to 2.0 times the fp32 kernel's time (6.3 with the
// operands of an instruction loaded one by one), and 1.02 to 1.15 times this kernel's for one NaN pixel, 1.8 to 2.0 for one
// filter with values near 2^-110 beside others (its sixteen filters only are formed again), 1.0 to 1.25 for a bank of
// filters of one weight, 1.0 for filters of two or twelve.
//
// split_kernel.h reduces over sixteen channels of one tap at a time, which few channels cannot fill; here
// the reduction runs over TAPS: an instruction takes 32 of them, in whatever order a table gives, so that the
// kernel is one for all filter sides and channel counts.
//  * The image block of a tile is staged once for all its taps: per part, dword x of a row holds the
//    pair (pixel x, pixel x + 1), so that the two taps (i, j), (i, j + 1) of an output pixel are one
//    aligned LDS read whatever the parity of x + j.  Rows are ordered [image row][channel]: tap row
//    r = i * C + c of any pixel lies r rows below its first one.
//  * A step's sixteen pairs are four per group of sixteen lanes.  Lane groups next to each other take
//    pairs of two rows next to each other where they can: with a row stride of 16 (mod 32) dwords
//    their reads share no bank.  A filter side that is odd leaves one column per row to a zero weight.
//  * Pixels are the rows of an instruction's result and filters its columns: a lane ends with four
//    pixels of a row next to each other, which leave in one 16-byte store.
//  * Tile: 256 pixels (numbered along (image, y, x) of a column strip) x up to 64 filters, a wave 64
//    pixels of it with all filters; filters come in blocks of sixteen, so 40 filters are 48 columns.
//    Two workgroups per CU: one computes while the other stages or stores.
//  * Filters: split once per workgroup into LDS where all of a block's fit, else by a small kernel in front
//    into the workspace, from where a ring of three steps runs ahead in LDS.
//
// Measured: 64 x 3 x 224 x 224, 64 11x11 filters 1133 -> 737 us = 185 TFLOP/s (120 on the fp32 instructions; 530 would be
// the six products at the rate of a bare loop of these instructions); one image of 1081 x 1917, 40 9x9 filters 224 -> 127 us.
// Beside the arithmetic both are bound by their stores: 750 and 328 MB in pieces of 64 bytes that share lines with other
// tiles; whole lines through LDS were no faster up to 1 GB, and the order of tiles below was worth 5 to 10 % there.
#include <algorithm>
#include <cmath>
#include "split_kernel.h"

namespace dconv {

namespace {

constexpr int kTapsNT = 256;                    // pixels of a tile
// bytes of an image block's part in LDS (no multiple of 256: reads of two parts do not pair up, which would
// leave the operands' words in the wrong registers): the smaller size, and what the LDS has room for beside a ring
// of three steps of the filters
constexpr int kTapsPartSmall = 11600;
constexpr int taps_part_large(int MB) { return MB == 4 ? 14384 : MB == 3 ? 17424 : 19888; }
constexpr int kTapsLds = 81920;                 // half of a CU's
constexpr int kTapsSteps = 16;                  // 512 taps, which the line for tiny values counts on
constexpr int kTapsStatic = 1024;               // set aside for the kernel's static LDS

// The smallest magnitude that is not zero, among values: their bits, doubled, less one.
__device__ __forceinline__ uint32_t taps_least(uint32_t least, float x) { return min(least, (__builtin_bit_cast(uint32_t, x) << 1) - 1u); }
// ... is it below 2^-103, so that a value's last part may fall below the smallest bf16?
__device__ __forceinline__ bool taps_tiny(uint32_t least) { return least < (uint32_t)(2 * (127 - 103)) * 0x800000u - 1u; }
constexpr float kTapsHuge = 0x1p40f;

struct TapsParams {
    const float* in;
    const float* filt;
    float* out;
    const v4u* bank;     // ring: the split filters, [filter block][step][part][16 filters][lane]
    const int* notes;    // ring: what is noted of each filter
    int N, C, H, W, K, F, Ho, Wo;
    int bw, nstrips, LS, ptiles, tiles, tpg, grows;     // tpg: tiles per strip of a group of `grows` rows
    int P, RC, nc, steps;        // pairs per tap row, pairs of rows, couples of pairs, steps
    FastDiv d_strips, d_pt, d_tpg, d_bw, d_ho, d_q, d_c, d_h, d_p, d_f, d_ff;
};

// Couple u of a step's lane groups 2 * hf, 2 * hf + 1 -> tap row and first column of group parity b; -1: none.
// Couples of two rows come first, then the pairs of an odd last row, two a couple.
__device__ __forceinline__ int taps_pair(const TapsParams& p, int u, int b, int* j)
{
    const int rho = fdiv(u, p.d_p), whole = p.RC * p.P;
    if (u < whole) {
        *j = 2 * (u - rho * p.P);
        return 2 * rho + b;
    }
    const int v = 2 * (u - whole) + b;
    *j = 2 * v;
    return (p.C * p.F & 1) && v < p.P ? p.C * p.F - 1 : -1;
}

// The 32 taps of step s for lane group g of a filter whose weights are at w: their parts.
__device__ __forceinline__ void taps_filter_piece(const TapsParams& p, const float* w, bool there, int s, int g, v4u (&part)[3])
{
    float x[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int j;
        const int r = taps_pair(p, s * 8 + (g >> 1) * 4 + q, g & 1, &j);
        const int i = fdiv(max(r, 0), p.d_c), c = r - i * p.C;
        const int at = (c * p.F + i) * p.F + j;
        x[2 * q] = there && r >= 0 ? w[at] : 0.f;
        x[2 * q + 1] = there && r >= 0 && j + 1 < p.F ? w[at + 1] : 0.f;
    }
    SplitRange range;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t h, m, l;
        split_pair(x[2 * q], x[2 * q + 1], h, m, l, range);
        part[0][q] = h;
        part[1][q] = m;
        part[2][q] = l;
    }
}

// What is noted of a filter: it has tiny values, one weight that is not zero (whose tap stands from kNoteTap on), huge
// values.
constexpr int kNoteTiny = 1, kNoteOne = 2, kNoteHuge = 4, kNoteTap = 3;
// The note of the filter whose T weights are at w; PER threads next to
// each other (a power of two), each with its number `at` among them, work on a filter.
template <int PER>
__device__ __forceinline__ int taps_filter_note(const float* w, int T, int at)
{
    float most = 0.f;
    uint32_t least = 0xFFFFFFFFu;
    int count = 0, tap = 0;
#pragma unroll 4
    for (int t = at; t < T; t += PER) {
        most = fmaxf(most, fabsf(w[t]));
        least = taps_least(least, w[t]);
        count += w[t] != 0.f;
        tap = w[t] != 0.f ? t : tap;
    }
#pragma unroll
    for (int d = 1; d < PER; d *= 2) {
        most = fmaxf(most, __shfl_xor(most, d));
        least = min(least, (uint32_t)__shfl_xor((int)least, d));
        count += __shfl_xor(count, d);
        tap = max(tap, __shfl_xor(tap, d));
    }
    return (taps_tiny(least) ? kNoteTiny : 0) | (count == 1 ? kNoteOne | tap << kNoteTap : 0) | (most > kTapsHuge ? kNoteHuge : 0);
}

// A workgroup per sixteen filters and four steps: a piece a thread.
template <int MB>
__global__ void __launch_bounds__(256)
taps_bank_kernel(TapsParams p, v4u* bank, int* notes)
{
    const int groups = (p.steps + 3) / 4, km = blockIdx.x / groups, s0 = blockIdx.x % groups * 4;
    const int T = p.C * p.F * p.F, tid = threadIdx.x;
    if (s0 == 0) {                                      // uniform
        const int k = km * 16 + (tid >> 4);
        const int note = taps_filter_note<16>(p.filt + (int64_t)min(k, p.K - 1) * T, k < p.K ? T : 0, tid & 15);
        if ((tid & 15) == 0) notes[k] = note;
    }
    const int s = s0 + (tid >> 6), l = tid & 63, k = km * 16 + (l & 15), kb = km / MB, m = km % MB;
    if (s >= p.steps) return;
    v4u part[3];
    taps_filter_piece(p, p.filt + (int64_t)min(k, p.K - 1) * T, k < p.K, s, l >> 4, part);
    v4u* d = bank + ((int64_t)(kb * p.steps + s) * 3 * MB + m) * 64 + l;
#pragma unroll
    for (int q = 0; q < 3; ++q) d[q * MB * 64] = part[q];
}

template <int MB, bool RES, int PSB>
__global__ void __launch_bounds__(256, 2)
split_taps_kernel(TapsParams p)
{
    constexpr int NT = kTapsNT, NB = 4;
    constexpr int NQ = (PSB / 16 + 255) / 256;          // quads of image dwords a thread stages
    constexpr int SLOT = 3 * MB * 64;                   // 16-byte pieces of a step's filters
    constexpr uint32_t kNowhere = 0xC0000000u;
    constexpr int kRsrcFlags = 0x00020000;

    extern __shared__ __attribute__((aligned(16))) v4u lds_pieces[];
    char* const img = (char*)lds_pieces;
    v4u* const fl = lds_pieces + 3 * PSB / 16;          // filters: all steps, or a ring of three
    v4u* const table = fl + (RES ? p.steps : 3) * SLOT; // [step][lane group]: byte offsets of its four pairs
    __shared__ int s_range[2];                          // by tile parity: whether the image block has tiny, huge values
    __shared__ int s_notes[MB * 16];                    // of the filter block

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, l16 = lane & 15;
    // Each XCD has a range of tiles and its workgroups take them in turn: tiles next to each other are written
    // at about the same time, and the lines that they share leave that XCD's L2 whole.
    const int G = gridDim.x, nx = G % 8 == 0 ? 8 : 1;
    const int t0 = range_start(blockIdx.x % nx, p.tiles, nx) + (int)(blockIdx.x / nx), t1 = range_start(blockIdx.x % nx + 1, p.tiles, nx), dt = G / nx;
    if (t0 >= t1) return;                               // uniform: before any barrier

    const int HW = p.H * p.W;
    const int64_t plane = (int64_t)p.Ho * p.Wo;
    const int64_t in_bytes = (int64_t)p.N * p.C * HW * 4;

    if (tid < 2) s_range[tid] = 0;
    for (int e = tid; e < p.steps * 16; e += 256) {
        int j;
        const int r = taps_pair(p, (e >> 4) * 8 + ((e >> 3) & 1) * 4 + (e & 3), (e >> 2) & 1, &j);
        ((uint32_t*)table)[e] = r >= 0 ? (uint32_t)(r * p.LS + j) * 4u : 0u;
    }

    // a tile's place: strip, pixels, first and last row
    struct Place { int kb, x0, ws, p0, n_base, n_first, y_first, nslots; };
    const int total = p.grows * p.bw;                   // numbered pixels of a group's strip
    auto place = [&](int tile) __attribute__((always_inline)) {
        Place t;
        t.kb = fdiv(tile, p.d_pt);
        const int pt = tile - t.kb * p.ptiles;
        const int down = fdiv(pt, p.d_strips);          // tiles next to each other in a row follow each other
        t.x0 = (pt - down * p.nstrips) * p.bw;
        t.ws = min(p.bw, p.Wo - t.x0);
        t.n_base = fdiv(down, p.d_tpg);
        t.p0 = (down - t.n_base * p.tpg) * NT;
        const int Q0 = fdiv(t.p0, p.d_bw);
        const int im = fdiv(Q0, p.d_ho);
        t.n_first = t.n_base + im;
        t.y_first = Q0 - im * p.Ho;
        const int Ql = fdiv(min(t.p0 + NT, total) - 1, p.d_bw);
        const int nl = fdiv(Ql, p.d_ho);
        t.nslots = (nl - im) * p.H + (Ql - nl * p.Ho) - t.y_first + p.F;
        return t;
    };
    // pixel pp of a tile's strip: column, row, image past the tile's first one
    auto pixel = [&](const Place& t, int pp, int* x, int* y) __attribute__((always_inline)) {
        const int Q = fdiv(pp, p.d_bw);
        *x = pp - Q * p.bw;
        const int im = fdiv(Q, p.d_ho);
        *y = Q - im * p.Ho;
        return t.n_base + im - t.n_first;
    };

    // ---- image staging: a thread brings quads of dwords, five values each.  Reads past the tensor's
    // end give zero, those past a row's end whatever follows: only unused dwords hold it, or zero
    // weights meet it (should it be infinite, the outputs are formed again).
    v4f ra[NQ];
    float rb[NQ];
    uint32_t pre[NQ];                                   // byte offset of the quad from the tile's first image, row and column
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int e = tid + i * 256;
        const int row = fdiv(e, p.d_q), col = 4 * e - row * p.LS;
        const int slot = fdiv(row, p.d_c), c = row - slot * p.C;
        pre[i] = (uint32_t)((c * p.H + slot) * p.W + col) * 4u;
    }
    auto fetch = [&](const Place& t) __attribute__((always_inline)) {
        const int64_t ifirst = (int64_t)t.n_first * p.C * HW * 4;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.in + ifirst), 0,
                                                         (int)min(in_bytes - ifirst, (int64_t)0x7FFFFFFF), kRsrcFlags);
        const int quads = t.nslots * p.C * p.LS >> 2;
        const int so = (t.y_first * p.W + t.x0) * 4;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            if (i * 256 >= quads) continue;             // uniform
            uint32_t o = pre[i] + (uint32_t)so;
            if (p.C > 1 && t.y_first + t.nslots > p.H) {         // uniform: rows of further images, C images apart
                const int slot = fdiv(fdiv(tid + i * 256, p.d_q), p.d_c);
                o += (uint32_t)(fdiv(t.y_first + slot, p.d_h) * (p.C - 1) * HW) * 4u;
            }
            ra[i] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0));
            rb[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, o + 16u, 0, 0));
        }
    };
    auto commit = [&](const Place& t, int par) __attribute__((always_inline)) {
        const int quads = t.nslots * p.C * p.LS >> 2;
        uint32_t least = 0xFFFFFFFFu;
        float most = 0.f;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            if (i * 256 >= quads) continue;             // uniform
            const float x[6] = {ra[i][0], ra[i][1], ra[i][2], ra[i][3], rb[i], 0.f};
            uint32_t part[3][3];
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                least = taps_least(least, x[q]);
                most = fmaxf(most, fabsf(x[q]));
            }
            SplitRange range;
#pragma unroll
            for (int q = 0; q < 3; ++q) split_pair(x[2 * q], x[2 * q + 1], part[0][q], part[1][q], part[2][q], range);
            const int e = tid + i * 256;
            if (e < PSB / 16) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const uint32_t (&w)[3] = part[k];
                    *(v4u*)(img + k * PSB + e * 16) = v4u{w[0], __builtin_amdgcn_alignbit(w[1], w[0], 16), w[1], __builtin_amdgcn_alignbit(w[2], w[1], 16)};
                }
            }
        }
        const int range = (taps_tiny(least) ? kNoteTiny : 0) | (most > kTapsHuge ? kNoteHuge : 0);
        if (range) atomicOr(&s_range[par], range);
    };

    // ---- filters
    // By the whole workgroup, and complete behind the next barrier.  RES: the weights of as many filters as the
    // image block's place holds are brought there, split from there.
    auto load_filters = [&](int kb) {
        if constexpr (!RES) {
            if (tid < MB * 16) s_notes[tid] = p.notes[kb * MB * 16 + tid];
        } else {
            const int T = p.C * p.F * p.F;
            float* const raw = (float*)img;
            const int mg = min(MB, 3 * PSB / 4 / (16 * T));                 // blocks of sixteen at a time (the plan sees to one or more)
            for (int m0 = 0; m0 < MB; m0 += mg) {
                const int k0 = (kb * MB + m0) * 16, nf = min(mg, MB - m0) * 16;
                const int words = min(nf, p.K - k0) * T;                    // (none beyond K)
                if (m0 > 0) __syncthreads();
#pragma unroll 8
                for (int e = tid; e < words; e += 256) raw[e] = p.filt[(int64_t)k0 * T + e];
                __syncthreads();
                if (tid < nf * 4) {
                    const int f = tid >> 2;
                    const int note = taps_filter_note<4>(raw + f * T, k0 + f < p.K ? T : 0, tid & 3);
                    if ((tid & 3) == 0) s_notes[m0 * 16 + f] = note;
                }
                for (int e = tid; e < p.steps * nf * 4; e += 256) {
                    const int l = e & 63, m = (e >> 6) % (nf >> 4), s = (e >> 6) / (nf >> 4), f = m * 16 + (l & 15);
                    v4u part[3];
                    taps_filter_piece(p, raw + f * T, k0 + f < p.K, s, l >> 4, part);
#pragma unroll
                    for (int q = 0; q < 3; ++q) fl[s * SLOT + (q * MB + m0 + m) * 64 + l] = part[q];
                }
            }
            __syncthreads();
        }
    };
    typedef __attribute__((address_space(3))) void* lds_ptr;
    const int nload = (3 * MB - wave + 3) / 4;          // ring: loads of 64 pieces per step, this wave's
    const auto brs = __builtin_amdgcn_make_buffer_rsrc((void*)p.bank, 0, RES ? 0 : 0x7FFFFFFF, kRsrcFlags);
    int lkb = 0, lstep = 0, lslot = 0, ltile = t0;      // ring: what is requested next, and where it goes
    auto request = [&]() __attribute__((always_inline)) {
        const int at = (lkb * p.steps + lstep) * (SLOT * 16);
#pragma unroll
        for (int i = 0; i < (3 * MB + 3) / 4; ++i) {
            const int k = i * 4 + wave;
            if (k < 3 * MB)                             // uniform
                __builtin_amdgcn_raw_ptr_buffer_load_lds(brs, (lds_ptr)(fl + lslot * SLOT + k * 64), 16, lane * 16, at + k * 1024, 0, 0);
        }
        lslot = lslot == 2 ? 0 : lslot + 1;
        if (++lstep == p.steps) {
            lstep = 0;
            ltile += dt;
            lkb = ltile < t1 ? fdiv(ltile, p.d_pt) : 0;
        }
    };
    auto wait_loads = [](int later) __attribute__((always_inline)) {      // vmcnt(later)
        switch (later) {
        case 1: __builtin_amdgcn_s_waitcnt(0x0F71); break;
        case 2: __builtin_amdgcn_s_waitcnt(0x0F72); break;
        case 3: __builtin_amdgcn_s_waitcnt(0x0F73); break;
        default: __builtin_amdgcn_s_waitcnt(0x0F70); break;
        }
    };
    auto meet = []() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };

    // Tiles with outputs to be formed again (see general_split_kernel).
    uint64_t redo = 0;
    uint32_t redo_blocks = 0;                           // blocks of sixteen filters that they are in
    auto redo_bit = [&](int t) __attribute__((always_inline)) { return 1ull << ((t - t0) / dt % 64); };
    // Where an operand is tiny (it lost 2^-134 at most), sums below this are formed again: 512 products with values of
    // up to 2^40 may be off by 2^-85.  With larger ones beside them, all are.
    auto redo_line = [](int notes) __attribute__((always_inline)) {
        return notes & kNoteTiny ? (notes & kNoteHuge ? __builtin_inff() : 0x1p-60f) : 0.f;
    };

    // The lane's quad of outputs in block n of the wave: byte offset of out[n][k0 + l16][y][x] from
    // out[n_first][k0][0][0]; how many of the four are there.
    auto out_quad = [&](const Place& t, int n, uint32_t* o) __attribute__((always_inline)) {
        const int pp = t.p0 + wave * 64 + n * 16 + 4 * g;
        int x, y;
        const int dn = pixel(t, min(pp, total - 4), &x, &y);
        *o = ((uint32_t)(dn * p.K + l16) * (uint32_t)plane + (uint32_t)(y * p.Wo + t.x0 + x)) * 4u;
        return pp < total ? min(t.ws - x, 4) : 0;
    };

    int kb = -1, slot = 0;
    Place t = place(t0);
    fetch(t);
    if constexpr (!RES) {
        lkb = fdiv(t0, p.d_pt);
        request();
        request();
        __builtin_amdgcn_s_waitcnt(0x0F70);
    }
    __syncthreads();                                    // s_range is clear
    for (int tile = t0, par = 0; tile < t1; tile += dt, par ^= 1) {
        meet();                                         // the last tile's operands have been read
        if (t.kb != kb) {                               // uniform
            kb = t.kb;
            load_filters(kb);
        }
        commit(t, par);
        const Place next = place(tile + dt < t1 ? tile + dt : tile);
        fetch(next);
        // The lane's pixel of the wave's 64: its LDS byte address at tap (0, 0), its output's byte offset from
        // out[n_first][0][0][0].  A lane works with the address of pixel 16 n + l16 and, filters being columns
        // of the result, writes pixels 16 n + 4 g and the three behind.
        uint32_t base[NB], obase;
        int px;
        {
            const int pp = t.p0 + wave * 64 + lane;
            int y;
            const int dn = pixel(t, min(pp, total - 1), &px, &y);
            const uint32_t mine = (uint32_t)((dn * p.H + y - t.y_first) * p.C * p.LS + px) * 4u;
            obase = (uint32_t)(dn * p.K * (int)plane + y * p.Wo + t.x0 + px) * 4u;
            if (pp >= total) px = 0x10000;              // (not there)
#pragma unroll
            for (int n = 0; n < NB; ++n) base[n] = (uint32_t)__builtin_amdgcn_ds_bpermute((n * 16 + l16) * 4, (int)mine);
        }
        v4f hi[MB][NB], lo[MB][NB];
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n) { hi[m][n] = v4f{}; lo[m][n] = v4f{}; }
        meet();
        const int range = s_range[par];
        if (tid == 0) s_range[par ^ 1] = 0;             // (read before the barrier above, set behind the next)

        // A step: its image operands were requested during the step before where registers allow that, its
        // filters go sixteen at a time, the next sixteen on their way.
        constexpr int DB = MB == 1 ? 2 : 1;
        v4u b[DB][NB][3], off = table[g];
        auto load_b = [&](v4u (&b)[NB][3]) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const char* at = img + (base[n] + off[q]);
#pragma unroll
                    for (int k = 0; k < 3; ++k) b[n][k][q] = *(const uint32_t*)(at + k * PSB);
                }
        };
        auto step = [&](int s, v4u (&b)[NB][3], v4u (&bnext)[NB][3]) __attribute__((always_inline)) {
            if constexpr (!RES) {
                if (s >= 2) wait_loads(nload);          // this step's filters; the next step's may be on their way
                meet();
                request();
            }
            const v4u* f = fl + (RES ? s : slot) * SLOT + lane;
            v4u a[2][3];
            auto load_a = [&](int m) __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k < 3; ++k) a[m & 1][k] = f[(k * MB + m) * 64];
            };
            load_a(0);
            if constexpr (DB == 1) load_b(b);
            const v4u* const noff = table + min(s + 1, p.steps - 1) * 4 + g;
            if constexpr (DB == 1) off = *noff;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                if (m + 1 < MB) load_a(m + 1);
                if (DB == 2 && m == 0) {
                    load_b(bnext);
                    off = table[min(s + 2, p.steps - 1) * 4 + g];
                }
                __builtin_amdgcn_sched_barrier(0);              // (the next operands are on their way before these products)
                auto mfma = [](v4u x, v4u w, v4f c) __attribute__((always_inline)) {
                    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, x), __builtin_bit_cast(v8bf, w), c, 0, 0, 0);
                };
                const v4u (&w)[3] = a[m & 1];
                constexpr int kSmall[5][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}};
#pragma unroll
                for (int q = 0; q < 5; ++q)
#pragma unroll
                    for (int n = 0; n < NB; ++n) lo[m][n] = mfma(b[n][kSmall[q][0]], w[kSmall[q][1]], lo[m][n]);
#pragma unroll
                for (int n = 0; n < NB; ++n) hi[m][n] = mfma(b[n][0], w[0], hi[m][n]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (!RES) slot = slot == 2 ? 0 : slot + 1;
        };
        if constexpr (DB == 2) {
            load_b(b[0]);
            off = table[min(1, p.steps - 1) * 4 + g];
            for (int s = 0; s < p.steps; s += 2) {
                step(s, b[0], b[1]);
                if (s + 1 < p.steps) step(s + 1, b[1], b[0]);
            }
        } else {
            for (int s = 0; s < p.steps; ++s) step(s, b[0], b[0]);
        }
        if constexpr (!RES) __builtin_amdgcn_s_waitcnt(0x0F70);      // the next tile's first two steps are in LDS

        // (a buffer's range check keeps what isn't there from being written)
        float bad = 0.f;
        uint32_t again = 0;                             // blocks of sixteen filters with sums below the line
        const uint32_t whole = px + 4 <= t.ws ? obase : kNowhere;
        uint32_t o[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const uint32_t ob = (uint32_t)__builtin_amdgcn_ds_bpermute((n * 16 + 4 * g) * 4, (int)whole);
            o[n] = ob == kNowhere ? kNowhere : ob + (uint32_t)l16 * (uint32_t)plane * 4u;
        }
        // A lane's quad of outputs in block (m, n), whole or what a row's end leaves of it.
        auto put = [&](auto ors, int n, v4f v, bool has) __attribute__((always_inline)) {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), ors, has ? o[n] : kNowhere, 0, 0);
            if (t.ws & 3) {                             // uniform: quads that a row's end cuts
                const int x = __builtin_amdgcn_ds_bpermute((n * 16 + 4 * g) * 4, px);
                const uint32_t ob = (uint32_t)__builtin_amdgcn_ds_bpermute((n * 16 + 4 * g) * 4, (int)obase) + (uint32_t)l16 * (uint32_t)plane * 4u;
                if (x < t.ws && x + 4 > t.ws && has)
#pragma unroll
                    for (int r = 0; r < 3; ++r)
                        if (x + r < t.ws) {
                            const float value = v[r];
                            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, value), ors, ob + 4u * r, 0, 0);
                        }
            }
        };
        auto out_of = [&](int m) __attribute__((always_inline)) {
            return __builtin_amdgcn_make_buffer_rsrc((void*)(p.out + ((int64_t)t.n_first * p.K + (t.kb * MB + m) * 16) * plane), 0, 0x7FFFFFFF, kRsrcFlags);
        };
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const auto ors = out_of(m);
            const int note = s_notes[m * 16 + l16];
            const bool has = (t.kb * MB + m) * 16 + l16 < p.K && (note & kNoteOne) == 0;
            const float line = has ? redo_line(range | note) : 0.f;
            bool below = false;
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                v4f v;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = hi[m][n][r] + lo[m][n][r];
                    bad = __builtin_fmaf(v[r], 0.f, bad);        // NaN behind anything not finite
                    below |= fabsf(v[r]) < line;
                }
                put(ors, n, v, has);
            }
            if (__any(below)) again |= 1u << m;
        }
        // Filters of one weight give their pixels, rounded once: those are read again, four a lane like its outputs.
        if (__any(lane < MB * 16 && (s_notes[min(lane, MB * 16 - 1)] & kNoteOne) != 0)) {
            const int64_t ifirst = (int64_t)t.n_first * p.C * HW * 4;
            const auto irs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.in + ifirst), 0,
                                                              (int)min(in_bytes - ifirst, (int64_t)0x7FFFFFFF), kRsrcFlags);
            const int pp = t.p0 + wave * 64 + lane;
            int x, y;
            const int dn = pixel(t, min(pp, total - 1), &x, &y);
            const uint32_t ib = pp < total && x < t.ws ? (uint32_t)(dn * p.C * HW + y * p.W + t.x0 + x) * 4u : kNowhere;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const int note = s_notes[m * 16 + l16];
                const bool one = (note & kNoteOne) != 0;          // (no filter beyond K is one)
                const int tap = one ? note >> kNoteTap : 0, k = (t.kb * MB + m) * 16 + l16;
                const int c = fdiv(tap, p.d_ff), ij = tap - c * p.F * p.F, i = fdiv(ij, p.d_f);
                const uint32_t at = (uint32_t)(c * HW + i * p.W + ij - i * p.F) * 4u;
                const float w = p.filt[(int64_t)min(k, p.K - 1) * (p.C * p.F * p.F) + tap];
                v4f v[NB];
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    const uint32_t quad = (uint32_t)__builtin_amdgcn_ds_bpermute((n * 16 + 4 * g) * 4, (int)ib);
                    v[n] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(irs, one && quad != kNowhere ? quad + at : kNowhere, 0, 0));
                }
                const auto ors = out_of(m);
#pragma unroll
                for (int n = 0; n < NB; ++n) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[n][r] *= w;
                    put(ors, n, v[n], one);
                }
            }
        }
        if (__any(!(bad == 0.f))) again = (1u << MB) - 1u;
        if (again != 0) {                               // uniform
            redo |= redo_bit(tile);
            redo_blocks |= again;
        }
        t = next;
    }

    // ---- outputs that the split cannot form: a wave's blocks again, on the fp32 matrix cores
    if (redo == 0) return;
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // this wave's outputs are in memory
    // Sixteen taps a time: lane (g, l) brings weights 4 g .. 4 g + 3 of filter l and, for each of the four, pixel l of the
    // wave's four blocks; instruction q takes word q, so that its reduction index g is tap 4 g + q.  The next sixteen are on their way.
    const int T = p.C * p.F * p.F;
    const auto wrs = __builtin_amdgcn_make_buffer_rsrc((void*)p.filt, 0, (int)min((int64_t)p.K * T * 4, (int64_t)0x7FFFFFFF), kRsrcFlags);
    for (int tile = t0; tile < t1; tile += dt) {
        if ((redo & redo_bit(tile)) == 0) continue;     // uniform
        const Place t = place(tile);
        const int64_t ifirst = (int64_t)t.n_first * p.C * HW * 4;
        const auto irs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.in + ifirst), 0,
                                                          (int)min(in_bytes - ifirst, (int64_t)0x7FFFFFFF), kRsrcFlags);
        uint32_t pix[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int pp = t.p0 + wave * 64 + n * 16 + l16;
            int x, y;
            const int dn = pixel(t, min(pp, total - 1), &x, &y);
            pix[n] = pp < total && x < t.ws ? (uint32_t)(dn * p.C * HW + y * p.W + t.x0 + x) * 4u : kNowhere;
        }
        v4f acc[MB][NB] = {}, x[2][NB], w[2][MB];
        auto bring = [&](int s, v4f (&x)[NB], v4f (&w)[MB]) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const int k = (t.kb * MB + m) * 16 + l16;
                // (beyond the last tap another filter's, against pixels that are zero: set to zero below)
                w[m] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                    wrs, k < p.K && (redo_blocks >> m & 1) ? (uint32_t)(k * T + s * 16 + 4 * g) * 4u : kNowhere, 0, 0));
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int tap = s * 16 + 4 * g + q;
                const int c = fdiv(tap, p.d_ff), ij = tap - c * p.F * p.F, i = fdiv(ij, p.d_f);
                const uint32_t at = (uint32_t)(c * HW + i * p.W + ij - i * p.F) * 4u;
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    x[n][q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(irs, tap < T && pix[n] != kNowhere ? pix[n] + at : kNowhere, 0, 0));
#pragma unroll
                for (int m = 0; m < MB; ++m) w[m][q] = tap < T ? w[m][q] : 0.f;
            }
        };
        const int groups = (T + 15) / 16;
        bring(0, x[0], w[0]);
        for (int s0 = 0; s0 < groups; s0 += 2)
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                if (s0 + d >= groups) break;            // uniform
                bring(s0 + d + 1, x[d ^ 1], w[d ^ 1]);  // (behind the last one: nothing is read)
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    if (redo_blocks >> m & 1)           // uniform
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int n = 0; n < NB; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[d][n][q], w[d][m][q], acc[m][n], 0, 0, 0);
            }
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            uint32_t ob;
            const int there = out_quad(t, n, &ob);
            float* const o = p.out + ((int64_t)t.n_first * p.K + t.kb * MB * 16) * plane + ob / 4u;
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (r < there && (redo_blocks >> m & 1) && (t.kb * MB + m) * 16 + l16 < p.K) o[(int64_t)(m * 16) * plane + r] = acc[m][n][r];
        }
    }
}

// ---- host side -----------------------------------------------------------------------------------

// Filters and steps of a layer.
struct TapsSteps { int MB, KB, P, RC, nc, steps; };
TapsSteps taps_steps(const Shape& s)
{
    TapsSteps t{};
    const int k16 = (s.K + 15) / 16, R = s.C * s.F;
    t.KB = (k16 + 3) / 4;
    t.MB = (k16 + t.KB - 1) / t.KB;
    t.P = (s.F + 1) / 2;
    t.RC = R / 2;
    t.nc = t.RC * t.P + (R & 1 ? (t.P + 1) / 2 : 0);
    t.steps = (t.nc + 7) / 8;
    return t;
}
bool taps_fits(const TapsSteps& t, int ahead, int psb) { return ahead * 3 * t.MB * 1024 + t.steps * 64 + kTapsStatic + 3 * psb <= kTapsLds; }

// Column strips, and where filters and image block lie, at the least cost.
TapsPlan make_taps_plan(const Shape& s)
{
    const TapsSteps t = taps_steps(s);
    TapsPlan best{t.MB, t.KB, t.P, t.RC, t.nc, t.steps, 0, 0, 0, 0, 0, 0, 0, false, false};
    if (s.C > 16 || s.F < 2 || s.F > 11 || t.steps > kTapsSteps || (int64_t)s.K * s.C * s.F * s.F >= 1LL << 29) return best;
    const int64_t all_rows = (int64_t)s.N * s.Ho;
    double least = 1e300;
    for (int mode = 0; mode < 3; ++mode) {
        const bool res = mode < 2;
        const int psb = mode == 0 ? kTapsPartSmall : taps_part_large(t.MB);
        if ((!res && t.steps < 3) || !taps_fits(t, res ? t.steps : 3, psb)) continue;
        if (res && 16LL * s.C * s.F * s.F * 4 > 3 * psb) continue;           // sixteen filters' weights go through the image block's place
        int last = 0;
        for (int about : {16, 32, 48, 64, 96, 128, 192, 256}) {
            const int nstrips = (s.Wo + about - 1) / about, bw = ((s.Wo + nstrips - 1) / nstrips + 3) / 4 * 4;
            if (bw == last || (s.Wo + bw - 1) / bw != nstrips) continue;
            last = bw;
            const int need = bw + 2 * t.P - 2;
            // pixels numbered through the batch (a tile may reach over several images, each with rows of its own),
            // or image by image (the last tile of each ends early)
            for (int each = 0; each < (s.N > 1 ? 2 : 1); ++each) {
                const int64_t grows = each ? s.Ho : all_rows;
                const int64_t rows = std::min<int64_t>((kTapsNT - 2) / bw + 2, grows);
                const int64_t cross = each ? 0 : std::min<int64_t>(rows >= 2 ? (rows - 2) / s.Ho + 1 : 0, s.N - 1);
                const int64_t slots = rows + (s.F - 1) * (cross + 1);
                const int64_t tpg = (grows * bw + kTapsNT - 1) / kTapsNT, ptiles = tpg * nstrips * (each ? s.N : 1);
                if (ptiles * t.KB > 2147483647LL) continue;
                // (a row stride without bank conflicts if there is room for it)
                int LS = (need + 15) / 32 * 32 + 16;
                if (LS < need) LS += 32;
                if (slots * s.C * LS * 4 > psb) LS = (need + 3) / 4 * 4;
                if (slots * s.C * LS * 4 > psb) continue;
                // cycles of a tile times what its stores cost with rows cut into pieces of that length, fitted to eleven
                // shapes with every width: 2 % above the best width on average, 9 % at most
                const double quads = ((double)kTapsNT / bw + 1 + s.F) * s.C * LS / 4;
                const double cost = (double)ptiles * (t.steps * t.MB * 300.0 + 2000.0 + 140.0 * std::ceil(quads / 256.0)) *
                                    (1.0 + 2.5 / bw + 1e-4 * bw + (bw % 16 ? 0.04 : 0.0)) * (LS % 32 == 16 ? 1.0 : 1.005) * (res ? 1.0 : 1.02);
                if (cost < least) {
                    least = cost;
                    best.bw = bw;
                    best.nstrips = nstrips;
                    best.LS = LS;
                    best.ptiles = (int)ptiles;
                    best.tpg = (int)tpg;
                    best.grows = (int)grows;
                    best.psb = psb;
                    best.res = res;
                    best.ok = true;
                }
            }
        }
    }
    return best;
}

template <int MB, bool RES, int PSB>
int taps_launch(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, const TapsPlan& pl, bool static_ws)
{
    TapsParams p{in, filt, out, nullptr, nullptr, s.N, s.C, s.H, s.W, s.K, s.F, s.Ho, s.Wo,
                 pl.bw, pl.nstrips, pl.LS, pl.ptiles, pl.ptiles * pl.KB, pl.tpg, pl.grows, pl.P, pl.RC, pl.nc, pl.steps,
                 make_fastdiv(pl.nstrips), make_fastdiv(pl.ptiles), make_fastdiv(pl.tpg), make_fastdiv(pl.bw),
                 make_fastdiv(s.Ho), make_fastdiv(pl.LS / 4), make_fastdiv(s.C), make_fastdiv(s.H), make_fastdiv(pl.P),
                 make_fastdiv(s.F), make_fastdiv(s.F * s.F)};
    const int cus = gen_cus();
    if (cus <= 0) return DCONV_LAUNCH_FAILED;
    auto kern = split_taps_kernel<MB, RES, PSB>;
    static std::atomic<uint64_t> lds_limit_raised{0};
    if (!raise_lds_limit((const void*)kern, kTapsLds, lds_limit_raised)) return DCONV_LAUNCH_FAILED;
    GenWorkspace ws;
    if constexpr (!RES) {
        const size_t bank_floats = (size_t)pl.KB * pl.steps * 3 * MB * 256, floats = bank_floats + (size_t)pl.KB * MB * 16;
        if (floats > kGenWorkspaceFloats) return DCONV_UNSUPPORTED;
        if (static_ws) {
            if (gen_static_workspace(st, floats, 0, &ws) != DCONV_OK) return DCONV_UNSUPPORTED;
        } else {
            ws = gen_workspace(st, floats, 0);
            if (!ws.part) return DCONV_UNSUPPORTED;
        }
        p.bank = (const v4u*)ws.part;
        p.notes = (const int*)(ws.part + bank_floats);
        begin_launch();
        hipLaunchKernelGGL((taps_bank_kernel<MB>), dim3((unsigned)(pl.KB * MB * ((pl.steps + 3) / 4))), dim3(256), 0, st, p, (v4u*)ws.part, (int*)(ws.part + bank_floats));
        if (const int rc = launch_status(); rc != DCONV_OK) return rc;
    }
    const int lds = pl.steps * 64 + (RES ? pl.steps : 3) * 3 * MB * 1024 + 3 * PSB;
    begin_launch();
    hipLaunchKernelGGL(kern, dim3((unsigned)std::min(p.tiles, 2 * cus)), dim3(256), (size_t)lds, st, p);
    return launch_status();
}

}  // namespace

static bool taps_plan_fits(const Shape& s, const TapsPlan& pl)
{
    if (!pl.ok) return false;
    // pixels are numbered in 32 bits; lanes address the image with 32-bit byte offsets from the tile's first image
    if ((int64_t)s.N * s.Ho * pl.bw > 2147483647LL) return false;
    // and of the outputs
    const int64_t span = std::min<int64_t>(kTapsNT / ((int64_t)s.Ho * pl.bw) + 2, pl.grows == s.Ho ? 1 : s.N), plane = (int64_t)s.Ho * s.Wo;
    return (span * s.C + 1) * s.H * s.W < 1LL << 29 && ((span - 1) * s.K + 17) * plane < 1LL << 29;
}

TapsPlan split_taps_plan(const Shape& s)
{
    TapsPlan pl = make_taps_plan(s);
    pl.ok = taps_plan_fits(s, pl);
    return pl;
}

// When this kernel goes before the others, by estimates of its time and of theirs fitted to 1544 layers drawn at
// random (half of them one image of 64^2 .. 4096^2, half 1 to 64 images of 1 to 16 channels; 2x2 to 11x11, 9 to 256
// filters; rms 9 and 16 %).  Here: 6.2 us and 0.30 us per step and block of sixteen filters to split them (or 2.5 us for
// the small kernel), per round of tiles 0.89 us, 0.39 us per step and block and 0.037 us per row of taps, 6.6 us per GB of
// output, two thirds more beyond the memory-side cache.  The others: 8.4 us per GFLOP and the output.  It has to promise
// a tenth: then 317 layers are chosen, 1.33 times faster than the fastest other kernel on average, six of them 3 % or more
// slower (four images with sixteen filters or fewer, which the last term of `there` is for since); at a twentieth 361, 21
// slower.  Layers that the fit did not see: profiles/rule_few_channels.txt.
double split_taps_time_if_preferred(const Shape& s, TapsPlan* plan)
{
    if (s.C > 16 || s.F < 2 || s.F > 11 || s.K < 9) return 1e300;
    const TapsSteps t = taps_steps(s);
    if (t.steps > kTapsSteps) return 1e300;
    const double px = (double)s.N * s.Ho * s.Wo, mb = px * s.K * 4e-6;
    // (few multiply-adds per output of a large volume: bound by its stores, which the special case's kernel arranges
    // better: 4096 x 4096 with 64 8x8 filters 1337 us there, 1588 here, 3008 x 2282 with 48 7x7 457 and 500; with 9x9
    // filters 1632 and 1367, 913 and 776 on 3000 x 3000)
    if (s.N == 1 && s.C == 1 && mb > 1000 && s.F < 9) return 1e300;
    const double tiles = std::ceil(px * 1.04 / kTapsNT) * t.KB, work = t.steps * t.MB;
    const double rounds = tiles > 1536 ? tiles / 512 : std::ceil(tiles / 512);
    const bool res = taps_fits(t, t.steps, kTapsPartSmall);
    const double here = 6.2 + rounds * (0.386 * work + 0.89 + 0.0369 * s.C * (s.F + 4)) + (res ? 0.3 * work : 2.45 + 0.064 * t.steps) + 0.152 * mb +
                        0.098 * std::max(0.0, mb - 250);
    const double taps = (double)s.C * s.F * s.F;
    // (one image of one channel has kernels with blocks of sixteen filters)
    const int block = s.N == 1 && s.C == 1 && s.K <= 16 ? 16 : 32;
    const double there = 4.74 + 0.00839e-6 * 2 * px * ((s.K + block - 1) / block * block) * taps + 0.169 * mb + 0.0062 * taps;
    if (here >= 0.9 * there) return 1e300;
    *plan = split_taps_plan(s);
    return plan->ok ? here : 1e300;
}

int launch_split_taps(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, bool static_ws, const TapsPlan& pl)
{
    if (!pl.ok) return DCONV_UNSUPPORTED;
    // (filters split into the workspace: see try_split)
    if (!pl.res && !static_ws && gen_capturing(st)) return DCONV_UNSUPPORTED;
    switch (pl.MB * 4 + (!pl.res ? 0 : pl.psb == kTapsPartSmall ? 1 : 2)) {
    case 4: return taps_launch<1, false, taps_part_large(1)>(in, filt, out, s, st, pl, static_ws);
    case 5: return taps_launch<1, true, kTapsPartSmall>(in, filt, out, s, st, pl, static_ws);
    case 6: return taps_launch<1, true, taps_part_large(1)>(in, filt, out, s, st, pl, static_ws);
    case 8: return taps_launch<2, false, taps_part_large(2)>(in, filt, out, s, st, pl, static_ws);
    case 9: return taps_launch<2, true, kTapsPartSmall>(in, filt, out, s, st, pl, static_ws);
    case 10: return taps_launch<2, true, taps_part_large(2)>(in, filt, out, s, st, pl, static_ws);
    case 12: return taps_launch<3, false, taps_part_large(3)>(in, filt, out, s, st, pl, static_ws);
    case 13: return taps_launch<3, true, kTapsPartSmall>(in, filt, out, s, st, pl, static_ws);
    case 14: return taps_launch<3, true, taps_part_large(3)>(in, filt, out, s, st, pl, static_ws);
    case 16: return taps_launch<4, false, taps_part_large(4)>(in, filt, out, s, st, pl, static_ws);
    case 17: return taps_launch<4, true, kTapsPartSmall>(in, filt, out, s, st, pl, static_ws);
    case 18: return taps_launch<4, true, taps_part_large(4)>(in, filt, out, s, st, pl, static_ws);
    default: return DCONV_UNSUPPORTED;
    }
}

}  // namespace dconv
