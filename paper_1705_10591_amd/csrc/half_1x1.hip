// 1x1 filters of the general case for short data types (fp16, bf16, int8): every output pixel is a
// product of the filter matrix with the pixel's channel run, with no neighbourhood, so the maps are
// numbered as one run of N * H * W pixels and a tile's image block is exactly its pixels.
//
// What bounds such a layer is memory latency: general_half_kernel takes 32 bytes of every pixel per
// chunk, one matrix-core step per barrier, one chunk ahead.  Here a chunk is CB such blocks (128 bytes
// of a pixel's run: whole lines of a channels-last image), three chunks share a ring in LDS, and
// chunk u + 2 is requested, straight into LDS, when chunk u begins.
//
// LDS.  A 16-byte load with the LDS bit set writes lane l's piece to place l, so consecutive lanes have
// to bring consecutive places; for coalesced loads they should bring the Q = 2 * CB pieces of one
// pixel.  Rows of Q pieces read at one piece per lane would all fall on the same few banks, so row r
// keeps its piece q at place q ^ ((r / R) % Q), R = 16 / Q: sixteen consecutive rows then cover all
// 64 banks, and a load still brings whole runs, in another order.
//
// Measured (general_half_kernel -> this one; the sums are taken in the same order, so the bits are the
// same): 32 x 512 x 28 x 28, 128 filters, fp16, channels last 24.0 -> 10.3 us (3.8 TB/s); 64 x 2048 x
// 7 x 7, 512 filters 75 -> 15 us; one image of 512 x 28 x 28, 512 filters 19.9 -> 4.9 us; 400 layers
// drawn at random (16 to 1024 channels and filters, both layouts, 8 and 16 bits) 1.74 times faster
// on average.
#include "half_kernel.h"

namespace dconv {

namespace {

struct PointParams {
    const char* in;      // [N][HW][C], or blocked [N][C/cb][HW][cb]
    const char* filt;    // [K][C] in both layouts
    float* out;          // [N][K][HW]
    int N, C, HW, K;
    int KB;              // filter tiles
    int tiles, per_xcd;
    int blocked;
    FastDiv d_kb, d_hw;
};

template <int DT, int MT, int NT, int WM, int WN, int CB>
__global__ void __launch_bounds__(kWave * WM * WN, 2)
general_point_kernel(PointParams p)
{
    constexpr int THREADS = kWave * WM * WN;
    constexpr int MW = MT / (32 * WM), NW = NT / (32 * WN);
    constexpr int Q = 2 * CB, R = 16 / Q;
    constexpr int NFI = MT * Q / THREADS, NII = NT * Q / THREADS, NI = NFI + NII;   // loads per thread and chunk
    constexpr int SLOT = (MT + NT) * Q;                      // 16-byte pieces: filters, pixels
    constexpr uint32_t kNowhere = 0xC0000000u;
    constexpr int kRsrcFlags = 0x00020000;
    static_assert(MT * Q % THREADS == 0 && NT * Q % THREADS == 0 && THREADS / Q % 16 == 0, "whole loads, one key per thread");

    extern __shared__ __attribute__((aligned(16))) v4f ring[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l32 = lane & 31;
    const int wm = wave / WN, wn = wave % WN;

    const int tile = (int)(blockIdx.x % 8) * p.per_xcd + (int)(blockIdx.x / 8);
    if (tile >= p.tiles) return;                             // uniform: before any barrier
    const int ptile = fdiv(tile, p.d_kb), kb = tile - ptile * p.KB;
    const int p0 = ptile * NT, k0 = kb * MT;
    const int total = p.N * p.HW;
    const int CBY = p.C * elem_bytes(DT);                    // bytes of a pixel's channel run
    const int nch = CBY / (CB * kHalfChunkBytes);
    const int n_first = fdiv(p0, p.d_hw);

    // ---- staging: load `it` of a thread brings the piece of row tid / Q + it * THREADS / Q for place tid % Q
    const int row0 = tid / Q, q = (tid % Q) ^ ((row0 / R) % Q);
    const int64_t image = (int64_t)p.HW * CBY;
    uint32_t ig[NII];
#pragma unroll
    for (int it = 0; it < NII; ++it) {
        const int pp = p0 + row0 + it * (THREADS / Q);
        uint32_t g = kNowhere;
        if (pp < total) {
            const int n = fdiv(pp, p.d_hw), yx = pp - n * p.HW;
            g = p.blocked ? (uint32_t)((n - n_first) * (int)image + (q >> 1) * p.HW * kHalfChunkBytes + yx * kHalfChunkBytes + (q & 1) * 16)
                          : (uint32_t)((pp - n_first * p.HW) * CBY + q * 16);
        }
        ig[it] = g;
    }
    const uint32_t wg = (uint32_t)(row0 * CBY + q * 16);     // (filters beyond K lie beyond the end of the bank)
    const int64_t ifirst = n_first * image, wfirst = (int64_t)k0 * CBY;
    const int64_t in_left = p.N * image - ifirst, filt_left = (int64_t)p.K * CBY - wfirst;
    const int istep = p.blocked ? CB * p.HW * kHalfChunkBytes : CB * kHalfChunkBytes;
    typedef __attribute__((address_space(3))) void* lds_ptr;
    auto fetch = [&](int chunk, v4f* slot) __attribute__((always_inline)) {
        const int64_t ioff = (int64_t)chunk * istep, woff = (int64_t)chunk * (CB * kHalfChunkBytes);
        auto irs = __builtin_amdgcn_make_buffer_rsrc((void*)(p.in + ifirst + ioff), 0,
                                                     (int)min(in_left - ioff, (int64_t)0x7FFFFFFF), kRsrcFlags);
        auto wrs = __builtin_amdgcn_make_buffer_rsrc((void*)(p.filt + wfirst + woff), 0,
                                                     (int)min(filt_left - woff, (int64_t)0x7FFFFFFF), kRsrcFlags);
#pragma unroll
        for (int it = 0; it < NFI; ++it)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lds_ptr)(slot + it * THREADS + wave * kWave), 16, (int)wg,
                                                     it * (THREADS / Q) * CBY, 0, 0);
#pragma unroll
        for (int it = 0; it < NII; ++it)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(irs, (lds_ptr)(slot + MT * Q + it * THREADS + wave * kWave), 16, (int)ig[it], 0, 0, 0);
    };

    // ---- operands: piece 2 cb + h of row 32 i + l32 lies at place (2 cb + h) ^ key of the row
    int place[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) place[cb] = l32 * Q + ((2 * cb + h) ^ ((l32 / R) % Q));

    v16f acc[MW][NW];
#pragma unroll
    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
        for (int nt = 0; nt < NW; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mt][nt][r] = 0.f;

    fetch(0, ring);
    if (nch > 1) fetch(1, ring + SLOT);
    int sc = 0;                                              // slot of the chunk being consumed
    for (int u = 0; u < nch; ++u) {
        // Chunk u is in LDS: this wave waits for its own loads (those of chunk u + 1 may be on their
        // way), the barrier for everybody's.  All have then left chunk u - 1, whose slot chunk u + 2
        // takes.  A bare barrier: a fence would wait for every outstanding load.
        if (u + 1 < nch) __builtin_amdgcn_s_waitcnt(0x0F70 | (NI & 15) | ((NI >> 4) << 14));
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (u + 2 < nch) fetch(u + 2, ring + (sc == 0 ? 2 : sc - 1) * SLOT);
        const v4f* slot = ring + sc * SLOT;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            v4f a[MW], b[NW];
#pragma unroll
            for (int mt = 0; mt < MW; ++mt) a[mt] = slot[place[cb] + (wm * MW + mt) * 32 * Q];
#pragma unroll
            for (int nt = 0; nt < NW; ++nt) b[nt] = slot[MT * Q + place[cb] + (wn * NW + nt) * 32 * Q];
#pragma unroll
            for (int mt = 0; mt < MW; ++mt)
#pragma unroll
                for (int nt = 0; nt < NW; ++nt) acc[mt][nt] = mfma_16B<DT>(a[mt], b[nt], acc[mt][nt]);
        }
        sc = sc == 2 ? 0 : sc + 1;
    }

    // ---- write back: 32 lanes hold 32 consecutive pixels of one output map
    const int kleft = p.K - k0 - 32 * wm * MW - 4 * h;
#pragma unroll
    for (int nt = 0; nt < NW; ++nt) {
        const int pp = p0 + (wn * NW + nt) * 32 + l32;
        if (pp >= total) continue;
        const int n = fdiv(pp, p.d_hw);
        float* o = p.out + ((int64_t)n * p.K + k0 + 32 * wm * MW + 4 * h) * p.HW + (pp - n * p.HW);
#pragma unroll
        for (int mt = 0; mt < MW; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kk = mt * 32 + mfma_row(r, 0);
                if (kk < kleft) o[(int64_t)kk * p.HW] = acc[mt][nt][r];
            }
    }
}

template <int DT, int MT, int NT, int WM, int WN, int CB>
int launch_point_tile(const void* in, const void* filt, float* out, const Shape& s, hipStream_t st, bool blocked)
{
    const int64_t total = (int64_t)s.N * s.H * s.W;
    const int KB = (s.K + MT - 1) / MT;
    const int64_t tiles = (total + NT - 1) / NT * KB;
    const int CBY = s.C * elem_bytes(DT);
    const int64_t image = (int64_t)s.H * s.W * CBY;
    const int64_t span = std::min<int64_t>(NT / ((int64_t)s.H * s.W) + 2, s.N);      // images a tile reaches
    if (CBY % (CB * kHalfChunkBytes) != 0 || total > 2147483647LL - NT || tiles > 2000000000LL ||
        span * image >= (1LL << 31) || (int64_t)(MT + 1) * CBY >= (1LL << 31))
        return DCONV_UNSUPPORTED;
    if ((((uintptr_t)in) & 15) != 0 || (((uintptr_t)filt) & 15) != 0) return DCONV_UNSUPPORTED;
    const int nch = CBY / (CB * kHalfChunkBytes);
    const size_t lds_bytes = (size_t)std::min(nch, 3) * (MT + NT) * 2 * CB * 16;
    auto kern = general_point_kernel<DT, MT, NT, WM, WN, CB>;
    static std::atomic<uint64_t> lds_limit_raised{0};
    if (!raise_lds_limit((const void*)kern, kGenLdsLimit, lds_limit_raised)) return DCONV_LAUNCH_FAILED;
    const int per_xcd = (int)((tiles + 7) / 8);
    PointParams p{(const char*)in, (const char*)filt, out, s.N, s.C, s.H * s.W, s.K, KB, (int)tiles, per_xcd,
                  blocked ? 1 : 0, make_fastdiv(KB), make_fastdiv(s.H * s.W)};
    begin_launch();
    hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(kWave * WM * WN), lds_bytes, st, p);
    return launch_status();
}

template <int DT>
int launch_point_dtype(const void* in, const void* filt, float* out, const Shape& s, hipStream_t st, bool blocked, int tile)
{
    const bool four = s.C * elem_bytes(DT) % (4 * kHalfChunkBytes) == 0;
    switch (tile) {
    case 0: return four ? launch_point_tile<DT, 64, 128, 1, 4, 4>(in, filt, out, s, st, blocked)
                        : launch_point_tile<DT, 64, 128, 1, 4, 2>(in, filt, out, s, st, blocked);
    case 1: return four ? launch_point_tile<DT, 128, 128, 2, 2, 4>(in, filt, out, s, st, blocked)
                        : launch_point_tile<DT, 128, 128, 2, 2, 2>(in, filt, out, s, st, blocked);
    case 2: return four ? launch_point_tile<DT, 128, 64, 2, 2, 4>(in, filt, out, s, st, blocked)
                        : launch_point_tile<DT, 128, 64, 2, 2, 2>(in, filt, out, s, st, blocked);
    case 3: return four ? launch_point_tile<DT, 64, 64, 2, 2, 4>(in, filt, out, s, st, blocked)
                        : launch_point_tile<DT, 64, 64, 2, 2, 2>(in, filt, out, s, st, blocked);
    default: return DCONV_UNSUPPORTED;
    }
}

// Which tile: by T, the number of 64 x 64 tiles, fitted to the 400 layers above (1.2 % above the
// fastest tile on average).  The smallest has the most loads in flight; larger ones read an operand
// less often, which counts where the layer reads more than it writes or has work enough.  -1: the
// output is beyond the memory-side cache, where general_half_kernel's longer runs of a map win
// (16 x 128 x 89 x 89, 656 filters: 116 against 122-136 us).
int point_tile(const Shape& s, int dtype)
{
    const double out_bytes = 4.0 * s.N * s.K * s.H * s.W;
    if (out_bytes > 256e6) return -1;
    const int64_t T = ((int64_t)s.N * s.H * s.W + 63) / 64 * ((s.K + 63) / 64);
    const int run = s.C * elem_bytes(dtype);                               // bytes of a pixel's channels
    const bool whole = s.K > 64 && (s.K + 127) / 128 * 10 <= (s.K + 63) / 64 * 6;   // 128 filters: little padding
    if (whole && T >= 1200 && run >= 800) return 1;
    if (whole && T >= 640 && run >= 4 * s.K) return 2;
    if (T >= 6000) return run <= 256 && s.K > 64 ? 2 : 0;
    return 3;
}

}  // namespace

int launch_general_point(const void* in, const void* filt, float* out, const Shape& s, hipStream_t st, int dtype, bool blocked)
{
    if (s.F != 1) return DCONV_UNSUPPORTED;
    const int tile = point_tile(s, dtype);
    if (tile < 0) return DCONV_UNSUPPORTED;
    switch (dtype) {
    case kF16: return launch_point_dtype<kF16>(in, filt, out, s, st, blocked, tile);
    case kBF16: return launch_point_dtype<kBF16>(in, filt, out, s, st, blocked, tile);
    case kI8: return launch_point_dtype<kI8>(in, filt, out, s, st, blocked, tile);
    default: return DCONV_UNSUPPORTED;
    }
}

}  // namespace dconv
