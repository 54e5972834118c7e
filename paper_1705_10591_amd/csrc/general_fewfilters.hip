// The few-filters kernel of the general case (general_few_kernel.h): when it runs.
#include "general_few_kernel.h"
#include "few_taps_kernel.h"

#include <algorithm>

namespace dconv {

// Filter sides with a window that fits the register file comfortably, up to sixteen filters.
bool general_few_supports(const Shape& s)
{
    return s.F >= 1 && s.F <= 7 && s.K >= 1 && s.K <= 16;
}

// Worth it when its estimated kernel time is below the matrix-core kernel's (below 95 % of it
// for launches of under 768 tiles).  Both estimates are fitted to the kernel times of 1015 layers
// measured from replayed graphs, so that launches of a few microseconds count as what they take
// on the GPU and not as what the host needs to issue them (1 to 16 filters of 1x1 to 7x7, 2 to
// 256 channels, 14 x 14 to 512 x 640 maps, 1 to 512 images, 3 us to 2 ms; this kernel's within
// 16 % rms, the other's 23 %), in microseconds:
//   this kernel: 3.4 plus the largest of three bounds --
//     the chain of one workgroup, C channels of a barrier and a round of LDS latencies (0.30,
//     shared by two channels where two go per barrier), the staging of the tile's rows (0.010
//     a row), the tile's multiply-adds (0.0105 x K x F x F x rows per band) and the filters'
//     weights (0.03 x K), K rounded up to the counts it is compiled for, times the rounds of
//     tiles over 430 workgroups;
//     input and output at 5.1 TB/s;
//     K x F x F multiply-adds per pixel and channel, divided by the share of its lanes that
//     fall inside the map, at 70 TFLOP/s;
//   the matrix-core kernel: 7.1 plus the largest of a chain of 0.055 + 0.009 x F x F per channel
//     (it shares a tile's channels between workgroups), a 32-filter block at 88 TFLOP/s whatever
//     the filter count, and input and output at 2.6 TB/s.
// With the halves of the layers swapped between fitting and checking the choice is 1.2 to 1.6 %
// above the faster kernel on the checked half; on all 1015 layers 1.3 % (35 are 15 % or more off),
// against 3.8 % for the rule this replaces, which was fitted to times that included the host's
// launch cost (4 x 16 x 224 x 224 with one 1x1 filter: 13.3 -> 5.1 us).  Where this kernel is
// chosen it is up to 6 times faster (101 x 3 x 64 x 640, two 1x1 filters: 97 -> 16 us; 8 x 16 x 224
// x 224, one 7x7 filter: 189 -> 23 us; 8 x 64 x 224 x 224, three 3x3 filters: 139 -> 49 us; eight:
// 139 -> 81 us; 21 x 8 x 96 x 640, twelve 5x5: 174 -> 80 us).
static double few_time(const Shape& s, double* tiles_out)
{
    static const int kCompiled[17] = {0, 1, 2, 3, 4, 6, 6, 8, 8, 12, 12, 12, 12, 16, 16, 16, 16};
    const GfTile t = gf_tile_for(s);
    const double tiles = (double)gf_tiles(s, t.lpr, t.rpw);
    const int kc = kCompiled[s.K], ff = s.F * s.F;
    const int tw = 4 * t.lpr, tr = 4 * (kWave / t.lpr) * t.rpw;
    const double inside = (double)s.Wo * s.Ho /
                          ((double)((s.Wo + tw - 1) / tw) * tw * (double)((s.Ho + tr - 1) / tr) * tr);
    const double macs = (double)s.N * s.Ho * s.Wo * s.C * ff;             // per filter
    const double bytes = 4.0 * ((double)s.N * s.C * s.H * s.W + (double)s.N * s.K * s.Ho * s.Wo);
    const int per_barrier = (t.rpw == 1 && kc <= 8) ? 2 : 1;              // channels (see launch_gf)
    const double chain = s.C * (0.30 / per_barrier + 0.010 * (tr + s.F - 1) + 0.0105 * kc * ff * t.rpw + 0.03 * kc);
    *tiles_out = tiles;
    return 3.4 + std::max({chain * std::max(1.0, tiles / 430.0), bytes / 5.1e6, 2.0 * macs * kc / inside / 70e6});
}
bool general_few_preferred(const Shape& s)
{
    // (one image of one channel is the special case proper, which has its own few-filters kernel)
    if (!general_few_supports(s) || (s.C == 1 && s.N == 1)) return false;
    double tiles;
    const double few = few_time(s, &tiles);
    const int ff = s.F * s.F;
    const double macs = (double)s.N * s.Ho * s.Wo * s.C * ff;             // per filter
    const double bytes = 4.0 * ((double)s.N * s.C * s.H * s.W + (double)s.N * s.K * s.Ho * s.Wo);
    const double tiled = 7.1 + std::max({0.055 * s.C + 0.009 * s.C * ff, 2.0 * macs * 32 / 88e6, bytes / 2.6e6});
    return few < (tiles >= 768 ? 1.0 : 0.95) * tiled;
}

// When the taps of all filters go to the matrix cores (few_taps_kernel.h) instead: where its estimated time is
// below 95 % of the vector-ALU kernel's, for layers that are that one's, or 85 % of the general matrix-core
// kernel's, for the others (up to 64 taps there: with more, sums of many channels are no closer to the exact
// ones).  Fitted to kernel times of 1600 layers from replayed graphs (1 to 16 filters of 1x1 to 7x7, 2 to 512
// channels, 14 x 14 to 256 x 512 maps, 1 to 64 images), in microseconds; rms 15 % for this kernel, 22 % for the
// general one: 3.9, the larger one of the plan's estimate and of input and output at 4.4 TB/s with a third of
// the smaller one, 0.77 per thousand weights; 8.1, a 32-filter block at 137 TFLOP/s and the root of it, input
// and output at 4.2 TB/s and a chain per channel.  Launches of the vector-ALU kernel of over 200 us have to be beaten by 15 %, as its
// estimate is high where its tiles fill the chip many times over: 36 of 617 layers, one slower, where 5 % take four more,
// two of them slower by a quarter and no faster on average.
// Of 1722 layers that the fit did not see 617 were of the first kind: 176 are chosen, 1.47 times faster, 19 of them 3 % or
// more slower (most of them launches of under 15 us; the worst 5.8 -> 9.4); 1105 of the others: 544 chosen, twice as fast,
// eight slower, by up to 24 %.  Both estimates fitted anew (rms 13 and 14 %) with a line at 85 % had nine slower ones of 160, but
// left 46 layers to the vector-ALU kernel that were faster by 1.5 % on average here, and five times closer to the exact sums.
// A list of slower ones: profiles/rule_taps_of_few_filters.txt.
FewTapsPlan make_few_taps_plan(const Shape& s) { return few_taps_plan(s); }

FewFilters few_filters_for(const Shape& s)
{
    FewFilters r{false, 1e300, {}};
    if (s.K > 16 || s.F > 7 || (s.C == 1 && s.N == 1)) return r;
    r.alu = general_few_preferred(s);
    const FewTapsPlan pl = few_taps_plan(s);
    if (!pl.ok) return r;
    const double ff = (double)s.F * s.F, px = (double)s.N * s.Ho * s.Wo;
    const double mb = 4e-6 * ((double)s.N * s.C * s.H * s.W + px * s.K), memory = mb / 4.4;
    const double here = 3.9 + 0.99 * std::max(pl.cost, memory) + 0.357 * std::min(pl.cost, memory) + 0.77e-3 * s.K * ff * s.C;
    bool better;
    if (r.alu) {
        double tiles;
        const double few = few_time(s, &tiles);
        better = here < (few > 200 ? 0.85 : 0.95) * few;
    } else {
        const double mflop = 2e-6 * px * 32 * s.C * ff;
        better = pl.mb <= 4 && here < 0.85 * (8.1 + 0.0073 * mflop + 0.191 * std::sqrt(mflop) + 0.24 * mb + (0.0078 + 0.0183 * std::max(1.0, px / 256 / 512)) * s.C);
    }
    if (!better) return r;
    r.taps = here;
    r.plan = pl;
    return r;
}

int launch_few_taps(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, const FewTapsPlan& pl)
{
    if (!pl.ok) return DCONV_UNSUPPORTED;
    switch (s.F) {
    case 1: return few_taps_for_F<1>(in, filt, out, s, st, pl);
    case 2: return few_taps_for_F<2>(in, filt, out, s, st, pl);
    case 3: return few_taps_for_F<3>(in, filt, out, s, st, pl);
    case 4: return few_taps_for_F<4>(in, filt, out, s, st, pl);
    case 5: return few_taps_for_F<5>(in, filt, out, s, st, pl);
    case 6: return few_taps_for_F<6>(in, filt, out, s, st, pl);
    case 7: return few_taps_for_F<7>(in, filt, out, s, st, pl);
    default: return DCONV_UNSUPPORTED;
    }
}

int launch_general_few(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st)
{
    if (!general_few_supports(s)) return DCONV_UNSUPPORTED;
    switch (s.F) {
    case 1: return gf_launch_for_F<1>(in, filt, out, s, st);
    case 2: return gf_launch_for_F<2>(in, filt, out, s, st);
    case 3: return gf_launch_for_F<3>(in, filt, out, s, st);
    case 4: return gf_launch_for_F<4>(in, filt, out, s, st);
    case 5: return gf_launch_for_F<5>(in, filt, out, s, st);
    case 6: return gf_launch_for_F<6>(in, filt, out, s, st);
    case 7: return gf_launch_for_F<7>(in, filt, out, s, st);
    default: return DCONV_UNSUPPORTED;
    }
}

}  // namespace dconv
