// Instantiation of few_taps_kernel.h for ONE filter side (DCONV_F, given on the compiler command line).
#include "few_taps_kernel.h"

#ifndef DCONV_F
#error "compile with -DDCONV_F=<filter side>"
#endif

namespace dconv {

template <>
int few_taps_for_F<DCONV_F>(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, const FewTapsPlan& pl)
{
    switch (pl.mb) {
    case 1: return pl.nw == 8 ? few_taps_launch<DCONV_F, 1, 8>(in, filt, out, s, st, pl) : few_taps_launch<DCONV_F, 1, 4>(in, filt, out, s, st, pl);
    case 2: return pl.nw == 8 ? few_taps_launch<DCONV_F, 2, 8>(in, filt, out, s, st, pl) : few_taps_launch<DCONV_F, 2, 4>(in, filt, out, s, st, pl);
    case 3: return pl.nw == 8 ? few_taps_launch<DCONV_F, 3, 8>(in, filt, out, s, st, pl) : few_taps_launch<DCONV_F, 3, 4>(in, filt, out, s, st, pl);
    case 4: return pl.nw == 8 ? few_taps_launch<DCONV_F, 4, 8>(in, filt, out, s, st, pl) : few_taps_launch<DCONV_F, 4, 4>(in, filt, out, s, st, pl);
    case 5: return few_taps_launch<DCONV_F, 5, 4>(in, filt, out, s, st, pl);
    case 6: return few_taps_launch<DCONV_F, 6, 4>(in, filt, out, s, st, pl);
    case 7: return few_taps_launch<DCONV_F, 7, 4>(in, filt, out, s, st, pl);
    default: return DCONV_UNSUPPORTED;
    }
}

}  // namespace dconv
