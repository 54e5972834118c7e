// Instantiation of the split-operand kernel of the general case for ONE filter side (DCONV_F, given
// on the compiler command line).
#include "split_kernel.h"

#ifndef DCONV_F
#error "compile with -DDCONV_F=<filter side>"
#endif

namespace dconv {

template <>
int split_launch_for_F<DCONV_F>(const float* in, const float* filt, float* out, const Shape& s,
                                hipStream_t st, const GenSched& sched)
{
    return split_try_launch<DCONV_F, split_image_rows(DCONV_F), split_phase_rows(DCONV_F)>(in, filt, out, s, st, sched);
}

}  // namespace dconv
