// C ABI of libdconv.so: argument validation and kernel dispatch.
#include "common.h"
#include "../../include/dconv.h"

using dconv::FewTapsPlan;
using dconv::GeneralWay;
using dconv::Shape;
using dconv::ShortChoice;
using dconv::TapsPlan;

namespace {

constexpr int64_t kMaxElems = 2147483647LL;

int validate(const void* in, const void* filt, const void* out,
             int N, int C, int H, int W, int K, int F, Shape* s)
{
    if (!in || !filt || !out) return DCONV_NULL_POINTER;
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || K <= 0 || F <= 0) return DCONV_BAD_SHAPE;
    if (F > H || F > W) return DCONV_BAD_SHAPE;
    const int Ho = H - F + 1, Wo = W - F + 1;
    // sizes are checked in floating point first so the int64 products below cannot overflow
    const double in_elems = (double)N * C * H * W;
    const double filt_elems = (double)K * C * F * F;
    const double img_out = (double)K * Ho * Wo;
    if (in_elems > (double)kMaxElems || filt_elems > (double)kMaxElems ||
        img_out > (double)kMaxElems || (double)N * img_out > 9.0e18)
        return DCONV_BAD_SHAPE;
    *s = Shape{N, C, H, W, K, F, Ho, Wo};
    return DCONV_OK;
}

// What DCONV_VARIANT_AUTO runs for a shape: a kernel of the single-channel case (`single`) or of the general one,
// by the variant that names it (TILED of the general case: whichever of the tiling kernels general_way_for says), and what
// its launch has use for of the estimates.
struct Route {
    int variant;
    bool single;
    FewTapsPlan few;
    TapsPlan taps;
    ShortChoice small;
    bool has_small;
    bool in_place_of_tiles;      // FEW_TAPS: of the general kernel's, not of the vector-ALU kernel
};

// By shape alone; `taps`: the kernel for few channels is among the choices.
Route auto_route(const Shape& s, bool single_entry, bool taps)
{
    Route r{DCONV_VARIANT_SIMPLE, single_entry, {}, {}, {1e300, 0}, false, false};
    auto small = [&]() {
        if (!r.has_small) r.small = dconv::short_choice(s);
        r.has_small = true;
        return r.small.time;
    };
    double channels = -1.0;                          // estimate of the kernel for few channels, once it is asked for
    auto few_channels = [&]() {
        if (channels < 0.0) channels = taps ? dconv::split_taps_time_if_preferred(s, &r.taps) : 1e300;
        return channels;
    };
    if (!single_entry) {
        // one channel is the special case, layouts included (a batch of images: its kernel takes
        // the images as further work items); the same kernel takes two to four channels with small filters: such
        // shapes are bound by the output stream like the one-channel case
        const bool one = s.N == 1 && s.C == 1;
        // (with up to sixteen filters the vector-ALU kernel of the general case goes first: up to
        // eight it is 2 to 10 times faster than a mostly padded matrix-core block of either kernel,
        // from nine on up to 2.8 times on layers of few channels; or the taps of all filters as rows of a product,
        // also in place of the general matrix-core kernel)
        if (!one && s.K <= 16) {
            const dconv::FewFilters few = dconv::few_filters_for(s);
            if (few.alu) {
                r.variant = few.taps < 1e300 ? DCONV_VARIANT_FEW_TAPS : DCONV_VARIANT_FEW_FILTERS;
                r.few = few.plan;
                return r;
            }
            r.single = dconv::single_batch_preferred(s) || (dconv::single_tiled_supports(s) && !dconv::general_tiled_supports(s));
            if (!r.single && few.taps < 1e300 && few.taps < few_channels() && few.taps < small()) {
                r.variant = DCONV_VARIANT_FEW_TAPS;
                r.in_place_of_tiles = true;
                r.few = few.plan;
                return r;
            }
        } else {
            r.single = one || dconv::single_batch_preferred(s) ||
                       (dconv::single_tiled_supports(s) && !dconv::general_tiled_supports(s));
        }
    }
    if (r.single && dconv::single_few_preferred(s)) {
        r.variant = DCONV_VARIANT_FEW_FILTERS;
        return r;
    }
    // (few channels, where that is estimated to be faster than the general kernels and small tiles)
    if (few_channels() < 1e300 && (r.single || few_channels() < small())) {
        r.variant = DCONV_VARIANT_FEW_CHANNELS;
        return r;
    }
    // (filters beyond the special case's 11 x 11: the general kernel takes one channel too;
    // so do narrow or short images and large filters, where it is the faster one)
    const bool tiled_ok = r.single && dconv::single_tiled_supports(s);
    if (r.single && (!tiled_ok || dconv::single_general_preferred(s)) && dconv::general_tiled_supports(s)) {
        r.single = false;
        r.variant = DCONV_VARIANT_TILED;
    } else if (tiled_ok || (!r.single && dconv::general_tiled_supports(s))) {
        r.variant = DCONV_VARIANT_TILED;
    }
    return r;
}

int launch_auto(bool single_entry, const float* in, const float* filt, float* out, const Shape& s, hipStream_t st,
                bool static_ws)
{
    Route r = auto_route(s, single_entry, true);
    if (r.variant == DCONV_VARIANT_FEW_CHANNELS) {
        if (!static_ws && r.taps.res && (!r.single || dconv::single_general_preferred(s))) dconv::bring_workspace(s, st);
        const int rc = dconv::launch_split_taps(in, filt, out, s, st, static_ws, r.taps);
        if (rc != DCONV_UNSUPPORTED) return rc;
        r = auto_route(s, single_entry, false);
    }
    switch (r.variant) {
    case DCONV_VARIANT_FEW_FILTERS:
        return r.single ? dconv::launch_single_few(in, filt, out, s, st) : dconv::launch_general_few(in, filt, out, s, st);
    case DCONV_VARIANT_FEW_TAPS:
        if (!static_ws && r.in_place_of_tiles) dconv::bring_workspace(s, st);
        return dconv::launch_few_taps(in, filt, out, s, st, r.few);
    case DCONV_VARIANT_TILED:
        return r.single ? dconv::launch_single_tiled(in, filt, out, s, st, -1)
                        : dconv::launch_general_tiled(in, filt, out, s, st, -1, static_ws, GeneralWay::kAuto,
                                                      r.has_small ? &r.small : nullptr);
    default: return dconv::launch_simple(in, filt, out, s, st);
    }
}

// A kernel by its name, whatever the estimates say.
int launch_named(bool single, const float* in, const float* filt, float* out, const Shape& s, int variant, hipStream_t st,
                 bool static_ws)
{
    const bool tiled_ok = single ? dconv::single_tiled_supports(s) : dconv::general_tiled_supports(s);
    auto tiled = [&](int cfg, GeneralWay way) {
        if (!tiled_ok) return (int)DCONV_UNSUPPORTED;
        return single ? dconv::launch_single_tiled(in, filt, out, s, st, cfg)
                      : dconv::launch_general_tiled(in, filt, out, s, st, cfg, static_ws, way);
    };
    switch (variant) {
    case DCONV_VARIANT_FEW_FILTERS:
        if (!single) return dconv::launch_general_few(in, filt, out, s, st);   // (refuses what it cannot run)
        if (!dconv::single_few_supports(s)) return DCONV_UNSUPPORTED;
        return dconv::launch_single_few(in, filt, out, s, st);
    case DCONV_VARIANT_SIMPLE: return dconv::launch_simple(in, filt, out, s, st);
    case DCONV_VARIANT_TILED: return tiled(-1, GeneralWay::kTiled);
    case DCONV_VARIANT_FEW_CHANNELS: return dconv::launch_split_taps(in, filt, out, s, st, static_ws, dconv::split_taps_plan(s));
    case DCONV_VARIANT_SHORT: return single ? DCONV_UNSUPPORTED : tiled(-1, GeneralWay::kShort);
    case DCONV_VARIANT_PARTS: return single ? DCONV_UNSUPPORTED : tiled(-1, GeneralWay::kParts);
    case DCONV_VARIANT_FEW_TAPS:
        return single ? DCONV_UNSUPPORTED : dconv::launch_few_taps(in, filt, out, s, st, dconv::make_few_taps_plan(s));
    default: break;
    }
    const int ncfg = single ? dconv::single_tile_configs() : dconv::general_tile_configs();
    if (variant >= DCONV_VARIANT_TILED_CFG0 && variant < DCONV_VARIANT_TILED_CFG0 + ncfg)
        return tiled(variant - DCONV_VARIANT_TILED_CFG0, GeneralWay::kTiled);
    return DCONV_UNSUPPORTED;
}

int general_entry(const float* in, int N, int C, int H, int W, const float* filt, int K, int F,
                  float* out, int variant, void* stream, bool static_ws)
{
    Shape s;
    const int rc = validate(in, filt, out, N, C, H, W, K, F, &s);
    if (rc != DCONV_OK) return rc;
    const hipStream_t st = (hipStream_t)stream;
    if (variant == DCONV_VARIANT_AUTO) return launch_auto(false, in, filt, out, s, st, static_ws);
    if (variant == DCONV_VARIANT_SPECIAL_CASE ||
        (variant >= DCONV_VARIANT_SPECIAL_CASE_CFG0 &&
         variant < DCONV_VARIANT_SPECIAL_CASE_CFG0 + dconv::single_tile_configs())) {
        if (!dconv::single_tiled_supports(s)) return DCONV_UNSUPPORTED;
        return launch_named(true, in, filt, out, s,
                            variant == DCONV_VARIANT_SPECIAL_CASE
                                ? DCONV_VARIANT_TILED
                                : variant - DCONV_VARIANT_SPECIAL_CASE_CFG0 + DCONV_VARIANT_TILED_CFG0,
                            st, false);
    }
    return launch_named(false, in, filt, out, s, variant, st, static_ws);
}

}  // namespace

extern "C" {

int dconv_single_channel_v(const float* img, int H, int W, const float* filt, int K, int F,
                           float* out, int variant, void* stream)
{
    Shape s;
    const int rc = validate(img, filt, out, 1, 1, H, W, K, F, &s);
    if (rc != DCONV_OK) return rc;
    const hipStream_t st = (hipStream_t)stream;
    return variant == DCONV_VARIANT_AUTO ? launch_auto(true, img, filt, out, s, st, false)
                                         : launch_named(true, img, filt, out, s, variant, st, false);
}

int dconv_general_v(const float* in, int N, int C, int H, int W, const float* filt, int K, int F,
                    float* out, int variant, void* stream)
{
    return general_entry(in, N, C, H, W, filt, K, F, out, variant, stream, false);
}

int dconv_general_noalloc(const float* in, int N, int C, int H, int W, const float* filt, int K, int F,
                          float* out, int variant, void* stream)
{
    return general_entry(in, N, C, H, W, filt, K, F, out, variant, stream, true);
}

int dconv_single_channel(const float* img, int H, int W, const float* filt, int K, int F,
                         float* out, void* stream)
{
    return dconv_single_channel_v(img, H, W, filt, K, F, out, DCONV_VARIANT_AUTO, stream);
}

int dconv_general(const float* in, int N, int C, int H, int W, const float* filt, int K, int F,
                  float* out, void* stream)
{
    return dconv_general_v(in, N, C, H, W, filt, K, F, out, DCONV_VARIANT_AUTO, stream);
}

int dconv_general_half_v(const void* in, int N, int C, int H, int W, const void* filt, int K, int F,
                         float* out, int dtype, int variant, void* stream)
{
    Shape s;
    const int rc = validate(in, filt, out, N, C, H, W, K, F, &s);
    if (rc != DCONV_OK) return rc;
    if (dtype != DCONV_DTYPE_F16 && dtype != DCONV_DTYPE_BF16) return DCONV_UNSUPPORTED;
    if ((((uintptr_t)in) & 1) != 0 || (((uintptr_t)filt) & 1) != 0) return DCONV_BAD_SHAPE;
    return dconv::launch_general_half(in, filt, out, s, (hipStream_t)stream, dtype,
                                      DCONV_LAYOUT_CHANNELS_LAST, variant);
}

int dconv_general_lowp(const void* in, int N, int C, int H, int W, const void* filt, int K, int F,
                       void* out, int dtype, int layout, int variant, void* stream)
{
    Shape s;
    const int rc = validate(in, filt, out, N, C, H, W, K, F, &s);
    if (rc != DCONV_OK) return rc;
    if (dtype != DCONV_DTYPE_I8 && ((((uintptr_t)in) & 1) != 0 || (((uintptr_t)filt) & 1) != 0))
        return DCONV_BAD_SHAPE;
    return dconv::launch_general_half(in, filt, (float*)out, s, (hipStream_t)stream, dtype, layout, variant);
}

int dconv_general_i8_v(const void* in, int N, int C, int H, int W, const void* filt, int K, int F,
                       int* out, int variant, void* stream)
{
    Shape s;
    const int rc = validate(in, filt, out, N, C, H, W, K, F, &s);
    if (rc != DCONV_OK) return rc;
    return dconv::launch_general_half(in, filt, (float*)out, s, (hipStream_t)stream, DCONV_DTYPE_I8,
                                      DCONV_LAYOUT_CHANNELS_LAST, variant);
}

int dconv_general_i8(const void* in, int N, int C, int H, int W, const void* filt, int K, int F,
                     int* out, void* stream)
{
    return dconv_general_i8_v(in, N, C, H, W, filt, K, F, out, DCONV_VARIANT_AUTO, stream);
}

int dconv_general_f16(const void* in, int N, int C, int H, int W, const void* filt, int K, int F,
                      float* out, void* stream)
{
    return dconv_general_half_v(in, N, C, H, W, filt, K, F, out, DCONV_DTYPE_F16, DCONV_VARIANT_AUTO, stream);
}

int dconv_general_bf16(const void* in, int N, int C, int H, int W, const void* filt, int K, int F,
                       float* out, void* stream)
{
    return dconv_general_half_v(in, N, C, H, W, filt, K, F, out, DCONV_DTYPE_BF16, DCONV_VARIANT_AUTO, stream);
}

const char* dconv_status_string(int status)
{
    switch (status) {
    case DCONV_OK: return "ok";
    case DCONV_NULL_POINTER: return "null pointer argument";
    case DCONV_BAD_SHAPE: return "bad shape";
    case DCONV_UNSUPPORTED: return "variant does not support this shape";
    case DCONV_LAUNCH_FAILED: return "kernel launch failed";
    case DCONV_SCRATCH_EXCEEDED: return "shape needs more scratch memory than the static device array holds";
    default: return "unknown status";
    }
}

int dconv_tile_config_count(int single_channel)
{
    return single_channel ? dconv::single_tile_configs() : dconv::general_tile_configs();
}

int dconv_tile_choice(int single_channel, int N, int C, int H, int W, int K, int F)
{
    Shape s;
    const int dummy = 0;       // (validate only tests its pointers against null)
    if (validate(&dummy, &dummy, &dummy, N, C, H, W, K, F, &s) != DCONV_OK ||
        (single_channel && (N != 1 || C != 1)))
        return DCONV_CHOICE_INVALID;
    // (the tiling kernels' own rules; which kernel runs is dconv_kernel_choice's answer)
    if (!single_channel && !(N == 1 && C == 1) && dconv::general_few_preferred(s)) return DCONV_CHOICE_FEW_FILTERS;
    const bool special = single_channel || (N == 1 && C == 1) || dconv::single_batch_preferred(s) ||
                         (dconv::single_tiled_supports(s) && !dconv::general_tiled_supports(s));
    if (special) {
        if (dconv::single_few_preferred(s)) return DCONV_CHOICE_FEW_FILTERS;
        if (!dconv::general_tiled_supports(s) && !dconv::single_tiled_supports(s)) return DCONV_CHOICE_SIMPLE;
        // (one channel on the general-case kernel: dconv_general names the tile shape it runs with)
        if (dconv::general_tiled_supports(s) &&
            (!dconv::single_tiled_supports(s) || dconv::single_general_preferred(s)))
            return single_channel ? DCONV_CHOICE_GENERAL_CASE : dconv::general_auto_shape(s);
        if (!single_channel) return DCONV_CHOICE_SPECIAL_CASE;
        return dconv::single_auto_config(s);
    }
    if (!dconv::general_tiled_supports(s)) return DCONV_CHOICE_SIMPLE;
    return dconv::general_auto_shape(s);
}

int dconv_kernel_choice(int single_channel, int N, int C, int H, int W, int K, int F)
{
    Shape s;
    const int dummy = 0;
    if (validate(&dummy, &dummy, &dummy, N, C, H, W, K, F, &s) != DCONV_OK ||
        (single_channel && (N != 1 || C != 1)))
        return DCONV_CHOICE_INVALID;
    const bool single = single_channel != 0;
    const Route r = auto_route(s, single, true);
    if (r.variant == DCONV_VARIANT_FEW_CHANNELS || r.variant == DCONV_VARIANT_SIMPLE) return r.variant;
    if (single && !r.single) return DCONV_CHOICE_GENERAL_CASE;
    if (r.single && !single) return r.variant == DCONV_VARIANT_TILED ? DCONV_VARIANT_SPECIAL_CASE : DCONV_VARIANT_AUTO;
    if (r.variant != DCONV_VARIANT_TILED || single) return r.variant;
    switch (dconv::general_way_for(s)) {
    case GeneralWay::kParts: return DCONV_VARIANT_PARTS;
    case GeneralWay::kShort: return DCONV_VARIANT_SHORT;
    default: return DCONV_VARIANT_TILED;
    }
}

int dconv_release_workspace(void)
{
    dconv::release_general_workspaces();
    return DCONV_OK;
}

int dconv_version(void) { return 1015; }

}  // extern "C"
