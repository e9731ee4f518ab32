// Whole segments of small fp32 models as one launch (xcd_device.h).
#include "xcd_device.h"

bool xcd_f32_fits(const Dims &d) {
    if (!xcd_shape_fits(d) || d.S > 5 || d.Dj % 8 || d.H % 8) return false;
    const long hb = (long)d.U * 2 * (d.R + 1) * d.N * f32_row(d.H) * 4;
    return hb < (1l << 31) && lds_of<true>(d).bytes <= XR_LDS(true);
}

int xcd_f32_lds_bytes(const Dims &d) { return lds_of<true>(d).bytes + XR_STATIC_LDS(true); }

bool xcd_f32_gates_stay(const Dims &d) { return lds_of<true>(d).wG >= 0; }

hipError_t launch_xcd_decode_f32(hipStream_t st, const XcdArgs &g) {
    if (!xcd_f32_fits(g.d) || !xcd_batch_fits(g) || g.push_step) return hipErrorInvalidValue;
    return g.d.N <= 7 ? xcd_launch<512, true, true>(st, g) : xcd_launch<768, false, true>(st, g);
}
