// Whole segments of small bf16 models as one launch (xcd_device.h).
#include "xcd_device.h"

bool xcd_fits(const Dims &d) {
    if (!xcd_shape_fits(d) || d.Dj % 128 || d.H % 128) return false;
    const long hb = (long)d.U * 2 * (d.R + 1) * d.N * d.H * 2;   // (offsets into it are 32 bits)
    return hb < (1l << 31) && lds_of<false>(d).bytes <= XR_LDS(d.N > 7);
}

hipError_t launch_xcd_decode(hipStream_t st, const XcdArgs &g) {
    if (!xcd_fits(g.d) || !xcd_batch_fits(g)) return hipErrorInvalidValue;
    if (g.d.S > 5) return launch_xcd_decode_long(st, g);
    return g.d.N <= 7 ? xcd_launch<512, true, false>(st, g) : xcd_launch<768, false, false>(st, g);
}
