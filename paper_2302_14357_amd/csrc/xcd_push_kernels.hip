// A push of a stream as one launch (xcd_device.h), small bf16 models; what fits and what does not is checked by launch_xcd_decode.
#include "xcd_device.h"

hipError_t launch_xcd_push(hipStream_t st, const XcdArgs &g) {
    if (g.seg1 != g.seg0 + 1) return hipErrorInvalidValue;
    return g.d.N <= 7 ? xcd_launch<512, true, false, true>(st, g) : xcd_launch<768, false, false, true>(st, g);
}
