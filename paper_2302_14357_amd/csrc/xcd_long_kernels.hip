// Whole segments of 6 to 64 frames as one launch (bf16 models, xcd_device.h).
#include "xcd_device.h"

template <int NV4>
static hipError_t xcd_launch_long(hipStream_t st, const XcdArgs &g, int shm) {
    if (g.d.S <= 16) return xcd_launch_t<512, NV4, 16, true, false>(st, g, shm);
    if (g.d.S <= 32) return xcd_launch_t<512, NV4, 32, true, false>(st, g, shm);
    return xcd_launch_t<512, NV4, 64, true, false>(st, g, shm);
}

hipError_t launch_xcd_decode_long(hipStream_t st, const XcdArgs &g) {
    if (g.push_step) return hipErrorInvalidValue;
    const int nv4 = nv4_of(g.d), shm = lds_of<false>(g.d).bytes;
    if (nv4 == 1) return xcd_launch_long<1>(st, g, shm);
    if (nv4 == 2) return xcd_launch_long<2>(st, g, shm);
    return xcd_launch_long<4>(st, g, shm);
}
