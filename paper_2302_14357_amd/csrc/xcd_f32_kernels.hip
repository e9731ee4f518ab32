// Whole segments of small fp32 models as one launch (xcd_device.h).
#include "xcd_device.h"

int xcd_f32_row(int K) { return f32_row(K); }
long xcd_f32_frags(int rows, int K) { return (long)((rows + 15) / 16) * f32_pieces(K) * 256; }

bool xcd_f32_fits(const Dims &d) {
    if (!xcd_shape_fits(d) || d.S > 5 || d.Dj % 8 || d.H % 8) return false;
    const long hb = (long)d.U * 2 * (d.R + 1) * d.N * f32_row(d.H) * 4;
    return hb < (1l << 31) && lds_of<true>(d).bytes <= XR_LDS(true);
}

hipError_t launch_xcd_decode_f32(hipStream_t st, const XcdArgs &g) {
    if (!xcd_f32_fits(g.d) || !xcd_batch_fits(g)) return hipErrorInvalidValue;
    return g.d.N <= 7 ? xcd_launch<512, true, true>(st, g) : xcd_launch<768, false, true>(st, g);
}

// A weight matrix [rows, K] in the pieces that the products read: tile of 16 rows, piece of 16 columns, lane, 4 floats
__global__ void k_xcd_frags(const float *w, float *frags, int rows, int K, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int pieces = f32_pieces(K), j = (int)(i & 3), l = (int)(i >> 2) & 63;
    const long tm = i >> 8;
    const int m = (int)(tm % pieces), row = min((int)(tm / pieces) * 16 + (l & 15), rows - 1), q = l >> 4;
    const int k = m * 16 + (j >> 1) * 8 + (q & 1) * 4 + (q & 2) + (j & 1);
    frags[i] = k < K ? w[(long)row * K + k] : 0.f;
}

hipError_t launch_xcd_frags(hipStream_t st, const float *w, float *frags, int rows, int K) {
    const long n = xcd_f32_frags(rows, K);
    hipLaunchKernelGGL(k_xcd_frags, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w, frags, rows, K, n);
    return hipGetLastError();
}
