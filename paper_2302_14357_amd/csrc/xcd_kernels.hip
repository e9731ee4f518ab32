// Whole segments of small bf16 models as one launch (xcd_device.h).
#include "xcd_device.h"

bool xcd_fits(const Dims &d) {
    if (!xcd_shape_fits(d) || d.Dj % 128 || d.H % 128) return false;
    const long hb = (long)d.U * 2 * (d.R + 1) * d.N * d.H * 2;   // (offsets into it are 32 bits)
    return hb < (1l << 31) && lds_of<false>(d).bytes <= XR_LDS(d.N > 7);
}

hipError_t launch_xcd_decode(hipStream_t st, const XcdArgs &g) {
    if (!xcd_fits(g.d) || !xcd_batch_fits(g)) return hipErrorInvalidValue;
    if (g.d.S > 5) return g.push_step ? hipErrorInvalidValue : launch_xcd_decode_long(st, g);
    if (g.push_step) return launch_xcd_push(st, g);
    return g.d.N <= 7 ? xcd_launch<512, true, false>(st, g) : xcd_launch<768, false, false>(st, g);
}

// ------------------------------------------------------------------ both types
// (asked by a CPU test that runs the barrier in every order)
extern "C" int xcd_barrier_reads(u64 word, unsigned due, unsigned seen, int live) { return xcd_barrier_read(word, due, seen, live != 0); }

int xcd_lds_bytes(int dtype, const Dims &d) { return dtype == 1 ? lds_of<false>(d).bytes + XR_STATIC_LDS(d.N > 7) : xcd_f32_lds_bytes(d); }
long xcd_row_bytes(int dtype, int K) { return dtype == 1 ? 2l * K : 4l * f32_row(K); }
long xcd_frag_bytes(int dtype, int rows, int K) { return (long)((rows + 15) / 16) * 16 * xcd_row_bytes(dtype, K); }

// A weight matrix [rows, K] in the pieces that the products read: tile of 16 rows, piece, lane, 16 bytes
__global__ void k_xcd_frags(int f32, const void *w, void *frags, int rows, int K, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int pieces = f32 ? f32_pieces(K) : K >> 5, l = (int)i & 63;
    const long tm = i >> 6;
    const int m = (int)(tm % pieces), row = min((int)(tm / pieces) * 16 + (l & 15), rows - 1), q = l >> 4;
    if (f32) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        const int k = m * 16 + (q & 1) * 4 + (q & 2);
        const float *src = static_cast<const float *>(w) + (long)row * K;
        if (k < K) v.x = src[k], v.y = src[k + 1];           // (K is a multiple of 8)
        if (k + 8 < K) v.z = src[k + 8], v.w = src[k + 9];
        static_cast<float4 *>(frags)[i] = v;
    } else {
        static_cast<uint4 *>(frags)[i] = *reinterpret_cast<const uint4 *>(static_cast<const bf16_t *>(w) + (long)row * K + m * 32 + q * 8);
    }
}

hipError_t launch_xcd_frags(hipStream_t st, int dtype, const void *w, void *frags, int rows, int K) {
    const long n = xcd_frag_bytes(dtype, rows, K) / 16;
    hipLaunchKernelGGL(k_xcd_frags, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, dtype == 0, w, frags, rows, K, n);
    return hipGetLastError();
}
