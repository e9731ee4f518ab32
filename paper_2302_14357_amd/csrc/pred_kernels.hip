// UpdatePredictorOutput of Algorithm 1: for every hypothesis created in this
// round, run the prediction network one step from its parent's recurrent state
// (Section 3.1: g(u) = predictor(y)).  A state gather builds the LSTM input rows
// (the embedding's share of the gates is a table), the gate pre-activations are
// one GEMM against W_hh (later layers: the concatenated [W_ih | W_hh] matrix), the cell update is a pointwise kernel, and
// the projection to the joint space is a GEMM that scatters into the state pool.
#include "tbs_internal.h"

__device__ __forceinline__ bf16_t f2bf_p(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

__device__ __forceinline__ float sigmoidf_(float x) { return 1.f / (1.f + expf(-x)); }

// The embedding half of the first layer's gates is a table made once (embed * W_ih^T + b for every
// token), so the first layer's input row of a new hypothesis is its parent's h.
//
// W_hh h is the same for every hypothesis made from one parent, and a round's new hypotheses have far fewer parents than they are
// many (N best of N x V expansions: 0.39 parents a new hypothesis for 256 utterances N = 10 S = 3, 0.48 for 1024 utterances S = 5,
// 0.13 to 0.56 elsewhere).  So the recurrent products run over the parents' rows, each once, and the cell update picks a pair's by
// pair_par (ms per decode 256 / 1024 utterances of the large widths: 135 / 286 -> 125 / 265).
// (The kernel takes the number of rows from device memory and leaves when launched beyond it: the
// host enqueues it on the largest possible grid before it knows the count.  It is bound by memory: a thread takes 16 bytes.)
template <int VEC>
__global__ void __launch_bounds__(256)
k_pred_gather_h(Dims d, int dtype, RowView rv, HidRows g) {
    const int j = blockIdx.x, l = blockIdx.y;
    if (j >= rv.counts[g.parents ? TBS_CNT_PARS : TBS_CNT_PAIRS]) return;
    const long slot = (g.parents ? rv.par_slot : rv.pair_pslot)[j];
    const float *src = g.pool_h + (l * g.pool_rows + slot) * d.H;
    const long dst = ((long)l * g.stride + j) * d.H;
    for (int i = threadIdx.x * VEC; i < d.H; i += blockDim.x * VEC) {
        if constexpr (VEC == 4) {
            const float4 v = *reinterpret_cast<const float4 *>(src + i);
            if (dtype == 1)
                *reinterpret_cast<uint2 *>((bf16_t *)g.out + dst + i) =
                    make_uint2(f2bf_p(v.x) | ((unsigned)f2bf_p(v.y) << 16), f2bf_p(v.z) | ((unsigned)f2bf_p(v.w) << 16));
            else *reinterpret_cast<float4 *>((float *)g.out + dst + i) = v;
        } else {
            if (dtype == 1) ((bf16_t *)g.out)[dst + i] = f2bf_p(src[i]);
            else ((float *)g.out)[dst + i] = src[i];
        }
    }
}

static int pred_threads(int units) { return units >= 256 ? 256 : (units + 63) / 64 * 64; }

hipError_t launch_pred_gather_h(hipStream_t st, const Dims &d, int dtype, int rows, RowView rv, const HidRows &g) {
    if (rows <= 0) return hipSuccess;
    const dim3 grid(rows, g.parents ? d.L : 1);
    if ((d.H & 3) == 0)
        hipLaunchKernelGGL(k_pred_gather_h<4>, grid, dim3(pred_threads(d.H / 4)), 0, st, d, dtype, rv, g);
    else
        hipLaunchKernelGGL(k_pred_gather_h<1>, grid, dim3(pred_threads(d.H)), 0, st, d, dtype, rv, g);
    return hipGetLastError();
}

// LSTM cell, gate order i, f, g, o.  A workgroup per pair, VEC units a thread, everything it reads requested at once.
// (Workgroups go to the XCDs in turn: an XCD takes an eighth of the pairs in a row, so that hypotheses of one parent find its gates
// and cell state in their L2.)
template <int VEC>
__global__ void __launch_bounds__(256)
k_lstm_pointwise(Dims d, int dtype, int layer, int pairs, RowView rv, CellIn in, float *pool_h, float *pool_c, long pool_rows) {
    const int per = (pairs + 7) >> 3, j = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (j >= pairs || ((int)blockIdx.x >> 3) >= per) return;
    const long ps = rv.pair_pslot[j], ns = rv.pair_slot[j];   // parent's and own state slot
    const float *ga = in.ga + (long)(in.ga_row ? in.ga_row[j] : j) * 4 * d.H;
    const float *gb = in.gb ? in.gb + (long)(in.gb_row ? in.gb_row[j] : j) * 4 * d.H : nullptr;
    const float *c_par = pool_c + ((long)layer * pool_rows + ps) * d.H;
    float *c_new = pool_c + ((long)layer * pool_rows + ns) * d.H;
    float *h_new = pool_h + ((long)layer * pool_rows + ns) * d.H;
    const float *hp = in.h_par_next ? in.h_par_next + ps * d.H : nullptr;
    const long out = (long)j * d.H * (hp ? 2 : 1);
    for (int i = threadIdx.x * VEC; i < d.H; i += blockDim.x * VEC) {
        float x[4][VEC], y[4][VEC], c[VEC], h[VEC], hv[VEC];
        auto load = [](float (&v)[VEC], const float *p) {
            if constexpr (VEC == 4) {
                const float4 q = *reinterpret_cast<const float4 *>(p);
                v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
            } else {
                v[0] = *p;
            }
        };
        auto store16 = [&](long at, const float (&v)[VEC]) {   // (a row of the next product's input, in the model's type)
            if constexpr (VEC == 4) {
                if (dtype == 1)
                    *reinterpret_cast<uint2 *>((bf16_t *)in.out + at) =
                        make_uint2(f2bf_p(v[0]) | ((unsigned)f2bf_p(v[1]) << 16), f2bf_p(v[2]) | ((unsigned)f2bf_p(v[3]) << 16));
                else *reinterpret_cast<float4 *>((float *)in.out + at) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
                if (dtype == 1) ((bf16_t *)in.out)[at] = f2bf_p(v[0]);
                else ((float *)in.out)[at] = v[0];
            }
        };
#pragma unroll
        for (int q = 0; q < 4; ++q) load(x[q], ga + q * d.H + i);
        if (gb) {   // (uniform)
#pragma unroll
            for (int q = 0; q < 4; ++q) load(y[q], gb + q * d.H + i);
        }
        load(c, c_par + i);
        if (hp) load(hv, hp + i);
        if (gb) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int k = 0; k < VEC; ++k) x[q][k] += y[q][k];
        }
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            const float ig = sigmoidf_(x[0][k]), fg = sigmoidf_(x[1][k]), gg = tanhf(x[2][k]), og = sigmoidf_(x[3][k]);
            c[k] = fg * c[k] + ig * gg;
            h[k] = og * tanhf(c[k]);
        }
        if constexpr (VEC == 4) {
            *reinterpret_cast<float4 *>(c_new + i) = make_float4(c[0], c[1], c[2], c[3]);
            *reinterpret_cast<float4 *>(h_new + i) = make_float4(h[0], h[1], h[2], h[3]);
        } else {
            c_new[i] = c[0];
            h_new[i] = h[0];
        }
        store16(out + i, h);
        if (hp) store16(out + d.H + i, hv);
    }
}

hipError_t launch_lstm_pointwise(hipStream_t st, const Dims &d, int dtype, int pairs, int layer, RowView rv, const CellIn &in,
                                 float *pool_h, float *pool_c, long pool_rows) {
    if (pairs <= 0) return hipSuccess;
    const dim3 grid((pairs + 7) / 8 * 8);
    if ((d.H & 3) == 0)
        hipLaunchKernelGGL(k_lstm_pointwise<4>, grid, dim3(pred_threads(d.H / 4)), 0, st, d, dtype, layer, pairs, rv, in, pool_h,
                           pool_c, pool_rows);
    else
        hipLaunchKernelGGL(k_lstm_pointwise<1>, grid, dim3(pred_threads(d.H)), 0, st, d, dtype, layer, pairs, rv, in, pool_h,
                           pool_c, pool_rows);
    return hipGetLastError();
}

// wcat[r, :] = [ w_ih[r, 0:in] | w_hh[r, 0:hid] ], elements of 2 bytes
__global__ void k_concat16(const uint16_t *w_ih, const uint16_t *w_hh, uint16_t *wcat, int rows, int in_dim,
                           int hid) {
    long W = in_dim + hid;
    long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * W) return;
    long r = idx / W, c = idx % W;
    wcat[idx] = c < in_dim ? w_ih[r * in_dim + c] : w_hh[r * hid + (c - in_dim)];
}
__global__ void k_concat32(const uint32_t *w_ih, const uint32_t *w_hh, uint32_t *wcat, int rows, int in_dim,
                           int hid) {
    long W = in_dim + hid;
    long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * W) return;
    long r = idx / W, c = idx % W;
    wcat[idx] = c < in_dim ? w_ih[r * in_dim + c] : w_hh[r * hid + (c - in_dim)];
}

hipError_t launch_concat_weights(hipStream_t st, int elem_bytes, const void *w_ih, const void *w_hh, void *wcat,
                                 int rows, int in_dim, int hid) {
    long n = (long)rows * (in_dim + hid);
    unsigned blocks = (unsigned)((n + 255) / 256);
    if (elem_bytes == 2)
        hipLaunchKernelGGL(k_concat16, dim3(blocks), dim3(256), 0, st, (const uint16_t *)w_ih, (const uint16_t *)w_hh,
                           (uint16_t *)wcat, rows, in_dim, hid);
    else
        hipLaunchKernelGGL(k_concat32, dim3(blocks), dim3(256), 0, st, (const uint32_t *)w_ih, (const uint32_t *)w_hh,
                           (uint32_t *)wcat, rows, in_dim, hid);
    return hipGetLastError();
}

// dst row 4j+g = src row g*H+j (rows of row_bytes bytes, a multiple of 4): the gate-interleaved
// order the fused gate GEMM wants
__global__ void k_permute_gate_rows(const uint32_t *src, uint32_t *dst, int H, long row_words) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= 4L * H * row_words) return;
    const long r = idx / row_words, w = idx % row_words;
    const long j = r >> 2, g = r & 3;
    dst[idx] = src[(g * H + j) * row_words + w];
}

hipError_t launch_permute_gate_rows(hipStream_t st, const void *src, void *dst, int H, long row_bytes) {
    const long words = row_bytes / 4, n = 4L * H * words;
    hipLaunchKernelGGL(k_permute_gate_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const uint32_t *)src,
                       (uint32_t *)dst, H, words);
    return hipGetLastError();
}

// ------------------------------------------------------------------ streaming: frame buffer
// Copies whole frames (rows) between the caller's array, the per-utterance frame buffers and
// the spare area used to move leftovers to the front.  UNIT = 16 or 4 bytes.
template <typename UNIT>
__global__ void k_stream_copy(int U, const UNIT *__restrict__ src, UNIT *__restrict__ dst, const int *__restrict__ desc,
                              long row_units) {
    const int u = blockIdx.x;
    const long s0 = (long)desc[u] * row_units, d0 = (long)desc[U + u] * row_units;
    const long total = (long)desc[2 * U + u] * row_units;
    for (long i = (long)blockIdx.y * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.y * blockDim.x)
        dst[d0 + i] = src[s0 + i];
}

hipError_t launch_stream_copy(hipStream_t st, int U, const void *src, void *dst, const int *desc, long row_bytes) {
    if (U <= 0) return hipSuccess;
    const bool wide = row_bytes % 16 == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0 &&
                      (reinterpret_cast<uintptr_t>(dst) & 15) == 0;
    const dim3 grid(U, 4), block(256);
    if (wide)
        hipLaunchKernelGGL(k_stream_copy<uint4>, grid, block, 0, st, U, (const uint4 *)src, (uint4 *)dst, desc,
                           row_bytes / 16);
    else
        hipLaunchKernelGGL(k_stream_copy<unsigned>, grid, block, 0, st, U, (const unsigned *)src, (unsigned *)dst, desc,
                           row_bytes / 4);
    return hipGetLastError();
}

// ------------------------------------------------------------------ padding of the logit rows
__global__ void k_logit_pads(float *logits, long rows, int V, int Vl) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int pad = Vl - V;
    if (i < rows * pad) logits[(i / pad) * Vl + V + i % pad] = -INFINITY;
}
hipError_t launch_logit_pads(hipStream_t st, float *logits, long rows, int V, int Vl) {
    if (Vl <= V || rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_logit_pads, dim3((unsigned)((rows * (Vl - V) + 255) / 256)), dim3(256), 0, st, logits, rows, V, Vl);
    return hipGetLastError();
}

// ------------------------------------------------------------------ timing yardstick
__global__ void k_empty() {}
hipError_t launch_empty(hipStream_t st) {
    hipLaunchKernelGGL(k_empty, dim3(1), dim3(64), 0, st);
    return hipGetLastError();
}
