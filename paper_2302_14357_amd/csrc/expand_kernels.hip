// Expansion scores of token-wise RNN-T beam search (Eq. 3-7) for every live
// hypothesis of a joiner call, and its N best non-blank expansions.
//
// One workgroup owns one (utterance, hypothesis) pair, i.e. the S' logit rows
// of that hypothesis.  Softmax probabilities are never formed: with row
// maximum m_t, row sum Z_t = sum_k exp(l[t,k]-m_t) and blank probability b_t,
// the blank products of Eq. 3 collapse into a forward variable
//     alpha_1 = d_old[1],  alpha_t = alpha_{t-1} b_{t-1} + d_old[t]
// (alpha_t = sum_{t1<=t} d_old[t1] Bl(t1,t)), so that
//     delta_blank   = alpha_S' b_S'                                  (Eq. 7; handed on as its logarithm)
//     d[k][t]       = alpha_t exp(l[t,k]-m_t) / Z_t                   (Eq. 4-5)
//     delta_nb[k]   = sum_t d[k][t] = sum_t exp(l[t,k] + lc_t)        (Eq. 6)
// with lc_t = log(alpha_t / Z_t) - m_t.  The [S+1,S+1] table, the [V,S] tensor
// d and the normalised J are never built; the logits are streamed from memory
// and each costs one exp and one add.
#include "tbs_internal.h"

#include "expand_device.h"

__global__ void __launch_bounds__(EXP_THREADS)
k_expand(Dims d, const float *__restrict__ logits, AView A, RowView rv, float *__restrict__ row_lc,
         float *__restrict__ dphi, float *__restrict__ cand_score, int *__restrict__ cand_tok,
         float *__restrict__ row_stats, float *__restrict__ delta_nb, const int *__restrict__ pairs_dev,
         int pair_base) {
    extern __shared__ __attribute__((aligned(16))) float s_dnb[];  // [Vl]
    __shared__ float s_m[TBS_MAX_SEG], s_z[TBS_MAX_SEG], s_b[TBS_MAX_SEG], s_lc[TBS_MAX_SEG];
    __shared__ float s_rv[EXP_WAVES];
    __shared__ int s_rk[EXP_WAVES];
    const int pair = pair_base + blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (pairs_dev && pair >= *pairs_dev) return;   // (enqueued on an upper-bound grid, see k_expand_reg)
    const int u = rv.pair_u[pair], h = rv.pair_h[pair];
    const int row0 = rv.pair_row0[pair], sp = rv.pair_len[pair];
    const int V = d.V, Vl = d.Vl;   // (the columns past V hold -inf: they add nothing and score 0)
    const float *L = logits + (long)row0 * Vl;

    // ---- softmax statistics of each row: one wave per row, no barriers inside
    for (int t = wave; t < sp; t += EXP_WAVES) {
        const float4 *r4 = reinterpret_cast<const float4 *>(L + (long)t * Vl);
        float m = -INFINITY, z = 0.f;
        for (int i = lane; i < Vl / 4; i += 64) {
            float4 x = r4[i];
            float mx = fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w));
            float mn = fmaxf(m, mx);
            z = z * __expf(m - mn) + __expf(x.x - mn) + __expf(x.y - mn) + __expf(x.z - mn) + __expf(x.w - mn);
            m = mn;
        }
        for (int off = 32; off > 0; off >>= 1) {
            float m2 = __shfl_xor(m, off), z2 = __shfl_xor(z, off);
            ms_combine(m, z, m2, z2);
        }
        if (lane == 0) {
            s_m[t] = m;
            s_z[t] = z;
            s_b[t] = __expf(L[(long)t * Vl + d.blank] - m) / z;
        }
    }
    __syncthreads();

    // ---- forward variable over the segment (Eq. 3 folded into a scan) and Eq. 7
    if (tid == 0) {
        const float *dold = A.dhat + ((long)u * d.N + h) * d.S;
        ScanAlpha al;
        al.start();
        for (int t = 0; t < sp; ++t) {
            al.step(t == 0 ? 0.f : s_b[t - 1], dold[t]);
            float lc = al.log_value() - __logf(s_z[t]) - s_m[t];   // log(alpha_t / Z_t) - m_t, no underflow
            s_lc[t] = lc;
            row_lc[row0 + t] = lc;
            if (row_stats) {
                row_stats[(long)(row0 + t) * 3 + 0] = s_m[t];
                row_stats[(long)(row0 + t) * 3 + 1] = s_z[t];
                row_stats[(long)(row0 + t) * 3 + 2] = s_b[t];
            }
        }
        dphi[pair] = al.log_times(s_b[sp - 1]);
    }
    __syncthreads();

    // ---- Eq. 4-6: delta_nb[k] = sum_t exp(l[t,k] + lc_t), streamed
    for (int i = tid; i < Vl / 4; i += EXP_THREADS) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int t = 0; t < sp; ++t) {
            float4 x = reinterpret_cast<const float4 *>(L + (long)t * Vl)[i];
            float lc = s_lc[t];
            acc.x += __expf(x.x + lc);
            acc.y += __expf(x.y + lc);
            acc.z += __expf(x.z + lc);
            acc.w += __expf(x.w + lc);
        }
        reinterpret_cast<float4 *>(s_dnb)[i] = acc;
    }
    __syncthreads();
    if (tid == 0) s_dnb[d.blank] = 0.f;  // blank is not a non-blank expansion
    __syncthreads();
    if (delta_nb)
        for (int k = tid; k < V; k += EXP_THREADS) delta_nb[(long)pair * V + k] = s_dnb[k];

    // ---- the N best expansions of this hypothesis: N rounds of workgroup arg-max
    for (int n = 0; n < d.N; ++n) {
        float bv = 0.f;  // only strictly positive scores are candidates
        int bk = 0x7fffffff;
        for (int k = tid; k < V; k += EXP_THREADS) {
            float v = s_dnb[k];
            if (v > bv) { bv = v; bk = k; }  // ascending k: the smallest token wins a tie
        }
        for (int off = 32; off > 0; off >>= 1) {
            float ov = __shfl_xor(bv, off);
            int ok = __shfl_xor(bk, off);
            if (ov > bv || (ov == bv && ok < bk)) { bv = ov; bk = ok; }
        }
        if (lane == 0) { s_rv[wave] = bv; s_rk[wave] = bk; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < EXP_WAVES; ++w)
                if (s_rv[w] > bv || (s_rv[w] == bv && s_rk[w] < bk)) { bv = s_rv[w]; bk = s_rk[w]; }
            if (bk != 0x7fffffff) {
                cand_score[(long)pair * d.N + n] = __logf(bv);
                cand_tok[(long)pair * d.N + n] = bk;
                s_dnb[bk] = -1.f;
            } else {
                cand_score[(long)pair * d.N + n] = -INFINITY;
                cand_tok[(long)pair * d.N + n] = -1;
            }
        }
        __syncthreads();
    }
}

template <int NV4, int SMAX>
__global__ void __launch_bounds__(EXP_THREADS, (NV4 * SMAX == 20 ? 5 : 1))   // 80 logits per thread: five waves per SIMD still fit
k_expand_reg(Dims d, const float *__restrict__ logits, AView A, RowView rv, float *__restrict__ row_lc,
             float *__restrict__ dphi, float *__restrict__ cand_score, int *__restrict__ cand_tok,
             float *__restrict__ row_stats, float *__restrict__ delta_nb, const int *__restrict__ pairs_dev,
             int pair_base) {
    __shared__ ExpandShared<SMAX, EXP_WAVES> sm;
    // Workgroup b runs on XCD b % 8.  The joiner GEMM before this kernel gave XCD x the x-th eighth
    // of the rows, in increasing order; here XCD x walks the pairs of the same eighth backwards, so
    // that what it reads first is what was written last (still in its L2 and in the memory-side
    // cache) and is read before this kernel's own traffic evicts it.  Measured: 196 -> 184 us at
    // 51200 rows x 4096.
    // (eighth x holds as many pairs as there are workgroups with b % 8 == x: every pair gets one)
    // (pairs_dev not null: the launch went out before the host knew the number of pairs; the grid is
    // an upper bound and the workgroups beyond the count in device memory leave)
    // (pair_base: the grid covers the pairs pair_base .. pair_base + gridDim.x - 1, one piece of a
    // large call, joined by a GEMM launch of its own over exactly these pairs' rows)
    int pair = blockIdx.x;
    if (pairs_dev) {
        if (pair >= *pairs_dev) return;
    } else {
        const int pairs = gridDim.x, q = pairs >> 3, r = pairs & 7, x = blockIdx.x & 7;
        const int first = x * q + min(x, r), count = q + (x < r);
        pair = first + count - 1 - (int)(blockIdx.x >> 3);
    }
    pair += pair_base;
    ExpandPair<SMAX> pi;
    expand_pair_info(pi, pair, d, A, rv, logits);
    float e[SMAX][NV4 * 4];
    expand_load<NV4, SMAX, EXP_THREADS>(e, logits, pi.row0, pi.sp, d.Vl, (int)threadIdx.x);
    expand_pair<NV4, SMAX, EXP_THREADS>(e, pi, sm, d, (int)threadIdx.x, true, row_lc + pi.row0, dphi + pi.pair,
                                        cand_score + (long)pi.pair * d.N, cand_tok + (long)pi.pair * d.N, row_stats,
                                        delta_nb);
}

// ------------------------------------------------------------------ long segments
// Segments too long for the registers of four waves: a wave takes whole rows (up to RPW of them, NQ
// 16-byte pieces a lane and row), so a row's maximum and sum never leave its wave and every logit is
// read from memory and exponentiated once.  The forward variable of Eq. 3 is a chain of S' steps; here it is
// a prefix scan over the lanes of one wave, alpha_t = alpha_{t-1} b_{t-1} + d_old[t] as the composition
// of the maps x -> x B + A, which takes log2(S') steps instead.  A and B are kept as mantissa * 2^exponent
// (see ScanAlpha: the products leave the range of float).  The waves' shares of delta_nb (Eq. 6) meet in LDS,
// and the first four waves take the N best.
struct ScanPart {
    float m;   // mantissa in [0.5, 1), or 0
    int e;
};
__device__ __forceinline__ ScanPart scan_norm(float m, int e) {
    int k;
    m = frexpf(m, &k);
    return {m, m != 0.f ? e + k : 0};
}
__device__ __forceinline__ ScanPart scan_mul(ScanPart a, ScanPart b) { return scan_norm(a.m * b.m, a.e + b.e); }
__device__ __forceinline__ ScanPart scan_add(ScanPart a, ScanPart b) {
    if (a.m == 0.f) return b;
    if (b.m == 0.f) return a;
    const int e = max(a.e, b.e);
    return scan_norm(ldexpf(a.m, a.e - e) + ldexpf(b.m, b.e - e), e);
}
__device__ __forceinline__ ScanPart scan_up(ScanPart a, int by) { return {__shfl_up(a.m, by), __shfl_up(a.e, by)}; }
__device__ __forceinline__ float scan_log(ScanPart a) {
    return a.m > 0.f ? __logf(a.m) + (float)a.e * 0.69314718055994531f : -INFINITY;
}
// 2^l2 / z; zero for l2 = -inf
__device__ __forceinline__ ScanPart scan_exp2(float l2, float z) {
    if (!(l2 > -INFINITY)) return {0.f, 0};
    const float fl = floorf(l2);
    return scan_norm(__builtin_amdgcn_exp2f(l2 - fl) / z, (int)fl);
}

#define LONG_FRAMES 64     // a lane per frame in the scan
#define LONG_MIN_WAVES 4   // the N best are taken by the first four waves
template <int NQ, int RPW>
__global__ void __launch_bounds__(1024)
k_expand_long(Dims d, const float *__restrict__ logits, AView A, RowView rv, float *__restrict__ row_lc,
              float *__restrict__ dphi, float *__restrict__ cand_score, int *__restrict__ cand_tok,
              float *__restrict__ row_stats, float *__restrict__ delta_nb, const int *__restrict__ pairs_dev,
              int pair_base) {
    extern __shared__ __attribute__((aligned(16))) float4 s_part[];   // [waves][Vl / 4]
    __shared__ ExpandBest<EXP_WAVES> sm;
    __shared__ float s_m[LONG_FRAMES], s_z[LONG_FRAMES], s_lb[LONG_FRAMES], s_cf[LONG_FRAMES];
    const int pair = pair_base + blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)blockDim.x >> 6;
    if (pairs_dev && pair >= *pairs_dev) return;   // (enqueued on an upper-bound grid, see k_expand_reg)
    const int u = ((cint_p)rv.pair_u)[pair], h = ((cint_p)rv.pair_h)[pair];
    const int row0 = ((cint_p)rv.pair_row0)[pair], sp = ((cint_p)rv.pair_len)[pair];
    const int V = d.V, Vl = d.Vl, V4 = Vl >> 2;
    const float *L = logits + (long)row0 * Vl;
    // this wave's rows: wave, wave + waves, ... (rows past S' repeat the last one, pieces past V the last piece)
    float4 e[RPW][NQ];
    float lblank[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const float *row = L + (long)min(wave + i * waves, sp - 1) * Vl;
#pragma unroll
        for (int q = 0; q < NQ; ++q) e[i][q] = reinterpret_cast<const float4 *>(row)[min(lane + 64 * q, V4 - 1)];
        lblank[i] = row[d.blank];
    }
    const float ld = wave == 0 ? A.dhat[((long)u * d.N + h) * d.S + min(lane, d.S - 1)] : 0.f;
    if (tid == 0) sm.jn = 0;
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int t = wave + i * waves;
        if (t >= sp) continue;   // (uniform)
        float m = -INFINITY;
#pragma unroll
        for (int q = 0; q < NQ; ++q) m = fmaxf(m, fmaxf(fmaxf(e[i][q].x, e[i][q].y), fmaxf(e[i][q].z, e[i][q].w)));
        m = wave_max_ord(m);
        const float nm = -m * 1.44269504088896341f;
        float z = 0.f;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            float4 &x = e[i][q];
            x.x = __builtin_amdgcn_exp2f(fmaf(x.x, 1.44269504088896341f, nm));
            x.y = __builtin_amdgcn_exp2f(fmaf(x.y, 1.44269504088896341f, nm));
            x.z = __builtin_amdgcn_exp2f(fmaf(x.z, 1.44269504088896341f, nm));
            x.w = __builtin_amdgcn_exp2f(fmaf(x.w, 1.44269504088896341f, nm));
            if (lane + 64 * q < V4) z += (x.x + x.y) + (x.z + x.w);
        }
        z = wave_sum(z);
        if (lane == 0) {
            s_m[t] = m;
            s_z[t] = z;
            s_lb[t] = fmaf(lblank[i], 1.44269504088896341f, nm);   // (log2 of the blank's e: with the row's common factor, see expand_pair)
        }
    }
    __syncthreads();
    if (wave == 0) {   // lane t: frame t
        const bool have = lane < sp;
        const int t = min(lane, sp - 1);
        const float m = s_m[t], z = s_z[t];
        const ScanPart b = scan_exp2(s_lb[t], z);             // blank probability of the frame
        ScanPart a = scan_exp2(have ? ld * 1.44269504088896341f : -INFINITY, 1.f), f = scan_up(b, 1);   // alpha_t = alpha_{t-1} f + a
        for (int by = 1; by < sp; by <<= 1) {
            const ScanPart a2 = scan_up(a, by), f2 = scan_up(f, by);
            if (lane >= by) {
                a = scan_add(scan_mul(a2, f), a);
                f = scan_mul(f2, f);
            }
        }
        const float lc = scan_log(a) - __logf(z);             // log(alpha_t / Z_t)
        if (have) {
            s_cf[t] = __expf(lc);
            row_lc[row0 + t] = fmaf(-m * 1.44269504088896341f, 0.69314718055994531f, lc);
            if (lane == sp - 1) dphi[pair] = scan_log(scan_mul(a, b));   // Eq. 7
            if (row_stats) {
                row_stats[(long)(row0 + t) * 3 + 0] = m;
                row_stats[(long)(row0 + t) * 3 + 1] = z;
                row_stats[(long)(row0 + t) * 3 + 2] = ldexpf(b.m, b.e);
            }
        }
    }
    __syncthreads();
    {   // this wave's share of Eq. 4-6
        float4 acc[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int t = wave + i * waves;
            if (t >= sp) continue;   // (uniform)
            const float cf = s_cf[t];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                acc[q].x += cf * e[i][q].x;
                acc[q].y += cf * e[i][q].y;
                acc[q].z += cf * e[i][q].z;
                acc[q].w += cf * e[i][q].w;
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (lane + 64 * q < V4) s_part[wave * V4 + lane + 64 * q] = acc[q];
    }
    __syncthreads();
    if (wave >= EXP_WAVES) {
        __syncthreads();   // (the barrier inside expand_best)
        return;
    }
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (tid < V4) {
        const int shares = min(waves, sp);   // (a wave beyond S' had no row)
        for (int w = 0; w < shares; ++w) {
            const float4 x = s_part[w * V4 + tid];
            v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int col = 4 * tid + c;
        if (col == d.blank || col >= V) v[c] = 0.f;   // blank is not a non-blank expansion
        if (delta_nb && col < V) delta_nb[(long)pair * V + col] = v[c];
    }
    expand_best<1, EXP_THREADS>(v, sm, d, tid, true, cand_score + (long)pair * d.N, cand_tok + (long)pair * d.N);
}

template <int NQ, int RPW>
static hipError_t expand_long_launch(hipStream_t st, const Dims &d, int pairs, const float *logits, AView A, RowView rv,
                                     float *row_lc, float *dphi, float *cand_score, int *cand_tok, float *row_stats,
                                     float *delta_nb, const int *pairs_dev, int pair_base) {
    int waves = (d.S + RPW - 1) / RPW;
    if (waves < LONG_MIN_WAVES) waves = LONG_MIN_WAVES;
    if (waves > 16) return hipErrorInvalidValue;
    const size_t shm = (size_t)waves * d.Vl * sizeof(float);   // (at most 64 KB)
    static size_t attr_for = 0;
    if (shm > attr_for) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_expand_long<NQ, RPW>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
        if (e != hipSuccess) return e;
        attr_for = shm;
    }
    hipLaunchKernelGGL((k_expand_long<NQ, RPW>), dim3(pairs), dim3(64 * waves), shm, st, d, logits, A, rv, row_lc, dphi,
                       cand_score, cand_tok, row_stats, delta_nb, pairs_dev, pair_base);
    return hipGetLastError();
}

template <int NV4, int SMAX>
static void expand_reg_launch(hipStream_t st, const Dims &d, int pairs, const float *logits, AView A, RowView rv,
                              float *row_lc, float *dphi, float *cand_score, int *cand_tok, float *row_stats,
                              float *delta_nb, const int *pairs_dev, int pair_base) {
    hipLaunchKernelGGL((k_expand_reg<NV4, SMAX>), dim3(pairs), dim3(EXP_THREADS), 0, st, d, logits, A, rv, row_lc, dphi,
                       cand_score, cand_tok, row_stats, delta_nb, pairs_dev, pair_base);
}

// The kernel that expands segments of S frames of logit rows of Vl floats (tests ask it by this name).
// Register forms (EXPAND_REG: 16-byte pieces a thread, most frames): the whole hypothesis in the registers of four waves.
// Longer segments of a vocabulary that fits a lane's four pieces (EXPAND_LONG: pieces a lane, rows a wave): two rows a
// wave up to 32 frames, four up to 64 (a workgroup has at most 16 waves).  Measured on the Librispeech-like batch of 64
// at N = 5 (ms per decode; one / two / four rows a wave; four waves with eight / sixteen frames' columns in registers):
// S = 6: 19.6 / 19.7 / 19.8 / 20.3 / 21.7, 8: 19.3 / 19.5 / - / 20.0 / 21.3, 12: 19.7 / 19.7 / 19.8 / - / 21.8, 16: 20.4 /
// 20.4 / 20.6 / - / 22.7, 20: - / 21.8 / 22.1, 32: - / 24.4 / 24.5; the two-pass kernel took 28.0 at 20, 33.5 at 32 and
// 44.3 (four rows a wave 30.9) at 50.  S = 8 elsewhere (two rows a wave / eight frames in registers): 4 utterances
// 15.3 / 16.0, 200 25.9 / 27.0, 320 32.2 / 33.6, V = 500 20.0 / 20.8, V = 200 19.8 / 20.9, N = 10 26.0 / 27.0, 1000 shorter
// utterances at N = 10 36.4 / 37.3.  (The body for 2048 columns, half of them copies here: 20.7 at S = 6, 20.4 at 8.)
extern "C" int expand_form(int Vl, int S) {
    const int nv4 = (Vl / 4 + EXP_THREADS - 1) / EXP_THREADS;
    if (nv4 <= 1) {
        if (S <= 3) return EXPAND_REG(1, 3);
        if (S <= 5) return EXPAND_REG(1, 5);
        if (S <= LONG_FRAMES) return EXPAND_LONG(Vl <= 256 ? 1 : (Vl <= 512 ? 2 : 4), S <= 32 ? 2 : 4);
    }
    if (nv4 <= 2 && S <= 8) return EXPAND_REG(2, 8);
    if (nv4 <= 4 && S <= 3) return EXPAND_REG(4, 3);
    if (nv4 <= 4 && S <= 5) return EXPAND_REG(4, 5);
    return EXPAND_TWO_PASS;
}

hipError_t launch_expand(hipStream_t st, const Dims &d, int pairs, const float *logits, AView A, RowView rv,
                         float *row_lc, float *dphi, float *cand_score, int *cand_tok, float *row_stats,
                         float *delta_nb, int force_generic, const int *pairs_dev, int pair_base) {
    if (pairs <= 0) return hipSuccess;
    if (pairs_dev && pair_base) return hipErrorInvalidValue;   // (a piece is launched with its size known)
    size_t shm = (size_t)d.Vl * sizeof(float);
    if (!force_generic) {
#define TBS_EXPAND_REG(NV4, SMAX)                                                                                      \
    case EXPAND_REG(NV4, SMAX):                                                                                        \
        expand_reg_launch<NV4, SMAX>(st, d, pairs, logits, A, rv, row_lc, dphi, cand_score, cand_tok, row_stats,       \
                                     delta_nb, pairs_dev, pair_base);                                                  \
        return hipGetLastError();
#define TBS_EXPAND_LONG(NQ, RPW)                                                                                       \
    case EXPAND_LONG(NQ, RPW):                                                                                         \
        return expand_long_launch<NQ, RPW>(st, d, pairs, logits, A, rv, row_lc, dphi, cand_score, cand_tok, row_stats, \
                                           delta_nb, pairs_dev, pair_base);
        switch (expand_form(d.Vl, d.S)) {
            TBS_EXPAND_REG(1, 3) TBS_EXPAND_REG(1, 5) TBS_EXPAND_REG(2, 8) TBS_EXPAND_REG(4, 3) TBS_EXPAND_REG(4, 5)
            TBS_EXPAND_LONG(1, 2) TBS_EXPAND_LONG(1, 4)
            TBS_EXPAND_LONG(2, 2) TBS_EXPAND_LONG(2, 4)
            TBS_EXPAND_LONG(4, 2) TBS_EXPAND_LONG(4, 4)
            default: break;
        }
#undef TBS_EXPAND_REG
#undef TBS_EXPAND_LONG
    }
    hipLaunchKernelGGL(k_expand, dim3(pairs), dim3(EXP_THREADS), shm, st, d, logits, A, rv, row_lc, dphi, cand_score,
                       cand_tok, row_stats, delta_nb, pairs_dev, pair_base);
    return hipGetLastError();
}
