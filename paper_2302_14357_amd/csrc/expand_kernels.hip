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
// (FOLD: as the launch over whole segments adds up, for batches that it may decode)
template <int NQ, int RPW, bool FOLD>
__global__ void __launch_bounds__(FOLD ? 64 * LONG_FOLD_WAVES : 1024)
k_expand_long(Dims d, const float *__restrict__ logits, AView A, RowView rv, float *__restrict__ row_lc,
              float *__restrict__ dphi, float *__restrict__ cand_score, int *__restrict__ cand_tok,
              float *__restrict__ row_stats, float *__restrict__ delta_nb, const int *__restrict__ pairs_dev,
              int pair_base) {
    extern __shared__ __attribute__((aligned(16))) float4 s_part[];   // [shares][Vl / 4]
    __shared__ LongShared sm;
    const int pair = pair_base + blockIdx.x, tid = threadIdx.x;
    const int waves = FOLD ? LONG_FOLD_WAVES : (int)blockDim.x >> 6, shares = FOLD ? LONG_FOLD_SHARES : waves;
    if (pairs_dev && pair >= *pairs_dev) return;   // (enqueued on an upper-bound grid, see k_expand_reg)
    const int u = ((cint_p)rv.pair_u)[pair], h = ((cint_p)rv.pair_h)[pair];
    const int row0 = ((cint_p)rv.pair_row0)[pair], sp = ((cint_p)rv.pair_len)[pair];
    const float *L = logits + (long)row0 * d.Vl;
    expand_long<NQ, RPW, FOLD>(
        d, sp, waves, shares, tid, sm, s_part, [&](int t) { return A.dhat[((long)u * d.N + h) * d.S + t]; },
        [&](int t, int piece) { return reinterpret_cast<const float4 *>(L + (long)t * d.Vl)[piece]; },
        [&](int t, int col) { return L[(long)t * d.Vl + col]; }, row_lc + row0, dphi + pair, cand_score + (long)pair * d.N,
        cand_tok + (long)pair * d.N, row_stats ? row_stats + (long)row0 * 3 : nullptr, delta_nb ? delta_nb + (long)pair * d.V : nullptr);
}

template <int NQ, int RPW, bool FOLD = false>
static hipError_t expand_long_launch(hipStream_t st, const Dims &d, int pairs, const float *logits, AView A, RowView rv,
                                     float *row_lc, float *dphi, float *cand_score, int *cand_tok, float *row_stats,
                                     float *delta_nb, const int *pairs_dev, int pair_base) {
    int waves = (d.S + RPW - 1) / RPW;
    if (waves < LONG_MIN_WAVES) waves = LONG_MIN_WAVES;
    if (waves > (FOLD ? LONG_FOLD_WAVES : 16)) return hipErrorInvalidValue;
    if (FOLD) waves = LONG_FOLD_WAVES;
    const size_t shm = (size_t)(FOLD ? LONG_FOLD_SHARES : waves) * d.Vl * sizeof(float);   // (at most 64 KB)
    static size_t attr_for = 0;
    if (shm > attr_for) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_expand_long<NQ, RPW, FOLD>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
        if (e != hipSuccess) return e;
        attr_for = shm;
    }
    hipLaunchKernelGGL((k_expand_long<NQ, RPW, FOLD>), dim3(pairs), dim3(64 * waves), shm, st, d, logits, A, rv, row_lc, dphi,
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
                         float *delta_nb, int force_generic, const int *pairs_dev, int pair_base, bool fold) {
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
        const int form = expand_form(d.Vl, d.S);
        if (fold && form >= EXPAND_LONG(1, 0)) {   // (rows a wave: those of the launch's bodies for 16, 32 and 64 frames)
#define TBS_EXPAND_FOLD(NQ, RPW)                                                                                        \
    case EXPAND_LONG(NQ, RPW):                                                                                          \
        return expand_long_launch<NQ, RPW, true>(st, d, pairs, logits, A, rv, row_lc, dphi, cand_score, cand_tok,       \
                                                 row_stats, delta_nb, pairs_dev, pair_base);
            switch (EXPAND_LONG((form - 1000) / 10, d.S <= 16 ? 2 : (d.S <= 32 ? 4 : 8))) {
                TBS_EXPAND_FOLD(1, 2) TBS_EXPAND_FOLD(1, 4) TBS_EXPAND_FOLD(1, 8)
                TBS_EXPAND_FOLD(2, 2) TBS_EXPAND_FOLD(2, 4) TBS_EXPAND_FOLD(2, 8)
                TBS_EXPAND_FOLD(4, 2) TBS_EXPAND_FOLD(4, 4) TBS_EXPAND_FOLD(4, 8)
                default: return hipErrorInvalidValue;
            }
#undef TBS_EXPAND_FOLD
        }
        switch (form) {
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
