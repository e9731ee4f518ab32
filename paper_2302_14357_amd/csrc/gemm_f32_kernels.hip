// Dense layers of fp32 models:
//   C[M,N] = A[M,K] * B[N,K]^T + bias[N],  fp32 throughout (v_mfma_f32_32x32x2_f32)
// (optionally rows scattered through out_row).
//
// The matrix cores take 64 cycles for a 32x32x2 step, a sixteenth of their bf16 rate, so at the sizes
// of a decode (80 to 400 rows) what bounds a product is how many SIMDs work on it.  A workgroup
// therefore owns one 32x32 tile and its four waves share K: wave w multiplies the w-th quarter of
// every K tile and the four partial tiles are added up through LDS at the end, where a thread owns
// four neighbouring columns of a row.  Measured at 16 utterances x 5 hypotheses x 3 frames of
// the Librispeech-like widths (240 x 1024 x 512, 80 x 2560 x 1280, 80 x 512 x 640): 10.5 us a launch on
// average against 122 us for the kernel of scalar multiply-adds on 64x64 tiles at the end of this file.
// With the fused epilogues (gates 80 x 2560 x 640 and the cell update 12.3 us, projection and joiner
// input rows 8.9 us, joiner 7.4 us) a round is four launches instead of nine.
// K tiles of 128 floats go from global memory straight into LDS, as many requested at once as there are
// stages; rows are 512 bytes, chunk c (16 bytes) of row r sits at position c ^ (r & 15), so that the
// 16-byte fragment reads of 16 neighbouring rows fall into different banks.  A lane takes 4 consecutive K
// elements per read and the MFMA steps take them in the order in which they lie (any order of K that A and B
// share is the same sum).  Products of every size run in these tiles; larger ones were not measured.
#include "tbs_internal.h"
#include <climits>

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

#define GF_BK 128                         // floats of K per stage
#define GF_CH (GF_BK / 4)                 // 16-byte chunks per LDS row
#define GF_STAGE (2 * GF_TILE * GF_BK)    // floats of one stage: A rows, then B rows
#define GF_LOADS 8                        // direct loads per wave and stage
#define GF_PAD 36                         // floats per row of a partial tile in LDS

// s_waitcnt operand that waits for all but n vector-memory operations and for nothing else
#define GF_VMCNT(n) (((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))

// workgroup barrier that orders LDS traffic only (the direct loads of later stages stay in flight)
__device__ __forceinline__ void gf_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ float gf_sigmoid(float x) { return 1.f / (1.f + expf(-x)); }

// MODE 0: C[out_row[r], :] = A[r, :] B^T + bias.
// MODE 1: the product is the gate pre-activations of an LSTM layer (gate-interleaved columns, see
// LstmEp), a thread's four columns are the gates of one hidden unit, and the epilogue is the cell update.
// MODE 2: the product is the predictor projection of new hypotheses (row r = pair r); the epilogue also
// forms the joiner input rows of the pair's frames (see JoinEp).
// m_dev not null: M is an upper bound and the rows that exist are the first *m_dev; any_dev not null: rows
// may be dead (state slot < 0) anywhere and the launch leaves at once when *any_dev is zero.
// xcd_rows (MODE 0): every XCD computes a range of rows of its own, all their columns (see PartEp).
template <int MODE>
__global__ void __launch_bounds__(256)
k_gemm_f32_mfma(const float *__restrict__ A, const float *__restrict__ B, const float *__restrict__ bias,
                float *__restrict__ C, int M, int N, int K, const int *__restrict__ out_row, long ldc, int tiles_m,
                int tiles_n, int ns, LstmEp ep, JoinEp jp, const int *__restrict__ m_dev,
                const int *__restrict__ any_dev, int xcd_rows) {
    extern __shared__ __attribute__((aligned(16))) float gf_smem[];   // ns stages
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The 8 XCDs (workgroup id modulo 8) form a 2 x 4 grid over the tiles, so that each XCD's L2
    // fetches half of A and a quarter of B instead of all of both.
    const int tmx = (tiles_m + 1) >> 1, tnx = (tiles_n + 3) >> 2;
    // (MODE 2 may run several workgroups per tile: the grid is then that many copies of the tile grid)
    const int base_grid = 8 * tmx * tnx;
    const int fgroup = MODE == 2 ? (int)blockIdx.x / base_grid : 0;
    const int bid = (int)blockIdx.x - fgroup * base_grid;
    const int xcd = bid & 7, j = bid >> 3;
    int tile_m = (xcd >> 2) * tmx + j % tmx, tile_n = (xcd & 3) * tnx + j / tmx;
    if (MODE == 0 && xcd_rows) {   // a row range per XCD, all its columns
        const int tpx = (tiles_m + 7) >> 3;
        tile_m = xcd * tpx + j % tpx;
        tile_n = j / tpx;
    }
    if (tile_m >= tiles_m || tile_n >= tiles_n) return;   // before any barrier
    const int kt = (K + GF_BK - 1) / GF_BK, kch = K >> 2;   // (K is a multiple of 4)

    // what the epilogue needs is requested first: loads retire in order, so it is there before the tiles
    const int erow = tile_m * GF_TILE + (tid >> 3), ecol = tile_n * GF_TILE + (tid & 7) * 4;
    const int erc = min(erow, M - 1);
    int orow = erc;                              // MODE 0 and 2: destination row
    int e_ps = 0, e_ns = 0, e_tok = 0;           // MODE 1: parent's and own state slot, last token
    int e_row0 = 0, e_len = 0, e_f0 = 0;         // MODE 2: first joiner row, frames, first frame
    if (MODE == 1) {
        e_ps = ep.pslot[erc];
        e_ns = ep.slot[erc];
        e_tok = ep.tok[erc];   // (unconditionally: a load behind a condition would be waited for at once)
    } else if (MODE == 2) {
        orow = out_row[erc];
        e_row0 = jp.pair_row0[erc];
        e_len = jp.pair_len[erc];
        e_f0 = jp.pair_frame0[erc];
    } else if (out_row) {
        orow = out_row[erc];
    }
    float bv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bv[i] = bias ? bias[min(ecol + i, N - 1)] : 0.f;
    asm volatile("" ::: "memory");
    const int m_live = m_dev ? min(*m_dev, M) : M;     // (the same in every lane)
    if (tile_m * GF_TILE >= m_live) return;            // no row of this tile exists
    if (any_dev && *any_dev == 0) return;

    // Direct loads: one instruction fills 1 KB of LDS = 2 rows of 512 bytes, lane l the 16 bytes at row
    // l/32, position l%32; the position holds chunk (l%32) ^ (row & 15) of the K tile.  Rows and
    // chunks beyond the matrices are clamped to ones that exist.
    const int lrow = lane >> 5, lpos = lane & 31;
    auto fetch = [&](int c, int stage) {
        float *dst = gf_smem + stage * GF_STAGE + wave * 2 * GF_BK;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = (i & 3) * 8 + wave * 2 + lrow;
            const int ch = min(c * GF_CH + (lpos ^ (row & 15)), kch - 1);
            const float *src = i < 4 ? A + (long)min(tile_m * GF_TILE + row, M - 1) * K
                                     : B + (long)min(tile_n * GF_TILE + row, N - 1) * K;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + ch * 4),
                                             (__attribute__((address_space(3))) void *)(dst + i * 8 * GF_BK), 16, 0, 0);
        }
    };
    const int first = min(ns, kt);
    for (int c = 0; c < first; ++c) fetch(c, c);
    floatx16 acc, acc1;   // (two, so that consecutive MFMAs do not wait for each other)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = acc1[r] = 0.f;
    const int frow = lane & 31, fsel = lane >> 5, fsw = frow & 15;
    int stage = 0;
    for (int c = 0; c < kt; ++c) {
        const int after = min(kt, c + ns) - 1 - c;   // K tiles requested after this one
        if (after >= 3) __builtin_amdgcn_s_waitcnt(GF_VMCNT(3 * GF_LOADS));
        else if (after == 2) __builtin_amdgcn_s_waitcnt(GF_VMCNT(2 * GF_LOADS));
        else if (after == 1) __builtin_amdgcn_s_waitcnt(GF_VMCNT(1 * GF_LOADS));
        else __builtin_amdgcn_s_waitcnt(GF_VMCNT(0));
        gf_barrier();      // every wave's share of this K tile is in LDS
        const float *cur = gf_smem + stage * GF_STAGE + frow * GF_BK;
        float4 af[4], bf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int cpos = ((wave * 8 + i * 2 + fsel) ^ fsw) * 4;
            af[i] = *reinterpret_cast<const float4 *>(cur + cpos);
            bf[i] = *reinterpret_cast<const float4 *>(cur + GF_TILE * GF_BK + cpos);
        }
        if ((c + 1) * GF_CH > kch) {   // (uniform) the last K tile is short: chunks beyond K count as zero
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (c * GF_CH + wave * 8 + i * 2 + fsel >= kch) {
                    af[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                    bf[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i].x, bf[i].x, acc, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i].y, bf[i].y, acc1, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i].z, bf[i].z, acc, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i].w, bf[i].w, acc1, 0, 0, 0);
        }
        if (c + ns < kt) {
            gf_barrier();      // every wave has read this stage
            fetch(c + ns, stage);
        }
        stage = stage + 1 == ns ? 0 : stage + 1;
    }
    // The four partial tiles meet in LDS (the stages are free once every wave is past its last K tile);
    // thread t takes row t/8 and the columns 4(t%8) .. +3.
    gf_barrier();
    float *sp = gf_smem + wave * (GF_TILE * GF_PAD);
#pragma unroll
    for (int r = 0; r < 16; ++r) sp[((r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) * GF_PAD + (lane & 31)] = acc[r] + acc1[r];
    gf_barrier();
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float4 q = *reinterpret_cast<const float4 *>(gf_smem + w * (GF_TILE * GF_PAD) + (tid >> 3) * GF_PAD + (tid & 7) * 4);
        v[0] += q.x; v[1] += q.y; v[2] += q.z; v[3] += q.w;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] += bv[i];
    if (erow >= m_live) return;
    if (MODE == 1) {
        const int H = ep.H, unit = ecol >> 2;
        if (unit >= H || e_ns < 0) return;
        // everything the update reads from memory is requested before any of it is used (from addresses
        // that are valid whether it is needed or not)
        const float cp = ep.c_par[(long)e_ps * H + unit];
        const float hp = (ep.h_par_next ? ep.h_par_next : ep.c_par)[(long)e_ps * H + unit];
        if (ep.emb_gates) {
            const float4 e = *reinterpret_cast<const float4 *>(ep.emb_gates + (long)e_tok * 4 * H + ecol);
            v[0] += e.x; v[1] += e.y; v[2] += e.z; v[3] += e.w;
        }
        const float cn = gf_sigmoid(v[1]) * cp + gf_sigmoid(v[0]) * tanhf(v[2]);
        const float hn = gf_sigmoid(v[3]) * tanhf(cn);
        ep.c_new[(long)e_ns * H + unit] = cn;
        ep.h_new[(long)e_ns * H + unit] = hn;
        float *out = static_cast<float *>(ep.out);
        if (ep.h_par_next == nullptr) {
            out[(long)erow * H + unit] = hn;
        } else {
            out[(long)erow * 2 * H + unit] = hn;
            out[(long)erow * 2 * H + H + unit] = hp;
        }
        return;
    }
    if (MODE == 2) {
        if (ecol >= N || orow < 0) return;   // (N is a multiple of 4)
        const int fgs = jp.fgroups > 1 ? jp.fgroups : 1;   // this workgroup's frames: fgroup, fgroup + fgs, ...
        const float *enc = static_cast<const float *>(jp.enc) + (long)e_f0 * N + ecol;
        float *amat = static_cast<float *>(jp.amat) + (long)e_row0 * N + ecol;
        for (int t0 = fgroup; t0 < e_len; t0 += 4 * fgs) {
            float4 e[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) e[q] = *reinterpret_cast<const float4 *>(enc + (long)min(t0 + q * fgs, e_len - 1) * N);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t0 + q * fgs < e_len)
                    *reinterpret_cast<float4 *>(amat + (long)(t0 + q * fgs) * N) =
                        make_float4(tbs_joiner_act_f32(e[q].x + v[0], jp.act), tbs_joiner_act_f32(e[q].y + v[1], jp.act),
                                    tbs_joiner_act_f32(e[q].z + v[2], jp.act), tbs_joiner_act_f32(e[q].w + v[3], jp.act));
        }
        if (fgroup == 0) *reinterpret_cast<float4 *>(C + (long)orow * ldc + ecol) = make_float4(v[0], v[1], v[2], v[3]);
        return;
    }
    float *dst = C + (long)orow * ldc + ecol;
    if (ecol + 3 < N && (ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0) {
        *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (ecol + i < N) dst[i] = v[i];
    }
}

// Rows that are not whole 16-byte pieces (K not a multiple of 4, or an operand at an odd address):
// 64x64 tile, 4x4 outputs per thread, any K.
__global__ void __launch_bounds__(256)
k_gemm_f32_any(const float *__restrict__ A, const float *__restrict__ B, const float *__restrict__ bias,
               float *__restrict__ C, int M, int N, int K, const int *__restrict__ out_row, long ldc) {
    __shared__ float sA[16][64 + 1], sB[16][64 + 1];
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += 16) {
        for (int i = tid; i < 64 * 16; i += 256) {
            int r = i / 16, k = i % 16;
            int gm = m0 + r, gn = n0 + r, gk = k0 + k;
            sA[k][r] = (gm < M && gk < K) ? A[(long)gm * K + gk] : 0.f;
            sB[k][r] = (gn < N && gk < K) ? B[(long)gn * K + gk] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = sA[k][ty * 4 + i]; b[i] = sB[k][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    for (int i = 0; i < 4; ++i) {
        int gm = m0 + ty * 4 + i;
        if (gm >= M) continue;
        long orow = out_row ? out_row[gm] : gm;
        for (int j = 0; j < 4; ++j) {
            int gn = n0 + tx * 4 + j;
            if (gn < N) C[orow * ldc + gn] = acc[i][j] + (bias ? bias[gn] : 0.f);
        }
    }
}

// LDS stages the MFMA kernel may use on the current device (0 = not usable)
static int gf_stages() {
    static int stages = -1;
    if (stages < 0) {
        int found = 0;
        for (int ns = 5; ns >= 2 && !found; --ns) {
            const int bytes = (int)(ns * GF_STAGE * sizeof(float));
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_f32_mfma<0>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess &&
                hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_f32_mfma<1>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess &&
                hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_f32_mfma<2>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess)
                found = ns;
        }
        (void)hipGetLastError();
        stages = found;
    }
    return stages;
}

// Stages of a launch: up to 256 workgroups every CU has one and all K tiles (up to five) are asked for
// at once; with more of them two stages, so that two workgroups share a CU.
static int gf_ns(long wgs, int K) {
    const int kt = (K + GF_BK - 1) / GF_BK, ns_max = gf_stages();
    if (wgs > 256 || kt < 2) return 2;
    return kt < ns_max ? kt : ns_max;
}

static long gf_tiles(int n) { return (n + GF_TILE - 1) / GF_TILE; }

// can the MFMA kernel run the product, and has it at most max_tiles tiles?
bool gemm_f32_fits(const void *A, const void *B, int M, int N, int K, int max_tiles) {
    return K % 4 == 0 && ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) & 15) == 0 && gf_stages() >= 2 &&
           gf_tiles(M) * gf_tiles(N) <= max_tiles;
}

template <int MODE>
static hipError_t gf_launch(hipStream_t st, const float *A, const float *B, const float *bias, float *C, int M, int N, int K,
                            const int *out_row, long ldc, const LstmEp &ep, const JoinEp &jp, const int *m_dev,
                            const int *any_dev, bool xcd_rows, int copies) {
    const long tm = gf_tiles(M), tn = gf_tiles(N);
    const int ns = gf_ns(tm * tn * copies, K);
    const long grid = xcd_rows ? 8 * ((tm + 7) / 8) * tn : 8 * ((tm + 1) / 2) * ((tn + 3) / 4) * copies;
    hipLaunchKernelGGL(k_gemm_f32_mfma<MODE>, dim3((unsigned)grid), dim3(256), ns * GF_STAGE * sizeof(float), st, A, B, bias,
                       C, M, N, K, out_row, ldc, (int)tm, (int)tn, ns, ep, jp, m_dev, any_dev, xcd_rows ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_gemm_f32(hipStream_t st, const float *A, const float *B, const float *bias, float *C, int M, int N,
                           int K, const int *out_row, long ldc, const int *m_dev, bool xcd_rows) {
    if (M <= 0) return hipSuccess;
    if (gemm_f32_fits(A, B, M, N, K, INT_MAX))
        return gf_launch<0>(st, A, B, bias, C, M, N, K, out_row, ldc, LstmEp{}, JoinEp{}, m_dev, nullptr, xcd_rows, 1);
    if (m_dev || xcd_rows) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gemm_f32_any, dim3((N + 63) / 64, (M + 63) / 64), dim3(256), 0, st, A, B, bias, C, M, N, K,
                       out_row, ldc);
    return hipGetLastError();
}

hipError_t launch_gemm_lstm_f32(hipStream_t st, const float *A, const float *Wp, const float *biasp, int M, int K,
                                const LstmEp &ep, const int *m_dev, const int *any_dev) {
    if (M <= 0) return hipSuccess;
    if (!gemm_f32_fits(A, Wp, M, 4 * ep.H, K, INT_MAX)) return hipErrorInvalidValue;
    return gf_launch<1>(st, A, Wp, biasp, nullptr, M, 4 * ep.H, K, nullptr, 0, ep, JoinEp{}, m_dev, any_dev, false, 1);
}

hipError_t launch_gemm_join_f32(hipStream_t st, const float *A, const float *B, const float *bias, float *C, int M, int N,
                                int K, const int *out_row, long ldc, const JoinEp &jp, const int *m_dev,
                                const int *any_dev) {
    if (M <= 0) return hipSuccess;
    if (!gemm_f32_fits(A, B, M, N, K, INT_MAX) || N % 4 || ldc % 4 || !out_row ||
        (reinterpret_cast<uintptr_t>(jp.enc) & 15) || (reinterpret_cast<uintptr_t>(jp.amat) & 15))
        return hipErrorInvalidValue;
    return gf_launch<2>(st, A, B, bias, C, M, N, K, out_row, ldc, LstmEp{}, jp, m_dev, any_dev, false,
                        jp.fgroups > 1 ? jp.fgroups : 1);
}
