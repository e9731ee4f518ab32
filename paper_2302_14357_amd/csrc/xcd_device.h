// Whole segments of small models as one launch: the rounds of Algorithm 1 run inside a kernel whose
// workgroups stay on their CUs, one per CU, and every XCD decodes utterances of its own.
//
// In the slot layout a round is four dependent kernels, and what bounds them is not their work but what
// lies around it: about 3.5 us of launch each, and the weights, which every launch fetches again
// (64 utterances of the Librispeech-like widths, N = 5, S = 3: 32 us a round).  Here the 32 workgroups of an XCD divide the
// columns of the three products among them and hold their slices of the gate and joiner weights in LDS for the whole launch
// (640 x 2560 and 512 x 1024 bf16 are 132 KB a CU); activations, logits and descriptors travel
// through the L2 that the XCD's CUs share, and a step ends with a barrier of those 32 workgroups alone,
// a counter in that L2: 0.7-1.0 us, where a barrier of the whole chip took 10 us (its release writes the L2
// back to memory) and a kernel boundary takes 3.5 us.  Measured, ms per decode, four kernels a round (row lists for S > 5) and
// in one launch: one utterance 10.2 and 4.9, 64 utterances 17.4 and 10.2 (S = 1 28.3 and 12.9, S = 20 21.2 and 14.5), 200
// utterances 24.6 and 15.3, 16 utterances fp32 20.4 and 12.5.  What bounds a round now is the expansion and the select step (one
// wave's chain of instructions per hypothesis, 6.5 of 19 us), the barriers (5 us with the wait for the last CU) and what the
// products read from LDS and L2.
//
// What one CU writes and another of the XCD reads goes out by ordinary stores (they go through the L1 to the L2; the
// barrier waits for their acknowledgement) and comes in by loads of device scope (`fresh` below), which
// pass by the reader's L1: loads of wave or workgroup scope were seen to return lines the L1 had kept from
// the round before.  What only one CU ever writes and reads (an utterance's lists A and B, its trie nodes, the
// columns of p, h and c that belong to a CU's share of the products) needs no such care.
//
// The workgroups must all run at once.  A launch begins by counting them: when all have come, and 32 on
// every XCD, it goes on; when they have not come in time (somebody else holds CUs) it ends with nothing changed, and the
// caller runs the batch in the slot layout.  Every later wait is bounded too.
#pragma once
#include "expand_device.h"
#include "select_device.h"
#include "xcd_barrier.h"
#include <algorithm>
#include <type_traits>

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned uintx4;

#define XR_CANDS 128                    // candidates of a select step (N <= 11)
#define XR_LDS(wide) (160 * 1024 - XR_STATIC_LDS(wide))
#define XR_STATIC_LDS(wide) ((wide) ? 7424 : 6144)   // the kernel's own arrays: the select step's and the figures
#define XR_TURNS (XR_POS / XR_WGS)      // utterances a workgroup may own

// ------------------------------------------------------------------ memory shared by the CUs of an XCD
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t rsrc_of(const void *p, long bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}
#define XR_DEVICE_SCOPE 16   // cache policy of a buffer load: device scope (past the L1)
__device__ __forceinline__ uintx4 fresh16(rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, XR_DEVICE_SCOPE));
}
__device__ __forceinline__ float fresh4(rsrc_t r, unsigned voff, unsigned soff) {
    return __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, XR_DEVICE_SCOPE));
}
__device__ __forceinline__ float4 as_float4(const uintx4 &v) {
    return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
}
#define XR_TICKS 100000ull   // wall_clock64 ticks per millisecond

// Barrier of the XCD's workgroups, in two halves: every wave waits for its stores (they are in the L2 then) and one thread
// counts the workgroup in; later that thread waits for the others.  What is asked for between the halves is on its way
// meanwhile.  At the barrier that ends a round (LIVE) `live` is added up over the workgroups and the wait returns the sum; at the
// others it returns 0; -1 if the others did not come (bounded: nobody here takes anywhere near that long).
struct XcdBarrier {
    u64 *word;        // low half: arrivals, high half: sum of live, both since the launch began
    unsigned due;     // arrivals that end the coming barrier
    unsigned seen;    // sum of live up to the last one that ended a round
};
__device__ __forceinline__ void xcd_arrive(XcdBarrier &b, int live) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    b.due += XR_WGS;
    if (threadIdx.x == 0)
        __hip_atomic_fetch_add(b.word, 1ull | ((u64)(unsigned)live << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool LIVE>
__device__ __forceinline__ int xcd_wait(XcdBarrier &b, int &s_sum) {
    if (threadIdx.x == 0) {
        unsigned spin = 0;
        u64 t0 = 0;
        int sum = 0;
        while ((sum = xcd_barrier_read(__hip_atomic_load(b.word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), b.due, b.seen, LIVE)) ==
               XR_NOT_YET) {
            if ((++spin & 1023u) == 0) {
                const u64 t = wall_clock64();
                if (t0 == 0) t0 = t;
                else if (t - t0 > 10000ull * XR_TICKS) {
                    sum = -1;
                    break;
                }
            }
        }
        s_sum = sum;
    }
    __syncthreads();
    const int sum = __builtin_amdgcn_readfirstlane(s_sum);
    asm volatile("" ::: "memory");
    if (LIVE && sum > 0) b.seen += (unsigned)sum;
    return sum;
}
__device__ __forceinline__ int xcd_barrier(XcdBarrier &b, int &s_sum) {
    xcd_arrive(b, 0);
    return xcd_wait<false>(b, s_sum);
}

// ------------------------------------------------------------------ arithmetic shared with the kernels of the slot layout
__device__ __forceinline__ float xr_sigmoid(float x) { return 1.f / (1.f + expf(-x)); }
__device__ __forceinline__ unsigned xr_bf16(float f) {   // nearest, ties to even
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
// four values of a frame or of a joiner input row, in the storage type of the model
template <bool F32> struct XcdType { typedef uint2 quad; };
template <> struct XcdType<true> { typedef float4 quad; };

// Joiner input rows lie in memory as the matrix instructions read them, in pieces of 1 KB: lane l of the wave that reads a
// piece takes the 16 bytes at 16 l.  bf16: 16 rows x 32 columns, the lane row l % 16 and columns 8 (l / 16) on.  Byte offset of
// column c0 (a multiple of 4) of a row, steps = Dj / 32:
__device__ __forceinline__ unsigned amat_at(int row, int c0, int steps) {
    return (((unsigned)(row >> 4) * steps + (c0 >> 5)) * 64 + ((c0 & 31) >> 3) * 16 + (row & 15)) * 16 + (c0 & 7) * 2;
}
// fp32: 16 rows x 16 columns.  A matrix instruction takes 4 columns, one a lane; the fp32 GEMM of the slot layout adds up
// columns k, k + 4, k + 2, k + 6 of every eight in one sum and those behind them (k + 1, ...) in another, so lane l holds, of
// eight columns, number (l / 16) of each sum, and a piece two such eights.  Place of column k in its piece's row of 16
// floats, four a lane (with the pieces ahead); a row of K columns takes f32_row(K) floats.
__host__ __device__ __forceinline__ int f32_pieces(int K) { return (K + 15) >> 4; }
__host__ __device__ __forceinline__ int f32_row(int K) { return f32_pieces(K) * 16; }
__host__ __device__ __forceinline__ int f32_at(int k) {
    return (k & ~15) + (((k >> 2) & 1) | (k & 2)) * 4 + ((k >> 3) & 1) * 2 + (k & 1);
}
__device__ __forceinline__ void put_joiner_quad(unsigned char *amat, int row, int c0, int Dj, const uint2 &e, const float4 &p, int act) {
    const float x[4] = {__uint_as_float(e.x << 16) + p.x, __uint_as_float(e.x & 0xFFFF0000u) + p.y, __uint_as_float(e.y << 16) + p.z,
                        __uint_as_float(e.y & 0xFFFF0000u) + p.w};
    unsigned o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = xr_bf16(tbs_joiner_act(x[q], act));
    *reinterpret_cast<uint2 *>(amat + amat_at(row, c0, Dj >> 5)) = make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
}
__device__ __forceinline__ void put_joiner_quad(unsigned char *amat, int row, int c0, int Dj, const float4 &e, const float4 &p, int act) {
    float *at = reinterpret_cast<float *>(amat) + (((long)(row >> 4) * f32_pieces(Dj) + (c0 >> 4)) * 64 + (row & 15)) * 4;
    const int l0 = ((c0 >> 2) & 1) * 16, i = ((c0 >> 3) & 1) * 2;   // (lanes l0 and l0 + 32)
    *reinterpret_cast<float2 *>(at + l0 * 4 + i) = make_float2(tbs_joiner_act_f32(e.x + p.x, act), tbs_joiner_act_f32(e.y + p.y, act));
    *reinterpret_cast<float2 *>(at + (l0 + 32) * 4 + i) = make_float2(tbs_joiner_act_f32(e.z + p.z, act), tbs_joiner_act_f32(e.w + p.w, act));
}

// 16 activation rows times one or two tiles of 16 weight rows in LDS, C chunks of 128 of K (same order of the sums over K as
// the 32 x 32 tiles of the slot layout's kernels: the same bits).  Lane l of a result holds weight rows 4 (l / 16) .. + 3 of
// activation row l % 16.
template <int TILES, int C>
__device__ __forceinline__ void mma(floatx4 (&acc)[2], const bf16x8 (&x)[4 * C], const unsigned char *w0, const unsigned char *w1, int lane) {
    acc[0] = acc[1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4 * C; ++s) {
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(w0 + s * 1024 + lane * 16), x[s], acc[0], 0, 0, 0);
        if (TILES == 2)
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(w1 + s * 1024 + lane * 16), x[s], acc[1], 0, 0, 0);
    }
}

// fn<C>() for the C chunks of 128 that K has
template <class F>
__device__ __forceinline__ void by_chunks(int K, F fn) {
    static_assert(XR_KMAX == 5 * 128, "a case for every width");
    switch (K >> 7) {
        case 1: fn(std::integral_constant<int, 1>()); break;
        case 2: fn(std::integral_constant<int, 2>()); break;
        case 3: fn(std::integral_constant<int, 3>()); break;
        case 4: fn(std::integral_constant<int, 4>()); break;
        default: fn(std::integral_constant<int, 5>()); break;
    }
}

// This workgroup's slice of a weight matrix [rows, K] in LDS: tiles r, r + 32, ... of 16 rows, each in pieces of 1 KB as the
// matrix instructions read them (see amat_at, f32_at).  Pieces [from, to) of it; they are there behind the next barrier that has
// waited for them.  The gates' lie in memory in that order; the output matrix and the projection, which may change from one
// decode to the next, come from their rows.
__device__ __forceinline__ void load_frags(unsigned char *lds, const void *frags, int pieces, int from, int to, int r, int wave, int nw, int lane) {
    const float rcp_p = __builtin_amdgcn_rcpf((float)pieces);   // (exact quotients of fewer than 2^12 pieces)
#pragma unroll 4
    for (int i = from + wave; i < to; i += nw) {
        const int t = (int)(((float)i + 0.5f) * rcp_p), m = i - t * pieces;
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void *)(static_cast<const float4 *>(frags) + ((long)(r + t * XR_WGS) * pieces + m) * 64 + lane),
            (__attribute__((address_space(3))) void *)(lds + (size_t)i * 1024), 16, 0, 0);
    }
}
template <bool F32>
__device__ __forceinline__ void load_rows(unsigned char *lds, const void *w, int rows, int K, int own, int r, int wave, int nw, int lane) {
    const int pieces = F32 ? f32_pieces(K) : K >> 5;
    const float rcp_p = __builtin_amdgcn_rcpf((float)pieces);
#pragma unroll 4
    for (int i = wave; i < own * pieces; i += nw) {
        const int t = (int)(((float)i + 0.5f) * rcp_p), m = i - t * pieces;
        const long row = min((r + t * XR_WGS) * 16 + (lane & 15), rows - 1);
        if constexpr (F32) {   // (K is a multiple of 8: a piece's second half may lie beyond it)
            const int q = lane >> 4, k = m * 16 + (q & 1) * 4 + (q & 2);
            const float *src = static_cast<const float *>(w) + row * K + k;
            const float2 lo = *reinterpret_cast<const float2 *>(src);
            float2 hi = *reinterpret_cast<const float2 *>(k + 8 < K ? src + 8 : src);
            if (k + 8 >= K) hi = make_float2(0.f, 0.f);
            *reinterpret_cast<float4 *>(lds + (size_t)i * 1024 + lane * 16) = make_float4(lo.x, lo.y, hi.x, hi.y);
        } else {
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(static_cast<const bf16_t *>(w) + row * K + m * 32 + (lane >> 4) * 8),
                (__attribute__((address_space(3))) void *)(lds + (size_t)i * 1024), 16, 0, 0);
        }
    }
}

__device__ __forceinline__ int own_tiles(int tiles, int r) { return r < tiles ? (tiles - r + XR_WGS - 1) / XR_WGS : 0; }

template <int NV4, int SMAX>
__device__ __forceinline__ void expand_load_fresh(float (&e)[SMAX][NV4 * 4], rsrc_t logits, int row0, int S, int Vl, int tid) {
    const int V4 = Vl >> 2;
    unsigned off[NV4];
#pragma unroll
    for (int q = 0; q < NV4; ++q) off[q] = 16u * (unsigned)min(tid + 64 * q, V4 - 1);
#pragma unroll
    for (int t = 0; t < SMAX; ++t) {
        const unsigned row = (unsigned)(row0 + min(t, S - 1)) * (unsigned)Vl * 4u;
#pragma unroll
        for (int q = 0; q < NV4; ++q) {
            const uintx4 x = fresh16(logits, off[q], row);
#pragma unroll
            for (int c = 0; c < 4; ++c) e[t][4 * q + c] = __uint_as_float(x[c]);
        }
    }
}

// ------------------------------------------------------------------ the kernel
// The kernel's arguments fill more scalar registers than a wave has.  A step reads those it needs from the argument memory
// (through the scalar cache) when it begins; without the detour below the compiler reads all of them ahead of the loops and
// keeps them in lanes of vector registers, two instructions for every use.
typedef const __attribute__((address_space(4))) void *kernarg_p;
__device__ __forceinline__ const XcdArgs &xcd_args() {
    kernarg_p p = (kernarg_p)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const XcdArgs *)p;
}

// what a workgroup knows of its place and of the segment under way
struct XcdPlace {
    int x, r;        // XCD, workgroup within it
    int u_base, nu;  // its utterances in `order`
    int n_act;       // those up to the last that has frames in this segment
    int half;        // of the descriptors: this segment's (the next one's lists are made while others still read this one's)
    int N;           // beam
    int tid, lane, wave;
};

struct XcdShared {   // LDS
    int where[3];
    int sum, made;
    int sp[XR_POS], f0[XR_POS], utt[XR_POS];
    int fig[XR_TURNS][TBS_FIG_SIZE];   // (of this workgroup's utterances)
    int more[XR_TURNS], next[XR_TURNS];   // and whether this launch has another segment of theirs, and the list A that it begins with
};
__device__ __forceinline__ int4 *desc_of(const XcdArgs &g, const XcdPlace &w, int half) {
    return g.desc + (long)half * g.desc_half + (long)w.u_base * g.d.N;
}

// LDS behind the weights
template <int SMAX>
struct XcdScratch {
    static constexpr bool LONG = SMAX > 5;   // (long segments: a hypothesis by a workgroup, in a step of its own)
    unsigned char *b_list;             // B of an utterance (head of a segment: its scores)
    ExpandShared<SMAX, 1> *teams;      // (not for long segments)
    float *lc, *dphi, *cs;             // what the teams hand to the select step: [H, S'], [H], [H, N]
    int *ct;                           // [H, N]
    __device__ __forceinline__ XcdScratch(unsigned char *at, const Dims &d) {
        const size_t list = ((size_t)d.BCAP * (sizeof(double) + sizeof(u64) + 3 * sizeof(int)) + 15) & ~(size_t)15;
        b_list = at;
        teams = reinterpret_cast<ExpandShared<SMAX, 1> *>(at + list);
        lc = reinterpret_cast<float *>(teams + (LONG ? 0 : d.N));
        dphi = lc + d.N * SMAX;
        cs = dphi + d.N;
        ct = reinterpret_cast<int *>(cs + d.N * d.N);
    }
};

#define XR_PROJ_BYTES(nw) ((nw) * (1024 + 64))   // LDS for the projection's tiles
__host__ __device__ __forceinline__ int tiles_gate(const Dims &d) { return d.H >> 2; }         // (four units' four gates)
__host__ __device__ __forceinline__ int tiles_joiner(const Dims &d) { return (d.V + 15) >> 4; }
__host__ __device__ __forceinline__ int tiles_proj(const Dims &d) { return (d.Dj + 15) >> 4; }
// LDS of the slices (of the workgroup that has most)
__host__ __device__ __forceinline__ int slice_bytes(int tiles, int K) { return (tiles + XR_WGS - 1) / XR_WGS * (K >> 5) * 1024; }
__host__ __device__ __forceinline__ int gate_bytes(const Dims &d, int nw) {
    const int n = slice_bytes(tiles_gate(d), d.H), p = XR_PROJ_BYTES(nw);
    return n > p ? n : p;
}
__host__ __device__ __forceinline__ int joiner_bytes(const Dims &d) { return slice_bytes(tiles_joiner(d), d.Dj); }

// LDS of a launch.  bf16: the slices of the three weight matrices; the round's scratch lies over the projection's slice and the
// projection's tiles over the first pieces of the gates', and what was written over is fetched again (from the L2) before it
// is next needed.  fp32: the joiner's and the projection's slices, the gates' where they fit too (else they come from the
// L2 and the memory-side cache every round, straight into registers), and a scratch for the round and for `tiles` products of
// 16 x 16 whose K is shared by up to four waves.
struct XcdLds {
    int wG, wJ, wP, scratch, proj, bytes;   // offsets, and all of it
    int tiles;
};
template <int SMAX>
__host__ __device__ inline size_t scratch_bytes(int N, int BCAP) {
    const size_t b_list = ((size_t)BCAP * (sizeof(double) + sizeof(u64) + 3 * sizeof(int)) + 15) & ~(size_t)15;
    return b_list + (SMAX > 5 ? 0 : (size_t)N * sizeof(ExpandShared<SMAX, 1>)) + sizeof(float) * ((size_t)N * SMAX + N + 2 * (size_t)N * N);
}
__host__ __device__ __forceinline__ int long_bytes(int Vl) { return (int)((sizeof(LongShared) + 15) & ~(size_t)15) + LONG_FOLD_SHARES * Vl * 4; }
__host__ __device__ __forceinline__ int slice_bytes_f32(int tiles, int K) { return (tiles + XR_WGS - 1) / XR_WGS * f32_pieces(K) * 1024; }
template <int SMAX, bool F32>
__host__ __device__ inline XcdLds xcd_lds(const Dims &d, int nw, int limit) {
    XcdLds l{};
    int round = ((int)scratch_bytes<SMAX>(d.N, d.BCAP) + 15) & ~15;
    if (SMAX > 5 && long_bytes(d.Vl) > round) round = long_bytes(d.Vl);
    if (!F32) {
        l.wJ = gate_bytes(d, nw);
        l.wP = l.scratch = l.wJ + joiner_bytes(d);
        const int p = slice_bytes(tiles_proj(d), d.H);
        l.bytes = l.wP + (p > round ? p : round);
        return l;
    }
    const int g = slice_bytes_f32(tiles_gate(d), d.H), j = slice_bytes_f32(tiles_joiner(d), d.Dj), p = slice_bytes_f32(tiles_proj(d), d.H);
    for (int stay = 1; stay >= 0; --stay)
        for (l.tiles = nw; l.tiles >= 2; --l.tiles) {   // (fewer tiles at a time: more turns)
            const int part = l.tiles * 4096, s = part > round ? part : round;
            l.wG = stay ? 0 : -1;
            l.wJ = stay ? g : 0;
            l.wP = l.wJ + j;
            l.scratch = l.proj = l.wP + p;
            l.bytes = l.scratch + s;
            if (l.bytes <= limit && (l.tiles >= 4 || !stay)) return l;
        }
    return l;
}

template <bool F32>
__device__ __forceinline__ unsigned char *amat_of(const XcdArgs &g, const XcdPlace &w) {
    return static_cast<unsigned char *>(g.amat) + (long)g.tile0[w.x] * 16 * (F32 ? f32_row(g.d.Dj) * 4 : g.d.Dj * 2);
}
template <bool F32>
__device__ __forceinline__ long amat_size(const XcdArgs &g, const XcdPlace &w) {
    return (long)((w.nu * g.d.N * g.d.S + 15) >> 4) * 16 * (F32 ? f32_row(g.d.Dj) * 4 : g.d.Dj * 2);
}
template <bool F32>
__device__ __forceinline__ const typename XcdType<F32>::quad *enc_of(const XcdArgs &g, int frame, int c0) {
    return static_cast<const typename XcdType<F32>::quad *>(g.enc) + ((long)frame * g.d.Dj + c0) / 4;
}

// A = ChooseNBest(B); B = []; d = (s, 0, ..., 0)   (Algorithm 1, head of the outer loop), a workgroup per utterance: of a
// launch's first segment.  Those behind it find it done, see xcd_next.
template <int NT>
__device__ __forceinline__ void xcd_head(const XcdPlace &w, XcdShared &sh, double *s_bl) {
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int N = d.N, S = d.S, tid = w.tid;
    int4 *desc = desc_of(g, w, w.half);
    for (int i = w.r, k = 0; i < w.n_act; i += XR_WGS, ++k) {
        const int u = __builtin_amdgcn_readfirstlane(sh.utt[i]), sp = __builtin_amdgcn_readfirstlane(sh.sp[i]);
        const int nB = __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_NB]);
        const int parity = __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_PAR]) ^ 1;
        __syncthreads();   // (everybody has read the figures, and the scores of the utterance before)
        if (sp == 0) {
            if (tid < N) desc[i * N + tid] = make_int4(-1, 0, 0, 0);
            if (tid == 0) {
                sh.fig[k][TBS_FIG_SP] = 0;
                sh.fig[k][TBS_FIG_CNT] = 0;
            }
            continue;
        }
        const long bb = (long)u * d.BCAP;
        for (int e = tid; e < nB; e += NT) s_bl[e] = g.B.logs[bb + e];
        // (what a survivor takes along is asked for beside the scores)
        const int e0 = min(tid, nB - 1);
        const int my_slot = g.B.slot[bb + e0], my_node = g.B.node[bb + e0], my_len = g.B.len[bb + e0];
        const u64 my_hash = g.B.hash[bb + e0];
        __syncthreads();
        const int cnt = min(nB, N);
        for (int e = tid; e < nB; e += NT) {
            const double si = s_bl[e];
            const int rank = rank_in_list<4>(s_bl, nB, e);
            if (rank < N) {
                const bool mine = e == tid;
                const long at = (long)u * N + rank, b = bb + e;
                const int slot = mine ? my_slot : g.B.slot[b], dst = tbs_slot_id(u, parity, 0, rank, d.R, N);
                g.A[0].logs[at] = si;
                g.A[0].node[at] = mine ? my_node : g.B.node[b];
                g.A[0].hash[at] = mine ? my_hash : g.B.hash[b];
                g.A[0].len[at] = mine ? my_len : g.B.len[b];
                g.A[0].pslot[at] = slot;
                g.A[0].slot[at] = dst;
                g.A[0].pnode[at] = -1;
                g.A[0].token[at] = -1;
                float *dh = g.A[0].dhat + at * S;
                dh[0] = 0.f;
                for (int t = 1; t < S; ++t) dh[t] = -INFINITY;
                desc[i * N + rank] = make_int4(dst, slot, 0, 0);
            }
        }
        if (tid < N && tid >= cnt) desc[i * N + tid] = make_int4(-1, 0, 0, 0);
        if (tid == 0) {
            g.A[0].count[u] = cnt;
            g.rv.utt_par[u] = parity;
            sh.fig[k][TBS_FIG_SP] = sp;
            sh.fig[k][TBS_FIG_CNT] = cnt;
            sh.fig[k][TBS_FIG_NB] = 0;
            sh.fig[k][TBS_FIG_PAR] = parity;
        }
    }
}

// The survivors' state into this segment's arena, and the joiner input rows of the first round: every CU moves the
// columns that it makes and reads itself (16 of p, and 4 of h and c, per tile of its shares).  (The segment's frames, which nobody has touched
// yet, are asked for beside the descriptors, not behind them: 64 utterances S = 3 9.86 -> 9.72 ms per decode, S = 20 14.3 -> 14.2.)
template <int NT, int SMAX, bool F32>
__device__ __forceinline__ void xcd_carry(const XcdPlace &w, XcdShared &sh) {
    typedef typename XcdType<F32>::quad quad;
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int N = d.N, S = d.S, P = w.n_act * N;
    const rsrc_t r_desc = rsrc_of(desc_of(g, w, w.half), (long)w.nu * N * 16);
    unsigned char *amat = amat_of<F32>(g, w);
    const float rcp_n = __builtin_amdgcn_rcpf((float)N);   // p / N as (p + 0.5) * (1 / N): exact for p < 1024
    const int ownG = own_tiles(tiles_gate(d), w.r), nP = own_tiles(tiles_proj(d), w.r) * 4, per = nP + ownG;
    const float rcp_i = __builtin_amdgcn_rcpf((float)per);
    for (int it = w.tid; it < P * per; it += NT) {
        const int p = (int)(((float)it + 0.5f) * rcp_i), j = it - p * per;   // (exact: fewer than 2^16 items)
        const uintx4 ds = fresh16(r_desc, (unsigned)p * 16u, 0u);
        if (j < nP) {
            const int c0 = (w.r + (j >> 2) * XR_WGS) * 16 + (j & 3) * 4;
            if (F32 && c0 >= d.Dj) continue;
            const int i = (int)(((float)p + 0.5f) * rcp_n), sp = sh.sp[i];
            const quad *ef = enc_of<F32>(g, sp > 0 ? sh.f0[i] : 0, c0);
            constexpr int FR = SMAX > 5 ? 4 : SMAX;   // frames asked for at a time: the first before anything else has come
            quad ev[FR];
#pragma unroll
            for (int t = 0; t < FR; ++t) ev[t] = ef[(long)max(min(t, sp - 1), 0) * (d.Dj >> 2)];
            if ((int)ds[0] < 0) continue;
            const long dst = (int)ds[0], src = (int)ds[1];
            const float4 v = *reinterpret_cast<const float4 *>(g.pool_p + src * d.Dj + c0);
            for (int t0 = 0; t0 < (SMAX > 5 ? sp : 1); t0 += FR) {
                if (t0 > 0)
#pragma unroll
                    for (int t = 0; t < FR; ++t) ev[t] = ef[(long)min(t0 + t, sp - 1) * (d.Dj >> 2)];
                if (t0 == 0) *reinterpret_cast<float4 *>(g.pool_p + dst * d.Dj + c0) = v;
#pragma unroll
                for (int t = 0; t < FR; ++t)
                    if (t0 + t < sp) put_joiner_quad(amat, p * S + t0 + t, c0, d.Dj, ev[t], v, g.act);
            }
        } else if ((int)ds[0] >= 0) {
            const long dst = (int)ds[0], src = (int)ds[1];
            const int c0 = (w.r + (j - nP) * XR_WGS) * 4;
            const float4 h = *reinterpret_cast<const float4 *>(g.pool_h + src * d.H + c0);
            const float4 c = *reinterpret_cast<const float4 *>(g.pool_c + src * d.H + c0);
            *reinterpret_cast<float4 *>(g.pool_h + dst * d.H + c0) = h;
            *reinterpret_cast<float4 *>(g.pool_c + dst * d.H + c0) = c;
            if constexpr (F32) {
                float *row = static_cast<float *>(g.hb) + dst * f32_row(d.H);
                *reinterpret_cast<float2 *>(row + f32_at(c0)) = make_float2(h.x, h.y);
                *reinterpret_cast<float2 *>(row + f32_at(c0 + 2)) = make_float2(h.z, h.w);
            } else {
                *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(g.hb) + dst * d.H + c0) =
                    make_uint2(xr_bf16(h.x) | (xr_bf16(h.y) << 16), xr_bf16(h.z) | (xr_bf16(h.w) << 16));
            }
        }
    }
}

// Joiner: the logits of all rows (Section 3.1).  A wave takes 16 rows at a time, all of K in registers.
template <int NT, int C>
__device__ __forceinline__ void xcd_joiner(const XcdPlace &w, const unsigned char *wJ) {
    constexpr int NW = NT / 64, steps = 4 * C;
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int own = own_tiles(tiles_joiner(d), w.r), lane = w.lane;
    const int M = w.n_act * d.N * d.S, rtiles = (M + 15) >> 4;
    const rsrc_t r_amat = rsrc_of(amat_of<false>(g, w), amat_size<false>(g, w));
    float *logits = g.logits + (long)w.u_base * d.N * d.S * d.Vl;
    const int groups = own > 1 && rtiles < NW ? own : 1;   // (few rows: the tiles of columns by different waves)
    if (own == 0) return;
    for (int task = w.wave; task < rtiles * groups; task += NW) {
        const int rt = groups > 1 ? task / groups : task, gi = task - rt * groups;
        bf16x8 xf[steps];
#pragma unroll
        for (int s = 0; s < steps; ++s)
            xf[s] = __builtin_bit_cast(bf16x8, fresh16(r_amat, (unsigned)lane * 16u, (unsigned)(rt * steps + s) * 1024u));
        const int row = rt * 16 + (lane & 15);
        for (int i = gi; i < own; i += 2 * groups) {
            const int i1 = i + groups;
            float b[2][4];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    b[q][c] = g.b_out[min((w.r + min(q ? i1 : i, own - 1) * XR_WGS) * 16 + (lane >> 4) * 4 + c, d.V - 1)];
            floatx4 acc[2];
            if (i1 < own) mma<2, C>(acc, xf, wJ + (size_t)i * steps * 1024, wJ + (size_t)i1 * steps * 1024, lane);
            else mma<1, C>(acc, xf, wJ + (size_t)i * steps * 1024, nullptr, lane);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int ii = q ? i1 : i, col = (w.r + ii * XR_WGS) * 16 + (lane >> 4) * 4;
                if (ii < own && row < M && col < d.Vl) {
                    float o[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) o[c] = col + c < d.V ? acc[q][c] + b[q][c] : -INFINITY;
                    *reinterpret_cast<float4 *>(logits + (long)row * d.Vl + col) = make_float4(o[0], o[1], o[2], o[3]);
                }
            }
        }
    }
}

// The head of the outer loop for an utterance whose list A is empty, by a wave beside the select wave (xcd_finish, which then has
// little to do) while the other utterances' rounds go on: what the select step left of B in LDS and its ranking make the next
// segment's list.  The segment itself then begins with xcd_carry.  As a step of its own, behind the last round's barrier and with a
// barrier of its own: ms per decode, 64 utterances N = 5 S = 1 13.0 (now 12.1), S = 3 9.97 (9.86), S = 20 the same, 200 utterances 15.2 (14.9),
// 16 fp32 12.4 (12.1), one 4.82 (4.70).  (By the select wave behind its own part: S = 1 12.3.)
template <int SMAX, class SM>
__device__ __forceinline__ void xcd_next(const XcdPlace &w, XcdShared &sh, const SM &sm, const SelectOut &s_out, unsigned char *scratch, int round,
                                         int i, int k) {
    if (!__builtin_amdgcn_readfirstlane(sh.more[k])) return;
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int lane = w.lane, N = w.N;
    if (!(g.max_rounds > 0 && round >= g.max_rounds)) {   // (does the select wave keep a candidate? its test, see select_merge_utt)
        const int c = lane < N ? sm.s_sel[lane] : -1;
        const bool have_thr = sm.have_thr() != 0;
        if (__ballot(c >= 0 && (!have_thr || sm.s_key[max(c, 0)] > sm.thr())) != 0) return;
    }
    const XcdScratch<SMAX> sc(scratch, d);
    const int S = d.S, cnt = min(__builtin_amdgcn_readfirstlane(s_out.nB), N), u = __builtin_amdgcn_readfirstlane(sh.utt[i]);
    const int parity = __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_PAR]) ^ 1;
    const double *blogs = reinterpret_cast<const double *>(sc.b_list);
    const u64 *bhash = reinterpret_cast<const u64 *>(blogs + d.BCAP);
    const int *bnode = reinterpret_cast<const int *>(bhash + d.BCAP), *blen = bnode + d.BCAP, *bslot = blen + d.BCAP;
    // (places that no number has taken: scores that are NaN, behind all numbers, so that every place of the list has an entry)
    if (__builtin_expect(__ballot(lane < cnt && sm.s_match[min(lane, cnt - 1)] < 0) != 0, 0)) {
        const int nB = __builtin_amdgcn_readfirstlane(s_out.nB);
        for (int i = lane; i < nB; i += 64) {
            const double v = blogs[i];
            const int rank = v != v ? rank_placed(blogs, nB, v, i, 0) : N;
            if (rank < N) sm.s_match[rank] = i;
        }
        sel_sync();
    }
    if (lane < N) {
        int4 ds = make_int4(-1, 0, 0, 0);
        if (lane < cnt) {
            const int e = sm.s_match[lane], slot = bslot[e], dst = tbs_slot_id(u, parity, 0, lane, d.R, N);
            const long at = (long)u * N + lane;
            g.A[0].logs[at] = blogs[e];
            g.A[0].node[at] = bnode[e];
            g.A[0].hash[at] = bhash[e];
            g.A[0].len[at] = blen[e];
            g.A[0].pslot[at] = slot;
            g.A[0].slot[at] = dst;
            g.A[0].pnode[at] = -1;
            g.A[0].token[at] = -1;
            ds = make_int4(dst, slot, 0, 0);
        }
        desc_of(g, w, w.half ^ 1)[i * N + lane] = ds;
    }
    for (int h = 0; h < cnt; ++h)
        if (lane < S) g.A[0].dhat[((long)u * N + h) * S + lane] = lane == 0 ? 0.f : -INFINITY;   // (S <= 64)
    if (lane == 0) {   // (the figures take their values when the segment begins)
        g.rv.utt_par[u] = parity;
        sh.next[k] = cnt;
    }
}

// Threshold test, the new list A and what depends on it (trie nodes, descriptors, the figures), by the select wave.
template <int SMAX, bool FEW, class SM>
__device__ __forceinline__ void xcd_finish(const XcdPlace &w, XcdShared &sh, SM &sm, SelectOut &s_out, unsigned char *scratch, int round,
                                           int a, int i, int k, int sp, int H) {
    const int lane = w.lane, N = w.N;
    const XcdArgs &g = xcd_args();
    const XcdScratch<SMAX> sc(scratch, g.d);
    const int drop = g.max_rounds > 0 && round >= g.max_rounds, u = __builtin_amdgcn_readfirstlane(sh.utt[i]);
    AView An = g.A[a ^ 1];
    An.parents = nullptr;   // (the gates of every new hypothesis are formed whole)
    SelectIn in{};
    in.lc = sc.lc;
    in.slot_rows = 1;
    const SelectFigs fg{sp, H, i * N * g.d.S, 0, __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_PAR])};
    // (its logits are in LDS already; that it has some is all it needs to know)
    select_merge_utt(sm, 5, g.d, round, drop, u, lane, LogitsPlain{g.logits}, in, fg, An, An, g.B, g.rv, g.nodes, sc.b_list, &s_out,
                     FEW, true);
    sel_sync();
    const int used0 = sh.fig[k][TBS_FIG_USED], ncap = sh.fig[k][TBS_FIG_CAP], nbase = sh.fig[k][TBS_FIG_BASE];
    const int total = s_out.total;
    bool full = false;
    if (lane < N) {
        int4 ds = make_int4(-1, 0, 0, 0);
        if (lane < total) {
            const int tok = s_out.tok[lane];
            full = used0 + lane >= ncap;
            const int node = full ? 0 : nbase + used0 + lane;
            if (!full) g.nodes[node] = make_int2(s_out.pnode[lane], tok);
            An.node[(long)u * N + lane] = node;
            ds = make_int4(s_out.slot[lane], s_out.pslot[lane], tok, 0);
        }
        desc_of(g, w, w.half)[i * N + lane] = ds;
    }
    const bool any_full = __ballot(full) != 0;
    if (lane == 0) {
        sh.fig[k][TBS_FIG_CNT] = total;
        sh.fig[k][TBS_FIG_NB] = s_out.nB;
        sh.fig[k][TBS_FIG_USED] = min(used0 + total, ncap);
        sh.made = total | (any_full ? XR_FULL_TRIE : 0);
    }
}

// Eq. 3-7, the N best expansions, AddAndMerge, the new list A: a workgroup per utterance, a wave per hypothesis and one for
// the select step, which stages the lists while the others expand, and merges the blank expansions and finds the threshold while
// they pick their N best.  Then all the others rank the candidates, 16 a wave, four lanes sharing one, and the select wave
// makes the new list.
// (Each role reads the arguments it needs for itself and asks for what it waits for longest before all else.)
// Returns the hypotheses made (and XR_FULL_TRIE where an utterance's share of the trie was full).
template <int NT, int NV4, int SMAX, bool FEW, bool PUSH, class SM>
__device__ __forceinline__ int xcd_round(const XcdPlace &w, XcdShared &sh, SM &sm, SelectOut &s_out, unsigned char *scratch, int round,
                                         int a, int &calls, int &joined, int &nodes_made) {
    constexpr int NW = NT / 64;
    int live = 0;
    for (int i = w.r, k = 0; i < w.n_act; i += XR_WGS, ++k) {
        const int tid = w.tid, lane = w.lane, wave = w.wave, N = w.N;
        float xpre = 0.f;
        if (wave < N) {
            const XcdArgs &g = xcd_args();
            const Dims &d = g.d;
            const int S = d.S, row0 = (i * N + wave) * S;
            const rsrc_t r_logits = rsrc_of(g.logits + (long)w.u_base * N * S * d.Vl, (long)w.nu * N * S * d.Vl * 4);
            float e[SMAX][NV4 * 4];
            expand_load_fresh<NV4, SMAX>(e, r_logits, row0, S, d.Vl, lane);
            const int t = min(lane, S - 1);
            const float lbv = fresh4(r_logits, (unsigned)((row0 + t) * d.Vl + d.blank) * 4u, 0u);
            const float doldv = g.A[a].dhat[((long)sh.utt[i] * N + wave) * S + t];
            asm volatile("" ::: "memory");   // (the requests go out here, not behind the branch)
            const int sp = __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_SP]);
            const int H = sp > 0 ? __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_CNT]) : 0;
            if (H > 0) {   // (the same for the whole workgroup)
                const bool live_team = wave < H;
                const XcdScratch<SMAX> sc(scratch, d);
                ExpandPair<SMAX> pi;
                pi.pair = 0;
                pi.row0 = row0;
                pi.sp = live_team ? sp : 0;
#pragma unroll
                for (int q = 0; q < SMAX; ++q) {
                    pi.dold[q] = q < pi.sp ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(doldv), q)) : -INFINITY;
                    pi.lblank[q] = q < pi.sp ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lbv), q)) : 0.f;
                }
#pragma unroll
                for (int q = 0; q < SMAX; ++q)
                    if (q >= pi.sp) {   // (uniform) not a frame: whatever was read, it must be a number
#pragma unroll
                        for (int c = 0; c < NV4 * 4; ++c) e[q][c] = 0.f;
                    }
                float cf[SMAX];
                expand_front<NV4, SMAX, 64>(e, cf, pi, sc.teams[wave], d, lane, live_team, sc.lc + wave * sp, sc.dphi + wave, nullptr);
                __syncthreads();
                expand_back<NV4, SMAX, 64>(e, cf, pi, sc.teams[wave], d, lane, live_team, sc.cs + wave * N, sc.ct + wave * N, nullptr);
                if (live_team) {
                    // the team's candidates as keys of the joint ranking; the logits of their tokens at the segment's frames,
                    // a lane each (N S <= 64), wait in a register until the ranking is done
                    sel_sync();
                    if (lane < N) {
                        const int tok = sc.ct[wave * N + lane];
                        sm.s_ctok[wave * N + lane] = tok;
                        sm.s_key[wave * N + lane] = tok >= 0 ? sm.s_alogs[wave] + (double)sc.cs[wave * N + lane] : nan("");
                    }
                    const int q = min(lane / SMAX, N - 1), tq = lane - lane / SMAX * SMAX;
                    const int tok = max(sc.ct[wave * N + q], 0);
                    xpre = fresh4(r_logits, (unsigned)((row0 + min(tq, sp - 1)) * d.Vl + tok) * 4u, 0u);
                }
            }
        } else {
            const int sp = __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_SP]);
            const int H = sp > 0 ? __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_CNT]) : 0;
            if (H > 0) {
                if (wave == N) {
                    const XcdArgs &g = xcd_args();
                    const XcdScratch<SMAX> sc(scratch, g.d);
                    const int u = __builtin_amdgcn_readfirstlane(sh.utt[i]);
                    SelectIn in{};
                    in.dphi = sc.dphi;
                    const SelectFigs fg{sp, H, i * N * g.d.S, __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_NB]), 0};
                    select_merge_utt(sm, 1, g.d, round, 0, u, lane, LogitsPlain{nullptr}, in, fg, g.A[a], g.A[a ^ 1], g.B, g.rv, g.nodes,
                                     sc.b_list, &s_out, FEW, true);
                    __syncthreads();
                    select_merge_utt(sm, 6, g.d, round, 0, u, lane, LogitsPlain{nullptr}, in, fg, g.A[a], g.A[a ^ 1], g.B, g.rv, g.nodes,
                                     sc.b_list, &s_out, FEW, true);
                } else {
                    __syncthreads();
                }
            }
        }
        const int sp = __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_SP]);
        const int H = sp > 0 ? __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_CNT]) : 0;
        if (H == 0) {   // (the same for the whole workgroup)
            const XcdArgs &g = xcd_args();
            if (tid < N) desc_of(g, w, w.half)[i * N + tid] = make_int4(-1, 0, 0, 0);
            continue;
        }
        __syncthreads();
        if (wave != N) {
            sel_rank_waves(sm, reinterpret_cast<const double *>(scratch), s_out.nB, H * N, N, wave < N ? wave : wave - 1, NW - 1, lane);
            if (wave < H) {
                const int q = lane / SMAX, tq = lane - q * SMAX;
                if (q < N) sm.s_xpre[tq * SM::pc + wave * N + q] = xpre;
            }
        }
        __syncthreads();
        if (wave == N) xcd_finish<SMAX, FEW>(w, sh, sm, s_out, scratch, round, a, i, k, sp, H);
        else if (!PUSH && wave == 0) xcd_next<SMAX>(w, sh, sm, s_out, scratch, round, i, k);
        __syncthreads();
        const int made = __builtin_amdgcn_readfirstlane(sh.made);
        live += made;
        calls += 1;
        joined += sp;
        nodes_made += made & (XR_FULL_TRIE - 1);
    }
    return live;
}

// Long segments: the hypotheses of the XCD's utterances by its workgroups in turn (a hypothesis has up to 64 rows of logits;
// the utterance's own workgroup would be alone with all of them).
template <int NT, int NQ, int SMAX>
__device__ __forceinline__ void xcd_expand_long(const XcdPlace &w, XcdShared &sh, unsigned char *scratch, int a) {
    static_assert(SMAX <= LONG_FRAMES && SMAX % (NT / 64) == 0 && NT / 64 == LONG_FOLD_WAVES, "rows of a wave");
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int N = w.N, S = d.S, P = w.n_act * N;
    const long pair0 = (long)w.u_base * N;
    const rsrc_t r_desc = rsrc_of(desc_of(g, w, w.half), (long)w.nu * N * 16);
    const rsrc_t r_logits = rsrc_of(g.logits + pair0 * S * d.Vl, (long)w.nu * N * S * d.Vl * 4);
    const rsrc_t r_dhat = rsrc_of(g.A[a].dhat, (long)g.all_utts * N * S * 4);
    LongShared &sm = *reinterpret_cast<LongShared *>(scratch);
    float4 *s_part = reinterpret_cast<float4 *>(scratch + ((sizeof(LongShared) + 15) & ~(size_t)15));
    for (int p = w.r; p < P; p += XR_WGS) {
        const int i = p / N, h = p - i * N;
        const int slot = __builtin_amdgcn_readfirstlane((int)fresh16(r_desc, (unsigned)p * 16u, 0u)[0]);
        const int sp = __builtin_amdgcn_readfirstlane(sh.sp[i]), u = __builtin_amdgcn_readfirstlane(sh.utt[i]);
        if (slot < 0 || sp == 0) continue;   // (the same for the whole workgroup)
        expand_long<NQ, SMAX / (NT / 64), true>(
            d, sp, NT / 64, LONG_FOLD_SHARES, w.tid, sm, s_part,
            [&](int t) { return fresh4(r_dhat, (unsigned)((u * N + h) * S + t) * 4u, 0u); },
            [&](int t, int piece) { return as_float4(fresh16(r_logits, (unsigned)piece * 16u, (unsigned)(p * S + t) * (unsigned)d.Vl * 4u)); },
            [&](int t, int col) { return fresh4(r_logits, (unsigned)((p * S + t) * d.Vl + col) * 4u, 0u); }, g.row_lc + (pair0 + p) * S,
            g.dphi + pair0 + p, g.cand_score + (pair0 + p) * N, g.cand_tok + (pair0 + p) * N, nullptr, nullptr);
        __syncthreads();
    }
}

// ... and the select step of an utterance by its own workgroup, whose waves then make the frame distributions of the new
// hypotheses, one each.
template <int NT, int SMAX, class SM>
__device__ __forceinline__ int xcd_select_long(const XcdPlace &w, XcdShared &sh, SM &sm, SelectOut &s_out, unsigned char *scratch, int round,
                                               int a, int &calls, int &joined, int &nodes_made) {
    constexpr int NW = NT / 64;
    int live = 0;
    for (int i = w.r, k = 0; i < w.n_act; i += XR_WGS, ++k) {
        const int tid = w.tid, lane = w.lane, wave = w.wave, N = w.N;
        const int sp = __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_SP]);
        const int H = sp > 0 ? __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_CNT]) : 0;
        const XcdArgs &g = xcd_args();
        const Dims &d = g.d;
        const long pair = (long)w.u_base * N + (long)i * N;
        if (H == 0) {   // (the same for the whole workgroup)
            if (tid < N) desc_of(g, w, w.half)[i * N + tid] = make_int4(-1, 0, 0, 0);
            continue;
        }
        const XcdScratch<SMAX> sc(scratch, d);
        const int u = __builtin_amdgcn_readfirstlane(sh.utt[i]), nc = H * N;
        SelectIn in{};
        in.dphi = sc.dphi;
        const SelectFigs fg{sp, H, i * N * d.S, __builtin_amdgcn_readfirstlane(sh.fig[k][TBS_FIG_NB]), 0};
        if (wave == N) {
            select_merge_utt(sm, 1, d, round, 0, u, lane, LogitsPlain{nullptr}, in, fg, g.A[a], g.A[a ^ 1], g.B, g.rv, g.nodes, sc.b_list,
                             &s_out, true, false);
        } else {   // what the expansion left, from the L2
            const rsrc_t r_cs = rsrc_of(g.cand_score + pair * N, N * N * 4), r_ct = rsrc_of(g.cand_tok + pair * N, N * N * 4);
            const rsrc_t r_dphi = rsrc_of(g.dphi + pair, N * 4), r_lc = rsrc_of(g.row_lc + pair * d.S, (long)N * d.S * 4);
            const int tt = (wave < N ? wave : wave - 1) * 64 + lane, n = (NW - 1) * 64;
            if (tt < nc) {
                sc.cs[tt] = fresh4(r_cs, (unsigned)tt * 4u, 0u);
                sc.ct[tt] = __float_as_int(fresh4(r_ct, (unsigned)tt * 4u, 0u));
            }
            if (tt < H) sc.dphi[tt] = fresh4(r_dphi, (unsigned)tt * 4u, 0u);
            const float rcp_sp = __builtin_amdgcn_rcpf((float)sp);   // (exact quotients of up to 7 x 64 rows)
            for (int e = tt; e < H * sp; e += n) {
                const int h = (int)(((float)e + 0.5f) * rcp_sp);
                sc.lc[e] = fresh4(r_lc, (unsigned)(h * d.S + e - h * sp) * 4u, 0u);
            }
        }
        __syncthreads();
        if (wave == N) {
            select_merge_utt(sm, 6, d, round, 0, u, lane, LogitsPlain{nullptr}, in, fg, g.A[a], g.A[a ^ 1], g.B, g.rv, g.nodes, sc.b_list,
                             &s_out, true, false);
        } else if (wave < H && lane < N) {
            const int c = wave * N + lane, tok = sc.ct[c];
            sm.s_ctok[c] = tok;
            sm.s_key[c] = tok >= 0 ? sm.s_alogs[wave] + (double)sc.cs[c] : nan("");
        }
        __syncthreads();
        if (wave != N) sel_rank_waves(sm, reinterpret_cast<const double *>(scratch), s_out.nB, nc, N, wave < N ? wave : wave - 1, NW - 1, lane);
        __syncthreads();
        if (wave == N) xcd_finish<SMAX, true>(w, sh, sm, s_out, scratch, round, a, i, k, sp, H);
        else if (wave == 0) xcd_next<SMAX>(w, sh, sm, s_out, scratch, round, i, k);
        __syncthreads();
        const int made = __builtin_amdgcn_readfirstlane(sh.made), total = made & (XR_FULL_TRIE - 1);
        if (wave < total) {   // (at most N < NW)
            const rsrc_t r_logits = rsrc_of(g.logits + pair * d.S * d.Vl, (long)N * d.S * d.Vl * 4);
            const int h = __builtin_amdgcn_readfirstlane(sm.s_kh[wave]), tok = __builtin_amdgcn_readfirstlane(sm.s_ktok[wave]);
            const int t = min(lane, sp - 1);
            const float xv = fresh4(r_logits, (unsigned)((h * d.S + t) * d.Vl + tok) * 4u, 0u) + sc.lc[h * sp + t];
            const float xx = lane < sp ? xv : -INFINITY;
            const float mx = wave_max(xx);
            const float ex = lane < sp ? __expf(xx - mx) : 0.f;
            float sum = 0.f;   // (in the order of the select step: one after the other, or by a butterfly over the frames)
            if (sp <= SEL_PRE_FRAMES) {
#pragma unroll
                for (int q = 0; q < SEL_PRE_FRAMES; ++q) sum += lane_f(ex, q);   // (zero beyond S')
            } else {
                sum = wave_sum_far(ex);
            }
            const float lz = mx + __logf(sum);
            float *dh = g.A[a ^ 1].dhat + ((long)u * N + wave) * d.S;
            if (lane < d.S) dh[lane] = lane < sp ? xx - lz : -INFINITY;
        }
        __syncthreads();
        live += made;
        calls += 1;
        joined += sp;
        nodes_made += total;
    }
    return live;
}

// UpdatePredictorOutput: the LSTM layer.  Lane l of a tile's result holds the four gates of one unit of one hypothesis.
template <int NT, int C>
__device__ __forceinline__ void xcd_gates(const XcdPlace &w, const unsigned char *wG) {
    constexpr int NW = NT / 64, steps = 4 * C;
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int own = own_tiles(tiles_gate(d), w.r), lane = w.lane;
    const int P = w.n_act * d.N, ptiles = (P + 15) >> 4;
    const rsrc_t r_desc = rsrc_of(desc_of(g, w, w.half), (long)w.nu * d.N * 16), r_hb = rsrc_of(g.hb, g.hb_bytes);
    const int groups = min(own, max(1, NW / ptiles));   // (few rows: the tiles of columns by different waves)
    for (int task = w.wave; task < ptiles * groups; task += NW) {
        const int rt = task / groups, gi = task - rt * groups;
        const int p = rt * 16 + (lane & 15);
        const uintx4 ds = fresh16(r_desc, (unsigned)min(p, P - 1) * 16u, 0u);
        const bool on = p < P && (int)ds[0] >= 0;
        const long slot = (int)ds[0], pslot = (int)ds[1], tok = (int)ds[2];
        bf16x8 xf[steps];
        const unsigned at = (unsigned)pslot * (unsigned)d.H * 2u + (unsigned)(lane >> 4) * 16u;
#pragma unroll
        for (int s = 0; s < steps; ++s) xf[s] = __builtin_bit_cast(bf16x8, fresh16(r_hb, at, (unsigned)s * 64u));
#pragma unroll 1
        for (int i = gi; i < own; i += 2 * groups) {
            const int i1 = i + groups;
            float4 e4[2];
            float cp[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int unit = (w.r + min(q ? i1 : i, own - 1) * XR_WGS) * 4 + (lane >> 4);
                e4[q] = *reinterpret_cast<const float4 *>(g.emb_gates + (tok * d.H + unit) * 4);
                cp[q] = g.pool_c[pslot * d.H + unit];
            }
            floatx4 acc[2];
            if (i1 < own) mma<2, C>(acc, xf, wG + (size_t)i * steps * 1024, wG + (size_t)i1 * steps * 1024, lane);
            else mma<1, C>(acc, xf, wG + (size_t)i * steps * 1024, nullptr, lane);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int ii = q ? i1 : i;
                if (ii < own && on) {
                    const int unit = (w.r + ii * XR_WGS) * 4 + (lane >> 4);
                    const float ig = xr_sigmoid(acc[q][0] + e4[q].x), fgt = xr_sigmoid(acc[q][1] + e4[q].y),
                                gg = tanhf(acc[q][2] + e4[q].z), og = xr_sigmoid(acc[q][3] + e4[q].w);
                    const float cn = fgt * cp[q] + ig * gg;
                    const float hn = og * tanhf(cn);
                    g.pool_c[slot * d.H + unit] = cn;
                    g.pool_h[slot * d.H + unit] = hn;
                    static_cast<bf16_t *>(g.hb)[slot * d.H + unit] = (bf16_t)xr_bf16(hn);
                }
            }
        }
    }
}

// UpdatePredictorOutput: the projection, and the joiner input rows of the next round.  A wave makes a tile of 16 hypotheses x
// 16 columns, as many at a time as there are waves, and leaves it in LDS; then all threads form the rows, four
// columns of one frame each (the few waves that have tiles would take longer over the activations than over the products).
// The first frames are asked for between the halves of the barrier ahead.
template <int NT, int C, int FR>
__device__ __forceinline__ int xcd_project(const XcdPlace &w, XcdShared &sh, XcdBarrier &bar, const unsigned char *wP, unsigned char *scratch) {
    constexpr int NW = NT / 64, steps = 4 * C;
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int own = own_tiles(d.Dj >> 4, w.r), lane = w.lane, S = d.S;
    const int P = w.n_act * w.N, ptiles = (P + 15) >> 4;
    const int per = own > 0 ? NW / own : 0;                  // row tiles at a time (own <= 2)
    const rsrc_t r_desc = rsrc_of(desc_of(g, w, w.half), (long)w.nu * w.N * 16), r_hb = rsrc_of(g.hb, g.hb_bytes);
    unsigned char *amat = amat_of<false>(g, w);
    const float rcp_n = __builtin_amdgcn_rcpf((float)w.N);
    float *s_p = reinterpret_cast<float *>(scratch);         // [per * 16 hypotheses][own * 16]
    int *s_on = reinterpret_cast<int *>(s_p + NW * 256);     // [per * 16]
    // item of the second half: columns 4 q .. of hypothesis p0 + h at frames f .. f + FR - 1
    const int q_n = own * 4, fg_n = (S + FR - 1) / FR;
    int q = 0, h = 0, f = 0, p0 = 0, n = 0, left = 0;
    uint2 ev[FR];
    auto item = [&](int it) {
        const float rq = __builtin_amdgcn_rcpf((float)q_n), rn = __builtin_amdgcn_rcpf((float)n);
        const int hf = (int)(((float)it + 0.5f) * rq);       // (exact: fewer than 2^16 items)
        q = it - hf * q_n;
        f = (int)(((float)hf + 0.5f) * rn);
        h = hf - f * n;
        f *= FR;
    };
    auto frames = [&]() {   // asks for them, and how many there are
        const int i = (int)(((float)(p0 + h) + 0.5f) * rcp_n), sp = sh.sp[i], c0 = (w.r + (q >> 2) * XR_WGS) * 16 + (q & 3) * 4;
        // (beyond the utterance's frames any frame that exists will do)
#pragma unroll
        for (int t = 0; t < FR; ++t) ev[t] = *enc_of<false>(g, sp > 0 ? sh.f0[i] + min(f + t, sp - 1) : 0, c0);
        return sp - f;
    };
    n = min(P, per * 16);
    if (w.tid < n * q_n * fg_n) {
        item(w.tid);
        left = frames();
    }
    const int sum = xcd_wait<false>(bar, sh.sum);
    if (sum < 0) return sum;
    if (own == 0) return 0;
    for (int rt0 = 0; rt0 < ptiles; rt0 += per) {
        const int rt = rt0 + w.wave / own;
        p0 = rt0 * 16;
        n = min(P - p0, per * 16);
        if (w.wave < per * own && rt < ptiles) {
            const int ti = w.wave % own, p = rt * 16 + (lane & 15), c0 = (w.r + ti * XR_WGS) * 16 + (lane >> 4) * 4;
            const float4 b = *reinterpret_cast<const float4 *>(g.b_proj + c0);
            const uintx4 ds = fresh16(r_desc, (unsigned)min(p, P - 1) * 16u, 0u);
            const bool on = p < P && (int)ds[0] >= 0;
            const long slot = max((int)ds[0], 0);
            const unsigned at = (unsigned)slot * (unsigned)d.H * 2u + (unsigned)(lane >> 4) * 16u;
            bf16x8 xf[steps];
#pragma unroll
            for (int s = 0; s < steps; ++s) xf[s] = __builtin_bit_cast(bf16x8, fresh16(r_hb, at, (unsigned)s * 64u));
            floatx4 acc[2];
            mma<1, C>(acc, xf, wP + (size_t)ti * steps * 1024, nullptr, lane);
            const float4 pv = make_float4(acc[0][0] + b.x, acc[0][1] + b.y, acc[0][2] + b.z, acc[0][3] + b.w);
            *reinterpret_cast<float4 *>(s_p + ((rt - rt0) * 16 + (lane & 15)) * own * 16 + ti * 16 + (lane >> 4) * 4) = pv;
            if (ti == 0 && lane < 16) s_on[(rt - rt0) * 16 + lane] = on;
            if (on) *reinterpret_cast<float4 *>(g.pool_p + slot * d.Dj + c0) = pv;
        }
        __syncthreads();
        for (int it = w.tid; it < n * q_n * fg_n; it += NT) {
            if (rt0 > 0 || it >= NT) {
                item(it);
                left = frames();
            }
            if (left > 0 && s_on[h]) {
                const float4 v = *reinterpret_cast<const float4 *>(s_p + h * own * 16 + q * 4);
#pragma unroll
                for (int t = 0; t < FR; ++t)
                    if (t < left)
                        put_joiner_quad(amat, (p0 + h) * S + f + t, (w.r + (q >> 2) * XR_WGS) * 16 + (q & 3) * 4, d.Dj, ev[t], v, g.act);
            }
        }
        if (rt0 + per < ptiles) __syncthreads();
    }
    return 0;
}

// ------------------------------------------------------------------ fp32 products
// Products of fp32 models: 16 x 16 tiles, K in the four shares and two sums a share of the slot layout's fp32 GEMM (the same
// bits).  A task is a tile's share: its sum goes to LDS, part[tile][share][lane], where whoever goes on with the tile adds the
// shares up.  C chunks of 128 of K; x(tile, piece) and wt(tile, piece) ask for 16 bytes a lane.
template <int NT, int C, class X, class W>
__device__ __forceinline__ void f32_shares(float4 *part, int tiles, int K, int wave, int lane, X x, W wt) {
    const int eights = K >> 3, pieces = f32_pieces(K), shares = min(4, (eights + 3) >> 2);
    for (int task = wave; task < tiles * shares; task += NT / 64) {
        const int tile = task / shares, s = task - tile * shares;
        float4 wv[2 * C], xv[2 * C];
#pragma unroll
        for (int q = 0; q < 2 * C; ++q) wv[q] = wt(tile, min((q >> 1) * 8 + s * 2 + (q & 1), pieces - 1));
#pragma unroll
        for (int q = 0; q < 2 * C; ++q) xv[q] = x(tile, min((q >> 1) * 8 + s * 2 + (q & 1), pieces - 1));
        floatx4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
#pragma unroll
        for (int q = 0; q < 2 * C; ++q) {
            const int e = ((q >> 1) * 8 + s * 2 + (q & 1)) * 2;
            if (q < 2 * C - 2 || e < eights) {       // (uniform; only the last chunk can be short)
                a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[q].x, xv[q].x, a0, 0, 0, 0);
                a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[q].y, xv[q].y, a1, 0, 0, 0);
            }
            if (q < 2 * C - 2 || e + 1 < eights) {
                a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[q].z, xv[q].z, a0, 0, 0, 0);
                a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[q].w, xv[q].w, a1, 0, 0, 0);
            }
        }
        part[(tile * 4 + s) * 64 + lane] = make_float4(a0[0] + a1[0], a0[1] + a1[1], a0[2] + a1[2], a0[3] + a1[3]);
    }
}
__device__ __forceinline__ float4 f32_sum(const float4 *part, int tile, int lane, int K) {
    const int shares = min(4, ((K >> 3) + 3) >> 2);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < shares; ++s) {
        const float4 q = part[(tile * 4 + s) * 64 + lane];
        v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
    }
    return v;
}
template <class F>
__device__ __forceinline__ void by_chunks_f32(int K, F fn) { by_chunks((K + 127) & ~127, fn); }

template <int NT, int C>
__device__ __forceinline__ void xcd_joiner_f32(const XcdPlace &w, const float4 *wJ, float4 *part, int at_once) {
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int own = own_tiles(tiles_joiner(d), w.r), lane = w.lane, pieces = f32_pieces(d.Dj);
    const int M = w.n_act * d.N * d.S, tiles = ((M + 15) >> 4) * own;
    const rsrc_t r_amat = rsrc_of(amat_of<true>(g, w), amat_size<true>(g, w));
    float *logits = g.logits + (long)w.u_base * d.N * d.S * d.Vl;
    for (int t0 = 0; t0 < tiles; t0 += at_once) {
        const int n = min(at_once, tiles - t0);
        f32_shares<NT, C>(part, n, d.Dj, w.wave, lane,
                          [&](int t, int m) { return as_float4(fresh16(r_amat, (unsigned)lane * 16u, (unsigned)((t0 + t) / own * pieces + m) * 1024u)); },
                          [&](int t, int m) { return wJ[((t0 + t) % own * pieces + m) * 64 + lane]; });
        __syncthreads();
        for (int t = w.wave; t < n; t += NT / 64) {
            const int row = (t0 + t) / own * 16 + (lane & 15), col = (w.r + (t0 + t) % own * XR_WGS) * 16 + (lane >> 4) * 4;
            const float4 v = f32_sum(part, t, lane, d.Dj);
            if (row < M && col < d.Vl) {
                const float v4[4] = {v.x, v.y, v.z, v.w};
                float o[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) o[c] = col + c < d.V ? v4[c] + g.b_out[min(col + c, d.V - 1)] : -INFINITY;
                *reinterpret_cast<float4 *>(logits + (long)row * d.Vl + col) = make_float4(o[0], o[1], o[2], o[3]);
            }
        }
        if (t0 + at_once < tiles) __syncthreads();
    }
}

// (wG null: the gates' slice is read from memory)
template <int NT, int C>
__device__ __forceinline__ void xcd_gates_f32(const XcdPlace &w, const float4 *wG, float4 *part, int at_once) {
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int own = own_tiles(tiles_gate(d), w.r), lane = w.lane, pieces = f32_pieces(d.H);
    const int P = w.n_act * d.N, tiles = ((P + 15) >> 4) * own;
    const rsrc_t r_desc = rsrc_of(desc_of(g, w, w.half), (long)w.nu * d.N * 16), r_hb = rsrc_of(g.hb, g.hb_bytes);
    const float4 *wfrag = static_cast<const float4 *>(g.w_gate);
    for (int t0 = 0; t0 < tiles; t0 += at_once) {
        const int n = min(at_once, tiles - t0);
        int rt_of = -1;
        unsigned at = 0;
        f32_shares<NT, C>(part, n, d.H, w.wave, lane,
                          [&](int t, int m) {
                              const int rt = (t0 + t) / own;
                              if (rt != rt_of) {   // (uniform)
                                  const uintx4 ds = fresh16(r_desc, (unsigned)min(rt * 16 + (lane & 15), P - 1) * 16u, 0u);
                                  at = ds[1] * (unsigned)f32_row(d.H) * 4u + (unsigned)(lane >> 4) * 16u;
                                  rt_of = rt;
                              }
                              return as_float4(fresh16(r_hb, at, (unsigned)m * 64u));
                          },
                          [&](int t, int m) {
                              const int i = (t0 + t) % own;
                              return wG ? wG[(i * pieces + m) * 64 + lane] : wfrag[((long)(w.r + i * XR_WGS) * pieces + m) * 64 + lane];
                          });
        __syncthreads();
        for (int t = w.wave; t < n; t += NT / 64) {
            const int p = (t0 + t) / own * 16 + (lane & 15), unit = (w.r + (t0 + t) % own * XR_WGS) * 4 + (lane >> 4);
            const uintx4 ds = fresh16(r_desc, (unsigned)min(p, P - 1) * 16u, 0u);
            if (p >= P || (int)ds[0] < 0) continue;
            const long slot = (int)ds[0], pslot = (int)ds[1], tok = (int)ds[2];
            const float4 e4 = *reinterpret_cast<const float4 *>(g.emb_gates + (tok * d.H + unit) * 4);
            const float cp = g.pool_c[pslot * d.H + unit];
            const float4 v = f32_sum(part, t, lane, d.H);
            const float cn = xr_sigmoid(v.y + e4.y) * cp + xr_sigmoid(v.x + e4.x) * tanhf(v.z + e4.z);
            const float hn = xr_sigmoid(v.w + e4.w) * tanhf(cn);
            g.pool_c[slot * d.H + unit] = cn;
            g.pool_h[slot * d.H + unit] = hn;
            static_cast<float *>(g.hb)[slot * f32_row(d.H) + f32_at(unit)] = hn;
        }
        if (t0 + at_once < tiles) __syncthreads();
    }
}

template <int NT, int C>
__device__ __forceinline__ void xcd_project_f32(const XcdPlace &w, XcdShared &sh, const float4 *wP, float4 *part, int at_once) {
    const XcdArgs &g = xcd_args();
    const Dims &d = g.d;
    const int own = own_tiles(tiles_proj(d), w.r), lane = w.lane, pieces = f32_pieces(d.H), S = d.S;
    const int P = w.n_act * d.N, ptiles = (P + 15) >> 4;
    const rsrc_t r_desc = rsrc_of(desc_of(g, w, w.half), (long)w.nu * d.N * 16), r_hb = rsrc_of(g.hb, g.hb_bytes);
    unsigned char *amat = amat_of<true>(g, w);
    const float rcp_n = __builtin_amdgcn_rcpf((float)w.N);
    if (own == 0) return;
    const int per = max(1, at_once / own);   // row tiles at a time
    for (int rt0 = 0; rt0 < ptiles; rt0 += per) {
        const int nr = min(per, ptiles - rt0), n = nr * own, p0 = rt0 * 16;
        int rt_of = -1;
        unsigned at = 0;
        f32_shares<NT, C>(part, n, d.H, w.wave, lane,
                          [&](int t, int m) {
                              const int rt = rt0 + t / own;
                              if (rt != rt_of) {   // (uniform)
                                  const uintx4 ds = fresh16(r_desc, (unsigned)min(rt * 16 + (lane & 15), P - 1) * 16u, 0u);
                                  at = (unsigned)max((int)ds[0], 0) * (unsigned)f32_row(d.H) * 4u + (unsigned)(lane >> 4) * 16u;
                                  rt_of = rt;
                              }
                              return as_float4(fresh16(r_hb, at, (unsigned)m * 64u));
                          },
                          [&](int t, int m) { return wP[(t % own * pieces + m) * 64 + lane]; });
        __syncthreads();
        // columns 4 q .. of hypothesis p0 + h at frame f; the first frame's also stores the projection
        const int hs = min(P - p0, nr * 16), q_n = own * 4;
        const float rq = __builtin_amdgcn_rcpf((float)q_n), rn = __builtin_amdgcn_rcpf((float)hs);
        for (int it = w.tid; it < hs * q_n * S; it += NT) {
            const int hf = (int)(((float)it + 0.5f) * rq), q = it - hf * q_n;       // (exact: fewer than 2^14 items)
            const int f = (int)(((float)hf + 0.5f) * rn), h = hf - f * hs, p = p0 + h;
            const int c0 = (w.r + (q >> 2) * XR_WGS) * 16 + (q & 3) * 4;
            if (c0 >= d.Dj) continue;
            const int i = (int)(((float)p + 0.5f) * rcp_n), sp = sh.sp[i];
            const uintx4 ds = fresh16(r_desc, (unsigned)p * 16u, 0u);
            const float4 ev = *enc_of<true>(g, sp > 0 ? sh.f0[i] + min(f, sp - 1) : 0, c0);
            const float4 b = *reinterpret_cast<const float4 *>(g.b_proj + c0);
            if ((int)ds[0] < 0 || f >= sp) continue;
            float4 v = f32_sum(part, (h >> 4) * own + (q >> 2), (q & 3) * 16 + (h & 15), d.H);
            v = make_float4(v.x + b.x, v.y + b.y, v.z + b.z, v.w + b.w);
            if (f == 0) *reinterpret_cast<float4 *>(g.pool_p + (long)(int)ds[0] * d.Dj + c0) = v;
            put_joiner_quad(amat, p * S + f, c0, d.Dj, ev, v, g.act);
        }
        if (rt0 + per < ptiles) __syncthreads();
    }
}

// NT threads, room for a wave per hypothesis and one for the select step; FEW: beams up to 8 (see select_merge_utt).
// PUSH: a push of a stream, one segment whose figures and frames come with the launch.  (A kernel of its own: a launch runs through its code
// once for a push, and what the one does not need of the other's, it does not fetch.  Utterances of 60 to 150 frames, ms: 64 streams N = 5 S = 3, three
// frames a push, 5.74 -> 5.56, 100 of N = 8 8.22 -> 7.87, 64 utterances as a batch 3.83 -> 3.78.)
template <int NT, int NV4, int SMAX, bool FEW, bool F32, bool PUSH>
__global__ void __launch_bounds__(NT)
k_xcd_decode(XcdArgs args) {
    static_assert(!PUSH || (!F32 && SMAX <= 5), "other models' streams have row lists");
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    __shared__ XcdShared sh;
    __shared__ SelectOut s_out;
    TBS_SELECT_ARRAYS(s_select, (SMAX > 5 ? 64 : XR_CANDS), (SMAX > 5 ? 0 : 1), (SMAX > 5 ? 1 : SMAX), (FEW ? 64 : XR_CANDS));
    XcdPlace w;
    w.tid = threadIdx.x;
    w.lane = w.tid & 63;
    w.wave = __builtin_amdgcn_readfirstlane(w.tid >> 6);
    w.N = args.d.N;
    const int tid = w.tid, lane = w.lane;

    // ---- all here?
    if (tid == 0) {
        XcdCtl *ctl = args.ctl;
        const int x = (int)(__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u);   // (the number of this CU's XCD: hwreg 20, 4 bits)
        const int xc = min(x, XR_XCDS - 1);
        // (Places are counted per XCD; the last of an XCD's workgroups counts the XCD, waits for the others' and tells its own.
        // A word that all 256 count in takes them one after the other: 10.5 -> 4.7 us a launch until the first segment with the
        // small fp32 configuration, 12.4 -> 8.5 with 64 utterances.)
        const unsigned r = __hip_atomic_fetch_add(&ctl->place[xc * 32], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool leads = r == XR_WGS - 1;
        unsigned st = 0;
        if (leads && __hip_atomic_fetch_add(&ctl->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)args.expect - 1) {
            unsigned none = 0;
            __hip_atomic_compare_exchange_strong(&ctl->state, &none, 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        unsigned *word = leads ? &ctl->state : &ctl->told[xc * 32];
        const u64 t0 = wall_clock64();
        while ((st = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
            if (wall_clock64() - t0 > XR_PATIENCE_MS * XR_TICKS) {   // (who decides first decides for all)
                unsigned none = 0;
                __hip_atomic_compare_exchange_strong(&ctl->state, &none, 2u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                word = &ctl->state;
            }
        }
        if (leads) __hip_atomic_store(&ctl->told[xc * 32], st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool ok = st == 1 && x < XR_XCDS && r < XR_WGS;
        sh.where[0] = xc;
        sh.where[1] = (int)r;
        sh.where[2] = ok;
    }
    __syncthreads();
    w.x = __builtin_amdgcn_readfirstlane(sh.where[0]);
    w.r = __builtin_amdgcn_readfirstlane(sh.where[1]);
    if (!sh.where[2]) {
        if (tid == 0) store_host(args.host + 4 * (int)blockIdx.x + 3, (args.seq << 8) | XR_ABSENT);
        return;
    }
    // (the words of the launch after this one; the launch before it has ended)
    if (w.x == 0 && w.r == 0)
        for (int i = tid; i < (int)(sizeof(XcdCtl) / sizeof(unsigned)); i += NT) reinterpret_cast<unsigned *>(args.ctl_next)[i] = 0u;

    w.u_base = args.first[w.x];
    w.nu = args.first[w.x + 1] - w.u_base;
    int status = XR_DONE, calls = 0, joined = 0, nodes_made = 0;   // (of this workgroup's utterances)
    if (w.nu > 0) {
        constexpr int NW = NT / 64;
        unsigned char *wG, *wJ, *wP, *scratch;
        int at_once = 0;
        {
            const XcdArgs &g = xcd_args();
            const Dims &d = g.d;
            const XcdLds l = xcd_lds<SMAX, F32>(d, NW, XR_LDS(F32 || d.N > 7));
            wG = s_dyn + l.wG;
            wJ = s_dyn + l.wJ;
            wP = s_dyn + l.wP;
            scratch = s_dyn + l.scratch;
            at_once = l.tiles;
            const int pH = F32 ? f32_pieces(d.H) : d.H >> 5;
            int2 step = make_int2(0, 0);
            int4 rows = make_int4(0, 0, 0, 0);
            if (PUSH && tid < w.nu) step = g.push_step[w.u_base + tid];
            if (PUSH && w.r < w.nu) rows = g.push_rows[w.u_base + w.r];
            if (l.wG < 0) wG = nullptr;
            else load_frags(wG, g.w_gate, pH, 0, own_tiles(tiles_gate(d), w.r) * pH, w.r, w.wave, NW, lane);
            load_rows<F32>(wJ, g.w_out, d.V, d.Dj, own_tiles(tiles_joiner(d), w.r), w.r, w.wave, NW, lane);
            if (F32) load_rows<F32>(wP, g.w_proj, d.Dj, d.H, own_tiles(tiles_proj(d), w.r), w.r, w.wave, NW, lane);
            if (tid < w.nu) sh.utt[tid] = g.order[w.u_base + tid];
            // A push brings its frames and figures with it: who has the utterance appends the frames to its buffer, while the
            // weights come (the first that reads them does so behind a barrier).  With a copy of the figures and a kernel that
            // appends in front of the launch a push of one segment of 64 streams took 116 us, now 107.
            if (PUSH) {
                if (tid < w.nu) {
                    sh.sp[tid] = step.x;
                    sh.f0[tid] = step.y;
                    if (w.r == 0) {
                        g.utt_T[sh.utt[tid]] = step.x;
                        g.utt_off[sh.utt[tid]] = step.y;
                    }
                }
                for (int i = w.r; i < w.nu; i += XR_WGS) {
                    if (i != w.r) rows = g.push_rows[w.u_base + i];
                    const uint4 *from = g.push_from + (long)rows.x * g.push_units;
                    uint4 *to = g.push_to + (long)rows.y * g.push_units;
                    for (int j = tid; j < rows.z * g.push_units; j += NT) to[j] = from[j];
                }
            }
            __syncthreads();
            for (int i = w.r, k = 0; i < w.nu; i += XR_WGS, ++k)
                if (tid < TBS_FIG_SIZE) {
                    const int u = sh.utt[i];
                    sh.fig[k][tid] = tid == TBS_FIG_NB ? g.B.count[u] : (tid == TBS_FIG_PAR ? g.rv.utt_par[u] : g.fig[u * TBS_FIG_SIZE + tid]);
                }
        }
        // (thread i: length and first frame of utterance i, for every segment of the launch)
        int my_T = 0, my_off = 0;
        if (tid < w.nu && !PUSH) {
            my_T = args.utt_T[sh.utt[tid]];
            my_off = args.utt_off[sh.utt[tid]];
        }
        XcdBarrier bar{&args.ctl->bar[w.x * 16], 0u, 0u};
        const int seg0 = args.seg0, seg1 = args.seg1, R = args.d.R, Dj = args.d.Dj, Hh = args.d.H;
        for (int seg = seg0; seg < seg1 && status == XR_DONE; ++seg) {
            // frames of the XCD's utterances in this segment; utterances beyond the last that has any are left out
            {
                const XcdArgs &g = xcd_args();
                const int left = my_T - seg * g.d.S;   // (a push has one segment, and its figures already)
                if (tid < w.nu && !PUSH) {
                    sh.sp[tid] = left < 0 ? 0 : min(left, g.d.S);
                    sh.f0[tid] = my_off + seg * g.d.S;
                }
                if (!PUSH && tid < w.nu && (tid & (XR_WGS - 1)) == w.r) {   // (one of this workgroup's)
                    const int k = tid / XR_WGS;
                    sh.more[k] = seg + 1 < seg1 && left > g.d.S;
                    if (seg > seg0) {
                        sh.fig[k][TBS_FIG_SP] = left < 0 ? 0 : min(left, g.d.S);
                        sh.fig[k][TBS_FIG_CNT] = 0;
                        if (left > 0) {
                            sh.fig[k][TBS_FIG_CNT] = sh.next[k];
                            sh.fig[k][TBS_FIG_NB] = 0;
                            sh.fig[k][TBS_FIG_PAR] ^= 1;
                        }
                    }
                }
                w.half = seg & 1;
                __syncthreads();
                const u64 some = __ballot(lane < w.nu && sh.sp[min(lane, w.nu - 1)] > 0);
                w.n_act = some ? 64 - __clzll(some) : 0;
                if (w.n_act == 0) break;   // (the same for the whole XCD; utterances come in falling length, or there is one step)
            }
            if (seg == seg0) {
                xcd_head<NT>(w, sh, reinterpret_cast<double *>(scratch));
                if (xcd_barrier(bar, sh.sum) < 0) { status = XR_STUCK; break; }
            }
            xcd_carry<NT, SMAX, F32>(w, sh);
            if (xcd_barrier(bar, sh.sum) < 0) { status = XR_STUCK; break; }
            int a = 0, round = 0;
            while (true) {   // while Length(A) > 0
                if (round + 1 > R) { status = XR_ROUNDS; break; }
                round += 1;
                if constexpr (F32)
                    by_chunks_f32(Dj, [&](auto c) {
                        xcd_joiner_f32<NT, c.value>(w, reinterpret_cast<const float4 *>(wJ), reinterpret_cast<float4 *>(scratch), at_once);
                    });
                else
                    by_chunks(Dj, [&](auto c) { xcd_joiner<NT, c.value>(w, wJ); });
                if (xcd_barrier(bar, sh.sum) < 0) { status = XR_STUCK; break; }
                int live;
                if constexpr (SMAX > 5) {
                    xcd_expand_long<NT, NV4, SMAX>(w, sh, scratch, a);
                    if (xcd_barrier(bar, sh.sum) < 0) { status = XR_STUCK; break; }
                    live = xcd_select_long<NT, SMAX>(w, sh, s_select, s_out, scratch, round, a, calls, joined, nodes_made);
                } else {
                    live = xcd_round<NT, NV4, SMAX, FEW, PUSH>(w, sh, s_select, s_out, scratch, round, a, calls, joined, nodes_made);
                }
                a ^= 1;
                xcd_arrive(bar, live);
                // The projection's slice again, where the round's scratch lies over it (only who has utterances of its own, or
                // hypotheses, writes over it): asked for in front of the wait where hypotheses go on, behind it where none of
                // one's own do, for then it is mostly the segment's last round, which needs it no more and would wait for it (64 utterances
                // S = 3 as streams 15.4 -> 14.8 ms, as a batch 10.57 -> 10.51, one utterance 5.26 -> 5.17; segments of one frame, whose other
                // utterances go on more often, 13.15 -> 13.25, of 20, where most workgroups have none, 14.27 -> 14.36: those ask in front).
                const bool refetch = !F32 && (SMAX > 5 || w.r < w.n_act || round == 1), now = SMAX == 1 || SMAX > 5 || live > 0 || round == 1;
                auto fetch = [&]() {
                    const XcdArgs &g = xcd_args();
                    load_rows<false>(wP, g.w_proj, g.d.Dj, g.d.H, own_tiles(g.d.Dj >> 4, w.r), w.r, w.wave, NW, lane);
                };
                if (refetch && now) fetch();
                const int sum = xcd_wait<true>(bar, sh.sum);
                if (sum < 0) { status = XR_STUCK; break; }
                if (sum >= XR_FULL_TRIE) { status = XR_TRIE; break; }
                if (sum == 0) break;
                if (refetch && !now) fetch();
                if constexpr (F32) {
                    by_chunks_f32(Hh, [&](auto c) {
                        xcd_gates_f32<NT, c.value>(w, reinterpret_cast<const float4 *>(wG), reinterpret_cast<float4 *>(scratch), at_once);
                    });
                    if (xcd_barrier(bar, sh.sum) < 0) { status = XR_STUCK; break; }
                    by_chunks_f32(Hh, [&](auto c) {
                        xcd_project_f32<NT, c.value>(w, sh, reinterpret_cast<const float4 *>(wP), reinterpret_cast<float4 *>(scratch), at_once);
                    });
                    if (xcd_barrier(bar, sh.sum) < 0) { status = XR_STUCK; break; }
                } else {
                    by_chunks(Hh, [&](auto c) { xcd_gates<NT, c.value>(w, wG); });
                    xcd_arrive(bar, 0);
                    int there = 0;
                    by_chunks(Hh, [&](auto c) { there = xcd_project<NT, c.value, (SMAX > 5 ? 4 : 1)>(w, sh, bar, wP, wG); });
                    if (there < 0) { status = XR_STUCK; break; }
                    xcd_arrive(bar, 0);
                    {
                        const XcdArgs &g = xcd_args();
                        const int all = own_tiles(tiles_gate(g.d), w.r) * (g.d.H >> 5);
                        load_frags(wG, g.w_gate, g.d.H >> 5, 0, min(all, (XR_PROJ_BYTES(NW) + 1023) / 1024), w.r, w.wave, NW, lane);
                    }
                    if (xcd_wait<false>(bar, sh.sum) < 0) { status = XR_STUCK; break; }
                }
            }
            if (w.r == 0 && tid == 0) store_host(args.host_rounds + w.x * XR_SEGS + (seg - seg0), round);
        }
        // what the next launch, or the kernels of the slot layout, go on from
        __syncthreads();
        const XcdArgs &g = xcd_args();
        for (int i = w.r, k = 0; i < w.nu; i += XR_WGS, ++k) {
            const int u = sh.utt[i];
            if (tid < TBS_FIG_SIZE) g.fig[u * TBS_FIG_SIZE + tid] = sh.fig[k][tid];
            if (tid == 0) {
                g.B.count[u] = sh.fig[k][TBS_FIG_NB];
                g.A[0].count[u] = 0;
                g.A[1].count[u] = 0;
            }
        }
    }
    if (tid == 0) {
        int *host = args.host + 4 * (int)blockIdx.x;
        store_host(host + 0, calls);
        store_host(host + 1, joined);
        store_host(host + 2, nodes_made);
        __builtin_amdgcn_s_waitcnt(0);   // the figures are acknowledged before the word that says so goes out
        store_host(host + 3, (args.seq << 8) | status);
    }
}

// ------------------------------------------------------------------ host
static int nv4_of(const Dims &d) {   // (as the round kernel of the slot layout: the same order of the sums)
    const int v4 = d.Vl / 4;
    return v4 <= 64 ? 1 : (v4 <= 128 ? 2 : 4);
}

template <bool F32>
static XcdLds lds_of(const Dims &d) {
    const int nw = d.N <= 7 ? 8 : 12, limit = XR_LDS(F32 || d.N > 7);
    if (d.S > 5) return d.S <= 16 ? xcd_lds<16, F32>(d, nw, limit) : d.S <= 32 ? xcd_lds<32, F32>(d, nw, limit) : xcd_lds<64, F32>(d, nw, limit);
    return d.S == 1 ? xcd_lds<1, F32>(d, nw, limit) : d.S <= 3 ? xcd_lds<3, F32>(d, nw, limit) : xcd_lds<5, F32>(d, nw, limit);
}

template <int NT, int NV4, int SMAX, bool FEW, bool F32, bool PUSH = false>
static hipError_t xcd_launch_t(hipStream_t st, const XcdArgs &g, int shm) {
    static int attr_for = 0;
    if (shm > attr_for) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_xcd_decode<NT, NV4, SMAX, FEW, F32, PUSH>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, shm);
        if (e != hipSuccess) return e;
        attr_for = shm;
    }
    hipLaunchKernelGGL((k_xcd_decode<NT, NV4, SMAX, FEW, F32, PUSH>), dim3(XR_XCDS * XR_WGS), dim3(NT), shm, st, g);
    return hipGetLastError();
}

template <int NT, int NV4, bool FEW, bool F32, bool PUSH>
static hipError_t xcd_launch_s(hipStream_t st, const XcdArgs &g, int shm) {
    if (g.d.S == 1) return xcd_launch_t<NT, NV4, 1, FEW, F32, PUSH>(st, g, shm);
    if (g.d.S <= 3) return xcd_launch_t<NT, NV4, 3, FEW, F32, PUSH>(st, g, shm);
    return xcd_launch_t<NT, NV4, 5, FEW, F32, PUSH>(st, g, shm);
}

template <int NT, bool FEW, bool F32, bool PUSH = false>
static hipError_t xcd_launch(hipStream_t st, const XcdArgs &g) {
    const int nv4 = nv4_of(g.d), shm = lds_of<F32>(g.d).bytes;
    if (nv4 == 1) return xcd_launch_s<NT, 1, FEW, F32, PUSH>(st, g, shm);
    if (nv4 == 2) return xcd_launch_s<NT, 2, FEW, F32, PUSH>(st, g, shm);
    return xcd_launch_s<NT, 4, FEW, F32, PUSH>(st, g, shm);
}

// the shapes both types have in common
[[maybe_unused]] static bool xcd_shape_fits(const Dims &d) {
    return d.L == 1 && (d.S <= 5 ? d.N <= 11 : d.S <= LONG_FRAMES && d.N <= 7) && d.V <= 1024 && d.Dj <= XR_KMAX && d.H <= XR_KMAX && d.BCAP <= 2048;
}
[[maybe_unused]] static bool xcd_batch_fits(const XcdArgs &g) {
    if (g.d.U > XR_XCDS * XR_POS) return false;
    for (int x = 0; x < XR_XCDS; ++x)
        if (g.first[x + 1] - g.first[x] > XR_POS) return false;
    return true;
}
