// Beam bookkeeping kernels of token-wise RNN-T beam search (Algorithm 1):
// ChooseNBest at the head of a segment, the row list of a joiner call,
// AddAndMerge / ChooseNthScore / ChooseNBestExpansions with the threshold
// test, and reading the N-best out of the token trie.
//
// One 64-lane wavefront owns one utterance, so every list operation of the
// algorithm is a few lane-parallel passes and nothing needs a grid-wide
// barrier.  Token sequences live in a trie of (parent, token) nodes; a
// hypothesis carries its node, length and a 64-bit hash; two hypotheses are
// "the same tokens" when hash and length agree and a walk up the trie agrees.
#include "tbs_internal.h"
#include "select_device.h"
#include <algorithm>

// ------------------------------------------------------------------ batch init
__global__ void k_init_batch(Dims d, BView B, AView A0, AView A1, RowView rv, int2 *nodes, float *pool_p,
                             float *pool_h, float *pool_c, const float *pred_init, long pool_rows, const int *told, int *fig,
                             int *order, int *utt_T, int *utt_off, int *live_sum) {
    int u = blockIdx.x;
    int tid = threadIdx.x;
    // the batch's figures, order of utterances, lengths and first frames from the host's memory
    if (tid < TBS_FIG_SIZE) fig[u * TBS_FIG_SIZE + tid] = told[u * TBS_FIG_SIZE + tid];
    const int *rest = told + d.U * TBS_FIG_SIZE;
    if (tid == 64) order[u] = rest[u];
    if (tid == 65) utt_T[u] = rest[d.U + u];
    if (tid == 66) utt_off[u] = rest[2 * d.U + u];
    if (tid == 67 && u == d.U - 1) utt_off[d.U] = rest[3 * d.U];
    if (tid < 2 && u == 0) live_sum[tid] = 0;
    // B = [([], 1, InitPredictor(), Null)]: the empty sequence is trie node 0;
    // its predictor state sits in the "previous segment" arena (parity 1).
    int slot = tbs_slot_id(u, 1, 0, 0, d.R, d.N);
    if (tid == 0) {
        B.count[u] = 1;
        B.logs[(long)u * d.BCAP] = 0.0;
        B.node[(long)u * d.BCAP] = 0;
        B.hash[(long)u * d.BCAP] = 0ull;
        B.len[(long)u * d.BCAP] = 0;
        B.slot[(long)u * d.BCAP] = slot;
        A0.count[u] = 0;
        A1.count[u] = 0;
        rv.utt_sp[u] = 0;
        rv.utt_pair0[u] = 0;
        rv.utt_par[u] = 1;
        if (u == 0) {
            nodes[0] = make_int2(-1, -1);
            rv.counts[TBS_CNT_PAIRS] = 0;
            rv.counts[TBS_CNT_ROWS] = 0;
            rv.counts[TBS_CNT_NODES] = 1;
            rv.counts[TBS_CNT_ERR] = 0;
            rv.counts[TBS_CNT_UTTS] = 0;
            rv.counts[TBS_CNT_FRAMES] = 0;
            rv.counts[TBS_CNT_SEQ] = 0;
            rv.counts[TBS_CNT_NODE_BASE] = 1;
            rv.counts[TBS_CNT_ACC_CALLS] = 0;
            rv.counts[TBS_CNT_ACC_JOINED] = 0;
            rv.counts[TBS_CNT_PARS] = 0;
        }
    }
    for (int j = tid; j < d.Dj; j += blockDim.x) pool_p[(long)slot * d.Dj + j] = pred_init[j];
    for (int l = 0; l < d.L; ++l)
        for (int j = tid; j < d.H; j += blockDim.x) {
            pool_h[((long)l * pool_rows + slot) * d.H + j] = 0.f;
            pool_c[((long)l * pool_rows + slot) * d.H + j] = 0.f;
        }
}

hipError_t launch_init_batch(hipStream_t st, const Dims &d, BView B, AView A0, AView A1, RowView rv, int2 *nodes,
                             float *pool_p, float *pool_h, float *pool_c, const float *pred_init,
                             long pool_rows, const int *told, int *fig, int *order, int *utt_T, int *utt_off, int *live_sum) {
    hipLaunchKernelGGL(k_init_batch, dim3(d.U), dim3(256), 0, st, d, B, A0, A1, rv, nodes, pool_p, pool_h, pool_c,
                       pred_init, pool_rows, told, fig, order, utt_T, utt_off, live_sum);
    return hipGetLastError();
}

// ------------------------------------------------------------------ segment head
// A = ChooseNBest(B); B = []; d = (s, 0, ..., 0)   (Algorithm 1, head of the outer loop)
// The workgroup ranks B and writes A; then it moves the survivors' predictor state into this
// segment's arena (slot r=0): the arena of the segment before last is reused, and a survivor may have
// been carried, untouched, from there.  In the slot layout it also forms the joiner input rows of the
// segment's first round, act(e_t + p) (Section 3.1), from the p values it is moving.
// A SIMD issues an instruction of one of its waves every few cycles, so what counts in a kernel of
// this size is the number of instructions per SIMD: a workgroup is four waves, one per SIMD, and in
// the slot layout, where a small batch leaves most of the chip idle, `parts` workgroups share an
// utterance: each ranks B for itself (a few hundred instructions) and moves its share of the
// survivors' rows, a 16-byte piece of one row per thread; the first also writes A and the
// descriptors.  With parts > 1 nothing that the other workgroups of the utterance still have to read
// is changed here: B's count and the arena flag are left to the round kernel that follows.
__device__ __forceinline__ unsigned seg_bf16(float f) {   // nearest, ties to even
    unsigned v = __float_as_uint(f);
    v += 0x7FFFu + ((v >> 16) & 1u);
    return v >> 16;
}
#define SEG_THREADS 256
// Row lists: one workgroup moves all of an utterance's survivors, 120 to 200 KB read and written at the large widths, and 256 utterances are one
// workgroup a CU: 16 waves keep four times the requests in flight (256 utterances, two layers 34.5 -> 30.6 us a launch; 1024, where four
// workgroups of 256 threads shared a CU, 70.0 and 70.4: 3.6 TB/s).
#define SEG_THREADS_WIDE 1024
#define SEG_ENC_LOADS ((TBS_FIXED_SMAX * 1024 / 4 + SEG_THREADS - 1) / SEG_THREADS)   // 8-byte pieces of S rows of up to 1024 columns, per thread
// four encoder values of a frame, in the storage type of the model
template <bool F32> struct SegPiece { typedef uint2 type; };
template <> struct SegPiece<true> { typedef float4 type; };
template <bool F32, int NT>
__global__ void __launch_bounds__(NT)
k_segment_begin(Dims d, int seg, const int *utt_T, BView B, AView A, RowView rv, float *pool_p,
                float *pool_h, float *pool_c, long pool_rows, FixedView fx) {
    __shared__ int s_src[TBS_MAX_BEAM], s_dst[TBS_MAX_BEAM];
    __shared__ int s_n;
    typedef typename SegPiece<F32>::type EP;
    constexpr bool ROWS = NT == SEG_THREADS;   // (joiner input rows: the slot layout alone)
    __shared__ EP s_enc[ROWS ? TBS_FIXED_SMAX * 1024 / 4 : 1];   // the segment's frames, [frame][4 columns]
    const int parts = fx.parts > 1 ? fx.parts : 1;
    const int u = blockIdx.x / parts, part = blockIdx.x - u * parts, tid = threadIdx.x;
    const bool first = part == 0;
    // Everything the head of the kernel needs is requested at once, before anything is known:
    // the utterance's figures and, per thread, one entry of B (the first NT entries
    // cover every list but the very longest), so that the ranking below starts after one memory
    // round trip instead of four.
    __shared__ double s_bl[2048];           // BCAP is at most 2048
    const long bb = (long)u * d.BCAP;
    const int e0 = min(tid, d.BCAP - 1);
    const int T_u = utt_T[u], nB = B.count[u], par_old = rv.utt_par[u];
    const double my_logs = B.logs[bb + e0];
    const int my_slot = B.slot[bb + e0], my_node = B.node[bb + e0], my_len = B.len[bb + e0];
    const u64 my_hash = B.hash[bb + e0];
    int left = T_u - seg * d.S;
    int sp = left < 0 ? 0 : (left > d.S ? d.S : left);
    // The frames of the segment come from memory nobody has touched yet, the slowest request of the
    // kernel: they are asked for now, behind the entries of B (requests come back in order), and wait
    // in registers until the ranking is done.  Asked for whether wanted or not, from an address that
    // exists in either case: a request behind a condition would make every later wait a wait for all.
    const bool rows_here = ROWS && fx.on && fx.amat != nullptr && sp > 0;
    const int cp = d.Dj >> 2;   // pieces of four columns in a row
    EP ev[SEG_ENC_LOADS];
    if constexpr (ROWS) {
        const EP *ebase = rows_here ? static_cast<const EP *>(fx.enc) + ((long)fx.utt_off[u] + (long)seg * d.S) * cp
                                    : reinterpret_cast<const EP *>(pool_p);
        const int pieces = rows_here ? sp * cp : 1;
#pragma unroll
        for (int q = 0; q < SEG_ENC_LOADS; ++q)
            ev[q] = ebase[min(tid + q * NT, pieces - 1)];   // (rows follow each other)
    }
    if (tid == 0) {
        if (first) rv.utt_sp[u] = sp;
        s_n = 0;
    }
    if (fx.on && tid == 0 && first) {
        rv.utt_pair0[u] = u * d.N;
        rv.utt_row0[u] = u * d.N * d.S;
        if (u == 0) fx.live_sum[(fx.seq + 1) & 1] = 0;   // the counter of the launch after this one
    }
    if (sp == 0) {  // finished (or empty) utterance: B keeps the final list
        if (!first) return;
        if (tid == 0) A.count[u] = 0;
        if (fx.on) {
            if (tid == 0) {
                int *fig = fx.fig + u * TBS_FIG_SIZE;
                fig[TBS_FIG_SP] = 0;
                fig[TBS_FIG_CNT] = 0;
            }
            if (tid < d.N) pair_mark_dead(rv, u * d.N + tid, u, d.S);
            if (tid == 0) store_host(fx.host_live + (fx.seq & 1) * d.U + u, fx.seq << 8);
        }
        return;
    }
    const int parity = par_old ^ 1;   // the arena the survivors are not in
    // the scores go through LDS: ranking by counting reads every score once per entry
    if (tid < nB) s_bl[tid] = my_logs;
    for (int i = tid + NT; i < nB; i += NT) s_bl[i] = B.logs[bb + i];
    __syncthreads();
    for (int i = tid; i < nB; i += NT) {
        const double si = s_bl[i];
        const int rank = rank_in_list<8>(s_bl, nB, i);
        if (rank < d.N) {
            const long a = (long)u * d.N + rank, b = bb + i;
            const bool mine = i == tid;
            const int src = mine ? my_slot : B.slot[b], dst = tbs_slot_id(u, parity, 0, rank, d.R, d.N);
            s_src[rank] = src;
            s_dst[rank] = dst;
            if (first) {
                A.logs[a] = si;
                A.node[a] = mine ? my_node : B.node[b];
                A.hash[a] = mine ? my_hash : B.hash[b];
                A.len[a] = mine ? my_len : B.len[b];
                A.pslot[a] = src;
                A.slot[a] = dst;
                A.pnode[a] = -1;
                A.token[a] = -1;
                float *dh = A.dhat + a * d.S;
                dh[0] = 0.f;   // d = (s, 0, ..., 0), normalised and as logarithms
                for (int t = 1; t < d.S; ++t) dh[t] = -INFINITY;
            }
        }
    }
    if (tid == 0) {
        if (first) A.count[u] = nB < d.N ? nB : d.N;
        s_n = nB < d.N ? nB : d.N;
    }
    if (rows_here) {
#pragma unroll
        for (int q = 0; q < SEG_ENC_LOADS; ++q)
            if (tid + q * NT < sp * cp) s_enc[tid + q * NT] = ev[q];
    }
    __syncthreads();
    if (tid == 0 && parts == 1) {   // (every thread has read the old values by now)
        rv.utt_par[u] = parity;
        B.count[u] = 0;
    }
    if (fx.on && first) {   // slot layout: this utterance's pair descriptors for the first round, its count to the host
        const int cnt = s_n;
        if (tid < d.N) {
            const int j = u * d.N + tid;
            if (tid < cnt) {
                rv.pair_u[j] = u;
                rv.pair_h[j] = tid;
                rv.pair_row0[j] = j * d.S;
                rv.pair_len[j] = sp;
                rv.pair_slot[j] = s_dst[tid];
                rv.pair_pslot[j] = s_src[tid];
                rv.pair_frame0[j] = fx.utt_off[u] + seg * d.S;
                rv.pair_tok[j] = -1;
            } else {
                pair_mark_dead(rv, j, u, d.S);
            }
        }
        if (tid == 0) {
            int *fig = fx.fig + u * TBS_FIG_SIZE;
            fig[TBS_FIG_SP] = sp;
            fig[TBS_FIG_CNT] = cnt;
            fig[TBS_FIG_NB] = 0;
            fig[TBS_FIG_PAR] = parity;
            atomicAdd(fx.live_sum + (fx.seq & 1), cnt);
            store_host(fx.host_live + (fx.seq & 1) * d.U + u, (fx.seq << 8) | cnt);
        }
    }
    // The survivors' predictor outputs and LSTM states move to their new slots: item (survivor k,
    // piece j) moves piece j (16 bytes where the widths allow) of the survivor's output row and of
    // its h and c rows of every layer, all requested before the first is stored.
    const int n = s_n;
    auto copy_all = [&](auto unit_tag, int w) {   // w = floats per unit
        using UNIT = decltype(unit_tag);
        const int up = d.Dj / w, uh = d.H / w, widest = max(up, uh);
        const float rcp_w = __builtin_amdgcn_rcpf((float)widest);   // (item / widest exactly, items < 2^16)
        for (int it = part * NT + tid; it < n * widest; it += parts * NT) {
            const int k = (int)(((float)it + 0.5f) * rcp_w), j = it - k * widest;
            const long src = s_src[k], dst = s_dst[k];
            const int jp = min(j, up - 1), jh = min(j, uh - 1);
            const UNIT vp = reinterpret_cast<const UNIT *>(pool_p + src * d.Dj)[jp];
            UNIT vh[TBS_MAX_LAYERS], vc[TBS_MAX_LAYERS];
#pragma unroll
            for (int l = 0; l < TBS_MAX_LAYERS; ++l)
                if (l < d.L) {   // (uniform)
                    vh[l] = reinterpret_cast<const UNIT *>(pool_h + ((long)l * pool_rows + src) * d.H)[jh];
                    vc[l] = reinterpret_cast<const UNIT *>(pool_c + ((long)l * pool_rows + src) * d.H)[jh];
                }
            if (j < up) reinterpret_cast<UNIT *>(pool_p + dst * d.Dj)[j] = vp;
            if (j < uh) {
#pragma unroll
                for (int l = 0; l < TBS_MAX_LAYERS; ++l)
                    if (l < d.L) {
                        reinterpret_cast<UNIT *>(pool_h + ((long)l * pool_rows + dst) * d.H)[j] = vh[l];
                        reinterpret_cast<UNIT *>(pool_c + ((long)l * pool_rows + dst) * d.H)[j] = vc[l];
                    }
            }
            if constexpr (sizeof(UNIT) == 16) {
                if (rows_here && j < up) {
                    // (hypothesis k of the utterance is pair u*N + k: rows from pair * S)
                    const float p4[4] = {vp.x, vp.y, vp.z, vp.w};
                    EP *arow = static_cast<EP *>(fx.amat) + (long)(u * d.N + k) * d.S * cp + j;
                    for (int t = 0; t < sp; ++t) {
                        const EP e = s_enc[t * cp + j];
                        if constexpr (F32) {
                            arow[(long)t * cp] = make_float4(
                                tbs_joiner_act_f32(e.x + p4[0], fx.act), tbs_joiner_act_f32(e.y + p4[1], fx.act),
                                tbs_joiner_act_f32(e.z + p4[2], fx.act), tbs_joiner_act_f32(e.w + p4[3], fx.act));
                        } else {
                            const float e4[4] = {__uint_as_float(e.x << 16), __uint_as_float(e.x & 0xFFFF0000u),
                                                 __uint_as_float(e.y << 16), __uint_as_float(e.y & 0xFFFF0000u)};
                            unsigned o[4];
#pragma unroll
                            for (int q = 0; q < 4; ++q) o[q] = seg_bf16(tbs_joiner_act(e4[q] + p4[q], fx.act));
                            arow[(long)t * cp] = make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
                        }
                    }
                }
            }
        }
    };
    if (((d.Dj | d.H) & 3) == 0) copy_all(float4{}, 4);
    else copy_all(float{}, 1);
}

hipError_t launch_segment_begin(hipStream_t st, const Dims &d, int seg, const int *utt_T, BView B,
                                AView A, RowView rv, float *pool_p, float *pool_h, float *pool_c, long pool_rows,
                                const FixedView *fx) {
    FixedView f{};
    if (fx) f = *fx;
    if (f.parts > 1 && !f.on) return hipErrorInvalidValue;   // (only the slot layout's round kernel finishes what the parts leave)
    const dim3 grid(d.U * (f.parts > 1 ? f.parts : 1)), block(SEG_THREADS);
    if (f.on && f.f32)
        hipLaunchKernelGGL((k_segment_begin<true, SEG_THREADS>), grid, block, 0, st, d, seg, utt_T, B, A, rv, pool_p, pool_h, pool_c,
                           pool_rows, f);
    else if (f.on)
        hipLaunchKernelGGL((k_segment_begin<false, SEG_THREADS>), grid, block, 0, st, d, seg, utt_T, B, A, rv, pool_p, pool_h, pool_c,
                           pool_rows, f);
    else
        hipLaunchKernelGGL((k_segment_begin<false, SEG_THREADS_WIDE>), grid, dim3(SEG_THREADS_WIDE), 0, st, d, seg, utt_T, B, A, rv, pool_p, pool_h,
                           pool_c, pool_rows, f);
    return hipGetLastError();
}

// ------------------------------------------------------------------ row list
// The joiner rows of a round are the (pair, frame) combinations of the live
// (utterance, hypothesis) pairs, compacted.  One workgroup (a wave) per
// utterance: each reads the counts of ALL utterances, which the kernel before it
// wrote, and sums those ahead of its own, so no workgroup waits for another and
// nothing travels between them; it then fills its pairs and rows and gives new
// hypotheses their trie nodes.  The first workgroup also owns the totals: it
// publishes them to the host, with the number of this launch last, before it
// fills anything.
__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ void rowfill_lists(const Dims &d, int seg, const int *utt_off, AView A, RowView rv, int2 *nodes,
                                              int assign_nodes, int *host_counts, int seq, int u, int lane, bool share,
                                              bool by_parent, int *s_pslot, int *s_pair0, int *s_cnt) {
    // trie nodes handed out so far: launches alternate between two slots, so that the first
    // workgroup can store the new figure while others still read the old one
    const int slot_old = (seq & 1) ? TBS_CNT_NODE_BASE : TBS_CNT_NODES;
    const int slot_new = (seq & 1) ? TBS_CNT_NODES : TBS_CNT_NODE_BASE;
    const bool by_list = A.parents != nullptr;   // (the parents of the new hypotheses are wanted)
    const int node_base = rv.counts[slot_old];
    const int frame0 = utt_off[u] + seg * d.S;
    // what the fill below needs of this utterance's hypotheses, lane h holding hypothesis h:
    // requested together with the counts, so the kernel costs one memory round trip, not two
    const long ah = (long)u * d.N + min(lane, d.N - 1);
    const int h_slot = A.slot[ah], h_pslot = A.pslot[ah], h_tok = A.token[ah], h_pnode = A.pnode[ah];
    int before_p = 0, before_r = 0, tot_p = 0, tot_r = 0, utts = 0, frames = 0, my_sp = 0, my_cnt = 0, before_q = 0, tot_q = 0;
    // (every request is made whatever the others bring, four turns at a time: 1024 utterances 12.7 -> 6.8 us a launch)
    const int *parents = by_list ? A.parents : A.count;
#pragma unroll 4
    for (int base = 0; base < d.U; base += WAVE) {
        const int v = base + lane, vc = min(v, d.U - 1);
        const int v_sp = rv.utt_sp[vc], v_cnt = A.count[vc], v_par = parents[vc];
        const int sp = v < d.U ? v_sp : 0;
        const int c = sp > 0 ? v_cnt : 0;
        const int r = c * sp, q = c > 0 ? v_par : 0;
        if (v < u) { before_p += c; before_r += r; before_q += q; }
        if (v == u) { my_sp = sp; my_cnt = c; }
        tot_p += c;
        tot_r += r;
        tot_q += q;
        utts += c > 0;
        frames += c > 0 ? sp : 0;
    }
    const int pair0 = wave_sum_int(before_p), row0 = wave_sum_int(before_r);
    const int sp = wave_sum_int(my_sp), cnt = wave_sum_int(my_cnt);
    if (u == 0) {
        tot_p = wave_sum_int(tot_p);
        tot_r = wave_sum_int(tot_r);
        utts = wave_sum_int(utts);
        frames = wave_sum_int(frames);
        tot_q = by_list ? wave_sum_int(tot_q) : 0;
        if (lane == 0) {
            int err = rv.counts[TBS_CNT_ERR];
            int nodes_used = node_base;
            if (assign_nodes) {
                nodes_used = node_base + tot_p;
                if (nodes_used > d.max_nodes) { err |= TBS_ERRF_NODES; nodes_used = d.max_nodes; }
            }
            // every row list is followed by one joiner call over its rows: the counters of Section
            // 4.2 (invocations, frames joined; per utterance summed) are kept here, so that the host
            // need not see every row list
            const int acc_calls = rv.counts[TBS_CNT_ACC_CALLS] + utts, acc_joined = rv.counts[TBS_CNT_ACC_JOINED] + frames;
            rv.counts[TBS_CNT_ACC_CALLS] = acc_calls;
            rv.counts[TBS_CNT_ACC_JOINED] = acc_joined;
            if (host_counts) {
                store_host(host_counts + TBS_CNT_ACC_CALLS, acc_calls);
                store_host(host_counts + TBS_CNT_ACC_JOINED, acc_joined);
                store_host(host_counts + TBS_CNT_PARS, tot_q);
                store_host(host_counts + TBS_CNT_PAIRS, tot_p);
                store_host(host_counts + TBS_CNT_ROWS, tot_r);
                store_host(host_counts + TBS_CNT_NODES, nodes_used);
                store_host(host_counts + TBS_CNT_ERR, err);
                store_host(host_counts + TBS_CNT_UTTS, utts);
                store_host(host_counts + TBS_CNT_FRAMES, frames);
                __builtin_amdgcn_s_waitcnt(0);   // the figures are acknowledged before their number goes out
                store_host(host_counts + TBS_CNT_SEQ, seq);
            }
            rv.counts[TBS_CNT_PARS] = tot_q;
            rv.counts[TBS_CNT_PAIRS] = tot_p;
            rv.counts[TBS_CNT_ROWS] = tot_r;
            rv.counts[slot_new] = nodes_used;
            rv.counts[TBS_CNT_ERR] = err;
            rv.counts[TBS_CNT_UTTS] = utts;
            rv.counts[TBS_CNT_FRAMES] = frames;
        }
    }
    if (lane == 0) {
        rv.utt_pair0[u] = pair0;
        rv.utt_row0[u] = row0;
    }
    // the hypotheses that this utterance's new ones were made from, in the order of their first ones
    int par0 = 0, n_par = 0, par_of = -1;
    if (by_list) {
        par0 = wave_sum_int(before_q);
        int first_of = lane;   // the first new hypothesis with this one's parent
        for (int g = cnt - 1; g >= 0; --g)
            if (__builtin_amdgcn_readlane(h_pslot, g) == h_pslot) first_of = g;
        const u64 firsts = __ballot(lane < cnt && first_of == lane);
        n_par = __popcll(firsts);
        par_of = __popcll(firsts & ((1ull << first_of) - 1ull));
        if (lane < cnt) {
            rv.pair_par[pair0 + lane] = par0 + par_of;
            if (first_of == lane) rv.par_slot[par0 + par_of] = h_pslot;
        }
        if (share && by_parent && lane < cnt && first_of == lane) s_pslot[par_of] = h_pslot;
    }
    for (int base = 0; base < cnt * sp; base += WAVE) {   // (cnt and sp are the same in every lane)
        const int idx = base + lane;
        const bool valid = idx < cnt * sp;
        const int h = valid ? idx / sp : 0, t = idx - h * sp;
        // every lane takes part in the exchanges, whatever it does with the result
        const int slot = __shfl(h_slot, h), pslot = __shfl(h_pslot, h), tok = __shfl(h_tok, h),
                  pnode = __shfl(h_pnode, h);
        if (!valid) continue;
        const long a = (long)u * d.N + h;
        rv.row_enc[row0 + idx] = frame0 + t;
        rv.row_slot[row0 + idx] = slot;
        if (t == 0) {
            const int j = pair0 + h;
            rv.pair_u[j] = u;
            rv.pair_h[j] = h;
            rv.pair_row0[j] = row0 + h * sp;
            rv.pair_len[j] = sp;
            rv.pair_slot[j] = slot;
            rv.pair_pslot[j] = pslot;
            rv.pair_frame0[j] = frame0;
            rv.pair_tok[j] = tok;
            if (assign_nodes) {
                const int node = node_base + j;
                if (node < d.max_nodes) {
                    nodes[node] = make_int2(pnode, tok);
                    A.node[a] = node;
                } else {
                    A.node[a] = 0;
                }
            }
        }
    }
    if (share) {   // for the other waves of the workgroup
        if (!by_parent && lane < d.N) s_pslot[lane] = h_pslot;
        if (lane == 0) {
            *s_pair0 = by_parent ? par0 : pair0;
            *s_cnt = by_parent ? n_par : cnt;
        }
    }
}

// With `gather` the workgroup has four waves: the first does all of the above, then all
// four write the rows of h that the gate products of this utterance's new hypotheses read (see HidRows), which would otherwise
// take a kernel of its own between this one and the gate GEMM.
__device__ __forceinline__ unsigned rowfill_bf16(float f) {
    unsigned v = __float_as_uint(f);
    v += 0x7FFFu + ((v >> 16) & 1u);   // round to nearest, ties to even
    return v >> 16;
}

__global__ void __launch_bounds__(256)
k_rowfill(Dims d, int seg, const int *utt_off, AView A, RowView rv, int2 *nodes, int assign_nodes, int *host_counts,
          int seq, HidRows gather) {
    __shared__ int s_pslot[TBS_MAX_BEAM];
    __shared__ int s_row0, s_rows;
    const int u = blockIdx.x;
    if (threadIdx.x < WAVE) rowfill_lists(d, seg, utt_off, A, rv, nodes, assign_nodes, host_counts, seq, u, threadIdx.x,
                                          gather.out != nullptr, gather.parents != 0, s_pslot, &s_row0, &s_rows);
    if (gather.out == nullptr) return;   // (one wave launched)
    __syncthreads();
    const int row0 = s_row0, H4 = d.H >> 2, total = s_rows * H4;
    for (int l = 0; l < (gather.parents ? d.L : 1); ++l) {
        const float *src = gather.pool_h + l * gather.pool_rows * d.H;
        uint2 *dst = static_cast<uint2 *>(gather.out) + l * gather.stride * H4;
        for (int base = threadIdx.x; base < total; base += 256 * 4) {
            float4 v[4];
            int at[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int idx = min(base + k * 256, total - 1);
                const int h = idx / H4, i = idx - h * H4;
                v[k] = reinterpret_cast<const float4 *>(src + (long)s_pslot[h] * d.H)[i];
                at[k] = (row0 + h) * H4 + i;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (base + k * 256 < total)
                    dst[at[k]] = make_uint2(rowfill_bf16(v[k].x) | (rowfill_bf16(v[k].y) << 16),
                                            rowfill_bf16(v[k].z) | (rowfill_bf16(v[k].w) << 16));
        }
    }
}

hipError_t launch_rowfill(hipStream_t st, const Dims &d, int seg, const int *utt_off, AView A, RowView rv,
                          int2 *nodes, int assign_nodes, int *host_counts, int seq, const HidRows *gather) {
    if (gather && ((d.H & 3) || (gather->parents && !A.parents))) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rowfill, dim3(d.U), dim3(gather ? 256 : WAVE), 0, st, d, seg, utt_off, A, rv, nodes,
                       assign_nodes, host_counts, seq, gather ? *gather : HidRows{});
    return hipGetLastError();
}

// ------------------------------------------------------------------ select + merge
// Second half of the inner loop of Algorithm 1, one utterance per workgroup of four
// waves: the first stages the lists and merges the blank expansions while the
// second builds the candidates' keys, all rank both lists, and the first goes on (a chain of
// dependent instructions everywhere: 256 utterances N = 10 S = 3 14.2 us with one
// wave, 12.1 with two of which the second ranked the candidates, 9.5 so; 1024
// utterances S = 5 20.2 with two, 19.1).  The
// utterance's B list, its A entries and its H*N candidates are staged in LDS
// with one round of parallel loads, all list work happens there, and B and the
// new A are written back once, so the kernel costs a handful of memory round
// trips instead of one per list operation.

// SMALL: at most SEL_PRE_FRAMES frames and SEL_PRE_CANDS candidates, whose distributions are made ahead: what the longest segments
// and widest beams need is left out, 13 KB of LDS instead of 41 beside list B (so that more than three workgroups fit a CU: 1024
// utterances N = 10 S = 5 25.6 -> 20.6 us a launch).
#define SEL_WAVES 4
template <bool SMALL>
__global__ void __launch_bounds__(SEL_WAVES * WAVE)
k_select_merge(Dims d, int round, int drop, const float *logits, const float *row_lc,
               const float *dphi, const float *cand_score, const int *cand_tok, AView A, AView An, BView B,
               RowView rv, const int2 *nodes) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];   // B list of this utterance
    TBS_SELECT_ARRAYS(s_select, (SMALL ? SEL_PRE_CANDS : CAND_MAX), (SMALL ? 1 : TBS_MAX_SEG * TBS_MAX_BEAM), SEL_PRE_FRAMES, SEL_PRE_CANDS);
    const int u = blockIdx.x;
    const int pair0 = rv.utt_pair0[u];
    const SelectFigs fg = select_figs(u, A, B, rv);
    SelectIn in;
    in.cand_score = cand_score + (long)pair0 * d.N;
    in.cand_tok = cand_tok + (long)pair0 * d.N;
    in.dphi = dphi + pair0;
    in.lc = row_lc + fg.urow0;
    in.slot_rows = 0;
    const int lane = (int)threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x) / WAVE;
    auto phase = [&](const int p) {
        select_merge_utt(s_select, p, d, round, drop, u, lane, LogitsPlain{logits}, in, fg, A, An, B, rv, nodes, s_dyn, nullptr, false, SMALL);
    };
    const int H = fg.sp > 0 ? fg.cntA : 0;   // (the same for the whole workgroup)
    if (H > 0) {
        if (wave == 0) phase(1);
        __syncthreads();
        if (wave == 0) phase(6);
        else if (wave == 1) phase(7);
        __syncthreads();
        sel_rank_waves(s_select, reinterpret_cast<const double *>(s_dyn), *s_select.s_nb, H * d.N, d.N, wave, SEL_WAVES, lane);
        __syncthreads();
    }
    if (wave == 0) phase(5);
}

// the rank of entry i, counted by `parts` lanes (tests ask it; holes: NaN marks a place without an entry)
extern "C" int rank_of_entry(const double *v, int n, int parts, int holes, int i) {
    int beaten = 0;
    for (int p = 0, per = (n + parts - 1) / parts; p < parts; ++p)
        beaten += rank_beaten<4>(v, std::min(p * per, n), std::min((p + 1) * per, n), v[i], i);
    return holes ? beaten : rank_placed(v, n, v[i], i, beaten);
}

extern "C" int select_dist_form(int candidates, int frames) { return sel_dist_form(candidates, frames); }

hipError_t launch_select_merge(hipStream_t st, const Dims &d, int round, int drop, const float *logits,
                               const float *row_lc, const float *dphi, const float *cand_score,
                               const int *cand_tok, AView A, AView An, BView B, RowView rv, const int2 *nodes) {
    const size_t shm = (size_t)d.BCAP * (sizeof(double) + sizeof(u64) + 3 * sizeof(int));
    const bool small = sel_dist_form(d.N * d.N, d.S) == SEL_AHEAD;
    // the longest B list the library accepts (2048 entries) needs 56 KB of dynamic LDS on top of
    // the kernel's static arrays: more than the default limit, so the limit is raised once
    static bool attr_set = false;
    if (!attr_set) {
        const int most = 2048 * (int)(sizeof(double) + sizeof(u64) + 3 * sizeof(int));
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_select_merge<false>), hipFuncAttributeMaxDynamicSharedMemorySize, most);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_select_merge<true>), hipFuncAttributeMaxDynamicSharedMemorySize, most);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    if (small)
        hipLaunchKernelGGL(k_select_merge<true>, dim3(d.U), dim3(SEL_WAVES * WAVE), shm, st, d, round, drop, logits, row_lc, dphi,
                           cand_score, cand_tok, A, An, B, rv, nodes);
    else
        hipLaunchKernelGGL(k_select_merge<false>, dim3(d.U), dim3(SEL_WAVES * WAVE), shm, st, d, round, drop, logits, row_lc, dphi,
                           cand_score, cand_tok, A, An, B, rv, nodes);
    return hipGetLastError();
}

// ------------------------------------------------------------------ results
__device__ void write_tokens(const int2 *nodes, int node, int len, int max_len, int *out) {
    // walk from the last token to the first
    int pos = len - 1;
    while (node > 0 && pos >= 0) {
        int2 nd = nodes[node];
        if (pos < max_len) out[pos] = nd.y;
        node = nd.x;
        --pos;
    }
}

// return ChooseNBest(B)   (Algorithm 1, last line)
// One wave per utterance writes every output entry of that utterance exactly once: ranks that
// exist get their score, length and tokens, everything else (ranks beyond the list, positions
// beyond a sequence) the neutral value, so the caller's buffers need no clearing beforehand.
__global__ void __launch_bounds__(WAVE)
k_finalize(Dims d, BView B, const int2 *nodes, int *res_count, int *res_len, double *res_logs,
           int *res_tok, int max_len) {
    __shared__ int s_len[TBS_MAX_BEAM];
    const int u = blockIdx.x, lane = threadIdx.x;
    const int nB = B.count[u];
    const double *bl = B.logs + (long)u * d.BCAP;
    if (lane < d.N) s_len[lane] = 0;
    __syncthreads();
    for (int i = lane; i < nB; i += WAVE) {
        const double si = bl[i];
        const int rank = rank_in_list<1>(bl, nB, i);
        if (rank < d.N) {
            long o = (long)u * d.N + rank;
            int len = B.len[(long)u * d.BCAP + i];
            res_logs[o] = si;
            res_len[o] = len;
            s_len[rank] = len;
            write_tokens(nodes, B.node[(long)u * d.BCAP + i], len, max_len, res_tok + o * max_len);
        }
    }
    __syncthreads();
    const int cnt = nB < d.N ? nB : d.N;
    if (lane < d.N && lane >= cnt) {
        res_logs[(long)u * d.N + lane] = 0.0;
        res_len[(long)u * d.N + lane] = 0;
    }
    for (int idx = lane; idx < d.N * max_len; idx += WAVE) {
        const int r = idx / max_len, p = idx - r * max_len;
        if (p >= s_len[r]) res_tok[((long)u * d.N + r) * max_len + p] = -1;
    }
    if (lane == 0) res_count[u] = cnt;
}

hipError_t launch_finalize(hipStream_t st, const Dims &d, BView B, const int2 *nodes, int *res_count, int *res_len,
                           double *res_logs, int *res_tok, int max_len) {
    hipLaunchKernelGGL(k_finalize, dim3(d.U), dim3(WAVE), 0, st, d, B, nodes, res_count, res_len, res_logs, res_tok,
                       max_len);
    return hipGetLastError();
}

// Every entry of the four outputs is written exactly once (entries past the list and positions
// past a sequence get the neutral value), so the buffers need no clearing beforehand.
__global__ void __launch_bounds__(WAVE)
k_hyps_dump(Dims d, int group, AView A, BView B, const int2 *nodes, int cap, int max_len, int *tok,
            int *len, double *logs, int *count) {
    int u = blockIdx.x, lane = threadIdx.x;
    int n = group == 0 ? A.count[u] : B.count[u];
    int stride = group == 0 ? d.N : d.BCAP;
    if (n > cap) n = cap;
    for (int i = lane; i < cap; i += WAVE) {
        long s = (long)u * stride + i, o = (long)u * cap + i;
        if (i < n) {
            int ln = group == 0 ? A.len[s] : B.len[s];
            int nd = group == 0 ? A.node[s] : B.node[s];
            logs[o] = group == 0 ? A.logs[s] : B.logs[s];
            len[o] = ln;
            write_tokens(nodes, nd, ln, max_len, tok + o * max_len);
        } else {
            logs[o] = 0.0;
            len[o] = 0;
        }
    }
    for (int idx = lane; idx < cap * max_len; idx += WAVE) {
        const int i = idx / max_len, p = idx - i * max_len;
        int ln = 0;
        if (i < n) ln = group == 0 ? A.len[(long)u * stride + i] : B.len[(long)u * stride + i];
        if (p >= ln) tok[((long)u * cap + i) * max_len + p] = -1;
    }
    if (lane == 0) count[u] = n;
}

hipError_t launch_hyps_dump(hipStream_t st, const Dims &d, int group, AView A, BView B, const int2 *nodes, int cap,
                            int max_len, int *tok, int *len, double *logs, int *count) {
    hipLaunchKernelGGL(k_hyps_dump, dim3(d.U), dim3(WAVE), 0, st, d, group, A, B, nodes, cap, max_len, tok, len,
                       logs, count);
    return hipGetLastError();
}

// A_PRED view for tests: gather (scatter=0) or scatter (scatter=1) the projected
// predictor outputs of group A between the state pool and a dense [U,N,Dj] array.
__global__ void k_gather_pred(Dims d, AView A, float *pool_p, float *dense, int scatter) {
    int u = blockIdx.x / d.N, i = blockIdx.x % d.N;
    if (i >= A.count[u]) return;
    long a = (long)u * d.N + i;
    long slot = A.slot[a];
    for (int j = threadIdx.x; j < d.Dj; j += blockDim.x) {
        if (scatter) pool_p[slot * d.Dj + j] = dense[a * d.Dj + j];
        else dense[a * d.Dj + j] = pool_p[slot * d.Dj + j];
    }
}

hipError_t launch_gather_pred(hipStream_t st, const Dims &d, AView A, const float *pool_p, float *out, int scatter) {
    hipLaunchKernelGGL(k_gather_pred, dim3(d.U * d.N), dim3(256), 0, st, d, A, const_cast<float *>(pool_p), out,
                       scatter);
    return hipGetLastError();
}

// ------------------------------------------------------------------ test support
// After a test has written A_COUNT: give every entry of A a state slot of its
// own (arena 0, region 0) and the empty token sequence.
__global__ void k_debug_fill_a(Dims d, AView A) {
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= d.U * d.N) return;
    int u = idx / d.N, i = idx % d.N;
    A.slot[idx] = tbs_slot_id(u, 0, 0, i, d.R, d.N);
    A.pslot[idx] = A.slot[idx];
    A.node[idx] = 0;
    A.pnode[idx] = -1;
    A.token[idx] = -1;
    A.hash[idx] = 0ull;
    A.len[idx] = 0;
}

__global__ void k_set_sp(Dims d, int seg, const int *utt_T, RowView rv) {
    int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= d.U) return;
    int left = utt_T[u] - seg * d.S;
    rv.utt_sp[u] = left < 0 ? 0 : (left > d.S ? d.S : left);
    rv.utt_par[u] = 0;   // the arena k_debug_fill_a puts the hypotheses' states in
}

hipError_t launch_debug_fill_a(hipStream_t st, const Dims &d, AView A) {
    hipLaunchKernelGGL(k_debug_fill_a, dim3((d.U * d.N + 255) / 256), dim3(256), 0, st, d, A);
    return hipGetLastError();
}

hipError_t launch_set_sp(hipStream_t st, const Dims &d, int seg, const int *utt_T, RowView rv) {
    hipLaunchKernelGGL(k_set_sp, dim3((d.U + 255) / 256), dim3(256), 0, st, d, seg, utt_T, rv);
    return hipGetLastError();
}
