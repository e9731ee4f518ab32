// Internal declarations shared by the host code and the kernel files of libtbs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tbs.h"

typedef unsigned long long u64;
typedef uint16_t bf16_t;  // raw bf16 bit pattern

// Group A (hypotheses still emitting in this segment), structure of arrays, [U, N].
struct AView {
    int *count;     // [U]
    int *parents;   // [U] different hypotheses that those of the list were made from (row lists only; null: not wanted)
    double *logs;   // log score
    int *node;      // trie node of the token sequence
    u64 *hash;      // hash of the token sequence
    int *len;       // number of tokens
    int *slot;      // predictor-state slot of this hypothesis
    int *pslot;     // slot of the hypothesis it was made from (source of the recurrent state)
    int *pnode;     // trie node of the hypothesis it was made from
    int *token;     // last token (-1 for hypotheses carried into the segment)
    float *dhat;    // [U, N, S] frame distribution of the last token, normalised, as natural logarithms
};

// Group B (hypotheses that took their blank for this segment), [U, BCAP].
struct BView {
    int *count;
    double *logs;
    int *node;
    u64 *hash;
    int *len;
    int *slot;
};

// Row/pair lists of the current round.
struct RowView {
    int *utt_pair0;  // [U]  first pair of each utterance
    int *utt_row0;   // [U]  first joiner row of each utterance
    int *utt_sp;     // [U]  frames of each utterance in this segment (0 = finished)
    int *utt_par;    // [U]  which of the two state arenas the utterance's current segment writes to; flips each
                     //      time the utterance starts a segment (survivors sit in the other one)
    int *pair_u, *pair_h, *pair_row0, *pair_len;  // [pairs]
    int *pair_slot;  // [pairs] predictor-state slot of the pair's hypothesis
    int *pair_pslot; // [pairs] slot of the hypothesis it was made from (source of the recurrent state)
    int *pair_frame0; // [pairs] row in enc_proj of the pair's first frame of the segment
    int *pair_tok;   // [pairs] last token of the pair's hypothesis (-1 if carried into the segment)
    int *pair_par;   // [pairs] place of the hypothesis it was made from among the parents ...
    int *par_slot;   // [parents] ... every hypothesis that new ones were made from, once: its predictor-state slot
    int *row_enc;    // [rows] frame row in enc_proj
    int *row_slot;   // [rows] predictor-state slot
    int *counts;     // [8]: 0 pairs, 1 rows, 2 trie nodes used, 3 error flags, 4 live utterances,
                     //      5 frames joined (sum of S' over live utterances), 6 number of the launch that
                     //      published the figures (host mirror), 7 the other slot of 2 (they alternate),
                     //      8 and 9 running sums of 4 and 5 over the row lists made since the batch began
                     //      (joiner invocations and frames joined, per utterance summed), 10 parents
};

enum { TBS_CNT_PAIRS = 0, TBS_CNT_ROWS = 1, TBS_CNT_NODES = 2, TBS_CNT_ERR = 3, TBS_CNT_UTTS = 4, TBS_CNT_FRAMES = 5,
       TBS_CNT_SEQ = 6, TBS_CNT_NODE_BASE = 7, TBS_CNT_ACC_CALLS = 8, TBS_CNT_ACC_JOINED = 9, TBS_CNT_PARS = 10, TBS_CNT_SIZE = 11 };
enum { TBS_ERRF_BCAP = 1, TBS_ERRF_NODES = 2 };

// Slot layout of small shapes: hypothesis i of utterance u is pair j = u*N + i whether or not it
// exists, its frames are the joiner rows j*S .. j*S + S' - 1.  Nothing depends on the other utterances'
// counts, so no kernel has to sum them: the kernel that makes a list A also writes the descriptors of
// its pairs, takes trie nodes from the utterance's own range and tells the host its count.
struct FixedView {
    int on;
    int seg;
    const int *utt_off;   // [U] first frame row of each utterance
    int *fig;             // [U, 8] what a round needs to know of an utterance before it can start, side by side so
                          //        that one request brings all of it (indices TBS_FIG_*): S' of the segment, the
                          //        hypotheses in A, the entries of B, the state arena, then the trie nodes the
                          //        utterance has taken from its range, the range's size and its first node (the
                          //        ranges share the trie in proportion to the utterances' lengths)
    int *live_sum;        // [2] hypotheses made by all utterances in launch seq (slot seq & 1): kernels queued
                          //     behind it leave at once when it is zero
    int *host_live;       // pinned [2, U], half seq & 1: (seq << 8) | (trie full << 6) | hypotheses made
    int seq;
    const float *pool_h;  // first LSTM layer's h by state slot, and where the new hypotheses' input rows go:
    void *xh;             // xh[j, :] = h of the parent of pair j, as bf16 or fp32 by `f32`   (null: not wanted)
    int f32;              // fp32 model: xh, amat and enc hold floats, otherwise bf16
    // head of a segment only: where the joiner input rows of the survivors go (null: a kernel of its own
    // makes them), the projected encoder frames and the joiner activation
    void *amat;
    const void *enc;
    int act;
    int parts;            // workgroups per utterance of the kernel that starts a segment (0 = 1)
    int xcd_rows;         // round kernel: not 0 = joiner rows per XCD (workgroup b runs on XCD b % 8 and takes an
                          // utterance whose first row lies in that XCD's range; see PartEp)
};
#define TBS_FIXED_SMAX 5   // longest segment the slot layout serves

enum { TBS_FIG_SP = 0, TBS_FIG_CNT = 1, TBS_FIG_NB = 2, TBS_FIG_PAR = 3, TBS_FIG_USED = 4, TBS_FIG_CAP = 5,
       TBS_FIG_BASE = 6, TBS_FIG_SIZE = 8 };

struct Dims {
    int U, N, S, V, Dj, blank;
    int Vl;     // floats from one row of logits to the next: V rounded up to whole 16-byte pieces; the columns past V
                // hold -inf from tbs_init on, so that a reader may take them for logits of probability 0
    int R;      // rounds capacity
    int BCAP;   // entries of B per utterance
    int E, H, L;
    int max_nodes;
};

__host__ __device__ inline int tbs_slot_id(int u, int parity, int r, int i, int R, int N) {
    return ((u * 2 + parity) * (R + 1) + r) * N + i;
}

// Joiner activation of the bf16 path.  tanh x = 1 - 2 / (exp(2x) + 1) with the hardware exponential
// and reciprocal: the absolute error is a few fp32 units of 1, far below the bf16 rounding the
// result goes through; both kernels that form joiner input rows use it, so they agree bit for bit.
__device__ __forceinline__ float tbs_joiner_act(float x, int act) {
    if (act != 0) return fmaxf(x, 0.f);
    const float t = __expf(2.f * x);
    return 1.f - 2.f * __builtin_amdgcn_rcpf(t + 1.f);
}

// ... and of fp32 models
__device__ __forceinline__ float tbs_joiner_act_f32(float x, int act) { return act == 0 ? tanhf(x) : fmaxf(x, 0.f); }

// LSTM cell update done in the epilogue of the gate GEMM (small problems): the weight rows are
// stored gate-interleaved (row 4j+g = gate g of hidden unit j, gate order i, f, g, o), so a 64-wide
// output tile holds all four gates of 16 units.
struct LstmEp {
    const int *pslot, *slot, *tok;   // per row: parent's state slot, own state slot, last token
    const float *emb_gates;          // [V, 4H] gate-interleaved input half of the gates (+ bias), or null
    const float *c_par;              // cell states of this layer, indexed by slot
    float *c_new, *h_new;            // the same pools, written at the row's own slot
    const float *h_par_next;         // hidden states of the next layer (null for the last layer)
    void *out;                       // bf16 or fp32 by the model: last layer [rows, H] top hidden state, else
                                     // [rows, 2H] next layer's input
    int H;
};

// Joiner input rows made in the epilogue of the predictor projection (small problems): row r of
// the product is the projection of pair r, whose frames pair_frame0[r] .. + pair_len[r] - 1 give
// the joiner rows pair_row0[r] ..: amat[row, :] = act(enc[frame, :] + projection).
struct JoinEp {
    const int *pair_row0, *pair_len, *pair_frame0;
    const void *enc;     // [frames, Dj], bf16 or fp32 by the model
    void *amat;          // [rows, Dj], likewise
    int act;             // 0 tanh, 1 relu
    int fgroups;         // workgroups per tile (0 = 1): each computes the tile and forms the joiner input rows of
                         // the frames t = its number, + fgroups, ...; the first also stores the projection
};

// Segments of one frame (the standard breadth-first search, Eq. 1): the joiner GEMM keeps no logits.
// Its epilogue leaves, per row and per tile of 64 columns, what the expansion of a one-frame segment
// needs of them: part[(row * tiles_n + tile) * PW ..] = maximum, sum of exp(l - maximum), the blank
// logit (-inf if blank is in another tile), a spare, then the NP largest non-blank logits in
// descending order (-inf where there are fewer) and their tokens (as integer bit patterns, -1).
struct PartEp {
    float *part;
    int np;      // NP = beam size
    int blank;
    int pieces;     // 1: the partials of a tile's four 16-column pieces go out as they are (four partials per
                    // tile, in column order), for a reader that has a lane for each; 0: merged into one
    int xcd_rows;   // (also for the joiner GEMM that stores logits) not 0: every XCD computes a range of rows
                    // of its own, all their columns, so that the logits or partials of an utterance lie in
                    // the L2 of the XCD whose workgroup of the round kernel reads them (see FixedView)
};
__host__ __device__ inline int part_width(int np) { return (4 + 2 * np + 3) & ~3; }   // (whole 16-byte pieces)

// Whole segments of a batch as one launch, every XCD decoding utterances of its own (xcd_kernels.hip).
#define XR_XCDS 8
#define XR_WGS 32      // workgroups per XCD, one on each of its CUs
#define XR_POS 64      // most utterances an XCD decodes
#define XR_KMAX 640    // widest joint space and LSTM
#define XR_SEGS 4096   // most segments of a launch
#define XR_PATIENCE_MS 5   // how long a launch's workgroups wait for each other to come
struct XcdCtl {        // device memory, zero when the launch begins
    u64 bar[XR_XCDS * 16];            // an XCD's barriers (a line each)
    unsigned place[XR_XCDS * 32];     // workgroups that came on each XCD
    unsigned told[XR_XCDS * 32];      // what became of it, as `state`
    unsigned arrived, state;          // XCDs that are complete; 1: all are, 2: given up
    unsigned pad[30];
};
enum { XR_DONE = 1, XR_ABSENT = 2, XR_TRIE = 3, XR_ROUNDS = 4, XR_STUCK = 5 };   // how a workgroup ended
#define XR_FULL_TRIE (1 << 20)
struct XcdArgs {
    Dims d;
    int seg0, seg1;         // segments of this launch
    int max_rounds;         // limit on the rounds of a segment (0: none)
    int act, seq;
    int expect;             // XCDs that have to be complete before anything is done
    int first[XR_XCDS + 1]; // the XCDs' parts of `order` [U]: utterances in falling length
    int tile0[XR_XCDS];     // and of amat, in tiles of 16 rows
    const int *order;
    int *utt_T, *utt_off;
    // a push of a stream (pinned, by place in `order`; null: none): frames to decode and the first of them, and rows to append
    // first: source row, destination row, how many, of push_units pieces of 16 bytes each
    const int2 *push_step;
    const int4 *push_rows;
    const uint4 *push_from;
    uint4 *push_to;
    int push_units;
    const void *enc;        // frames; the caller's output and projection weights, and the recurrent gate weights
                            // (rows interleaved, see LstmEp) in the pieces the products read (launch_xcd_frags)
    const void *w_out, *w_gate, *w_proj;
    const float *b_out, *b_proj, *emb_gates;
    AView A[2];
    BView B;
    RowView rv;
    int *fig;
    int2 *nodes;
    float *pool_p, *pool_h, *pool_c;
    void *hb;               // [slots] rows of h as the products read it (xcd_row_bytes)
    long hb_bytes;
    void *amat;             // joiner input rows, in pieces of 16 rows x 32 columns (fp32: 16)
    float *logits;
    float *row_lc, *dphi, *cand_score;   // long segments: what the expansion leaves [U*N, S], [U*N], [U*N, N] ...
    int *cand_tok;                       // ... for the select step
    int all_utts;           // utterances there is room for in A and B
    int4 *desc;             // [2][desc_half >= U*N] state slot (-1: no hypothesis), parent's slot, last token: of even and odd segments
    int desc_half;
    XcdCtl *ctl, *ctl_next;
    int *host;              // pinned [workgroups, 4]: joiner calls, frames joined, nodes taken, (seq << 8) | how it ended
    int *host_rounds;       // pinned [XCDs, XR_SEGS]: rounds of each segment
};
bool xcd_fits(const Dims &d);
hipError_t launch_xcd_decode(hipStream_t st, const XcdArgs &g);
hipError_t launch_xcd_push(hipStream_t st, const XcdArgs &g);          // (a push of a stream: one segment, push_step not null)
hipError_t launch_xcd_decode_long(hipStream_t st, const XcdArgs &g);   // (its segments of more than five frames)
bool xcd_f32_fits(const Dims &d);
int xcd_f32_lds_bytes(const Dims &d);
bool xcd_f32_gates_stay(const Dims &d);
int xcd_lds_bytes(int dtype, const Dims &d);   // LDS a workgroup takes
hipError_t launch_xcd_decode_f32(hipStream_t st, const XcdArgs &g);
long xcd_row_bytes(int dtype, int K);                // bytes of a row of K columns as the products read it
long xcd_frag_bytes(int dtype, int rows, int K);     // and of a weight matrix in pieces
hipError_t launch_xcd_frags(hipStream_t st, int dtype, const void *w, void *frags, int rows, int K);

// ---- launchers (each enqueues on `st` and returns the HIP status) ----
// told: pinned, as a batch's [U, TBS_FIG_SIZE] figures, [U] order, [U] lengths and [U + 1] first frames; they go to the others
hipError_t launch_init_batch(hipStream_t st, const Dims &d, BView B, AView A0, AView A1, RowView rv, int2 *nodes,
                             float *pool_p, float *pool_h, float *pool_c, const float *pred_init,
                             long pool_rows,
                             const int *told, int *fig, int *order, int *utt_T, int *utt_off, int *live_sum);
hipError_t launch_segment_begin(hipStream_t st, const Dims &d, int seg, const int *utt_T, BView B,
                                AView A, RowView rv, float *pool_p, float *pool_h, float *pool_c, long pool_rows,
                                const FixedView *fx = nullptr);
// joiner input rows in the slot layout: every row j*S + t with t < pair_len[j]
// the same by pairs (bf16; the pair count is read from the row lists' counts in device memory, at most `pairs`)
hipError_t launch_joiner_prep_pairs(hipStream_t st, const Dims &d, int act, const bf16_t *enc, const float *pool_p,
                                    RowView rv, bf16_t *amat, int pairs);
hipError_t launch_joiner_prep_fixed(hipStream_t st, const Dims &d, int dtype, int act, const void *enc, const float *pool_p,
                                    RowView rv, void *amat);
// Rows of h that the gate products of new hypotheses read, as bf16 or fp32 (fp32 models): row j the parent's of pair j (parents
// 0, the first layer only), or row p that of parent p, for every layer (out: [layers, stride, H]).
struct HidRows {
    const float *pool_h;
    void *out;
    long pool_rows, stride;
    int parents;
};
// gather not null (bf16, H a multiple of 4): also writes those rows
hipError_t launch_rowfill(hipStream_t st, const Dims &d, int seg, const int *utt_off, AView A, RowView rv,
                          int2 *nodes, int assign_nodes, int *host_counts, int seq, const HidRows *gather = nullptr);
// row_begin (bf16 only, with rows_dev): only the rows [*row_begin, *rows_dev), `rows` sizing the launch
hipError_t launch_joiner_prep(hipStream_t st, const Dims &d, int dtype, int act, int rows, const void *enc,
                              const float *pool_p, RowView rv, void *amat, const int *rows_dev = nullptr,
                              const int *row_begin = nullptr);
// m_dev, xcd_rows as for launch_gemm_bf16 below
hipError_t launch_gemm_f32(hipStream_t st, const float *A, const float *B, const float *bias, float *C, int M, int N,
                           int K, const int *out_row, long ldc, const int *m_dev = nullptr, bool xcd_rows = false);
// the fp32 forms of the fused GEMMs below (operands of which every row starts at a 16-byte boundary)
bool gemm_f32_fits(const void *A, const void *B, int M, int N, int K, int max_tiles);
hipError_t launch_gemm_lstm_f32(hipStream_t st, const float *A, const float *Wp, const float *biasp, int M, int K,
                                const LstmEp &ep, const int *m_dev, const int *any_dev);
hipError_t launch_gemm_join_f32(hipStream_t st, const float *A, const float *B, const float *bias, float *C, int M, int N,
                                int K, const int *out_row, long ldc, const JoinEp &jp, const int *m_dev,
                                const int *any_dev);
#define GF_TILE 32            // fp32: edge of a tile
#define GF_TILES 1024         // fp32: tiles of 32 x 32 up to which the fused forms serve the row lists: ms per decode fused /
                              // separate by the most tiles of a round's products, Librispeech-like widths N = 5 S = 3
                              // 256: 6.4 / 6.9, 736: 7.9 / 8.1, 1024: 8.6 / 9.0, 1152: 9.0 / 9.3, 1440: 10.0 / 10.1, 1920:
                              // 11.7 / 11.6, 4512: 20.8 / 19.9; large widths N = 8 1024: 10.6 / 10.8, 1536: 11.9 / 12.3,
                              // 3072: 17.6 / 16.9; widths of 256 2400: 11.5 / 11.9, 4000: 16.6 / 16.6.  Fused is no slower
                              // anywhere up to here; the two cross between 1440 and 4000, by the widths.
#define GF_TILES_FIXED 1280   // ... and the slot layout: measured at N = 5 on the Librispeech-like widths (most tiles of
                              // a round's products: ms per decode with slots / row lists) 640: 12.5 / 16.0, 800: 10.6 /
                              // 11.4, 960: 12.5 / 13.5, 1200: 20.8 / 22.1, 1440: 15.4 / 15.2, 1600: 13.9 / 13.4 and
                              // 25.5 / 24.5, 1920: 18.8 / 17.3
// m_dev: the launch is enqueued before the host knows the row count; M is an upper bound and the count is read from *m_dev
// m_likely: rows to choose the kernel for, 0: M.  (Products without a bias have the same bits whichever it is.  The bias is added last by
// k_gemm_small, in products that k_gemm_tile serves up to 768 tiles of 256 x 256, and with bias_late; otherwise it comes first.)
hipError_t launch_gemm_bf16(hipStream_t st, const bf16_t *A, const bf16_t *B, const float *bias, float *C, int M,
                            int N, int K, const int *out_row, long ldc, int kernel = 0, const int *m_dev = nullptr,
                            bool xcd_rows = false, bool bias_late = false, int m_likely = 0);
// further products of a launch: the i-th takes A + (i + 1) a and B[i] to C + i c
struct GemmBatch {
    int n;
    const bf16_t *B[TBS_MAX_LAYERS - 1];
    float *C;
    long a, c;
};
hipError_t launch_gemm_bf16_batch(hipStream_t st, const bf16_t *A, const bf16_t *B, float *C, int M, int N, int K, long ldc, const int *m_dev,
                                  int m_likely, const GemmBatch &more);
// rows per XCD when k_gemm_small gives every XCD a row range of its own (PartEp::xcd_rows)
inline int gemm_small_xcd_rows(int M, int tile) { return tile * ((((M + tile - 1) / tile) + 7) / 8); }
hipError_t launch_gemm_bf16_rows(hipStream_t st, const bf16_t *A, const bf16_t *B, const float *bias, float *C,
                                 int m_max, int N, int K, long ldc, const int *m_begin, const int *m_end);
#define GS_TILES 320          // tiles of 64 x 64 up to which the row lists take the small-problem GEMM kernel's fused forms
#define GS_TILES_FIXED 1024   // the same for the slot layout (measured on the Librispeech-like shape: 96 to 256
                              // utterances decode 5-16 % faster in it than with row lists, 320 the same)
bool gemm_small_fits(int M, int N, int K, int max_tiles = GS_TILES);
// true if launch_gemm_lstm can run this problem (small, K a multiple of 128 that fits the LDS stages)
bool gemm_lstm_fits(int M, int H, int K, int max_tiles = GS_TILES);
// any_dev (both fused forms): rows may be dead (state slot < 0) anywhere, and if *any_dev is zero
// the whole launch leaves at once
hipError_t launch_gemm_lstm(hipStream_t st, const bf16_t *A, const bf16_t *Wp, const float *biasp, int M, int K,
                            const LstmEp &ep, const int *m_dev = nullptr, const int *any_dev = nullptr);
// the same for the projection GEMM that also makes the next joiner call's input rows (bf16 models)
bool gemm_join_fits(int M, int N, int K, int max_tiles = GS_TILES);
hipError_t launch_gemm_join(hipStream_t st, const bf16_t *A, const bf16_t *B, const float *bias, float *C, int M,
                            int N, int K, const int *out_row, long ldc, const JoinEp &jp, const int *m_dev = nullptr,
                            const int *any_dev = nullptr);
// joiner GEMM of one-frame segments: row partials instead of logits (see PartEp)
bool gemm_part_fits(int M, int N, int K, int np, int max_tiles = GS_TILES);
hipError_t launch_gemm_part(hipStream_t st, const bf16_t *A, const bf16_t *B, const float *bias, int M, int N, int K,
                            const PartEp &pe);
hipError_t launch_permute_gate_rows(hipStream_t st, const void *src, void *dst, int H, long row_bytes);
// which kernel expands segments of S frames of logit rows of Vl floats
#define EXPAND_TWO_PASS 0
#define EXPAND_REG(NV4, SMAX) (100 * (NV4) + (SMAX))
#define EXPAND_LONG(NQ, RPW) (1000 + 10 * (NQ) + (RPW))
extern "C" int expand_form(int Vl, int S);
hipError_t launch_expand(hipStream_t st, const Dims &d, int pairs, const float *logits, AView A, RowView rv,
                         float *row_lc, float *dphi, float *cand_score, int *cand_tok, float *row_stats,
                         float *delta_nb, int force_generic, const int *pairs_dev = nullptr, int pair_base = 0,
                         bool fold = false);
// how the select step makes the frame distributions of new hypotheses: 0 ahead of the ranking, 1 by lane, 2 by frame
extern "C" int select_dist_form(int candidates, int frames);
hipError_t launch_select_merge(hipStream_t st, const Dims &d, int round, int drop, const float *logits,
                               const float *row_lc, const float *dphi, const float *cand_score,
                               const int *cand_tok, AView A, AView An, BView B, RowView rv, const int2 *nodes);
// expansion and select/merge of a round in one kernel, a workgroup per utterance (small shapes:
// round_fits says whether the shape is served)
bool round_fits(const Dims &d);
hipError_t launch_round(hipStream_t st, const Dims &d, int round, int drop, const float *logits, AView A, AView An,
                        BView B, RowView rv, int2 *nodes, float *row_stats, float *delta_nb,
                        const FixedView *fx = nullptr);
// the same for one-frame segments in the slot layout, from the joiner GEMM's row partials
bool round_s1_fits(const Dims &d);
// (tiles_n: partials per row, in column order: the vocabulary's 64-column tiles, or their 16-column pieces)
hipError_t launch_round_s1(hipStream_t st, const Dims &d, int round, int drop, const float *part, int tiles_n, AView A,
                           AView An, BView B, RowView rv, int2 *nodes, const FixedView *fx);
// rows: the most there can be
hipError_t launch_pred_gather_h(hipStream_t st, const Dims &d, int dtype, int rows, RowView rv, const HidRows &g);
// Cell update of one layer: the gates of pair j are ga[ga_row[j]] + gb[gb_row[j]] (row j where a list of rows is null, the first
// alone where gb is).  out [pairs, H], or with h_par_next [pairs, 2H] = the next layer's input and its parent's h.
struct CellIn {
    const float *ga, *gb;
    const int *ga_row, *gb_row;
    const float *h_par_next;   // h of the next layer, by state slot
    void *out;
};
hipError_t launch_lstm_pointwise(hipStream_t st, const Dims &d, int dtype, int pairs, int layer, RowView rv, const CellIn &in,
                                 float *pool_h, float *pool_c, long pool_rows);
hipError_t launch_finalize(hipStream_t st, const Dims &d, BView B, const int2 *nodes, int *res_count, int *res_len,
                           double *res_logs, int *res_tok, int max_len);
hipError_t launch_hyps_dump(hipStream_t st, const Dims &d, int group, AView A, BView B, const int2 *nodes, int cap,
                            int max_len, int *tok, int *len, double *logs, int *count);
hipError_t launch_gather_pred(hipStream_t st, const Dims &d, AView A, const float *pool_p, float *out, int scatter);
hipError_t launch_concat_weights(hipStream_t st, int elem_bytes, const void *w_ih, const void *w_hh, void *wcat,
                                 int rows, int in_dim, int hid);
hipError_t launch_debug_fill_a(hipStream_t st, const Dims &d, AView A);
// rows of row_bytes bytes: for every utterance u, n[u] rows from src row src_row[u] on to dst row
// dst_row[u] on (desc = [src_row | dst_row | n], each [U]); the ranges of src and dst must not overlap
hipError_t launch_stream_copy(hipStream_t st, int U, const void *src, void *dst, const int *desc, long row_bytes);
hipError_t launch_logit_pads(hipStream_t st, float *logits, long rows, int V, int Vl);   // -inf into the columns past V
hipError_t launch_empty(hipStream_t st);   // a kernel that does nothing (timing yardstick)
hipError_t launch_set_sp(hipStream_t st, const Dims &d, int seg, const int *utt_T, RowView rv);
