"""GPU parity: the HIP path through the C ABI against the CPU oracle, element
by element, on the same seeded inputs.

Tolerances.  Expansion scores: relative 1e-3 on scores
relative to the hypothesis score, i.e. |log gpu - log oracle| <= 1e-3, for
entries above 1e-30.  For bf16 models the oracle rounds act(e+p) and the
recurrent inputs to bf16 at the same points as the kernels; what remains is
fp32 accumulation order and exp/log/tanh rounding (~1e-6), plus rare bf16
rounding flips.  fp32 models: the same checks at 1e-4.  Integer results
(tokens, candidate sets, list sizes) must match exactly wherever the oracle's
own decision margin exceeds the tolerance.
"""

import math

import numpy as np
import pytest

import oracle
from tbs_inputs import SHAPES, TbsShape, make_model, make_utterances
from helpers import (build_case, oracle_weights, make_tbs, compare_nbest, small_bf16_shape, tolerance,
                     strict_prefixes, assert_all_agree, nbest_agrees)

pytestmark = pytest.mark.gpu


def _bf16_values(rng, shape, scale=1.0):
    import torch
    x = (rng.standard_normal(shape) * scale).astype(np.float32)
    return torch.from_numpy(x).to(torch.bfloat16)


# ------------------------------------------------------------------ the MFMA GEMM on its own

@pytest.mark.parametrize("kernel", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (200, 192, 128), (37, 100, 72), (1000, 1024, 512), (300, 2560, 640),
                                   (4100, 4096, 1024), (513, 257, 256)])
def test_gemm_bf16_tiles(M, N, K, kernel):
    """Every GEMM kernel (0 = the one the decode would pick; 64x64, 128x128, 256x256 tiles of the
    persistent kernel; the multi-stage kernel for small problems) on shapes with ragged edges."""
    import torch
    from paper_2302_14357_amd import gemm_bf16
    if kernel == 4 and K % 128:
        pytest.skip("the multi-stage kernel takes K in multiples of 128")
    rng = np.random.default_rng(M + N + K)
    a, b = _bf16_values(rng, (M, K)), _bf16_values(rng, (N, K), 0.1)
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32))
    got = gemm_bf16(a.cuda(), b.cuda(), bias.cuda(), kernel=kernel).cpu().numpy()
    want = a.to(torch.float64).numpy() @ b.to(torch.float64).numpy().T + bias.numpy().astype(np.float64)
    np.testing.assert_allclose(got, want, rtol=1e-4, atol=1e-4 * math.sqrt(K))


@pytest.mark.parametrize("tm,tn,ns", [(8, 4, 2), (7, 4, 2), (6, 4, 2), (5, 4, 2), (4, 4, 2), (3, 4, 2), (4, 2, 2), (3, 2, 2), (2, 2, 2),
                                      (1, 2, 2), (4, 2, 4), (3, 2, 4), (2, 2, 4), (1, 2, 4)])
def test_gemm_bf16_tile_shapes(tm, tn, ns):
    """Every tile shape of the kernel for products of a few tiles a CU: one row and a few columns past whole tiles, one short of
    them, a single row, several tiles on every XCD, as few K tiles as it has stages, one more, and many; rows scattered, fewer rows than
    the launch is sized for, and nothing written beside the result.  Against fp64 as above, and bit for bit against the kernel for
    small problems, whose sums it keeps."""
    import ctypes
    import torch
    from paper_2302_14357_amd import gemm_bf16, load_library
    run = load_library().gemm_tile_run
    run.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 4 + [ctypes.c_int] * 3 + [ctypes.c_void_p, ctypes.c_long] + [ctypes.c_void_p] * 2
    bm, bn = 32 * tm, 64 * tn
    rng = np.random.default_rng(100 * tm + 10 * tn + ns)
    for M, N, K, live in [(1, 3, 64 * ns, 1), (bm, bn, 64 * (ns + 1), bm), (bm + 1, bn + 5, 64 * ns + 64, bm + 1),
                          (5 * bm - 1, 9 * bn - 2, 640, 5 * bm - 1), (3 * bm + 7, 2 * bn, 256, bm + 2), (2 * bm, bn, 256, 0)]:
        a, b = _bf16_values(rng, (M, K)), _bf16_values(rng, (N, K), 0.1)
        bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32))
        ldc = (N + 3) // 4 * 4 + 4
        where = torch.from_numpy(rng.permutation(M + 3)[:M].astype(np.int32)) if M % 2 == 0 else None
        out = torch.full((M + 3, ldc), 7.0, device="cuda")
        da, db, dbias, n = a.cuda(), b.cuda(), bias.cuda(), torch.tensor([live], dtype=torch.int32, device="cuda")
        dwhere = where.cuda() if where is not None else None
        rc = run(100 * tm + 10 * tn + ns, da.data_ptr(), db.data_ptr(), dbias.data_ptr(), out.data_ptr(), M, N, K,
                 dwhere.data_ptr() if where is not None else None, ldc, n.data_ptr() if live < M else None, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        rows = (where if where is not None else torch.arange(M))[:live].long()
        want = torch.full((M + 3, ldc), 7.0)
        want[rows, :N] = (a[:live].double() @ b.double().T + bias.double()).float()
        np.testing.assert_allclose(out.cpu().numpy(), want.numpy(), rtol=1e-4, atol=1e-4 * math.sqrt(K))
        untouched = torch.ones(M + 3, ldc, dtype=torch.bool)
        untouched[rows, :N] = False
        assert (out.cpu()[untouched] == 7.0).all()
        if K % 128 == 0 and live > 0:
            assert torch.equal(out[rows.cuda(), :N], gemm_bf16(da, db, dbias, kernel=4)[:live]), (M, N, K)


# ------------------------------------------------------------------ joiner + expansion on chosen inputs

def _teacher_forced_state(rng, U, N, S, Dj):
    counts = rng.integers(0, N + 1, size=U).astype(np.int32)
    counts[0] = N
    if U > 1:
        counts[1] = 1
    pred = (rng.standard_normal((U, N, Dj)) * 0.5).astype(np.float32)
    dhat = rng.random((U, N, S)).astype(np.float32)
    dhat[rng.random((U, N, S)) < 0.35] = 0.0
    dhat[:, :, 0] += 0.05
    logs = -rng.random((U, N)) * 50.0
    return counts, pred, dhat, logs


_EXPAND_DEBUG = {"auto": 1, "generic": 3}   # tbs_config.debug: statistics kept + kernel choice


def _check_joiner_expand(shape, U, N, S, seg, sample_pairs=None, tol=1e-3, kernel="auto", flat=False, **kw):
    model, offsets, enc = build_case(shape, n_utts=U)
    if flat:   # every logit equal: every expansion ties, the smallest tokens must win
        model["w_out"] = np.zeros_like(model["w_out"])
        model["b_out"] = np.zeros_like(model["b_out"])
    W = oracle_weights(shape, model)
    tbs = make_tbs(shape, model, offsets, N, S, debug=_EXPAND_DEBUG[kernel], **kw)
    enc_dev = tbs.upload_frames(enc)
    rng = np.random.default_rng(11)
    counts, pred, dhat, logs = _teacher_forced_state(rng, U, N, S, shape.d_joint)
    tbs.begin(enc_dev, offsets)
    from paper_2302_14357_amd import BUF
    tbs.debug_write(BUF.A_COUNT, counts)
    tbs.debug_write(BUF.A_LOGS, logs)
    tbs.debug_write(BUF.A_PRED, pred)
    tbs.debug_write(BUF.A_DHAT, dhat)
    rows = tbs.debug_rebuild(seg)
    lens = np.diff(offsets)
    sp = np.clip(lens - seg * S, 0, S)
    assert rows == int(np.sum(np.where(sp > 0, counts, 0) * sp))
    np.testing.assert_array_equal(tbs.debug_read(BUF.A_PRED)[0, :N], pred[0, :N])
    tbs.joiner_segment()
    tbs.expand()
    pu, ph = tbs.debug_read(BUF.PAIR_UTT), tbs.debug_read(BUF.PAIR_HYP)
    row0, plen = tbs.debug_read(BUF.PAIR_ROW0), tbs.debug_read(BUF.PAIR_LEN)
    logits = tbs.debug_read(BUF.LOGITS)
    stats = tbs.debug_read(BUF.ROW_STATS)
    dphi = tbs.debug_read(BUF.DELTA_BLANK)
    dnb = tbs.debug_read(BUF.DELTA_NB)
    cs, ct = tbs.debug_read(BUF.CAND_SCORE), tbs.debug_read(BUF.CAND_TOKEN)
    pairs = len(pu)
    # pair list: utterances in order, hypotheses in order, finished utterances absent
    want_pairs = [(u, h) for u in range(U) if sp[u] > 0 for h in range(counts[u])]
    assert list(zip(pu.tolist(), ph.tolist())) == want_pairs
    which = range(pairs) if sample_pairs is None else rng.choice(pairs, size=min(sample_pairs, pairs), replace=False)
    worst = 0.0
    for j in which:
        u, h, r0, L = int(pu[j]), int(ph[j]), int(row0[j]), int(plen[j])
        assert L == sp[u]
        ref_logits = np.stack([W.joiner_vec(enc[offsets[u] + seg * S + t], pred[u, h]) for t in range(L)])
        np.testing.assert_allclose(logits[r0:r0 + L], ref_logits, rtol=0, atol=tol)
        d_old = dhat[u, h, :L].astype(np.float64)
        J, Bl, d, ref_nb, ref_phi = oracle.expansion_scores(ref_logits[None], d_old[None], shape.blank_id)
        np.testing.assert_allclose(stats[r0:r0 + L, 2], J[0, :, shape.blank_id], rtol=tol)
        assert abs(dphi[j] - math.log(ref_phi[0])) <= tol   # the kernel hands on log delta_blank
        ref_nb = ref_nb[0]
        big = ref_nb > 1e-30
        err = np.abs(np.log(dnb[j][big]) - np.log(ref_nb[big]))
        worst = max(worst, float(err.max()))
        assert err.max() <= tol
        assert dnb[j][shape.blank_id] == 0.0
        # the N best expansions of this hypothesis: same set wherever the margin is clear
        order = np.argsort(-ref_nb, kind="stable")
        n_take = min(N, shape.vocab - 1)
        margin = math.log(ref_nb[order[n_take - 1]]) - math.log(ref_nb[order[n_take]]) if n_take < shape.vocab - 1 else 1.0
        if margin > 2 * tol:
            assert set(ct[j][:n_take].tolist()) == set(order[:n_take].tolist())
        if flat:
            assert ct[j][:n_take].tolist() == list(range(1, n_take + 1))
        got_sorted = cs[j][:n_take]
        assert np.all(np.diff(got_sorted) <= 0)
        np.testing.assert_allclose(got_sorted, np.log(ref_nb[ct[j][:n_take]]), rtol=0, atol=tol)
    tbs.close()
    return worst


def test_joiner_expand_tiny_fp32():
    _check_joiner_expand(SHAPES["tiny"], U=1, N=2, S=3, seg=2, tol=1e-4)
    _check_joiner_expand(SHAPES["tiny"], U=1, N=2, S=3, seg=16, tol=1e-4)  # ragged last segment (2 frames)


@pytest.mark.parametrize("d,V,U,N,S", [(4, 20, 1, 2, 1), (128, 64, 3, 4, 3), (132, 33, 2, 3, 2), (640, 70, 4, 5, 3), (772, 1028, 13, 5, 5),
                                       (6, 31, 2, 3, 3), (1030, 129, 3, 4, 2)])
def test_fp32_dense_layers_widths(d, V, U, N, S):
    """The fp32 GEMM at the edges of its K tiles (one chunk, one tile, a tile and a chunk, as many tiles as
    stages, more; widths that are no whole 16-byte chunks take the other kernel) and of its 32x32 tiles."""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=U, vocab=V, d=d, hidden=d), dtype="f32")
    _check_joiner_expand(shape, U=U, N=N, S=S, seg=0, tol=1e-4, sample_pairs=8)
    model, offsets, enc = build_case(shape, n_utts=U, lengths=np.minimum(np.arange(U) + 4, 9))
    _check_decode(shape, model, offsets, enc, N, S)


@pytest.mark.parametrize("kernel", ["auto", "generic"])
@pytest.mark.parametrize("N,S", [(5, 3), (2, 1), (10, 5), (3, 50), (4, 12), (32, 2)])
def test_joiner_expand_small_bf16(N, S, kernel):
    """Both expansion kernels (the one that holds a hypothesis' logits in registers, which gives
    way to the other where S is beyond its range, and the two-pass kernel for any shape)."""
    shape = small_bf16_shape(n_utts=5, vocab=200, d=128, hidden=64)
    _check_joiner_expand(shape, U=5, N=N, S=S, seg=1 if S < 20 else 0, kernel=kernel)


@pytest.mark.parametrize("V,N,S", [(2048, 8, 7), (1028, 3, 2), (4096, 10, 5), (3000, 4, 3), (2000, 6, 5), (4096, 20, 3),
                                   (1024, 16, 4), (4096, 32, 2), (16000, 3, 2), (5001, 4, 3)])
def test_joiner_expand_wide_vocab(V, N, S):
    """Vocabulary widths that exercise every register-kernel instantiation and a ragged last column block."""
    shape = small_bf16_shape(n_utts=4, vocab=V, d=64, hidden=64)
    _check_joiner_expand(shape, U=4, N=N, S=S, seg=1, sample_pairs=6)


@pytest.mark.parametrize("kernel", ["auto", "generic"])
def test_expand_all_scores_equal(kernel):
    """Degenerate input: every expansion of a hypothesis has the same score (exercises the
    tie order and the selection path taken when too many candidates reach the threshold)."""
    shape = small_bf16_shape(n_utts=3, vocab=1024, d=64, hidden=64)
    _check_joiner_expand(shape, U=3, N=6, S=3, seg=0, kernel=kernel, flat=True)


@pytest.mark.parametrize("V,N,S", [(3, 2, 2), (257, 5, 3), (1023, 16, 5), (1021, 3, 1), (2049, 4, 3), (3001, 10, 5)])
def test_vocabularies_that_are_no_whole_pieces(V, N, S):
    """Logit rows padded to 16-byte pieces: vocabularies one, two and three columns short of a piece or just
    past one, in the kernels that hold the logits in registers (the round kernel among them), against the
    oracle; the padding must neither enter a softmax nor become a token."""
    shape = small_bf16_shape(n_utts=4, vocab=V, d=128, hidden=128)
    _check_joiner_expand(shape, U=4, N=N, S=S, seg=0, sample_pairs=6)
    model, offsets, enc = build_case(shape, n_utts=4, lengths=np.array([7, 1, 9, 4]))
    _, st = _gpu_decode(shape, model, offsets, enc, N, S)
    assert st["path"]["fixed_places"] == (V <= 1024)
    _check_decode(shape, model, offsets, enc, N, S)


@pytest.mark.parametrize("V,S,scale", [(1021, 5, 8), (64, 5, 8), (2049, 3, 8), (1024, 8, 8), (1024, 17, 8), (1023, 50, 4), (200, 64, 4)])
def test_blank_expansion_error_of_peaked_models(V, S, scale):
    """log delta_blank (Eq. 7) against fp64 on the kernel's own logits, for peaked distributions with large logits: the
    rounding of a row's maximum must not enter the blank probabilities, whose errors add up over the segment.  Bound on
    the rms over hypotheses: a frame's log blank probability has three roundings (the blank's exponential, the row
    sum, its logarithm) of values about one, at most 2^-23 each and evenly spread, so 3^0.5 2^-23 / 3^0.5 = 2^-23 rms;
    S of them are independent; the result is rounded once more to its own last place."""
    import dataclasses
    from paper_2302_14357_amd import BUF
    U, N, Dj = 16, 5, 128
    shape = dataclasses.replace(small_bf16_shape(n_utts=U, vocab=V, d=Dj, hidden=64), len_lo=S, len_hi=S, logit_scale=float(scale),
                                blank_bias=3.0 * scale)
    model, offsets, enc = build_case(shape, n_utts=U)
    tbs = make_tbs(shape, model, offsets, N, S, debug=1, rounds_capacity=4 * S)
    rng = np.random.default_rng(4)
    pred = (rng.standard_normal((U, N, Dj)) * 0.5).astype(np.float32)
    dhat = rng.random((U, N, S)).astype(np.float32)
    dhat[rng.random((U, N, S)) < 0.3] = 0.0
    dhat[:, :, 0] += 0.05
    tbs.begin(tbs.upload_frames(enc), offsets)
    tbs.debug_write(BUF.A_COUNT, np.full(U, N, np.int32))
    tbs.debug_write(BUF.A_LOGS, -rng.random((U, N)))
    tbs.debug_write(BUF.A_PRED, pred)
    tbs.debug_write(BUF.A_DHAT, dhat)
    tbs.debug_rebuild(0)
    tbs.joiner_segment()
    tbs.expand()
    logits, dphi = tbs.debug_read(BUF.LOGITS).astype(np.float64), tbs.debug_read(BUF.DELTA_BLANK)
    pu, ph, row0 = tbs.debug_read(BUF.PAIR_UTT), tbs.debug_read(BUF.PAIR_HYP), tbs.debug_read(BUF.PAIR_ROW0)
    tbs.close()
    want = np.array([math.log(oracle.expansion_scores(logits[r:r + S][None], dhat[u, h].astype(np.float64)[None], shape.blank_id)[4][0])
                     for u, h, r in zip(pu, ph, row0)])
    err = math.sqrt(np.mean((dphi - want) ** 2))
    bound = math.sqrt(S) * 2.0 ** -23 + 2.0 ** -24 * math.sqrt(np.mean(want ** 2))
    print(f"V={V} S={S} scale={scale}: rms error {err:.2e}, bound {bound:.2e}")
    assert err <= bound


def test_joiner_expand_odd_vocab():
    shape = small_bf16_shape(n_utts=3, vocab=77, d=64, hidden=64)
    _check_joiner_expand(shape, U=3, N=4, S=3, seg=0)


def test_joiner_expand_librispeech_full_size_sampled():
    """Headline configuration at full size (64 utterances, V=1024, Dj=512,
    N=5, S=3): sampled hypotheses against the oracle."""
    _check_joiner_expand(SHAPES["librispeech"], U=64, N=5, S=3, seg=10, sample_pairs=12)


def test_joiner_expand_assistant_full_width_sampled():
    """Large-assistant widths (V=4096, Dj=1024, N=10, S=3) with a multi-tile row count."""
    _check_joiner_expand(SHAPES["assistant"].with_utts(48), U=48, N=10, S=3, seg=5, sample_pairs=6)
    _check_joiner_expand(SHAPES["assistant"].with_utts(48), U=48, N=10, S=3, seg=5, sample_pairs=4, kernel="generic")


@pytest.mark.parametrize("kernel", ["auto", "generic"])
@pytest.mark.parametrize("N,S,chunk", [(5, 3, 16), (10, 5, 37), (3, 50, 60), (4, 12, 1), (6, 2, 7)])
def test_joiner_expand_in_pieces(N, S, chunk, kernel):
    """A joiner call run in pieces (input rows, GEMM and expansion of some hypotheses, then of the
    next): piece sizes that are no multiple of the segment size, ragged last segments, a piece of a
    single hypothesis, finished utterances in the batch."""
    shape = small_bf16_shape(n_utts=5, vocab=200, d=128, hidden=64)
    _check_joiner_expand(shape, U=5, N=N, S=S, seg=1 if S < 20 else 0, kernel=kernel, joiner_chunk_rows=chunk)


def test_joiner_expand_throughput_shape_in_pieces():
    """The largest configuration's widths with ~8000 rows in two pieces of 6144 rows at most: each
    piece runs on the 256x256-tile persistent GEMM over a row range read from device memory."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["throughput"], n_utts=320, len_lo=25, len_hi=25)
    _check_joiner_expand(shape, U=320, N=10, S=5, seg=3, sample_pairs=10, joiner_chunk_rows=6144)


def test_joiner_expand_throughput_shape_sampled():
    """The largest configuration's widths (Dj=1024, V=4096, N=10, S=5) with enough rows (320
    utterances, ~8000 rows) that the joiner runs on the 256x256-tile persistent GEMM and the
    expansion on the 80-logits-per-thread kernel: the two kernels the at-scale roofline figures
    are measured on, sampled hypotheses against the oracle."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["throughput"], n_utts=320, len_lo=25, len_hi=25)
    _check_joiner_expand(shape, U=320, N=10, S=5, seg=3, sample_pairs=8)


# ------------------------------------------------------------------ whole decode

def _oracle_decode(shape, model, offsets, enc, N, S, threads=16, **kw):
    W = oracle_weights(shape, model)
    kw.setdefault("trace", True)   # the per-round decision gaps decide how strictly results are compared
    res, _ = oracle.decode_lstm_batch(W, enc, offsets, N, S, threads=min(threads, oracle.max_threads()), **kw)
    return res


def _gpu_decode(shape, model, offsets, enc, N, S, **kw):
    tbs = make_tbs(shape, model, offsets, N, S, **kw)
    out = tbs.decode(tbs.upload_frames(enc), offsets)
    st = tbs.stats()
    st["path"] = tbs.path()
    tbs.close()
    return out, st


def _check_decode(shape, model, offsets, enc, N, S, max_rounds=0, report=None, **kw):
    """tbs_decode against the oracle under the gap rule, in two steps.  (1) The whole batch:
    utterances all of whose decisions were clear must agree.  (2) Every utterance cut back to the
    whole segments before its first close decision, decoded again by both sides: now every
    decision is clear, so every utterance must agree and the joiner-call counters must be equal.
    Returns a dict of what was seen (for assertions on coverage, e.g. hypothesis lengths)."""
    tol, score_tol = tolerance(shape, model)
    okw = dict(max_rounds=max_rounds) if max_rounds else {}
    gkw = dict(kw)
    if max_rounds:
        gkw["max_rounds_per_segment"] = max_rounds
    ref = _oracle_decode(shape, model, offsets, enc, N, S, **okw)
    U = len(offsets) - 1
    tbs = make_tbs(shape, model, offsets, N, S, **gkw)
    got = tbs.decode(tbs.upload_frames(enc), offsets)
    st = tbs.stats()
    same, amb, tot = compare_nbest(got, ref, score_tol=score_tol, gap_tol=tol)
    clear = [u for u in range(U) if ref[u].first_ambiguous_segment(tol) is None]
    info = {"same": same, "amb": amb, "tot": tot, "clear": len(clear),
            "max_len_checked": max([len(y) for u in clear for y, _ in ref[u].nbest], default=0)}
    if len(clear) == U:
        assert same == tot
        assert st["joiner_calls"] == sum(r.joiner_calls for r in ref)
        assert st["joined_frames"] == sum(r.joined_frames for r in ref)
    else:
        off2, enc2, keep = strict_prefixes(ref, offsets, enc, S, tol)
        ref2 = _oracle_decode(shape, model, off2, enc2, N, S, **okw)
        got2 = tbs.decode(tbs.upload_frames(enc2), off2)
        st2 = tbs.stats()
        assert_all_agree(got2, ref2, score_tol, tol)
        assert st2["joiner_calls"] == sum(r.joiner_calls for r in ref2)
        assert st2["joined_frames"] == sum(r.joined_frames for r in ref2)
        info["prefix_frames"] = int(keep.sum())
        info["max_len_checked"] = max(info["max_len_checked"],
                                      max([len(y) for r in ref2 for y, _ in r.nbest], default=0))
    tbs.close()
    if report:
        print(f"{report}: identical {same}/{tot}, differing after a close decision {amb}, "
              f"utterances with every decision clear {len(clear)}, "
              f"frames checked strictly {info.get('prefix_frames', int(offsets[-1]))}/{int(offsets[-1])}, "
              f"longest hypothesis checked {info['max_len_checked']}")
    return info


def test_decode_tiny_reference_config():
    shape = SHAPES["tiny"]
    model, offsets, enc = build_case(shape)
    info = _check_decode(shape, model, offsets, enc, 2, 3, report="tiny")
    assert info["tot"] == 1


@pytest.mark.parametrize("N,S", [(1, 1), (2, 2), (5, 3), (3, 7), (4, 30)])
def test_decode_small_bf16_and_edges(N, S):
    """Ragged batch with an empty utterance, one shorter than a segment and
    lengths that leave ragged last segments."""
    shape = small_bf16_shape(n_utts=6, vocab=64, d=64, hidden=64, layers=2)
    lengths = np.array([0, 1, 2, 7, 12, 23])
    model, offsets, enc = build_case(shape, n_utts=6, lengths=lengths)
    got, _ = _gpu_decode(shape, model, offsets, enc, N, S)
    assert got[0] == [((), 0.0)]
    _check_decode(shape, model, offsets, enc, N, S)


# ------------------------------------------------------------------ peaked models: long hypotheses

def _peaked(shape, scale, blank_bias):
    """A model with peaked output distributions (the output matrix scaled up, the blank bias with it):
    hypotheses then grow to many tokens, which the benchmark models' flat distributions never
    produce.  Such a model keeps emitting within a frame, so these runs cap the rounds of a
    segment on both sides (Section 3.2 mentions such a cap)."""
    import dataclasses
    return dataclasses.replace(shape, logit_scale=scale, blank_bias=blank_bias)


@pytest.mark.parametrize("dtype,N,S,cap,bb,min_len", [("f32", 5, 3, 8, 8.0, 5), ("bf16", 5, 3, 8, 8.0, 4),
                                                     ("bf16", 4, 2, 6, 12.0, 5), ("f32", 8, 5, 8, 12.0, 5),
                                                     ("bf16", 3, 1, 5, 10.0, 4)])
def test_decode_peaked_model_long_hypotheses(dtype, N, S, cap, bb, min_len):
    """Whole decodes whose N-best lists hold sequences of five and more tokens: deep walks of the
    token trie in AddAndMerge, hash-and-walk matches between long sequences, token read-out.
    (The list kernels are the same for both storage types; the fp32 models, whose tolerance is
    ten times tighter, are the ones that stay comparable over whole utterances; bf16 models meet a
    close decision sooner and are compared strictly on shorter prefixes.)"""
    import dataclasses
    shape = _peaked(dataclasses.replace(small_bf16_shape(n_utts=8, vocab=96, d=64, hidden=64), dtype=dtype), 8.0, bb)
    lengths = np.array([23, 17, 30, 9, 41, 26, 12, 35])
    model, offsets, enc = build_case(shape, n_utts=8, lengths=lengths)
    info = _check_decode(shape, model, offsets, enc, N, S, max_rounds=cap, report=f"peaked {dtype} N={N} S={S}")
    assert info["max_len_checked"] >= min_len, info


@pytest.mark.parametrize("debug", [0, 8, 16, 1024, 2048])
@pytest.mark.parametrize("d,hidden,layers,V,U,N,S", [(64, 64, 1, 32, 1, 2, 3), (132, 36, 2, 100, 5, 5, 5), (1028, 68, 1, 64, 3, 3, 2),
                                                     (64, 128, 3, 1024, 9, 16, 1)])
def test_decode_fp32_fixed_places(d, hidden, layers, V, U, N, S, debug):
    """fp32 models in the slot layout and, by debug bits, with row lists (8), with the cell update and the
    joiner input rows as kernels of their own (16), the first round's rows as a kernel of its own (1024; it
    serves d > 1024 in any case), one workgroup per projection tile (2048): same arithmetic, same oracle."""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=U, vocab=V, d=d, hidden=hidden, layers=layers), dtype="f32")
    model, offsets, enc = build_case(shape, n_utts=U, lengths=np.arange(U) * 2 + 3)
    _, st = _gpu_decode(shape, model, offsets, enc, N, S, debug=debug)
    assert st["path"]["fixed_places"] == (debug not in (8, 16))
    _check_decode(shape, model, offsets, enc, N, S, debug=debug)


@pytest.mark.parametrize("U,N,S,V,xcd", [(3, 9, 3, 64, False), (2, 15, 5, 1000, False), (15, 5, 3, 100, True), (50, 5, 2, 33, True),
                                         (20, 12, 1, 1024, True)])
def test_decode_fp32_fixed_places_beams_and_row_ranges(U, N, S, V, xcd):
    """fp32 models in the slot layout with beams of 9 to 15 (more candidates than lanes) and, from 225 joiner rows
    on, with a range of rows per XCD in the joiner GEMM and the round kernel; the row ranges can be left out (debug
    4096) and change nothing."""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=U, vocab=V, d=64, hidden=64), dtype="f32")
    model, offsets, enc = build_case(shape, n_utts=U, lengths=(np.arange(U) * 5) % 11 + 2)
    got, st = _gpu_decode(shape, model, offsets, enc, N, S)
    assert st["path"]["fixed_places"] and xcd == (U * N * S >= 225)
    if xcd:
        assert _gpu_decode(shape, model, offsets, enc, N, S, debug=4096)[0] == got
    _check_decode(shape, model, offsets, enc, N, S)


@pytest.mark.parametrize("dtype,V,S", [("f32", 64, 3), ("bf16", 64, 3), ("bf16", 63, 3), ("bf16", 63, 1)])
def test_counters_of_steps_driven_by_the_caller(dtype, V, S):
    """tbs_stats, and the trie nodes of TBS_BUF_COUNTS, say the same whether the step functions or tbs_decode ran the
    batch, and in which layout (a batch that tbs_decode would run in the slot layout has row lists when stepped)."""
    import dataclasses
    N = 4
    shape = dataclasses.replace(small_bf16_shape(n_utts=3, vocab=V, d=128, hidden=128), dtype=dtype)
    model, offsets, enc = build_case(shape, n_utts=3, lengths=np.array([7, 4, 11]))
    seen = []
    for debug, steps in ((256, False), (0, False), (0, True)):
        tbs = make_tbs(shape, model, offsets, N, S, debug=debug)
        frames = tbs.upload_frames(enc)
        if steps:
            tbs.begin(frames, offsets)
            for seg in range(-(-11 // S)):
                rows = tbs.segment_begin(seg)
                while rows > 0:
                    tbs.joiner_segment()
                    tbs.expand()
                    tbs.select_merge()
                    tbs.predictor_step()
                    rows = tbs.counts()["rows"]
        else:
            tbs.decode(frames, offsets)
            assert tbs.path()["fixed_places"] == (debug == 0)
        seen.append((tbs.stats(), tbs.counts()["nodes"]))
        tbs.close()
    assert seen[0][0]["joiner_calls"] > 0 and seen[0][1] > 1
    assert seen[0] == seen[1] == seen[2]


@pytest.mark.parametrize("dtype,V", [("f32", 64), ("bf16", 63)])
def test_small_trie_that_one_list_of_nodes_fits(dtype, V):
    """A trie just large enough for all utterances together, too small for a share of each: fp32 models
    and vocabularies that are no whole 16-byte pieces then decode with row lists, to the same result; a stream of theirs
    runs with row lists from the start."""
    import dataclasses
    N, S = 4, 3
    shape = dataclasses.replace(small_bf16_shape(n_utts=5, vocab=V, d=128, hidden=128), dtype=dtype)
    model, offsets, enc = build_case(shape, n_utts=5, lengths=np.array([3, 40, 8, 21, 13]))

    def run(**kw):
        """(token sequences, slot layout?) or None where the trie is too small"""
        try:
            got, st = _gpu_decode(shape, model, offsets, enc, N, S, **kw)
        except RuntimeError:
            return None
        return [[y for y, _ in u] for u in got], st["path"]["fixed_places"]

    want, slots = run()
    assert slots
    lo, hi = 16, 4 * N * (85 + 5 * S) + 16   # (row lists with lo nodes overflow, with hi they do not)
    assert run(max_nodes=lo, debug=256) is None and run(max_nodes=hi, debug=256) == (want, False)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if run(max_nodes=mid, debug=256) is None else (lo, mid)
    assert run(max_nodes=hi) == (want, False)
    assert run(max_nodes=lo) is None
    tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=8)
    tbs.stream_begin(5)
    assert not tbs.path()["fixed_places"]
    tbs.close()


@pytest.mark.parametrize("dtype,V", [("f32", 64), ("bf16", 63)])
def test_small_trie_is_decoded_once(dtype, V):
    """A context whose trie is smaller than the default sizing: fp32 models and vocabularies that are no whole pieces run
    every decode once, with row lists (counted by the work of the joiner launches)."""
    import dataclasses
    from paper_2302_14357_amd.tbs import KERNEL
    N, S = 4, 3
    shape = dataclasses.replace(small_bf16_shape(n_utts=5, vocab=V, d=128, hidden=128), dtype=dtype)
    model, offsets, enc = build_case(shape, n_utts=5, lengths=np.array([3, 40, 8, 21, 13]))

    def work(**kw):
        tbs = make_tbs(shape, model, offsets, N, S, **kw)
        frames, seen = tbs.upload_frames(enc), []
        tbs.decode(frames, offsets)
        nodes = tbs.counts()["nodes"]
        tbs.profile_select(KERNEL.JOINER)
        for _ in range(2):
            tbs.decode(frames, offsets)
            p = tbs.profile_read()
            seen.append((p["launches"], p["units"]))
        assert not tbs.path()["fixed_places"]
        tbs.close()
        return nodes, seen

    nodes, want = work(debug=256)
    assert work(debug=256, max_nodes=nodes + 1) == (nodes, want)   # (as many nodes as one trie for all needs)
    assert work(max_nodes=nodes + 1) == (nodes, want)


def test_share_of_the_trie_that_was_too_small_is_remembered():
    """One utterance that emits more than its share of a trie of the default size: the first decode falls back to row
    lists, and its work is counted once; later ones of no larger shares start with row lists; a batch with larger shares
    runs in the slot layout again."""
    import dataclasses
    from paper_2302_14357_amd.tbs import KERNEL
    N, S, U, cap = 2, 1, 9, 24
    shape = dataclasses.replace(small_bf16_shape(n_utts=U, vocab=32, d=64, hidden=64), dtype="f32", act="relu")
    model, offsets, enc = build_case(shape, n_utts=U, lengths=np.full(U, 6))
    # (a blank logit that the frames alone decide: the first utterance's make it hopeless, the others' certain)
    model["w_out"] = np.zeros_like(model["w_out"])
    model["w_out"][0, :] = 0.5
    model["b_out"] = np.linspace(0.0, 0.3, 32).astype(np.float32)
    model["b_out"][0] = -60.0
    enc = np.full_like(enc, 8.0)
    enc[:6] = -64.0

    def contexts(debug, lens):
        tbs = make_tbs(shape, model, offsets, N, S, max_rounds_per_segment=cap, debug=debug, max_utts=U,
                       max_frames_total=int(offsets[-1]))
        tbs.profile_select(KERNEL.JOINER)
        out = []
        for T in lens:
            off = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
            got = tbs.decode(tbs.upload_frames(enc[:off[-1]]), off)
            p = tbs.profile_read()
            out.append((got, p["units"], tbs.path()["fixed_places"]))
        tbs.close()
        return out

    whole = np.full(U, 6)
    # (alone and two frames long, the first utterance has the whole trie: its share is larger than it needs)
    lists = contexts(256, [whole, whole, np.array([2])])
    slots = contexts(0, [whole, whole, np.array([2])])
    assert [s[2] for s in slots] == [False, False, True]
    for a, b in zip(lists, slots):
        assert a[1] == b[1]
        for x, y in zip(a[0], b[0]):
            assert [h[0] for h in x] == [h[0] for h in y]
            np.testing.assert_allclose([h[1] for h in x], [h[1] for h in y], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("N,S", [(8, 3), (9, 5), (11, 8), (12, 8), (12, 2), (16, 5), (3, 9), (2, 64), (2, 65)])
def test_decode_select_forms(N, S):
    """The frame distributions of new hypotheses: from logits asked for ahead of the ranking (one or two
    candidates a lane: beams to 8 and to 11, segments to 8 frames), by (hypothesis, frame) pairs (to 64
    frames) and by a lane per hypothesis; on each side of the lines, in both layouts where both serve."""
    shape = _peaked(small_bf16_shape(n_utts=3, vocab=64, d=128, hidden=128), 4.0, 6.0)
    model, offsets, enc = build_case(shape, n_utts=3, lengths=np.array([S + 3, 2 * S, max(S - 1, 1)]))
    for debug in (0, 256):   # (256: row lists also for small batches)
        _check_decode(shape, model, offsets, enc, N, S, max_rounds=4, debug=debug)


def test_decode_peaked_model_librispeech_widths():
    """The same at the headline widths (Dj=512, V=1024, LSTM 640, N=5, S=3)."""
    import dataclasses
    shape = _peaked(dataclasses.replace(SHAPES["librispeech"], n_utts=6), 16.0, 20.0)
    lengths = np.array([60, 90, 45, 33, 75, 52])
    model, offsets, enc = build_case(shape, n_utts=6, lengths=lengths)
    info = _check_decode(shape, model, offsets, enc, 5, 3, max_rounds=4, report="peaked, Librispeech widths")
    assert info["max_len_checked"] >= 5, info


def test_decode_truncation_and_capacity_codes():
    """Results longer than max_len come back truncated to their first max_len tokens, with their
    true lengths, and the call says TBS_EOVERFLOW; a list B or a token trie too small for the run
    is reported as the same code, not as a crash or a wrong result."""
    from paper_2302_14357_amd import TbsError
    shape = _peaked(small_bf16_shape(n_utts=3, vocab=96, d=64, hidden=64), 8.0, 8.0)
    lengths = np.array([23, 17, 30])
    model, offsets, enc = build_case(shape, n_utts=3, lengths=lengths)
    N, S, cap = 5, 3, 8
    tol, score_tol = tolerance(shape, model)
    ref = _oracle_decode(shape, model, offsets, enc, N, S, max_rounds=cap)
    longest = max(len(y) for r in ref for y, _ in r.nbest)
    assert longest >= 5
    tbs = make_tbs(shape, model, offsets, N, S, max_rounds_per_segment=cap)
    enc_dev = tbs.upload_frames(enc)
    full = tbs.decode(enc_dev, offsets)
    cut = 3
    tok = np.full((3, N, cut), -7, np.int32)
    lens = np.zeros((3, N), np.int32)
    logs = np.zeros((3, N), np.float64)
    cnt = np.zeros(3, np.int32)
    rc = tbs.decode_raw(enc_dev, offsets, tok, lens, logs, cnt, cut)
    assert rc == -5
    for u in range(3):
        assert cnt[u] == len(full[u])
        for i, (y, sc) in enumerate(full[u]):
            assert lens[u, i] == len(y) and logs[u, i] == sc
            assert tok[u, i, :min(cut, len(y))].tolist() == list(y[:cut])
            assert (tok[u, i, len(y):] == -1).all()
    with pytest.raises(TbsError) as e:
        tbs.result(max_len=257)          # beyond the configuration's max_result_len (256)
    assert e.value.code == -1
    tbs.close()
    # a trie with room for a handful of sequences only
    tbs = make_tbs(shape, model, offsets, N, S, max_rounds_per_segment=cap, max_nodes=40)
    with pytest.raises(TbsError) as e:
        tbs.decode(tbs.upload_frames(enc), offsets)
    assert e.value.code == -5
    tbs.close()
    # the same where every utterance takes nodes from a range of its own (width 128: the layout with
    # every hypothesis in a fixed place)
    shape128 = _peaked(small_bf16_shape(n_utts=3, vocab=96, d=128, hidden=128), 8.0, 8.0)
    model128, off128, enc128 = build_case(shape128, n_utts=3, lengths=lengths)
    tbs = make_tbs(shape128, model128, off128, N, S, max_rounds_per_segment=cap, max_nodes=40)
    with pytest.raises(TbsError) as e:
        tbs.decode(tbs.upload_frames(enc128), off128)
    assert e.value.code == -5
    tbs.close()
    # a list B smaller than a segment's blank expansions: the rounds of a segment are not capped,
    # the workspaces are sized for two
    tbs = make_tbs(shape, model, offsets, N, S, rounds_capacity=2)
    with pytest.raises(TbsError) as e:
        tbs.decode(tbs.upload_frames(enc), offsets)
    assert e.value.code == -5
    tbs.close()


def test_longest_list_b():
    """N * rounds capacity = 2048 entries of B per utterance, the most the library accepts."""
    shape = small_bf16_shape(n_utts=2, vocab=48, d=64, hidden=64)
    model, offsets, enc = build_case(shape, n_utts=2, lengths=np.array([9, 14]))
    _check_decode(shape, model, offsets, enc, 4, 3, rounds_capacity=512)
    from paper_2302_14357_amd import TbsError
    with pytest.raises(TbsError) as e:
        make_tbs(shape, model, offsets, 4, 3, rounds_capacity=513)
    assert e.value.code == -1


@pytest.mark.parametrize("debug", [0, 8, 32, 64, 8 + 16 + 32])
def test_decode_cell_update_inside_and_outside_the_gate_gemm(debug):
    """Two LSTM layers of 128 units: both layers fit the gate GEMM whose epilogue updates the cell
    (debug=0); debug=8 keeps the cell update a kernel of its own, 32 the gather of the first layer's
    input rows (otherwise part of the row list kernel), 64 the predictor step behind the host's wait
    for the counts (otherwise enqueued ahead of it), 56 every step that has a fused form.  All
    against the oracle."""
    shape = small_bf16_shape(n_utts=5, vocab=96, d=128, hidden=128, layers=2)
    lengths = np.array([4, 9, 15, 22, 31])
    model, offsets, enc = build_case(shape, n_utts=5, lengths=lengths)
    _check_decode(shape, model, offsets, enc, 4, 3, debug=debug)


@pytest.mark.parametrize("U,N,layers", [(103, 10, 1), (256, 16, 2), (241, 17, 1)])
def test_rows_gathered_in_the_row_list_kernel_equal_those_of_their_own(U, N, layers):
    """The parents' rows of h gathered by the row list kernel, the recurrent products behind it enqueued ahead of the counts, and (debug
    bit 5) by a kernel of their own: one hypothesis list's size over 1024, the largest that is gathered so, and one beyond."""
    shape = small_bf16_shape(n_utts=U, vocab=96, d=128, hidden=512, layers=layers)
    lengths = np.random.default_rng(U).integers(0, 9, U)
    model, offsets, enc = build_case(shape, n_utts=U, lengths=lengths)
    one, st1 = _gpu_decode(shape, model, offsets, enc, N, 2, debug=256)
    two, st2 = _gpu_decode(shape, model, offsets, enc, N, 2, debug=256 | 32)
    assert not st1["path"]["fixed_places"] and st1["joiner_calls"] == st2["joiner_calls"]
    tol, score_tol = tolerance(shape, model)
    differ = [u for u, (g, r) in enumerate(zip(one, two)) if [y for y, _ in g] != [y for y, _ in r]]
    assert len(differ) <= U // 32   # (a product may run in another kernel: decisions closer than the arithmetic can tell apart)
    assert all(abs(a[1] - b[1]) <= score_tol for u, (g, r) in enumerate(zip(one, two)) if u not in differ for a, b in zip(g, r))


@pytest.mark.parametrize("dtype,hidden,layers,V,U,N,S,debug,peaked", [
    ("bf16", 64, 1, 96, 6, 5, 3, 256, True), ("bf16", 72, 2, 96, 70, 16, 2, 256, False), ("bf16", 64, 3, 96, 6, 2, 4, 256, True),
    ("bf16", 128, 4, 96, 5, 32, 3, 256 + 8, False), ("bf16", 128, 2, 2100, 7, 5, 3, 8 + 32, True), ("bf16", 1024, 2, 300, 130, 8, 1, 512, False),
    ("f32", 36, 2, 60, 5, 4, 5, 256 + 8, True), ("f32", 37, 1, 60, 4, 3, 7, 256 + 8, True), ("f32", 64, 3, 1100, 66, 16, 2, 8, False)])
def test_recurrent_products_by_parents_equal_those_by_hypothesis(dtype, hidden, layers, V, U, N, S, debug, peaked):
    """The recurrent half of the gates once per parent (as wherever a layer does not update the cell inside its product) and, with
    debug bit 18, for every new hypothesis: batches over 1024 hypotheses and under (whose row list kernel gathers the rows), one to
    four layers, widths that are no whole pieces, beams up to the largest, empty utterances.  One layer is the same sum: the same
    bits.  More layers add the two halves separately; a gate moves by a few fp32 units, which moves a score by no more than what
    `tolerance` derives.  And the oracle's results on the default form."""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=U, vocab=V, d=64, hidden=hidden, layers=layers), dtype=dtype)
    if peaked:
        shape = _peaked(shape, 8.0, 8.0)
    lengths = np.random.default_rng(hidden + U).integers(0, 8 if U > 50 else 20, U)
    model, offsets, enc = build_case(shape, n_utts=U, lengths=lengths)
    kw = dict(max_rounds_per_segment=5)
    one, st1 = _gpu_decode(shape, model, offsets, enc, N, S, debug=debug, **kw)
    two, st2 = _gpu_decode(shape, model, offsets, enc, N, S, debug=debug | (1 << 18), **kw)
    assert not st1["path"]["fixed_places"]
    if layers == 1:
        assert one == two and st1["joiner_calls"] == st2["joiner_calls"]
    else:
        tol, score_tol = tolerance(shape, model)
        close = [u for u, (g, r) in enumerate(zip(one, two)) if [y for y, _ in g] != [y for y, _ in r]]
        assert len(close) <= U // 8   # (a decision closer than the arithmetic can tell apart)
        for u, (g, r) in enumerate(zip(one, two)):
            assert u in close or all(abs(a[1] - b[1]) <= score_tol for a, b in zip(g, r)), u
    _check_decode(shape, model, offsets, enc, N, S, max_rounds=5, debug=debug)


@pytest.mark.parametrize("d,hidden,N,S", [(128, 128, 4, 3), (144, 128, 5, 7), (80, 256, 8, 2)])
def test_decode_joiner_rows_from_the_projection_epilogue(d, hidden, N, S):
    """Where the predictor projection is a small GEMM its epilogue also forms the joiner input rows
    of the coming round; debug=16 keeps them a kernel of their own.  Widths that leave a ragged
    column tile, segments longer than the epilogue's chunk of four frames, more pairs than one
    row tile.  The two variants do the same arithmetic: identical results, and both against the
    oracle."""
    shape = small_bf16_shape(n_utts=14, vocab=96, d=d, hidden=hidden, layers=1)
    lengths = np.array([0, 1, 3, 5, 8, 9, 11, 14, 15, 17, 20, 23, 26, 29])
    model, offsets, enc = build_case(shape, n_utts=14, lengths=lengths)
    got, st = _gpu_decode(shape, model, offsets, enc, N, S)
    own, st2 = _gpu_decode(shape, model, offsets, enc, N, S, debug=16)
    for a, b in zip(got, own):
        assert [h[0] for h in a] == [h[0] for h in b]
        np.testing.assert_allclose([h[1] for h in a], [h[1] for h in b], rtol=1e-6, atol=1e-6)
    assert st["joiner_calls"] == st2["joiner_calls"]
    _check_decode(shape, model, offsets, enc, N, S)
    _check_decode(shape, model, offsets, enc, N, S, debug=16)


@pytest.mark.parametrize("base,N,S", [("tiny", 2, 3), ("small64", 4, 3), ("small128", 5, 4)])
def test_decode_relu_joiner(base, N, S):
    """The joiner with a ReLU in place of tanh (the activation of the paper's Librispeech model,
    Section 4): fp32 model, bf16 model with the input rows from their own kernel (width 64) and
    from the projection's epilogue (width 128)."""
    import dataclasses
    if base == "tiny":
        shape, kw = dataclasses.replace(SHAPES["tiny"], act="relu"), {}
    else:
        w = int(base[5:])
        shape = dataclasses.replace(small_bf16_shape(n_utts=6, vocab=80, d=w, hidden=w), act="relu")
        kw = dict(n_utts=6, lengths=np.array([2, 5, 9, 14, 20, 27]))
    model, offsets, enc = build_case(shape, **kw)
    _check_decode(shape, model, offsets, enc, N, S)


# ------------------------------------------------------------------ streaming

def _push_in_pieces(tbs, shape, offsets, enc, piece_of, flush_last=True):
    """Feed every utterance its frames in pieces of piece_of(u, call) frames until all are in."""
    U = len(offsets) - 1
    T = np.diff(offsets)
    sent = np.zeros(U, dtype=np.int64)
    tbs.stream_begin(U)
    call = 0
    while (sent < T).any():
        n = np.array([min(int(piece_of(u, call)), int(T[u] - sent[u])) for u in range(U)])
        off = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
        rows = np.concatenate([enc[offsets[u] + sent[u]: offsets[u] + sent[u] + n[u]] for u in range(U)]) \
            if n.sum() else np.zeros((0, enc.shape[1]), np.float32)
        sent += n
        last = not (sent < T).any()
        tbs.push_segment(tbs.upload_frames(rows), off, flush=(last and flush_last))
        call += 1
    if T.sum() == 0:
        tbs.push_segment(None, np.zeros(U + 1, np.int32), flush=True)


@pytest.mark.parametrize("N,S,pieces", [(4, 3, "random"), (3, 4, "one"), (5, 3, "segment"), (2, 5, "uneven")])
def test_streaming_in_pieces_equals_decode(N, S, pieces):
    """Encoder frames arriving in pieces (frame by frame, in decoder-sized segments, in random
    sizes different per utterance, or some utterances much faster than others) and a flush at
    the end give what tbs_decode gives on the whole utterances (Section 3.2: the encoder's
    segment size need not be the decoder's): the segments of an utterance are the same either
    way, so the results are required to be identical; tbs_decode itself is checked against the
    oracle."""
    shape = small_bf16_shape(n_utts=7, vocab=64, d=128, hidden=128, layers=1)
    lengths = np.array([0, 1, 4, 9, 13, 22, 30])
    model, offsets, enc = build_case(shape, n_utts=7, lengths=lengths)
    rng = np.random.default_rng(5)
    draws = rng.integers(0, 2 * S + 2, size=(7, 200))
    piece_of = {"random": lambda u, c: draws[u, c], "one": lambda u, c: 1, "segment": lambda u, c: S,
                "uneven": lambda u, c: (u % 3) * 3 + 1}[pieces]
    whole, st0 = _gpu_decode(shape, model, offsets, enc, N, S)
    tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=3 * S + 2)
    _push_in_pieces(tbs, shape, offsets, enc, piece_of)
    got = tbs.result()
    st = tbs.stats()
    tbs.close()
    for a, b in zip(got, whole):
        assert [h[0] for h in a] == [h[0] for h in b]
        np.testing.assert_allclose([h[1] for h in a], [h[1] for h in b], rtol=1e-5, atol=1e-5)
    assert st["frames"] == int(lengths.sum()) and st["joined_frames"] == st0["joined_frames"]
    _check_decode(shape, model, offsets, enc, N, S)


@pytest.mark.parametrize("N,V", [(3, 63), (5, 63), (4, 1030), (6, 1030)])
def test_streams_of_single_frames_in_fixed_places(N, V):
    """Segments of one frame of a bf16 model run in the slot layout whatever the vocabulary, as a stream too (the form
    without logits serves any), and a stream gives what the whole decode gives."""
    shape = small_bf16_shape(n_utts=3, vocab=V, d=128, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=3, lengths=np.array([7, 1, 12]))
    whole, st = _gpu_decode(shape, model, offsets, enc, N, 1)
    assert st["path"]["fixed_places"]
    tbs = make_tbs(shape, model, offsets, N, 1, stream_buffer_frames=4)
    _push_in_pieces(tbs, shape, offsets, enc, lambda u, c: 1 + (u + c) % 3)
    assert tbs.path() == st["path"]
    assert tbs.result() == whole
    tbs.close()
    _check_decode(shape, model, offsets, enc, N, 1)


def test_streaming_partial_results_and_limits():
    """Between pushes B holds the result for the frames decoded so far: with no flush, that is the
    decode of each utterance's whole segments.  A push beyond the buffer is refused and
    changes nothing; step calls and pushes do not mix."""
    from paper_2302_14357_amd.tbs import TbsError
    shape = small_bf16_shape(n_utts=3, vocab=48, d=64, hidden=64)
    N, S = 3, 4
    lengths = np.array([10, 17, 6])
    model, offsets, enc = build_case(shape, n_utts=3, lengths=lengths)
    tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=12)
    with pytest.raises(TbsError):
        tbs.push_segment(None, np.zeros(4, np.int32))          # no stream begun
    _push_in_pieces(tbs, shape, offsets, enc, lambda u, c: 5, flush_last=False)
    got = tbs.result()
    done = (lengths // S) * S
    off2 = np.concatenate([[0], np.cumsum(done)]).astype(np.int32)
    enc2 = np.concatenate([enc[offsets[u]: offsets[u] + done[u]] for u in range(3)])
    part, _ = _gpu_decode(shape, model, off2, enc2, N, S)
    for a, b in zip(got, part):
        assert [h[0] for h in a] == [h[0] for h in b]
        np.testing.assert_allclose([h[1] for h in a], [h[1] for h in b], rtol=1e-5, atol=1e-5)
    _check_decode(shape, model, off2, enc2, N, S)
    # 2, 1, 2 frames are still buffered; 11 more do not fit into 12
    with pytest.raises(TbsError):
        tbs.push_segment(tbs.upload_frames(np.zeros((11, 64), np.float32)), np.array([0, 11, 11, 11], np.int32))
    with pytest.raises(TbsError):
        tbs.segment_begin(0)
    assert tbs.result() == got
    # the rest of the stream still decodes: flush the leftovers
    tbs.push_segment(None, np.zeros(4, np.int32), flush=True)
    rest = tbs.result()
    tbs.close()
    whole, _ = _gpu_decode(shape, model, offsets, enc, N, S)
    for a, b in zip(rest, whole):
        assert [h[0] for h in a] == [h[0] for h in b]
        np.testing.assert_allclose([h[1] for h in a], [h[1] for h in b], rtol=1e-5, atol=1e-5)
    _check_decode(shape, model, offsets, enc, N, S)


def _step_by_step(shape, model, offsets, enc, N, S, max_rounds=0, **kw):
    """Drive the step entry points over a batch and compare A and B of every utterance with the
    oracle's trace after every round, up to the utterance's first close decision (from there on its
    run may legitimately differ and it is only followed).  Lists are compared as sets of token
    sequences with their scores: the order inside A changes no score.  Returns what was covered."""
    from paper_2302_14357_amd import BUF
    tol, score_tol = tolerance(shape, model)
    U = len(offsets) - 1
    T = np.diff(offsets)
    okw = dict(max_rounds=max_rounds) if max_rounds else {}
    ref = _oracle_decode(shape, model, offsets, enc, N, S, **okw)
    gkw = dict(kw)
    if max_rounds:
        gkw["max_rounds_per_segment"] = max_rounds
    tbs = make_tbs(shape, model, offsets, N, S, debug=1, **gkw)
    tbs.begin(tbs.upload_frames(enc), offsets)
    trace = [{(r.seg, r.round): r for r in ref[u].rounds} for u in range(U)]
    stop = [ref[u].first_ambiguous_segment(tol) for u in range(U)]
    cov = {"rounds": 0, "merges": 0, "max_len": 0, "deep_merges": 0}
    nseg = (int(T.max()) + S - 1) // S if U else 0
    for seg in range(nseg):
        rows = tbs.segment_begin(seg)
        rnd = 0
        prev_nb = [0] * U
        while rows > 0:
            rnd += 1
            a_now = tbs.debug_hyps(0)
            tbs.joiner_segment()
            tbs.expand()
            live = tbs.select_merge()
            b_now = tbs.debug_hyps(1, cap=N * (max_rounds or 32))
            a_new = tbs.debug_hyps(0)
            dh = tbs.debug_read(BUF.A_DHAT)
            for u in range(U):
                if stop[u] is not None and seg >= stop[u]:
                    continue
                r = trace[u].get((seg, rnd))
                if r is None:
                    assert a_now[u] == [] or seg * S >= T[u], (u, seg, rnd)
                    continue
                cov["rounds"] += 1
                assert {y for y, _ in a_now[u]} == set(r.a_tokens), (u, seg, rnd)
                want = dict(zip(r.a_tokens, r.a_scores))
                for y, sc in a_now[u]:
                    assert abs(sc - want[y]) <= score_tol, (u, seg, rnd, y)
                assert [y for y, _ in b_now[u]] == r.b_tokens, (u, seg, rnd)     # insertion order is unique
                np.testing.assert_allclose([sc for _, sc in b_now[u]], r.b_scores, atol=score_tol)
                new_tokens = [r.a_tokens[h] + (k,) for h, k in r.new_pairs]
                if max_rounds and rnd >= max_rounds:
                    new_tokens = []      # the round cap: what the last allowed round creates is dropped
                assert {y for y, _ in a_new[u]} == set(new_tokens), (u, seg, rnd)
                for i, (y, sc) in enumerate(a_new[u]):
                    j = new_tokens.index(y)
                    assert abs(sc - r.new_scores[j]) <= score_tol
                    np.testing.assert_allclose(dh[u, i, :r.S], r.new_d[j], rtol=10 * tol, atol=1e-7)
                merged = prev_nb[u] + len(r.a_tokens) - len(r.b_tokens)
                cov["merges"] += merged
                if merged:
                    cov["deep_merges"] += sum(1 for y in r.a_tokens if len(y) >= 3 and y in r.b_tokens[:prev_nb[u]])
                prev_nb[u] = len(r.b_tokens)
                cov["max_len"] = max([cov["max_len"]] + [len(y) for y in r.b_tokens])
            tbs.predictor_step()
            rows = tbs.counts()["rows"]
    final = tbs.result()
    for u in range(U):
        if stop[u] is None:
            why = nbest_agrees(final[u], ref[u], score_tol, tol)
            assert why is None, (u, why)
    tbs.close()
    return cov


def test_decode_step_by_step_matches_oracle_trace():
    """One utterance at the benchmark models' scale: A and B after every round."""
    shape = small_bf16_shape(n_utts=1, vocab=48, d=64, hidden=64)
    model, offsets, enc = build_case(shape, n_utts=1, lengths=np.array([38]))
    cov = _step_by_step(shape, model, offsets, enc, 3, 4)
    assert cov["merges"] > 0 and cov["rounds"] > 10, cov


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_step_by_step_peaked_batch(dtype):
    """A batch with a peaked model: A and B of every utterance after every round while the
    hypotheses grow long, including merges between sequences of three and more tokens (a sequence
    carried into a segment meeting the same sequence re-created in it)."""
    import dataclasses
    shape = _peaked(dataclasses.replace(small_bf16_shape(n_utts=5, vocab=12, d=64, hidden=64), dtype=dtype), 8.0, 8.0)
    lengths = np.array([30, 21, 38, 14, 26])
    model, offsets, enc = build_case(shape, n_utts=5, lengths=lengths)
    cov = _step_by_step(shape, model, offsets, enc, 5, 3, max_rounds=6)
    print(cov)
    assert cov["max_len"] >= 5, cov
    if dtype == "f32":   # (the tighter tolerance keeps these runs comparable to their ends)
        assert cov["deep_merges"] >= 10 and cov["max_len"] >= 10, cov


@pytest.mark.parametrize("d,limit", [(64, 2), (128, 2), (128, 1)])
def test_round_limit_matches_oracle(d, limit):
    """Hypotheses still emitting after `limit` rounds of a segment are dropped (Section 3.2 mentions
    such a limit).  Width 128 takes the path on which a segment's head and first round are enqueued
    in one go (with limit 1 the drop falls into that first round), width 64 the step-by-step one."""
    shape = small_bf16_shape(n_utts=2, vocab=32, d=d, hidden=d)
    model, offsets, enc = build_case(shape, n_utts=2, lengths=np.array([9, 6]))
    _check_decode(shape, model, offsets, enc, 4, 3, max_rounds=limit)


def test_batch_equals_each_alone_and_is_deterministic():
    shape = small_bf16_shape(n_utts=4, vocab=64, d=64, hidden=64)
    model, offsets, enc = build_case(shape, n_utts=4, lengths=np.array([11, 4, 17, 8]))
    together, _ = _gpu_decode(shape, model, offsets, enc, 3, 3)
    again, _ = _gpu_decode(shape, model, offsets, enc, 3, 3)
    assert together == again
    for u in range(4):
        o = np.array([0, offsets[u + 1] - offsets[u]], np.int32)
        alone, _ = _gpu_decode(shape, model, o, enc[offsets[u]:offsets[u + 1]], 3, 3)
        assert [y for y, _ in alone[0]] == [y for y, _ in together[u]]
        np.testing.assert_allclose([s for _, s in alone[0]], [s for _, s in together[u]], atol=1e-5)


def test_decode_librispeech_headline_batch():
    """The benchmark's own batch in the benchmark's launch configuration (64 utterances, 17983
    frames, Dj=512, V=1024, LSTM 640, N=5, S=3): every utterance against the oracle, whole where
    all its decisions were clear and up to its first close decision otherwise."""
    shape = SHAPES["librispeech"]
    model = make_model(shape)
    offsets, enc = make_utterances(shape, model)
    info = _check_decode(shape, model, offsets, enc, 5, 3, report="Librispeech-like headline batch")
    assert info["tot"] == 64
    # flat synthetic distributions put thousands of expansion scores within 1e-3 of each other, so
    # every utterance meets a close decision within its first segments and the part the rule
    # makes strict is short; the whole-utterance count above it is reported (the kernels' actual
    # error is ~1e-6, so in practice the whole batch agrees)
    assert info.get("prefix_frames", int(offsets[-1])) >= 500, info


@pytest.mark.parametrize("index,N,S", [(11, 5, 3), (23, 5, 3), (37, 4, 5), (41, 10, 2)])
def test_decode_librispeech_widths_other_draws(index, N, S):
    """The headline widths (Dj=512, V=1024, LSTM 640) with other draws of the model and of the frames
    than the benchmark's, and utterance lengths around the segment size and its multiples (empty,
    shorter than a segment, a ragged last segment, one frame more or less than whole segments):
    the fixed-place form against the oracle."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["librispeech"], index=index, n_utts=12)
    lengths = np.array([0, 1, 2, S, S + 1, 2 * S - 1, 40, 77, 30 * S, 30 * S + 1, 30 * S - 1, 211])
    model, offsets, enc = build_case(shape, n_utts=12, lengths=lengths)
    _, st = _gpu_decode(shape, model, offsets, enc, N, S)
    assert st["path"]["fixed_places"]
    _check_decode(shape, model, offsets, enc, N, S)


@pytest.mark.parametrize("U,N,S", [(70, 5, 3), (100, 5, 3), (273, 5, 3), (274, 5, 3), (90, 4, 1)])
def test_decode_fixed_places_with_more_tiles_than_cus(U, N, S):
    """The headline widths with so many utterances that the GEMMs of a round have more 64x64 tiles
    than the chip has CUs (up to 1024 joiner tiles: the fixed-place form still runs, its GEMMs with two
    LDS stages a workgroup and two workgroups a CU, K tiles refilled as they are read), one utterance
    more (the row-list form), and one-frame segments without logits: short utterances, all against
    the oracle."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["librispeech"], index=53, n_utts=U)
    rng = np.random.default_rng(U)
    lengths = rng.integers(0, 14, size=U)
    model, offsets, enc = build_case(shape, n_utts=U, lengths=lengths)
    _, st = _gpu_decode(shape, model, offsets, enc, N, S)
    assert st["path"]["fixed_places"] == (U <= 273)
    _check_decode(shape, model, offsets, enc, N, S)


@pytest.mark.parametrize("name,N,S", [("assistant", 10, 3), ("throughput", 10, 5)])
def test_decode_large_shapes_short_utterances(name, N, S):
    """Whole decodes at the widths of the two large configurations (V=4096, Dj=1024, LSTM 2x1024 /
    1x1024) on a few short utterances, against the oracle."""
    import dataclasses
    shape = dataclasses.replace(SHAPES[name], n_utts=4)
    lengths = np.array([7, 16, 23, 30])
    model, offsets, enc = build_case(shape, n_utts=4, lengths=lengths)
    _check_decode(shape, model, offsets, enc, N, S, report=name)


@pytest.mark.parametrize("N,S", [(2, 1), (2, 5), (10, 1), (10, 2), (10, 5), (5, 2), (5, 5)])
def test_decode_librispeech_like_beam_and_segment_sweep(N, S):
    """The Librispeech-like configuration's sweep of beam and segment sizes, at its widths, on three
    utterances of 30-60 frames, whole decode against the oracle."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["librispeech"], n_utts=3)
    lengths = np.array([31, 44, 60])
    model, offsets, enc = build_case(shape, n_utts=3, lengths=lengths)
    _check_decode(shape, model, offsets, enc, N, S)


@pytest.mark.parametrize("S", [10, 20, 50])
def test_decode_long_segments(S):
    """The long-segment configuration (Librispeech-like widths, N=5, S in {10, 20, 50}): the scan of
    Eq. 3 over long segments and the expansion kernels for S beyond the register-resident range."""
    import dataclasses
    shape = dataclasses.replace(SHAPES["librispeech"], n_utts=2)
    lengths = np.array([75, 128])
    model, offsets, enc = build_case(shape, n_utts=2, lengths=lengths)
    # a segment of S frames can take more rounds than the default workspace is sized for
    # (with blank probabilities of a few percent the blank products over such segments span ~1e-85:
    # this is the case that needs the forward variable and d carried with extended range)
    _check_decode(shape, model, offsets, enc, 5, S, rounds_capacity=4 * S, report=f"S={S}")


@pytest.mark.parametrize("V,S,blank", [(1024, 6, 0), (1024, 7, 5), (500, 8, 0), (200, 8, 199), (257, 9, 0), (511, 32, 17), (512, 33, 0),
                                       (500, 64, 0), (1000, 9, 999), (1023, 33, 0), (1021, 64, 1020), (1024, 32, 1023)])
def test_joiner_expand_long_segments(V, S, blank):
    """k_expand_long over what it serves: one, two and four 16-byte pieces a lane, two and four rows a wave, each at the
    edges of its range of frames, vocabularies that leave lanes without a piece or a piece partly beyond the vocabulary,
    a blank that is not token 0; full and ragged segments (the utterances' lengths differ), then every score equal."""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=5, vocab=V, d=64, hidden=64), blank_id=blank, len_lo=2, len_hi=S + 3)
    _check_joiner_expand(shape, U=5, N=5, S=S, seg=0, sample_pairs=8, rounds_capacity=4 * S)
    if blank == 0:
        _check_joiner_expand(shape, U=3, N=6, S=S, seg=0, sample_pairs=3, flat=True, rounds_capacity=4 * S)


@pytest.mark.parametrize("V,S,N", [(1000, 7, 3), (400, 8, 10), (257, 12, 4), (1023, 40, 3)])
def test_decode_long_segments_other_vocabularies(V, S, N):
    """Whole decodes whose expansions run in k_expand_long, on vocabularies that are no power of two."""
    shape = small_bf16_shape(n_utts=3, vocab=V, d=128, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=3, lengths=np.array([S + 3, 2 * S, 1]))
    _check_decode(shape, model, offsets, enc, N, S, rounds_capacity=4 * S)


def test_decode_largest_segment_and_smallest_vocabulary():
    """The limits of the configuration: S = 128 (the largest segment the library takes; one full
    segment and a ragged one) with a small model, and V = 2 (blank and one token: every hypothesis
    has one expansion, top-N and threshold degenerate) at several beam widths."""
    shape = small_bf16_shape(n_utts=2, vocab=24, d=64, hidden=64)
    lengths = np.array([140, 131])
    model, offsets, enc = build_case(shape, n_utts=2, lengths=lengths)
    _check_decode(shape, model, offsets, enc, 3, 128, rounds_capacity=512)
    shape2 = small_bf16_shape(n_utts=3, vocab=2, d=64, hidden=64)
    model2, off2, enc2 = build_case(shape2, n_utts=3, lengths=np.array([5, 11, 2]))
    for N, S in ((1, 1), (3, 2), (4, 5)):
        _check_decode(shape2, model2, off2, enc2, N, S)


@pytest.mark.parametrize("name,N,S,U", [("assistant", 10, 3, 300), ("throughput", 10, 5, 200)])
def test_decode_large_batch_contains_the_small_one(name, N, S, U):
    """The large configurations' widths with enough utterances that every round runs on the kernels
    chosen at scale (256x256-tile joiner GEMM, 80- or 48-logit-per-thread expansion, LSTM cell
    update as its own kernel behind a large gate GEMM): the first eight utterances against the
    oracle under the gap rule, decoded inside the large batch."""
    import dataclasses
    shape = dataclasses.replace(SHAPES[name], n_utts=U)
    lengths = np.concatenate([np.array([7, 16, 23, 30, 5, 11, 19, 26]), np.full(U - 8, 12)])
    model, offsets, enc = build_case(shape, n_utts=U, lengths=lengths)
    tol, score_tol = tolerance(shape, model)
    full, st = _gpu_decode(shape, model, offsets, enc, N, S)
    assert st["frames"] == int(offsets[-1])
    off8 = offsets[:9].copy()
    ref = _oracle_decode(shape, model, off8, enc[:off8[-1]], N, S)
    same, amb, tot = compare_nbest(full[:8], ref, score_tol=score_tol, gap_tol=tol)
    # the same eight cut back to before their first close decision, again inside a large batch
    offp, encp, keep = strict_prefixes(ref, off8, enc[:off8[-1]], S, tol)
    lengths2 = np.concatenate([keep, np.full(U - 8, 12)])
    off2 = np.concatenate([[0], np.cumsum(lengths2)]).astype(np.int32)
    enc2 = np.concatenate([encp, enc[off8[-1]:]])
    full2, _ = _gpu_decode(shape, model, off2, enc2, N, S)
    ref2 = _oracle_decode(shape, model, offp, encp, N, S)
    assert_all_agree(full2[:8], ref2, score_tol, tol)
    print(f"{name}: identical {same}/{tot} whole, strict prefix frames {int(keep.sum())}/{int(off8[-1])}")


@pytest.mark.parametrize("N,S,V,peaked", [(3, 3, 96, False), (4, 5, 1024, False), (5, 3, 1024, False), (8, 5, 512, True),
                                          (10, 3, 1024, False), (16, 4, 200, True), (5, 3, 96, True), (2, 1, 64, True)])
def test_round_in_one_kernel_equals_separate_kernels(N, S, V, peaked):
    """Inside tbs_decode, expansion and select/merge of a round run as one kernel (a workgroup per
    utterance) where the shape allows; debug bit 7 keeps them two kernels.  Beam widths and
    vocabularies that take each of the kernel's forms (4, 8 or 16 columns per thread, with and without
    a wave of its own for the select step), ragged utterances, flat and peaked models: the two forms must give the same hypotheses, and the
    one-kernel form is checked against the oracle."""
    shape = small_bf16_shape(n_utts=6, vocab=V, d=128, hidden=128)
    cap = 0
    if peaked:
        shape, cap = _peaked(shape, 8.0, 8.0), 5
    lengths = np.array([0, 2, 7, 12, 23, 31])
    model, offsets, enc = build_case(shape, n_utts=6, lengths=lengths)
    kw = dict(max_rounds_per_segment=cap) if cap else {}
    # default: every hypothesis in a fixed place, four kernels a round; 256: the one-kernel round with
    # row lists made by a kernel of their own; 128: expansion and select/merge as two kernels as well
    one, st1 = _gpu_decode(shape, model, offsets, enc, N, S, **kw)
    for dbg in (256, 128):
        two, st2 = _gpu_decode(shape, model, offsets, enc, N, S, debug=dbg, **kw)
        for a, b in zip(one, two):
            assert [h[0] for h in a] == [h[0] for h in b], dbg
            np.testing.assert_allclose([h[1] for h in a], [h[1] for h in b], rtol=1e-6, atol=1e-5)
        assert st1["joiner_calls"] == st2["joiner_calls"] and st1["joined_frames"] == st2["joined_frames"], dbg
        assert st1["launches"] == st2["launches"] and st1["frames"] == st2["frames"], dbg
    _check_decode(shape, model, offsets, enc, N, S, max_rounds=cap)
    _check_decode(shape, model, offsets, enc, N, S, max_rounds=cap, debug=256)
    _check_decode(shape, model, offsets, enc, N, S, max_rounds=cap, debug=128)


@pytest.mark.parametrize("N,V,blank,peaked", [(1, 64, 0, False), (2, 96, 0, True), (4, 1024, 0, False), (5, 1024, 0, True),
                                              (5, 200, 7, True), (8, 512, 511, True), (10, 4096, 0, False),
                                              (16, 100, 64, True), (3, 68, 67, False)])
def test_standard_search_without_logits_equals_the_one_with(N, V, blank, peaked):
    """S = 1 is the standard breadth-first search (Eq. 1).  The joiner GEMM can then keep no logits: its
    epilogue leaves each row's softmax sums, blank logit and N best tokens per 16-column piece (or, debug
    bit 14, merged per tile of 64 columns) and the round kernel merges them.  That form runs by default
    for beams up to 4 and where the vocabulary is too large for the form with logits, and with debug bit
    15 everywhere; debug bit 9 asks for the logits.  Vocabularies of one tile, of many and with a ragged last tile, blank
    first, last, at a tile edge and inside a tile, every list length the round kernel has (4, 8, 16),
    flat and peaked models, ragged and empty utterances: the forms give the same hypotheses, and each is
    checked against the oracle."""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=6, vocab=V, d=128, hidden=128), blank_id=blank)
    cap = 0
    if peaked:
        shape, cap = _peaked(shape, 8.0, 8.0), 5
    lengths = np.array([0, 1, 7, 12, 23, 31])
    model, offsets, enc = build_case(shape, n_utts=6, lengths=lengths)
    kw = dict(max_rounds_per_segment=cap) if cap else {}
    dflt, st0 = _gpu_decode(shape, model, offsets, enc, N, 1, **kw)
    one, st1 = _gpu_decode(shape, model, offsets, enc, N, 1, debug=32768, **kw)
    two, st2 = _gpu_decode(shape, model, offsets, enc, N, 1, debug=512, **kw)
    # (the form with logits keeps a hypothesis' logits in registers: vocabularies up to 1024 entries)
    # (by default the form without logits serves beams up to 4 and the vocabularies the other cannot hold)
    assert st0["path"] == {"fixed_places": True, "one_frame_no_logits": V > 1024 or N <= 4}
    assert st1["path"] == {"fixed_places": True, "one_frame_no_logits": True}
    assert st2["path"] == {"fixed_places": V <= 1024, "one_frame_no_logits": False}
    assert dflt == (one if (V > 1024 or N <= 4) else two)
    tol, score_tol = tolerance(shape, model)
    # (bit 14: the partials of a tile's four 16-column pieces merged by the GEMM instead of the round kernel:
    # the same arithmetic in another order of the sums)
    three, st3 = _gpu_decode(shape, model, offsets, enc, N, 1, debug=32768 + 16384, **kw)
    assert st3["path"] == st1["path"]
    for other in (two, three):
        for a, b in zip(one, other):
            # (the forms round differently: log(exp(l - m) / Z) against (l - m) - log Z)
            assert [h[0] for h in a] == [h[0] for h in b]
            np.testing.assert_allclose([h[1] for h in a], [h[1] for h in b], rtol=0, atol=score_tol)
    assert st1["joiner_calls"] == st2["joiner_calls"] and st1["joined_frames"] == st2["joined_frames"]
    assert st1["launches"] == st2["launches"] and st1["frames"] == st2["frames"]
    _check_decode(shape, model, offsets, enc, N, 1, max_rounds=cap, debug=32768)
    _check_decode(shape, model, offsets, enc, N, 1, max_rounds=cap, debug=512)
    _check_decode(shape, model, offsets, enc, N, 1, max_rounds=cap, debug=32768 + 16384)


def test_standard_search_without_logits_librispeech_batch():
    """The in-house baseline of the benchmark (64 Librispeech-like utterances, N = 5, S = 1) in the form
    without logits agrees with the oracle under the gap rule."""
    shape = SHAPES["librispeech"]
    model, offsets, enc = build_case(shape)
    _, st = _gpu_decode(shape, model, offsets[:3], enc[:offsets[2]], 5, 1, debug=32768)
    assert st["path"]["one_frame_no_logits"]
    info = _check_decode(shape, model, offsets, enc, 5, 1, report="Librispeech-like, standard search (S=1)",
                         debug=32768)
    assert info["tot"] == 64


@pytest.mark.parametrize("N,S,U", [(5, 3, 6), (4, 5, 6), (10, 2, 70), (3, 1, 130)])
def test_first_round_rows_from_the_segment_head_equal_those_of_their_own_kernel(N, S, U):
    """In the layout with fixed places the kernel that starts a segment also forms the joiner input
    rows of the segment's first round, with one, two or four workgroups per utterance depending on the
    batch; debug bit 10 forms them in a kernel of their own.  Ragged and empty utterances, batches of
    every workgroup count: identical hypotheses, and the oracle on the first utterances."""
    shape = small_bf16_shape(n_utts=U, vocab=128, d=128, hidden=128)
    rng = np.random.default_rng(7)
    lengths = rng.integers(0, 20, size=U)
    lengths[:6] = [0, 1, 7, 12, 23, 31]
    model, offsets, enc = build_case(shape, n_utts=U, lengths=lengths)
    one, st1 = _gpu_decode(shape, model, offsets, enc, N, S)
    # (bit 11: the later rounds' rows, from the projection's epilogue, by one workgroup per tile instead of
    # one per tile and frame)
    # (bit 12: the joiner GEMM's tiles spread over the XCDs as the other GEMMs' are, instead of a range of
    # rows per XCD with the round kernel's workgroups placed to match)
    for dbg in (1024, 2048, 4096, 1024 + 2048 + 4096):
        two, st2 = _gpu_decode(shape, model, offsets, enc, N, S, debug=dbg)
        assert st1["path"]["fixed_places"] and st2["path"]["fixed_places"]
        assert one == two, dbg
        assert st1["joiner_calls"] == st2["joiner_calls"] and st1["joined_frames"] == st2["joined_frames"]
    _check_decode(shape, model, offsets[:7], enc[:offsets[6]], N, S)


@pytest.mark.parametrize("N,S,d", [(5, 3, 64), (3, 12, 64), (10, 2, 128), (4, 5, 144)])
def test_joiner_rows_by_pair_equal_those_by_row(N, S, d):
    """With row lists the joiner input rows act(e + p) come from a kernel of their own: a thread per
    pair and 8 columns (all frames of the pair), or with debug bit 13 a thread per row and 8 columns.
    Identical hypotheses required, and the oracle's on the default form."""
    shape = small_bf16_shape(n_utts=6, vocab=96, d=d, hidden=64)
    lengths = np.array([0, 1, 7, 12, 23, 31])
    model, offsets, enc = build_case(shape, n_utts=6, lengths=lengths)
    kw = dict(rounds_capacity=4 * S) if S > 8 else {}
    one, st1 = _gpu_decode(shape, model, offsets, enc, N, S, debug=256, **kw)
    two, st2 = _gpu_decode(shape, model, offsets, enc, N, S, debug=256 + 8192, **kw)
    assert not st1["path"]["fixed_places"]
    assert one == two
    assert st1["joiner_calls"] == st2["joiner_calls"] and st1["joined_frames"] == st2["joined_frames"]
    _check_decode(shape, model, offsets, enc, N, S, debug=256, **kw)


@pytest.mark.parametrize("chunk", [1, 11, 40])
def test_decode_with_joiner_calls_in_pieces(chunk):
    """Whole decodes whose every joiner call of more than `chunk` rows runs in pieces."""
    shape = small_bf16_shape(n_utts=6, vocab=64, d=64, hidden=64, layers=2)
    lengths = np.array([0, 1, 2, 7, 12, 23])
    model, offsets, enc = build_case(shape, n_utts=6, lengths=lengths)
    _check_decode(shape, model, offsets, enc, 5, 3, joiner_chunk_rows=chunk)
    whole, _ = _gpu_decode(shape, model, offsets, enc, 5, 3, joiner_chunk_rows=0)
    parts, _ = _gpu_decode(shape, model, offsets, enc, 5, 3, joiner_chunk_rows=chunk)
    assert whole == parts      # the same arithmetic per row, whatever the pieces


@pytest.mark.parametrize("N,S", [(32, 2), (17, 3)])
def test_decode_wide_beams(N, S):
    """Beams up to the library's maximum: the list kernels' general paths (more than 64 candidates
    per utterance, B lists of hundreds of entries)."""
    shape = small_bf16_shape(n_utts=3, vocab=96, d=64, hidden=64)
    lengths = np.array([5, 11, 18])
    model, offsets, enc = build_case(shape, n_utts=3, lengths=lengths)
    _check_decode(shape, model, offsets, enc, N, S)


def test_errors_are_codes_not_crashes():
    from paper_2302_14357_amd import TbsError
    shape = small_bf16_shape(n_utts=2)
    model, offsets, enc = build_case(shape, n_utts=2, lengths=np.array([5, 6]))
    tbs = make_tbs(shape, model, offsets, 2, 2)
    with pytest.raises(TbsError) as e:
        tbs.expand()            # before begin / joiner
    assert e.value.code == -2
    enc_dev = tbs.upload_frames(enc)
    tbs.begin(enc_dev, offsets)
    with pytest.raises(TbsError) as e:
        tbs.joiner_segment()    # before segment_begin
    assert e.value.code == -2
    with pytest.raises(TbsError) as e:
        tbs.begin(enc_dev, np.array([0, 5, 11, 12], np.int32))   # more utterances than capacity
    assert e.value.code == -1
    tbs.close()
    # rounds capacity of one: the second round of a segment overflows cleanly
    tbs = make_tbs(shape, model, offsets, 2, 2, rounds_capacity=1)
    with pytest.raises(TbsError) as e:
        tbs.decode(tbs.upload_frames(enc), offsets)
    assert e.value.code == -5
    tbs.close()
    # the same at a width whose segments are enqueued head and first round in one go, and the
    # context still decodes afterwards when given the room
    shape = small_bf16_shape(n_utts=2, d=128, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=2, lengths=np.array([5, 6]))
    tbs = make_tbs(shape, model, offsets, 2, 2, rounds_capacity=1)
    with pytest.raises(TbsError) as e:
        tbs.decode(tbs.upload_frames(enc), offsets)
    assert e.value.code == -5
    tbs.close()
    _check_decode(shape, model, offsets, enc, 2, 2)


def _assert_one_launch(tbs, segments, debug=0):
    """The batch's segments ran inside one launch, every one of them, or (debug bit 16) in no launch, or (bit 17) in launches
    that gave up: what ran, not what could have."""
    ran = tbs.one_launch()
    assert ran["may"] == (debug != 65536)
    assert ran["segments"] == (segments if debug == 0 else 0) and (ran["gave_up"] > 0) == (debug == 131072), ran


def _segments(offsets, S):
    return -(-int(np.diff(offsets).max()) // S)


@pytest.mark.parametrize("dtype,d,hidden,V,N,S,lengths,peaked", [
    ("f32", 64, 64, 32, 2, 3, [50], False), ("f32", 72, 72, 37, 8, 5, [9, 12, 33, 1, 0, 31], True), ("f32", 96, 136, 97, 3, 1, [9, 2, 31], False),
    ("f32", 256, 200, 500, 10, 4, [7, 30, 12], False), ("f32", 512, 640, 1001, 5, 3, [6, 40, 11], False),
    ("f32", 520, 384, 1024, 11, 5, [4, 9], True), ("f32", 64, 128, 60, 5, 2, [2 + i % 9 for i in range(50)], False)] + [("bf16",) + c for c in [
    (128, 128, 17, 1, 2, [5], False), (128, 256, 96, 5, 3, [0, 1, 7, 12, 23, 31], True), (256, 128, 200, 5, 1, [3] * 9, False),
    (384, 384, 257, 7, 5, list(range(1, 18)), True), (512, 640, 1024, 5, 3, [8] * 3 + [40] * 6, False), (640, 512, 1023, 3, 2, [9, 30], False),
    (512, 640, 1000, 10, 3, [17] * 5, False), (512, 640, 500, 10, 5, [21, 20, 19, 5], True), (128, 128, 512, 8, 4, [6, 33], True),
    (128, 128, 33, 11, 5, [11, 12], True), (256, 384, 40, 4, 3, [3 + i % 7 for i in range(300)], False), (128, 128, 64, 6, 1, [9, 2, 31], True)]])
def test_segments_in_one_launch_equal_four_kernels_a_round(dtype, d, hidden, V, N, S, lengths, peaked):
    """Whole segments inside one launch, every XCD with utterances of its own: the same bits as the four kernels a round (debug
    bit 16), whose arithmetic and order of sums it keeps, and the same counters; every width of K, ragged tiles of rows,
    columns and utterances (none, fewer than XCDs, more than workgroups), beams on both sides of the workgroup sizes; fp32
    with K of no whole chunks and with gate weights that do not fit the LDS."""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=len(lengths), vocab=V, d=d, hidden=hidden), dtype=dtype)
    cap = 0
    if peaked:
        shape, cap = _peaked(shape, 8.0, 8.0), 5
    model, offsets, enc = build_case(shape, n_utts=len(lengths), lengths=np.array(lengths))
    kw = dict(max_rounds_per_segment=cap) if cap else {}
    seen = []
    for debug in (0, 65536, 131072):
        tbs = make_tbs(shape, model, offsets, N, S, debug=debug, **kw)
        frames = tbs.upload_frames(enc)
        got = [tbs.decode(frames, offsets)]
        _assert_one_launch(tbs, _segments(offsets, S), debug)
        got.append(tbs.decode(frames, offsets))
        assert tbs.path()["fixed_places"] and got[0] == got[1]
        seen.append((got[0], tbs.stats(), tbs.counts()["nodes"]))
        tbs.close()
    assert seen[0] == seen[1] == seen[2]   # (131072: the launch gives up and the batch runs with four kernels a round)
    if len(lengths) < 20:
        _check_decode(shape, model, offsets, enc, N, S, max_rounds=cap)


@pytest.mark.parametrize("debug", [0, 131072])
def test_streams_in_one_launch_a_step(debug):
    """A stream pushed in uneven pieces, utterances starting and ending segments at different steps, gives what the four
    kernels a round give for the whole batch; tries, lists and states are left as those kernels go on from them."""
    N, S = 5, 3
    shape = _peaked(small_bf16_shape(n_utts=11, vocab=120, d=256, hidden=128), 8.0, 8.0)
    model, offsets, enc = build_case(shape, n_utts=11, lengths=np.array([0, 1, 3, 4, 9, 10, 14, 21, 22, 5, 30]))
    want, _ = _gpu_decode(shape, model, offsets, enc, N, S, debug=65536, max_rounds_per_segment=5)
    tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=12, max_rounds_per_segment=5, debug=debug)
    _push_in_pieces(tbs, shape, offsets, enc, lambda u, c: (u + 2 * c) % 5)
    assert tbs.result() == want
    _assert_one_launch(tbs, max(tbs.one_launch()["segments"], _segments(offsets, S)), debug)   # (at least: a step need not be all utterances')
    tbs.close()


@pytest.mark.parametrize("U,piece,offset,debug", [(300, 4, 0, 0), (20, 130, 0, 0), (20, 7, 2, 0), (9, 5, 0, 0), (20, 7, 0, 131072)])
def test_pushes_whose_frames_go_with_the_launch(U, piece, offset, debug):
    """Frames appended inside the launch (two utterances of a workgroup too), or by a kernel in front of it: pieces of more
    than 64 KB, frames that begin off 16 bytes, a launch that gives up.  Every utterance brings another number of frames."""
    import torch
    N, S = 3, 3
    shape = small_bf16_shape(n_utts=U, vocab=40, d=256, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=U, lengths=np.array([piece + 2 + (i * 7) % 11 for i in range(U)]))
    want, _ = _gpu_decode(shape, model, offsets, enc, N, S, debug=65536)
    tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=piece + S, debug=debug)
    tbs.stream_begin(U)
    at, c = offsets[:-1].copy(), 0
    while (at < offsets[1:]).any():
        n = np.minimum([piece - (u + c) % 3 for u in range(U)], offsets[1:] - at)
        rows = tbs.upload_frames(np.concatenate([enc[at[u]:at[u] + n[u]] for u in range(U)]))
        space = torch.empty(rows.numel() + offset, dtype=rows.dtype, device=rows.device)
        space[offset:].copy_(rows.reshape(-1))
        torch.cuda.synchronize()
        at, c = at + n, c + 1
        tbs.push_segment(space[offset:], np.concatenate([[0], np.cumsum(n)]), flush=bool((at == offsets[1:]).all()))
    _assert_one_launch(tbs, max(tbs.one_launch()["segments"], _segments(offsets, S)), debug)
    got = tbs.result()
    tbs.close()
    assert got == want


def test_contexts_that_decode_at_the_same_time():
    """Two threads, each with a context on a stream of its own: whoever finds the other's launch under way takes four kernels a
    round; both get the results they get alone."""
    import threading
    import torch
    N, S = 5, 3
    shape = small_bf16_shape(n_utts=9, vocab=200, d=256, hidden=256)
    model, offsets, enc = build_case(shape, n_utts=9, lengths=np.arange(20, 29))
    want, _ = _gpu_decode(shape, model, offsets, enc, N, S)
    out, streams = [None, None], [torch.cuda.Stream(), torch.cuda.Stream()]
    ctx = []
    for st in streams:
        with torch.cuda.stream(st):
            ctx.append(make_tbs(shape, model, offsets, N, S))
    frames = [t.upload_frames(enc) for t in ctx]
    torch.cuda.synchronize()

    def work(i):
        out[i] = [ctx[i].decode(frames[i], offsets) for _ in range(8)]

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert out[i] is not None and all(g == want for g in out[i])
        ctx[i].close()


def test_codes_of_segments_in_one_launch():
    """Rounds beyond the capacity and a full share of the trie are the same codes as with four kernels a round."""
    from paper_2302_14357_amd.tbs import TbsError
    shape = small_bf16_shape(n_utts=5, vocab=64, d=128, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=5, lengths=np.array([3, 40, 8, 21, 13]))
    for kw in (dict(rounds_capacity=2), dict(max_nodes=60)):
        for debug in (0, 65536):
            tbs = make_tbs(shape, model, offsets, 4, 3, debug=debug, **kw)
            frames = tbs.upload_frames(enc)
            for _ in range(2):
                with pytest.raises(TbsError) as e:
                    tbs.decode(frames, offsets)
                assert e.value.code == -5
            tbs.close()


@pytest.mark.parametrize("d,hidden,V,N,S,lengths,peaked", [
    (128, 128, 96, 4, 7, [0, 2, 7, 12, 23, 31], False), (128, 256, 200, 7, 16, [5, 16, 17, 40], True), (256, 128, 1023, 2, 17, [34, 3, 18], False),
    (384, 128, 500, 5, 33, [33, 70, 1], False), (128, 128, 64, 3, 64, [64, 65, 130, 20], False), (512, 640, 1024, 5, 20, [25] * 9, False),
    (128, 128, 40, 5, 6, [3 + i % 10 for i in range(270)], False), (128, 128, 700, 10, 5, [4 + i % 5 for i in range(140)], False),
    (128, 128, 1000, 5, 3, [2 + i % 5 for i in range(300)], False)])
def test_one_launch_beyond_the_fixed_places(d, hidden, V, N, S, lengths, peaked):
    """Segments of 6 to 64 frames (a wave's rows one to eight, hypotheses spread over the XCD's workgroups, more of them than
    those) and batches too large for the layout with fixed places: what row lists give (debug bit 16), and the oracle."""
    shape = small_bf16_shape(n_utts=len(lengths), vocab=V, d=d, hidden=hidden)
    kw, cap = {}, 0
    if peaked:
        shape, cap = _peaked(shape, 8.0, 8.0), 5
        kw = dict(max_rounds_per_segment=cap)
    elif S > 16:
        kw = dict(rounds_capacity=4 * S)
    model, offsets, enc = build_case(shape, n_utts=len(lengths), lengths=np.array(lengths))
    seen = []
    for debug in (0, 65536, 131072):
        tbs = make_tbs(shape, model, offsets, N, S, debug=debug, **kw)
        got = tbs.decode(tbs.upload_frames(enc), offsets)
        _assert_one_launch(tbs, _segments(offsets, S), debug)
        assert not tbs.path()["fixed_places"]
        seen.append((got, tbs.stats(), tbs.counts()["nodes"]))
        tbs.close()
    for other in seen[1:]:
        for a, b in zip(seen[0][0], other[0]):
            assert [h[0] for h in a] == [h[0] for h in b]
            np.testing.assert_allclose([h[1] for h in a], [h[1] for h in b], rtol=1e-6, atol=1e-5)
        assert seen[0][1:] == other[1:]
    n = min(len(lengths), 6)
    okw = {k: v for k, v in kw.items() if k != "max_rounds_per_segment"}
    _check_decode(shape, model, offsets[:n + 1], enc[:offsets[n]], N, S, max_rounds=cap, **okw)


def test_one_launch_with_a_trie_that_one_list_of_nodes_fits():
    """A trie just large enough for all utterances together, too small for a share of each: decodes of long segments and of
    batches beyond the fixed places run with row lists then, with the same result; nothing that was accepted is refused."""
    N, S = 4, 7
    shape = small_bf16_shape(n_utts=5, vocab=64, d=128, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=5, lengths=np.array([3, 40, 8, 21, 13]))

    def run(**kw):
        try:
            got, _ = _gpu_decode(shape, model, offsets, enc, N, S, **kw)
        except RuntimeError:
            return None
        return [[y for y, _ in u] for u in got]

    want = run()
    lo, hi = 16, 4 * N * (85 + 5 * S) + 16
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if run(max_nodes=mid, debug=65536) is None else (lo, mid)
    assert run(max_nodes=hi) == want
    assert run(max_nodes=lo) is None
    # (one utterance that emits more than its share of a trie of the default size: decoded again with row lists)
    cap = 24
    model["w_out"] = np.zeros_like(model["w_out"])
    model["w_out"][0, :] = 0.5
    model["b_out"] = np.linspace(0.0, 0.3, 64).astype(np.float32)
    model["b_out"][0] = -60.0
    enc = np.full_like(enc, 8.0)
    enc[offsets[1]:offsets[2]] = -64.0
    import dataclasses
    shape = dataclasses.replace(shape, act="relu")
    one, two = (_gpu_decode(shape, model, offsets, enc, 2, 6, max_rounds_per_segment=cap, debug=dbg) for dbg in (0, 65536))
    assert [[h[0] for h in u] for u in one[0]] == [[h[0] for h in u] for u in two[0]]
    assert one[1]["joiner_calls"] == two[1]["joiner_calls"]


@pytest.mark.parametrize("dtype,S", [("bf16", 3), ("f32", 3), ("bf16", 8)])
def test_output_and_projection_weights_may_change_between_decodes(dtype, S):
    """The output matrix and the projection are read when a batch is decoded: a change in place is seen by the next decode."""
    import dataclasses
    import torch
    shape = dataclasses.replace(small_bf16_shape(n_utts=3, vocab=96, d=128, hidden=128), dtype=dtype)
    model, offsets, enc = build_case(shape, lengths=np.array([9, 17, 4]))
    other = make_model(dataclasses.replace(shape, index=8))
    changed = dict(model, w_out=other["w_out"], w_proj=other["w_proj"])
    want, _ = _gpu_decode(shape, changed, offsets, enc, 4, S)
    tbs = make_tbs(shape, model, offsets, 4, S)
    frames = tbs.upload_frames(enc)
    before = tbs.decode(frames, offsets)
    _assert_one_launch(tbs, _segments(offsets, S))
    for name in ("w_out", "w_proj"):
        tbs.t[name].copy_(torch.from_numpy(changed[name]))
    torch.cuda.synchronize()
    after = tbs.decode(frames, offsets)
    tbs.close()
    assert after == want and after != before


@pytest.mark.parametrize("dtype,d,hidden,V,N,S,lengths,peaked", [
    ("bf16", 128, 128, 96, 4, 7, [0, 2, 7, 12, 23, 31], False), ("bf16", 128, 256, 200, 7, 16, [5, 16, 17, 40], True),
    ("bf16", 256, 128, 1023, 2, 17, [34, 3, 18, 24, 26], False), ("bf16", 384, 128, 500, 5, 33, [33, 70, 1, 42], False),
    ("bf16", 128, 128, 64, 3, 64, [64, 65, 130, 20, 73], False), ("bf16", 512, 640, 1024, 5, 20, [9 + i for i in range(64)], False),
    ("bf16", 512, 640, 1000, 5, 8, [9 + i for i in range(64)], True), ("bf16", 128, 128, 40, 5, 6, [3 + i % 10 for i in range(270)], False),
    ("bf16", 128, 128, 700, 10, 5, [4 + i % 5 for i in range(140)], False), ("bf16", 128, 128, 1000, 5, 3, [2 + i % 5 for i in range(300)], True),
    ("bf16", 512, 640, 1024, 10, 5, [4 + i % 5 for i in range(320)], False), ("bf16", 256, 128, 300, 5, 1, [1 + i % 3 for i in range(512)], False),
    ("f32", 64, 64, 32, 4, 3, [2 + i % 5 for i in range(300)], False), ("f32", 128, 256, 500, 10, 5, [4 + i % 4 for i in range(200)], False)])
def test_results_do_not_hang_on_what_the_gpu_is_doing(dtype, d, hidden, V, N, S, lengths, peaked):
    """Where the slot layout does not reach (long segments, large batches), row lists take the place of a launch that gives up
    (debug bit 17) or is not made (bit 16): the same bits, for products of every tile size, and as a stream, which has row lists
    there in any case."""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=len(lengths), vocab=V, d=d, hidden=hidden), dtype=dtype)
    kw = dict(rounds_capacity=4 * S) if S > 16 else {}
    if peaked:
        shape = _peaked(shape, 8.0, 8.0)
        kw = dict(max_rounds_per_segment=5)
    model, offsets, enc = build_case(shape, n_utts=len(lengths), lengths=np.array(lengths))
    seen = []
    for debug in (0, 65536, 131072):
        tbs = make_tbs(shape, model, offsets, N, S, debug=debug, **kw)
        seen.append(tbs.decode(tbs.upload_frames(enc), offsets))
        _assert_one_launch(tbs, _segments(offsets, S), debug)
        tbs.close()
    assert seen[0] == seen[1] == seen[2]
    if S > 5:
        tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=2 * S, **kw)
        _push_in_pieces(tbs, shape, offsets, enc, lambda u, c: 1 + (u + 3 * c) % S)
        assert tbs.result() == seen[0]
        tbs.close()


@pytest.mark.parametrize("dtype,S", [("bf16", 3), ("bf16", 8), ("f32", 3)])
def test_contexts_at_the_same_time_share_the_gpu(dtype, S):
    """Two threads that decode in a loop at widths whose launch takes all of the CUs' LDS: when one is done the other has come
    a third as far or more (it stood still while the launch went to whoever asked first), and both get what they get alone."""
    import dataclasses
    import threading
    import torch
    N, rounds, max_len = 5, 12, 256
    shape = dataclasses.replace(small_bf16_shape(n_utts=16, vocab=1024, d=512, hidden=640), dtype=dtype)
    model, offsets, enc = build_case(shape, n_utts=16, lengths=np.arange(220, 236))
    offsets = np.asarray(offsets, np.int32)
    ctx = []
    for st in [torch.cuda.Stream(), torch.cuda.Stream()]:
        with torch.cuda.stream(st):
            ctx.append(make_tbs(shape, model, offsets, N, S))
    frames = [t.upload_frames(enc) for t in ctx]

    def decode(i):
        ctx[i].U = len(offsets) - 1
        out = ctx[i]._result_arrays(max_len)
        assert ctx[i].decode_raw(frames[i], offsets, *out, max_len) == 0
        return out

    want = decode(0)
    decode(1)
    _assert_one_launch(ctx[0], _segments(offsets, S))
    done, at_end, out, start = [0, 0], [], [None, None], threading.Barrier(2)

    def work(i):
        start.wait()
        for _ in range(rounds):
            out[i] = decode(i)
            done[i] += 1
        at_end.append(min(done))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for t in ctx:
        t.close()
    for got in out:
        assert all(np.array_equal(a, b) for a, b in zip(got, want))
    assert at_end[0] >= rounds // 3, at_end   # (8 to 11 of 12; 0 while it stood still)


def test_a_launch_that_gave_up_is_not_tried_at_every_push():
    """Where the GPU is not free for the launch (debug bit 17) a stream waits for it once in 100 ms, not at every push."""
    import time
    N, S = 3, 3
    shape = small_bf16_shape(n_utts=4, vocab=40, d=256, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=4, lengths=np.full(4, 120))
    want, _ = _gpu_decode(shape, model, offsets, enc, N, S)
    tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=6, debug=131072)
    t0 = time.monotonic()
    _push_in_pieces(tbs, shape, offsets, enc, lambda u, c: 3)   # (40 pushes)
    most = 1 + int((time.monotonic() - t0) / 0.1)
    _assert_one_launch(tbs, 0, 131072)
    assert tbs.one_launch()["gave_up"] <= most and tbs.result() == want
    tbs.close()


@pytest.mark.parametrize("dtype,S,lengths", [("bf16", 1, [4100, 30, 0, 7, 4097, 1, 2, 3, 5000]), ("f32", 1, [4099]), ("bf16", 64, [66 * 1024 // 64 * 64 + 5])])
def test_decodes_of_several_launches(dtype, S, lengths):
    """More segments than one launch takes: what the kernels without it give."""
    import dataclasses
    N = 5
    shape = dataclasses.replace(small_bf16_shape(n_utts=len(lengths), vocab=24, d=128, hidden=128), dtype=dtype)
    model, offsets, enc = build_case(shape, n_utts=len(lengths), lengths=np.array(lengths))
    seen = []
    for debug in (0, 65536):
        tbs = make_tbs(shape, model, offsets, N, S, debug=debug, max_result_len=20000, **(dict(rounds_capacity=4 * S) if S > 16 else {}))
        seen.append((tbs.decode(tbs.upload_frames(enc), offsets, max_len=20000), tbs.stats()))
        _assert_one_launch(tbs, _segments(offsets, S), debug)
        tbs.close()
    assert seen[0] == seen[1]


@pytest.mark.parametrize("S,peaked", [(3, True), (1, False), (5, False)])
def test_streams_that_change_form_between_pushes(S, peaked):
    """Pushes in a launch, with four kernels a round (a timed kernel family is not there in a launch) and back, as where another
    context comes and goes: the stream's result, and its counters, are those of the batch."""
    N = 5
    shape = small_bf16_shape(n_utts=11, vocab=120, d=256, hidden=128)
    kw = {}
    if peaked:
        shape, kw = _peaked(shape, 8.0, 8.0), dict(max_rounds_per_segment=5)
    model, offsets, enc = build_case(shape, n_utts=11, lengths=np.array([0, 1, 3, 4, 9, 10, 14, 21, 22, 5, 30]))
    want, st = _gpu_decode(shape, model, offsets, enc, N, S, debug=65536, **kw)
    steps = None
    for turn in (1000, 1, 2, 3):
        tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=12, **kw)
        push, calls = tbs.push_segment, []

        def one(*a, **k):
            tbs.profile_select(0 if len(calls) // turn % 2 else -1)
            calls.append(0)
            push(*a, **k)

        tbs.push_segment = one
        _push_in_pieces(tbs, shape, offsets, enc, lambda u, c: (u + 2 * c) % 5)
        ran = tbs.one_launch()
        steps = steps or ran["segments"]   # (all of them in a launch)
        assert ran["gave_up"] == 0 and (turn == 1000 or 0 < ran["segments"] < steps)
        assert tbs.result() == want
        assert {k: tbs.stats()[k] for k in ("joiner_calls", "joined_frames", "frames")} == {k: st[k] for k in ("joiner_calls", "joined_frames", "frames")}
        tbs.close()


def test_memory_of_the_launch_ends_with_its_utterances():
    """A context for 1500 utterances takes no more for the launch, which decodes up to 512, than those need (state rows of
    4 x 2 x 33 places of 256 bytes an utterance, input rows of 12 x 256), and batches on both sides of the limit decode."""
    import torch
    N, S = 4, 3
    shape = small_bf16_shape(n_utts=520, vocab=40, d=128, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=520, lengths=np.array([1 + i % 4 for i in range(520)]))
    taken, got = [], []
    for debug in (0, 65536, 0):   # (the first for what a process takes once)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        tbs = make_tbs(shape, model, offsets, N, S, max_utts=1500, debug=debug)
        taken.append(free - torch.cuda.mem_get_info()[0])
        out = []
        for U in (512, 513):
            out.append(tbs.decode(tbs.upload_frames(enc[:offsets[U]]), offsets[:U + 1]))
            assert tbs.one_launch()["segments"] == (2 if debug == 0 and U == 512 else 0)
        got.append(out)
        tbs.close()
    assert got[0] == got[1] == got[2] and got[0][0] == got[0][1][:512]
    assert taken[2] - taken[1] <= 512 * (N * 2 * 33 + N * S) * 256 + (8 << 20), taken


@pytest.mark.parametrize("dtype,N,S,few,many", [("bf16", 5, 20, 128, 129), ("f32", 7, 5, 176, 177)])
def test_large_batches_keep_to_the_other_forms(dtype, N, S, few, many):
    """Batches on both sides of the line up to which the launch is faster: one runs in it and one does not.  (A batch beyond the line
    adds up in the order of its own forms, whoever else is on the GPU: the same hypotheses, scores to the last digits.)"""
    import dataclasses
    shape = dataclasses.replace(small_bf16_shape(n_utts=many, vocab=32, d=128, hidden=128), dtype=dtype)
    model, offsets, enc = build_case(shape, n_utts=many, lengths=np.array([1 + i % 23 for i in range(many)]))
    kw = dict(rounds_capacity=4 * S) if S > 16 else {}
    tbs = make_tbs(shape, model, offsets, N, S, **kw)
    got = []
    for U in (few, many):
        got.append(tbs.decode(tbs.upload_frames(enc[:offsets[U]]), offsets[:U + 1]))
        assert tbs.one_launch()["may"] == (U == few) and (tbs.one_launch()["segments"] > 0) == (U == few)
    tbs.close()
    for a, b in zip(got[0], got[1]):
        assert [h[0] for h in a] == [h[0] for h in b]
        np.testing.assert_allclose([h[1] for h in a], [h[1] for h in b], rtol=1e-6, atol=1e-5)


def _bad_batches(offsets, enc, u, S, act):
    """The frames of a batch with some of utterance u's that are no numbers (or, where the activation makes numbers of those,
    infinite): the last one of its second segment, all of that segment's, all it has."""
    lo, hi = int(offsets[u]), int(offsets[u + 1])
    assert hi - lo > 2 * S
    for a, b in [(lo + 2 * S - 1, lo + 2 * S), (lo + S, lo + 2 * S), (lo, hi)]:
        bad = enc.copy()
        bad[a:b] = math.nan if act == "tanh" else math.inf
        if act == "relu":
            bad[a:b, ::2] = -math.inf
        yield bad


def _check_bad_utterance(got, clean, bad_u, V, N):
    for u, (g, c) in enumerate(zip(got, clean)):
        if u != bad_u:
            assert g == c, u
    assert 1 <= len(got[bad_u]) <= N
    assert len({y for y, _ in got[bad_u]}) == len(got[bad_u])
    assert all(0 < k < V for y, _ in got[bad_u] for k in y)


@pytest.mark.parametrize("dtype,act,d,hidden,layers,V,N,S,debugs", [
    ("bf16", "tanh", 128, 128, 1, 96, 5, 1, (0, 65536, 256)), ("bf16", "tanh", 128, 128, 1, 96, 4, 1, (0, 32768 + 65536, 512 + 256)),
    ("bf16", "tanh", 128, 256, 1, 96, 5, 3, (0, 65536, 131072, 256, 256 + 128)), ("bf16", "relu", 128, 128, 1, 200, 10, 5, (0, 65536, 256)),
    ("bf16", "tanh", 128, 128, 1, 96, 5, 8, (0, 65536)), ("bf16", "relu", 128, 128, 1, 96, 3, 40, (0, 65536)),
    ("f32", "tanh", 64, 64, 1, 40, 5, 3, (0, 65536, 256)), ("bf16", "tanh", 64, 72, 2, 96, 20, 2, (0, 2)),
    ("bf16", "tanh", 64, 64, 3, 2100, 5, 3, (0, 8)), ("bf16", "tanh", 64, 64, 1, 4200, 12, 9, (0,))])
def test_an_utterance_whose_frames_are_no_numbers(dtype, act, d, hidden, layers, V, N, S, debugs):
    """Encoder frames come from the caller and nobody looks at them.  An utterance some of whose are NaN (or infinite) has scores that are
    NaN; it is decoded to an end, the same twice, and the others of the batch give the bits they give without it: whole
    segments in one launch, in four kernels a round and by row lists, every form of the expansion and the select step."""
    import dataclasses
    lengths = np.array([2 * S + 1 + (7 * i) % (2 * S + 5) for i in range(9)])
    shape = dataclasses.replace(small_bf16_shape(n_utts=9, vocab=V, d=d, hidden=hidden, layers=layers), dtype=dtype, act=act)
    model, offsets, enc = build_case(shape, n_utts=9, lengths=lengths)
    kw = dict(rounds_capacity=64 if S > 16 else 0)
    by_form = []
    for debug in debugs:
        tbs = make_tbs(shape, model, offsets, N, S, debug=debug, **kw)
        clean = tbs.decode(tbs.upload_frames(enc), offsets)
        bad_results = []
        for bad in _bad_batches(offsets, enc, 4, S, act):
            frames = tbs.upload_frames(bad)
            got = tbs.decode(frames, offsets)
            _check_bad_utterance(got, clean, 4, V, N)
            assert repr(tbs.decode(frames, offsets)) == repr(got)
            bad_results.append(repr(got[4]))
        tbs.close()
        by_form.append(bad_results)
    if len(debugs) > 1 and debugs[:2] == (0, 65536):   # (these keep the order of sums)
        assert by_form[0] == by_form[1]


@pytest.mark.parametrize("debug", [0, 65536, 256])
def test_a_stream_whose_frames_are_no_numbers(debug):
    """The same pushed in pieces."""
    N, S = 5, 3
    shape = small_bf16_shape(n_utts=9, vocab=120, d=256, hidden=128)
    model, offsets, enc = build_case(shape, n_utts=9, lengths=np.array([7 + 3 * i for i in range(9)]))
    tbs = make_tbs(shape, model, offsets, N, S, stream_buffer_frames=12, debug=debug)
    _push_in_pieces(tbs, shape, offsets, enc, lambda u, c: 1 + (u + 2 * c) % 5)
    clean = tbs.result()
    for bad in _bad_batches(offsets, enc, 4, S, "tanh"):
        _push_in_pieces(tbs, shape, offsets, bad, lambda u, c: 1 + (u + 2 * c) % 5)
        _check_bad_utterance(tbs.result(), clean, 4, 120, N)
    tbs.close()


@pytest.mark.parametrize("dtype,S,debug", [("bf16", 3, 0), ("bf16", 3, 8192), ("bf16", 1, 0), ("f32", 3, 0)])
def test_a_round_without_hypotheses_is_no_error(dtype, S, debug):
    """A caller that drives the steps may make one more round behind the one that made nothing, or one over lists that it has emptied:
    every step has nothing to do and says so, and the next segment begins as if the round had not been."""
    import dataclasses
    from paper_2302_14357_amd import BUF
    N = 4
    shape = dataclasses.replace(small_bf16_shape(n_utts=3, vocab=60), dtype=dtype)
    model, offsets, enc = build_case(shape, n_utts=3, lengths=np.array([2 * S, 2 * S - 1, 0]))
    want = None
    for extra in (0, 2):
        tbs = make_tbs(shape, model, offsets, N, S, debug=debug)
        tbs.begin(tbs.upload_frames(enc), offsets)
        for seg in range(2):
            rows = tbs.segment_begin(seg)
            while rows > 0:
                tbs.joiner_segment()
                tbs.expand()
                live = tbs.select_merge()
                tbs.predictor_step()
                rows = tbs.counts()["rows"]
                assert (rows > 0) == (live > 0)
            for _ in range(extra):
                tbs.joiner_segment()
                tbs.expand()
                assert tbs.select_merge() == 0
                tbs.predictor_step()
                assert tbs.counts()["rows"] == 0
        got = tbs.result()
        want = want or got
        assert got == want
        if extra:
            tbs.debug_write(BUF.A_COUNT, np.zeros(3, np.int32))
            assert tbs.debug_rebuild(0) == 0
            tbs.joiner_segment()
            tbs.expand()
            assert tbs.select_merge() == 0
        tbs.close()


@pytest.mark.parametrize("M,N,K", [(64, 64, 128), (300, 200, 256), (1000, 1025, 640), (2050, 4096, 1024), (37, 100, 72), (700, 513, 520)])
def test_gemm_bf16_kernels_give_the_same_bits(M, N, K):
    """Whichever kernel makes a product without a bias: all add up K in the same order.  (The recurrent products' is chosen for the rows
    that the segment before had.)"""
    import torch
    from paper_2302_14357_amd import gemm_bf16
    rng = np.random.default_rng(M + N + K)
    a, b = _bf16_values(rng, (M, K)).cuda(), _bf16_values(rng, (N, K), 0.1).cuda()
    first = gemm_bf16(a, b, kernel=1)
    for kernel in (0, 2, 3) + ((4,) if K % 128 == 0 else ()):
        assert torch.equal(first, gemm_bf16(a, b, kernel=kernel)), kernel


@pytest.mark.parametrize("U,N,S,d,hidden,layers,V", [(400, 10, 5, 128, 64, 1, 4096), (240, 10, 5, 128, 64, 1, 4096), (400, 10, 5, 64, 64, 1, 4096),
                                                     (130, 8, 3, 64, 64, 2, 300), (60, 6, 7, 72, 72, 1, 96)])
def test_decode_equals_its_steps(U, N, S, d, hidden, layers, V):
    """tbs_decode, whose segments' first rounds may be enqueued for the most rows there can be (here also where that is beyond what tiles
    of a few a CU serve and the rows there are do not reach it), and the same driven step by step: the same bits.
    (Expansion and select step as two kernels throughout: the one for both, which steps do without, adds up a row in another order.)"""
    shape = small_bf16_shape(n_utts=U, vocab=V, d=d, hidden=hidden, layers=layers)
    lengths = np.random.default_rng(U).integers(S, 2 * S + 2, U)
    model, offsets, enc = build_case(shape, n_utts=U, lengths=lengths)
    results = []
    for debug in (128, 128 + 64):   # (64: nothing is enqueued ahead)
        tbs = make_tbs(shape, model, offsets, N, S, debug=debug)
        frames = tbs.upload_frames(enc)
        results.append(tbs.decode(frames, offsets))
        assert not tbs.path()["fixed_places"]
        if len(results) == 1:
            tbs.begin(frames, offsets)
            for seg in range(_segments(offsets, S)):
                rows = tbs.segment_begin(seg)
                while rows > 0:
                    tbs.joiner_segment()
                    tbs.expand()
                    tbs.select_merge()
                    tbs.predictor_step()
                    rows = tbs.counts()["rows"]
            results.append(tbs.result())
        tbs.close()
    for other in results[1:]:
        assert results[0] == other


def test_what_goes_out_ahead_does_not_hang_on_the_batch_before():
    """The recurrent products go out ahead of a round's counts where the same round of the segment before made hypotheses: of this
    batch's segments.  Batches of one segment have none before theirs, so each has as many launches behind any other batch as on
    its own (a batch's last round, which makes nothing, would otherwise have one more behind a batch with more rounds)."""
    from paper_2302_14357_amd import KERNEL
    shape = small_bf16_shape(n_utts=1, vocab=60, hidden=72)   # (three or four rounds a segment)
    N, S = 4, 4
    model, offsets, enc = build_case(shape, n_utts=12, lengths=np.full(12, S))
    tbs = make_tbs(shape, model, offsets, N, S, debug=256)
    frames = [tbs.upload_frames(enc[u * S:(u + 1) * S]) for u in range(12)]
    one = np.array([0, S], np.int32)

    def decode(u):
        tbs.profile_select(KERNEL.GEMM)
        tbs.decode(frames[u], one)
        return tbs.profile_read()["launches"], tbs.stats()["launches"]

    alone = [decode(u) for u in range(12)]
    rounds = [r for _, r in alone]
    most, least = int(np.argmax(rounds)), int(np.argmin(rounds))
    assert rounds[most] > rounds[least]
    fresh = {}
    for u in (most, least):
        tbs.close()
        tbs = make_tbs(shape, model, offsets, N, S, debug=256)
        fresh[u] = decode(u)
    for first in (most, least):
        for then in (most, least):
            decode(first)
            assert decode(then) == fresh[then], (first, then)
    tbs.close()


@pytest.mark.parametrize("kernel", [1, 2, 3, 4])
@pytest.mark.parametrize("M,N,K,lives", [(300, 200, 128, (0, 1, 64, 255, 299)), (9000, 4096, 128, (0, 4097, 8999)), (700, 130, 200, (0, 513))])
def test_gemm_bf16_with_a_row_count_from_device_memory(M, N, K, lives, kernel):
    """Fewer rows than the launch is sized for, down to none and up to several tiles of a persistent workgroup, rows scattered or in
    place: the same bits as a product of those rows, and nothing written beside them."""
    import ctypes
    import torch
    from paper_2302_14357_amd import gemm_bf16, load_library
    if kernel == 4 and K % 128:
        return
    run = load_library().gemm_tile_run
    run.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 4 + [ctypes.c_int] * 3 + [ctypes.c_void_p, ctypes.c_long] + [ctypes.c_void_p] * 2
    rng = np.random.default_rng(M + kernel)
    a, b = _bf16_values(rng, (M, K)).cuda(), _bf16_values(rng, (N, K), 0.1).cuda()
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).cuda()
    ldc = N + 5
    for live in lives:
        where = torch.from_numpy(rng.permutation(M + 3)[:M].astype(np.int32)).cuda() if live % 2 else None
        n, out = torch.tensor([live], dtype=torch.int32, device="cuda"), torch.full((M + 3, ldc), 7.0, device="cuda")
        rc = run(kernel, a.data_ptr(), b.data_ptr(), bias.data_ptr(), out.data_ptr(), M, N, K, where.data_ptr() if where is not None else None, ldc,
                 n.data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        rows = (where if where is not None else torch.arange(M, device="cuda"))[:live].long()
        want = torch.full((M + 3, ldc), 7.0, device="cuda")
        if live:
            want[rows, :N] = gemm_bf16(a[:live].contiguous(), b, bias, kernel=kernel)
        assert torch.equal(out, want), live


@pytest.mark.parametrize("U,N,layers", [(103, 10, 1), (256, 16, 2), (241, 17, 1)])
def test_rows_gathered_by_either_kernel_give_the_same_bits(U, N, layers):
    """The parents' rows of h gathered by the row list kernel, with the products behind it enqueued ahead of the counts, and by a kernel of
    their own: the same rows, and products that add up in the same order whichever kernel makes them."""
    shape = small_bf16_shape(n_utts=U, vocab=96, d=128, hidden=512, layers=layers)
    model, offsets, enc = build_case(shape, n_utts=U, lengths=np.random.default_rng(U).integers(0, 9, U))
    one, st1 = _gpu_decode(shape, model, offsets, enc, N, 2, debug=256)
    two, st2 = _gpu_decode(shape, model, offsets, enc, N, 2, debug=256 | 32)
    assert not st1["path"]["fixed_places"]
    assert one == two and st1["joiner_calls"] == st2["joiner_calls"]


@pytest.mark.parametrize("M,N,K", [(6000, 2560, 512), (12000, 2560, 256), (7680, 4096, 256), (4500, 4096, 320), (2560, 2560, 192)])
def test_gemm_bf16_by_size_keeps_the_bits_of_the_tiles(M, N, K):
    """Up to 768 tiles of 256 x 256 a product is made by tiles chosen for it or by the persistent kernel, whichever is the faster: with
    the bias in the same place."""
    import ctypes
    import torch
    from paper_2302_14357_amd import gemm_bf16, load_library
    run = load_library().gemm_tile_run
    run.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 4 + [ctypes.c_int] * 3 + [ctypes.c_void_p, ctypes.c_long] + [ctypes.c_void_p] * 2
    rng = np.random.default_rng(M)
    a, b = _bf16_values(rng, (M, K)).cuda(), _bf16_values(rng, (N, K), 0.1).cuda()
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).cuda()
    out = torch.empty(M, N, device="cuda")
    assert run(442, a.data_ptr(), b.data_ptr(), bias.data_ptr(), out.data_ptr(), M, N, K, None, N, None, torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(gemm_bf16(a, b, bias, kernel=0), out)
