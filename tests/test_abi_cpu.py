"""CPU-side checks of the C-ABI library: it loads, exports every symbol the
header declares, and rejects bad configurations before touching a GPU."""

import ctypes as C
import math
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _lib():
    from paper_2302_14357_amd import tbs
    return tbs.load_library(), tbs


def test_library_exports_every_declared_symbol():
    L, tbs = _lib()
    header = open(os.path.join(ROOT, "include", "tbs.h")).read()
    declared = set(re.findall(r"\b(tbs_[a-z0-9_]+)\s*\(", header))
    assert declared, "no declarations found"
    assert declared == set(tbs.EXPORTED_SYMBOLS)
    for name in declared:
        assert hasattr(L, name), name


def test_strerror_and_invalid_configs():
    L, tbs = _lib()
    assert L.tbs_strerror(0) == b"ok"
    assert b"order" in L.tbs_strerror(-2)
    cfg = tbs._Config()
    w = tbs._Weights()
    ctx = C.c_void_p()
    assert L.tbs_init(None, None, None) == -1
    # all-zero configuration
    assert L.tbs_init(C.byref(cfg), C.byref(w), C.byref(ctx)) == -1
    good = dict(d_joint=64, vocab=32, blank_id=0, beam_n=2, seg_s=3, max_utts=1, max_frames_total=50,
                pred_layers=1, pred_hidden=64, pred_embed=64, act=0, dtype=0)
    for bad in (dict(beam_n=0), dict(beam_n=33), dict(seg_s=0), dict(vocab=1), dict(blank_id=32),
                dict(pred_layers=5), dict(dtype=2), dict(act=3), dict(max_utts=0), dict(dtype=1, d_joint=60),
                dict(stream_buffer_frames=2), dict(stream_buffer_frames=-1)):
        c = tbs._Config(**{**good, **bad})
        assert L.tbs_init(C.byref(c), C.byref(w), C.byref(ctx)) == -1, bad
        assert not ctx.value
    # good shape but null weight pointers
    c = tbs._Config(**good)
    assert L.tbs_init(C.byref(c), C.byref(w), C.byref(ctx)) == -1
    # null context on every entry point
    assert L.tbs_joiner_segment(None) == -1 and L.tbs_expand(None) == -1
    assert L.tbs_select_merge(None, None) == -1 and L.tbs_predictor_step(None) == -1
    assert L.tbs_gemm_bf16(None, None, None, None, 1, 1, 8, 0, None) == -1
    assert L.tbs_path(None) == -1 and L.tbs_one_launch(None, None, None) == -1
    assert L.tbs_stream_begin(None, 1) == -1 and L.tbs_push_segment(None, None, None, 0) == -1
    L.tbs_free(None)


@pytest.mark.parametrize("V,S,form", [
    (1024, 3, "reg 1 3"), (1024, 4, "reg 1 5"), (1024, 5, "reg 1 5"),
    (1024, 6, "long 4 2"), (1024, 7, "long 4 2"), (1024, 8, "long 4 2"), (256, 6, "long 1 2"), (260, 8, "long 2 2"), (2, 8, "long 1 2"),
    (256, 32, "long 1 2"), (257, 33, "long 2 4"), (512, 64, "long 2 4"), (513, 32, "long 4 2"), (1023, 64, "long 4 4"),
    (1024, 65, "two pass"), (1025, 3, "reg 2 8"), (1025, 8, "reg 2 8"), (2048, 8, "reg 2 8"), (1025, 9, "two pass"),
    (2049, 3, "reg 4 3"), (4096, 5, "reg 4 5"), (2049, 6, "two pass"), (4097, 1, "two pass")])
def test_expansion_kernel_by_size(V, S, form):
    """Which kernel expands a call, on both sides of every line: four waves with the logits in registers to 5 frames (wider
    vocabularies: to 8), k_expand_long from 6 to 64 frames of vocabularies up to 1024, two passes beyond."""
    L, _ = _lib()
    code = L.expand_form((V + 3) // 4 * 4, S)
    kind, _, args = form.partition(" ")
    if kind == "two":
        assert code == 0
    else:
        a, b = (int(x) for x in args.split())
        assert code == (100 * a + b if kind == "reg" else 1000 + 10 * a + b)


@pytest.mark.parametrize("N,frames,form", [(1, 1, 0), (8, 8, 0), (11, 8, 0), (12, 1, 1), (12, 8, 1), (16, 3, 1), (32, 8, 1),
                                           (1, 9, 2), (11, 9, 2), (32, 64, 2), (1, 65, 1), (32, 128, 1)])
def test_distributions_of_new_hypotheses_by_size(N, frames, form):
    """How the select step makes them, on both sides of every line: ahead of the ranking (0) to 8 frames and 128
    candidates, by (hypothesis, frame) pairs (2) from 9 to 64 frames only, by a lane per hypothesis (1) otherwise."""
    L, _ = _lib()
    assert L.select_dist_form(N * N, frames) == form


@pytest.mark.parametrize("inside,lds,may", [(1, 160 * 1024, 1), (2, 160 * 1024, 0), (8, 81921, 0), (2, 81920, 1), (8, 20000, 1)])
def test_when_a_call_may_take_every_cu(inside, lds, may):
    """A launch over whole segments where no other call runs rounds on the GPU, or where it leaves those half of every CU's LDS."""
    L, _ = _lib()
    assert L.xcd_may_launch(inside, lds) == may


@pytest.mark.parametrize("utts,S,segments", [(1, 1, 4096), (1, 16, 4096), (8, 2, 4096), (1, 17, 3855), (8, 3, 2730), (25, 3, 873), (64, 64, 16)])
def test_segments_of_a_launch(utts, S, segments):
    """A launch holds the GPU, so its work is bounded: 4096 segments, 65536 frames of an XCD's utterances."""
    L, _ = _lib()
    assert L.xcd_launch_segments(utts, S) == segments


@pytest.mark.parametrize("f32,stay,N,S,most", [
    (0, 1, 11, 5, 64), (0, 1, 1, 1, 64), (0, 1, 5, 6, 37), (0, 1, 7, 8, 20), (0, 1, 5, 9, 24), (0, 1, 7, 16, 17), (0, 1, 5, 17, 16), (0, 1, 5, 32, 16),
    (0, 1, 5, 33, 8), (0, 1, 1, 64, 40), (1, 0, 5, 3, 16), (1, 0, 7, 1, 22), (1, 0, 2, 5, 24), (1, 0, 8, 1, 25), (1, 0, 10, 5, 9),
    (1, 1, 5, 5, 32), (1, 1, 2, 1, 64), (1, 1, 8, 5, 35), (1, 1, 11, 5, 25)])
def test_batches_the_launch_is_faster_for(f32, stay, N, S, most):
    """Utterances an XCD up to which whole segments run in one launch: bf16 of up to 5 frames all (64 are its limit anyway),
    longer segments by hypotheses, fp32 by rows, fewer where the gates' weights do not stay in LDS."""
    L, _ = _lib()
    assert [u for u in range(1, 65) if L.xcd_pays(f32, stay, N, S, u)] == list(range(1, most + 1))


def test_binding_has_no_oracle_or_cpu_path():
    """The product package must not import the oracle."""
    import paper_2302_14357_amd
    pkg = os.path.dirname(paper_2302_14357_amd.__file__)
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "import oracle" not in text and "from oracle" not in text and "liborc" not in text, f


def _barrier_runs(read, groups, live, ahead, behind):
    """All interleavings of `groups` workgroups on one XCD that run rounds of barriers: `ahead` of them, the one that ends the
    round and carries live[round][workgroup], `behind` more; a round whose sum is 0 is the last.  read(word, due, seen, ends):
    what the kernel makes of the word.  Yields what each workgroup got, by round, at every end of a run."""
    per = ahead + 1 + behind
    # a workgroup: barriers passed, has it arrived at the coming one, sum seen, sums by round (or None: it has left)
    first = (0, 0, tuple((0, False, 0, ()) for _ in range(groups)))
    stack, known, ends = [first], {first}, set()
    while stack:
        low, high, wgs = stack.pop()
        moved = False
        for i, (passed, there, seen, sums) in enumerate(wgs):
            rnd, step = divmod(passed, per)
            if rnd == len(live) or (sums and sums[-1] == 0):
                continue
            if not there:
                add = live[rnd][i] if step == ahead else 0
                after = (low + 1, (high + add) & 0xffffffff, (passed, True, seen, sums))
            else:
                got = read(low | high << 32, groups * (passed + 1), seen, step == ahead)
                if got == -2:
                    continue
                after = (low, high, (passed + 1, False, (seen + got) & 0xffffffff if got > 0 else seen,
                                     sums + (got,) if step == ahead else sums))
            moved = True
            state = (after[0], after[1], wgs[:i] + (after[2],) + wgs[i + 1:])
            if state not in known:
                known.add(state)
                stack.append(state)
        if not moved:
            ends.add(tuple(w[3] for w in wgs))
    return ends


@pytest.mark.parametrize("ahead,behind", [(1, 2), (2, 2), (1, 1)])
@pytest.mark.parametrize("live", [[(5, 0), (0, 0)], [(5, 3), (2, 0), (0, 0)], [(5 + (1 << 20), 0, 3), (0, 0, 0)], [(0, 7, 0), (0, 4, 0), (0, 0, 0)]])
def test_barrier_of_an_xcd_in_every_order(ahead, behind, live):
    """Every workgroup of an XCD gets every round's sum, whoever is late to look at the word (the barrier of the joiner, or of the
    joiner and a long segment's expansion, in front of the round's; the predictor's behind it)."""
    L, _ = _lib()
    L.xcd_barrier_reads.argtypes = [C.c_uint64, C.c_uint32, C.c_uint32, C.c_int]
    groups = len(live[0])
    want = {tuple(tuple(sum(r) for r in live) for _ in range(groups))}
    assert _barrier_runs(L.xcd_barrier_reads, groups, live, ahead, behind) == want
    # (the model sees the mistake it is here for: a sum taken at every barrier)
    assert _barrier_runs(lambda w, due, seen, ends: L.xcd_barrier_reads(w, due, seen, 1), groups, live, ahead, behind) != want


def _rank_lists():
    """Lists of scores as a call with frames that are no numbers makes them, among others."""
    nan, inf = math.nan, math.inf
    rng = np.random.default_rng(5)
    lists = [[nan] * 5, [nan], [-1.0, nan, -3.0, nan, -2.0], [nan, nan, -5.0, -1.0, -1.0], [-inf] * 4, [-inf, nan, -inf], [-2.0] * 6,
             [inf, nan, -inf, inf, 0.0], [-4.0, -1.0, -1.0, -9.0]]
    for n in (16, 17, 32, 33, 64, 85, 320):
        v = rng.integers(-6, 0, n).astype(float)
        v[rng.random(n) < 0.3] = nan
        v[rng.random(n) < 0.1] = -inf
        lists.append(v.tolist())
    return lists


@pytest.mark.parametrize("parts", [1, 2, 4])
def test_ranks_of_scores_that_are_no_numbers(parts):
    """Every entry of a list B has a rank of its own, whatever the scores are: larger first, equal ones by place, NaN behind all.  Who makes the
    next segment's list reads the entry of every rank below the list's length; with NaN that beats nothing and that nothing beats,
    the order of candidate lists, whose NaN mark places without a candidate, some ranks have several entries and others none."""
    L, _ = _lib()
    L.rank_of_entry.argtypes = [C.c_void_p] + [C.c_int] * 4
    holes = False
    for values in _rank_lists():
        v = np.array(values, np.float64)
        n = len(v)
        got = [L.rank_of_entry(v.ctypes.data, n, parts, 0, i) for i in range(n)]
        order = sorted(range(n), key=lambda i: (math.isnan(v[i]), 0.0 if math.isnan(v[i]) else -v[i], i))
        assert [order.index(i) for i in range(n)] == got, values
        cands = [L.rank_of_entry(v.ctypes.data, n, parts, 1, i) for i in range(n)]
        assert [r for r, x in zip(cands, v) if x == x] == [r for r, x in zip(got, v) if x == x]   # (numbers have the same ranks)
        holes = holes or sorted(cands) != list(range(n))
    assert holes   # (the lists see the mistake they are here for)
