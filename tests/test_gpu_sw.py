"""Parity of the HIP Smith-Waterman path with the CPU oracle (Section IV-E).

Every record field is compared element by element; all of it is integer work,
so the bar is bit-exact.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FIELDS = ("score", "beg_a", "end_a", "beg_b", "end_b", "matches", "columns", "seed_used", "passed", "swapped", "cells")


def _to_dev(x, dev, dtype=None):
    import torch

    a = np.ascontiguousarray(x)
    if a.dtype == np.uint32:
        a = a.view(np.int32)
    return torch.from_numpy(a).to(dev)


def _gpu_records(dev, s, lo, hi, s1=None, s2=None, tuning=None, **params):
    import paper_2009_14467_amd as P

    ctx = P.Context(P.Params(**params))
    if tuning:
        ctx.set_tuning(**tuning)
    out = ctx.align_pairs(
        _to_dev(s.residues, dev), _to_dev(s.offsets, dev), _to_dev(lo, dev), _to_dev(hi, dev),
        None if s1 is None else _to_dev(s1, dev), None if s2 is None else _to_dev(s2, dev),
    )
    return P.records_to_numpy(out)


def _compare(got, want, fields=FIELDS, mask=None):
    assert got.shape == want.shape
    for f in fields:
        g, w = got[f], want[f]
        if mask is not None:
            g, w = g[mask], w[mask]
        bad = np.nonzero(g != w)[0]
        assert bad.size == 0, f"{f}: {bad.size} mismatches, first at {bad[:5]}: got {g[bad[:5]]} want {w[bad[:5]]}"


@pytest.fixture(scope="module")
def tiny(orc):
    from synth import workload

    s = workload("tiny")
    codes = orc.encode(s.residues)
    cand = orc.candidates(codes, s.offsets, 6, ck_min=1)
    want = orc.align_pairs(codes, s.offsets, cand["lo"], cand["hi"], mode="sw")
    return s, cand, want


def test_sw_full_records_tiny(gpu, tiny):
    s, cand, want = tiny
    got = _gpu_records(gpu, s, cand["lo"], cand["hi"], full_records=True)
    _compare(got, want)


def test_sw_fast_records_tiny(gpu, tiny):
    s, cand, want = tiny
    got = _gpu_records(gpu, s, cand["lo"], cand["hi"], full_records=False)
    _compare(got, want, ("score", "end_a", "end_b", "passed", "swapped", "cells"))
    _compare(got, want, FIELDS, mask=want["passed"] == 1)


def test_sw_reversed_pair_order(gpu, tiny):
    """(j, i) gives the same alignment as (i, j): orientation is by length."""
    s, cand, want = tiny
    got = _gpu_records(gpu, s, cand["hi"], cand["lo"], full_records=True)
    w2 = want.copy()
    # same rows/columns unless the lengths tie, where the first of the pair is a
    L = np.diff(s.offsets)
    tie = L[cand["lo"]] == L[cand["hi"]]
    _compare(got[~tie], w2[~tie], tuple(f for f in FIELDS if f != "swapped"))
    assert (got["swapped"][~tie] == 1 - w2["swapped"][~tie]).all()


def test_sw_multi_strip_long_pairs(gpu, orc):
    """Rows beyond 512 cross strips through the global boundary buffer."""
    from synth import make_family_set

    s = make_family_set(n_families=4, family_size=4, mean_len=900, min_len=500, max_len=1800, divergence=0.3,
                        stream=91)
    codes = orc.encode(s.residues)
    n = s.n
    lo, hi = np.triu_indices(n, 1)
    lo = lo.astype(np.uint32)
    hi = hi.astype(np.uint32)
    want = orc.align_pairs(codes, s.offsets, lo, hi, mode="sw")
    got = _gpu_records(gpu, s, lo, hi, full_records=True)
    assert (want["end_a"] >= 512).any()
    _compare(got, want)


def test_sw_edge_cases(gpu, orc):
    from synth.families import FamilySet

    seqs = [b"", b"W", b"WW", b"A", b"WWWWWWWWWW", b"WWWWWGWWWWW", b"PPP", b"X*BZ", b"A" * 700, b"A" * 700 + b"W"]
    lens = np.array([len(x) for x in seqs])
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    s = FamilySet(np.frombuffer(b"".join(seqs), np.uint8).copy(), off, np.zeros(len(seqs), np.int32), {})
    codes = orc.encode(s.residues)
    lo, hi = np.triu_indices(len(seqs), 1)
    lo = lo.astype(np.uint32)
    hi = hi.astype(np.uint32)
    want = orc.align_pairs(codes, s.offsets, lo, hi, mode="sw")
    got = _gpu_records(gpu, s, lo, hi, full_records=True)
    _compare(got, want)


def test_sw_rejects_bad_input(gpu):
    import paper_2009_14467_amd as P
    from synth.families import FamilySet

    res = np.frombuffer(b"ACDEFJKL", np.uint8).copy()
    off = np.array([0, 4, 8], np.int64)
    s = FamilySet(res, off, np.zeros(2, np.int32), {})
    with pytest.raises(P.PastisError, match="BAD_RESIDUE"):
        _gpu_records(gpu, s, np.array([0], np.uint32), np.array([1], np.uint32))
    s = FamilySet(np.frombuffer(b"ACDEFGKL", np.uint8).copy(), off, np.zeros(2, np.int32), {})
    with pytest.raises(P.PastisError, match="INVAL"):
        _gpu_records(gpu, s, np.array([0], np.uint32), np.array([2], np.uint32))
    with pytest.raises(P.PastisError, match="INVAL"):
        _gpu_records(gpu, s, np.array([1], np.uint32), np.array([1], np.uint32))


def test_sw_every_length_bin(gpu, orc):
    """One pair per side of every bin boundary (64 R rows in one strip; 2, 3
    and 4 strips of 64 R rows, R = 5..8), against the oracle."""
    from synth.families import FamilySet

    rng = np.random.default_rng(5)
    lens = [1, 64, 65, 128, 129, 448, 449, 512, 513, 640, 641, 768, 769, 896, 897, 1024, 1025, 1152, 1153, 1344,
            1345, 1536, 1537, 1792, 2048, 2049, 2500]
    seqs = []
    for L in lens:
        a = rng.integers(0, 20, L)
        b = a.copy()
        sub = rng.random(L) < 0.25
        b[sub] = rng.integers(0, 20, int(sub.sum()))
        b = np.concatenate([rng.integers(0, 20, 7), b, rng.integers(0, 20, 11)])
        seqs += [a, b]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    res = np.concatenate([letters[x] for x in seqs]).astype(np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(res, off, np.zeros(len(seqs), np.int32), {})
    codes = orc.encode(s.residues)
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    hi = lo + 1
    want = orc.align_pairs(codes, s.offsets, lo, hi, mode="sw")
    for full in (True, False):
        got = _gpu_records(gpu, s, lo, hi, full_records=full)
        if full:
            _compare(got, want)
        else:
            _compare(got, want, ("score", "end_a", "end_b", "passed", "swapped", "cells"))


def _check16(got, want):
    """16-bit pass 1: score, end row and the cut are exact for every pair; the
    end column and statistics exist where the statistics pass ran, and every
    pair without them fails the cut."""
    _compare(got, want, ("score", "end_a", "passed", "swapped", "cells"))
    have = got["beg_a"] >= 0
    assert (want["passed"][~have] == 0).all()
    _compare(got, want, ("beg_a", "beg_b", "matches", "columns"), mask=have)
    _compare(got, want, ("end_b",), mask=got["end_b"] != -1)
    assert (got["end_b"][have] >= 0).all()
    return have


def test_sw16_records_tiny(gpu, tiny):
    s, cand, want = tiny
    got = _gpu_records(gpu, s, cand["lo"], cand["hi"], score_width=16)
    have = _check16(got, want)
    assert have.sum() >= (want["passed"] == 1).sum() > 0


@pytest.mark.parametrize("narrow", [0, 4])
def test_sw16_every_one_strip_bin_and_odd_counts(gpu, orc, narrow):
    """Rows 1..1024 (one-strip bins R = 1..16) with odd pair counts per bin,
    so the last wave of a bin carries one pair, and several pairs sharing
    their shorter sequence (the 16-bit pass pairs those in one wave).  Bins
    of up to 8 rows per lane run in two rows classes (up to 64 R - 32 rows,
    and more): both sides of every class boundary are here, in strips of 32
    lanes (narrow 0) and, up to 4 rows per lane, of 16 (narrow 4)."""
    from synth.families import FamilySet

    rng = np.random.default_rng(8)
    lens = [1, 2, 63, 64, 65, 100, 128, 129, 191, 192, 193, 255, 256, 257, 320, 321, 383, 384, 385, 448, 449, 511,
            512, 513, 640, 641, 768, 769, 896, 897, 1023, 1024]
    lens += [64 * R - 32 + d for R in range(1, 9) for d in (0, 1)]
    seqs = []
    for L in lens:
        a = rng.integers(0, 20, L)
        b = a.copy()
        sub = rng.random(L) < 0.3
        b[sub] = rng.integers(0, 20, int(sub.sum()))
        b = np.concatenate([rng.integers(0, 20, int(rng.integers(0, 40))), b, rng.integers(0, 20, 5)])
        seqs += [a, b]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    res = np.concatenate([letters[x] for x in seqs]).astype(np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(res, off, np.zeros(len(seqs), np.int32), {})
    codes = orc.encode(s.residues)
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    hi = lo + 1
    # plus every cross pair among the first 16 sequences: many pairs per bin
    a, b = np.triu_indices(16, 1)
    lo = np.concatenate([lo, a.astype(np.uint32)])
    hi = np.concatenate([hi, b.astype(np.uint32)])
    want = orc.align_pairs(codes, s.offsets, lo, hi, mode="sw")
    tuning = dict(sw16_max_rows=16, sw16_narrow_rows=narrow)
    got = _gpu_records(gpu, s, lo, hi, tuning=tuning, score_width=16)
    _check16(got, want)


def test_sw16_multi_strip_bins(gpu, orc):
    """Rows 1025..2978 run in 16-bit lanes over strips of 64 R rows (R = 9..16)
    with the boundary row passed through a per-wave buffer; 2979 rows and more
    stay in 32 bits.  Identical runs of W (11 per row) put the score at the
    16-bit limit: 11 * 2978 = 32758 in 16 bits, 32769 in 32."""
    from synth.families import FamilySet

    rng = np.random.default_rng(9)
    lens = [1025, 1100, 1152, 1153, 1344, 1345, 1536, 1537, 1792, 2048, 2049, 2500, 2977, 2978, 2979, 3100]
    seqs = []
    for L in lens:
        a = rng.integers(0, 20, L)
        b = a.copy()
        sub = rng.random(L) < 0.3
        b[sub] = rng.integers(0, 20, int(sub.sum()))
        b = np.concatenate([rng.integers(0, 20, int(rng.integers(0, 40))), b, rng.integers(0, 20, 5)])
        seqs += [a, b]
    w = np.full(2978, 17)  # W
    seqs += [w, w.copy(), np.full(2979, 17), np.full(2979, 17)]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    res = np.concatenate([letters[x] for x in seqs]).astype(np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(res, off, np.zeros(len(seqs), np.int32), {})
    codes = orc.encode(s.residues)
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    hi = lo + 1
    # several pairs sharing their shorter sequence (1025 rows), one wave apart
    a = np.zeros(9, np.uint32)
    lo = np.concatenate([lo, a])
    hi = np.concatenate([hi, np.arange(3, 30, 3, dtype=np.uint32)])
    want = orc.align_pairs(codes, s.offsets, lo, hi, mode="sw")
    assert want["score"][len(lens)] == 11 * 2978 and want["score"][len(lens) + 1] == 11 * 2979
    got = _gpu_records(gpu, s, lo, hi, score_width=16)
    _check16(got, want)
    _compare(_gpu_records(gpu, s, lo, hi, full_records=True, score_width=16), want)


def test_intra_pair_mode(gpu, orc):
    """One workgroup per pair (strips pipelined across four waves) for
    sequences a over 2,978 rows, and for every multi-strip pair once 16-bit
    lanes are off: 1 to 20 strips, pairs sharing sequences, against the oracle."""
    from synth.families import FamilySet

    rng = np.random.default_rng(13)
    lens = [1100, 2500, 2979, 3100, 4100, 5000, 9000, 20000]
    seqs = []
    for L in lens:
        a = rng.integers(0, 20, L)
        b = a.copy()
        sub = rng.random(L) < 0.25
        b[sub] = rng.integers(0, 20, int(sub.sum()))
        b = np.concatenate([rng.integers(0, 20, int(rng.integers(0, 60))), b, rng.integers(0, 20, 9)])
        seqs += [a, b]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    res = np.concatenate([letters[x] for x in seqs]).astype(np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(res, off, np.zeros(len(seqs), np.int32), {})
    codes = orc.encode(s.residues)
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    hi = lo + 1
    # unrelated pairs and pairs sharing their shorter sequence
    lo = np.concatenate([lo, np.array([4, 4, 6, 8, 10], np.uint32)])
    hi = np.concatenate([hi, np.array([9, 13, 11, 15, 13], np.uint32)])
    want = orc.align_pairs(codes, s.offsets, lo, hi, mode="sw")
    intra = dict(sw_intra_pair=1)
    _compare(_gpu_records(gpu, s, lo, hi, tuning=intra, full_records=True), want)
    _compare(_gpu_records(gpu, s, lo, hi, tuning=intra), want, ("score", "end_a", "end_b", "passed", "swapped", "cells"))
    _check16(_gpu_records(gpu, s, lo, hi, tuning=intra, score_width=16), want)


def test_search_same_edges_in_16_and_32_bits(gpu):
    import paper_2009_14467_amd as P
    from synth import workload

    s = workload("tiny", n_families=15)
    res, off = _to_dev(s.residues, gpu), _to_dev(s.offsets, gpu)
    e16 = P.Context(P.Params(k=6, ck_min=1, score_width=16)).search(res, off)
    e32 = P.Context(P.Params(k=6, ck_min=1, score_width=32)).search(res, off)
    assert e16.size == e32.size > 0
    assert e16.tobytes() == e32.tobytes()


def test_longest_pairs_sw_and_xd(gpu, orc):
    """Pairs of 20,000-30,000 residues (the heavy tail's range): many strips
    of 1024 rows, scores far beyond 16 bits, the start bound skipped for
    rectangles taller than its packing allows; SW and XD against the oracle."""
    from synth.families import FamilySet

    rng = np.random.default_rng(12)
    anc = rng.integers(0, 20, 30000)
    a = anc.copy()
    sub = rng.random(a.size) < 0.2
    a[sub] = rng.integers(0, 20, int(sub.sum()))
    b = np.concatenate([anc[:12000], rng.integers(0, 20, 40), anc[12000:29000]])
    c = rng.integers(0, 20, 20000)
    seqs = [a, b, c]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    res = np.concatenate([letters[x] for x in seqs]).astype(np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(res, off, np.zeros(len(seqs), np.int32), {})
    codes = orc.encode(s.residues)
    lo = np.array([0, 0, 1], np.uint32)
    hi = np.array([1, 2, 2], np.uint32)
    want = orc.align_pairs(codes, s.offsets, lo, hi, mode="sw")
    assert want["score"][0] > 1 << 16 and want["passed"][0] == 1
    _compare(_gpu_records(gpu, s, lo, hi, full_records=True), want)
    _compare(_gpu_records(gpu, s, lo, hi), want, ("score", "end_a", "end_b", "passed", "swapped", "cells"))
    p = orc.pair_counts(codes, s.offsets, lo, hi, 6)
    wx = orc.align_pairs(codes, s.offsets, lo, hi, p["seed1"], p["seed2"], mode="xd", k=6)
    gx = _gpu_records(gpu, s, lo, hi, p["seed1"], p["seed2"], align_mode="xd", full_records=True)
    _compare(gx, wx)


def test_rejects_sequences_beyond_u16_positions(gpu):
    import paper_2009_14467_amd as P
    from synth.families import FamilySet

    res = np.full(65536 + 10, ord("A"), np.uint8)
    off = np.array([0, 65536, 65546], np.int64)
    s = FamilySet(res, off, np.zeros(2, np.int32), {})
    with pytest.raises(P.PastisError):
        _gpu_records(gpu, s, np.array([0], np.uint32), np.array([1], np.uint32))
    ctx = P.Context(P.Params())
    with pytest.raises(P.PastisError):
        ctx.search(_to_dev(s.residues, gpu), _to_dev(s.offsets, gpu))


@pytest.mark.parametrize("go,ge", [(5, 2), (250, 10), (2, 1), (240, 4)])
def test_sw_other_gap_costs(gpu, orc, tiny, go, ge):
    """Gap costs away from 11/1: the 16-bit profile holds s + o + e in a byte,
    so o + e above 244 (and below 4) must run in 32-bit lanes; every width and
    record mode still matches the oracle, and so do the search's edges."""
    import paper_2009_14467_amd as P

    s, cand, _ = tiny
    codes = orc.encode(s.residues)
    want = orc.align_pairs(codes, s.offsets, cand["lo"], cand["hi"], mode="sw", gap_open=go, gap_extend=ge)
    gaps = dict(gap_open=go, gap_extend=ge)
    _compare(_gpu_records(gpu, s, cand["lo"], cand["hi"], full_records=True, **gaps), want)
    for width in (0, 16, 32):
        _check16(_gpu_records(gpu, s, cand["lo"], cand["hi"], score_width=width, **gaps), want)
    res, off = _to_dev(s.residues, gpu), _to_dev(s.offsets, gpu)
    want_e = orc.search(s.residues, s.offsets, k=6, ck_min=1, mode="sw", **gaps)
    for width in (0, 16):
        got_e = P.Context(P.Params(k=6, ck_min=1, score_width=width, **gaps)).search(res, off)
        assert got_e.size == want_e.size and got_e.tobytes() == want_e.tobytes()


@pytest.mark.parametrize("copies", [1, 80])
@pytest.mark.parametrize("params", [dict(full_records=True), dict(score_width=16), dict(full_records=True, gap_open=5,
                                                                                        gap_extend=2)])
def test_sw_traced_statistics(gpu, orc, params, copies):
    """The traceback's edges: rows at both sides of its fetches and of a lane's,
    a strip's and a rows class's end, long gaps either way (walks that leave a
    fetch sideways), alignments that start or end inside the sequences, columns
    at both sides of the direction buffers' limits (2048 for one strip, 4096 for
    several: longer pairs take the statistics kernels), one strip and several;
    as one call of few pairs (two to a wave over 64 lanes) and, with copies, of
    more than 8,192 (strips of 16 and 32 lanes)."""
    from synth.families import FamilySet

    rng = np.random.default_rng(17)

    def related(L, pre, post, gaps):
        a = rng.integers(0, 20, L)
        b = a.copy()
        sub = rng.random(L) < 0.2
        b[sub] = rng.integers(0, 20, int(sub.sum()))
        for at, g in gaps:  # g > 0: residues inserted into b, g < 0: removed from it
            at = int(at * b.size)
            b = np.concatenate([b[:at], rng.integers(0, 20, g), b[at:]]) if g > 0 else np.delete(
                b, slice(at, at - g))
        return [a, np.concatenate([rng.integers(0, 20, pre), b, rng.integers(0, 20, post)])]

    pairs = []
    for L in (1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 161, 224, 225, 256, 257, 353,
              480, 481, 512, 513, 640, 769, 1023, 1024, 1025, 1537, 2049):
        pairs.append(related(L, int(rng.integers(0, 40)), int(rng.integers(0, 40)), []))
    for L in (90, 200, 300, 500, 700, 1000, 1300):  # long gaps: both ways, single residues, several
        pairs.append(related(L, 3, 0, [(0.5, 40)]))
        pairs.append(related(L, 0, 9, [(0.5, -25)]))
        pairs.append(related(L, 0, 0, [(0.3, 1), (0.5, -1), (0.7, 17), (0.8, -9)]))
    for total in (2047, 2048, 2049):
        pairs.append(related(300, total - 300 - 50, 50, []))
    for total in (4095, 4096, 4097):
        pairs.append(related(1100, total - 1100 - 50, 50, []))
    for _ in range(40):  # unrelated: short local alignments anywhere
        pairs.append([rng.integers(0, 20, int(rng.integers(20, 600))), rng.integers(0, 20, int(rng.integers(20, 900)))])
    seqs = [x for p in pairs for x in p]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(np.concatenate([letters[x] for x in seqs]).astype(np.uint8), off, np.zeros(len(seqs), np.int32), {})
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    hi = lo + 1
    # pairs that share their shorter sequence: several to a window
    lo = np.concatenate([lo, np.full(11, 60, np.uint32)])
    hi = np.concatenate([hi, np.arange(63, 85, 2, dtype=np.uint32)])
    gaps = {k: v for k, v in params.items() if k.startswith("gap")}
    want = orc.align_pairs(orc.encode(s.residues), s.offsets, lo, hi, mode="sw", **gaps)
    got = _gpu_records(gpu, s, np.tile(lo, copies), np.tile(hi, copies), **params)
    assert copies == 1 or got.size > 8192
    for c in range(copies):
        part = got[c * lo.size : (c + 1) * lo.size]
        if params.get("full_records"):
            _compare(part, want)
        else:
            _check16(part, want)


@pytest.mark.parametrize("width", [0, 32])
@pytest.mark.parametrize("gaps", [dict(), dict(gap_open=1, gap_extend=1)])
def test_start_bound_keeps_every_edge(gpu, orc, width, gaps):
    """The backward start bound at the coverage cut's two sides, with the
    alignment's rows at both sides of the 256 that it sweeps, a known end column
    (32-bit pass 1) and a window of columns (16-bit), and end rows that tie with
    the next one (a residue pair of score 0 follows); every pair takes it."""
    import paper_2009_14467_amd as P

    rng = np.random.default_rng(5)
    seqs = []
    for L in (40, 90, 181, 255, 256, 257, 300, 364, 365, 366, 367, 500, 900, 1100, 3100):
        for share in (0.6, 0.695, 0.7, 0.705, 0.8, 1.0):
            n = max(int(round(share * L)), 1)
            core = rng.integers(0, 20, n)
            other = core.copy()
            sub = rng.random(n) < 0.15
            other[sub] = rng.integers(0, 20, int(sub.sum()))
            before = int(rng.integers(0, L - n + 1))
            tie = L - n - before > 0 and rng.random() < 0.5  # A against T scores 0
            a = np.concatenate([rng.integers(0, 20, before), core, rng.integers(0, 20, L - n - before)])
            b = np.concatenate([rng.integers(0, 20, int(rng.integers(0, 60))), other, rng.integers(0, 20, L // 2 + 9)])
            if tie:
                a[before + n] = 0
                b[b.size - (L // 2 + 9)] = 16
            seqs += [a, b]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    res = letters[np.concatenate(seqs)]
    want = orc.search(res, off, k=6, ck_min=1, mode="sw", **gaps)
    ctx = P.Context(P.Params(k=6, ck_min=1, score_width=width, **gaps))
    ctx.set_tuning(sw_direct_pct=100000)
    got = ctx.search(_to_dev(res, gpu), _to_dev(off, gpu))
    st = ctx.stats()
    assert st["bound_pass_pairs"] > 0 and want.size > 0
    assert got.size == want.size and got.tobytes() == want.tobytes()


@pytest.mark.parametrize("copies", [1, 130])
def test_sw16_windows(gpu, orc, copies):
    """Windows of pairs that share sequence a: groups of one to nine pairs, in
    one-strip bins (both rows classes) and multi-strip bins, and, with copies,
    groups that span the blocks in which the windows are cut (1,024 items); rows
    at both sides of strip heights, b far longer than a (one past the
    traceback's 4,096 columns)."""
    from synth.families import FamilySet

    rng = np.random.default_rng(23)
    seqs = []
    shapes = [(L, L + d) for L in (1025, 1280, 1281, 1536, 1537, 1793, 2305, 2560, 2561, 2816, 2817, 2978)
              for d in (0, int(rng.integers(1, 90)))]
    shapes += [(1025, n) for n in (1087, 1088, 1089, 1151, 1152, 1153, 4096, 4097)]
    for la, lb in shapes:
        n = int(rng.integers(la // 3, la + 1))  # the shared segment
        at, bt = int(rng.integers(0, la - n + 1)), int(rng.integers(0, lb - n + 1))
        a, b = rng.integers(0, 20, la), rng.integers(0, 20, lb)
        seg = a[at : at + n].copy()
        sub = rng.random(n) < 0.25
        seg[sub] = rng.integers(0, 20, int(sub.sum()))
        b[bt : bt + n] = seg
        seqs += [a, b]
    short = len(seqs)
    for L in (20, 33, 64, 65, 97, 129, 200, 300, 449, 512, 700, 1000):
        seqs += [rng.integers(0, 20, L), rng.integers(0, 20, L)]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(letters[np.concatenate(seqs)].astype(np.uint8), off, np.zeros(len(seqs), np.int32), {})
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    hi = lo + 1
    group = rng.permutation(np.repeat(np.arange(12), [1, 1, 2, 3, 3, 4, 4, 5, 5, 7, 8, 9]))
    shares = short + 2 * group.astype(np.uint32)  # as a, against every longer sequence
    lo, hi = np.concatenate([lo, shares]), np.concatenate([hi, np.arange(shares.size, dtype=np.uint32)])
    want = orc.align_pairs(orc.encode(s.residues), s.offsets, lo, hi, mode="sw")
    for params in (dict(full_records=True), dict(score_width=16)):
        got = _gpu_records(gpu, s, np.tile(lo, copies), np.tile(hi, copies), **params)
        assert copies == 1 or got.size > 8192
        for c in range(copies):
            part = got[c * lo.size : (c + 1) * lo.size]
            if params.get("full_records"):
                _compare(part, want)
            else:
                _check16(part, want)


@pytest.mark.parametrize("copies", [1, 130])
def test_long_pairs_in_a_block(gpu, orc, copies):
    """Pairs of several strips in 32-bit lanes, one block of eight waves each
    (few pairs) and one wave each (with copies, more than 2,048): rows at both
    sides of a strip (512) and of eight of them (a wave's second strip), columns
    at both sides of a tile (512 steps), gaps that leave a tile or a strip,
    alignments that begin and end inside, unrelated pairs."""
    from synth.families import FamilySet

    rng = np.random.default_rng(29)
    seqs = []

    def add(a, b):
        sub = rng.random(b.size) < 0.2
        b = b.copy()
        b[sub] = rng.integers(0, 20, int(sub.sum()))
        seqs.extend([a, b])

    for L in (1025, 1536, 1537, 2047, 2560, 4095, 4096, 4097, 4609):
        a = rng.integers(0, 20, L)
        add(a, np.concatenate([rng.integers(0, 20, int(rng.integers(0, 70))), a, rng.integers(0, 20, 5)]))
    for L, g in ((2600, 700), (2600, -600), (1500, 1), (1500, -1)):
        a = rng.integers(0, 20, L)
        m = L // 2
        add(a, np.concatenate([a[:m], rng.integers(0, 20, g), a[m:]]) if g > 0 else np.delete(a, slice(m, m - g)))
    a = rng.integers(0, 20, 3000)
    add(np.concatenate([rng.integers(0, 20, 700), a[500:2000], rng.integers(0, 20, 900)]), a)
    add(rng.integers(0, 20, 1300), rng.integers(0, 20, 1800))
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(letters[np.concatenate(seqs)].astype(np.uint8), off, np.zeros(len(seqs), np.int32), {})
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    hi = lo + 1
    lo, hi = np.concatenate([lo, [0, 12]]).astype(np.uint32), np.concatenate([hi, [14, 16]]).astype(np.uint32)
    want = orc.align_pairs(orc.encode(s.residues), s.offsets, lo, hi, mode="sw")
    assert copies == 1 or copies * lo.size > 2048
    for full in (True, False):
        got = _gpu_records(gpu, s, np.tile(lo, copies), np.tile(hi, copies), full_records=full, score_width=32)
        fields = FIELDS if full else ("score", "end_a", "end_b", "passed", "swapped", "cells")
        for c in range(copies):
            _compare(got[c * lo.size : (c + 1) * lo.size], want, fields)


def test_records_do_not_depend_on_the_bound(gpu):
    """Which pairs of an alignment call carry statistics is a matter of their
    scores and of the coverage that the start bound leaves, in either score
    width: weakly similar segments of 100 to 700 rows at and under the coverage
    cut (far beyond the rows a shortened sweep would see)."""
    from synth.families import FamilySet

    rng = np.random.default_rng(31)
    seqs = []
    for L in (300, 420, 600, 800, 1000):
        for share in (0.3, 0.5, 0.6, 0.66, 0.69, 0.72):
            for rate in (0.55, 0.62, 0.68, 0.72):
                n = int(share * L)
                a, b = rng.integers(0, 20, L), rng.integers(0, 20, L + 10)
                at = L - n  # the segment ends with a, so that pass 1 alone cannot tell
                seg = a[at:].copy()
                sub = rng.random(n) < rate
                seg[sub] = rng.integers(0, 20, int(sub.sum()))
                b[5 : 5 + n] = seg
                seqs += [a, b]
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    s = FamilySet(letters[np.concatenate(seqs)].astype(np.uint8), off, np.zeros(len(seqs), np.int32), {})
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    full = _gpu_records(gpu, s, lo, lo + 1, full_records=True)
    for width in (0, 16, 32):
        got = _gpu_records(gpu, s, lo, lo + 1, score_width=width)
        span = full["end_a"] - full["beg_a"] + 1
        la = np.diff(off)[::2]
        assert 0 < (got["beg_a"] < 0).sum() < got.size
        none = got["beg_a"] < 0
        assert np.all(100 * span[none] < 70 * la[none])
        _compare(got, full, FIELDS, ~none)
        if width == 0:
            first = none
        np.testing.assert_array_equal(none, first)


def _family_of(seqs):
    from synth.families import FamilySet

    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    return FamilySet(letters[np.concatenate(seqs)].astype(np.uint8), off, np.zeros(len(seqs), np.int32), {})


def _related(rng, L, rate=0.2, pre=20, post=9):
    a = rng.integers(0, 20, L)
    b = a.copy()
    sub = rng.random(L) < rate
    b[sub] = rng.integers(0, 20, int(sub.sum()))
    return [a, np.concatenate([rng.integers(0, 20, pre), b, rng.integers(0, 20, post)])]


def test_calls_without_room_for_the_extra_buffers(gpu, orc):
    """A device too full (here: a limit of the context) for the traceback's
    direction bits, or for the long pairs' slots as well, gives the same records
    without an error left behind, and the few blocks planned for the few long
    pairs do not get the statistics of every other pair of several strips."""
    import time

    import torch

    import paper_2009_14467_amd as P

    rng = np.random.default_rng(37)
    seqs = []
    for L in (1030, 1100, 1152, 1153, 1200, 1281, 90, 300, 700, 1000):
        seqs += _related(rng, L)
    several = len(seqs)
    for L in (3000, 3100, 3200):  # 32-bit lanes
        seqs += _related(rng, L)
    s = _family_of(seqs)
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    want = orc.align_pairs(orc.encode(s.residues), s.offsets, lo, lo + 1, mode="sw")
    copies = 400  # 2,400 pairs of several strips in 16-bit lanes, and three long ones
    at = np.concatenate([np.tile(np.arange(several // 2), copies), np.arange(several // 2, lo.size)])
    args = [_to_dev(x, gpu) for x in (s.residues, s.offsets, lo[at], lo[at] + 1)]
    times = {}
    for mib in (0, 64, 1):  # all fits; no direction bits; no slots either
        ctx = P.Context(P.Params(full_records=True))
        ctx.set_tuning(sw_extra_mib=mib)
        for rep in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            out = ctx.align_pairs(*args)
            torch.cuda.synchronize()
            dt = time.perf_counter() - t0
            times[mib] = min(times.get(mib, dt), dt)
        _compare(P.records_to_numpy(out), want[at])
        assert P.lib().pastis_last_error(ctx._ctx) == b""
    print({k: round(1e3 * v, 2) for k, v in times.items()}, "ms")
    assert times[64] < 12 * times[0] and times[1] < 12 * times[0], times


def test_calls_in_32_bit_lanes_hold_no_rows_for_16_bits(gpu):
    """Boundary rows of the 16-bit kernels belong to calls that have pairs of
    several strips in 16-bit lanes: a long pair in 32-bit lanes holds those of the
    32-bit kernels alone (24 bytes per residue of the longest sequence and each of
    1,536 waves, and a quarter's headroom)."""
    import torch

    import paper_2009_14467_amd as P

    rng = np.random.default_rng(41)
    s = _family_of(_related(rng, 20000))
    args = [_to_dev(x, gpu) for x in (s.residues, s.offsets, np.array([0], np.uint32), np.array([1], np.uint32))]
    ctx = P.Context(P.Params(score_width=32))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    ctx.align_pairs(*args)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = before - torch.cuda.mem_get_info()[0]
    rows = 24 * 20029 * 1536 * 5 // 4
    print(held, rows)
    assert held < rows + (100 << 20)


def _best_ms(f, reps=4):
    import time

    import torch

    best = 1e9
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, 1e3 * (time.perf_counter() - t0))
    return best


def test_long_pairs_run_beside_the_others_in_any_program(gpu):
    """The launches of a pass overlap whatever streams the program has made and
    destroyed: contexts that came after others had gone, beside others, and on
    streams of the caller's own take the time of the first (a quarter more where
    the long pairs and the 16-bit bins shared a hardware queue)."""
    import torch

    import paper_2009_14467_amd as P

    rng = np.random.default_rng(43)
    seqs = []
    for _ in range(8):
        seqs += _related(rng, 12000 + int(rng.integers(0, 50)))
    long = len(seqs)
    for _ in range(40):
        seqs += _related(rng, int(rng.integers(300, 500)))
    s = _family_of(seqs)
    lo = np.concatenate([np.tile(np.arange(0, long, 2), 4), np.tile(np.arange(long, len(seqs), 2), 3000)])
    args = [_to_dev(x, gpu) for x in (s.residues, s.offsets, lo.astype(np.uint32), (lo + 1).astype(np.uint32))]

    def context():
        return P.Context(P.Params(full_records=True))

    first = context()
    alone = _best_ms(lambda: first.align_pairs(*args))
    times = {}
    others = [context() for _ in range(5)]
    for k, c in enumerate(others):
        times[f"beside {k + 1}"] = _best_ms(lambda: c.align_pairs(*args))
    del others[1], others[2]
    for k in range(3):
        c = context()
        times[f"after others {k}"] = _best_ms(lambda: c.align_pairs(*args))
        others.append(c)
    streams = [torch.cuda.Stream() for _ in range(6)]
    for k, q in enumerate(streams):
        with torch.cuda.stream(q):
            times[f"stream {k}"] = _best_ms(lambda: first.align_pairs(*args))
    print(round(alone, 2), {k: round(v, 2) for k, v in times.items()})
    assert max(times.values()) < 1.12 * alone, (alone, times)


def test_contexts_are_made_without_streams(gpu):
    """A context that never spreads a pass over several launches makes none of the
    streams for it: it costs less than making and destroying four streams."""
    import ctypes
    import time

    import torch

    import paper_2009_14467_amd as P

    hip = ctypes.CDLL("libamdhip64.so")
    keep = P.Context(P.Params())  # the library's one-time work

    def streams():
        made = []
        for _ in range(4):
            q = ctypes.c_void_p()
            assert hip.hipStreamCreateWithFlags(ctypes.byref(q), 1) == 0  # hipStreamNonBlocking
            made.append(q)
        for q in made:
            assert hip.hipStreamDestroy(q) == 0

    def context():
        c = P.Context(P.Params())
        del c

    def median(f):
        ts = []
        for _ in range(40):
            t0 = time.perf_counter()
            f()
            ts.append(1e6 * (time.perf_counter() - t0))
        return sorted(ts)[20]

    torch.cuda.synchronize()
    a, b = median(context), median(streams)
    print(f"context {a:.0f} us, four streams {b:.0f} us")
    assert a < b
    del keep


@pytest.mark.parametrize("graph", [False, True])
def test_contexts_of_two_threads_share_the_lanes(gpu, graph):
    """Two threads, a context and a stream each, with calls of several launches a
    pass at the same time: every result is that of a call alone, also while one of
    the contexts captures its passes as a graph."""
    import threading

    import torch

    import paper_2009_14467_amd as P

    rng = np.random.default_rng(47)

    def setting(k):
        seqs = []
        for _ in range(6):
            seqs += _related(rng, 3000 + 700 * k + int(rng.integers(0, 50)))
        for _ in range(60):
            seqs += _related(rng, int(rng.integers(40, 1500)))
        s = _family_of(seqs)
        return _to_dev(s.residues, gpu), _to_dev(s.offsets, gpu)

    sets = [setting(0), setting(1)]
    args = [dict(k=6, ck_min=1, score_width=32), dict(k=6, ck_min=1, graph_mode=graph)]
    want = [P.Context(P.Params(k=6, ck_min=1)).search(*x) for x in sets]
    ctxs = [P.Context(P.Params(**a)) for a in args]
    streams = [torch.cuda.Stream() for _ in sets]
    torch.cuda.synchronize()
    got = [[], []]
    errors = []

    def work(t):
        try:
            with torch.cuda.stream(streams[t]):
                for rep in range(12):
                    # (a set of the other thread's now and then: new pair counts, new captures)
                    k = t if rep % 3 else 1 - t
                    got[t].append((k, ctxs[t].search(*sets[k])))
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for t in range(2):
        assert len(got[t]) == 12
        for k, e in got[t]:
            assert e.size > 0 and e.tobytes() == want[k].tobytes()


@pytest.mark.parametrize("total", [2048, 2049])
@pytest.mark.parametrize("intra", [0, 1])
def test_long_pairs_at_the_block_limit(gpu, orc, total, intra):
    """Pairs of several strips in 32-bit lanes at the number up to which each has a
    block: beyond it, pass 1 runs one wave a pair or (sw_intra_pair) a workgroup of
    four waves, whose strips are pipelined; 2 to 9 strips, pairs that share
    sequences, unrelated pairs, rows at both sides of a strip and of a round of the
    workgroup's waves."""
    rng = np.random.default_rng(53)
    seqs = []
    for L in (1025, 1100, 2047, 2500, 2979, 3100, 4096, 4097, 5000, 9000):
        seqs += _related(rng, L, post=int(rng.integers(0, 60)))
    s = _family_of(seqs)
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    lo, hi = np.concatenate([lo, [4, 6, 8, 10]]).astype(np.uint32), np.concatenate([lo + 1, [9, 11, 15, 13]])
    hi = hi.astype(np.uint32)
    want = orc.align_pairs(orc.encode(s.residues), s.offsets, lo, hi, mode="sw")
    at = np.arange(total) % lo.size
    for full in (True, False):
        got = _gpu_records(gpu, s, lo[at], hi[at], tuning=dict(sw_intra_pair=intra), full_records=full, score_width=32)
        _compare(got, want[at], FIELDS if full else ("score", "end_a", "end_b", "passed", "swapped", "cells"))


@pytest.mark.parametrize("total", [4096, 4097, 8192, 8193])
@pytest.mark.parametrize("narrow", [0, 4])
def test_sw16_calls_at_the_sizes_of_its_layouts(gpu, orc, total, narrow):
    """16-bit calls at both sides of the numbers of pairs that choose the layout:
    traceback kernels for two waves per SIMD up to 4,096, bins of up to 8 rows per
    lane across all 64 lanes up to 8,192, in strips of 16 (narrow 4) and 32 lanes
    beyond; both rows classes of every bin, windows of one to five pairs of a
    sequence, several strips, and columns past the direction buffers' limit."""
    rng = np.random.default_rng(59)
    lens = [1, 2, 31, 33, 63, 64, 65, 1023, 1024, 1025, 1100, 1537, 2049, 2978]
    lens += [64 * R - 32 + d for R in range(1, 17) for d in (0, 1, 32)]
    seqs = []
    for L in lens:
        seqs += _related(rng, L, rate=0.25, pre=int(rng.integers(0, 40)), post=5)
    single = len(seqs)
    seqs += [rng.integers(0, 20, 300), rng.integers(0, 20, 2049), rng.integers(0, 20, 1100), rng.integers(0, 20, 4097)]
    s = _family_of(seqs)
    lo = np.arange(0, single, 2, dtype=np.uint32)
    hi = lo + 1
    # more pairs of some sequences: windows of several
    few = np.repeat(np.arange(14, 44, 2), np.arange(15) % 5)
    lo = np.concatenate([lo, few, [single, single + 2]]).astype(np.uint32)
    hi = np.concatenate([hi, few + 3 + 2 * (np.arange(few.size) % 7), [single + 1, single + 3]]).astype(np.uint32)
    want = orc.align_pairs(orc.encode(s.residues), s.offsets, lo, hi, mode="sw")
    at = np.arange(total) % lo.size
    tuning = dict(sw16_narrow_rows=narrow)
    _compare(_gpu_records(gpu, s, lo[at], hi[at], tuning=tuning, full_records=True), want[at])
    _check16(_gpu_records(gpu, s, lo[at], hi[at], tuning=tuning, score_width=16), want[at])


@pytest.mark.parametrize("width", [0, 32])
def test_few_long_pairs_among_many_shorter(gpu, orc, width):
    """Pairs of over 2,978 rows keep a block each when the multi-strip pairs of
    fewer rows (here of more columns than the traceback takes) are too many for
    blocks: the call takes about as long as the two kinds alone, not as long as
    single waves take for the longest pairs."""
    import paper_2009_14467_amd as P

    rng = np.random.default_rng(61)
    seqs = []
    for L in (3000, 4100, 5000, 12000, 11000, 10000):
        seqs += _related(rng, L)
    long = len(seqs)
    for L in (1030, 1100, 1200, 1300):
        a = rng.integers(0, 20, L)
        seqs += [a, np.concatenate([rng.integers(0, 20, 1700), a, rng.integers(0, 20, 1400)])]
    s = _family_of(seqs)
    lo = np.arange(0, len(seqs), 2, dtype=np.uint32)
    want = orc.align_pairs(orc.encode(s.residues), s.offsets, lo, lo + 1, mode="sw")
    few = np.arange(60) % (long // 2)
    many = long // 2 + np.arange(2100) % 4
    ctx = P.Context(P.Params(full_records=True, score_width=width))
    res, off = _to_dev(s.residues, gpu), _to_dev(s.offsets, gpu)
    ms = []
    for at in (few, many, np.concatenate([many[:1000], few, many[1000:]])):
        i, j = _to_dev(lo[at], gpu), _to_dev(lo[at] + 1, gpu)
        _compare(P.records_to_numpy(ctx.align_pairs(res, off, i, j)), want[at])
        ms.append(_best_ms(lambda: ctx.align_pairs(res, off, i, j), 3))
    print([round(x, 2) for x in ms], "ms")
    assert ms[2] < 1.5 * (ms[0] + ms[1]), ms
