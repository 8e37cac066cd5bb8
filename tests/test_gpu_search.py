"""End-to-end parity: sequences in, edges out (Section II problem, Section IV
pipeline) against the CPU oracle's search.  Every edge field is compared;
the float weights bit for bit (both sides divide in IEEE float32)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EDGE_FIELDS = ("i", "j", "score", "matches", "columns", "beg_i", "end_i", "beg_j", "end_j", "shared_kmers",
               "seed_used", "flags", "identity", "ns_weight")


def _dev(x, gpu):
    import torch

    return torch.from_numpy(np.ascontiguousarray(x)).to(gpu)


def _compare_edges(got, want):
    assert got.size == want.size, f"{got.size} edges vs {want.size}"
    for f in EDGE_FIELDS:
        g, w = got[f], want[f]
        if g.dtype == np.float32:
            g, w = g.view(np.uint32), w.view(np.uint32)
        bad = np.nonzero(g != w)[0]
        assert bad.size == 0, f"{f}: {bad.size} mismatches at {bad[:5]}: got {got[f][bad[:5]]} want {want[f][bad[:5]]}"


@pytest.mark.parametrize("weight", ["ani", "ns"])
def test_search_sw_tiny(gpu, orc, weight):
    import paper_2009_14467_amd as P
    from synth import workload

    s = workload("tiny")
    want = orc.search(s.residues, s.offsets, k=6, ck_min=1, mode="sw", weight=weight)
    ctx = P.Context(P.Params(k=6, ck_min=1, weight_mode=weight))
    got = ctx.search(_dev(s.residues, gpu), _dev(s.offsets, gpu))
    _compare_edges(got, want)
    if weight == "ani":
        st = ctx.stats()
        assert st["n_edges"] == want.size and st["n_candidates"] > 0


def test_search_sw_substitutes_host_input(gpu, orc):
    """Host-resident inputs take the staging path; substitute k-mers, ck >= 2."""
    import torch

    import paper_2009_14467_amd as P
    from synth import workload

    s = workload("tiny", n_families=8)
    want = orc.search(s.residues, s.offsets, k=6, n_subs=25, ck_min=2, mode="sw")
    ctx = P.Context(P.Params(k=6, n_subs=25, ck_min=2))
    got = ctx.search(torch.from_numpy(s.residues), torch.from_numpy(s.offsets))
    _compare_edges(got, want)


def test_search_repeatable(gpu):
    """The graph does not depend on scheduling: two runs give identical bytes."""
    import paper_2009_14467_amd as P
    from synth import workload

    s = workload("tiny", n_families=10)
    ctx = P.Context(P.Params(k=5, n_subs=10, ck_min=2))
    a = ctx.search(_dev(s.residues, gpu), _dev(s.offsets, gpu))
    b = P.Context(P.Params(k=5, n_subs=10, ck_min=2)).search(_dev(s.residues, gpu), _dev(s.offsets, gpu))
    assert a.tobytes() == b.tobytes()


@pytest.mark.parametrize("tuning", [dict(sw16_max_rows=0), dict(sw16_max_rows=8, sw_direct_pct=0),
                                    dict(sw16_max_rows=12, sw_direct_pct=1 << 20, sw_grid_scale=1),
                                    dict(sw16_max_rows=16, sw_direct_pct=25, sw_grid_scale=64, sw_grid_scale_wide=3),
                                    dict(sw16_max_rows=0, sw_intra_pair=1), dict(sw16_narrow_rows=0),
                                    dict(sw16_narrow_rows=2, sw_direct_pct=0), dict(sw_long_blocks=1),
                                    dict(sw16_max_rows=0, sw_long_blocks=2)])
def test_every_schedule_gives_the_same_edges(gpu, orc, tuning):
    """Schedule knobs move time, never results: each setting against the oracle."""
    import paper_2009_14467_amd as P
    from synth import make_family_set

    s = make_family_set(n_families=12, family_size=8, mean_len=500, min_len=30, max_len=1500, divergence=0.3,
                        stream=55)
    want = orc.search(s.residues, s.offsets, k=6, ck_min=1, mode="sw")
    ctx = P.Context(P.Params(k=6, ck_min=1))
    ctx.set_tuning(**tuning)
    got = ctx.search(_dev(s.residues, gpu), _dev(s.offsets, gpu))
    _compare_edges(got, want)


def test_autotune_picks_a_valid_schedule(gpu):
    import paper_2009_14467_amd as P
    from synth import workload

    s = workload("tiny")
    res, off = _dev(s.residues, gpu), _dev(s.offsets, gpu)
    ctx = P.Context(P.Params(k=6, ck_min=1))
    before = ctx.search(res, off)
    t = ctx.autotune(res, off, max_pairs=2000)
    assert t == ctx.get_tuning()
    assert t["sw16_max_rows"] in (0, 8, 12, 16) and t["sw_grid_scale"] in (1, 2, 4)
    assert t["sw_grid_scale_wide"] in (1, 2, 4) and t["sw16_narrow_rows"] in (0, 2, 4)
    assert before.tobytes() == ctx.search(res, off).tobytes()
    with pytest.raises(P.PastisError):
        ctx.set_tuning(sw16_max_rows=17)
    with pytest.raises(P.PastisError):
        ctx.set_tuning(sw16_narrow_rows=5)
    with pytest.raises(P.PastisError):
        ctx.set_tuning(sw_long_blocks=0)


def test_graph_mode_replays_match_direct_launches(gpu):
    """The SW stage captured once and replayed: every replay, with direct
    launches of another context in between, gives the direct result; a new
    pair count forces a new capture."""
    import paper_2009_14467_amd as P
    from synth import workload

    s = workload("tiny")
    res, off = _dev(s.residues, gpu), _dev(s.offsets, gpu)
    eager = P.Context(P.Params(k=6, ck_min=1))
    graph = P.Context(P.Params(k=6, ck_min=1, graph_mode=True))
    want = eager.search(res, off)
    modes = []
    for rep in range(4):
        got = graph.search(res, off)
        modes.append(graph.stats()["sw_graph"])
        _compare_edges(got, want)
        _compare_edges(eager.search(res, off), want)  # direct work between replays
    assert modes == [1, 2, 2, 2]
    s2 = workload("tiny", n_families=9)
    r2, o2 = _dev(s2.residues, gpu), _dev(s2.offsets, gpu)
    _compare_edges(graph.search(r2, o2), eager.search(r2, o2))
    assert graph.stats()["sw_graph"] == 1
    _compare_edges(graph.search(res, off), want)


ROW_BLOCK_CASES = {
    "exact-sw": dict(k=6, ck_min=1),
    "subs-sw": dict(k=6, n_subs=25, ck_min=2),
    "exact-xd": dict(k=6, ck_min=1, align_mode="xd"),
    "subs-ns-graph": dict(k=5, n_subs=10, ck_min=2, weight_mode="ns", graph_mode=True),
}


@pytest.mark.parametrize("case", sorted(ROW_BLOCK_CASES))
def test_row_blocks_give_the_same_edges(gpu, orc, case):
    """Discovery, alignment and the cut run block by block when the
    directional entries exceed block_entries (the pairs of a range of lower
    indices per block, halved until each fits): the same edges, counts and
    cells as one block, and the oracle's edges."""
    import paper_2009_14467_amd as P
    from synth import workload

    s = workload("tiny", n_families=8)
    res, off = _dev(s.residues, gpu), _dev(s.offsets, gpu)
    kw = ROW_BLOCK_CASES[case]
    one = P.Context(P.Params(**kw))
    want = one.search(res, off)
    st1 = one.stats()
    nc = int(st1["n_candidates"])
    assert nc > 200
    one.candidates(nc)  # one block keeps its candidates
    blocks = P.Context(P.Params(block_entries=max(nc // 6, 8), **kw))
    got = blocks.search(res, off)
    assert got.tobytes() == want.tobytes()
    st = blocks.stats()
    assert st1["n_row_blocks"] == 1 and st["n_row_blocks"] >= 4
    for f in ("n_candidates", "n_aligned", "n_edges", "cells", "stats_pass_pairs", "stats_pass_cells",
              "bound_pass_pairs", "bound_pass_cells"):
        assert st[f] == st1[f], f
    with pytest.raises(P.PastisError) as e:
        blocks.candidates(nc)  # several blocks: the candidate buffers hold only the last one
    assert e.value.status == 6  # PASTIS_E_STATE
    if case == "exact-sw":
        oracle_kw = {k: v for k, v in kw.items() if k != "align_mode"}
        _compare_edges(got, orc.search(s.residues, s.offsets, mode="sw", **oracle_kw))
    # the substitute product of a block counts both directions of its pairs:
    # a repeat of the blocked search is byte-identical too
    assert blocks.search(res, off).tobytes() == want.tobytes()


def test_row_block_of_one_sequence_over_the_limit_fails(gpu):
    import paper_2009_14467_amd as P
    from synth import make_family_set

    s = make_family_set(n_families=2, family_size=4, mean_len=200, min_len=100, max_len=300, divergence=0.2,
                        stream=91)
    ctx = P.Context(P.Params(k=4, ck_min=1, block_entries=1))
    with pytest.raises(P.PastisError) as e:
        ctx.search(_dev(s.residues, gpu), _dev(s.offsets, gpu))
    assert e.value.status == 5  # PASTIS_E_CAPACITY
    with pytest.raises(P.PastisError):
        P.Context(P.Params(block_entries=-1))


def test_counters_do_not_depend_on_the_run(gpu):
    """The counters of a search (pairs and cells of every pass) are those of its
    input: pairs that share a wave of the start bound, in whatever order its list
    was written, do not decide about one another."""
    import paper_2009_14467_amd as P
    from synth import make_family_set

    s = make_family_set(n_families=20, family_size=20, mean_len=500, min_len=30, max_len=3000, divergence=0.4,
                        stream=56)
    res, off = _dev(s.residues, gpu), _dev(s.offsets, gpu)
    ctx = P.Context(P.Params(k=5, n_subs=25, ck_min=2))
    ctx.set_tuning(sw_direct_pct=100000)  # every pair takes the bound
    seen = set()
    for _ in range(8):
        ctx.search(res, off)
        st = ctx.stats()
        seen.add(tuple(st[k] for k in ("n_aligned", "cells", "bound_pass_pairs", "bound_pass_cells",
                                       "stats_pass_pairs", "stats_pass_cells", "n_edges")))
    assert st["bound_pass_pairs"] > 10000
    assert len(seen) == 1, seen


def test_buffers_that_only_save_time_make_room(gpu):
    """The direction bits that an alignment call left with the context are given
    back when a later call of it finds the device full."""
    import torch

    import paper_2009_14467_amd as P
    from synth import make_family_set

    long = make_family_set(n_families=3, family_size=40, mean_len=1300, min_len=1100, max_len=1600, divergence=0.3,
                           stream=57)
    short = make_family_set(n_families=4, family_size=10, mean_len=40, min_len=20, max_len=60, divergence=0.3,
                            stream=58)
    lo, hi = (_dev(x.astype(np.uint32), gpu) for x in np.triu_indices(long.n, 1))
    lo2, hi2 = (_dev(x.astype(np.uint32), gpu) for x in np.triu_indices(short.n, 1))
    copies = 40000  # 31 million pairs, about 115 bytes each
    many = [_dev(short.residues, gpu), _dev(short.offsets, gpu), lo2.repeat(copies), hi2.repeat(copies)]
    want = P.Context(P.Params(full_records=True)).align_pairs(*many[:2], lo2, hi2)
    ctx = P.Context(P.Params(full_records=True))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    ctx.align_pairs(_dev(long.residues, gpu), _dev(long.offsets, gpu), lo, hi)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    assert before - free > 5 << 30
    full = None
    try:
        try:  # room for the records and 2 GiB
            full = torch.empty(free - copies * lo2.numel() * 48 - (2 << 30), dtype=torch.uint8, device=gpu)
        except torch.cuda.OutOfMemoryError:
            pytest.skip("the device is shared")
        got = ctx.align_pairs(*many).view(copies, -1)
        assert all(bool((part == want).all()) for part in got.split(4000))
    finally:
        del full
        torch.cuda.empty_cache()


def test_autotune_leaves_a_knob_without_effect(gpu):
    """A set with few or no long pairs runs the same kernels for both values of
    sw_intra_pair: the tuner keeps the value it finds, whichever runs faster that
    time."""
    import paper_2009_14467_amd as P
    from synth import workload

    s = workload("tiny")
    res, off = _dev(s.residues, gpu), _dev(s.offsets, gpu)
    ctx = P.Context(P.Params(k=6, ck_min=1))
    for rep in range(12):
        ctx.set_tuning(sw_intra_pair=rep % 2)
        assert ctx.autotune(res, off, max_pairs=500)["sw_intra_pair"] == rep % 2, rep


def test_graph_mode_with_passes_of_several_launches(gpu):
    """Replays of passes that spread over several streams (long pairs in blocks, then
    the traceback; statistics of several groups of bins), with eager searches and
    synchronizations in between, give the eager result every time, in both widths."""
    import torch

    import paper_2009_14467_amd as P
    from synth import make_family_set

    s = make_family_set(n_families=44, family_size=16, mean_len=900, min_len=30, max_len=2500, divergence=0.35,
                        long_frac=0.06, long_range=(3050, 3200), stream=9)
    res, off = _dev(s.residues, gpu), _dev(s.offsets, gpu)
    L = np.diff(s.offsets)
    assert (L > 2978).sum() > 1
    eager = P.Context(P.Params(k=5, ck_min=1))
    want = eager.search(res, off)
    bins = eager.stats()["sw_bins"]
    assert sum(b["pairs"] for b in bins if b["multi_strip"] and b["bits"] == 32) > 0
    assert sum(b["cells"] for b in bins if b["bits"] == 16) > 4096 * int(L.max()) ** 2
    for width in (0, 32):
        graph = P.Context(P.Params(k=5, ck_min=1, graph_mode=True, score_width=width))
        for rep in range(4):
            got = graph.search(res, off)
            assert got.tobytes() == want.tobytes(), (width, rep)
            assert graph.stats()["sw_graph"] == (1 if rep == 0 else 2)
            assert eager.search(res, off).tobytes() == want.tobytes()
            torch.cuda.synchronize()


def test_graph_mode_with_passes_led_by_different_lanes(gpu):
    """One capture whose pass 1 gives the long pairs a block each and whose statistics
    take them in single waves (too many pairs of fewer rows and a long b): the
    capture ends, and its replays give the eager result."""
    import torch

    import paper_2009_14467_amd as P

    rng = np.random.default_rng(67)
    letters = np.frombuffer(b"ARNDCQEGHILKMFPSTWYV", np.uint8)
    motif = rng.integers(0, 20, 60)
    seqs = []
    related = rng.integers(0, 20, 4300)
    for L, n in ((4300, 20), (1300, 130)):
        for _ in range(n):
            x = rng.integers(0, 20, L + int(rng.integers(0, 150)))
            if L == 4300:
                x[:L] = np.where(rng.random(L) < 0.2, x[:L], related)
            at = int(rng.integers(0, x.size - 60))
            x[at : at + 60] = motif
            seqs.append(x)
    off = np.zeros(len(seqs) + 1, np.int64)
    np.cumsum([len(x) for x in seqs], out=off[1:])
    res, offd = _dev(letters[np.concatenate(seqs)], gpu), _dev(off, gpu)
    eager = P.Context(P.Params(k=6, ck_min=2))
    eager.set_tuning(sw_direct_pct=0)  # every pair whose coverage can hold takes statistics
    want = eager.search(res, offd)
    st = eager.stats()
    L = np.diff(off)
    assert want.size >= 190 and st["n_aligned"] == len(seqs) * (len(seqs) - 1) // 2
    multi = [b for b in st["sw_bins"] if b["multi_strip"]]
    assert 0 < sum(b["pairs"] for b in multi if b["bits"] == 32) <= 2048 < 20 * 130
    assert sum(b["cells"] for b in multi) > 1024 * int(L.max()) ** 2
    graph = P.Context(P.Params(k=6, ck_min=2, graph_mode=True))
    graph.set_tuning(sw_direct_pct=0)
    for rep in range(4):
        assert graph.search(res, offd).tobytes() == want.tobytes(), rep
        assert graph.stats()["sw_graph"] == (1 if rep == 0 else 2)
        assert eager.search(res, offd).tobytes() == want.tobytes()
        torch.cuda.synchronize()
