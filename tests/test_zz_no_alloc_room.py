"""How many pairs the no-allocation workspace holds (through the C ABI)."""

import numpy as np
import pytest

from test_zz_no_alloc import _dev, _noalloc

pytestmark = pytest.mark.gpu


def _bytes(npairs, n_res):
    """What a call in 32-bit lanes carved from the workspace when its counters and
    tables took 1,856 bytes: the codes and 73 bytes per pair."""

    def up(b):
        return (b + 255) // 256 * 256

    per_pair = [48, 16, 1, 4, 4]
    return up(32) + up(n_res) + sum(up(b * npairs) for b in per_pair) + up(1856) + 256


def test_noalloc_holds_as_many_pairs_as_ever(gpu):
    import torch

    import paper_2009_14467_amd as P
    from synth.families import FamilySet

    seqs = [b"ACDEFGHIKL", b"ACDEFGHIKLM", b"MNPQRSTVWY"]
    off = np.array([0, 10, 21, 31], np.int64)
    s = FamilySet(np.frombuffer(b"".join(seqs), np.uint8).copy(), off, np.zeros(3, np.int32), {})
    res, offd = _dev(s.residues, gpu), _dev(s.offsets, gpu)
    most = (48 << 20) // 73
    while _bytes(most, 31) > 48 << 20:
        most -= 1
    assert most > 680000
    pairs = np.array([[0, 1], [0, 2], [1, 2]], np.uint32)[np.arange(most) % 3]
    pi, pj = _dev(pairs[:, 0], gpu), _dev(pairs[:, 1], gpu)
    out = torch.full((most * 48,), 0xAB, dtype=torch.uint8, device=gpu)
    ctx = P.Context(P.Params(k=6))
    st = _noalloc(P, ctx, res, offd, pi, pj, None, None, out)
    assert st == 0, P.lib().pastis_last_error(ctx._ctx)
    want = ctx.align_pairs(res, offd, pi, pj)
    torch.cuda.synchronize()
    assert (out == want).all()
