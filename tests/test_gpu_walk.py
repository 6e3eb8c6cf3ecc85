"""GPU parity of the long pairs' walk at its edges: runs of mismatches and gaps
around the 16 cells a round trip takes, matches around the 64 bases a lane
follows by itself and the 1024 of a wavefront, edits with no match between them
around the 64 runs are made of at a time, scores around the rows that cut a path
into pieces and where their distance doubles.  Integer results: byte-identical
to the oracle, exact and with the adaptive heuristic."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu


def _seq(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def _other(base):
    return np.array([b"ACGT"[(b"ACGT".index(bytes([x])) + 1) % 4] for x in base], np.uint8)


def _pairs(rng):
    pairs = []
    for n in (1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 130):
        p = _seq(rng, 1300 + 5 * n)
        swap = p.copy()
        swap[600:600 + n] = _other(p[600:600 + n])  # a run of mismatches (or a gap pair)
        gap = np.concatenate([p[:700], _seq(rng, n), p[700:]])
        pairs += [(p, swap), (p, gap), (gap, p), (swap, gap)]
        near = p.copy()  # edits one, and n, bases apart
        near[100:100 + 2 * n:2] = _other(near[100:100 + 2 * n:2])
        near[500:900:n + 1] = _other(near[500:900:n + 1])
        pairs += [(p, near), (near[n:], p)]
    for n in (62, 63, 64, 65, 66, 1023, 1024, 1025, 2050, 5000):
        p = _seq(rng, 3 * n + 40)
        t = p.copy()
        for at in (n, 2 * n + 1):
            t[at] = _other(t[at:at + 1])[0]
        pairs += [(p, p), (p, t), (p, np.delete(t, n // 2)), (np.delete(p, 0), t)]
    for edits in (5, 15, 16, 17, 60, 120, 245, 250, 260, 500, 520):
        p = _seq(rng, 6000)
        t = p.copy()
        at = np.sort(rng.choice(6000, edits, replace=False))
        t[at] = _other(t[at])
        pairs += [(p, t), (t, np.delete(p, at[::3]))]
    return pairs


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
@pytest.mark.parametrize("heur", [None, (10, 50)])
def test_walk_edges(oracle_lib, synth_lib, pen, heur):
    import paper_2204_02085_amd as wfa

    rng = np.random.default_rng(17)
    b = synth_lib.from_pairs([(bytes(p), bytes(t)) for p, t in _pairs(rng)])
    say(f"case: walk edges, penalties {pen}, heuristic {heur}, {len(b)} pairs")
    kw = {"adaptive": heur} if heur else {}
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8, **kw)
    al = wfa.Aligner(0)
    try:
        if heur:
            al.set_heuristic(*heur)
        got = al.align(b, pen, capacity=int(ref.offsets[-1]) + 8)
        assert al.stats()["general_pairs"] > 0
    finally:
        al.close()
    assert_same(got, ref, b, f"{pen} {heur}")


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
def test_bound_from_both_ends(oracle_lib, synth_lib, pen):
    """The score bound is found from both ends: lengths around the words of the
    reversed sequences, length differences of both parities, edits at either end or
    in the middle, where the two meet, and none."""
    import paper_2204_02085_amd as wfa

    rng = np.random.default_rng(23)
    pairs = [(_seq(rng, 2500), _seq(rng, 2500)[:100])]  # the batch is the long kernels'
    for n in (1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 1000, 2401):
        p = _seq(rng, n)
        pairs += [(p, p), (p, p[:0]), (p[:0], p), (p, _other(p[:1])), (p, _seq(rng, max(1, n - 1)))]
        for at in (0, n // 2, n - 1):
            t = p.copy()
            t[at] = _other(t[at:at + 1])[0]
            pairs += [(p, t), (p, np.delete(p, at)), (np.delete(t, at), p)]
            for gap in (1, 2, 7, 64, 131):
                pairs.append((p, np.concatenate([t[:at], _seq(rng, gap), t[at:]])))
    b = synth_lib.from_pairs([(bytes(p), bytes(t)) for p, t in pairs])
    say(f"case: bounds from both ends, penalties {pen}, {len(b)} pairs")
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8)
    al = wfa.Aligner(0)
    try:
        got = al.align(b, pen, capacity=int(ref.offsets[-1]) + 8)
        assert al.stats()["general_pairs"] == len(b)
    finally:
        al.close()
    assert_same(got, ref, b, f"{pen}")
