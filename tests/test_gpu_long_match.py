"""GPU parity of the long pairs' kernels on near-exact reads: matches around what a
lane and a wavefront take at a time, ends of the matrix amid them, repeats in which
many diagonals match far at once, offsets doubled and as they are, few pairs and
enough to fill the chip, exact and adaptive.  Integer results: byte-identical to the
oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu


def _seq(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def _edited(rng, p, at, i):
    """`p` with one edit at `at`, of the kind `i`."""
    if i % 3 == 0:
        base = np.frombuffer(b"ACGT"[(b"ACGT".index(bytes([p[at]])) + 1) % 4:][:1], np.uint8)
        return np.concatenate([p[:at], base, p[at + 1:]])
    if i % 3 == 1:
        return np.concatenate([p[:at], p[at + 1:]])
    return np.concatenate([p[:at], _seq(rng, 1), p[at:]])


def _pairs(rng, longest):
    pairs = []
    for i, run in enumerate((14, 15, 16, 30, 31, 32, 62, 63, 64, 127, 128, 254, 255, 256, 257, 286, 287, 511, 512,
                             1278, 1279, 1280, 1281, 2302, 2303, 2304, 2305)):
        p = _seq(rng, 2500 + 37 * i)
        t = _edited(rng, p, run, i)  # from the front, from the back, and from an edit on
        t = _edited(rng, t, len(t) - 1 - run, i + 1)
        pairs += [(p, t), (t[:run + 1300], p)]
    for n in (2450, 3000, longest):
        p = _seq(rng, n)
        pairs += [(p, p), (p, p[:-1]), (p[255:], p), (p, _edited(rng, p, n // 2, 0)),
                  (p, _edited(rng, _edited(rng, p, n // 4, 1), n // 2, 2))]
    for unit in (1, 2, 7, 33):  # at a period's distance every diagonal matches to the end
        r = np.tile(_seq(rng, unit), 2600 // unit + 1)
        pairs += [(r[:2500], r[:2560]), (r[:2561], r[3:2500]), (r[:2500], _edited(rng, r[:2500], 1300, 0))]
    return [(bytes(p), bytes(t)) for p, t in pairs]


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
@pytest.mark.parametrize("heur", [None, (10, 50), (10, 300)])
@pytest.mark.parametrize("longest,copies", [(16383, 1), (17000, 1), (6000, 9)])
def test_long_matches(oracle_lib, synth_lib, longest, copies, pen, heur):
    import paper_2204_02085_amd as wfa

    pairs = _pairs(np.random.default_rng(31), longest)
    small = synth_lib.from_pairs(pairs)
    ref = oracle_lib.align_batch(small, pen, cigar=True, threads=8, adaptive=heur)
    b = synth_lib.from_pairs(pairs * copies)
    say(f"case: long matches to {longest}, penalties {pen}, heuristic {heur}, {len(b)} pairs")
    al = wfa.Aligner(0)
    try:
        if heur:
            al.set_heuristic(*heur)
        sc, runs, off = al.align(b, pen, capacity=copies * int(ref.offsets[-1]) + 8)
        for c in range(copies):
            lo, hi = c * len(small), (c + 1) * len(small)
            at = off[lo:hi + 1]
            assert_same((sc[lo:hi], runs[at[0]:at[-1]], at - at[0]), ref, small, f"{pen} {heur} copy {c}")
        sc, _, _ = al.align(b, pen, cigar=False)
        assert np.array_equal(sc, np.tile(ref.scores, copies))
    finally:
        al.close()
