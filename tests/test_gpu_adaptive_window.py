"""GPU parity of the adaptive kernel where its window matters: gaps that widen
the kept ranges past one block of 128 diagonals and past both, thresholds that
drop almost nothing (the general kernel's pairs), 16-bit offsets doubled and
as they are, length differences that pull the window along.  Integer results:
byte-identical to the oracle under the same heuristic."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def aligner():
    import paper_2204_02085_amd as wfa

    al = wfa.Aligner(0)
    yield al
    al.close()


@pytest.fixture(autouse=True)
def _defaults(aligner):
    aligner.set_options()
    aligner.set_heuristic()
    yield
    aligner.set_options()
    aligner.set_heuristic()


def _seq(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def _noisy(rng, p, rate):
    t = p[rng.random(len(p)) >= rate / 2]
    hit = rng.random(len(t)) < rate / 2
    return np.where(hit, _seq(rng, len(t)), t).astype(np.uint8)


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
@pytest.mark.parametrize("heur", [(10, 50), (1, 0), (10, 400), (40, 10)])
def test_windows(aligner, oracle_lib, synth_lib, pen, heur):
    rng = np.random.default_rng(3)
    pairs = [(b"", b""), (b"", _seq(rng, 700)), (_seq(rng, 400), b""), (b"A", b"C"),
             (_seq(rng, 600), _seq(rng, 500))]
    for gap in (20, 60, 90, 150, 320):
        p = _seq(rng, 1800)
        t = _noisy(rng, p, 0.06)
        for at in (100, 1200):
            pairs += [(p, np.delete(t, slice(at, at + gap))), (np.delete(p, slice(at, at + gap)), t)]
        pairs.append((p, np.concatenate([t[:500], _seq(rng, gap), t[500:1200], t[1200 + gap:]])))
    for n in (16383, 16384):
        p = _seq(rng, n)
        pairs += [(p, p), (_noisy(rng, p, 0.01), p)]
    b = synth_lib.from_pairs([(bytes(p), bytes(t)) for p, t in pairs])
    say(f"case: adaptive windows, penalties {pen}, heuristic {heur}, {len(b)} pairs")
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8, adaptive=heur)
    aligner.set_heuristic(*heur)
    assert_same(aligner.align(b, pen, capacity=int(ref.offsets[-1]) + 8), ref, b, f"{pen} {heur}")
    sc, _, _ = aligner.align(b, pen, cigar=False)
    assert np.array_equal(sc, ref.scores)
    assert aligner.stats()["general_pairs"] == len(b)


@pytest.mark.parametrize("heur", [(10, 50), (10, 80)])
def test_every_width(aligner, oracle_lib, synth_lib, heur):
    """Gaps of every length about one block: the kept ranges take every width up
    to it, at both parities, so the window is placed with nothing to spare."""
    rng = np.random.default_rng(29)
    pairs = []
    for gap in range(90, 150):
        p = _seq(rng, 1600)
        t = np.concatenate([p[:700], _seq(rng, gap), p[700:]])
        pairs += [(p, t), (t, p), (_noisy(rng, p, 0.02), t)]
    b = synth_lib.from_pairs([(bytes(p), bytes(t)) for p, t in pairs])
    say(f"case: adaptive windows of every width, heuristic {heur}, {len(b)} pairs")
    ref = oracle_lib.align_batch(b, (4, 6, 2), cigar=True, threads=8, adaptive=heur)
    aligner.set_heuristic(*heur)
    assert_same(aligner.align(b, (4, 6, 2), capacity=int(ref.offsets[-1]) + 8), ref, b, f"{heur}")
