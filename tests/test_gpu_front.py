"""GPU parity of the front kernel at its edges: lengths around what 16-bit
offsets hold doubled and as they are, row widths around the forms' (blocks per
wavefront, diagonals per lane, the widest), gaps the bound's band cannot see
across, empty sequences, batches that fill the chip and that do not, and an
arena that takes the batch in several parts.  Integer results: byte-identical
to the oracle."""
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
    yield
    aligner.set_options()


def _seq(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def _noisy(rng, p, rate):
    t = p[rng.random(len(p)) >= rate / 2]
    hit = rng.random(len(t)) < rate / 2
    return np.where(hit, _seq(rng, len(t)), t).astype(np.uint8)


def _check(aligner, oracle_lib, synth_lib, pairs, pen, label):
    b = synth_lib.from_pairs([(bytes(p), bytes(t)) for p, t in pairs])
    say(f"case: front {label}, penalties {pen}, {len(b)} pairs")
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8)
    assert_same(aligner.align(b, pen, capacity=int(ref.offsets[-1]) + 8), ref, b, label)
    sc, _, _ = aligner.align(b, pen, cigar=False)
    assert np.array_equal(sc, ref.scores), label
    assert aligner.stats()["general_pairs"] > 0


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
def test_lengths(aligner, oracle_lib, synth_lib, pen):
    rng = np.random.default_rng(5)
    pairs = [(_seq(rng, 3000), b""), (b"", _seq(rng, 2500)), (b"", b""), (b"A", b"C")]
    for n in (2401, 16382, 16383, 16384, 32765, 32766, 32767, 33000):
        p = _seq(rng, n)
        pairs += [(p, p), (p, np.delete(p, [n // 3, n // 2])), (_noisy(rng, p, 0.004), p)]
    _check(aligner, oracle_lib, synth_lib, pairs, pen, "lengths")


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
def test_widths_and_gaps(aligner, oracle_lib, synth_lib, pen):
    """Unrelated pairs (rows as wide as both sequences), and a gap of 70 to
    600 bases in either sequence, early and late."""
    rng = np.random.default_rng(6)
    pairs = [(_seq(rng, a), _seq(rng, b)) for a, b in
             ((1000, 1040), (1020, 1030), (1023, 1024), (1024, 1025), (1500, 900), (2000, 2100),
              (3000, 1500), (2600, 2600), (40, 2500), (2500, 3))]
    for gap in (70, 130, 600):
        p = _seq(rng, 3000)
        t = _noisy(rng, p, 0.05)
        for at in (200, 2500):
            pairs += [(p, np.delete(t, slice(at, at + gap))), (np.delete(p, slice(at, at + gap)), t)]
        both = np.concatenate([t[:700], _seq(rng, gap), t[700:2000], t[2000 + gap:]])
        pairs.append((p, both))
    _check(aligner, oracle_lib, synth_lib, pairs, pen, "widths")


def test_many_pairs(aligner, oracle_lib, synth_lib):
    """More pairs than compute units: two blocks per wavefront, launches by
    workgroup size; the general schedule takes short pairs the same way."""
    rng = np.random.default_rng(7)
    pairs = []
    for n in [50, 300, 900, 1500, 2500] * 80:
        p = _seq(rng, int(n + rng.integers(0, 60)))
        pairs.append((p, _noisy(rng, p, 0.09)))
    pairs += [(_seq(rng, 1800), _seq(rng, 1700)) for _ in range(8)]
    _check(aligner, oracle_lib, synth_lib, pairs, (4, 6, 2), "many")
    aligner.set_options(schedule=3)
    _check(aligner, oracle_lib, synth_lib, pairs[:300], (4, 6, 2), "many, general schedule")


def test_small_arena(oracle_lib, synth_lib):
    """A budget that holds the records of a few pairs at a time."""
    import paper_2204_02085_amd as wfa

    rng = np.random.default_rng(8)
    pairs = []
    for _ in range(300):
        p = _seq(rng, 2600)
        pairs.append((p, _noisy(rng, p, 0.08)))
    al = wfa.Aligner(0, hbm_budget_bytes=64 << 20)
    try:
        _check(al, oracle_lib, synth_lib, pairs, (4, 6, 2), "small arena")
    finally:
        al.close()
