"""GPU parity of the band kernel at the edges where it can go wrong: pairs
whose score lies at, one below and one above what a band is exact for (the
excursion to the band's edge and back), lengths around the words and the
windows' length classes, free ends against the band's edge, both launch forms
and both modes.  Integer results: byte-identical to the oracle."""
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
    aligner.set_ends_free()
    yield
    aligner.set_options()
    aligner.set_ends_free()


def _excursions(rng):
    """Pairs that gain g text bases near the start and lose g (or g - 1, g + 1)
    near the end, g around half of each window, and a few mismatches."""
    pairs = []
    for half in (16, 32, 64):
        for g in range(half - 3, half + 3):
            for back in (g - 1, g, g + 1):
                core = rng.choice(list(b"ACGT"), 150 + half).astype(np.uint8)
                extra = rng.choice(list(b"ACGT"), g).astype(np.uint8)
                tail = rng.choice(list(b"ACGT"), back).astype(np.uint8)
                text = np.concatenate([core[:40], extra, core[40:]])
                pat = np.concatenate([core[:120], tail, core[120:]])
                for mism in range(3):
                    t2 = text.copy()
                    for _ in range(mism):
                        i = int(rng.integers(0, len(t2)))
                        t2[i] = b"ACGT"[(b"ACGT".index(bytes([t2[i]])) + 1) % 4]
                    pairs.append((pat.tobytes(), t2.tobytes()))
                    pairs.append((t2.tobytes(), pat.tobytes()))
    return pairs


def _lengths(synth_lib, rng):
    pairs = [(b"", b""), (b"", b"ACGTACGT"), (b"ACG", b""), (b"A", b"A"), (b"A", b"G")]
    for n in (15, 16, 17, 31, 32, 33, 127, 128, 129, 159, 160, 161):
        p = rng.choice(list(b"ACGT"), n).astype(np.uint8)
        t = np.delete(p, n // 2)
        pairs += [(p.tobytes(), p.tobytes()), (p.tobytes(), t.tobytes()), (t.tobytes(), p.tobytes())]
    pairs += synth_lib.random_pairs(rng, 300, 60)
    pairs += synth_lib.random_pairs(rng, 100, 300)
    pairs += synth_lib.random_pairs(rng, 60, 160, related=False)
    return pairs


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
@pytest.mark.parametrize("ends", [None, (5, 5, 5, 5), (0, 9, 13, 0)])
def test_band_edges(aligner, oracle_lib, synth_lib, pen, ends):
    rng = np.random.default_rng(11)
    b = synth_lib.from_pairs(_excursions(rng) + _lengths(synth_lib, rng))
    kw = {"ends": ends} if ends else {}
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8, **kw)
    if ends:
        aligner.set_ends_free(*ends)
    for schedule in (0, 1):  # persistent, plain
        say(f"case: band edges, penalties {pen}, ends {ends}, schedule {schedule}")
        aligner.set_options(schedule=schedule, lane_kernel=-1)
        assert_same(aligner.align(b, pen), ref, b, f"{pen} {ends} {schedule}")
        sc, _, _ = aligner.align(b, pen, cigar=False)
        assert np.array_equal(sc, ref.scores)


@pytest.mark.parametrize("top", [400, 401, 1200, 1201, 2400])
def test_band_length_classes(aligner, oracle_lib, synth_lib, top):
    """The largest length of a batch picks the first window; short and long
    pairs share it, at error rates that stay in and run past it."""
    say(f"case: band length class {top}")
    rng = np.random.default_rng(top)
    pairs = [(b"A" * top, b"A" * top), (b"C" * top, b"C" * (top - 7)), (b"", b"T" * 20)]
    for rate in (0.01, 0.04, 0.15):
        p = rng.choice(list(b"ACGT"), top).astype(np.uint8)
        for _ in range(3):
            keep = p[rng.random(top) >= rate / 2]
            t = keep.copy()
            hit = rng.random(len(t)) < rate / 2
            t[hit] = rng.choice(list(b"ACGT"), int(hit.sum())).astype(np.uint8)
            pairs.append((p.tobytes(), t.tobytes()))
    pairs += synth_lib.random_pairs(rng, 40, 200)
    b = synth_lib.from_pairs([(p[:top], t[:top]) for p, t in pairs])
    ref = oracle_lib.align_batch(b, (4, 6, 2), cigar=True, threads=8)
    assert_same(aligner.align(b, (4, 6, 2)), ref, b, f"class {top}")
