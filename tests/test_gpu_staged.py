"""ASCII batches packed by the first pass as it stages them, at the batch sizes
where the kernels change (256 pairs: one launch for offsets and runs; 64 pairs
per CU: one lane per pair; 256 per CU: uneven batches in buckets): unaligned
byte offsets and lower case against the oracle, the same pairs as packed words,
and the lowest bad pair whichever pass reads it.  Integer results: identical."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu
PEN = (4, 6, 2)
CUS = 256


@pytest.fixture(scope="module")
def wfa():
    import paper_2204_02085_amd as w

    return w


@pytest.fixture(scope="module")
def aligner(wfa):
    al = wfa.Aligner(0)
    yield al
    al.close()


def _pairs(synth_lib, n, uneven):
    rng = np.random.default_rng(n)
    b = synth_lib.workload("pairs100_e4_5m", min(n, 3000), first=5)
    base = [b.pair(i) for i in range(len(b))]
    base[: min(40, n)] = synth_lib.random_pairs(rng, min(40, n), 126)
    base = [(p[:127], t[:127]) for p, t in base]
    pairs = [base[i % len(base)] for i in range(n)]
    if uneven:  # lengths past the lane kernel's, and a pair for the last kernels
        pairs = [(p * (1 + i % 3), t * (1 + i % 3)) for i, (p, t) in enumerate(pairs)]
        pairs[n // 2] = synth_lib.random_pairs(rng, 1, 900, related=False)[0]
    return pairs


def _mixed_case(pairs):
    return [(p.lower() if i % 3 else p, t.lower() if i % 2 else t) for i, (p, t) in enumerate(pairs)]


@pytest.mark.parametrize("uneven", [False, True])
@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 64 * CUS, 64 * CUS + 1, 256 * CUS, 256 * CUS + 1])
def test_staged_ascii(aligner, oracle_lib, synth_lib, n, uneven):
    say(f"case: staged ASCII, {n} pairs, uneven {uneven}")
    pairs = _pairs(synth_lib, n, uneven)
    b = synth_lib.from_pairs(pairs)
    ref = oracle_lib.align_batch(b, PEN, cigar=True, threads=8)
    low = synth_lib.from_pairs(_mixed_case(pairs))
    cap = len(ref.runs)
    for _ in range(2):  # the second call starts from the first one's plan
        assert_same(aligner.align(low, PEN, capacity=cap), ref, b, f"{n} {uneven}")
    sc, _, _ = aligner.align(low, PEN, cigar=False)
    assert np.array_equal(sc, ref.scores)


@pytest.mark.parametrize("n", [300, 64 * CUS + 1])
def test_lowest_bad_pair(aligner, synth_lib, wfa, n):
    """Bad bytes in pairs the first pass reads, hands on unread (900 bases), or
    hands on after reading (unrelated sequences); each order of the two."""
    rng = np.random.default_rng(3)
    good = _pairs(synth_lib, n, False)
    far = synth_lib.random_pairs(rng, 1, 120, related=False)[0]
    long = (b"ACGT" * 600, b"ACGA" * 600)

    def spoil(pair, side, at):
        p = [bytearray(pair[0]), bytearray(pair[1])]
        p[side][at % len(p[side])] = ord("N")
        return bytes(p[0]), bytes(p[1])

    plain = good[50]
    for first, second in ((plain, long), (long, plain), (far, plain), (long, far), (far, long)):
        for side, at in ((0, 0), (1, -1)):
            pairs = list(good)
            pairs[n // 3] = spoil(first, side, at)
            pairs[n // 3 + 7] = spoil(second, 1 - side, at)
            b = synth_lib.from_pairs(pairs)
            say(f"case: bad bytes, {n} pairs, lengths {len(first[0])} before {len(second[0])}, side {side}")
            with pytest.raises(wfa.WFAError) as ei:
                aligner.align(b, PEN)
            assert ei.value.status == wfa.WFA_E_ALPHABET and ei.value.bad == n // 3
    # only a pair that the first pass never reads
    pairs = list(good)
    pairs[n - 2] = spoil(long, 1, 2000)
    with pytest.raises(wfa.WFAError) as ei:
        aligner.align(synth_lib.from_pairs(pairs), PEN)
    assert ei.value.bad == n - 2
    aligner.align(synth_lib.from_pairs(good), PEN)  # and the context goes on
