"""GPU parity of the one-pair-per-lane kernel on reads with one longer gap: end
diagonals past the narrow form's, to the last one that the step cap can reach.
Reads that the cap holds finish in the first pass, and a batch keeps to the narrow
form where such reads are rare among pairs a few bases apart.  Integer results:
byte-identical to the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu
PEN = (4, 6, 2)


def _seq(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def _pair(rng, gap, subs):
    """100 bases with a gap of `gap` bases in the text (below 0: in the pattern) and
    `subs` substitutions."""
    p = _seq(rng, 100)
    at = int(rng.integers(0, 100 - abs(gap)))
    t = np.delete(p, slice(at, at + abs(gap)))
    for i in rng.choice(len(t), subs, replace=False):
        t[i] = b"ACGT"[(b"ACGT".index(bytes([t[i]])) + 1) % 4]
    return (bytes(p), bytes(t)) if gap > 0 else (bytes(t), bytes(p))


def _gapped(rng, cap, count):
    """Pairs of at most `cap` steps: a gap of g bases is g + 3 of them, a substitution 2."""
    pairs = []
    for i in range(count):
        g = int(rng.integers(1, cap - 2))
        pairs.append(_pair(rng, g if i & 1 else -g, (cap - g - 3) // 2))
    return pairs


def _aligned(al, b, cap, cigar, packed):
    import paper_2204_02085_amd as wfa

    if not packed:
        return al.align(b, PEN, cigar=cigar, capacity=cap)
    pat, txt, desc = al.to_device_packed(b)
    scores, runs, off = al.alloc_outputs(len(b), cap, cigar)
    need = al.align_device(pat, txt, desc, len(b), scores, runs, off, PEN, cigar=cigar,
                           encoding=wfa.WFA_PACKED2)
    if not cigar:
        return scores.cpu().numpy(), None, None
    return (scores.cpu().numpy(), runs[:need].cpu().numpy().view(np.uint32),
            off.cpu().numpy().astype(np.uint64))


@pytest.fixture()
def aligner():
    import paper_2204_02085_amd as wfa

    al = wfa.Aligner(0)
    yield al
    al.close()


@pytest.mark.parametrize("cap", [8, 16])
@pytest.mark.parametrize("cigar", [True, False])
@pytest.mark.parametrize("packed", [True, False])
def test_gapped_reads_stay(aligner, oracle_lib, synth_lib, cap, cigar, packed):
    rng = np.random.default_rng(cap)
    b = synth_lib.from_pairs(_gapped(rng, cap, 5000))
    say(f"case: gapped reads, cap {cap}, cigar {cigar}, packed {packed}")
    ref = oracle_lib.align_batch(b, PEN, cigar=cigar, threads=8)
    assert int(ref.scores.max()) <= 2 * cap
    aligner.set_options(lane_kernel=1, step_cap=cap)
    got = _aligned(aligner, b, len(b) * 40, cigar, packed)
    st = aligner.stats()
    assert st["lane_kernel"] == 1 and st["requeued"] == 0
    assert_same(got, ref, b, f"cap {cap}")


def test_rare_among_reads_of_several_edits(aligner, oracle_lib, synth_lib):
    """One gap of nine bases in 5000 pairs, most of them two or three bases apart:
    the narrow form, which hands that pair over."""
    rng = np.random.default_rng(3)
    pairs = [_pair(rng, int(rng.integers(2, 4)), 2) for _ in range(4999)]
    pairs.insert(1234, _pair(rng, 9, 0))
    b = synth_lib.from_pairs(pairs)
    say("case: one gapped read among reads of several edits")
    ref = oracle_lib.align_batch(b, PEN, cigar=True, threads=8)
    aligner.set_options(lane_kernel=1)
    got = _aligned(aligner, b, len(b) * 40, True, True)
    st = aligner.stats()
    assert st["lane_kernel"] == 1 and st["requeued"] == 1
    assert_same(got, ref, b, "rare")
