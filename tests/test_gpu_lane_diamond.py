"""GPU parity of the one-pair-per-lane kernel over its diamond of cells: every
mix of up to four edits at the edge of what a step cap allows, end diagonals up to
and past the ones it holds, sequences shorter than the diamond is wide, edits at
both ends, matches around the 15 and 32 bases of its compares.  Integer results:
byte-identical to the oracle."""
import itertools

import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu
PEN = (4, 6, 2)


def _seq(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def _edited(rng, p, edits, at):
    t = p.copy()
    for (kind, length), pos in sorted(zip(edits, at), key=lambda x: -x[1]):
        if kind == "X":
            t[pos] = b"ACGT"[(b"ACGT".index(bytes([t[pos]])) + 1) % 4]
        elif kind == "I":
            t = np.concatenate([t[:pos], _seq(rng, length), t[pos:]])
        else:
            t = np.delete(t, slice(pos, pos + length))
    return t


def _pairs(rng):
    pairs = []
    kinds = [("X", 1), ("I", 1), ("D", 1), ("I", 2), ("D", 3)]
    for r in range(5):  # costs 0 to past 16 steps
        for edits in itertools.combinations_with_replacement(kinds, r):
            p = _seq(rng, int(rng.integers(60, 121)))
            at = np.sort(rng.choice(len(p) - 4, r, replace=False))
            pairs.append((p, _edited(rng, p, edits, at)))
            pairs.append((p, _edited(rng, p, edits, np.arange(r) * 4)))          # at the start
            pairs.append((p, _edited(rng, p, edits, len(p) - 4 - np.arange(r) * 4)))  # at the end
    for length in range(1, 15):  # one gap, and a gap there and back
        p = _seq(rng, 100)
        pairs += [(p, np.delete(p, slice(40, 40 + length))), (np.delete(p, slice(40, 40 + length)), p)]
        t = np.delete(p, slice(30, 30 + length))
        pairs.append((p, np.concatenate([t[:60], _seq(rng, length), t[60:]])))
    for n in (14, 15, 16, 17, 30, 31, 32, 33, 46, 47, 48, 62, 63, 64):  # matches of n bases
        p = _seq(rng, 126)
        at = [n] + ([2 * n + 1] if 2 * n + 1 < 126 else [])
        pairs.append((p, _edited(rng, p, [("X", 1)] * len(at), at)))
    for n in range(13):  # narrower than the diamond
        for m in range(13):
            p = _seq(rng, n)
            t = p[:m] if m <= n else np.concatenate([p, _seq(rng, m - n)])
            pairs += [(p, t), (p, _seq(rng, m))]
    return [(bytes(p), bytes(t)) for p, t in pairs if len(p) <= 127 and len(t) <= 127]


@pytest.mark.parametrize("cap", [8, 16])
@pytest.mark.parametrize("ascii_input", [True, False])
def test_diamond(oracle_lib, synth_lib, cap, ascii_input):
    import paper_2204_02085_amd as wfa

    rng = np.random.default_rng(cap)
    base = _pairs(rng)
    pairs = [base[i] for i in rng.permutation(len(base))] * 3
    b = synth_lib.from_pairs(pairs)
    ref = oracle_lib.align_batch(b, PEN, cigar=True, threads=8)
    say(f"case: lane diamond, cap {cap}, ASCII {ascii_input}, {len(pairs)} pairs")
    al = wfa.Aligner(0)
    try:
        al.set_options(lane_kernel=1, step_cap=cap)
        if ascii_input:
            got = al.align(b, PEN, capacity=len(ref.runs))
            sc = al.align(b, PEN, cigar=False)[0]
        else:
            n = len(pairs)
            pat, txt, desc = al.to_device_packed(b)
            scores, runs, off = al.alloc_outputs(n, len(ref.runs), True)
            need = al.align_device(pat, txt, desc, n, scores, runs, off, PEN, encoding=wfa.WFA_PACKED2)
            got = (scores.cpu().numpy(), runs[:need].cpu().numpy().view(np.uint32),
                   off.cpu().numpy().astype(np.uint64))
            al.align_device(pat, txt, desc, n, scores, penalties=PEN, cigar=False,
                            encoding=wfa.WFA_PACKED2)
            sc = scores.cpu().numpy()
        assert al.stats()["lane_kernel"] == 1 and al.stats()["step_cap"] == cap
    finally:
        al.close()
    assert_same(got, ref, b, f"cap {cap}")
    assert np.array_equal(sc, ref.scores)
