"""GPU parity of the adaptive kernel on pairs that need more steps than the first
records hold, or more diagonals than the first window: they are aligned again with
longer records in a wider one, not by the general kernel (the count that the library
reports on stderr).  Integer results: byte-identical to the oracle under the same
heuristic."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu
HEUR = (10, 50)


def _left(err):
    """Pairs the adaptive kernel left for the general kernel."""
    line = [x for x in err.splitlines() if x.startswith("libwfa adaptive:")][-1]
    return int(line.split()[2])


def _seq(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def _divergent(rng, n, rate):
    """A sequence and one with `rate` of its bases replaced, deleted or preceded by
    another, a third each."""
    p = _seq(rng, n)
    r = rng.random(n) * 3
    t = np.where(r < rate, _seq(rng, n), p)
    t = np.stack([_seq(rng, n), t], 1)
    keep = np.stack([(r >= 1) & (r < 1 + rate), ~((r >= 2) & (r < 2 + rate))], 1)
    return p, t[keep].astype(np.uint8)


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
@pytest.mark.parametrize("budget", [0, 48 << 20])
def test_divergent(oracle_lib, synth_lib, capfd, monkeypatch, pen, budget):
    import paper_2204_02085_amd as wfa

    rng = np.random.default_rng(41)
    pairs = [_divergent(rng, n, rate) for n in (100, 700, 1500, 2500) for rate in (0.05, 0.35, 0.5)
             for _ in range(8)]
    pairs += [_divergent(rng, 17000, 0.002), _divergent(rng, 60, 0.8)]
    b = synth_lib.from_pairs([(bytes(p), bytes(t)) for p, t in pairs])
    say(f"case: adaptive kernel, divergent pairs, penalties {pen}, budget {budget}")
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8, adaptive=HEUR)
    monkeypatch.setenv("WFA_DEBUG", "1")
    al = wfa.Aligner(0, hbm_budget_bytes=budget)
    try:
        al.set_heuristic(*HEUR)
        capfd.readouterr()
        got = al.align(b, pen, capacity=int(ref.offsets[-1]) + 8)
        err = capfd.readouterr().err
        sc, _, _ = al.align(b, pen, cigar=False)
    finally:
        al.close()
    assert _left(err) == 0
    assert_same(got, ref, b, f"{pen}")
    assert np.array_equal(sc, ref.scores)


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
@pytest.mark.parametrize("mdt,left", [(50, 0), (500, 11)])
def test_outgrown(oracle_lib, synth_lib, capfd, monkeypatch, pen, mdt, left):
    """Gaps of hundreds of bases, unrelated pairs and a short text against a long
    pattern; with a threshold that drops next to nothing, ranges that span both sequences:
    about the first window's 256 diagonals, four blocks' 512 and the wide window's
    1024 (ten of them are margins; pairs past these are left)."""
    import paper_2204_02085_amd as wfa

    rng = np.random.default_rng(43)
    if mdt == 50:
        pairs = [(_seq(rng, n), _seq(rng, n - 30)) for n in (600, 2000) for _ in range(3)]
        for gap in (200, 320, 600):
            p, t = _divergent(rng, 2200, 0.06)
            pairs += [(p, np.delete(t, slice(700, 700 + gap))), (np.delete(p, slice(700, 700 + gap)), t)]
        pairs += [(_seq(rng, 900), _seq(rng, 5)), (_seq(rng, 5), _seq(rng, 900))]
    else:
        pairs = [(_seq(rng, total // 2), _seq(rng, total - total // 2))
                 for total in [*range(240, 252), *range(495, 507), *range(1003, 1014), *range(1014, 1025)]]
    b = synth_lib.from_pairs([(bytes(p), bytes(t)) for p, t in pairs])
    say(f"case: adaptive kernel, wide ranges, penalties {pen}, threshold {mdt}")
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8, adaptive=(10, mdt))
    monkeypatch.setenv("WFA_DEBUG", "1")
    al = wfa.Aligner(0)
    try:
        al.set_heuristic(10, mdt)
        capfd.readouterr()
        got = al.align(b, pen, capacity=int(ref.offsets[-1]) + 8)
        err = capfd.readouterr().err
        sc, _, _ = al.align(b, pen, cigar=False)
    finally:
        al.close()
    say(err)
    assert _left(err) <= left
    assert_same(got, ref, b, f"{pen}")
    assert np.array_equal(sc, ref.scores)


@pytest.mark.parametrize("mdt", [512, 513, 1 << 20])
def test_wide_thresholds(oracle_lib, synth_lib, mdt):
    """Thresholds on either side of what goes to the adaptive kernel at all."""
    import paper_2204_02085_amd as wfa

    rng = np.random.default_rng(47)
    b = synth_lib.from_pairs([tuple(map(bytes, _divergent(rng, n, 0.1))) for n in (90, 800, 1800) for _ in range(4)])
    say(f"case: adaptive kernel, threshold {mdt}")
    ref = oracle_lib.align_batch(b, (4, 6, 2), cigar=True, threads=8, adaptive=(10, mdt))
    al = wfa.Aligner(0)
    try:
        al.set_heuristic(10, mdt)
        assert_same(al.align(b, (4, 6, 2), capacity=int(ref.offsets[-1]) + 8), ref, b, f"{mdt}")
    finally:
        al.close()
