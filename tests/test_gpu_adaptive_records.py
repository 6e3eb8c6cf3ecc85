"""GPU parity of the adaptive kernel on pairs that need more steps than the first
records hold: they are aligned again with longer ones, not by the general kernel
(the count that the library reports on stderr).  Integer results: byte-identical to
the oracle under the same heuristic."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu
HEUR = (10, 50)


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
    assert "libwfa adaptive: 0 pairs left for the general kernel" in err, err
    assert_same(got, ref, b, f"{pen}")
    assert np.array_equal(sc, ref.scores)
