"""The workgroup-per-pair kernel itself, for penalties and pairs that kernels with
rows in registers take otherwise: an option of its memory sends every pair past them
(the kernel reports its pairs on stderr).  Each workgroup size score-only, the
penalty sets of those kernels in both modes, the heuristic.  Integer results:
byte-identical to the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu
GENERAL = 3  # WFA_SCHED_GENERAL


@pytest.fixture(scope="module")
def aligner():
    import paper_2204_02085_amd as wfa

    al = wfa.Aligner(0)
    yield al
    al.close()


@pytest.fixture(autouse=True)
def _options(aligner, monkeypatch):
    monkeypatch.setenv("WFA_DEBUG", "1")
    aligner.set_options(schedule=GENERAL, general_checkpoint=-1)
    yield
    aligner.set_options()
    aligner.set_heuristic()


def _ran(capfd, count):
    err = capfd.readouterr().err
    assert f"libwfa general: {count} pairs" in err, err


# 256 compute units: 1024 threads per pair up to 8 pairs per unit, 512 up to 24, 256 beyond
@pytest.mark.parametrize("count", [400, 3000, 7000])
def test_workgroup_sizes_score_only(aligner, oracle_lib, synth_lib, capfd, count):
    b = synth_lib.generate(synth_lib.long_reads(601, 1200, 0.02, 0.08), 5100 + count, count)
    assert int(np.maximum(b.p_len, b.t_len).min()) > 600
    say(f"case: general kernel, {count} pairs of 601-1200 bp, score only")
    ref = oracle_lib.align_batch(b, (4, 6, 2), cigar=False, threads=16)
    capfd.readouterr()
    sc, _, _ = aligner.align(b, (4, 6, 2), cigar=False)
    _ran(capfd, count)
    assert np.array_equal(sc, ref.scores)


@pytest.mark.parametrize("pen", [(4, 6, 2), (1, 0, 1), (2, 3, 1)])
@pytest.mark.parametrize("heur", [None, (10, 50)])
def test_penalty_sets(aligner, oracle_lib, synth_lib, capfd, pen, heur):
    say(f"case: general kernel, penalties {pen}, heuristic {heur}")
    b = synth_lib.workload("uneven50_300_2m", 1500, first=4321)
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8, adaptive=heur)
    aligner.set_heuristic(*(heur or ()))
    capfd.readouterr()
    got = aligner.align(b, pen, capacity=int(ref.offsets[-1]) + 8)
    _ran(capfd, len(b))
    assert_same(got, ref, b, f"{pen}")
    sc, _, _ = aligner.align(b, pen, cigar=False)
    _ran(capfd, len(b))
    assert np.array_equal(sc, ref.scores)
