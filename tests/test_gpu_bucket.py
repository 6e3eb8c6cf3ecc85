"""Which batches are sorted by length and length difference before the first pass
(the plan as the library reports it on stderr), with results byte-identical to the
oracle either way."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu


@pytest.fixture()
def aligner():
    import paper_2204_02085_amd as wfa

    al = wfa.Aligner(0)
    yield al
    al.close()


def _check(al, oracle_lib, b, pen, capfd, monkeypatch, kernel, bucketed):
    monkeypatch.setenv("WFA_DEBUG", "1")
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8)
    capfd.readouterr()
    got = al.align(b, pen, capacity=int(ref.offsets[-1]) + 8)
    err = capfd.readouterr().err
    plan = [line for line in err.splitlines() if line.startswith("libwfa plan")]
    assert plan and kernel in plan[0], err
    assert plan[0].endswith(", bucketed") == bucketed, plan[0]
    assert_same(got, ref, b, f"{len(b)} pairs, {pen}")


# 256 compute units: lane groups with rows in LDS from 8 pairs per CU on, even lengths too
@pytest.mark.parametrize("count,bucketed", [(2047, False), (2048, True)])
def test_short_kernel(aligner, oracle_lib, synth_lib, capfd, monkeypatch, count, bucketed):
    say(f"case: bucketing of the short kernel, {count} pairs")
    b = synth_lib.workload("pairs100_e4_5m", count, first=5)
    _check(aligner, oracle_lib, b, (5, 7, 1), capfd, monkeypatch, "short kernel", bucketed)


# 256 compute units: the lane kernel past 2048 pairs per CU, from one read in 128
# with a gap of four bases on
@pytest.mark.parametrize("count,gapped,bucketed", [(524_289, 4097, True), (524_289, 4096, False),
                                                   (524_288, 8000, False)])
def test_lane_kernel_gaps(aligner, oracle_lib, synth_lib, capfd, monkeypatch, count, gapped, bucketed):
    say(f"case: bucketing of the lane kernel, {count} pairs, {gapped} with a gap")
    rng = np.random.default_rng(9)
    L = 40
    pat = rng.choice(np.frombuffer(b"ACGT", np.uint8), (count, L))
    txt = pat.copy()
    txt[:, 7] = pat[:, 8]  # a substitution in three of four reads
    lens = np.full(count, L, np.uint32)
    lens[rng.permutation(count)[:gapped]] = L - 4  # four bases at the end
    off = np.arange(count, dtype=np.uint64) * L
    b = synth_lib.Batch(np.ascontiguousarray(pat).reshape(-1), np.ascontiguousarray(txt).reshape(-1), off,
                        np.full(count, L, np.uint32), off, lens)
    _check(aligner, oracle_lib, b, (4, 6, 2), capfd, monkeypatch, "lane kernel", bucketed)
