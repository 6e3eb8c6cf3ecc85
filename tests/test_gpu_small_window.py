"""The band kernel's first window for small batches: wide enough that no pair of
moderate divergence needs a further pass, and the narrow one again once a batch
fills the chip.  Scores, runs and offsets byte-identical to the oracle."""
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


# 256 compute units of four SIMDs: two pairs per wavefront in the window of 128
# diagonals, four in that of 64
@pytest.mark.parametrize("count,window", [(1, 128), (18, 128), (2048, 128), (2049, 64), (4096, 64), (4097, 32)])
@pytest.mark.parametrize("pen", [(4, 6, 2), (2, 3, 1), (1, 0, 1)])
def test_window(aligner, oracle_lib, synth_lib, count, window, pen):
    b = synth_lib.generate(synth_lib.uneven(154, 323, 0.0, 0.05), 77, count)
    assert int(np.maximum(b.p_len, b.t_len).max()) <= 400
    say(f"case: small batch, {count} pairs, penalties {pen}")
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=8)
    got = aligner.align(b, pen, capacity=int(ref.offsets[-1]) + 8)
    st = aligner.stats()
    assert st["window"] == window
    if window == 128:
        assert st["requeued"] == 0 and st["cascade_window"] == 0
    assert_same(got, ref, b, f"{count} pairs")
    sc, _, _ = aligner.align(b, pen, cigar=False)
    assert np.array_equal(sc, ref.scores)


def test_ends_free(aligner, oracle_lib, synth_lib):
    """Free ends wider than the narrow window's slack."""
    ends = (20, 20, 20, 20)
    b = synth_lib.generate(synth_lib.fixed(250, 8), 5, 64)
    say("case: small batch, free ends")
    aligner.set_ends_free(*ends)
    ref = oracle_lib.align_batch(b, (4, 6, 2), cigar=True, threads=8, ends=ends)
    got = aligner.align(b, (4, 6, 2), capacity=int(ref.offsets[-1]) + 8)
    assert aligner.stats()["window"] == 128
    assert_same(got, ref, b, "free ends")


@pytest.mark.parametrize("cap", [8, 30, 90])
def test_step_cap(aligner, oracle_lib, synth_lib, cap):
    """What a step cap hands over is held by the same window without it: no pair goes
    on to the kernels for long pairs."""
    b = synth_lib.generate(synth_lib.uneven(154, 323, 0.0, 0.05), 78, 1000)
    say(f"case: small batch, step cap {cap}")
    ref = oracle_lib.align_batch(b, (4, 6, 2), cigar=True, threads=8)
    aligner.set_options(step_cap=cap)
    got = aligner.align(b, (4, 6, 2), capacity=int(ref.offsets[-1]) + 8)
    st = aligner.stats()
    assert st["window"] == 128 and st["step_cap"] == cap and st["general_pairs"] == 0
    assert (st["requeued"] > 0) == (cap <= 30)
    assert_same(got, ref, b, f"cap {cap}")
