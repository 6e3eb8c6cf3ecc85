"""GPU parity of the front kernel's large batches, which go in two parts on three
streams: around the number of pairs where that begins, with an arena that grows
between the parts, that takes a part in several rounds and that holds few pairs, and
with enough pairs that the second part follows the first on its stream.  Score-only
too.  Integer results: byte-identical to the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu
GENERAL = 3  # WFA_SCHED_GENERAL: pairs of any length on the front kernel


def _check(oracle_lib, synth_lib, spec, count, budget, calls, pen=(4, 6, 2)):
    import paper_2204_02085_amd as wfa

    b = synth_lib.generate(spec, 900 + count, count)
    say(f"case: front kernel in parts, {count} pairs, budget {budget >> 20} MiB")
    ref = oracle_lib.align_batch(b, pen, cigar=True, threads=16)
    cap = int(ref.offsets[-1]) + 8
    al = wfa.Aligner(0, hbm_budget_bytes=budget)
    try:
        al.set_options(schedule=GENERAL)
        for call in range(calls):
            say(f"  call {call}")
            assert_same(al.align(b, pen, capacity=cap), ref, b, f"{count} pairs, call {call}")
            sc, _, _ = al.align(b, pen, cigar=False)
            assert np.array_equal(sc, ref.scores)
        assert al.stats()["general_pairs"] == count
    finally:
        al.close()


# 256 compute units: two parts past 8 pairs per unit, the first part 2 per unit
@pytest.mark.parametrize("count", [2048, 2049, 2600])
def test_first_call_grows_the_arena(oracle_lib, synth_lib, count):
    """A new context: the first part sizes the arena, the second outgrows it; then
    again with the arena as it is."""
    _check(oracle_lib, synth_lib, synth_lib.long_reads(300, 1200, 0.04, 0.10), count, 0, 2)


@pytest.mark.parametrize("mib", [24, 64, 160])
def test_arena_in_rounds(oracle_lib, synth_lib, mib):
    """Budgets whose arena holds a few pairs, the first part, most of both."""
    _check(oracle_lib, synth_lib, synth_lib.long_reads(300, 1200, 0.04, 0.10), 2300, mib << 20, 2)


def test_many_pairs(oracle_lib, synth_lib):
    """Past 64 pairs per unit, where the second part follows the first on its stream."""
    _check(oracle_lib, synth_lib, synth_lib.uneven(40, 400, 0.0, 0.08), 16_500, 0, 2)
    _check(oracle_lib, synth_lib, synth_lib.uneven(40, 400, 0.0, 0.08), 16_500, 48 << 20, 1, (2, 3, 1))
