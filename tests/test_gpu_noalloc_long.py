"""The allocation-free entry point, and a small budget, on batches of many short
reads and a few long pairs, which all go to the kernels for long pairs: calls that
hold the limit of the entry point are not refused for want of memory.  Results equal
the oracle's byte for byte."""
import ctypes

import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu
PEN = (4, 6, 2)


def _mixed(synth_lib, count, length, longest):
    """`count` reads of `length` bases and (unless 0) one pair of `longest`."""
    b = synth_lib.generate(synth_lib.fixed(length, 4), 3, count)
    if not longest:
        return b
    c = synth_lib.generate(synth_lib.fixed(longest, longest // 20), 4, 1)
    return synth_lib.Batch(
        np.concatenate([b.patterns, c.patterns]), np.concatenate([b.texts, c.texts]),
        np.concatenate([b.p_off, c.p_off + np.uint64(len(b.patterns))]), np.concatenate([b.p_len, c.p_len]),
        np.concatenate([b.t_off, c.t_off + np.uint64(len(b.texts))]), np.concatenate([b.t_len, c.t_len]))


@pytest.mark.parametrize("heur", [None, (10, 50)])
@pytest.mark.parametrize("count,length,longest", [(200_000, 100, 2500), (262_143, 100, 2500), (250_000, 100, 0),
                                                  (100_000, 127, 20_000)])
def test_noalloc(oracle_lib, synth_lib, heur, count, length, longest):
    import torch

    import paper_2204_02085_amd as wfa

    b = _mixed(synth_lib, count, length, longest)
    say(f"case: noalloc, {count} reads of {length}, one of {longest}, heuristic {heur}")
    ref = oracle_lib.align_batch(b, PEN, cigar=True, threads=16, adaptive=heur)
    al = wfa.Aligner(0)
    try:
        al.set_heuristic(*(heur or ()))
        pat, txt, pairs = al.to_device(b)
        scores, runs, off = al.alloc_outputs(len(b), int(ref.offsets[-1]))
        need, bad = ctypes.c_size_t(0), ctypes.c_int64(-1)
        rc = wfa.wfa_align_batch_noalloc(
            al.ctx, pat.data_ptr(), txt.data_ptr(), pairs.data_ptr(), len(b), wfa.WFA_ASCII,
            wfa.wfa_penalties(*PEN), wfa.WFA_CIGAR, scores.data_ptr(), runs.data_ptr(), runs.numel(),
            off.data_ptr(), ctypes.byref(need), ctypes.byref(bad), None)
        torch.cuda.synchronize()
        assert rc == wfa.WFA_OK, (rc, bad.value)
        got = (scores.cpu().numpy(), runs[: need.value].cpu().numpy().view(np.uint32),
               off.cpu().numpy().view(np.uint64))
    finally:
        al.close()
    assert_same(got, ref, b, "noalloc")


@pytest.mark.parametrize("heur", [None, (10, 50)])
@pytest.mark.parametrize("mib", [6, 12, 24])
def test_small_budget(oracle_lib, synth_lib, heur, mib):
    """Budgets that these kernels run out of in some place: the call succeeds where
    the general kernel's does."""
    import paper_2204_02085_amd as wfa

    b = _mixed(synth_lib, 20_000, 60, 2500)
    say(f"case: budget of {mib} MiB, heuristic {heur}")
    ref = oracle_lib.align_batch(b, PEN, cigar=True, threads=16, adaptive=heur)
    results = []
    for options in ({}, {"general_checkpoint": -1}):
        al = wfa.Aligner(0, hbm_budget_bytes=mib << 20)
        try:
            al.set_options(**options)
            al.set_heuristic(*(heur or ()))
            results.append(al.align(b, PEN, capacity=int(ref.offsets[-1])))
        except wfa.WFAError as err:
            assert err.status == wfa.WFA_E_NOMEM
            results.append(None)
        finally:
            al.close()
    say(f"  default {results[0] is not None}, general kernel {results[1] is not None}")
    assert results[0] is not None or results[1] is None
    for got in results:
        if got is not None:
            assert_same(got, ref, b, f"{mib} MiB")
