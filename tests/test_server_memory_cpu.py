"""Host memory of the server's workers: what one very large request took is given
back once its results are handed over, and later requests are served as before."""
import numpy as np
import pytest


def _rss():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[1]) * 4096


def _match_executor(b):
    """One match run per pair: the scheduler is what is looked at."""
    n = len(b["pairs"])
    lens = b["pairs"]["p_len"].astype(np.uint32)
    return np.zeros(n, np.int32), lens << 4, np.arange(n + 1, dtype=np.uint64)


@pytest.mark.parametrize("cigar", [True, False])
def test_large_request_is_given_back(synth_lib, cigar):
    import paper_2204_02085_amd as wfa

    n = 40 << 20  # two of these are past what a worker keeps
    srv = wfa.Server(None, streams=1, cigar=cigar, hbm_budget_bytes=1 << 60, executor=_match_executor)
    try:
        small = synth_lib.workload("pairs100_e2_10k", 50)
        tk = srv.submit(small)
        assert srv.poll(tk)["status"] == 0
        srv.release(tk)
        before = _rss()
        seq = np.full(n, ord("A"), np.uint8)
        lens, starts = np.full(2, n, np.uint32), np.zeros(2, np.uint64)
        big = synth_lib.Batch(seq, seq, starts, lens, starts, lens)
        tk = srv.submit(big)
        res = srv.poll(tk)
        assert res["status"] == 0
        if cigar:
            assert list(res["runs"]) == [n << 4] * 2
        srv.release(tk)
        assert srv.stats()["batches"] == 2
        del seq, big, res
        tk = srv.submit(small)  # (the worker has gone on)
        res = srv.poll(tk)
        assert res["status"] == 0 and len(res["scores"]) == 50
        srv.release(tk)
        assert _rss() - before < 2 * n
    finally:
        srv.close()
