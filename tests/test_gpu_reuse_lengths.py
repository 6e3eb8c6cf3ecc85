"""Calls that reuse the same device buffers for longer reads: the captured graph of
the shorter ones is not replayed on them, so that every pair stays in the first pass
that a fresh context plans, and results are byte-identical to the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu

N = 3000


@pytest.fixture()
def aligner():
    import paper_2204_02085_amd as wfa

    al = wfa.Aligner(0)
    yield al
    al.close()


def _reads(synth_lib, longest, seed):
    """Reads of up to exactly `longest` bases, two edits each."""
    b = synth_lib.generate(synth_lib.fixed(longest - 2, 2), seed, N - 1)
    p = b.pair(0)[0][: longest - 2] + b"AC"
    return synth_lib.from_pairs([b.pair(i) for i in range(N - 1)] + [(p, p)])


def _run(al, bufs, b, pen, packed, cigar):
    import torch

    import paper_2204_02085_amd as wfa

    P, T, D, scores, runs, offsets = bufs
    pat, txt, pairs = al.to_device_packed(b) if packed else al.to_device(b)
    P.view(pat.dtype)[: pat.numel()].copy_(pat.reshape(-1))
    T.view(txt.dtype)[: txt.numel()].copy_(txt.reshape(-1))
    D.copy_(pairs.reshape(-1).view(torch.uint8))
    scores.fill_(-7)
    need = al.align_device(P, T, D, N, scores, runs, offsets, pen, cigar,
                           wfa.WFA_PACKED2 if packed else wfa.WFA_ASCII)
    torch.cuda.synchronize()
    if not cigar:
        return scores.cpu().numpy(), None, None
    return (scores.cpu().numpy(), runs[:need].cpu().numpy().view(np.uint32),
            offsets.cpu().numpy().view(np.uint64))


# lengths on either side of what 32-base words, and offsets of one byte, hold
@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("pen,lengths", [((4, 6, 2), (150, 250, 150)), ((1, 0, 1), (64, 65, 200)),
                                         ((5, 7, 1), (127, 128, 159))])
def test_longer_reads(aligner, oracle_lib, synth_lib, packed, pen, lengths):
    import torch

    import paper_2204_02085_amd as wfa

    cigar = True
    bufs = [torch.zeros(64 * N, dtype=torch.int64, device="cuda") for _ in range(2)]
    bufs.append(torch.zeros(24 * N, dtype=torch.uint8, device="cuda"))
    bufs += aligner.alloc_outputs(N, 200 * N, cigar)
    for i, longest in enumerate(lengths):
        b = _reads(synth_lib, longest, 31 + i)
        assert int(max(b.p_len.max(), b.t_len.max())) == longest
        say(f"case: reused buffers, reads of up to {longest}, penalties {pen}, packed {packed}")
        got = _run(aligner, bufs, b, pen, packed, cigar)
        fresh = wfa.Aligner(0)
        try:
            _run(fresh, bufs, b, pen, packed, cigar)
            assert aligner.stats()["requeued"] == fresh.stats()["requeued"] < N // 4
        finally:
            fresh.close()
        assert_same(got, oracle_lib.align_batch(b, pen, cigar=cigar, threads=8), b, f"{longest}")
