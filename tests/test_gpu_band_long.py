"""GPU parity of the band kernel on middling reads in small batches: the window of 256
diagonals, matches around what its compares and a lane group take at a time, pairs
about the most steps a window holds, free ends, batches about the sizes where the
window changes.  Integer results: byte-identical to the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def aligner():
    import paper_2204_02085_amd as wfa

    al = wfa.Aligner(0)
    yield al
    al.close()


@pytest.fixture(autouse=True)
def _global(aligner):
    aligner.set_ends_free()
    yield
    aligner.set_ends_free()


def _seq(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def _broken(rng, p, gaps):
    """`p` with an edit after every so many matching bases."""
    out, at = [], 0
    for i, g in enumerate(gaps):
        out.append(p[at:at + g])
        at += g
        if at >= len(p):
            break
        kind = i % 3
        if kind == 0:
            out.append(np.frombuffer(bytes([b"ACGT"[(b"ACGT".index(bytes([p[at]])) + 1) % 4]]), np.uint8))
            at += 1
        elif kind == 1:
            at += 1
        else:
            out.append(_seq(rng, 1))
    out.append(p[at:])
    return np.concatenate(out)


def _pairs(rng, longest):
    pairs = [(_seq(rng, longest), b""), (b"", _seq(rng, 700)), (b"", b""), (b"A", b"C")]
    for n in (401, 640, longest):
        p = _seq(rng, n)
        pairs += [(p, p), (p, p[1:]), (p[:-1], p)]
    for run in (14, 15, 16, 30, 31, 32, 33, 46, 47, 48, 62, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024,
                1025, 2047, 2048, 2049):
        p = _seq(rng, longest - 40)
        pairs.append((p, _broken(rng, p, [run] + [run + 1] * (2 if run < 60 else 1))))
    for rate in (0.02, 0.05, 0.08, 0.11, 0.14):  # up to and past the steps of a window
        for n in (420, 700, 900):
            p = _seq(rng, n)
            pairs.append((p, _broken(rng, p, rng.geometric(rate, 400))))
    pairs += [(_seq(rng, 170), _seq(rng, 175)), (_seq(rng, 500), _seq(rng, 260))]
    return [(bytes(p), bytes(t)) for p, t in pairs if len(t) <= longest]


# 256 compute units: past 400 bases two wavefronts per SIMD in the windows of 256 and 128
@pytest.mark.parametrize("count,window", [(100, 256), (2048, 256), (2049, 128), (4096, 128), (4097, 64)])
@pytest.mark.parametrize("pen", [(4, 6, 2), (2, 3, 1), (1, 0, 1)])
@pytest.mark.parametrize("longest,cigar", [(1200, True), (2400, False)])
def test_windows(aligner, oracle_lib, synth_lib, count, window, pen, longest, cigar):
    rng = np.random.default_rng(61)
    pairs = _pairs(rng, longest)
    reads = synth_lib.generate(synth_lib.uneven(100, 300, 0.0, 0.02), 7, count)
    pairs += [reads.pair(i) for i in range(count - len(pairs))]
    b = synth_lib.from_pairs(pairs)
    assert len(b) == count and int(np.maximum(b.p_len, b.t_len).max()) == longest
    say(f"case: band kernel, reads of up to {longest}, {count} pairs, penalties {pen}, cigar {cigar}")
    ref = oracle_lib.align_batch(b, pen, cigar=cigar, threads=8)
    got = aligner.align(b, pen, cigar=cigar, capacity=int(ref.offsets[-1]) + 8 if cigar else None)
    # (past 1200 bases a batch starts with 128 diagonals at any size)
    assert aligner.stats()["window"] == (window if longest <= 1200 else max(window, 128))
    assert_same(got, ref, b, f"{count} pairs")


@pytest.mark.parametrize("free", [10, 50])
def test_free_ends(aligner, oracle_lib, synth_lib, free):
    rng = np.random.default_rng(67)
    pairs = []
    for run in (31, 64, 256, 600):
        p = _seq(rng, 900)
        t = _broken(rng, p, [run] * 3)
        pairs += [(p, np.concatenate([_seq(rng, free), t])), (p[free:], t), (p, t[: len(t) - free]),
                  (np.concatenate([_seq(rng, free // 2), p]), np.concatenate([t, _seq(rng, free)]))]
    b = synth_lib.from_pairs([(bytes(p), bytes(t)) for p, t in pairs])
    say(f"case: band kernel, middling reads, {free} free bases")
    ref = oracle_lib.align_batch(b, (4, 6, 2), cigar=True, threads=8, ends=(free,) * 4)
    aligner.set_ends_free(free, free, free, free)
    got = aligner.align(b, (4, 6, 2), capacity=int(ref.offsets[-1]) + 8)
    assert aligner.stats()["window"] == 256
    assert_same(got, ref, b, f"{free} free")
    sc, _, _ = aligner.align(b, (4, 6, 2), cigar=False)
    assert np.array_equal(sc, ref.scores)
