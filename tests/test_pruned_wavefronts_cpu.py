"""The rules by which the band and front kernels leave cells out, as a plain
model on the CPU against the oracle: offsets past the matrix dropped after the
maximum, a band exact up to the cheapest way out of it and back, the diamond of
cells that can still reach the end within a bound, decisions kept at a gap's
source and edits replayed along matches.  Scores and runs must be the oracle's
for every penalty set, free ends, bound slack and band width."""
import numpy as np
import pytest

NUL = -10**6


def model(P, T, pen, ends=(0, 0, 0, 0), band=None, bound=None):
    """(score, runs) of P against T, or None where the band hands the pair over.
    band: width; bound: slack above the score the diamond is cut to."""
    x, o, e = pen
    g = int(np.gcd.reduce([x, o, e]))
    X, OE, E = x // g, (o + e) // g, e // g
    n, m = len(P), len(T)
    kt = m - n
    pb, pe, tb, te = min(ends[0], n), min(ends[1], n), min(ends[2], m), min(ends[3], m)
    ks0, ks1, ke0, ke1 = -pb, tb, kt - te, kt + pe
    if band:
        k0 = (kt >> 1) - band // 2
        out0, out1 = k0 - 1, k0 + band
        ways = (2 * (OE - E) + E * ((out1 - ks1) + (out1 - ke1)),
                2 * (OE - E) + E * ((ks0 - out0) + (ke0 - out0)))
        smax = min(ways) - 1
        if ks1 >= out1 or ke1 >= out1 or ks0 <= out0 or ke0 <= out0 or smax < 0:
            return None
        lim = lambda s: (k0, k0 + band - 1)
    else:
        smax = 10**6 if bound is None else bound
        def lim(s):
            reach = (1 + (s - OE) // E) if s >= OE else 0
            back = (smax - s) // E
            return (max(ks0 - reach, ke0 - back, -n), min(ks1 + reach, ke1 + back, m))
    M, I, D, rec = {}, {}, {}, {}
    get = lambda A, t, k: A.get((t, k), NUL) if t >= 0 else NUL
    s = 0
    while True:
        if s > smax:
            return None
        lo, hi = lim(s)
        for k in range(lo, hi + 1):
            L = min(m, n + k) if -n <= k <= m else -1
            if s == 0:
                mv = max(k, 0) if ks0 <= k <= ks1 else NUL
                iv = dv = NUL
            else:
                iv = max(get(M, s - OE, k - 1), get(I, s - E, k - 1)) + 1
                dv = max(get(M, s - OE, k + 1), get(D, s - E, k + 1))
                xv = get(M, s - X, k) + 1
                mv = max(xv, iv, dv)
                rec[s, k] = (mv == xv, mv == iv)
            if iv >= 0:
                I[s, k] = iv
            if dv >= 0:
                D[s, k] = dv
            if 0 <= mv <= L:
                while mv < m and mv - k < n and P[mv - k] == T[mv]:
                    mv += 1
                M[s, k] = mv
        hit = [k for k in range(max(ke0, lo), min(ke1, hi) + 1)
               if get(M, s, k) == min(m, n + k)]
        if hit:
            break
        s += 1
    S, k = s, hit[0]
    edits = []
    while s > 0:
        isx, isi = rec[s, k]
        if isx:
            edits.append((1, 1))
            s -= X
            continue
        dk, A, op = (-1, I, 2) if isi else (1, D, 3)
        length = 0
        while True:
            length += 1
            k += dk
            ext = get(A, s - E, k) > get(M, s - OE, k)  # kept at the gap's source diagonal
            s -= E if ext else OE
            if not ext:
                break
        edits.append((op, length))
    assert s == 0
    runs = []

    def emit(op, length):
        if length <= 0:
            return
        if runs and runs[-1][0] == op:
            runs[-1][1] += length
        else:
            runs.append([op, length])

    h, v = max(k, 0), max(k, 0) - k
    emit(2, k)
    emit(3, -k)
    for op, length in [*reversed(edits), (None, 0)]:
        while h < m and v < n and P[v] == T[h]:
            emit(0, 1)
            h += 1
            v += 1
        if op is None:
            break
        emit(op, length)
        h += length if op != 3 else 0
        v += length if op != 2 else 0
    assert h == m or v == n
    emit(3, n - v)
    emit(2, m - h)
    return S * g, [length << 4 | op for op, length in runs]


def _pairs(rng, count, top):
    for _ in range(count):
        n = int(rng.integers(0, top))
        p = rng.choice(list(b"ACGT"), n).astype(np.uint8)
        if rng.random() < 0.6:  # related
            t = p[rng.random(n) > 0.12]
            hit = rng.random(len(t)) < 0.12
            t = np.where(hit, rng.choice(list(b"ACGT"), len(t)), t).astype(np.uint8)
            at = int(rng.integers(0, len(t) + 1))
            t = np.concatenate([t[:at], rng.choice(list(b"AC"), int(rng.integers(0, 7))).astype(np.uint8),
                                t[at:]])
        else:
            t = rng.choice(list(b"ACGT"), int(rng.integers(0, top))).astype(np.uint8)
        yield p.tobytes(), t.tobytes()


PENALTIES = [(4, 6, 2), (1, 0, 1), (2, 3, 1), (3, 1, 4), (5, 2, 3)]
ENDS = [(0, 0, 0, 0), (3, 0, 0, 4), (2, 5, 3, 1)]


@pytest.mark.parametrize("pen", PENALTIES)
@pytest.mark.parametrize("ends", ENDS)
def test_band(oracle_lib, pen, ends):
    rng = np.random.default_rng(17)
    held = handed = 0
    for P, T in _pairs(rng, 150, 28):
        want = oracle_lib.align(P, T, pen, ends=ends) if any(ends) else oracle_lib.align(P, T, pen)
        for width in (8, 12, 16):
            got = model(P, T, pen, ends, band=width)
            if got is None:
                handed += 1
                continue
            held += 1
            assert got[0] == want[0] and got[1] == [int(r) for r in want[1]], (P, T, width, got, want)
    assert held > 40 and handed > 40


@pytest.mark.parametrize("pen", PENALTIES)
@pytest.mark.parametrize("ends", ENDS)
def test_diamond(oracle_lib, pen, ends):
    rng = np.random.default_rng(23)
    g = int(np.gcd.reduce(list(pen)))
    for P, T in _pairs(rng, 120, 26):
        want = oracle_lib.align(P, T, pen, ends=ends) if any(ends) else oracle_lib.align(P, T, pen)
        for slack in (0, 1, 5):
            got = model(P, T, pen, ends, bound=int(want[0]) // g + slack)
            assert got is not None
            assert got[0] == want[0] and got[1] == [int(r) for r in want[1]], (P, T, slack, got, want)
