// Staging and the CIGAR walk shared by the front and adaptive kernels
// (k_front.hip, k_adapt.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "kernels.h"
#include "rows.h"

namespace wfa {
namespace rows {

__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Both sequences into LDS: the text's words, then the pattern's, each followed
// by a zero word.  The pattern starts at least four words in, so a compare a
// little before its first base (a cell off the matrix) stays in the block.
__device__ __forceinline__ int text_words(int m) { return max((m + 31) / 32 + 1, 8); }
__device__ __forceinline__ void stage(lds_p<uint64_t> dst, const uint64_t* pw, const uint64_t* tw,
                                      const PairDesc& d, int tid, int bt) {
    const int nwt = ((int)d.t_len + 31) >> 5, nwp = ((int)d.p_len + 31) >> 5;
    const int tws = text_words((int)d.t_len);
    for (int w = tid; w < tws; w += bt) dst[w] = w < nwt ? tw[d.t_start + w] : 0ull;
    for (int w = tid; w <= nwp; w += bt) dst[tws + w] = w < nwp ? pw[d.p_start + w] : 0ull;
}

// 16-bit value of a packed register at a wave-uniform lane and half
__device__ __forceinline__ int half_at(uint32_t reg, int lane, int half) {
    const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)reg, lane);
    return (int)(short)(w >> (16 * half));
}

// largest of the lanes' values, in every lane
__device__ __forceinline__ int wave_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xF, 0xF, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// LDS bytes of both staged sequences, with a tail for compares past the
// pattern's end by cells off the matrix
inline int seq_lds_bytes(uint32_t n, uint32_t m) {
    return 8 * (int)(std::max((m + 31) / 32 + 1, 8u) + (n + 31) / 32 + 1) + 256;
}

constexpr int WALK_QUADS = 64;                     // quads of steps of the record window in LDS
constexpr int WALK_COLS = 16;                      // its diagonals
constexpr int WALK_DW = WALK_QUADS * WALK_COLS / 2;  // its dwords

// One pair's walk, by one wavefront: the records back to the list of edits,
// then the edits from the start along matches.  All but the loads, stores and
// compares is wave-uniform, so what bounds it is the chain of LDS round trips
// and of scalar instructions; each round trip takes as many edits as it can:
//   back     sixteen lanes each look at the next cells of a run of mismatches,
//            of an insertion and of a deletion from here;
//   forward  lane l compares 16 bases, 16 l on, and a run of mismatches on one
//            diagonal reads its matches from those bits.
// One edit per round trip took 300 us of a lone pair of 5 kbp at 10 % (1.13 ms in
// all).
//
// The records come through a window of 64 quads of steps by 16 diagonals in LDS
// (`win`); `load(q, k)` fills it with quad q and those before it, around
// diagonal k, and returns the first diagonal.  AT_DEST: the gap bits stand at the
// gap's own diagonal (else at its source's).  Events and runs go to
// evs[ev_words] and below runs_end; sequences at LDS bytes tb and pb.  Returns
// the runs written below runs_end, last to first, or -1.
template <int X, int OE, int E, bool AT_DEST, class Load>
__device__ int walk(Load&& load, int S, int n, int m, int lane, lds_p<uint32_t> win, uint32_t* evs,
                    int ev_words, uint32_t* runs_end, int run_words, uint32_t tb, uint32_t pb) {
    // ---- the edits, last to first; lane i keeps event i of the current 64
    bool bad = false;
    int s = S, k = m - n, ne = 0;
    uint32_t evreg = 0;
    auto event = [&](int kind, int len) {
        evreg = lane == (ne & 63) ? (uint32_t)(len << 2 | kind) : evreg;
        ne++;
        if (ne > ev_words) bad = true;
        if (!bad && (ne & 63) == 0) evs[ne - 64 + lane] = evreg;
    };
    int qtop = -1, kf = 0;
    auto refill = [&](int to) {
        qtop = s >> 2;
        wave_fence();
        kf = load(qtop, to);
        wave_fence();
    };
    // lanes 0-15: mismatches, 16-31: an insertion, 32-47: a deletion
    const int group = lane >> 4, j = lane & 15;
    const int ds = j * (group == 0 ? X : E);
    const int dk = (j + (AT_DEST ? 0 : 1)) * (group == 1 ? -1 : group == 2 ? 1 : 0);
    const uint32_t bit = group == 0 ? 1u : group == 1 ? 4u : 8u;
    int gap = -1, glen = 0;  // the gap the walk is in, its bases so far
    while (s > 0 && !bad) {
        if ((s >> 2) > qtop || (s >> 2) <= qtop - WALK_QUADS || k < kf || k >= kf + WALK_COLS) refill(k);
        const int sj = s - ds, row = qtop - (sj >> 2), col = k + dk - kf;
        const bool in = sj > 0 && row < WALK_QUADS && col >= 0 && col < WALK_COLS;
        const uint32_t word = in ? win[row * (WALK_COLS / 2) + (col >> 1)] : 0u;
        const uint32_t rec = record_of(word, sj, col);
        const uint64_t seen = lanes_where(in && group < 3);
        const uint64_t set = lanes_where(in && (rec & bit) != 0);
        if (gap < 0) {
            const int run = __builtin_ctz((~(uint32_t)seen | (uint32_t)set | 0x10000u));
            if (run > 0) {
                event(EV_X, run);
                s -= X * run;
                continue;
            }
            const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)rec, 0);
            if (!(seen & 1)) bad = true;  // outside the records (never, if they are whole)
            gap = (first & 2) ? EV_D : EV_I;
            glen = 0;
        }
        const int sh = 16 * gap;  // EV_I = 1, EV_D = 2
        const uint32_t gs = (uint32_t)(seen >> sh) & 0xFFFFu, ge = (uint32_t)(set >> sh) & 0xFFFFu;
        const int ext = __builtin_ctz(~ge | 0x10000u);
        const bool open = ext < 16 && ((gs >> ext) & 1);
        const int len = ext + (open ? 1 : 0), dir = gap == EV_I ? -1 : 1;
        glen += len;
        s -= E * ext + (open ? OE : 0);
        k += dir * len;
        if (open) {
            event(gap, glen);
            gap = -1;
        } else if (len == 0) {  // the window ends here
            refill(k + dir);
            const int c0 = k + (AT_DEST ? 0 : dir) - kf;
            if (c0 < 0 || c0 >= WALK_COLS) bad = true;
        }
    }
    if (s != 0 || k != 0 || gap >= 0) bad = true;

    // ---- replay; runs are stored downwards from the end, so that they stand
    // last to first
    int h = 0, v = 0, nr = 0, cop = -1, clen = 0;
    uint32_t rreg = 0;
    auto put = [&]() {
        rreg = lane == (nr & 63) ? ((uint32_t)clen << 4) | (uint32_t)cop : rreg;
        nr++;
        if (nr > run_words) bad = true;
        if (!bad && (nr & 63) == 0) runs_end[-(nr - 64) - 1 - lane] = rreg;
    };
    auto emit = [&](int op, int len) {
        if (len <= 0) return;
        if (op == cop) {
            clen += len;
        } else {
            if (cop >= 0) put();
            cop = op;
            clen = len;
        }
    };
    // 1024 bases from (h, v) on: two bits per base that differs (bases past
    // either end do); `at`: how many of them are taken
    uint32_t diff = 0;
    uint64_t some = 0;
    int at = 0, left = 0;
    auto compare = [&]() {
        left = min(n - v, m - h);
        uint32_t x = ~0u;
        if (16 * lane < left)
            x = win16(tb, 2 * (h + 16 * lane)) ^ win16(pb, 2 * (v + 16 * lane));
        diff = x;
        some = lanes_where(x != 0);
        at = 0;
    };
    auto advance = [&](int dh, int dv) {
        h += at + dh;
        v += at + dv;
        if (h > m || v > n) bad = true;
        if (!bad) compare();
    };
    auto matches = [&]() {
        int mm = 0;
        while (!bad) {
            int to = 1024;
            const int l0 = at >> 4;
            uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)diff, l0) & (~0u << (2 * (at & 15)));
            if (y) {
                to = 16 * l0 + (__builtin_ctz(y) >> 1);
            } else {
                const uint64_t later = some & (~1ull << l0);
                if (later) {
                    const int l1 = __builtin_ctzll(later);
                    y = (uint32_t)__builtin_amdgcn_readlane((int)diff, l1);
                    to = 16 * l1 + (__builtin_ctz(y) >> 1);
                }
            }
            to = min(to, left);
            mm += to - at;
            at = to;
            if (at < 1024 || at == left) break;
            advance(0, 0);
        }
        emit(0, mm);
    };
    if (!bad) compare();
    matches();
    for (int i = ne - 1; i >= 0 && !bad; i--) {
        if ((i & 63) == 63 && i != ne - 1) evreg = evs[i - 63 + lane];
        const uint32_t ev = (uint32_t)__builtin_amdgcn_readlane((int)evreg, i & 63);
        const int len = (int)(ev >> 2), kind = (int)(ev & 3);
        if (kind == EV_X) {
            for (int c = 0; c < len && !bad; c++) {
                if (at >= left) bad = true;
                emit(1, 1);
                if (++at == 1024) advance(0, 0);
                matches();
            }
        } else {
            emit(1 + kind, len);
            advance(kind == EV_I ? len : 0, kind == EV_D ? len : 0);
            matches();
        }
    }
    h += at;
    v += at;
    if (h != m || v != n) bad = true;
    if (cop >= 0) put();
    if (!bad && (nr & 63) && lane < (nr & 63)) runs_end[-(nr & ~63) - 1 - lane] = rreg;
    return bad ? -1 : nr;
}

// A job's walk ended with nr runs (-1: it did not): its results, or its place
// in the list of pairs for the general kernel.
__device__ __forceinline__ void walk_done(const FrontArgs& a, const FrontJob& job, int S, int nr,
                                          const uint32_t* runs_end, int lane) {
    if (lane != 0) return;
    if (nr < 0) {
        a.fail_list[atomicAdd(a.fail_count, 1u)] = job.pair;
        return;
    }
    a.scores[job.pair] = S * a.g;
    a.nruns[job.pair] = (uint32_t)nr;
    a.job_nruns[blockIdx.x] = (uint32_t)nr;
    a.run_src[job.pair] = (uint64_t)(runs_end - a.arena) - nr;  // arena words
}

}  // namespace rows
}  // namespace wfa
