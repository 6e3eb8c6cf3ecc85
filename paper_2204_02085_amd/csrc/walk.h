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

// sum of the lanes' values up to and with this one's
__device__ __forceinline__ int wave_sum_to(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
    return v;
}

// Matching bases from (h, v) on, at most `left`, for each lane with left > 0:
// 64 by the lane itself, the rest by the whole wavefront, 1024 at a time.
__device__ __forceinline__ int lane_matches(uint32_t tb, uint32_t pb, int h, int v, int left, int lane) {
    int mm = 0;
    bool more = left > 0;
    for (int i = 0; i < 2; i++) {
        if (more) {
            const uint32_t x0 = win16(tb, 2 * (h + mm)) ^ win16(pb, 2 * (v + mm));
            const uint32_t x1 = win16(tb, 2 * (h + mm) + 32) ^ win16(pb, 2 * (v + mm) + 32);
            const uint64_t x = ((uint64_t)x1 << 32) | x0;
            const int z = x ? __builtin_ctzll(x) >> 1 : 32;
            mm += z;
            more = z == 32 && mm < left;
        }
    }
    for (uint64_t on = lanes_where(more); on; on &= on - 1) {
        const int l = __builtin_ctzll(on);
        const int hl = __builtin_amdgcn_readlane(h + mm, l), vl = __builtin_amdgcn_readlane(v + mm, l);
        const int ll = __builtin_amdgcn_readlane(left - mm, l);
        int sum = 0;
        while (sum < ll) {
            uint32_t x = 1;
            if (sum + 16 * lane < ll)
                x = win16(tb, 2 * (hl + sum + 16 * lane)) ^ win16(pb, 2 * (vl + sum + 16 * lane));
            const uint64_t stop = lanes_where(x != 0);
            if (stop) {
                const int fl = __builtin_ctzll(stop);
                sum += 16 * fl + (__builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)x, fl)) >> 1);
                break;
            }
            sum += 1024;
        }
        if (lane == l) mm += sum;
    }
    return min(mm, left);
}

constexpr int WALK_QUADS = 64;                       // quads of steps of the record window in LDS
constexpr int WALK_COLS = 16;                        // its diagonals
constexpr int WALK_DW = WALK_QUADS * WALK_COLS / 2;  // its dwords

// One pair's walk, by one wavefront: the records back to the list of edits,
// from that the matches after every edit, then the runs.  What bounds it is the
// chain of LDS round trips and of scalar instructions, so each part takes many
// edits at a time:
//   back     sixteen lanes each look at the next cells of a run of mismatches,
//            of an insertion and of a deletion from here;
//   matches  the forward pass has left the M row of every 16th step
//            (`offset(s, k)`: the offset of cell k of such a row), so the cells
//            of those rows that the path goes through cut it into pieces, and
//            each lane follows one of them;
//   runs     64 edits at a time, places by a sum over the lanes.
// One edit at a time took 445 us of a lone pair of 5 kbp at 10 % (1.13 ms in
// all); with pieces only for the way back 325 us.
//
// The records come through a window of 64 quads of steps by 16 diagonals in LDS
// (`win`); `load(q, k)` fills it with quad q and those before it, around
// diagonal k, and returns the first diagonal.  AT_DEST: the gap bits stand at the
// gap's own diagonal (else at its source's).  Events and runs go to
// evs[ev_words] and below runs_end; sequences at LDS bytes tb and pb.  Returns
// the runs written below runs_end, last to first, or -1.
template <int X, int OE, int E, bool AT_DEST, class Load, class Offset>
__device__ int walk(Load&& load, Offset&& offset, int S, int n, int m, int lane, lds_p<uint32_t> win,
                    uint32_t* evs, int ev_words, uint32_t* runs_end, int run_words, uint32_t tb,
                    uint32_t pb) {
    // ---- the edits, last to first; lane i keeps event i of the current 64
    bool bad = false;
    int s = S, k = m - n, ne = 0;
    uint32_t evreg = 0;
    auto events = [&](int kind, int len, int count) {  // at most 64 of them
        const int at = ne & 63;
        const uint32_t ev = (uint32_t)(len << 2 | kind);
        evreg = (uint32_t)(lane - at) < (uint32_t)count ? ev : evreg;
        ne += count;
        if (ne > ev_words) bad = true;
        if (!bad && at + count >= 64) {
            evs[(ne & ~63) - 64 + lane] = evreg;
            evreg = ev;  // (of use in the lanes below ne & 63)
        }
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
    // cells on rows of every `every` steps; lane i: the i-th, and the events
    // before it (those nearer the end)
    int every = 16, nck = 0, cks = 0, ckk = 0, ckn = 0;
    while (S / every >= 62) every *= 2;
    while (s > 0 && !bad) {
        if ((s >> 2) > qtop || (s >> 2) <= qtop - WALK_QUADS || k < kf || k >= kf + WALK_COLS) refill(k);
        const int sj = s - ds, row = qtop - (sj >> 2), col = k + dk - kf;
        const bool in = sj > 0 && row < WALK_QUADS && col >= 0 && col < WALK_COLS;
        const uint32_t word = in ? win[row * (WALK_COLS / 2) + (col >> 1)] : 0u;
        const uint32_t rec = record_of(word, sj, col);
        const uint64_t seen = lanes_where(in && group < 3);
        const uint64_t set = lanes_where(in && (rec & bit) != 0);
        if (gap < 0) {
            if ((s & (every - 1)) == 3 && ne > 0) {
                cks = lane == nck ? s : cks;
                ckk = lane == nck ? k : ckk;
                ckn = lane == nck ? ne : ckn;
                nck++;
            }
            int run = __builtin_ctz((~(uint32_t)seen | (uint32_t)set | 0x10000u));
            // up to the next such row, if the mismatches meet it
            const int next = ((s - 4) & (every - 1)) + 1;
            if (next % X == 0) run = min(run, next / X);
            if (run > 0) {
                events(EV_X, 1, run);
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
            events(gap, glen, 1);
            gap = -1;
        } else if (len == 0) {  // the window ends here
            refill(k + dir);
            const int c0 = k + (AT_DEST ? 0 : dir) - kf;
            if (c0 < 0 || c0 >= WALK_COLS) bad = true;
        }
    }
    if (s != 0 || k != 0 || gap >= 0 || bad) return -1;
    if ((ne & 63) && lane < (ne & 63)) evs[(ne & ~63) + lane] = evreg;
    __threadfence_block();

    // ---- the matches after every edit, into the upper half of its event.
    // Lane i follows the events from cell i on to cell i - 1 (lane 0: to the
    // end); the lane after the last cell starts at the origin
    int h = 0, v = 0;
    if (lane == nck) ckn = ne;
    const int stop = (int)wave_prev(0u, (uint32_t)ckn);
    if (lane < nck) {
        h = offset(cks, ckk);
        v = h - ckk;
    }
    const int h0 = h, v0 = v;
    bool ok = lane > nck || (h >= 0 && v >= 0 && h <= m && v <= n);
    const int mm0 = lane_matches(tb, pb, h, v, lane == nck ? min(n, m) : 0, lane);
    h += mm0;
    v += mm0;
    int i = ckn - 1;
    bool on = lane <= nck && ok && i >= stop;
    uint32_t ev = on ? evs[i] : 0u;
    while (lanes_where(on)) {
        const uint32_t after = on && i > stop ? evs[i - 1] : 0u;
        if (on) {
            const int len = (int)(ev >> 2) & 0x7FFF;
            h += (ev & 3) == EV_D ? 0 : len;
            v += (ev & 3) == EV_I ? 0 : len;
            ok = h <= m && v <= n;
        }
        on = on && ok;
        const int mm = lane_matches(tb, pb, h, v, on ? min(n - v, m - h) : 0, lane);
        if (on) evs[i] = ev | (uint32_t)mm << 17;
        h += mm;
        v += mm;
        i--;
        on = on && i >= stop;
        ev = after;
    }
    // every piece ends where the next one starts
    const int hn = (int)wave_next(0u, (uint32_t)h), vn = (int)wave_next(0u, (uint32_t)v);
    if (lane < nck) ok = ok && hn == h0 && vn == v0;
    if (lane == 0) ok = ok && h == m && v == n;
    if (lanes_where(!ok)) return -1;
    __threadfence_block();

    // ---- the runs, stored downwards from the end, so that they stand last to
    // first.  An edit adds a run, unless it goes on with the one before, and its
    // matches another; buf[0] is the run the last 64 edits ended with.
    lds_p<uint32_t> buf = win;
    int nr = 0;
    uint32_t open_run = (uint32_t)__builtin_amdgcn_readlane(mm0, nck) << 4;
    int first = open_run ? 0 : 1;  // 1: there is none yet
    uint32_t before = ~0u;         // the event before
    for (int top = ne - 1; top >= 0; top -= 64) {
        const bool is = lane <= top;
        const uint32_t e = is ? evs[top - lane] : 0u;
        const uint32_t p = wave_prev(before, e);
        const bool head = is && ((p >> 17) || ((p ^ e) & 3));
        const bool match = is && (e >> 17);
        const int upto = wave_sum_to((head ? 1 : 0) + (match ? 1 : 0));
        const int total = __builtin_amdgcn_readlane(upto, 63);
        const int at = upto - (match ? 1 : 0);  // of the edit's run
        wave_fence();
        buf[lane] = lane == 0 ? open_run : 0u;
        buf[64 + lane] = 0u;
        if (lane == 0) buf[128] = 0u;
        wave_fence();
        if (is)
            __hip_atomic_fetch_add(buf + at, ((e >> 2) & 0x7FFF) << 4 | (head ? 1 + (e & 3) : 0u),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        if (match) buf[at + 1] = (e >> 17) << 4;
        wave_fence();
        const int count = total - first;
        if (nr + count + 1 > run_words) return -1;
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int r = lane + 64 * u;
            if (r >= first && r < total) runs_end[-(nr + r - first) - 1] = buf[r];
        }
        open_run = (uint32_t)__builtin_amdgcn_readfirstlane((int)buf[total]);
        nr += count;
        first = 0;
        before = (uint32_t)__builtin_amdgcn_readlane((int)e, min(top, 63));
    }
    if (first == 0) {
        if (nr + 1 > run_words) return -1;
        if (lane == 0) runs_end[-nr - 1] = open_run;
        nr++;
    }
    return nr;
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
