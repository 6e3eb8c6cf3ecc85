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

// One pair's walk, by one wavefront: the records back to the list of edits,
// then the edits from the start along matches, 1024 bases per compare.
// Everything but the loads and stores is wave-uniform.  `record(s, k, bad)`
// reads the record of a cell; AT_DEST: the gap bits stand at the gap's own
// diagonal (else at its source's).  Events and runs go to evs[ev_words] and
// below runs_end; sequences at LDS bytes tb and pb.  Returns the runs written
// below runs_end, last to first, or -1.
template <int X, int OE, int E, bool AT_DEST, class Record>
__device__ int walk(Record&& record, int S, int n, int m, int lane, uint32_t* evs, int ev_words,
                    uint32_t* runs_end, int run_words, uint32_t tb, uint32_t pb) {
    // ---- the edits, last to first; lane i keeps event i of the current 64
    bool bad = false;
    int s = S, k = m - n, ne = 0;
    uint32_t evreg = 0;
    while (s > 0 && !bad) {
        const uint32_t f = record(s, k, bad);
        int kind = EV_X, len = 1;
        if (!(f & 1)) {
            s -= X;
        } else {
            const bool ins = !(f & 2);
            kind = ins ? EV_I : EV_D;
            const uint32_t more = ins ? 4u : 8u;
            const int dk = ins ? -1 : 1;
            len = 0;
            for (;;) {
                len++;
                if (!AT_DEST) k += dk;
                if (s <= 0) bad = true;
                if (bad) break;
                const bool ext = (record(s, k, bad) & more) != 0;
                if (AT_DEST) k += dk;
                s -= ext ? E : OE;
                if (!ext) break;
            }
        }
        evreg = lane == (ne & 63) ? (uint32_t)(len << 2 | kind) : evreg;
        ne++;
        if (ne > ev_words) bad = true;
        if (!bad && (ne & 63) == 0) evs[ne - 64 + lane] = evreg;
    }
    if (s != 0 || k != 0) bad = true;

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
    for (int i = ne - 1; !bad; i--) {
        int left = min(n - v, m - h), mm = 0;
        while (left > 0) {  // lane l compares 16 bases, 16 l on
            uint32_t x = 1;
            if (16 * lane < left)
                x = win16(tb, 2 * (h + mm + 16 * lane)) ^ win16(pb, 2 * (v + mm + 16 * lane));
            const uint64_t stop = lanes_where(x != 0);
            int z = 1024;
            if (stop) {
                const int fl = __builtin_ctzll(stop);
                const uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)x, fl);
                z = 16 * fl + (__builtin_ctz(y) >> 1);
            }
            z = min(z, left);
            mm += z;
            left -= z;
            if (z < 1024) break;
        }
        emit(0, mm);
        h += mm;
        v += mm;
        if (i < 0) break;
        if ((i & 63) == 63 && i != ne - 1) evreg = evs[i - 63 + lane];
        const uint32_t ev = (uint32_t)__builtin_amdgcn_readlane((int)evreg, i & 63);
        const int len = (int)(ev >> 2), kind = (int)(ev & 3);
        emit(1 + kind, len);
        if (kind != EV_D) h += len;
        if (kind != EV_I) v += len;
        if (h > m || v > n) bad = true;
    }
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
