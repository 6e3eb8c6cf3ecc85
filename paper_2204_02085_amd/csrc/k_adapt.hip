// Adaptive kernel: the WF-adaptive heuristic, one wavefront per pair.
//
// The reduction keeps a wavefront to the diagonals near its furthest points,
// usually a few dozen, so a pair's rows fit the registers of one wavefront: a
// window of 128 diagonals, two per lane, that moves along with the reduced
// ranges, and further blocks of 128 beside it while they are wider.  Where
// k_general spent a workgroup, several barriers and row traffic on every step, a
// step here is about 130 instructions of one wavefront, the least distance by DPP
// and the kept range by two ballots.
//
// What bounds it: VALU issue, 0.91 of it over 10 k pairs of 1-10 kbp at 5-10 %
// under the thresholds (10, 50), whole call with CIGARs 3.6 ms (32.0 ms on the
// general kernel).  The second block inside the same kernel: 22 of those
// pairs outgrow 128 diagonals for a stretch, and aligning them again in a wider
// window took another 4.7 ms, the latency of their chains.
//
// The reduction measures every cell, on an optimal path or not, so offsets
// here follow the recurrences to the letter: a candidate past the matrix is
// dropped before the maximum (as an unsigned distance below the diagonal's
// limit, like the general kernel's), in I and D too, and the ranges of steps
// are those of the sources widened by one and clipped to the matrix.
//
// Two blocks first.  A pair whose ranges outgrow them (gaps of hundreds of bases,
// unrelated sequences), or that needs more steps than its records hold, is aligned
// again in a window of eight blocks, at one wavefront per SIMD instead of four, with
// records for every step it can need; what outgrows that goes to the general kernel.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "rows.h"
#include "walk.h"

namespace wfa {

namespace {

using namespace rows;

// smallest of the lanes' values, in every lane
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
    auto step = [&](int other) { v = min(v, (uint32_t)other); };
    step(__builtin_amdgcn_update_dpp((int)v, (int)v, 0x111, 0xF, 0xF, false));  // row_shr:1
    step(__builtin_amdgcn_update_dpp((int)v, (int)v, 0x112, 0xF, 0xF, false));
    step(__builtin_amdgcn_update_dpp((int)v, (int)v, 0x114, 0xF, 0xF, false));
    step(__builtin_amdgcn_update_dpp((int)v, (int)v, 0x118, 0xF, 0xF, false));
    step(__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xA, 0xF, false));  // row_bcast:15
    step(__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The window is NB blocks of 128 diagonals, two per lane and block; the second, the
// third and fourth, and the last four are computed only while the ranges do not fit
// those before.
template <int X, int OE, int E, int SH, int NB, bool CIGAR>
__global__ __launch_bounds__(64) void k_adapt(FrontArgs a) {
    constexpr int BW = 128, AW = NB * BW, QUAD = adapt_quad_words(NB);
    // the walk's window; columns of a wide window past the last diagonal compare from
    // up to AW bases before the pattern, which stays behind it
    constexpr bool HEAD = CIGAR || AW / 4 > 64;
    static_assert(AW / 4 <= 64 + 4 * WALK_DW, "compares stay in the workgroup's LDS");
    constexpr int RM = X > OE ? X : OE;
    constexpr int LONG = NB > ADAPT_BLOCKS ? LONG_LANE : LONG_WAVE;  // (no registers left for the other)
    constexpr uint32_t ONE = SH ? 0x00020002u : 0x00010001u;
    extern __shared__ __align__(16) unsigned char lds[];
    const FrontJob job = a.jobs[blockIdx.x];
    const PairDesc d = a.pairs[job.pair];
    const int n = (int)d.p_len, m = (int)d.t_len, kt = m - n;
    const int lane = threadIdx.x;
    lds_p<uint32_t> win = (lds_p<uint32_t>)lds;
    lds_p<uint64_t> seq = (lds_p<uint64_t>)(win + (HEAD ? WALK_DW : 0));
    stage(seq, a.pw, a.tw, d, lane, 64);
    wave_fence();
    const uint32_t tb = (uint32_t)(uintptr_t)seq, pb = tb + 8 * text_words(m);
    const int MWL = a.heur.mwl, MDT = a.heur.mdt;
    uint32_t* hist = CIGAR ? a.arena + job.hist : nullptr;  // per quad: the records, the window's base

    int kmin = -BW / 2;
    Place<2> pl[NB];
    uint32_t inside[NB];  // 0xffff in the halves whose diagonal is in the matrix
    uint32_t whole[NB];   // max(n + k, m), in the offsets' units: 16 bits without sign
    auto place = [&]() {
#pragma unroll
        for (int b = 0; b < NB; b++) {
            pl[b].template set<SH>(n, m, kmin + BW * b + 2 * lane);
            inside[b] = ~pk_sign(pl[b].lim[0]);
            const int k = kmin + BW * b + 2 * lane;
            whole[b] = pk_pair(max(n + k, m) << SH, max(n + k + 1, m) << SH);
        }
    };
    place();
    uint32_t M[RM][NB], I[E][NB], D[E][NB], acc[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        acc[b] = 0;
#pragma unroll
        for (int j = 0; j < RM; j++) M[j][b] = NUL16P;
#pragma unroll
        for (int j = 0; j < E; j++) I[j][b] = D[j][b] = NUL16P;
    }
    auto shift_up = [&](uint32_t (&r)[NB]) {  // one lane: the window moves two diagonals up
#pragma unroll
        for (int b = 0; b < NB; b++)
            r[b] = wave_next(b + 1 < NB ? (uint32_t)__builtin_amdgcn_readlane((int)r[b + 1 < NB ? b + 1 : b], 0) : NUL16P,
                             r[b]);
    };
    auto shift_down = [&](uint32_t (&r)[NB]) {
#pragma unroll
        for (int b = NB - 1; b >= 0; b--)
            r[b] = wave_prev(b ? (uint32_t)__builtin_amdgcn_readlane((int)r[b ? b - 1 : 0], 63) : NUL16P, r[b]);
    };
    // ranges of the last RM steps; lo > hi: no wavefront
    constexpr int NONE = 1 << 29;
    int lo[RM], hi[RM];
#pragma unroll
    for (int j = 0; j < RM; j++) {
        lo[j] = NONE;
        hi[j] = -NONE;
    }
    int S = -1;
    // four steps on the first nb blocks
    auto quad = [&](int s, auto blocks) {
        constexpr int nb = decltype(blocks)::value;
#pragma unroll
        for (int u = 0; u < 4; u++) {
            if (S >= 0) break;
            // the step's range: its sources', one wider, inside the matrix
            int l = min(min(lo[X - 1], lo[OE - 1]), lo[E - 1]);
            int h = max(max(hi[X - 1], hi[OE - 1]), hi[E - 1]);
            bool present = l <= h;
            l = max(l - 1, -n);
            h = min(h + 1, m);
            uint32_t cm[NB], ci[NB], cd[NB], rec[NB];
#pragma unroll
            for (int b = 0; b < NB; b++) {
                cm[b] = ci[b] = cd[b] = NUL16P;
                rec[b] = 0;
            }
            if (u == 0 && s == 0) {
                present = true;
                l = h = 0;
                if (lane == 32) cm[0] = 0xC0000000u;  // M_0[0] = 0
                uint32_t c1[1] = {cm[0]};
                extend<2, SH, LONG>(c1, pl[0], tb, pb);
                cm[0] = c1[0];
            } else if (present) {
#pragma unroll
                for (int b = 0; b < nb; b++) {
                    // the columns before and after, across the blocks' border
                    auto up = [&](const uint32_t (&r)[NB]) {
                        const uint32_t end = b ? (uint32_t)__builtin_amdgcn_readlane((int)r[b ? b - 1 : 0], 63) : NUL16P;
                        return __builtin_amdgcn_alignbit(r[b], wave_prev(end, r[b]), 16);
                    };
                    auto down = [&](const uint32_t (&r)[NB]) {
                        const uint32_t end = b + 1 < nb ? (uint32_t)__builtin_amdgcn_readlane((int)r[b + 1 < nb ? b + 1 : b], 0) : NUL16P;
                        return __builtin_amdgcn_alignbit(wave_next(end, r[b]), r[b], 16);
                    };
                    // distances below the limit: past it they wrap to huge,
                    // NULL is past L
                    const uint32_t L = pl[b].lim[0];
                    const uint32_t tio = pk_sub(L, pk_add(up(M[OE - 1]), ONE)), tdo = pk_sub(L, down(M[OE - 1]));
                    const uint32_t tx = pk_sub(L, pk_add(M[X - 1][b], ONE));
                    const uint32_t ti = pk_minu(tio, pk_sub(L, pk_add(up(I[E - 1]), ONE)));
                    const uint32_t td = pk_minu(tdo, pk_sub(L, down(D[E - 1])));
                    const uint32_t tm = pk_minu(pk_minu(tx, ti), td);
                    if (CIGAR)
                        rec[b] = shl_or<1>(shl_or<1>(shl_or<1>(pk_ne(tdo, td), pk_ne(tio, ti)), pk_ne(ti, tm)),
                                           pk_ne(tx, tm));
                    ci[b] = pk_sub(L, ti);
                    cd[b] = pk_sub(L, td);
                    ci[b] = bit_select(pk_sign(ci[b] | ti | ~inside[b]), NUL16P, ci[b]);
                    cd[b] = bit_select(pk_sign(cd[b] | td | ~inside[b]), NUL16P, cd[b]);
                    uint32_t c1[1] = {bit_select(inside[b], pk_sub(L, tm), NUL16P)};
                    extend<2, SH, LONG>(c1, pl[b], tb, pb);
                    cm[b] = c1[0];
                }
            }
            if (CIGAR) {
#pragma unroll
                for (int b = 0; b < nb; b++) acc[b] = u ? shl_or<4>(acc[b], rec[b]) : rec[b];
            }
            const int tc = kt - kmin;
            uint32_t treg = cm[0];
#pragma unroll
            for (int b = 1; b < nb; b++) treg = tc >= BW * b ? cm[b] : treg;
            if (tc >= 0 && tc < nb * BW && half_at(treg, (tc & (BW - 1)) >> 1, tc & 1) == m << SH) {
                S = s + u;  // the step that reaches the end is not reduced
            } else if (present && h - l + 1 >= MWL) {
                // distances to the end: max(n + k, m) - M, two to a register;
                // all ones where there is no offset
                constexpr uint32_t FAR = 0xFFFF;
                uint32_t dist[NB], least = FAR;
#pragma unroll
                for (int b = 0; b < nb; b++) {
                    dist[b] = pk_sub(whole[b], cm[b]) | pk_sign(cm[b]);
                    least = min(least, min(dist[b] & 0xffffu, dist[b] >> 16));
                }
                least = wave_min(least);
                if (least != FAR) {
                    const uint32_t lim = (uint32_t)min((long long)least + ((long long)MDT << SH), (long long)FAR - 1);
                    int rl = AW, rh = -1;  // kept columns
#pragma unroll
                    for (int c = 0; c < 2 * nb; c++) {
                        const uint64_t in = lanes_where(((c & 1) ? dist[c / 2] >> 16 : dist[c / 2] & 0xffffu) <= lim);
                        if (in) {
                            rl = min(rl, BW * (c / 2) + 2 * (int)__builtin_ctzll(in) + (c & 1));
                            rh = max(rh, BW * (c / 2) + 2 * (63 - (int)__builtin_clzll(in)) + (c & 1));
                        }
                    }
                    l = kmin + rl;
                    h = kmin + rh;
#pragma unroll
                    for (int b = 0; b < nb; b++) {
                        const int c = BW * b + 2 * lane;
                        const uint32_t keep = (c >= rl && c <= rh ? 0xffffu : 0u) |
                                              (c + 1 >= rl && c + 1 <= rh ? 0xffff0000u : 0u);
                        cm[b] = bit_select(keep, cm[b], NUL16P);
                        ci[b] = bit_select(keep, ci[b], NUL16P);
                        cd[b] = bit_select(keep, cd[b], NUL16P);
                    }
                }
            }
#pragma unroll
            for (int j = RM - 1; j > 0; j--) {
                lo[j] = lo[j - 1];
                hi[j] = hi[j - 1];
            }
            lo[0] = present ? l : NONE;
            hi[0] = present ? h : -NONE;
#pragma unroll
            for (int b = 0; b < nb; b++) {
#pragma unroll
                for (int j = RM - 1; j > 0; j--) M[j][b] = M[j - 1][b];
#pragma unroll
                for (int j = E - 1; j > 0; j--) {
                    I[j][b] = I[j - 1][b];
                    D[j][b] = D[j - 1][b];
                }
                M[0][b] = cm[b];
                I[0][b] = ci[b];
                D[0][b] = cd[b];
            }
            if (CIGAR && (u == 3 || S >= 0)) {
                uint32_t* q = hist + (uint64_t)(s >> 2) * QUAD;
#pragma unroll
                for (int b = 0; b < nb; b++) q[64 * b + lane] = acc[b] << (4 * (3 - u));
                if (lane == 0) q[64 * NB] = (uint32_t)kmin;
                if (u == 3 && (s & 15) == 0) {
                    uint32_t* r = hist + adapt_rec_words(job.bound, NB) + (uint64_t)(s >> 4) * (64 * NB);
#pragma unroll
                    for (int b = 0; b < nb; b++) r[64 * b + lane] = cm[b];
                }
            }
        }
    };
    for (int s = 0; S < 0; s += 4) {
        // the rows' ranges, four steps on, inside the first block or, if they
        // are wider, inside the first two, four or all
        int ul = NONE, uh = -NONE;
#pragma unroll
        for (int j = 0; j < RM; j++) {
            ul = min(ul, lo[j]);
            uh = max(uh, hi[j]);
        }
        if (s == 0) ul = uh = 0;
        const int width = uh - ul + 1 + 8;
        if (s > job.bound || ul > uh || width + 2 > AW) break;
        int room = BW;
        while (room < width + 2) room *= 2;
        if (ul - 4 < kmin || uh + 4 > kmin + room - 1) {
            // in the middle, rounded down to a lane: of the columns to spare
            // there are at least two, so both margins hold
            int shift = (ul - 4 - (room - width) / 2 - kmin) >> 1;  // lanes
            kmin += 2 * shift;
            for (; shift > 0; shift--) {
#pragma unroll
                for (int j = 0; j < RM; j++) shift_up(M[j]);
#pragma unroll
                for (int j = 0; j < E; j++) {
                    shift_up(I[j]);
                    shift_up(D[j]);
                }
            }
            for (; shift < 0; shift++) {
#pragma unroll
                for (int j = 0; j < RM; j++) shift_down(M[j]);
#pragma unroll
                for (int j = 0; j < E; j++) {
                    shift_down(I[j]);
                    shift_down(D[j]);
                }
            }
            place();
        }
        if (room == BW) quad(s, std::integral_constant<int, 1>{});
        else if (NB == 2 || room == 2 * BW) quad(s, std::integral_constant<int, 2>{});
        else if (room == 4 * BW) quad(s, std::integral_constant<int, NB < 4 ? NB : 4>{});
        else quad(s, std::integral_constant<int, NB>{});
    }
    if (S < 0) {  // outgrew its records, or the window
        if (lane == 0) a.fail_list[atomicAdd(a.fail_count, 1u)] = job.pair;
        return;
    }
    if (!CIGAR) {
        if (lane == 0) {
            a.scores[job.pair] = S * a.g;
            a.nruns[job.pair] = 0;
        }
        return;
    }
    // the walk (what a quad left unwritten of its later blocks is never on the
    // way; the windows of all quads start at an even diagonal)
    constexpr int QW = 64 * NB;
    __threadfence_block();
    uint32_t* evs = hist + job.hist_words;
    uint32_t* runs_end = evs + job.ev_words + job.run_words;
    auto load = [&](int q, int k) {
        const int kf = (k & ~1) - WALK_COLS / 2;
        if (q - lane >= 0) {
            const uint32_t* from = hist + (uint64_t)(q - lane) * QUAD;
            const int c0 = (kf - (int)from[QW]) >> 1;
#pragma unroll
            for (int i = 0; i < WALK_COLS / 2; i++)
                win[lane * (WALK_COLS / 2) + i] = c0 + i >= 0 && c0 + i < QW ? from[c0 + i] : 0u;
        }
        return kf;
    };
    auto offset = [&](int s, int k) {
        const int col = k - (int)hist[(uint64_t)(s >> 2) * QUAD + QW];
        const uint32_t w = col >= 0 && col < AW
                               ? hist[adapt_rec_words(job.bound, NB) + (uint64_t)(s >> 4) * QW + (col >> 1)]
                               : NUL16P;
        return (int)(short)(w >> (16 * (col & 1))) >> SH;
    };
    const int nr = walk<X, OE, E, true>(load, offset, S, n, m, lane, win, evs, job.ev_words, runs_end,
                                        job.run_words, tb, pb);
    walk_done(a, job, S, nr, runs_end, lane);
}

// Scaled penalties (x, o + e, e) the rows are built for.
#define WFA_ADAPT_PENS(F) \
    F(2, 4, 1)            \
    F(1, 1, 1)            \
    F(2, 5, 1)

}  // namespace

bool adapt_supported(const Pen& pen) {
#define WFA_CASE(PX, POE, PE) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE) return true;
    WFA_ADAPT_PENS(WFA_CASE)
#undef WFA_CASE
    return false;
}

hipError_t launch_adapt(const FrontArgs& a, const Pen& pen, bool cigar, int sh, int blocks, int jobs,
                        uint32_t n, uint32_t m, hipStream_t s) {
    if (!jobs) return hipSuccess;
    const int lds = (cigar || blocks > ADAPT_BLOCKS ? WALK_DW * 4 : 0) + seq_lds_bytes(n, m);
#define WFA_GO(PX, POE, PE, SHF, NB, CG) \
    hipLaunchKernelGGL((k_adapt<PX, POE, PE, SHF, NB, CG>), dim3(jobs), dim3(64), lds, s, a)
#define WFA_FORM(PX, POE, PE, NB)                                                                       \
    if (pen.x == PX && pen.oe == POE && pen.e == PE && blocks == NB) {                                  \
        if (cigar) { if (sh) WFA_GO(PX, POE, PE, 1, NB, true); else WFA_GO(PX, POE, PE, 0, NB, true); } \
        else { if (sh) WFA_GO(PX, POE, PE, 1, NB, false); else WFA_GO(PX, POE, PE, 0, NB, false); }     \
        return hipGetLastError();                                                                       \
    }
#define WFA_CASE(PX, POE, PE) WFA_FORM(PX, POE, PE, ADAPT_BLOCKS) WFA_FORM(PX, POE, PE, ADAPT_BLOCKS_WIDE)
    WFA_ADAPT_PENS(WFA_CASE)
#undef WFA_CASE
#undef WFA_FORM
#undef WFA_GO
    return hipErrorInvalidValue;
}

}  // namespace wfa
