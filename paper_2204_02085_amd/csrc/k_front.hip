// Front kernel: long and divergent pairs, a workgroup per pair, wavefront rows
// in registers (rows.h).
//
// Two kernels per batch of pairs:
//
//   k_bound       two wavefronts per pair align greedily, from either end, in
//                 bands of 128 diagonals that follow the furthest points.  Where
//                 they meet there is an alignment of the sum U of their scores,
//                 so no optimal one costs more.
//   k_front       one workgroup per pair.  A cell on diagonal k at step s lies
//                 on an optimal alignment only if a gap back to the end
//                 diagonal still fits, s + e |k - kt| <= U, and only if a gap
//                 from diagonal 0 has reached it.  Both cut the triangle of
//                 cells to a diamond, half of it when U is the score.  Every
//                 lane owns C neighbouring diagonals for the whole pair, so
//                 the rows stay in registers; neighbouring lanes exchange a
//                 column by DPP, neighbouring wavefronts through LDS, with one
//                 barrier per step.  In CIGAR mode the first wavefront then
//                 walks the decision records back (see walk).
//
// What bounds it: VALU issue and the chain of a step (the neighbour's column
// from LDS, the recurrences, two windows of each sequence from LDS, the barrier),
// hidden by the other workgroups of a CU: about 60 instructions per step and
// 128 diagonals, 0.65 to 0.76 of the issue slots in launches that fill the chip.
// Measured on whole calls against the general kernel, whose rows cross L2 and
// HBM and fill the whole triangle: 20 k pairs of 1-10 kbp at 5-10 % with CIGARs
// 24.4 ms (107.5), 5 k of them score-only 5.4 ms (25.0), 24 pairs of 10-20 kbp
// 7.9 to 8.3 ms (66.4).  k_bound takes 2 ms for the 20 k pairs, most of it beside the
// first alignments (from one end only, by one wavefront, the chain of a pair took
// twice as long: 5 k pairs score-only 5.8 ms, the 24 pairs 9.1 ms).
// Columns exchanged every four steps instead, with four columns computed twice on
// either side, saved three of four barriers and cost 7 % more cells: no gain; four
// diagonals per lane: 20 % slower.  The record walk in a kernel of its own took
// 2.8 ms more.
//
// Cells a pruned cell would have fed never beat those of an optimal
// alignment: a missing candidate only lowers offsets off the optimal paths,
// and a cell on one has all its sources on one.  So scores and tie-breaks are
// those of the full wavefronts.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "kernels.h"
#include "rows.h"
#include "walk.h"

namespace wfa {

namespace {

using namespace rows;

// A sequence of `len` bases from its last to its first, into LDS.
__device__ __forceinline__ void stage_reversed(lds_p<uint64_t> dst, const uint64_t* words, int len, int count,
                                               int tid, int bt) {
    for (int w = tid; w < count; w += bt) {
        const int q = len - 32 * (w + 1);  // the first of the word's bases (below 0: as many fewer)
        uint64_t x = 0;
        if (q > -32) {
            const int from = max(q, 0), i = from >> 5, sh = 2 * (from & 31);
            x = words[i] >> sh;
            if (sh && from + 31 < len && ((from + 31) >> 5) > i) x |= words[i + 1] << (64 - sh);
            if (q < 0) x <<= -2 * q;
            x = __builtin_bitreverse64(x);  // bases and the two bits of each; these back
            x = ((x >> 1) & 0x5555555555555555ull) | ((x & 0x5555555555555555ull) << 1);
        }
        dst[w] = x;
    }
}

constexpr int BOUND_ROWS = 5;  // M of four steps, and their maximum

// Two wavefronts per pair, one from either end: a pair's chain of steps is what
// this kernel costs where few pairs are in flight, and each goes half of it.  They
// meet where on one diagonal the offsets from both ends cover the text: an
// alignment of the sum of their scores exists then.
template <int X, int OE, int E, int SH>
__global__ __launch_bounds__(128) void k_bound(FrontArgs a) {
    constexpr int C = 2;
    extern __shared__ __align__(16) unsigned char lds[];
    const uint32_t pair = a.ids[blockIdx.x];
    const PairDesc d = a.pairs[pair];
    const int n = (int)d.p_len, m = (int)d.t_len, kt = m - n;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // LDS: the quad they met in and the reverse window's base per buffer, two
    // buffers of the reverse rows, the sequences, the sequences reversed
    lds_p<int> met = (lds_p<int>)lds;
    lds_p<int> base = met + 2;
    lds_p<uint32_t> rows = (lds_p<uint32_t>)(met + 4);
    lds_p<uint64_t> seq = (lds_p<uint64_t>)(rows + 2 * BOUND_ROWS * 64);
    const int tws = text_words(m), nwp = (n + 31) >> 5;
    lds_p<uint64_t> rev = seq + tws + nwp + 1;
    stage(seq, a.pw, a.tw, d, threadIdx.x, 128);
    stage_reversed(rev, a.tw + d.t_start, m, tws, threadIdx.x, 128);
    stage_reversed(rev + tws, a.pw + d.p_start, n, nwp + 1, threadIdx.x, 128);
    if (threadIdx.x == 0) *met = -1;
    __syncthreads();
    const uint32_t tb = (uint32_t)(uintptr_t)(w ? rev : seq);
    const uint32_t pb = tb + 8 * tws;
    // every base mismatched and the length difference in one gap
    int U = X * min(n, m) + (kt ? (OE - E) + E * abs(kt) : 0);
    const int last = min(U, SH ? 8000 : 16000);  // (the front kernel holds no more)
    int kmin = -64;
    Place<C> pl;
    pl.template set<SH>(n, m, kmin + C * lane);
    Rows<X, OE, E, C, SH, false> row;
    row.clear();
    for (int s = 0;; s += 4) {
        uint32_t mq[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            uint32_t sa[1], sb[1], cm[1], ci[1], cd[1];
            row.sources(sa, sb);
            row.cells(sa, sb, wave_prev(NUL16P, sa[0]), wave_next(NUL16P, sb[0]), cm, ci, cd, false);
            if (u == 0 && s == 0) {
                cm[0] = lane == 32 ? 0xC0000000u : NUL16P;  // M_0[0] = 0
                ci[0] = cd[0] = NUL16P;
            }
            extend<C, SH, LONG_WAVE>(cm, pl, tb, pb);
            row.push(cm, ci, cd);
            mq[u] = cm[0];
        }
        const uint32_t far = pk_max(pk_max(mq[0], mq[1]), pk_max(mq[2], mq[3]));
        lds_p<uint32_t> buf = rows + ((s >> 2) & 1) * (BOUND_ROWS * 64);
        if (w) {
#pragma unroll
            for (int u = 0; u < 4; u++) buf[u * 64 + lane] = mq[u];
            buf[4 * 64 + lane] = far;
            if (lane == 0) base[(s >> 2) & 1] = kmin;
        }
        __syncthreads();
        // (set by the forward wavefront after this quad's barrier at the earliest)
        const int at = __builtin_amdgcn_readfirstlane(*met);
        if ((at >= 0 && at < s) || 2 * s >= last) break;
        if (!w && at < 0) {
            // the reverse columns of this lane's diagonals k and k + 1: kt - k and
            // the one before it
            const int c = kt - (kmin + C * lane) - __builtin_amdgcn_readfirstlane(base[(s >> 2) & 1]);
            auto meets = [&](uint32_t mine, int r) -> bool {
                lds_p<const short> other = (lds_p<const short>)(buf + r * 64);
                const int o0 = c >= 0 && c < 128 ? other[c] : -1, o1 = c >= 1 && c <= 128 ? other[c - 1] : -1;
                const int m0 = (int)(short)mine, m1 = (int)(short)(mine >> 16);
                return (o0 >= 0 && m0 >= 0 && o0 + m0 >= m << SH) || (o1 >= 0 && m1 >= 0 && o1 + m1 >= m << SH);
            };
            if (lanes_where(meets(far, 4))) {
#pragma unroll
                for (int u = 0; u < 4; u++)
                    for (int r = 0; r < 4; r++)
                        if (2 * s + u + r < U && lanes_where(meets(mq[u], r))) U = 2 * s + u + r;
                if (lane == 0) *met = s;
            }
        }
        // follow the furthest point (2 h - k), a lane or two at a time
        const int k0 = kmin + C * lane;
        const int h0 = (int)(short)far << (1 - SH), h1 = (int)(short)(far >> 16) << (1 - SH);
        const int top = wave_max((max(h0 - k0, h1 - k0 - 1) << 6) | lane);
        int shift = top < 0 ? 0 : (top & 63) - 32;  // (below 0: no cell at these steps)
        shift = shift > 8 ? 2 : shift > 2 ? 1 : shift < -8 ? -2 : shift < -2 ? -1 : 0;
        if (shift) {
            for (; shift > 0; shift--, kmin += C) {
#pragma unroll
                for (int j = 0; j < Rows<X, OE, E, C, SH, false>::RM; j++)
                    row.M[j][0] = wave_next(NUL16P, row.M[j][0]);
#pragma unroll
                for (int j = 0; j < E; j++) {
                    row.I[j][0] = wave_next(NUL16P, row.I[j][0]);
                    row.D[j][0] = wave_next(NUL16P, row.D[j][0]);
                }
            }
            for (; shift < 0; shift++, kmin -= C) {
#pragma unroll
                for (int j = 0; j < Rows<X, OE, E, C, SH, false>::RM; j++)
                    row.M[j][0] = wave_prev(NUL16P, row.M[j][0]);
#pragma unroll
                for (int j = 0; j < E; j++) {
                    row.I[j][0] = wave_prev(NUL16P, row.I[j][0]);
                    row.D[j][0] = wave_prev(NUL16P, row.D[j][0]);
                }
            }
            pl.template set<SH>(n, m, kmin + C * lane);
        }
    }
    if (threadIdx.x == 0) a.bounds[blockIdx.x] = U;
}

// The walk over a pair's records.
template <int X, int OE, int E, int SH>
__device__ void walk_job(const FrontArgs& a, const FrontJob& job, int S, int n, int m, int lane,
                         lds_p<uint32_t> win, uint32_t tb, uint32_t pb) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int ROW = WALK_COLS / 2;
    const int rowdw = front_row_words(job.nw, job.cols);
    const uint32_t* hist = a.arena + job.hist;
    uint32_t* evs = a.arena + job.hist + job.hist_words;
    uint32_t* runs_end = evs + job.ev_words + job.run_words;
    auto load = [&](int q, int k) {
        const int c0 = min(max((((k - job.kbase) >> 1) - ROW / 2) & ~3, 0), rowdw - ROW);
        if (q - lane >= 0) {
            const u32x4* from = (const u32x4*)(hist + (uint64_t)front_row(4 * (q - lane)) * rowdw + c0);
            lds_p<u32x4> to = (lds_p<u32x4>)(win + lane * ROW);
#pragma unroll
            for (int i = 0; i < ROW / 4; i++) to[i] = from[i];
        }
        return job.kbase + 2 * c0;
    };
    auto offset = [&](int s, int k) {
        const int col = k - job.kbase;
        const uint32_t w = col >= 0 && (col >> 1) < rowdw ? hist[(uint64_t)(front_row(s) + 4) * rowdw + (col >> 1)] : NUL16P;
        return (int)(short)(w >> (16 * (col & 1))) >> SH;
    };
    const int nr = walk<X, OE, E, false>(load, offset, S, n, m, lane, win, evs, job.ev_words, runs_end,
                                         job.run_words, tb, pb);
    walk_done(a, job, S, nr, runs_end, lane);
}

// The rows of one block of 64 C diagonals, and where it stands.
template <int X, int OE, int E, int C, int SH, bool CIGAR>
struct Block {
    static constexpr int P = C / 2;
    Rows<X, OE, E, C, SH, CIGAR> row;
    Place<C> pl;
    uint32_t sa[P], sb[P];           // sources of the next step
    lds_p<uint32_t> xin, xout;       // the columns next to it
    int k0;                          // this lane's first diagonal
};

// NB blocks of diagonals per wavefront: block b is wavefront b mod nwv's, nwv
// the pair's wavefronts.  With NB = 2 a wavefront holds one block of either
// half of the diamond's diagonals, of which about one is active at a time, so
// no wavefront is idle for half of the pair's steps.
template <int X, int OE, int E, int C, int NB, int SH, bool CIGAR>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(C * NB <= 4 ? 8 : 4)))
void k_front(FrontArgs a) {
    constexpr int P = C / 2, WC = 64 * C;  // columns of a block
    using B = Block<X, OE, E, C, SH, CIGAR>;
    extern __shared__ __align__(16) unsigned char lds[];
    const FrontJob job = a.jobs[blockIdx.x];
    const PairDesc d = a.pairs[job.pair];
    const int n = (int)d.p_len, m = (int)d.t_len, kt = m - n;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nbb = NB * (blockDim.x >> 6);
    // LDS: the step the pair ended at, two buffers of the columns blocks
    // exchange (a block of NULL on either side), the window of the walk, the
    // sequences
    lds_p<int> done = (lds_p<int>)lds;
    lds_p<uint32_t> xch = (lds_p<uint32_t>)(done + 4);
    const int xb = 2 * (nbb + 2);  // words per buffer: {up, down} per block
    lds_p<uint32_t> win = xch + 2 * xb;
    lds_p<uint64_t> seq = (lds_p<uint64_t>)(win + (CIGAR ? WALK_DW : 0));
    stage(seq, a.pw, a.tw, d, threadIdx.x, blockDim.x);
    for (int i = threadIdx.x; i < 2 * xb; i += blockDim.x) xch[i] = NUL16P;
    if (threadIdx.x == 0) *done = -1;
    const uint32_t tb = (uint32_t)(uintptr_t)seq, pb = tb + 8 * text_words(m);
    int edge = lane == 0 || lane == 63;  // lanes that hand a column to the next block
    asm("" : "+v"(edge));

    const int U = job.bound, kbase = job.kbase, nwv = (job.nw + NB - 1) / NB;
    const int ct = kt - kbase;  // column of the end diagonal
    B blk[NB];
#pragma unroll
    for (int i = 0; i < NB; i++) {
        const int b = w + i * nwv;
        blk[i].k0 = kbase + b * WC + lane * C;
        blk[i].pl.template set<SH>(n, m, blk[i].k0);
        blk[i].row.clear();
#pragma unroll
        for (int p = 0; p < P; p++) blk[i].sa[p] = blk[i].sb[p] = NUL16P;
        // lane 0 takes the column below from the block before, lane 63 the one
        // above from the block after; the same lanes hand theirs out
        const int bx = min(b, nbb - 1);
        blk[i].xin = xch + (lane == 63 ? 2 * (bx + 2) + 1 : 2 * bx);
        blk[i].xout = xch + 2 * (bx + 1) + (lane == 63 ? 0 : 1);
    }
    // the block, lane and column of the end cell
    const int eb = ct / WC, elane = (ct % WC) / C, ecol = ct % C;
    int S = -1;
    // one step of block i (u: its place in the quad)
    auto step = [&](B& q, int s, int u, bool owner) {
        const uint32_t xv = q.xin[(u & 1) * xb];
        uint32_t cm[P], ci[P], cd[P];
        q.row.cells(q.sa, q.sb, wave_prev(xv, q.sa[P - 1]), wave_next(xv, q.sb[0]), cm, ci, cd, u == 0);
        if (u == 0 && s == 0) {  // M_0[0] = 0
#pragma unroll
            for (int p = 0; p < P; p++) {
                cm[p] = pk_pair(q.k0 + 2 * p == 0 ? 0 : -16384, q.k0 + 2 * p + 1 == 0 ? 0 : -16384);
                ci[p] = cd[p] = NUL16P;
            }
        }
        // (two blocks with events, or of four columns a lane, have no registers for the other)
        extend<C, SH, NB == 1 || (C == 2 && !CIGAR) ? LONG_WAVE : LONG_LANE>(cm, q.pl, tb, pb);
        q.row.push(cm, ci, cd);
        q.row.sources(q.sa, q.sb);
        if (edge) q.xout[((u + 1) & 1) * xb] = lane == 63 ? q.sa[P - 1] : q.sb[0];
        if (owner && S < 0) {
            uint32_t reg = cm[0];
#pragma unroll
            for (int p = 1; p < P; p++) reg = (ecol >> 1) == p ? cm[p] : reg;
            if (half_at(reg, elane, ecol & 1) == m << SH) S = s + u;
        }
    };
    auto flush = [&](B& q, int s, int b) {
        if (CIGAR) {
            uint32_t* h = a.arena + job.hist + ((uint64_t)front_row(s) * job.nw + b) * (64 * P) + lane * P;
#pragma unroll
            for (int p = 0; p < P; p++) h[p] = q.row.acc[p];
            if ((s & 15) == 0) {
                uint32_t* r = h + (uint64_t)(4 * job.nw) * (64 * P);
#pragma unroll
                for (int p = 0; p < P; p++) r[p] = q.row.M[0][p];
            }
        }
    };
    __syncthreads();
    // wavefronts past the pair's own (a launch's workgroups have one size) make
    // room for other workgroups: barriers count the wavefronts that are left
    if (w >= nwv) return;
    for (int s = 0;; s += 4) {
        if (__builtin_amdgcn_readfirstlane(*done) >= 0 || s > U) break;
        // diagonals of these four steps' cells, with one to spare on each side
        const int reach = s + 3 >= OE ? 1 + (s + 3 - OE) / E : 0;
        const int back = (U - s) / E;
        const int dlo = max(-reach, kt - back) - 1, dhi = min(reach, kt + back) + 1;
        bool act[NB], own[NB];
#pragma unroll
        for (int i = 0; i < NB; i++) {
            const int b = w + i * nwv, lo = kbase + b * WC;
            act[i] = b < job.nw && lo + WC - 1 >= dlo && lo <= dhi;
            own[i] = b == eb;
        }
        auto quad = [&](bool first, bool second) {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (first) step(blk[0], s, u, own[0]);
                if (second) step(blk[NB - 1], s, u, own[NB - 1]);
                if (u == 3) {
                    if (first) flush(blk[0], s, w);
                    if (second) flush(blk[NB - 1], s, w + nwv);
                    if (S >= 0 && lane == 0) *done = S;
                }
                __syncthreads();
            }
        };
        if (NB == 1) {
            if (act[0]) quad(true, false);
        } else {
            if (act[0] && act[NB - 1]) quad(true, true);
            else if (act[0]) quad(true, false);
            else if (act[NB - 1]) quad(false, true);
        }
        bool any = act[0];
#pragma unroll
        for (int i = 1; i < NB; i++) any = any || act[i];
        if (!any) {
#pragma unroll
            for (int u = 0; u < 4; u++) __syncthreads();
        }
    }
    const int S2 = __builtin_amdgcn_readfirstlane(*done);
    if (S2 < 0) {  // the bound did not hold (an internal error): the general kernel takes the pair
        if (threadIdx.x == 0) a.fail_list[atomicAdd(a.fail_count, 1u)] = job.pair;
        return;
    }
    if (!CIGAR) {
        if (threadIdx.x == 0) {
            a.scores[job.pair] = S2 * a.g;
            a.nruns[job.pair] = 0;
        }
        return;
    }
    // every wavefront's records are written; one wavefront walks them while
    // the others' slots go to the next workgroup
    __threadfence_block();
    __syncthreads();
    if (w == 0) walk_job<X, OE, E, SH>(a, job, S2, n, m, lane, win, tb, pb);
}

// Scaled penalties (x, o + e, e) the rows are built for.
#define WFA_FRONT_PENS(F) \
    F(2, 4, 1)            \
    F(1, 1, 1)            \
    F(2, 5, 1)

template <int X, int OE, int E>
struct FrontShape {
    template <int C, int NB, int SH>
    static hipError_t fwd(const FrontArgs& a, bool cigar, int jobs, int waves, int lds, hipStream_t s) {
        if (cigar)
            hipLaunchKernelGGL((k_front<X, OE, E, C, NB, SH, true>), dim3(jobs), dim3(64 * waves), lds, s, a);
        else
            hipLaunchKernelGGL((k_front<X, OE, E, C, NB, SH, false>), dim3(jobs), dim3(64 * waves), lds, s, a);
        return hipGetLastError();
    }
    static hipError_t launch(const FrontArgs& a, const FrontForm& f, bool cigar, int jobs, int waves,
                             int lds, hipStream_t s) {
        if (f.cols == 2 && f.blocks == 1)
            return f.sh ? fwd<2, 1, 1>(a, cigar, jobs, waves, lds, s) : fwd<2, 1, 0>(a, cigar, jobs, waves, lds, s);
        if (f.cols == 2 && f.blocks == 2)
            return f.sh ? fwd<2, 2, 1>(a, cigar, jobs, waves, lds, s) : fwd<2, 2, 0>(a, cigar, jobs, waves, lds, s);
        if (f.cols == 4 && f.blocks == 2)
            return f.sh ? fwd<4, 2, 1>(a, cigar, jobs, waves, lds, s) : fwd<4, 2, 0>(a, cigar, jobs, waves, lds, s);
        return hipErrorInvalidValue;
    }
};

}  // namespace

bool front_supported(const Pen& pen) {
#define WFA_CASE(PX, POE, PE) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE) return true;
    WFA_FRONT_PENS(WFA_CASE)
#undef WFA_CASE
    return false;
}

bool front_fits(uint32_t n, uint32_t m) { return std::max(n, m) <= FRONT_MAX_LEN; }

bool front_shape(const Pen& pen, uint32_t n, uint32_t m, int bound, FrontShapeInfo* f) {
    f->bound = bound;
    f->sh = std::max(n, m) <= 16383 ? 1 : 0;
    // NULL offsets drift up by 1 << sh per step and stay negative
    if (bound > (f->sh ? 8000 : 16000)) return false;
    const long long kt = (long long)m - n, og = pen.oe - pen.e;
    // the diamond's outermost diagonals: where the reach from diagonal 0 and
    // the way back to kt meet, with one to spare
    long long hi = (bound + pen.e * kt - og) / (2 * pen.e) + 2;
    long long lo = -((bound - pen.e * kt - og) / (2 * pen.e) + 2);
    hi = std::min<long long>(std::max<long long>(hi, std::max<long long>(kt, 0)), m);
    lo = std::max<long long>(std::min<long long>(lo, std::min<long long>(kt, 0)), -(long long)n);
    f->kbase = (int)lo;
    f->width = (int)(hi - lo + 1);
    f->ev_words = (uint32_t)(bound / std::min(pen.x, pen.oe) + 64) & ~63u;
    f->run_words = 2 * f->ev_words + 64;
    return f->width <= FRONT_MAX_WIDTH;
}

int front_blocks(int width, int cols) { return (width + 64 * cols - 1) / (64 * cols); }

hipError_t launch_bound(const FrontArgs& a, const Pen& pen, int sh, int jobs, uint32_t n, uint32_t m,
                        hipStream_t s) {
    if (!jobs) return hipSuccess;
    // (the rows; both sequences each way; compares read on past the last)
    const int lds = 16 + 2 * BOUND_ROWS * 256 + 2 * seq_lds_bytes(n, m);
#define WFA_CASE(PX, POE, PE)                                                                        \
    if (pen.x == PX && pen.oe == POE && pen.e == PE) {                                               \
        if (sh) hipLaunchKernelGGL((k_bound<PX, POE, PE, 1>), dim3(jobs), dim3(128), lds, s, a);      \
        else hipLaunchKernelGGL((k_bound<PX, POE, PE, 0>), dim3(jobs), dim3(128), lds, s, a);         \
        return hipGetLastError();                                                                    \
    }
    WFA_FRONT_PENS(WFA_CASE)
#undef WFA_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_front(const FrontArgs& a, const Pen& pen, bool cigar, const FrontForm& f, int jobs,
                        int waves, uint32_t n, uint32_t m, hipStream_t s) {
    if (!jobs) return hipSuccess;
    if (waves < 1 || waves > 16) return hipErrorInvalidValue;
    const int lds = 16 + 16 * (waves * f.blocks + 2) + (cigar ? WALK_DW * 4 : 0) +
                    seq_lds_bytes(n, m);
#define WFA_CASE(PX, POE, PE)                       \
    if (pen.x == PX && pen.oe == POE && pen.e == PE) \
        return FrontShape<PX, POE, PE>::launch(a, f, cigar, jobs, waves, lds, s);
    WFA_FRONT_PENS(WFA_CASE)
#undef WFA_CASE
    return hipErrorInvalidValue;
}

}  // namespace wfa
