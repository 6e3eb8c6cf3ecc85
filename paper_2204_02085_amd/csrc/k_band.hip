// Band kernel: short and middling pairs, a lane group per pair, wavefront rows
// in registers (rows.h).
//
// A group of G = 8, 16, 32 or 64 lanes holds a band of W = 4 G diagonals, four
// to a lane; 64 / G pairs share a wavefront and step through the scores
// together.  Recurrences run on 16-bit pairs in registers, neighbours exchange
// columns by DPP, only the sequences and (CIGAR) the decision records live in
// LDS.  There is no row traffic and no barrier.
//
// A band is exact up to a score its width gives: an alignment that leaves the
// band pays a gap to the first diagonal outside it and a gap back, so while
// the score stays below the cheaper of the two ways out, cells outside the
// band lie on no optimal alignment, and score and tie-breaks are unchanged.  For (4, 6, 2)
// and equal lengths W diagonals hold W + 5 steps; a rule that gives a pair up
// once the wavefront touches the window's edge stops near W / 2.  Pairs that
// need more leave through the overflow list.
//
// What bounds it: VALU issue (all of the issue slots on 1 M pairs of 100 bp with 10
// free bases at each end; about 100 instructions per step and wavefront plus the
// longer compares).  Measured, kernel alone: those pairs with CIGARs
// 0.82 ms, where the lane groups with rows in LDS (k_short, window 64) took
// 2.50 ms; 2 M pairs of 50-300 bp at 0-5 % 2.67 + 0.56 + 0.06 ms over windows
// 32, 64 and 128 against 8.62 + 3.77 ms over 64 and 128; 300 k pairs of 150 bp
// under (1, 0, 1) 0.19 ms against 0.47.  Five wavefronts per SIMD (96 VGPRs,
// some spills outside the steps) beat four (118) by 2 to 3 %.  One loop for
// every lane's longer compares instead of one per column: 25 % slower.
//
// Where few pairs are in flight, the chain of a pair sets the time, for long matches
// that of their compares: forward 32 bases a trip after the first 31, in the replay
// the whole group's lanes, 32 bases each.  100 pairs of 600-1200 bp at 0-1 % took
// 105 us in the kernel with 16 bases a trip and the replay by one lane, now 40; 1 M
// pairs with 10 free bases 0.82 ms either way, the uneven pairs 3.47 ms a call (3.65).
//
// CIGAR: the forward pass keeps four record bits per cell.  The group walks them
// back to the list of edits, then replays the edits from the start: after each edit
// the alignment runs along matches exactly as the forward pass extended, so no
// offset is stored.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include "kernels.h"
#include "pack.h"
#include "rows.h"

namespace wfa {

namespace {

using namespace rows;

constexpr int BAND_C = 4;           // diagonals per lane
constexpr int BAND_TAIL = 256;      // spare LDS bytes: compares of cells off the matrix read on

__device__ __forceinline__ void wave_fence() {
    // a wavefront's LDS traffic is in order; this keeps the compiler in order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int X, int OE, int E, int G, bool CIGAR, bool ENDS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_band(BandArgs a) {
    constexpr int C = BAND_C, P = C / 2, W = G * C, GPW = 64 / G;
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wpb = blockDim.x >> 6;
    const int grp = lane / G, gl = lane % G;
    const bool first = gl == 0, last = gl == G - 1;
    const uint64_t gmask = (~0ull >> (64 - G)) << (grp * G);

    // per group: the text, the pattern, (CIGAR) the records
    lds_p<unsigned char> gb = (lds_p<unsigned char>)lds + (wave * GPW + grp) * a.group_bytes;
    lds_p<uint64_t> ST = (lds_p<uint64_t>)gb;
    lds_p<uint64_t> SP = ST + a.seq_words;
    lds_p<uint32_t> HI = (lds_p<uint32_t>)(SP + a.seq_words);
    const uint32_t tb = (uint32_t)(uintptr_t)ST, pb = (uint32_t)(uintptr_t)SP;

    // persistent: LANE_QUEUES counters 128 bytes apart, wavefront w drawing from
    // counter w mod LANE_QUEUES; the i-th claim of counter c is round i * LANE_QUEUES + c
    // of 64 / G queue entries.  (With one counter for all a claim took 12 ns,
    // which set the time: 1 M pairs of 100 bp score-only 1.55 ms, now 0.59.)
    const uint32_t qid = (blockIdx.x * wpb + wave) % LANE_QUEUES;
    for (uint32_t iter = 0;; iter++) {
        uint32_t qbase;
        if (a.persistent) {
            uint32_t t = 0;
            if (lane == 0) t = atomicAdd(a.queue + qid * 32, 1u);
            const uint64_t r = (uint64_t)__builtin_amdgcn_readfirstlane(t) * LANE_QUEUES + qid;
            qbase = r * GPW >= a.num ? a.num : (uint32_t)(r * GPW);
        } else {
            if (iter) break;
            qbase = (blockIdx.x * wpb + wave) * GPW;
        }
        if (qbase >= a.num) break;
        const uint32_t q = qbase + grp;
        bool active = q < a.num;
        uint32_t pair = 0;
        int n = 0, m = 0;
        uint64_t ps = 0, ts = 0;
        if (active) {
            pair = a.order ? a.order[q] : q;
            if (pair >= a.npairs) {  // a corrupt permutation must not fault: skip the entry
                active = false;
                pair = 0;
            }
        }
        if (active) {
            const PairDesc d = a.pairs[pair];
            n = (int)d.p_len;
            m = (int)d.t_len;
            ps = d.p_start;
            ts = d.t_start;
        }
        const int nwp = (n + 31) >> 5, nwt = (m + 31) >> 5;
        const int kt = m - n;
        const int kmin = (kt >> 1) - W / 2;
        // start diagonals [ks0, ks1] and end diagonals [ke0, ke1]
        int ks0 = 0, ks1 = 0, ke0 = kt, ke1 = kt;
        if (ENDS) {
            ks0 = -min(a.ends.pb, n);
            ks1 = min(a.ends.tb, m);
            ke0 = kt - min(a.ends.te, m);
            ke1 = kt + min(a.ends.pe, n);
        }
        // the largest step at which no alignment has been outside the band
        int smax;
        {
            const int out0 = kmin - 1, out1 = kmin + W;
            const int hi = 2 * (OE - E) + E * ((out1 - ks1) + (out1 - ke1));
            const int lo = 2 * (OE - E) + E * ((ks0 - out0) + (ke0 - out0));
            smax = min(min(hi, lo) - 1, a.cap);
            if (ks1 >= out1 || ke1 >= out1 || ks0 <= out0 || ke0 <= out0) smax = -1;
        }
        bool run = active && smax >= 0 && nwp + 1 <= a.seq_words && nwt + 1 <= a.seq_words;
        if (a.ascii) {  // packed on the way in: no packed copy in memory
            bool ok = true;
            const uint8_t* pa = (const uint8_t*)a.pw;
            const uint8_t* ta = (const uint8_t*)a.tw;
            for (int w = gl; w < a.seq_words; w += G) {
                bool okt = true, okp = true;
                ST[w] = (run && w < nwt) ? pack_word(ta, ts + 32ull * w, min(32, m - 32 * w), okt) : 0ull;
                SP[w] = (run && w < nwp) ? pack_word(pa, ps + 32ull * w, min(32, n - 32 * w), okp) : 0ull;
                ok = ok && okt && okp;
            }
            if (!ok) atomicMin(a.err_pair, (unsigned long long)pair);
        } else {
            for (int w = gl; w < a.seq_words; w += G) {
                ST[w] = (run && w < nwt) ? a.tw[ts + w] : 0ull;
                SP[w] = (run && w < nwp) ? a.pw[ps + w] : 0ull;
            }
        }
        if (!run) {  // an idle group computes on two empty sequences
            n = m = 0;
        }
        wave_fence();

        const int k0 = (run ? kmin : -(W / 2)) + C * gl;
        Place<C> pl;
        pl.template set<1>(n, m, k0);
        // the limit at each end diagonal (reached: the alignment ends there),
        // a value no offset takes elsewhere
        uint32_t tg[P];
#pragma unroll
        for (int p = 0; p < P; p++) {
            const int ka = k0 + 2 * p, kb = ka + 1;
            tg[p] = pk_pair(ka >= ke0 && ka <= ke1 ? (int)(pl.lim[p] & 0xffffu) : 0x7fff,
                            kb >= ke0 && kb <= ke1 ? (int)(pl.lim[p] >> 16) : 0x7fff);
        }
        Rows<X, OE, E, C, 1, CIGAR> row;
        row.clear();
        int S = -1;
        int ecol = W;  // ends-free: lowest column of this lane that ends the alignment
        uint64_t running = lanes_where(run);  // lanes of groups still aligning
        // the first step at which one of them has to hand its pair over
        auto next_limit = [&]() -> int {
            int lim = run ? smax : INT_MAX;
#pragma unroll
            for (int off = 32; off >= G; off >>= 1) lim = min(lim, __shfl_xor(lim, off));
            return __builtin_amdgcn_readfirstlane(lim);
        };
        int limit = next_limit();
        int s = 0;
        while (running) {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (!running) break;
                uint32_t sa[P], sb[P], cm[P], ci[P], cd[P];
                row.sources(sa, sb);
                row.cells(sa, sb, group_prev<G>(sa[P - 1], first), group_next<G>(sb[0], last), cm,
                          ci, cd, u == 0);
                if (u == 0 && s == 0) {  // M_0[k] = max(k, 0) on the start diagonals
#pragma unroll
                    for (int p = 0; p < P; p++) {
                        const int ka = k0 + 2 * p, kb = ka + 1;
                        cm[p] = pk_pair(ka >= ks0 && ka <= ks1 ? 2 * max(ka, 0) : -16384,
                                        kb >= ks0 && kb <= ks1 ? 2 * max(kb, 0) : -16384);
                        ci[p] = cd[p] = NUL16P;
                    }
                }
                extend<C, 1, LONG_LANE>(cm, pl, tb, pb);
                row.push(cm, ci, cd);
                // a cell at its end diagonal's limit ends its pair
                uint32_t z = cm[0] ^ tg[0];
#pragma unroll
                for (int p = 1; p < P; p++) z = pk_minu(z, cm[p] ^ tg[p]);
                const uint64_t hits = (lanes_where((z & 0xffffu) == 0) | lanes_where(z < 0x10000u)) & running;
                if (hits) {
#pragma unroll
                    for (int p = P - 1; p >= 0; p--) {
                        const uint32_t y = cm[p] ^ tg[p];
                        if (run && y < 0x10000u) ecol = C * gl + 2 * p + 1;
                        if (run && (y & 0xffffu) == 0) ecol = C * gl + 2 * p;
                    }
                    if (run && (hits & gmask)) {
                        S = s;
                        run = false;
                    }
                    running = lanes_where(run);
                    if (s < limit) limit = next_limit();
                }
                if (s >= limit) {
                    if (run && s >= smax) run = false;  // hands the pair over (S < 0)
                    running = lanes_where(run);
                    limit = next_limit();
                }
                if (CIGAR && (u == 3 || !running)) {
                    lds_p<uint32_t> h = HI + (s >> 2) * (W / 2) + gl * P;
#pragma unroll
                    for (int p = 0; p < P; p++) h[p] = row.acc[p] << (4 * (3 - u));
                }
                s++;
            }
        }
        if (CIGAR) {
#pragma unroll
            for (int off = G / 2; off >= 1; off >>= 1) ecol = min(ecol, __shfl_xor(ecol, off));
            wave_fence();
        }

        bool overflow = active && S < 0;
        int cnt = 0;
        if (CIGAR && active && !overflow) {
            // walk: the edits from the end back to step 0, from the top of the
            // group's records down (the walk has consumed at least as many
            // steps as it has written words, and reads only below); every lane of
            // the group takes it alike, and stores the same words
            const int top = a.hist_words;
            int ws = S, k = kmin + ecol, ne = 0;
            bool bad = ecol >= W;
            while (!bad && ws > 0) {
                const int col = k - kmin;
                const uint32_t f = record_of(HI[(ws >> 2) * (W / 2) + (col >> 1)], ws, col);
                int kind = EV_X, len = 1;
                if (!(f & 1)) {
                    ws -= X;
                } else {
                    const bool ins = !(f & 2);
                    const int dk = ins ? -1 : 1;
                    const uint32_t more = ins ? 4u : 8u;
                    kind = ins ? EV_I : EV_D;
                    len = 0;
                    for (;;) {
                        len++;
                        k += dk;
                        const int cc = k - kmin;
                        if (ws <= 0 || (unsigned)cc >= (unsigned)W) {
                            bad = true;
                            break;
                        }
                        const uint32_t g = record_of(HI[(ws >> 2) * (W / 2) + (cc >> 1)], ws, cc);
                        ws -= (g & more) ? E : OE;
                        if (!(g & more)) break;
                    }
                }
                if (ws < 0) bad = true;
                if (!bad) HI[top - 1 - ne] = (uint32_t)(len << 2 | kind);
                ne++;
            }
            wave_fence();
            // replay: from the start along matches, edit by edit; runs go to
            // the front of the records, in alignment order.  32 bases a compare,
            // stores without branches (a store past the last run is overwritten);
            // a longer match is followed by the group, 32 bases to a lane.
            int h = max(k, 0), v = h - k;
            int nr = 0, last_op = -1;  // -1: a match run, or none
            uint32_t cur = 0;          // the last edit run
            auto edit = [&](int op, int len) {
                const bool same = op == last_op;
                cur = same ? cur + ((uint32_t)len << 4) : ((uint32_t)len << 4) | (uint32_t)op;
                nr += same ? 0 : 1;
                HI[nr - 1] = cur;
                last_op = op;
            };
            // matching bases from o on, at most 32
            auto match32 = [&](int o) -> int {
                const uint32_t x0 = win16(tb, 2 * (h + o)) ^ win16(pb, 2 * (v + o));
                const uint32_t x1 = win16(tb, 2 * (h + o) + 32) ^ win16(pb, 2 * (v + o) + 32);
                const uint64_t x = ((uint64_t)x1 << 32) | x0;
                return x ? (int)(__builtin_ctzll(x) >> 1) : 32;
            };
            if (!bad) {
                if (ENDS) {
                    if (k > 0) edit(2, k);
                    if (k < 0) edit(3, -k);
                }
                for (int e2 = ne;; e2--) {
                    // matches from (v, h) on
                    const int left = min(n - v, m - h);
                    int mm = match32(0);
                    for (bool on = mm == 32 && left > 32; on;) {
                        const int z = mm + 32 * gl < left ? match32(mm + 32 * gl) : 0;
                        const uint64_t stop = lanes_where(z < 32) & gmask;
                        on = stop == 0;
                        const int l = on ? lane : (int)__builtin_ctzll(stop);
                        mm += on ? 32 * G : 32 * (l - grp * G) + __shfl(z, l);
                    }
                    mm = min(mm, left);
                    HI[nr] = (uint32_t)mm << 4;
                    nr += mm > 0 ? 1 : 0;
                    last_op = mm > 0 ? -1 : last_op;
                    h += mm;
                    v += mm;
                    if (e2 == 0) break;
                    const uint32_t ev = HI[top - e2];
                    const int len = (int)(ev >> 2), kind = (int)(ev & 3);
                    edit(1 + kind, len);
                    h += kind != EV_D ? len : 0;
                    v += kind != EV_I ? len : 0;
                    if (h > m || v > n) {
                        bad = true;
                        break;
                    }
                }
                if (!ENDS && (h != m || v != n)) bad = true;
                if (ENDS && !bad) {
                    if (h < m && v < n) bad = true;
                    if (v < n) edit(3, n - v);
                    if (h < m) edit(2, m - h);
                }
            }
            if (bad || nr > a.slot_cap) overflow = true;
            cnt = nr;
        }
        if (overflow) cnt = 0;
        if (active && first) {
            if (overflow) {
                const uint32_t at = atomicAdd(a.ovf_count, 1u);
                a.ovf_list[at] = pair;
            } else {
                a.scores[pair] = S * a.g;
                a.nruns[pair] = (uint32_t)cnt;
            }
        }
        if (CIGAR) {
            // the groups' runs, last to first, packed one after another
            wave_fence();
            const bool done = active && first && !overflow;
            int pre = 0;
#pragma unroll
            for (int g2 = 0; g2 < GPW; g2++) {
                const int cg = __shfl(cnt, g2 * G);
                pre += g2 < grp ? cg : 0;
            }
            const int mine = __shfl(cnt, grp * G);
            const uint64_t base = (uint64_t)qbase * a.slot_cap + (uint64_t)pre;
            for (int r = gl; r < mine; r += G) a.slots[base + r] = HI[mine - 1 - r];
            if (done) a.run_src[pair] = base + a.run_src_add;
        }
        wave_fence();
    }
}

// LDS bytes of one group: both sequences, the records of `cap` + 1 steps and a
// spare quad of steps; an odd multiple of eight dwords, so that the groups of
// a wavefront start at different banks
int group_words(int seq_words, int hist_words) {
    int w = 4 * seq_words + hist_words;
    w = (w + 7) & ~7;
    if (!((w >> 3) & 1)) w += 8;
    return w;
}

template <int X, int OE, int E, int G>
struct BandShape {
    static hipError_t launch(const BandArgs& a, bool cigar, int bt, int grid, int lds, hipStream_t s) {
        const bool ends = a.ends.pb || a.ends.pe || a.ends.tb || a.ends.te;
        if (cigar && ends)
            hipLaunchKernelGGL((k_band<X, OE, E, G, true, true>), dim3(grid), dim3(bt), lds, s, a);
        else if (cigar)
            hipLaunchKernelGGL((k_band<X, OE, E, G, true, false>), dim3(grid), dim3(bt), lds, s, a);
        else if (ends)
            hipLaunchKernelGGL((k_band<X, OE, E, G, false, true>), dim3(grid), dim3(bt), lds, s, a);
        else
            hipLaunchKernelGGL((k_band<X, OE, E, G, false, false>), dim3(grid), dim3(bt), lds, s, a);
        return hipGetLastError();
    }
    static int occupancy(bool cigar, bool ends, int bt, int lds) {
        int blocks = 0;
        const void* f = cigar ? (ends ? (const void*)k_band<X, OE, E, G, true, true>
                                      : (const void*)k_band<X, OE, E, G, true, false>)
                              : (ends ? (const void*)k_band<X, OE, E, G, false, true>
                                      : (const void*)k_band<X, OE, E, G, false, false>);
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, f, bt, lds) == hipSuccess ? blocks
                                                                                               : 0;
    }
};

// Scaled penalties (x, o + e, e) the rows are built for.
#define WFA_BAND_PENS(F, G) \
    F(2, 4, 1, G)           \
    F(1, 1, 1, G)           \
    F(2, 5, 1, G)
#define WFA_BAND_SHAPES(F) \
    WFA_BAND_PENS(F, 8) WFA_BAND_PENS(F, 16) WFA_BAND_PENS(F, 32) WFA_BAND_PENS(F, 64)

}  // namespace

bool band_supported(const Pen& pen, int window) {
#define WFA_CASE(PX, POE, PE, G) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE && window == G * BAND_C) return true;
    WFA_BAND_SHAPES(WFA_CASE)
#undef WFA_CASE
    return false;
}

bool band_plan(const Pen& pen, bool cigar, int window, int step_cap, uint32_t max_len, int block_threads,
               bool ends, BandPlan* bp) {
    if (!band_supported(pen, window) || max_len > 16383) return false;
    const int G = window / BAND_C;
    bp->window = window;
    bp->lanes = G;
    // no pair of this band can run past this step (see smax in the kernel)
    bp->cap = 2 * (pen.oe - pen.e) + pen.e * window - 1;
    if (step_cap > 0 && step_cap < bp->cap) bp->cap = step_cap;
    bp->seq_words = (int)((max_len + 31) / 32) + 1;
    bp->hist_words = cigar ? (bp->cap / 4 + 2) * (window / 2) : 0;
    // an edit run and a match run per event, the match run and the free run at
    // either end
    bp->slot_cap = 2 * (bp->cap / (pen.x < pen.oe ? pen.x : pen.oe) + 1) + 2 + (ends ? 2 : 0);
    bp->group_bytes = 4 * group_words(bp->seq_words, bp->hist_words);
    int bt = block_threads ? block_threads : 256;
    const int gpw = 64 / G;
    while (bt > 64 && (bt / 64) * gpw * bp->group_bytes + BAND_TAIL > 64 * 1024) bt -= 64;
    bp->block_threads = bt;
    bp->lds_per_block = (bt / 64) * gpw * bp->group_bytes + BAND_TAIL;
    return bp->lds_per_block <= 64 * 1024;
}

int band_max_blocks_per_cu(const Pen& pen, const BandPlan& bp, bool cigar, bool ends) {
#define WFA_CASE(PX, POE, PE, G) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE && bp.lanes == G) \
        return BandShape<PX, POE, PE, G>::occupancy(cigar, ends, bp.block_threads, bp.lds_per_block);
    WFA_BAND_SHAPES(WFA_CASE)
#undef WFA_CASE
    return 0;
}

hipError_t launch_band(const BandArgs& a, const Pen& pen, const BandPlan& bp, bool cigar, int grid,
                       hipStream_t s) {
#define WFA_CASE(PX, POE, PE, G) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE && bp.lanes == G) \
        return BandShape<PX, POE, PE, G>::launch(a, cigar, bp.block_threads, grid, bp.lds_per_block, s);
    WFA_BAND_SHAPES(WFA_CASE)
#undef WFA_CASE
    return hipErrorInvalidValue;
}

}  // namespace wfa
