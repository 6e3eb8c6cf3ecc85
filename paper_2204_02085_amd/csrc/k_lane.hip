// One lane per pair: short reads under a fixed penalty set, every wavefront row
// of a pair in the registers of one lane, 64 pairs stepping together.
//
// The paper runs one pair per DPU thread (Introduction and Methods); on a
// GPU the same independence puts one pair on each lane.  What makes this pay on
// CDNA is that, for fixed scaled penalties (x', o'+e', e'), which (s, k) cells can
// matter does not depend on the sequences:
//
//   M_0[0] exists; I_s[k] exists if M_{s-o'-e'}[k-1] or I_{s-e'}[k-1] does;
//   D_s[k] exists if M_{s-o'-e'}[k+1] or D_{s-e'}[k+1] does; M_s[k] exists
//   if M_{s-x'}[k], I_s[k] or D_s[k] does;
//   and a pair that ends by step CAP on a diagonal kt of at most KT has no
//   cell of an optimal alignment with s + e' |k - kt| > CAP.
//
// So the kernel is unrolled at compile time over a diamond of registers, two
// neighbouring diagonals to each as 16-bit offsets (rows.h): 81 register-steps
// for steps 0..16 under (4, 6, 2), every source a constant register, the
// neighbour's column one funnel shift away, no data exchange between lanes.
// Offsets past the matrix are dropped from M after the maximum (rows.h has the
// argument), so scores and tie-breaks are those of the full wavefronts.
//
// What bounds it: VALU issue (0.9 of the slots with CIGARs, all of them without).
// About 50 instructions per register and step with CIGARs, 15 bases of each
// cell's matches among them; a wavefront follows longer matches, 32 bases at a
// time, while one of its lanes has some.  5 M pairs of 100 bp at E = 4 % in the
// kernel: 1.01 ms with CIGARs, 0.74 without, where a form with a byte per
// diagonal and a cell at a time, over all 167 cells that can hold an offset, took
// 1.48 and 1.03.
//
// With 16 steps there are two forms: KT = 4 as above, for reads of a few edits,
// and KT = 13, every diagonal 16 steps can reach, 106 register-steps, for reads
// with longer gaps (the rule between them stands where the batch is planned).
// 1 M pairs with a gap of 6 bases each 0.18 ms with CIGARs, by the form with a byte
// per diagonal 0.18, handed over by the narrow form 1.36.
// Steps past the last lane's end are skipped within a quad as well, by a branch
// around a step's cells, which also keeps the compiler from mixing two steps: no
// spills in the narrow form (20 bytes without), and those pairs 0.23 ms without.
//
// LDS per wavefront, lane-interleaved (dword q of lane l at q * 64 + l, so 64
// lanes reading "their" dword q hit 64 different banks): both sequences in 2-bit
// words, and (CIGAR) the runs.  Global memory per wavefront, interleaved the same
// way: the decision records, four bits a cell, four steps of a register to a
// dword.  Every lane walks its own pair's records back to at most eight edits, kept
// in a register pair, and replays these from the start along matches.
//
// A pair leaves through the overflow list (to the band kernel's passes) when a
// sequence is longer than LMAX bases, when its end diagonal lies beyond KT,
// or when it needs more than CAP steps.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "kernels.h"
#include "pack.h"
#include "rows.h"

namespace wfa {

namespace {

using namespace rows;

template <class T>
using lptr = lds_p<T>;
template <class T>
using gptr_t = __attribute__((address_space(1))) T*;

// Which registers (diagonals 2p and 2p + 1, p = index - PR) hold cells at each
// step, which have records, and where these go.
template <int X, int OE, int E, int CAP, int KT>
struct LanePlan {
    static constexpr int reach(int s) {  // largest |k| of the diamond at step s
        if (s < OE) return 0;
        const int out = 1 + (s - OE) / E, back = (CAP - s) / E + KT;
        return out < back ? out : back;
    }
    static constexpr int most() {
        int r = 0;
        for (int s = 0; s <= CAP; s++) r = reach(s) > r ? reach(s) : r;
        return r;
    }
    static constexpr int PR = (most() + 2) / 2;
    static constexpr int NP = 2 * PR, Q = CAP / 4;
    bool m[CAP + 1][NP] = {}, i[CAP + 1][NP] = {}, d[CAP + 1][NP] = {}, rec[CAP + 1][NP] = {};
    bool a[CAP + 1][NP] = {}, b[CAP + 1][NP] = {};  // sources of insertions, deletions
    // a record word of this quad of steps (4 q + 1 to 4 q + 4: so many single
    // edits end with a quad)
    bool acc[Q][NP] = {};
    int lo[Q] = {}, off[Q] = {};                    // its row: off + index
    int rows = 0;
    constexpr bool inside(int s, int p) const {
        const int k0 = 2 * (p - PR), k1 = k0 + 1;
        const int least = k0 >= 0 ? k0 : -k1;
        return least <= reach(s);
    }
    constexpr LanePlan() {
        m[0][PR] = true;
        for (int s = 1; s <= CAP; s++) {
            for (int p = 0; p < NP; p++) {
                a[s][p] = (s >= OE && m[s - OE][p]) || (s >= E && i[s - E][p]);
                b[s][p] = (s >= OE && m[s - OE][p]) || (s >= E && d[s - E][p]);
            }
            for (int p = 0; p < NP; p++) {
                if (!inside(s, p)) continue;
                i[s][p] = a[s][p] || (p > 0 && a[s][p - 1]);
                d[s][p] = b[s][p] || (p + 1 < NP && b[s][p + 1]);
                m[s][p] = (s >= X && m[s - X][p]) || i[s][p] || d[s][p];
            }
            for (int p = 0; p < NP; p++)
                rec[s][p] = s >= OE && (m[s][p] || (a[s][p] && p + 1 < NP && m[s][p + 1]) ||
                                        (b[s][p] && p > 0 && m[s][p - 1]));
        }
        for (int q = 0; q < Q; q++) {
            int first = NP, last = -1;
            for (int p = 0; p < NP; p++) {
                for (int s = 4 * q + 1; s <= 4 * q + 4; s++) acc[q][p] = acc[q][p] || rec[s][p];
                if (acc[q][p]) {
                    first = p < first ? p : first;
                    last = p;
                }
            }
            lo[q] = first;
            off[q] = last < 0 ? 0 : rows - first;
            if (last >= 0) rows += last - first + 1;
        }
    }
    // off of every quad, a byte each (they are above -NP)
    constexpr uint64_t offs() const {
        uint64_t w = 0;
        for (int q = 0; q < Q; q++) w |= (uint64_t)(off[q] + NP) << (8 * q);
        return w;
    }
};

template <int X, int OE, int E, int CAP, int KT, int LMAX, bool CIGAR>
struct LaneKernel {
    static_assert(E == 1 && CAP % 4 == 0 && CAP <= 16 && LMAX <= 127, "see the walk and the records");
    using Plan = LanePlan<X, OE, E, CAP, KT>;
    static constexpr Plan plan{};
    static constexpr int NP = Plan::NP, PR = Plan::PR;
    static constexpr int RM = X > OE ? X : OE;
    static constexpr int SQ = (LMAX >> 4) + 3;  // dwords per sequence column
    static_assert(SQ % 2 == 0, "staged by words");
    static constexpr int EDITS = CAP / (X < OE ? X : OE);
    static_assert(6 * EDITS <= 64, "the edits of a pair fill a register pair");
    // Rows of the runs, one to spare.  Until the runs are made they hold the
    // first record rows; the other records go to global memory.
    static constexpr int RUNS = CIGAR ? 2 * EDITS + 2 : 0;
    static constexpr int WAVE_BYTES = (2 * SQ + RUNS) * 256;
    static constexpr int HIST_DW = CIGAR && plan.rows > RUNS ? plan.rows - RUNS : 0;
    static constexpr uint32_t ONE = 0x00020002u;  // offsets are doubled
    static constexpr uint32_t STOP = 0x80000000u;
    static constexpr int TLO = PR - (KT + 1) / 2, THI = PR + KT / 2;  // registers of end diagonals

    struct St {
        uint32_t M[RM][NP], I[NP], D[NP];  // M of step s in row s % RM
        uint32_t acc[NP];
        uint32_t n2, m2;  // the lengths doubled, in both halves
        uint32_t tb, pb;  // LDS addresses of the lane's columns
        int tsh, tp;      // the end diagonal's half (a shift) and register
        int S;
        lptr<uint32_t> R;    // record row r at R[r * 64], from RUNS on
        gptr_t<uint32_t> H;  // at H[(r - RUNS) * 64]
    };

    // dwords q and q + 1 (and q + 2) of a lane's column
    static __device__ __forceinline__ lptr<const uint32_t> at(uint32_t col, uint32_t q) {
        return (lptr<const uint32_t>)(uintptr_t)(col + (q << 8));
    }
    static __device__ __forceinline__ uint32_t ffbl(uint32_t x) {
        uint32_t z;
        asm("v_ffbl_b32 %0, %1" : "=v"(z) : "v"(x));
        return z;
    }

    // Extension of one register's two cells (see rows.h).
    template <int PI>
    static __device__ __forceinline__ uint32_t extend(const St& st, uint32_t m) {
        constexpr int k0 = 2 * (PI - PR);
        constexpr uint32_t SAFE = k0 >= 0 ? (uint32_t)(2 * k0) | ((uint32_t)(2 * k0 + 2) << 16) : 0u;
        // the largest offset, min(m, n + k): below every offset on the diagonals
        // left of the matrix, and an offset on one to the right of it is past m
        constexpr uint32_t K2 = (uint32_t)(2 * k0 & 0xffff) | ((uint32_t)(2 * k0 + 2) << 16);
        const uint32_t lim = bits(__builtin_elementwise_min(as_s(st.m2), as_s(pk_add(st.n2, K2))));
        const uint32_t bad = pk_sign(m | pk_sub(lim, m));
        const uint32_t hv = (bad & SAFE) | (~bad & m);
        uint32_t t0[2], t1[2], p0[2], p1[2], h[2], v[2], x[2], r[2];
#pragma unroll
        for (int c = 0; c < 2; c++) {
            h[c] = c ? hv >> 16 : hv & 0xffffu;
            v[c] = h[c] - (uint32_t)(2 * (k0 + c));
            const lptr<const uint32_t> t = at(st.tb, c ? hv >> 21 : __builtin_amdgcn_ubfe(hv, 5, 11));
            const lptr<const uint32_t> p = at(st.pb, v[c] >> 5);
            t0[c] = t[0];
            t1[c] = t[64];
            p0[c] = p[0];
            p1[c] = p[64];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 2; c++) {
            x[c] = (__builtin_amdgcn_alignbit(t1[c], t0[c], h[c]) ^
                    __builtin_amdgcn_alignbit(p1[c], p0[c], v[c])) | STOP;
            r[c] = ffbl(x[c]);
        }
        if (lanes_where(min(x[0], x[1]) == STOP)) {
            const uint32_t left = pk_sub(lim, hv) & ~bad;
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const uint32_t end = c ? left >> 16 : left & 0xffffu;
                if (x[c] == STOP && end > 30) {
                    uint32_t done = 30, z;
                    do {
                        const uint32_t hd = h[c] + done, vd = v[c] + done;
                        const lptr<const uint32_t> t = at(st.tb, hd >> 5), p = at(st.pb, vd >> 5);
                        const uint32_t ta = t[0], tm = t[64], tz = t[128];
                        const uint32_t pa = p[0], pm = p[64], pz = p[128];
                        const uint32_t y0 = __builtin_amdgcn_alignbit(tm, ta, hd) ^ __builtin_amdgcn_alignbit(pm, pa, vd);
                        const uint32_t y1 = __builtin_amdgcn_alignbit(tz, tm, hd) ^ __builtin_amdgcn_alignbit(pz, pm, vd);
                        // ~0 for a zero word: the sum saturates
                        z = min(min(ffbl(y0), __builtin_elementwise_add_sat(ffbl(y1), 32u)), 64u);
                        done += z;
                    } while (z >= 64 && done < end);
                    r[c] = done;
                }
            }
        }
        const uint32_t rr = (r[0] | (r[1] << 16)) & 0xFFFEFFFEu;
        const uint32_t e = pk_minu(hv + rr, lim);
        return (bad & NUL16P) | (~bad & e);
    }

    // The best sources of step S of gaps into the next diagonals, and the M cells
    // they open from.
    template <int S, int PI>
    static __device__ __forceinline__ uint32_t opens(const St& st) {
        if constexpr (PI < NP && S >= OE && plan.m[S >= OE ? S - OE : 0][PI < NP ? PI : 0])
            return st.M[(S + RM - OE) % RM][PI];
        return NUL16P;
    }
    template <int S, int PI, bool INS>
    static __device__ __forceinline__ uint32_t source(const St& st) {
        if constexpr (PI < NP && S >= E) {
            constexpr bool gap = INS ? plan.i[S - E][PI] : plan.d[S - E][PI];
            constexpr bool open = S >= OE && plan.m[S >= OE ? S - OE : 0][PI];
            if constexpr (gap && open) return pk_max(opens<S, PI>(st), INS ? st.I[PI] : st.D[PI]);
            if constexpr (gap) return INS ? st.I[PI] : st.D[PI];
        }
        return opens<S, PI>(st);
    }

    // One register of step S: its cells from the rows, extended, in place.  The
    // registers go upwards; `ap` and `b` carry the insertion source of the one
    // before and the deletion source of this one.
    template <int S, int PI>
    static __device__ __forceinline__ void cells(St& st, uint32_t& ap, uint32_t& b, uint32_t& z) {
        const uint32_t open = opens<S, PI>(st), a = source<S, PI, true>(st);
        const uint32_t bn = source<S, PI + 1, false>(st);
        [[maybe_unused]] uint32_t nx = 0, ni = 0, ai = 0, ad = 0;
        if constexpr (CIGAR && plan.rec[S][PI]) {
            // gaps into the next diagonals up and down: extended (ties: opened)
            constexpr bool ho = S >= OE && plan.m[S >= OE ? S - OE : 0][PI];
            if constexpr (plan.a[S][PI]) ai = ho ? pk_ne(a, open) : 0x00010001u;
            if constexpr (plan.b[S][PI]) ad = ho ? pk_ne(b, open) : 0x00010001u;
        }
        uint32_t m = NUL16P, i = NUL16P, d = NUL16P;
        if constexpr (plan.m[S][PI]) {
            constexpr bool hx = S >= X && plan.m[S >= X ? S - X : 0][PI];
            constexpr bool hi = plan.i[S][PI], hd = plan.d[S][PI];
            uint32_t x = NUL16P;
            if constexpr (hx) m = x = pk_add(st.M[(S + RM - X) % RM][PI], ONE);
            if constexpr (hi) {
                i = pk_add(__builtin_amdgcn_alignbit(a, ap, 16), ONE);
                m = hx ? pk_max(m, i) : i;
            }
            if constexpr (hd) {
                d = __builtin_amdgcn_alignbit(bn, b, 16);
                m = hx || hi ? pk_max(m, d) : d;
            }
            if constexpr (CIGAR && plan.rec[S][PI]) {
                if constexpr (!hx) nx = 0x00010001u;
                else if constexpr (hi || hd) nx = pk_ne(m, x);
                if constexpr (!hi) ni = 0x00010001u;
                else if constexpr (hx || hd) ni = pk_ne(m, i);
            }
        }
        if constexpr (CIGAR && plan.rec[S][PI]) {
            const uint32_t rec = shl_or<1>(shl_or<1>(shl_or<1>(ad, ai), ni), nx);
            constexpr int sh = 4 * (3 - ((S - 1) & 3));
            if constexpr (fresh(S, PI)) st.acc[PI] = rec << sh;
            else st.acc[PI] = shl_or<sh>(rec, st.acc[PI]);
        }
        if constexpr (plan.m[S][PI]) {
            m = extend<PI>(st, m);
            st.M[S % RM][PI] = m;
            if constexpr (PI >= TLO && PI <= THI) z = st.tp == PI ? m : z;
        }
        if constexpr (plan.i[S][PI]) st.I[PI] = i;
        if constexpr (plan.d[S][PI]) st.D[PI] = d;
        ap = a;
        b = bn;
    }
    // no earlier step of S's quad has a record of this register
    static constexpr bool fresh(int S, int p) {
        for (int s = ((S - 1) & ~3) + 1; s < S; s++)
            if (plan.rec[s][p]) return false;
        return true;
    }

    template <int S, int... Ps>
    static __device__ __forceinline__ bool step(St& st, std::integer_sequence<int, Ps...>) {
        // (through an empty asm each step: else the compiler hoists the address of
        // every record row out of the pair loop and keeps them all in registers)
        asm volatile("" : "+v"(st.H));
        uint32_t z = ~0u;
        if constexpr (S == 0) {
            st.M[0][PR] = extend<PR>(st, 0xC0000000u);  // M_0[0] = 0
            z = st.tp == PR ? st.M[0][PR] : z;
        } else if (S % 4 == 1 || lanes_where(st.S < 0)) {  // (a quad begins with lanes that go on)
            uint32_t ap = NUL16P, b = source<S, 0, false>(st);
            (cells<S, Ps>(st, ap, b, z), ...);
        }
        const bool hit = ((z >> st.tsh) & 0xffffu) == (st.m2 & 0xffffu);
        st.S = st.S < 0 && hit ? S : st.S;
        // a quad's end: its record words, and whether any lane goes on (exits
        // within a quad, with record words to store, cost 50 spilled registers)
        if constexpr (S == 0 || S % 4 != 0) return true;
        if constexpr (CIGAR && S > 0) {
#pragma unroll
            for (int p = 0; p < NP; p++) {
                const int row = plan.off[(S - 1) >> 2] + p;
                if (!plan.acc[(S - 1) >> 2][p]) continue;
                if (row < RUNS) st.R[row * 64] = st.acc[p];
                else st.H[(row - RUNS) * 64] = st.acc[p];
            }
        }
        return lanes_where(st.S < 0) != 0;
    }
    template <int S>
    static __device__ __forceinline__ bool step_if(St& st) {
        if constexpr (has_step(S)) return step<S>(st, std::make_integer_sequence<int, NP>{});
        return true;
    }
    static constexpr bool has_step(int s) {
        for (int p = 0; p < NP; p++)
            if (plan.m[s][p]) return true;
        return false;
    }
    template <int... Ss>
    static __device__ __forceinline__ void forward(St& st, std::integer_sequence<int, Ss...>) {
        (step_if<Ss>(st) && ...);  // stops after the step where every lane finished
    }
};

// At most 128 VGPRs (four wavefronts per SIMD; the limits of the diagonals are
// made again where they are used, two instructions, to stay below).
template <int X, int OE, int E, int CAP, int KT, int LMAX, bool CIGAR, bool ASCII>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_lane(LaneArgs a,
                                                                                    int persistent) {
    using K = LaneKernel<X, OE, E, CAP, KT, LMAX, CIGAR>;
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wpb = blockDim.x >> 6;
    lptr<uint32_t> wbase = (lptr<uint32_t>)((lptr<unsigned char>)lds + wave * K::WAVE_BYTES) + lane;
    const lptr<uint32_t> colP = wbase, colT = wbase + K::SQ * 64, stage = wbase + 2 * K::SQ * 64;
    typename K::St st;
    st.pb = (uint32_t)(uintptr_t)colP;
    st.tb = (uint32_t)(uintptr_t)colT;
    st.R = stage;
    // this wavefront's records (HIST_DW rows of 64 dwords; one region per
    // launched wavefront)
    st.H = (gptr_t<uint32_t>)a.hist + (uint64_t)(blockIdx.x * wpb + wave) * K::HIST_DW * 64 + lane;
    // persistent: LANE_QUEUES counters (one per 128-byte line), wavefront w
    // drawing from counter w % LANE_QUEUES; the i-th claim from counter q is
    // the group of 64 queue entries number i * LANE_QUEUES + q, so every
    // counter serves an interleaved share of the queue (of the same mix of
    // costs) and no single address takes every wavefront's atomics
    const uint32_t qid = (blockIdx.x * wpb + wave) % LANE_QUEUES;
    for (uint32_t iter = 0;; iter++) {
        uint32_t qbase;
        if (persistent) {
            uint32_t t = 0;
            if (lane == 0) t = atomicAdd(a.queue + qid * 32, 1u);
            const uint32_t i = __builtin_amdgcn_readfirstlane(t);
            const uint64_t g = (uint64_t)i * LANE_QUEUES + qid;
            qbase = g * 64 >= a.num ? a.num : (uint32_t)(g * 64);
        } else {
            if (iter) break;
            qbase = (blockIdx.x * wpb + wave) * 64;
        }
        if (qbase >= a.num) break;
        const uint32_t q = qbase + lane;
        uint32_t pair = 0;
        bool active = q < a.num;
        if (active) {
            pair = a.order ? a.order[q] : q;
            if (pair >= a.npairs) {  // a corrupt permutation must not fault: skip the entry
                active = false;
                pair = 0;
            }
        }
        int n = 0, m = 0;
        uint64_t ps = 0, ts = 0;
        if (active) {
            const PairDesc d = a.pairs[pair];
            n = (int)d.p_len;
            m = (int)d.t_len;
            ps = d.p_start;
            ts = d.t_start;
        }
        const int kt = m - n;
        // pairs this kernel cannot hold leave at once
        const bool run = active && n <= LMAX && m <= LMAX && kt >= -KT && kt <= KT;
        // stage both sequences in the lane's columns (zero past their ends)
        if constexpr (ASCII) {
            // ASCII: packed on the way in, a word at a time by the pair's own
            // lane, so that all lanes are at the same word and whole words, most
            // of them, go without masks (the words spread over the lanes instead
            // took 57 % of a score-only call of 1 M pairs)
            bool ok = true;
#pragma unroll
            for (int w = 0; w < K::SQ / 2; w++) {
                auto word = [&](const uint64_t* base, uint64_t start, int len) -> uint64_t {
                    const int left = run ? len - 32 * w : 0;
                    uint64_t v = 0;
                    bool good = true;
                    if (lanes_where(left > 0 && left < 32)) {
                        if (left > 0) v = pack_word((const uint8_t*)base, start + 32 * w, min(left, 32), good);
                    } else if (left > 0) {
                        v = pack_full_word((const uint8_t*)base, start + 32 * w, good);
                    }
                    ok = ok && good;
                    return v;
                };
                const uint64_t pv = 32 * w < LMAX ? word(a.pw, ps, n) : 0ull;
                const uint64_t tv = 32 * w < LMAX ? word(a.tw, ts, m) : 0ull;
                colP[(2 * w) * 64] = (uint32_t)pv;
                colT[(2 * w) * 64] = (uint32_t)tv;
                colP[(2 * w + 1) * 64] = (uint32_t)(pv >> 32);
                colT[(2 * w + 1) * 64] = (uint32_t)(tv >> 32);
            }
            if (!ok) atomicMin(a.err_pair, (unsigned long long)pair);
        } else {
            const int nwp = run ? (n + 31) >> 5 : 0, nwt = run ? (m + 31) >> 5 : 0;
#pragma unroll
            for (int w = 0; w < (K::SQ + 1) / 2; w++) {
                const uint64_t pv = w < nwp ? a.pw[ps + w] : 0ull;
                const uint64_t tv = w < nwt ? a.tw[ts + w] : 0ull;
                if (2 * w < K::SQ) {
                    colP[(2 * w) * 64] = (uint32_t)pv;
                    colT[(2 * w) * 64] = (uint32_t)tv;
                }
                if (2 * w + 1 < K::SQ) {
                    colP[(2 * w + 1) * 64] = (uint32_t)(pv >> 32);
                    colT[(2 * w + 1) * 64] = (uint32_t)(tv >> 32);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // (lengths of an idle lane: two empty sequences)
        const int ln = run ? n : 0, lm = run ? m : 0;
        st.n2 = pk_pair(2 * ln, 2 * ln);
        st.m2 = pk_pair(2 * lm, 2 * lm);
        st.tsh = 16 * (kt & 1);
        st.tp = run ? (kt >> 1) + K::PR : -1;
        st.S = run ? -1 : CAP + 1;  // idle lanes hold up no other
        if (lanes_where(run)) K::forward(st, std::make_integer_sequence<int, CAP + 1>{});
        // lanes still running after CAP steps leave through the overflow list
        bool overflow = active && !(run && st.S >= 0 && st.S <= CAP);
        int nr = 0;
        if (CIGAR && active && !overflow) {
            // walk: the edits from the end back to step 0, the last one walked
            // (the first of the alignment) in the low six bits
            uint64_t edits = 0;
            int s = st.S, k = kt, ne = 0;
            bool bad = false;
            auto word = [&](int s2, int k2) -> uint32_t {
                constexpr uint64_t OFFS = K::plan.offs();
                const int row = (int)((OFFS >> (8 * ((s2 - 1) >> 2))) & 0xff) - K::NP + ((k2 + 2 * K::PR) >> 1);
                const int last = K::plan.rows - 1;
                const int r = min(max(row, 0), last);
                uint32_t w;
                if (r < K::RUNS) w = stage[r * 64];
                else w = st.H[(r - K::RUNS) * 64];
                return record_of(w, s2 - 1, k2);
            };
            while (s > 0 && !bad) {
                int kind = EV_X, len = 1;
                const uint32_t f = s >= OE ? word(s, k) : 0u;  // before OE: mismatches only
                if (!(f & 1)) {
                    s -= X;
                } else {
                    const bool ins = !(f & 2);
                    const uint32_t more = ins ? 4u : 8u;
                    kind = ins ? EV_I : EV_D;
                    len = 0;
                    for (;;) {
                        len++;
                        k += ins ? -1 : 1;
                        if (s < OE || k < -2 * K::PR || k >= 2 * K::PR) {
                            bad = true;
                            break;
                        }
                        const uint32_t g = word(s, k);
                        s -= (g & more) ? E : OE;
                        if (!(g & more)) break;
                    }
                }
                edits = edits << 6 | (uint32_t)((len & 15) << 2 | kind);
                ne++;
            }
            if (s != 0 || k != 0 || ne > K::EDITS) bad = true;
            // replay: from the start along matches, edit by edit (as in the band
            // kernel); runs in alignment order
            int h = 0, v = 0, last_op = -1;
            uint32_t cur = 0;
            while (!bad) {
                const int left = min(n - v, m - h);
                int mm = 0;
                for (;;) {
                    const uint32_t hd = 2 * (h + mm), vd = 2 * (v + mm);
                    const lptr<const uint32_t> t = K::at(st.tb, hd >> 5), p = K::at(st.pb, vd >> 5);
                    const uint32_t ta = t[0], tm = t[64], tz = t[128];
                    const uint32_t pa = p[0], pm = p[64], pz = p[128];
                    const uint32_t y0 = __builtin_amdgcn_alignbit(tm, ta, hd) ^ __builtin_amdgcn_alignbit(pm, pa, vd);
                    const uint32_t y1 = __builtin_amdgcn_alignbit(tz, tm, hd) ^ __builtin_amdgcn_alignbit(pz, pm, vd);
                    const uint32_t z = min(min(K::ffbl(y0), __builtin_elementwise_add_sat(K::ffbl(y1), 32u)), 64u);
                    mm += (int)(z >> 1);
                    if (z < 64 || mm >= left) break;
                }
                mm = min(mm, left);
                stage[nr * 64] = (uint32_t)mm << 4;
                nr += mm > 0 ? 1 : 0;
                last_op = mm > 0 ? -1 : last_op;
                h += mm;
                v += mm;
                if (ne == 0) break;
                const int len = (int)(edits >> 2) & 15, kind = (int)(edits & 3);
                edits >>= 6;
                ne--;
                const bool same = last_op == kind;
                cur = same ? cur + ((uint32_t)len << 4) : ((uint32_t)len << 4) | (uint32_t)(1 + kind);
                nr += same ? 0 : 1;
                stage[(nr - 1) * 64] = cur;
                last_op = kind;
                h += kind != EV_D ? len : 0;
                v += kind != EV_I ? len : 0;
                if (h > m || v > n) bad = true;
            }
            if (bad || h != m || v != n || nr > a.slot_cap) overflow = true;
        }
        // CIGAR: the 64 pairs' runs, last to first, packed one after another at
        // the start of the group's slot area (64 * slot_cap words from queue
        // position qbase on), so the compaction reads dense data
        uint64_t src = 0;
        if (CIGAR) {
            const int cnt = (active && !overflow) ? nr : 0;
            int incl = cnt;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int t = __shfl_up(incl, off);
                incl += lane >= off ? t : 0;
            }
            src = (uint64_t)qbase * a.slot_cap + (uint64_t)(incl - cnt);
            for (int r = 0; r < cnt; r++) a.slots[src + r] = stage[(cnt - 1 - r) * 64];
        }
        if (active) {
            if (overflow) {
                const uint32_t at = atomicAdd(a.ovf_count, 1u);
                a.ovf_list[at] = pair;
            } else {
                a.scores[pair] = st.S * a.pen.g;
                a.nruns[pair] = CIGAR ? (uint32_t)nr : 0u;
                if (CIGAR) a.run_src[pair] = src;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

template <int X, int OE, int E, int CAP, int KT, int LMAX>
struct LaneShape {
    static int lds_bytes(bool cigar, int waves) {
        return waves * (cigar ? LaneKernel<X, OE, E, CAP, KT, LMAX, true>::WAVE_BYTES
                              : LaneKernel<X, OE, E, CAP, KT, LMAX, false>::WAVE_BYTES);
    }
    // records of one wavefront
    static int hist_dwords(bool cigar) {
        return cigar ? LaneKernel<X, OE, E, CAP, KT, LMAX, true>::HIST_DW * 64 : 0;
    }
    template <bool CIGAR, bool ASCII>
    static hipError_t launch_t(const LaneArgs& a, bool persistent, int bt, int grid, hipStream_t s) {
        hipLaunchKernelGGL((k_lane<X, OE, E, CAP, KT, LMAX, CIGAR, ASCII>), dim3(grid), dim3(bt),
                           lds_bytes(CIGAR, bt / 64), s, a, persistent ? 1 : 0);
        return hipGetLastError();
    }
    static hipError_t launch(const LaneArgs& a, bool cigar, bool persistent, int bt, int grid,
                             hipStream_t s) {
        if (cigar)
            return a.ascii ? launch_t<true, true>(a, persistent, bt, grid, s)
                           : launch_t<true, false>(a, persistent, bt, grid, s);
        return a.ascii ? launch_t<false, true>(a, persistent, bt, grid, s)
                       : launch_t<false, false>(a, persistent, bt, grid, s);
    }
    static int occupancy(bool cigar, int bt) {
        // (the forms that pack ASCII as they stage hold the same LDS and wavefronts)
        int blocks = 0;
        const int lds = lds_bytes(cigar, bt / 64);
        const hipError_t e =
            cigar ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                        &blocks, (const void*)k_lane<X, OE, E, CAP, KT, LMAX, true, false>, bt, lds)
                  : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                        &blocks, (const void*)k_lane<X, OE, E, CAP, KT, LMAX, false, false>, bt, lds);
        return e == hipSuccess ? blocks : 0;
    }
};

// Shapes built: scaled penalties (2, 4, 1) -- x = 4, o = 6, e = 2 and their
// multiples -- with 8 or 16 score steps, sequences up to 127 bases.
#define WFA_LANE_SHAPES(F)                     \
    F(2, 4, 1, 8, LANE_KT_CAP8, false, 127)    \
    F(2, 4, 1, 16, LANE_KT, false, 127)        \
    F(2, 4, 1, 16, LANE_KT_WIDE, true, 127)

}  // namespace

bool lane_supported(const Pen& pen, int cap, uint32_t max_len) {
#define WFA_LANE_CASE(PX, POE, PE, PC, PKT, PW, PLM) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE && cap == PC && max_len <= (uint32_t)PLM) return true;
    WFA_LANE_SHAPES(WFA_LANE_CASE)
#undef WFA_LANE_CASE
    return false;
}

int lane_lds_bytes(const Pen& pen, int cap, bool cigar, int block_threads) {
    // (either form)
#define WFA_LANE_CASE(PX, POE, PE, PC, PKT, PW, PLM) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE && cap == PC) \
        return LaneShape<PX, POE, PE, PC, PKT, PLM>::lds_bytes(cigar, block_threads / 64);
    WFA_LANE_SHAPES(WFA_LANE_CASE)
#undef WFA_LANE_CASE
    return -1;
}

size_t lane_hist_bytes_per_wave(const Pen& pen, int cap, bool wide, bool cigar) {
#define WFA_LANE_CASE(PX, POE, PE, PC, PKT, PW, PLM) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE && cap == PC && wide == PW) \
        return (size_t)LaneShape<PX, POE, PE, PC, PKT, PLM>::hist_dwords(cigar) * 4;
    WFA_LANE_SHAPES(WFA_LANE_CASE)
#undef WFA_LANE_CASE
    return 0;
}

int lane_max_blocks_per_cu(const Pen& pen, int cap, bool wide, bool cigar, int block_threads) {
#define WFA_LANE_CASE(PX, POE, PE, PC, PKT, PW, PLM) \
    if (pen.x == PX && pen.oe == POE && pen.e == PE && cap == PC && wide == PW) \
        return LaneShape<PX, POE, PE, PC, PKT, PLM>::occupancy(cigar, block_threads);
    WFA_LANE_SHAPES(WFA_LANE_CASE)
#undef WFA_LANE_CASE
    return 0;
}

hipError_t launch_lane(const LaneArgs& a, int cap, bool wide, bool cigar, bool persistent,
                       int block_threads, int grid, hipStream_t s) {
#define WFA_LANE_CASE(PX, POE, PE, PC, PKT, PW, PLM) \
    if (a.pen.x == PX && a.pen.oe == POE && a.pen.e == PE && cap == PC && wide == PW) \
        return LaneShape<PX, POE, PE, PC, PKT, PLM>::launch(a, cigar, persistent, block_threads, grid, s);
    WFA_LANE_SHAPES(WFA_LANE_CASE)
#undef WFA_LANE_CASE
    return hipErrorInvalidValue;
}

}  // namespace wfa
