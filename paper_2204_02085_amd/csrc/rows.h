// Wavefront rows in registers, shared by the band kernel (k_band.hip), the front
// kernel (k_front.hip) and, for the packed operations and the extension, the
// adaptive kernel (k_adapt.hip) and the lane kernel (k_lane.hip).
//
// A lane owns C neighbouring diagonals; a row of offsets is C / 2 registers of
// two 16-bit offsets each, so the recurrences run two cells per instruction
// (v_pk_max_i16 and friends) and the M, I and D rows a step reads back live in
// registers for compile-time scaled penalties (X, OE, E).  Neighbouring lanes
// exchange one column per step with DPP moves.
//
// Offsets are stored shifted left by SH (0 or 1).  With SH = 1 an offset is
// twice the base position, i.e. the bit position in the 2-bit sequence: the
// funnel shift of a 16-base window takes it as it stands.  SH = 1 holds
// sequences up to 16383 bases, SH = 0 up to 32766.  NULL is any negative
// value: NUL16P when stored by the extension, drifting up by 1 << SH per step
// along a chain of I or D cells, so a kernel stops before 16384 >> SH steps.
//
// Candidates past the matrix (offset above L = min(m, n + k) on diagonal k) are
// dropped from M after the maximum and stay in the I and D rows.  That changes
// no result of an exact alignment: an I candidate past the last text column
// has passed, on a lower diagonal and at a lower score, an M cell on that
// column, from which the remaining deletions cost less than any way on from
// this diagonal; D past the last pattern row and a mismatch past either are
// the same argument.  So the cells such a candidate hides lie on no optimal
// alignment, and every cell on one keeps its offset and its tie-break.
// (The WF-adaptive reduction measures cells off the optimal paths too, so the
// adaptive kernel drops candidates before the maximum.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace wfa {
namespace rows {

constexpr uint32_t NUL16P = 0xC000C000u;  // two NULL offsets (-16384)
enum { EV_X = 0, EV_I = 1, EV_D = 2 };    // walk events: len << 2 | kind

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
template <class T>
using lds_p = __attribute__((address_space(3))) T*;

__device__ __forceinline__ s16x2 as_s(uint32_t a) { return __builtin_bit_cast(s16x2, a); }
__device__ __forceinline__ u16x2 as_u(uint32_t a) { return __builtin_bit_cast(u16x2, a); }
__device__ __forceinline__ uint32_t bits(s16x2 a) { return __builtin_bit_cast(uint32_t, a); }
__device__ __forceinline__ uint32_t bits(u16x2 a) { return __builtin_bit_cast(uint32_t, a); }
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    return bits(__builtin_elementwise_max(as_s(a), as_s(b)));
}
__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b) { return bits(as_u(a) + as_u(b)); }
__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b) { return bits(as_u(a) - as_u(b)); }
// The next ones are written as instructions: from vector code the compiler
// takes the halves apart again (a compare, a select and a permute for each) or
// spreads a mask over several operations.
__device__ __forceinline__ uint32_t pk_minu(uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// 0xffff in each half whose sign bit is set
__device__ __forceinline__ uint32_t pk_sign(uint32_t a) {
    uint32_t r;
    asm("v_pk_ashrrev_i16 %0, 15, %1 op_sel_hi:[0,1]" : "=v"(r) : "v"(a));
    return r;
}
// 1 in each half where a != b
__device__ __forceinline__ uint32_t pk_ne(uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_pk_min_u16 %0, %1, 1 op_sel_hi:[1,0]" : "=v"(r) : "v"(a ^ b));
    return r;
}
// (mask & a) | (~mask & b)
__device__ __forceinline__ uint32_t bit_select(uint32_t mask, uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(mask), "v"(a), "v"(b));
    return r;
}
// (a << n) | b
template <int N>
__device__ __forceinline__ uint32_t shl_or(uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_lshl_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "n"(N), "v"(b));
    return r;
}
// a wave-uniform mask of the lanes where c holds
__device__ __forceinline__ uint64_t lanes_where(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ uint32_t pk_pair(int lo, int hi) {
    return (uint32_t)(lo & 0xffff) | ((uint32_t)hi << 16);
}

// the value of the lane before / after (whole wavefront; the end lane keeps `end`)
__device__ __forceinline__ uint32_t wave_prev(uint32_t end, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)end, (int)x, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_next(uint32_t end, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)end, (int)x, 0x130, 0xF, 0xF, false);
}
// the same within groups of G = 8, 16, 32 or 64 lanes (`first` / `last`: this lane is at the
// group's end); the group's end lane reads NULL
template <int G>
__device__ __forceinline__ uint32_t group_prev(uint32_t x, bool first) {
    if constexpr (G == 64) {
        return wave_prev(NUL16P, x);
    } else if constexpr (G == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)NUL16P, (int)x, 0x111, 0xF, 0xF, false);
    } else if constexpr (G < 16) {
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp((int)NUL16P, (int)x, 0x111, 0xF, 0xF, false);
        return first ? NUL16P : y;
    } else {
        const uint32_t y = wave_prev(NUL16P, x);
        return first ? NUL16P : y;
    }
}
template <int G>
__device__ __forceinline__ uint32_t group_next(uint32_t x, bool last) {
    if constexpr (G == 64) {
        return wave_next(NUL16P, x);
    } else if constexpr (G == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)NUL16P, (int)x, 0x101, 0xF, 0xF, false);
    } else if constexpr (G < 16) {
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp((int)NUL16P, (int)x, 0x101, 0xF, 0xF, false);
        return last ? NUL16P : y;
    } else {
        const uint32_t y = wave_next(NUL16P, x);
        return last ? NUL16P : y;
    }
}

// The rows of one lane.  M[j], I[j], D[j] hold step s - 1 - j.
template <int X, int OE, int E, int C, int SH, bool CIGAR>
struct Rows {
    static constexpr int P = C / 2;
    static constexpr int RM = X > OE ? X : OE;
    static constexpr uint32_t ONE = SH ? 0x00020002u : 0x00010001u;
    uint32_t M[RM][P], I[E][P], D[E][P];
    uint32_t acc[P];  // decision records of up to four steps

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int p = 0; p < P; p++) {
#pragma unroll
            for (int j = 0; j < RM; j++) M[j][p] = NUL16P;
#pragma unroll
            for (int j = 0; j < E; j++) I[j][p] = D[j][p] = NUL16P;
            acc[p] = 0;
        }
    }
    // what a step hands to the next diagonal up (the best source of an
    // insertion) and down (of a deletion)
    __device__ __forceinline__ void sources(uint32_t (&a)[P], uint32_t (&b)[P]) const {
#pragma unroll
        for (int p = 0; p < P; p++) {
            a[p] = pk_max(M[OE - 1][p], I[E - 1][p]);
            b[p] = pk_max(M[OE - 1][p], D[E - 1][p]);
        }
    }
    // The cells of a step before extension: m (M), i, d, from sources a, b and
    // the neighbour lanes' columns (ap: the last register of a one lane down,
    // bn: the first of b one lane up).  CIGAR: four record bits per cell are
    // shifted into acc: M is not a mismatch / not the end of an insertion
    // (ties: mismatch, then insertion, then deletion), the insertion into the
    // next diagonal up extends one / the deletion into the next one down does
    // (ties: open).  The two gap bits stand at their source's diagonal.  acc
    // holds four steps; `fresh` starts the next four.
    __device__ __forceinline__ void cells(const uint32_t (&a)[P], const uint32_t (&b)[P], uint32_t ap,
                                          uint32_t bn, uint32_t (&m)[P], uint32_t (&i)[P],
                                          uint32_t (&d)[P], bool fresh) {
#pragma unroll
        for (int p = 0; p < P; p++) {
            i[p] = pk_add(__builtin_amdgcn_alignbit(a[p], p ? a[p - 1] : ap, 16), ONE);
            d[p] = __builtin_amdgcn_alignbit(p < P - 1 ? b[p + 1] : bn, b[p], 16);
            const uint32_t x = pk_add(M[X - 1][p], ONE);
            m[p] = pk_max(pk_max(x, i[p]), d[p]);
            if constexpr (CIGAR) {
                const uint32_t nx = pk_ne(m[p], x), ni = pk_ne(m[p], i[p]);
                const uint32_t ai = pk_ne(a[p], M[OE - 1][p]), ad = pk_ne(b[p], M[OE - 1][p]);
                const uint32_t rec = shl_or<1>(shl_or<1>(shl_or<1>(ad, ai), ni), nx);
                acc[p] = fresh ? rec : shl_or<4>(acc[p], rec);
            }
        }
    }
    __device__ __forceinline__ void push(const uint32_t (&m)[P], const uint32_t (&i)[P],
                                         const uint32_t (&d)[P]) {
#pragma unroll
        for (int p = 0; p < P; p++) {
#pragma unroll
            for (int j = RM - 1; j > 0; j--) M[j][p] = M[j - 1][p];
#pragma unroll
            for (int j = E - 1; j > 0; j--) {
                I[j][p] = I[j - 1][p];
                D[j][p] = D[j - 1][p];
            }
            M[0][p] = m[p];
            I[0][p] = i[p];
            D[0][p] = d[p];
        }
    }
};

// Where a lane's cells sit: packed limits (L << SH; -1 for a diagonal outside
// the matrix) and, for cells with no offset, a packed offset inside the text
// whose compares read staged bases; k2: twice each diagonal.
template <int C>
struct Place {
    static constexpr int P = C / 2;
    uint32_t lim[P], safe[P];
    int k2[C];
    template <int SH>
    __device__ __forceinline__ void set(int n, int m, int k0) {
#pragma unroll
        for (int c = 0; c < C; c++) {
            k2[c] = 2 * (k0 + c);
            // four registers, not one and an add per cell and step
            asm volatile("" : "+v"(k2[c]));
        }
#pragma unroll
        for (int p = 0; p < P; p++) {
            int l[2], z[2];
#pragma unroll
            for (int u = 0; u < 2; u++) {
                const int k = k0 + 2 * p + u;
                l[u] = (k < -n || k > m) ? -1 : min(m, n + k) << SH;
                z[u] = min(max(k, 0), m) << SH;
            }
            lim[p] = pk_pair(l[0], l[1]);
            safe[p] = pk_pair(z[0], z[1]);
        }
    }
};

// dwords q and q + 1 of a sequence at LDS byte `base`
__device__ __forceinline__ void two_dwords(uint32_t base, int q, uint32_t& w0, uint32_t& w1) {
    asm("" : "+v"(q));  // keeps q << 2 and the base in one instruction
    lds_p<const uint32_t> w = (lds_p<const uint32_t>)(uintptr_t)(base + ((uint32_t)q << 2));
    w0 = w[0];
    w1 = w[1];
}
// 16 bases from bit position `b` (twice the base) on
__device__ __forceinline__ uint32_t win16(uint32_t base, int b) {
    uint32_t w0, w1;
    two_dwords(base, b >> 5, w0, w1);
    return __builtin_amdgcn_alignbit(w1, w0, (uint32_t)b);
}

// Bits (two a base; an odd count: with one of a mismatch) that match from bit positions
// h and v on, at most 64.
__device__ __forceinline__ uint32_t match_bits(uint32_t tb, uint32_t pb, uint32_t h, uint32_t v) {
    lds_p<const uint32_t> t = (lds_p<const uint32_t>)(uintptr_t)(tb + ((h >> 5) << 2));
    lds_p<const uint32_t> p = (lds_p<const uint32_t>)(uintptr_t)(pb + ((v >> 5) << 2));
    uint32_t a[3], b[3], n = 64;
#pragma unroll
    for (int i = 0; i < 3; i++) {
        a[i] = t[i];
        b[i] = p[i];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const uint32_t y = __builtin_amdgcn_alignbit(a[i + 1], a[i], h) ^ __builtin_amdgcn_alignbit(b[i + 1], b[i], v);
        uint32_t z;
        asm("v_ffbl_b32 %0, %1" : "=v"(z) : "v"(y));  // ~0 for a zero word: the sum saturates
        n = min(n, __builtin_elementwise_add_sat(z, 32u * i));
    }
    return n;
}

// Extend the cells m of one step along matches (sequences in LDS at byte
// addresses tb, pb) and drop those past the matrix.  Fifteen bases first (a stop
// bit in place of the sixteenth bounds the count); a wavefront goes on only while
// one of its lanes still matches.  What runs past the matrix is cut off by one
// packed minimum at the end.  Past 31 bases a lane takes 32 at a time, some 400
// cycles of LDS latency and a short chain.  With LONG_WAVE a match of 255 bases or
// more (one or two lanes a step have one) is handed to the wavefront, which takes
// 1024 in that time: 600 reads of 8 to 20 kbp at up to 0.05 % divergence, score
// only, 345 us (899 without it, 1325 at 16 bases a trip).  It pays where a pair has
// the wavefront to itself; from 64 bases on it cost 1 % of 5 % divergent reads.
enum { LONG_LANE, LONG_WAVE };
template <int C, int SH, int LONG>
__device__ __forceinline__ void extend(uint32_t (&m)[C / 2], const Place<C>& pl, uint32_t tb,
                                       uint32_t pb) {
    constexpr int P = C / 2;
    constexpr uint32_t STOP = 0x80000000u;
    uint32_t bad[P], hv[P], x[C], r[C];
#pragma unroll
    for (int p = 0; p < P; p++) {
        bad[p] = pk_sign(m[p] | pk_sub(pl.lim[p], m[p]));
        hv[p] = bit_select(bad[p], pl.safe[p], m[p]);
    }
    // bit position of column c in the text
    auto pos = [&](int c) -> uint32_t {
        return ((c & 1) ? hv[c / 2] >> 16 : hv[c / 2] & 0xffffu) << (1 - SH);
    };
    // every column's loads go out before the first is used (left to itself the
    // compiler waits for each pair in turn)
    uint32_t t0[C], t1[C], p0[C], p1[C];
    int v[C];
#pragma unroll
    for (int c = 0; c < C; c++) {
        v[c] = (int)pos(c) - pl.k2[c];
        // the dword of the position straight from the packed offsets
        const uint32_t q = (c & 1) ? hv[c / 2] >> (20 + SH)
                                   : __builtin_amdgcn_ubfe(hv[c / 2], 4 + SH, 12 - SH);
        two_dwords(tb, (int)q, t0[c], t1[c]);
        two_dwords(pb, v[c] >> 5, p0[c], p1[c]);
    }
    __builtin_amdgcn_sched_barrier(0);
    uint32_t lo = ~0u;
#pragma unroll
    for (int c = 0; c < C; c++) {
        x[c] = (__builtin_amdgcn_alignbit(t1[c], t0[c], pos(c)) ^
                __builtin_amdgcn_alignbit(p1[c], p0[c], (uint32_t)v[c])) | STOP;
        // bits; an odd one rounds down below
        asm("v_ffbl_b32 %0, %1" : "=v"(r[c]) : "v"(x[c]));
        lo = min(lo, x[c]);
    }
    if (lanes_where(lo == STOP)) {
        auto to_end = [&](int c) -> uint32_t {  // bits from column c to the matrix' edge
            const uint32_t left = pk_sub(pl.lim[c / 2], hv[c / 2]) & ~bad[c / 2];
            return ((c & 1) ? left >> 16 : left & 0xffffu) << (1 - SH);
        };
        constexpr int TRIPS = 7;
        constexpr uint32_t FAR = 62 + 64 * TRIPS;
        uint32_t longest = 0;
#pragma unroll
        for (int c = 0; c < C; c++) {
            const uint32_t end = to_end(c);
            if (x[c] == STOP && end > 30) {
                const int h = (int)pos(c);
                uint32_t done = 30, z;
                const uint32_t y = win16(tb, h + (int)done) ^ win16(pb, v[c] + (int)done);
                asm("v_ffbl_b32 %0, %1" : "=v"(z) : "v"(y));  // ~0 for a zero word
                done += min(z, 32u);
                int trips = TRIPS;
                for (bool on = z >= 32 && done < end; on; on = z >= 64 && done < end) {
                    if (LONG == LONG_WAVE && !trips--) break;
                    z = match_bits(tb, pb, (uint32_t)h + done, (uint32_t)v[c] + done);
                    done += z;
                }
                r[c] = done;
            }
            longest = max(longest, r[c]);
        }
        if (LONG == LONG_WAVE && lanes_where(longest >= FAR)) {
            const uint32_t lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll
            for (int c = 0; c < C; c++) {
                const uint32_t end = to_end(c);
                for (uint64_t far = lanes_where(x[c] == STOP && r[c] >= FAR && r[c] < end); far; far &= far - 1) {
                    const int l = __builtin_ctzll(far);
                    const int hl = __builtin_amdgcn_readlane((int)pos(c) + (int)r[c], l);
                    const int vl = __builtin_amdgcn_readlane(v[c] + (int)r[c], l);
                    const uint32_t el = (uint32_t)__builtin_amdgcn_readlane((int)(end - r[c]), l);
                    uint32_t sum = 0;
                    for (;;) {
                        const uint32_t o = sum + 32 * lane;
                        uint32_t y = 1;
                        if (o < el) y = win16(tb, hl + (int)o) ^ win16(pb, vl + (int)o);
                        const uint64_t stop = lanes_where(y != 0);
                        if (stop) {
                            const int f = __builtin_ctzll(stop);
                            sum += 32 * f + __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)y, f));
                            break;
                        }
                        sum += 64 * 32;
                    }
                    if (lane == (uint32_t)l) r[c] += sum;
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < P; p++) {
        const uint32_t rr = SH ? (r[2 * p] | (r[2 * p + 1] << 16)) & 0xFFFEFFFEu
                               : (r[2 * p] >> 1) | ((r[2 * p + 1] >> 1) << 16);
        m[p] = bit_select(bad[p], NUL16P, pk_minu(hv[p] + rr, pl.lim[p]));
    }
}

// The record of cell (s, column) among the stored words: four steps of a
// register pair of columns to a dword, the first of the four on top.
__device__ __forceinline__ uint32_t record_of(uint32_t word, int s, int col) {
    return (word >> (16 * (col & 1) + 4 * (3 - (s & 3)))) & 15u;
}

}  // namespace rows
}  // namespace wfa
