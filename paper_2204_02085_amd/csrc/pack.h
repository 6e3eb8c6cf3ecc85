// ASCII -> 2-bit packing of one word (32 bases), shared by the packing kernels
// and by kernels that pack a pair as they stage it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace wfa {

// Codes of the 4 bytes of x (A/a=0, C/c=1, G/g=2, T/t=3) in 8 bits; `bad`
// collects the bits of bytes (among the low `keep` mask) that are not one of
// those letters.  The code of an ASCII letter is bits 1-2 of the byte folded
// ((c >> 1) ^ (c >> 2)) & 3; a byte is valid when the lowercase letter of its
// code (looked up bytewise with v_perm_b32) equals the byte in lowercase.
__device__ __forceinline__ uint32_t pack4(uint32_t x, uint32_t keep, uint32_t& bad) {
    const uint32_t c = ((x >> 1) ^ (x >> 2)) & 0x03030303u;
    // bytes 'a' 'c' 'g' 't' selected by c (selector values 0..3 pick bytes of src1)
    const uint32_t letters = __builtin_amdgcn_perm(0u, 0x74676361u, c);
    bad |= (letters ^ (x | 0x20202020u)) & keep;
    return __builtin_amdgcn_udot4(c & keep, 0x40100401u, 0u, false);  // a base's code times 4 to its place
}

// 32 bases starting at byte b0 of `ascii` (cnt of them valid, 1..32) as one
// 2-bit word.  Reads the aligned dwords covering the bases; near the end of
// the sequence the dword index is clamped to the last one holding a base,
// so no byte past the sequence is read.
__device__ __forceinline__ uint64_t pack_word(const uint8_t* __restrict__ ascii, uint64_t b0,
                                              int cnt, bool& ok) {
    const uint8_t* first = ascii + b0;
    const uint32_t sh = (uint32_t)((uintptr_t)first & 3u);
    const uint32_t* src = (const uint32_t*)(first - sh);
    const int lastd = (int)((sh + cnt - 1) >> 2);  // last dword holding a base
    uint32_t raw[9];
    if (lastd == 8) {
#pragma unroll
        for (int d = 0; d < 9; d++) raw[d] = src[d];
    } else {
#pragma unroll
        for (int d = 0; d < 9; d++) raw[d] = src[min(d, lastd)];
    }
    uint64_t word = 0;
    uint32_t bad = 0;
#pragma unroll
    for (int d = 0; d < 8; d++) {
        const uint32_t x = __builtin_amdgcn_alignbyte(raw[d + 1], raw[d], sh);
        const int c = min(max(cnt - 4 * d, 0), 4);
        const uint32_t keep = c >= 4 ? 0xFFFFFFFFu : ((1u << (8 * c)) - 1u);
        word |= (uint64_t)pack4(x, keep, bad) << (8 * d);
    }
    ok = bad == 0;
    return word;
}

// The same for a whole word (32 bases).
__device__ __forceinline__ uint64_t pack_full_word(const uint8_t* __restrict__ ascii, uint64_t b0, bool& ok) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
    const uint8_t* first = ascii + b0;
    const uint32_t sh = (uint32_t)((uintptr_t)first & 3u);
    const uint32_t* src = (const uint32_t*)(first - sh);
    const u32x4 lo = *(const u32x4*)src, hi = *(const u32x4*)(src + 4);
    const uint32_t raw[9] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3], src[sh ? 8 : 7]};
    uint32_t half[2] = {0, 0}, bad = 0;
#pragma unroll
    for (int d = 7; d >= 0; d--) {
        const uint32_t x = __builtin_amdgcn_alignbyte(raw[d + 1], raw[d], sh);
        half[d >> 2] = half[d >> 2] << 8 | pack4(x, ~0u, bad);
    }
    ok = bad == 0;
    return (uint64_t)half[1] << 32 | half[0];
}

}  // namespace wfa
