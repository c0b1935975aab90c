// Counter bands in LDS: pair terms of packed counter words and the slot
// scatter, shared by the kernels that count wedges.
#pragma once

#include "bbc_internal.h"

namespace bbc {

// Pair terms of the counter fields of LDS words: sum over fields x of
// C(x,2) = (x^2 - x) / 2.  The sum of x^2 over a word is one packed
// dot-product instruction (the word with itself), so no field is unpacked.
// In count mode (TWICE) only the squares are summed: the band's sum of x is
// its number of wedges, which the caller subtracts once, and the kernel
// carries twice the pair terms.  Otherwise the sum of x is the dot product
// with a word of ones and x^2 - x, always even, is halved per thread.
// Modes 0 and 1 keep 32-bit partial sums per band and thread (at most 64
// words per thread and band, each below 2^18); modes 2 and 3 widen per
// word (in mode 2, a + b <= 65535, so a^2 + b^2 fits 32 bits).
template <int MODE, bool TWICE>
struct PairSum {
    uint32_t sq = 0, lin = 0;
    unsigned long long wide = 0;
    __device__ __forceinline__ void add(uint32_t v) {
        if constexpr (MODE == 0) {  // eight 4-bit fields
            sq = __builtin_amdgcn_udot8(v, v, sq, false);
            if constexpr (!TWICE) lin = __builtin_amdgcn_udot8(v, 0x11111111u, lin, false);
        } else if constexpr (MODE == 1) {  // four 8-bit fields
            sq = __builtin_amdgcn_udot4(v, v, sq, false);
            if constexpr (!TWICE) lin = __builtin_amdgcn_udot4(v, 0x01010101u, lin, false);
        } else if constexpr (MODE == 2) {  // a and b of one endpoint
            typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
            const u16x2 h = __builtin_bit_cast(u16x2, v);
            const uint32_t q = __builtin_amdgcn_udot2(h, h, 0u, false);
            if constexpr (TWICE) wide += q;
            else wide += (q - ((v & 0xffffu) + (v >> 16))) >> 1;
        } else {  // one 32-bit field
            const unsigned long long a = v;
            if constexpr (TWICE) wide += a * a;
            else wide += a * (a - (a > 0)) / 2;
        }
    }
    // The sums added so far, and restarts.
    __device__ __forceinline__ unsigned long long take() {
        unsigned long long r = wide;
        if constexpr (MODE <= 1) r += TWICE ? (unsigned long long)sq : (unsigned long long)((sq - lin) >> 1);
        sq = lin = 0;
        wide = 0;
        return r;
    }
};

// Multiplier of the slot scatter.  Centre lists are sorted by rank, so the
// lanes of a wave read endpoints at a near-regular stride; mapped straight
// onto LDS words that stride lands on a few banks.  Any bijection between
// the endpoint ranks of a band and counter fields is valid (the reduction
// sums every touched field), so an endpoint's slot is its rank times an odd
// multiplier modulo the power-of-two band capacity: a band never spans more
// ranks than its capacity, and distinct residues stay distinct under the
// multiplication.
constexpr uint32_t kSlotMul = 0x9E377u;  // times 8 still below 2^24: a full-rate 24-bit multiply

// Inverse of an odd number modulo 2^32 (Newton iteration; each step doubles
// the number of correct low bits).
constexpr uint32_t inverse_odd(uint32_t m) {
    uint32_t x = m;  // correct to 3 bits
    for (int i = 0; i < 5; ++i) x *= 2u - m * x;
    return x;
}
constexpr uint32_t kSlotInv = inverse_odd(kSlotMul);
static_assert(kSlotMul * kSlotInv == 1u, "slot scatter must be invertible");
static_assert(kSlotMul * 8u < (1u << 24), "scaled multipliers must fit a 24-bit multiply");

// Low 32 bits of a 24 x 24-bit product (full rate; the compiler drops the
// masks that would let it pick this form, since only the low bits are used).
// The low k <= 24 bits of the product depend only on the low k bits of the
// operands, so ranks above 2^24 map correctly modulo the band capacity.
__device__ __forceinline__ uint32_t mul_u24(uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

}  // namespace bbc
