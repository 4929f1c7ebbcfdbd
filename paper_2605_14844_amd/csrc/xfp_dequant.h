// Dequantisation in registers: the codebook as byte planes, v_perm_b32 as the lookup (four weights per instruction).
#pragma once
#include "xfp_device.h"

namespace xfp {

typedef __attribute__((address_space(3))) uint32_t lds_u32_t;
typedef __attribute__((address_space(3))) const uint32_t lds_cu32_t;
// index words of 32 weights
template <int BITS>
struct WordsOf { typedef uint32_t type __attribute__((ext_vector_type(BITS))); };
template <int BITS>
using words_t = typename WordsOf<BITS>::type;

// position (0..31) in natural order of the weight in slot s of a dequantised run of 32
constexpr int slot_k(int bits, int s)
{
    const int c = s >> 3, t = s & 7;                       // 16-byte chunk, slot in it
    if (bits == 4) return 8 * c + (t < 4 ? 2 * t : 2 * (t - 4) + 1);
    if (bits == 3) return 2 * c + (t >> 2) + 8 * (t & 3);
    return 16 * (c >> 1) + 2 * (c & 1) + (t >> 2) + 4 * (t & 3);
}

// Byte planes of a codebook: lo[d] / hi[d] hold the low / high bytes of entries 4 d .. 4 d + 3.
template <int BITS>
struct Planes {
    static constexpr int ND = (1 << BITS) / 4;
    uint32_t lo[ND], hi[ND];
    // from the codebook's 2^BITS fp16 entries as dwords
    __device__ __forceinline__ void set(const uint32_t *c)
    {
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            lo[d] = __builtin_amdgcn_perm(c[2 * d + 1], c[2 * d], 0x06040200u);
            hi[d] = __builtin_amdgcn_perm(c[2 * d + 1], c[2 * d], 0x07050301u);
        }
    }
};

// Bytes (four at a time) of the entries that the selector bytes name: BITS = 4: low three index bits in s, the fourth
// as j + 4 * bit in byte j of up; fewer bits: the index itself in s.
template <int BITS>
__device__ __forceinline__ uint32_t pick(const uint32_t *p, uint32_t s, uint32_t up)
{
    if constexpr (BITS == 4)
        return __builtin_amdgcn_perm(__builtin_amdgcn_perm(p[3], p[2], s), __builtin_amdgcn_perm(p[1], p[0], s), up);
    else if constexpr (BITS == 3) return __builtin_amdgcn_perm(p[1], p[0], s);
    else return __builtin_amdgcn_perm(p[0], p[0], s);
}

// Four weights (two dwords of fp16 pairs) from four selectors.
template <int BITS>
__device__ __forceinline__ void four(const Planes<BITS> &P, uint32_t s, uint32_t up, uint32_t &d0, uint32_t &d1)
{
    const uint32_t l = pick<BITS>(P.lo, s, up), h = pick<BITS>(P.hi, s, up);
    d0 = __builtin_amdgcn_perm(h, l, 0x05010400u);
    d1 = __builtin_amdgcn_perm(h, l, 0x07030602u);
}

// Index words of 32 weights in the form chunk() wants them: 3 bits: bytes 0, 3, 6, 9 / 1, 4, 7, 10 / 2, 5, 8, 11 of
// the 12, so that fields 8 apart sit at one bit position of four bytes.
template <int BITS>
__device__ __forceinline__ void arrange(words_t<BITS> &w)
{
    if constexpr (BITS == 3) {
        const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x0c060300u), b = __builtin_amdgcn_perm(w[1], w[0], 0x0c070401u),
                       c = __builtin_amdgcn_perm(w[1], w[0], 0x0c0c0502u), x = w[2];
        w[0] = __builtin_amdgcn_perm(x, a, 0x05020100u);
        w[1] = __builtin_amdgcn_perm(x, b, 0x06020100u);
        w[2] = __builtin_amdgcn_perm(x, c, 0x07040100u);
    }
}

// Half of chunk c (0..3) of a run of 32: slots 8 c + 4 half .. 8 c + 4 half + 3 as fp16 pairs.
template <int BITS>
__device__ __forceinline__ void chunk_half(const Planes<BITS> &P, const words_t<BITS> &w, int c, int half, uint32_t &d0, uint32_t &d1)
{
    if constexpr (BITS == 4) {
        const uint32_t v = w[c], kTop = 0x03020100u;
        if (half == 0) four<4>(P, v & 0x07070707u, ((v >> 1) & 0x04040404u) | kTop, d0, d1);
        else four<4>(P, (v >> 4) & 0x07070707u, ((v >> 5) & 0x04040404u) | kTop, d0, d1);
    } else if constexpr (BITS == 3) {
        auto sel = [&](int k0) -> uint32_t {
            switch (k0) {
            case 0: return w[0] & 0x07070707u;
            case 1: return (w[0] >> 3) & 0x07070707u;
            case 2: return ((w[0] >> 6) & 0x03030303u) | ((w[1] << 2) & 0x04040404u);
            case 3: return (w[1] >> 1) & 0x07070707u;
            case 4: return (w[1] >> 4) & 0x07070707u;
            case 5: return ((w[1] >> 7) & 0x01010101u) | ((w[2] << 1) & 0x06060606u);
            case 6: return (w[2] >> 2) & 0x07070707u;
            default: return (w[2] >> 5) & 0x07070707u;
            }
        };
        four<3>(P, sel(2 * c + half), 0u, d0, d1);
    } else {
        four<2>(P, (w[c >> 1] >> (4 * (c & 1) + 2 * half)) & 0x03030303u, 0u, d0, d1);
    }
}

// The whole chunk.
template <int BITS>
__device__ __forceinline__ u32x4_t chunk(const Planes<BITS> &P, const words_t<BITS> &w, int c)
{
    uint32_t d0, d1, d2, d3;
    chunk_half<BITS>(P, w, c, 0, d0, d1);
    chunk_half<BITS>(P, w, c, 1, d2, d3);
    return u32x4_t{d0, d1, d2, d3};
}

// slot of column k (0..31) of such a run: the inverse of slot_k
template <int BITS>
__device__ __forceinline__ uint32_t slot_of(uint32_t k)
{
    if constexpr (BITS > 4) return k;                          // (looked up one by one, in natural order)
    else if constexpr (BITS == 4) return (k & 24u) + (k & 1u) * 4 + (k >> 1 & 3u);
    else if constexpr (BITS == 3) return (k >> 1 & 3u) * 8 + (k & 1u) * 4 + (k >> 3);
    else return (k & 16u) + (k >> 1 & 1u) * 8 + (k & 1u) * 4 + (k >> 2 & 3u);
}

}  // namespace xfp
