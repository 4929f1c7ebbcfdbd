// Up to 64 tokens against one matrix (V2 codebooks at 2 to 6 bits, a V2a library, a library with a scale and a mid-point per
// group at 2 to 4) in ONE launch, on the matrix cores, with the activations resident in LDS.
//
// Why: the other kernels for several tokens re-lay the activations in a launch of their own and build pair tables per 16 or 32
// rows before the first product; with few tokens, or few rows, those two are most of a call (7001 x 5504, 2 bits, 5 tokens:
// 16.2 us a call, of which the product's bytes need 1.9), and rows beyond 8192 columns were three launches.
//
// Work unit: a workgroup of RB x KW waves owns RB blocks of 16 rows (of one slice of K); the KW waves of a block share its
// columns in contiguous ranges and add their sums in LDS at the end.
//  - The activations are put into LDS once, converted, in the order that the dequantisation gives (slot_k); rows 16 bytes
//    more than a multiple of 256 apart, so that 16 tokens' chunks lie in 16 different places of the 64 banks.  B operands
//    and the outliers' activations are read from there: no re-laid copies, no second launch.
//  - Index words come by loads straight into LDS (load_to_lds), a ring of four units per wave, and are read back in the
//    operand's layout: no table, no transposition, and no barrier in the main loop.
//  - A lane dequantises 32 weights of its row in registers (xfp_dequant.h: 5, 5 and 10 VALU clocks per weight and SIMD at 2,
//    3 and 4 bits; a v_perm_b32 takes 4, a two-operand instruction 2).  At 5 and 6 bits 32 and 64 entries are too many for
//    that: one LDS lookup per weight, from a table in the lane's own bank, and 1.5 instructions to pair them up.
//  - Outliers: four rows of a wave at a time, an entry per lane, 16 tokens per entry from LDS.
//
// What bounds it: small matrices the launch (1.5 us), one round trip to memory and the instructions around the main loop
// (3000 x 2048, 3 bits, 8 tokens: 5.9 us, of which the main loop takes 0.8); large ones the VALU (28672 x 8192, 4 bits, one
// token: 36 us, HBM 22).  7001 x 5504 as above 9.9 us; 16384 x 3072, a scale and a mid-point per group, 24 tokens 36 -> 20.
// 5 and 6 bits the lookups (8192 x 4096, 5 bits, 16 tokens 95 us token by token in the general kernel, 26 here; 16257 x 6400,
// 9 tokens 227 / 56).
#pragma once
#include "xfp_dequant.h"

#include <atomic>
#include <type_traits>

namespace xfp {

struct FewArgs {
    DecodeArgs a;
    uint32_t M;            // tokens
    uint32_t RB, KW;       // blocks of 16 rows of a workgroup; waves that share a block's columns (the block's z and y)
    uint32_t J;            // rows whose outliers a wave adds
    uint32_t GS, per;      // groups of a slice of K (grid y); its units / KW
    uint32_t gsdiv, rwdiv; // 2^32 / GS, 2^32 / (16 RB), rounded up: quotients of numbers below 2^16 without a division
    uint32_t xpitch;       // bytes of a token's row in LDS
    uint32_t ringw;        // bytes of a wave's ring
    uint32_t o_lib, o_ids, o_rec, o_out, o_ring;               // LDS offsets
    int y_f32;
    float *part;           // several slices: fp32 planes [slice][M][N]; else null
};

namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const half8_t lds_ch8_t;
typedef __attribute__((address_space(3))) const u32x4_t lds_cu4_t;
typedef __attribute__((address_space(3))) const u32x2_t lds_cu2_t;
typedef __attribute__((address_space(3))) u32x4_t lds_u4_t;
typedef __attribute__((address_space(3))) float4_t lds_f4_t;
typedef __attribute__((address_space(3))) float lds_f32_t;
typedef __attribute__((address_space(3))) uint16_t lds_u16_t;
typedef __attribute__((address_space(3))) uint8_t lds_u8_t;

template <class T>
__device__ __forceinline__ T &at_lds(uint32_t o) { return *(T *)(uintptr_t)o; }

constexpr int kFewRing = 4;                                    // units of a wave in LDS
constexpr int few_loads(int bits) { return bits > 4 ? 2 : 1; } // loads of a unit: 64 lanes of 16 bytes (5 and 6 bits: 80 and 96, 3 bits: 48)
constexpr int few_unit(int bits) { return bits > 4 ? 256 * bits : 1024; }          // bytes of a unit there
constexpr int kFewOut = 256;                                   // outlier entries of a wave there
static_assert(kFewOut * 4 <= 1024, "");
template <int BITS>
constexpr int few_groups() { return BITS == 2 ? 2 : 1; }       // groups of a unit

// 8 activations (columns 8 p .. 8 p + 7 of a run of 32, natural order) to their slots of the run
template <int BITS>
__device__ __forceinline__ void put_x(uint32_t run, uint32_t p, const uint4 &w)
{
    constexpr uint32_t kLow = 0x05040100u, kHigh = 0x07060302u;
    if constexpr (BITS == 4) {
        at_lds<lds_u4_t>(run + 16 * p) = u32x4_t{__builtin_amdgcn_perm(w.y, w.x, kLow), __builtin_amdgcn_perm(w.w, w.z, kLow),
                                                 __builtin_amdgcn_perm(w.y, w.x, kHigh), __builtin_amdgcn_perm(w.w, w.z, kHigh)};
    } else if constexpr (BITS > 4) {
        at_lds<lds_u4_t>(run + 16 * p) = u32x4_t{w.x, w.y, w.z, w.w};
    } else if constexpr (BITS == 2) {
        const uint32_t o = run + 32 * (p >> 1) + 4 * (p & 1);
        at_lds<lds_u32_t>(o) = __builtin_amdgcn_perm(w.z, w.x, kLow);
        at_lds<lds_u32_t>(o + 8) = __builtin_amdgcn_perm(w.z, w.x, kHigh);
        at_lds<lds_u32_t>(o + 16) = __builtin_amdgcn_perm(w.w, w.y, kLow);
        at_lds<lds_u32_t>(o + 24) = __builtin_amdgcn_perm(w.w, w.y, kHigh);
    } else {
        const uint32_t v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            at_lds<lds_u16_t>(run + 16 * j + 2 * p) = (uint16_t)v[j];
            at_lds<lds_u16_t>(run + 16 * j + 8 + 2 * p) = (uint16_t)(v[j] >> 16);
        }
    }
}

// Chunk c (0..3) of a run of 32 at 5 and 6 bits: slots 8 c .. 8 c + 7 as fp16 pairs, looked up in a bank that no other lane of
// the half wave reads: entry e at table + 128 e.
template <int BITS, int C>
__device__ __forceinline__ u32x4_t look_up(const words_t<BITS> &w, uint32_t table)
{
    uint32_t v[8];
    auto one = [&](auto slot) {
        constexpr int t = decltype(slot)::value, bit = BITS * (8 * C + t), word = bit / 32, sh = bit % 32;
        uint32_t f;                                            // the field at bit 7
        if constexpr (sh + BITS > 32) f = __builtin_amdgcn_alignbit(w[word + 1], w[word], sh - 7);
        else if constexpr (sh >= 7) f = w[word] >> (sh - 7);
        else f = w[word] << (7 - sh);
        v[t] = at_lds<lds_cu32_t>((f & (((1u << BITS) - 1) << 7)) + table);
    };
    one(std::integral_constant<int, 0>{}); one(std::integral_constant<int, 1>{}); one(std::integral_constant<int, 2>{}); one(std::integral_constant<int, 3>{});
    one(std::integral_constant<int, 4>{}); one(std::integral_constant<int, 5>{}); one(std::integral_constant<int, 6>{}); one(std::integral_constant<int, 7>{});
    return u32x4_t{v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16};
}

// Waves of a workgroup at most (few_plan).  With more than 32 tokens the sums alone ask for more than the 128 registers that 16
// waves leave (2 bits, a scale and a mid-point per group: 146, spilled within 128).
constexpr int few_waves(int bits, int tokens) { return tokens <= 32 && bits <= 4 ? 16 : 8; }

template <int BITS, int MODE, int T>
__global__ __launch_bounds__(kWave * few_waves(BITS, 16 * T)) void decode_few_kernel(FewArgs fa)
{
    static_assert(BITS <= 4 || MODE == 0, "");
    constexpr int ND = Planes<BITS>::ND, GU = few_groups<BITS>(), NL = few_loads(BITS), kUnit = few_unit(BITS);
    extern __shared__ __align__(256) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const DecodeArgs &a = fa.a;
    const uint32_t lane = threadIdx.x, KW = fa.KW, kw = __builtin_amdgcn_readfirstlane(threadIdx.y), rb = __builtin_amdgcn_readfirstlane(threadIdx.z);
    const uint32_t wave = rb * KW + kw, tid = wave * 64 + lane, nw = KW * fa.RB, nt = nw * 64;
    const uint32_t i = lane & 15, q = lane >> 4;
    const uint32_t N = a.N, K = a.K, M = fa.M, G = K / kGroup, wpr = K / 32 * BITS;
    const uint32_t RW = 16 * fa.RB;
    const uint32_t r0 = blockIdx.x * RW, rows = min(N - r0, RW);
    const uint32_t g0 = blockIdx.y * fa.GS, gs = min(G - g0, fa.GS);
    const size_t row0 = r0;
    const uint16_t *x = a.x + (size_t)g0 * kGroup;

    // ---------------------------------------------------------------- requests
    // Loads complete in the order they are asked for: activations, then what is small, then the index words.  Nothing here
    // waits for a load.
    const uint32_t cpt = gs * (kGroup / 8), total = M * cpt;   // 16-byte chunks of a token, of all
    constexpr int XB = 4;
    uint4 xv[XB];
    uint32_t xm[XB], xc[XB];
    uint32_t m_ = 0, c_ = tid;
    auto request_x = [&](uint32_t done) {
#pragma unroll
        for (int b = 0; b < XB; ++b) {
            if (done + b * nt >= total) break;                 // wave-uniform
            while (c_ >= cpt) { c_ -= cpt; ++m_; }
            xm[b] = m_;
            xc[b] = c_;
            xv[b] = *reinterpret_cast<const uint4 *>(x + (size_t)min(m_, M - 1) * a.x_stride + 8 * c_);
            c_ += nt;
        }
    };
    auto put = [&](uint32_t done) {
#pragma unroll
        for (int b = 0; b < XB; ++b) {
            if (done + b * nt >= total) break;
            if (xm[b] >= M) continue;
            uint4 v = xv[b];
            if (a.x_bf16) v = make_uint4(bf16x2_to_f16x2(v.x), bf16x2_to_f16x2(v.y), bf16x2_to_f16x2(v.z), bf16x2_to_f16x2(v.w));
            put_x<BITS>(lds0 + xm[b] * fa.xpitch + (xc[b] >> 2) * 64, xc[b] & 3u, v);
        }
    };
    request_x(0);
    // row pointers of this wave's rows (for the outliers): lane l: first entry of row J wave + l
    const uint32_t J = fa.J;
    const int32_t rpv = a.rp[row0 + min(wave * J + min(lane, J), rows)];
    Planes<BITS> P;
    uint32_t cbw[BITS > 4 ? 1 : 1 << (BITS - 1)];
    uint2 libw = make_uint2(0u, 0u);
    uint32_t idw = 0;
    uint16_t scw = 0, miw = 0;
    const uint16_t *lib = a.cb;
    const uint8_t *gid = a.gid + row0 * G + g0;
    const uint16_t *gsc = a.gscale + row0 * G + g0, *gmi = a.gmid + row0 * G + g0;
    auto div_gs = [&](uint32_t v) { return gs == fa.GS && gs > 1 ? __umulhi(v, fa.gsdiv) : v / gs; };
    const uint32_t nid = rows * gs;                            // ids of the workgroup
    auto load_id4 = [&](uint32_t j) -> uint32_t {              // four of them, in the order of the rows
        uint32_t v = 0;
        if (gs == G) {
            if (4 * j + 3 < nid) __builtin_memcpy(&v, gid + 4 * j, 4);
            else for (uint32_t b = 0; 4 * j + b < nid; ++b) v |= (uint32_t)gid[4 * j + b] << (8 * b);
        } else {
#pragma unroll
            for (uint32_t b = 0; b < 4; ++b) {
                const uint32_t o = min(4 * j + b, nid - 1), r = div_gs(o);
                v |= (uint32_t)gid[(size_t)r * G + (o - r * gs)] << (8 * b);
            }
        }
        return v;
    };
    const uint32_t *cb = reinterpret_cast<const uint32_t *>(a.cb) + row0 * (1 << (BITS - 1));
    const uint32_t co = min(rb * 16 + i, rows - 1) * (1 << (BITS - 1));
    if constexpr (BITS > 4) {
        cbw[0] = cb[co + min(kw, (1u << (BITS - 1)) - 1)];
    } else if constexpr (MODE == 0) {
#pragma unroll
        for (int d = 0; d < (1 << (BITS - 1)); ++d) cbw[d] = cb[co + d];
    } else {
        const uint32_t j = min(tid, a.L * ND - 1);
        libw = *reinterpret_cast<const uint2 *>(lib + 4 * j);
        if (4 * tid < nid) idw = load_id4(tid);
    }
    if constexpr (MODE == 2) {
        const uint32_t j = min(tid, nid - 1), r = div_gs(j);
        const size_t o = (size_t)r * G + (j - r * gs);
        scw = gsc[o];
        miw = gmi[o];
    }

    // index words: a unit is 16 rows x 128 columns (2 bits: 256), 16 bytes per lane straight into the wave's ring.
    // Four (3 bits: three) neighbouring lanes take the 64 (48) bytes of a row; with 64 the chunk's place is turned by the
    // row, so that the 16 lanes that read one chunk of 16 rows later find them in different banks.
    const uint32_t U = (gs + GU - 1) / GU, per = gs == fa.GS ? fa.per : U / KW, rem = U - per * KW;
    const uint32_t u0 = kw * per + min(kw, rem), n = rb * 16 < rows ? per + (kw < rem) : 0u;
    const uint32_t ring = lds0 + fa.o_ring + wave * fa.ringw;
    const uint64_t base = (uint64_t)(uintptr_t)(a.idx + (row0 + rb * 16) * wpr);
    const u32x4_t ri = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base),
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(base >> 32) & 0xFFFFu)),
                        rb * 16 < rows ? min(16u, rows - rb * 16) * (wpr * 4) : 0u, 0x00020000u};
    uint32_t voff[NL];
#pragma unroll
    for (int d = 0; d < NL; ++d) {
        const uint32_t id = d * 64 + lane;
        if constexpr (BITS == 4 || BITS == 2) voff[d] = id / 4 * (wpr * 4) + ((id ^ (id >> 4)) & 3) * 16;
        else voff[d] = id < 16 * BITS ? id / BITS * (wpr * 4) + id % BITS * 16 : 0x7FFFFFF0u;
    }
    auto request = [&](uint32_t t) {                           // the wave's t-th unit
#pragma unroll
        for (int d = 0; d < NL; ++d)
            if (d == 0 || lane < 16 * BITS - 64)               // (a lane that is off writes nothing to LDS)
                load_to_lds(__builtin_amdgcn_readfirstlane(ring + (t % kFewRing) * kUnit + d * 1024), voff[d] + (g0 + (u0 + t) * GU) * (16 * BITS), ri, 0);
    };
#pragma unroll
    for (uint32_t t = 0; t < (uint32_t)kFewRing; ++t)
        if (t < n) request(t);

    // ---------------------------------------------------------------- what every wave reads: LDS
    put(0);
    for (uint32_t done = XB * nt; done < total; done += XB * nt) {
        request_x(done);
        put(done);
    }
    // outliers: this wave's entries (column | value << 16) are one run, of which kFewOut at a time pass through LDS behind the
    // main loop; the first are asked for here
    const int32_t ob = __builtin_amdgcn_readlane(rpv, 0), oend = __builtin_amdgcn_readlane(rpv, (int)J);
    uint32_t oc[kFewOut / 64], ov[kFewOut / 64];
    auto request_outliers = [&](int32_t from) {
#pragma unroll
        for (int b = 0; b < kFewOut / 64; ++b) {
            if (from + 64 * b >= oend) break;                  // wave-uniform
            const int32_t at = min(from + 64 * b + (int32_t)lane, oend - 1);
            oc[b] = (uint32_t)a.col[at];
            ov[b] = a.val[at];
        }
    };
    request_outliers(ob);
    if constexpr (MODE != 0) {
        // the library as byte planes: entry l at o_lib + l * 2^BITS * 2, low bytes first
        for (uint32_t j = tid; j < a.L * ND; j += nt) {
            if (j != tid) libw = *reinterpret_cast<const uint2 *>(lib + 4 * j);
            const uint32_t o = lds0 + fa.o_lib + (j / ND) * (2u << BITS) + (j % ND) * 4;
            at_lds<lds_u32_t>(o) = __builtin_amdgcn_perm(libw.y, libw.x, 0x06040200u);
            at_lds<lds_u32_t>(o + ND * 4) = __builtin_amdgcn_perm(libw.y, libw.x, 0x07050301u);
        }
        for (uint32_t j = tid; 4 * j < nid; j += nt) {
            if (j != tid) idw = load_id4(j);
            at_lds<lds_u32_t>(lds0 + fa.o_ids + 4 * j) = idw;
        }
    } else if constexpr (BITS > 4) {
        // a table per row, twice, in banks of its own (LDS serves 32 lanes at a time): entry e of lane l at e * 128 + l % 32 * 4;
        // lanes 0 to 31 write the first entry of a dword, the others the second
        for (uint32_t d = kw; d < (1u << (BITS - 1)); d += KW) {
            const uint32_t v = d == kw ? cbw[0] : cb[co + d];
            at_lds<lds_u32_t>(lds0 + fa.o_lib + rb * (128u << BITS) + d * 256 + (lane >> 5) * 128 + (lane & 31) * 4) = lane < 32 ? v & 0xFFFFu : v >> 16;
        }
    } else {
        P.set(cbw);
    }
    if constexpr (MODE == 2) {
        // scale | mid-point << 16 of row r, group g at o_rec + ((r / 16 * gs + g) * 20 + r % 16) * 4
        for (uint32_t j = tid; j < nid; j += nt) {
            const uint32_t r = div_gs(j), g = j - r * gs;
            const size_t o = (size_t)r * G + g;
            if (j != tid) { scw = gsc[o]; miw = gmi[o]; }
            at_lds<lds_u32_t>(lds0 + fa.o_rec + (((r >> 4) * gs + g) * 20 + (r & 15u)) * 4) = (uint32_t)scw | ((uint32_t)miw << 16);
        }
    }
    lds_barrier();

    // ---------------------------------------------------------------- main loop
    float4_t sum[T];
#pragma unroll
    for (int t = 0; t < T; ++t) sum[t] = float4_t{};
    uint32_t xb[T];
#pragma unroll
    for (int t = 0; t < T; ++t) xb[t] = lds0 + min(16u * t + i, M - 1) * fa.xpitch + 64 * q;
    const uint32_t ids = lds0 + fa.o_ids + (rb * 16 + min(i, rows - 1 - min(rb * 16, rows - 1))) * gs;
    const uint32_t recs = lds0 + fa.o_rec + (rb * gs * 20 + 4 * q) * 4;
    const uint32_t table = lds0 + fa.o_lib + rb * (128u << BITS) + (lane & 31) * 4;    // (5 and 6 bits)
    words_t<BITS> w[GU], wn[GU];
    auto take = [&](uint32_t t, words_t<BITS> (&v)[GU]) {      // a unit's words: lane (i, q): 32 weights of row i per group
        const uint32_t s = ring + (t % kFewRing) * kUnit;
        if constexpr (BITS == 4) v[0] = at_lds<lds_cu4_t>(s + i * 64 + ((q ^ (i >> 2)) & 3) * 16);
        else if constexpr (BITS != 2) {
#pragma unroll
            for (int d = 0; d < BITS; ++d) v[0][d] = at_lds<lds_cu32_t>(s + i * (16 * BITS) + q * (4 * BITS) + d * 4);
        } else {
#pragma unroll
            for (int g = 0; g < 2; ++g) v[g] = at_lds<lds_cu2_t>(s + i * 64 + (((2 * g + (q >> 1)) ^ (i >> 2)) & 3) * 16 + (q & 1) * 8);
        }
    };
    // unit t has landed; the min(kFewRing - 2, n - 1 - t) units behind it that have been requested may be under way
    auto wait = [&](uint32_t t) {
        if (t + kFewRing - 2 < n) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kFewRing - 2) * NL) : "memory");
        else if (t + 1 < n && kFewRing > 3) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    static_assert(kFewRing == 4, "the waits");
    if (n) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (the waits for the loads above have drained them already)
        take(0, w);
    }
#pragma unroll 1
    for (uint32_t t = 0; t < n; ++t) {
        if (t + 1 < n) {
            wait(t + 1);
            take(t + 1, wn);
        }
#pragma unroll
        for (int s = 0; s < GU; ++s) {
            const uint32_t g = (u0 + t) * GU + s;              // of the slice
            if (GU > 1 && g >= gs) break;
            if constexpr (MODE != 0) {
                const uint32_t o = lds0 + fa.o_lib + (uint32_t)at_lds<lds_u8_t>(ids + g) * (2u << BITS);
                if constexpr (BITS == 4) {
                    const u32x4_t l = at_lds<lds_cu4_t>(o), h = at_lds<lds_cu4_t>(o + 16);
#pragma unroll
                    for (int d = 0; d < 4; ++d) { P.lo[d] = l[d]; P.hi[d] = h[d]; }
                } else if constexpr (BITS == 3) {
                    const u32x4_t l = at_lds<lds_cu4_t>(o);
                    P.lo[0] = l[0]; P.lo[1] = l[1]; P.hi[0] = l[2]; P.hi[1] = l[3];
                } else {
                    const u32x2_t l = at_lds<lds_cu2_t>(o);
                    P.lo[0] = l[0]; P.hi[0] = l[1];
                }
            }
            if constexpr (BITS <= 4) arrange<BITS>(w[s]);
            // two chains of two steps: what a longer one loses shows in the results (512 columns: 8.9e-8 of them against 64 bits
            // with one chain of four, 7.5e-8 with two)
            float4_t acc[2][T], ones[2][MODE == 2 ? T : 1];
            auto step = [&](auto cc) {
                constexpr int c = decltype(cc)::value;
                half8_t af;
                if constexpr (BITS > 4) af = __builtin_bit_cast(half8_t, look_up<BITS, c>(w[s], table));
                else af = __builtin_bit_cast(half8_t, chunk<BITS>(P, w[s], c));
#pragma unroll
                for (int tt = 0; tt < T; ++tt) {
                    const half8_t bf = at_lds<lds_ch8_t>(xb[tt] + g * 256 + 16 * c);
                    acc[c / 2][tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af, bf, c % 2 == 0 ? float4_t{} : acc[c / 2][tt], 0, 0, 0);
                    if constexpr (MODE == 2) {
                        const half8_t one = {1, 1, 1, 1, 1, 1, 1, 1};
                        ones[c / 2][tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(one, bf, c % 2 == 0 ? float4_t{} : ones[c / 2][tt], 0, 0, 0);
                    }
                }
            };
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
            if constexpr (MODE == 2) {
                const u32x4_t rec = at_lds<lds_cu4_t>(recs + g * 80);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float sc = half_bits_to_float((uint16_t)rec[r]), mi = half_bits_to_float((uint16_t)(rec[r] >> 16));
#pragma unroll
                    for (int tt = 0; tt < T; ++tt)
                        sum[tt][r] += fmaf(sc, acc[0][tt][r] + acc[1][tt][r], mi * (ones[0][tt][r] + ones[1][tt][r]));
                }
            } else {
#pragma unroll
                for (int tt = 0; tt < T; ++tt) sum[tt] += acc[0][tt] + acc[1][tt];
            }
        }
        if (t + kFewRing < n) {
#pragma unroll
            for (int s = 0; s < GU; ++s) asm volatile("" : "+v"(w[s]));     // the slot's words are in registers
            request(t + kFewRing);
        }
#pragma unroll
        for (int s = 0; s < GU; ++s) w[s] = wn[s];
    }

    // ---------------------------------------------------------------- the outlier term, from the resident activations
    // Four of this wave's rows at a time, 16 lanes each, an entry per lane: its place in LDS is worked out once, then the 16
    // tokens of a chunk are a read and a multiply-add each.  The lanes of a row meet in a fixed tree.
    const uint32_t el = lane & 15, er = lane >> 4, op = (M + 3) & ~3u;
    int32_t from = ob;                                         // the entries in LDS: from .. from + kFewOut - 1
    auto keep = [&] {
#pragma unroll
        for (int b = 0; b < kFewOut / 64; ++b) {
            if (from + 64 * b >= oend) break;
            at_lds<lds_u32_t>(ring + (64 * b + lane) * 4) = oc[b] | (ov[b] << 16);
        }
    };
    if (ob < oend) keep();
#pragma unroll 1
    for (uint32_t t0 = 0, j0 = 0; t0 < M; j0 + 4 < J ? j0 += 4 : (j0 = 0, t0 += 16)) {
        float s[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) s[m] = 0.f;
        const int32_t first = __builtin_amdgcn_readlane(rpv, (int)min(j0, J)), all = __builtin_amdgcn_readlane(rpv, (int)min(j0 + 4, J));
        if (first < all) {
            if (first < from || first >= from + kFewOut) {     // (a later chunk of tokens whose entries have been replaced)
                from = first;
                request_outliers(from);
                keep();
            }
            int32_t at = __builtin_amdgcn_ds_bpermute((int)(min(j0 + er, J) * 4), rpv) + (int32_t)el;
            const int32_t ee = __builtin_amdgcn_ds_bpermute((int)(min(j0 + er + 1, J) * 4), rpv);
            for (;;) {
                const int32_t to = min(ee, from + kFewOut);
                for (; at < to; at += 16) {
                    const uint32_t en = at_lds<lds_u32_t>(ring + (uint32_t)(at - from) * 4), k = (en & 0xFFFFu) - g0 * kGroup;
                    if (k >= gs * kGroup) continue;            // another slice's column
                    const float v = half_bits_to_float((uint16_t)(en >> 16));
                    const uint32_t xo = lds0 + (k >> 5) * 64 + slot_of<BITS>(k & 31u) * 2;
                    // (one chunk: the tokens' rows do not change with t0 and are worked out once)
                    const uint32_t chunk0 = T == 1 ? 0u : t0;
#pragma unroll
                    for (int m4 = 0; m4 < 16; m4 += 4) {
                        if (t0 + m4 >= M) break;
                        uint16_t xw[4];
#pragma unroll
                        for (int m = 0; m < 4; ++m) xw[m] = at_lds<lds_u16_t>(xo + min(chunk0 + m4 + m, M - 1) * fa.xpitch);        // (past the last token: again the last)
#pragma unroll
                        for (int m = 0; m < 4; ++m) s[m4 + m] = fmaf(v, half_bits_to_float(xw[m]), s[m4 + m]);
                    }
                }
                if (all <= from + kFewOut) break;
                from += kFewOut;
                request_outliers(from);
                keep();
            }
#pragma unroll
            for (int m4 = 0; m4 < 16; m4 += 4) {
                if (t0 + m4 >= M) break;
#pragma unroll
                for (int m = m4; m < m4 + 4; ++m) s[m] = dpp_add<0x128>(s[m]);             // row_ror:8
#pragma unroll
                for (int m = m4; m < m4 + 4; ++m) s[m] = dpp_add<0x124>(s[m]);             // row_ror:4
#pragma unroll
                for (int m = m4; m < m4 + 4; ++m) s[m] = dpp_add<0x4E>(s[m]);              // quad_perm [2,3,0,1]
#pragma unroll
                for (int m = m4; m < m4 + 4; ++m) s[m] = dpp_add<0xB1>(s[m]);              // quad_perm [1,0,3,2]
            }
        }
        const uint32_t r = wave * J + j0 + er;
        if (el == 0 && j0 + er < J && r < RW) {
#pragma unroll
            for (int m4 = 0; m4 < 16; m4 += 4) {
                if (t0 + m4 >= M) break;
                at_lds<lds_f4_t>(lds0 + fa.o_out + (r * op + t0 + m4) * 4) = float4_t{s[m4], s[m4 + 1], s[m4 + 2], s[m4 + 3]};
            }
        }
    }

    // ---------------------------------------------------------------- the waves' sums, in their order, then the outliers
    // A wave's sums go where its ring was: [token][16 rows], rows 20 floats apart.
#pragma unroll
    for (int t = 0; t < T; ++t)
        if (16u * t + i < M) at_lds<lds_f4_t>(ring + ((16 * t + i) * 20 + 4 * q) * 4) = sum[t];
    lds_barrier();
    for (uint32_t o = tid; o < RW * M; o += nt) {
        const uint32_t m = __umulhi(o, fa.rwdiv), r = o - m * RW;
        if (r >= rows) continue;
        const uint32_t at = lds0 + fa.o_ring + (r >> 4) * KW * fa.ringw + (m * 20 + (r & 15u)) * 4;
        float part[4] = {0.f, 0.f, 0.f, 0.f};
        for (uint32_t k = 0; k < KW; k += 4)
#pragma unroll
            for (uint32_t b = 0; b < 4; ++b)
                if (k + b < KW) part[b] += at_lds<lds_f32_t>(at + (k + b) * fa.ringw);
        float s = (part[0] + part[1]) + (part[2] + part[3]);
        s += at_lds<lds_f32_t>(lds0 + fa.o_out + (r * op + m) * 4);
        if (fa.part) fa.part[((size_t)blockIdx.y * M + m) * N + r0 + r] = s;
        else store_out(a.y, (int64_t)m * a.y_stride + r0 + r, s, fa.y_f32 != 0, a.y_bf16 != 0);
    }
}

inline uint32_t few_up16(uint32_t v) { return (v + 15) & ~15u; }

// What follows from a call's tokens and its split (RB, KW, GS); returns the bytes of LDS a workgroup needs.
inline uint32_t few_layout(int bits, int mode, uint32_t L, uint32_t M, uint32_t RB, uint32_t KW, uint32_t GS, FewArgs &fa)
{
    const uint32_t nw = RB * KW, GU = bits == 2 ? 2 : 1, U = (GS + GU - 1) / GU, most = (U + KW - 1) / KW;
    fa.M = M;
    fa.RB = RB;
    fa.KW = KW;
    fa.GS = GS;
    fa.per = U / KW;
    fa.J = (16 * RB + nw - 1) / nw;
    fa.gsdiv = GS == 1 ? 0u : (uint32_t)(((1ull << 32) + GS - 1) / GS);
    fa.rwdiv = (uint32_t)(((1ull << 32) + 16 * RB - 1) / (16 * RB));
    fa.xpitch = GS * 256 + 16;
    uint32_t o = M * fa.xpitch;
    fa.o_lib = o;
    if (mode) o += L * (2u << bits);
    if (bits > 4) o += RB * (128u << bits);
    fa.o_ids = o;
    if (mode) o = few_up16(o + RB * 16 * GS + 4);
    fa.o_rec = o;
    if (mode == 2) o += RB * GS * 80;
    fa.ringw = (most < (uint32_t)kFewRing ? most : (uint32_t)kFewRing) * (uint32_t)few_unit(bits);
    if (fa.ringw < M * 80) fa.ringw = M * 80;                  // the wave's sums take its place
    fa.o_ring = o;
    o += nw * fa.ringw;
    fa.o_out = o;
    return o + RB * 16 * ((M + 3) & ~3u) * 4;
}

template <int BITS, int MODE, int T>
hipError_t launch_few_t(const FewArgs &fa, dim3 grid, int lds, hipStream_t s)
{
    auto kern = decode_few_kernel<BITS, MODE, T>;
    static std::atomic<int> configured[kMaxDevices];           // per device; idempotent attribute, benign race
    const int dev = current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    if (!configured[dev].load(std::memory_order_relaxed)) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (err != hipSuccess) return err;
        configured[dev].store(1, std::memory_order_relaxed);
    }
    hipLaunchKernelGGL(kern, grid, dim3(kWave, fa.KW, fa.RB), lds, s, fa);
    return hipGetLastError();
}

template <int BITS>
hipError_t launch_few_bits(int mode, const FewArgs &fa, dim3 grid, int lds, hipStream_t s)
{
    const int T = fa.M <= 16 ? 1 : fa.M <= 32 ? 2 : 4;
#define XFP_FEW(MODE) \
    (T == 1 ? launch_few_t<BITS, MODE, 1>(fa, grid, lds, s) : T == 2 ? launch_few_t<BITS, MODE, 2>(fa, grid, lds, s) \
                                                                             : launch_few_t<BITS, MODE, 4>(fa, grid, lds, s))
    if constexpr (BITS > 4) return mode == 0 ? XFP_FEW(0) : hipErrorInvalidValue;
    else return mode == 2 ? XFP_FEW(2) : mode == 1 ? XFP_FEW(1) : XFP_FEW(0);
#undef XFP_FEW
}

}  // namespace
}  // namespace xfp
