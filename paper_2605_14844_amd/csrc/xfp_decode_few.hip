// Host side of the kernel of xfp_decode_few.inc.h: which calls it is the faster one for, and how a call's rows and columns
// are shared out.
#include "xfp_decode_few.inc.h"

namespace xfp {

// defined in xfp_decode_few2.hip, xfp_decode_few3.hip, xfp_decode_few4.hip, xfp_decode_few56.hip
hipError_t launch_few2(int mode, const FewArgs &fa, dim3 grid, int lds, hipStream_t s);
hipError_t launch_few3(int mode, const FewArgs &fa, dim3 grid, int lds, hipStream_t s);
hipError_t launch_few4(int mode, const FewArgs &fa, dim3 grid, int lds, hipStream_t s);
hipError_t launch_few56(int bits, const FewArgs &fa, dim3 grid, int lds, hipStream_t s);

namespace {

constexpr uint32_t kLds = 160 * 1024;
constexpr uint32_t kCUs = 256;

// Blocks of 16 rows, waves per block, groups per slice of K: as few slices as the activations' place in LDS allows (a second
// launch adds the slices' sums), the blocks of all slices in one round of the 256 CUs (a slice's share of them rounded down:
// 86 x 3 workgroups of 3 blocks are two rounds, 4096 x 14336, 4 bits, 8 tokens 27.6 us, 64 x 3 of 4 blocks one, 20.1), and the
// 16 waves that a CU holds at this kernel's registers (8 from 33 tokens on, whose sums take 5 KB of LDS per wave) sharing the
// blocks' columns.  7001 x 5504, 2 bits, 5 tokens, us for blocks x waves: 2 x 8 9.9, 2 x 4 11.3, 1 x 8 10.6, 1 x 16 13.8, 4 x 4 14.1.
// A slice of one to three units has no work in the main loop for more waves than that, but activations to stage, outliers and
// sums to share out: eight waves all the same, us with a wave per unit / eight: 335 x 256, 2 bits, 30 tokens 15.1 / 6.3; 1627 x
// 128, 4 bits, 26 tokens 11.5 / 5.9; 4297 x 128, 3 bits, 40 17.6 / 9.1; not in matrices of more blocks than CUs with few tokens
// (4096 rows and more of one unit, 2 to 4 tokens, 1.14 of the time with eight; 5 to 16 of two units 1.0).
struct FewPlan {
    uint32_t slices, lds;
    FewArgs fa;
};

bool few_plan(int bits, int mode, uint32_t L, uint32_t N, uint32_t K, uint32_t M, FewPlan &p)
{
    const uint32_t G = K / kGroup, GU = bits == 2 ? 2 : 1, blocks = (N + 15) / 16, most = (uint32_t)few_waves(bits, (int)M);
    const uint32_t x_most = kLds - most * 1024 - (mode ? L * (2u << bits) : 0u) - (bits > 4 ? 128u << bits : 0u);
    for (uint32_t S = (uint32_t)(((uint64_t)M * G * 256 + x_most - 1) / x_most); S <= G; ++S) {
        uint32_t GS = (G + S - 1) / S;
        if (bits == 2) GS = (GS + 1) & ~1u;
        p.slices = (G + GS - 1) / GS;
        const uint32_t share = p.slices < kCUs ? kCUs / p.slices : 1;       // workgroups of a slice in one round
        uint32_t RB = (blocks + share - 1) / share, KW;
        if (RB > most) RB = most;
        KW = most / RB;
        const uint32_t units = (GS + GU - 1) / GU;
        if (KW > units) KW = units >= 4 || (blocks > kCUs && M <= 16) ? units : KW < 8 ? KW : 8;
        p.lds = few_layout(bits, mode, L, M, RB, KW, GS, p.fa);
        if (p.lds <= kLds) return true;
    }
    return false;
}

}  // namespace

// How many of `left` tokens the next launch takes in this kernel, 0: none (another kernel is faster).  plane: floats of the
// scratch plane for the sums of several slices.  general: the other kernel is the general one.
// One launch without a re-laid copy of the activations and without tables wins wherever the activations fit, and loses its
// edge with the slices that they are cut into otherwise: every slice stages its activations and reads its rows' outliers
// anew.  Measured, us in the other kernels / here (graph replay, cold weights):
//  - 2 to 8 tokens: 4096 x 2048 8.3 / 5.0, 7001 x 5504 16 / 9.9, 8192 x 8192 (2 slices) 24 / 18, 28672 x 4096 57 / 27, but
//    8192 x 14336 (3 slices) 38 / 51; rows beyond 8192 columns in matrices of up to 8160 rows, which are three launches
//    elsewhere, in any number of slices while a workgroup has no more than eight blocks (of 1353 such calls one lost more than
//    0.04; of 327 with nine and more, which leave its CU half of its waves, every fourth: 3000 x 28672 16 tokens 28 / 39): 4 bits
//    4096 x 14336 8 tokens 21.8 / 20.1, 16 22.3 / 23.2; 4096 x 20480 16 30 / 28; 4096 x 28672 6 33 / 28; 300 x 20480 2 to 16
//    16.4 .. 17.8 / 15.8 .. 12.1; 2 bits 8160 x 14336 8 29 / 21;
//  - 9 to 16: 4096 x 2048 9.8 / 7.4, 28672 x 1024 22 / 12, 12000 x 5504 (2 slices) 43 / 21, but 4096 x 8192 (3) 19.5 / 22;
//  - 17 to 32: 600 x 1536 11.2 / 7.7, 28672 x 1024 20.5 / 13.9, 600 x 14336 27 / 16, but 8192 x 4096 17 / 36;
//  - 33 to 64, where the other kernel's tables serve more tokens: 300 x 4096 15 / 13, 600 x 14336 52 / 21, 1200 x 14336
//    53 / 22, but 1200 x 4096 23 / 28 and 1200 x 640 10.6 / 13.7;
//  - a scale and a mid-point per group, which run token by token or 16 at a time elsewhere: 8 tokens 16384 x 3072 17.8 / 12.7,
//    24 4096 x 4096 30 / 14, 64 2000 x 2048 37 / 30 and 64 12000 x 5504 97 / 95 (16 at a time), but 2 to 4 tokens of
//    1200 x 4096 6.6 / 7.3 and 40 of 8192 x 8192 66 / 88; and few rows, which leave the token-by-token kernel room for all tokens
//    at once: 73 x 256 45 tokens 3.6 / 9, 387 x 2176 2 3.3 / 5.2, 1752 x 1664 2 4.4 / 5.6 but 16 14.6 / 7.5, 319 x 4480 8 5.3 / 8.1,
//    851 x 1024 16 8.6 / 6.3, 125 x 2560 16 4.1 / 8.6, 835 x 2048 48 15.7 / 23.5;
//  - 5 and 6 bits, which run token by token elsewhere: 8192 x 4096 2 tokens 13.3 / 13.0, 16 75 / 27 (8 at a time); 12933 x 1152 2 11.4 / 11.2;
//    16257 x 6400 9 164 / 58; 8192 x 8192 4 42 / 21; 2213 x 11392 28 101 / 100; but 617 x 14208 2 8.6 / 17; 500 x 8192 9
//    10 / 23; 300 x 1024 16 4.5 / 5.7; and of few long rows, in several launches that leave CUs idle, 1024 x 23424 42 155 / 463,
//    1526 x 14592 6 26 / 34, 32 95 / 137, 1201 x 7936 22 36 / 48, 827 x 3840 27 15 / 20.  As many tokens per launch as fit in one slice (these calls take no scratch elsewhere, so they get none here);
//  - one token: library rows that neither fit the registers of the streaming kernel nor leave it time for slices:
//    8192 x 28672 45 / 35 (4 bits), 57 / 32 (2 bits), with a scale and a mid-point 76 / 36; 4 bits 6411 x 19712 31 / 29,
//    but 5524 x 28672 35 / 39, 4577 x 21888 24 / 29; 3 bits 5310 x 23680 31 / 25, 4611 x 17280 18.7 / 20.1; 300 x 20480 6.7 / 12.
//    Rows of a length with no equal slices for that kernel, which one wave each of the general kernel walks: V2 2 bits 3300 x 22784
//    18 / 14, 3 bits 3300 x 21376 17.3 / 15.6, but 4 bits, V2a 300 x 21376 9.2 / 17; 3300 x 17024 16.9 / 16.7; a scale and a mid-point
//    3300 x 21376 21 / 18, but 1300 x 17792 10.4 / 15.3.  (The lines were drawn when the general kernel took up to twice that; by
//    these figures it would keep more: V2 2 bits 300 x 21376 8.3 / 11.7, 3 bits 1300 x 18688 9.2 / 13.3, 5000 x 17792 16.9 / 19.6, a scale and a
//    mid-point, 4 bits 2048 x 21376 13.5 / 20.2.)
int few_tokens(int bits, int mode, uint32_t L, uint32_t N, uint32_t K, int left, uint64_t plane, bool general)
{
    if (bits < 2 || (bits > 4 && mode != 0) || K > 65536 || left < 1) return 0;   // (an outlier's column is kept in 16 bits)
    FewPlan p;
    auto fits = [&](uint32_t m) { return few_plan(bits, mode, L, N, K, m, p) && (p.slices == 1 || (uint64_t)p.slices * m * N <= plane); };
    if (bits > 4) {
        const uint32_t all = left < 64 ? (uint32_t)left : 64u;
        if (N <= (K > 8192 ? 2048u : K >= 5632 ? 1280u : K >= 3072 ? 896u : 0u)) return 0;
        for (uint32_t c = 1; c < all; ++c) {
            const uint32_t m = (all + c - 1) / c;
            if (N < 4096 && (uint64_t)m * N * K < 40u << 20) return 0;
            if (fits(m) && p.slices == 1) return (int)m;
        }
        return 0;
    }
    if (left == 1) {
        if (K <= 16384) return 0;
        const bool faster = general ? (bits <= 3 && mode != 2) || (N >= 2048 && mode != 0)
                                    : mode != 0 && N >= (mode == 2 || bits == 2 ? 4096u : bits == 3 ? 4864u : 5632u);
        return faster && fits(1) ? 1 : 0;
    }
    const bool split = K > 8192 && N <= 8160;                  // three launches in the 16-token kernel
    const uint32_t m = left < 64 ? (uint32_t)left : 64u;
    if (mode == 2 && plane == 0 && !general && (N <= (m <= 8 || (m > 32 && K >= 1280) ? 1008u : 640u) || (m <= 5 && (uint64_t)N * m <= (bits == 4 ? 4096u : 6144u)))) return 0;
    if (m <= 16) {
        if (mode == 2 && m <= 4 && K >= 4096 && (uint64_t)N * m <= 8192) return 0;
        return fits(m) && (p.slices <= 2 || (split && p.fa.RB <= 8)) ? (int)m : 0;
    }
    if (m <= 32) {
        if (fits(m) && (p.slices == 1 || N <= 1008 || (mode == 2 && p.slices <= 2))) return (int)m;
    } else if (mode == 2 ? N <= 2048 : (N <= 1008 && K >= 8192) || (N <= 640 && K >= 4096)) {
        if (fits(m)) return (int)m;
    } else if (mode == 2) {
        if (fits(32) && p.slices <= 2) return 32;
    }
    if (mode == 2 && fits(16) && p.slices <= 2) return 16;
    return 0;
}

// M tokens (few_tokens), fp32 planes of the slices' sums in part
hipError_t launch_decode_few(int bits, int mode, const DecodeArgs &a, int M, bool y_f32, float *part, hipStream_t s)
{
    FewPlan p;
    if (!few_plan(bits, mode, a.L, a.N, a.K, (uint32_t)M, p) || (p.slices > 1 && !part)) return hipErrorInvalidValue;
    p.fa.a = a;
    p.fa.y_f32 = (int)y_f32;
    p.fa.part = p.slices > 1 ? part : nullptr;
    const dim3 grid((a.N + p.fa.RB * 16 - 1) / (p.fa.RB * 16), p.slices);
    hipError_t err = bits > 4    ? launch_few56(bits, p.fa, grid, (int)p.lds, s)
                     : bits == 4 ? launch_few4(mode, p.fa, grid, (int)p.lds, s)
                     : bits == 3 ? launch_few3(mode, p.fa, grid, (int)p.lds, s)
                                 : launch_few2(mode, p.fa, grid, (int)p.lds, s);
    if (err != hipSuccess || p.slices == 1) return err;
    return launch_splitk_sum(part, p.slices, a.N, M, a.y, a.y_stride, y_f32, a.y_bf16 != 0, s);
}

bool few_is_sliced(int bits, int mode, uint32_t L, uint32_t N, uint32_t K, int M)
{
    FewPlan p;
    return few_plan(bits, mode, L, N, K, (uint32_t)M, p) && p.slices > 1;
}

bool few_shares(int bits, int mode, uint32_t L, uint32_t N, uint32_t K, int M, unsigned *out)
{
    FewPlan p;
    if (!few_plan(bits, mode, L, N, K, (uint32_t)M, p)) return false;
    out[0] = p.slices;
    out[1] = p.fa.RB;
    out[2] = p.fa.KW;
    out[3] = (N + p.fa.RB * 16 - 1) / (p.fa.RB * 16) * p.slices;
    return true;
}

}  // namespace xfp
