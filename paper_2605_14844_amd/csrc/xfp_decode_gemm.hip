// Prompt form of the fused decode: any number of tokens against one matrix (V2 codebooks or a V2a library, 2 to 4
// bits), as a tiled matrix product on the matrix cores whose weight operand is dequantised on the way.
//
// Why: with hundreds of tokens the product is bound by arithmetic (28672 x 8192 with 2048 tokens: 0.96 TFLOP; the matrix
// cores and the VALU, which dequantises, each busy for half of the clocks), not by the weights' bytes, and the 64-token
// kernel reads and dequantises the whole matrix once per 64 tokens and fetches its activations from L2 once per 32 rows.
//
// Work unit: a workgroup of 8 or 16 waves owns BN output rows x BM tokens and walks K; a row's sum is taken in two or
// three steps (GemmTile).
//  - Every lane dequantises the weights it needs itself, straight into the A operand of v_mfma_f32_32x32x16_f16: lane
//    (i, h) owns row i of a block of 32 rows and one half of every 64 columns, the same rows for the whole kernel, so
//    a V2 row's codebook stays in registers, split into byte planes (low and high bytes of the fp16 entries):
//    v_perm_b32 then looks four entries up per instruction, with no LDS table, no bank conflict and no address (1.5,
//    1.8 and 2.9 VALU operations per weight at 2, 3 and 4 bits).  V2a: the planes of the group's library entry are
//    read from LDS once per block.  (An A tile in LDS, filled by all waves, was measured slower: ds_write_b128 takes
//    14 to 16 clocks per KB, against 4.5 for a read, and LDS bandwidth is what runs out next to the matrix cores.)
//  - The B tile (BM tokens) comes from a token-major copy of the activations straight into LDS
//    (buffer_load_dwordx4 ... lds: no registers, no VALU), through a ring of parts; its rows are XOR-swizzled in
//    16-byte chunks so that 16 consecutive lanes of a ds_read_b128 cover the 64 banks.
//  - 28672 x 8192, 4 bits, 2048 tokens: 1.17 ms (the library's own dense product of this shape 0.71 ms).  4096 x 4096, 2 bits, 333
//    tokens: 30 us against 90 in passes of 64.
//
// Order of k inside 32 weights: what the byte planes give cheaply is not the natural order (at 4 bits the even
// nibbles of a dword come before the odd ones).  A product does not care as long as both operands agree, so the copy
// of the activations is written in that order (slot_k), and by steps inside 64 columns.
//
// Outliers (fp32, not folded into the fp16 operand: that would round them): the waves share out the tile's rows; an
// entry's activations of all the tile's tokens are one contiguous read from a k-major copy of x; a row's sums meet in
// an LDS plane, which is added to the finished sums of the product.  No atomics, fixed orders.
#include "xfp_dequant.h"

#include <atomic>
#include <type_traits>
#include <utility>

namespace xfp {
namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4_t lds_u4_t;
typedef __attribute__((address_space(3))) const u32x4_t lds_cu4_t;
typedef __attribute__((address_space(3))) const half8_t lds_ch8_t;
typedef __attribute__((address_space(3))) const float lds_cf32_t;
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const u32x2_t lds_cu2_t;
typedef __attribute__((address_space(3))) const uint8_t lds_cu8_t;
typedef __attribute__((address_space(3))) float4_t lds_f4_t;
typedef __attribute__((address_space(4))) const int32_t const_i32_t;   // uniform reads go through the scalar cache

// Tile geometry: WN x WK waves; a wave owns 32 RB rows and all 32 TB tokens and takes every WK-th block of 256 columns
// (the waves that share rows add their sums in LDS at the end), a block in four turns of 64.  A part of the B tile is SP
// of a turn's four steps of 16 columns, for each of the WK waves; NBUF of them in LDS, NBUF - 1 requested ahead.
// Every block is a chain of its own, whose sums are added to a second set of registers: what one fp32 chain through all
// of a row's products of 16 loses grows with the root of its length (4096 columns: 3.1e-7 of the result, 1.2e-7 in two
// steps).  The second set halves the tokens that a dequantised weight meets in a wave (28672 x 8192, 2048 tokens, fp16:
// 256 x 256 tiles in one chain were 13 % faster than 256 x 128 in two steps).
template <int RB_, int TB_, int WN_, int WK_, int SP_, int NBUF_, int IBUF_, bool PLAIN_ = false>
struct GemmTile {
    static constexpr int RB = RB_, TB = TB_, WN = WN_, WK = WK_, SP = SP_, NBUF = NBUF_, IBUF = IBUF_;
    static constexpr int BN = 32 * RB * WN, BM = 32 * TB, NW = WN * WK, T = NW * kWave;
    static constexpr int KB = 16 * SP * WK, RSB = KB * 2, kB = BM * RSB;   // a part: columns, bytes of a row, bytes
    static constexpr int U = 4 / SP;                           // parts of a turn
    static_assert(SP == 2 || SP == 4, "");
    static constexpr int AHEAD = NBUF - 1;
    static constexpr int ND = kB / (NW * 1024);                // loads of a wave per part
    // LDS: the B tiles, then the index words (IBUF blocks of every wave); the outliers' plane or the waves' sums in the
    // same place later; then a V2a library and its ids
    static constexpr int kPlane = BN * BM * 4, kSums = (WK - 1) * BN * BM * 4, kTiles = NBUF * kB;
    template <int BITS> static constexpr int kWordBlock = RB * 1024 * BITS;            // bytes of a wave's block of index words
    template <int BITS> static constexpr int kLoop = kTiles + NW * IBUF * kWordBlock<BITS>;
    template <int BITS> static constexpr int kBase = kPlane > kSums ? (kLoop<BITS> > kPlane ? kLoop<BITS> : kPlane) : (kLoop<BITS> > kSums ? kLoop<BITS> : kSums);
    static constexpr int kIds = BN * 64;                       // ids of 64 groups
    // A step's VALU work is dealt out between its matrix instructions, which 64 columns of tokens need (4096 x 4096, 333 tokens, 3
    // bits 37 us in the compiler's order, 34).  With 128 both orders take the same clocks (28672 x 8192, 4 bits, 2048 tokens 1.69 M,
    // 1.67 M dealt out, 1081 / 1073 us without outliers) or the compiler's fewer (2 bits 878 / 931 us; 11008 x 4096, 2 bits, 700 tokens
    // 142 and 152 thousand, 120.5 / 125.6 us).
    // PLAIN: in the compiler's order all the same, with nothing asked for ahead (rows of a block or two: see kPlainTinyK).
    static constexpr bool DEAL = TB <= 2 && !PLAIN_;
    static constexpr bool EARLY = NW <= 8 && DEAL;             // there are registers for what is asked for ahead of its use
    static constexpr bool FINE = NW <= 8;                      // takes short rows (half blocks as chains)
    // A third set of sums for long rows: tiles of 32 tokens are taken for 17 and more, whose copies hold rows of up to 16384 columns.
    static constexpr bool DEEP = WK > 1 && NW <= 8 && TB > 1 && !PLAIN_;
    static_assert(kB % (NW * 1024) == 0 && AHEAD >= 1 && BN % NW == 0, "");
    // registers: accumulators and sums, operands (B twice), index words, planes; then waves per SIMD
    static constexpr int kRegs = (WK > 1 && NW <= 8 ? 48 : 32) * RB * TB + 16 * RB + 8 * TB + 4 * RB + 8 * RB + 56;
    static constexpr int kWavesPerSimd = kRegs <= 128 ? 4 : kRegs <= 168 ? 3 : kRegs <= 256 ? 2 : 1;
};

// Half a block is a chain where waves share their rows (their sums take few registers) and up to kFineK columns; above kDeepK
// eight waves or fewer take their sums in three steps (the third: every eighth block).  Error against 64 bits, 1e-8 of the
// result's norm, this kernel / passes of 64 tokens: 1024 rows, 512 columns 8.5 / 8.6; 1536 9.5 / 11.3; 4096 10.4 / 15.6; 8192
// 11.6 / 21.1; 28672 12.2 / 14.2; 8320 rows, 8192 columns 14.9 / 21.1.
constexpr uint32_t kFineK = 2048, kDeepK = 16384;

// Rows of a block or two for each of the waves that share them: a step dealt out between its matrix instructions stands behind each
// barrier with one instruction less to cover its reads, and asking ahead is only more to wait for.  us in the order above / plain:
// 64 x 64 tiles, 3 bits, 143 x 256, 150 tokens 12.2 / 11.7, 212 x 512, 92 12.2 / 11.7, but 300 x 1024, 200 12.7 / 13.1, 4096 columns
// 21.3 / 22.8; 4 bits, 300 x 512, 200 12.4 / 12.4; of 862 drawn calls of up to 2048 columns two are more than 2 % slower than with
// plain tiles alone (201 before; 2.8 % at most, 640 and 768 columns), the median 2 % faster.  128 x 64: 21235 x 128, 98 tokens 26.7 / 26.2,
// at 384 columns the same.
constexpr uint32_t kPlainTinyK = 512, kPlainSmallK = 256;

// 16-byte chunk c of row r of a tile with C chunks per row sits at position c ^ swz<C>(r)
template <int C>
__device__ __forceinline__ uint32_t swz(uint32_t r)
{
    if constexpr (C >= 16) return r & 15u;
    else return (r / (16 / C)) & (uint32_t)(C - 1);
}

constexpr uint64_t kCopyHalves = (uint64_t)kXtMaxK * kXtTokens;        // of a workspace's copies

struct GemmArgs {
    DecodeArgs a;
    const uint16_t *xp;    // [M][K rounded up to 256] fp16, every block of 256 columns in the order of the kernel's steps
    const uint16_t *xt;    // [K][MP] fp16
    uint32_t M, MP;        // tokens of this launch; row length of xt (a multiple of 8)
    uint32_t row0, tiles_n, tiles_m;                           // first row, tiles of this launch
    int y_f32;
    int fine;              // half blocks are chains of their own
    int deep;              // a third set of sums
};

template <class F, int... Is>
__device__ __forceinline__ void for_each_of(F &&f, std::integer_sequence<int, Is...>) { (f(std::integral_constant<int, Is>{}), ...); }
// f(0), .., f(n - 1) with compile-time arguments
template <int n, class F>
__device__ __forceinline__ void for_each(F &&f) { for_each_of(f, std::make_integer_sequence<int, n>{}); }

template <int BITS, int MODE, class C>
__device__ __forceinline__ void tile_product(const GemmArgs &ga)
{
    static_assert(MODE == 0 || MODE == 1, "V2, V2a");
    constexpr int BN = C::BN, BM = C::BM, RB = C::RB, TB = C::TB, WK = C::WK, NW = C::NW;
    constexpr int CB = C::KB / 8;                              // 16-byte chunks of a row of a part
    constexpr bool DEAL = C::DEAL, EARLY = C::EARLY;
    extern __shared__ __align__(256) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const DecodeArgs &a = ga.a;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t i = lane & 31, h = lane >> 5;
    const uint32_t wn = wave % C::WN, wk = wave / C::WN;
    const uint32_t N = a.N, K = a.K, M = ga.M;
    const uint32_t wpr = K / 32 * BITS, G = K / kGroup;
    const uint32_t NB = (K + 255) / 256, NS = (NB + WK - 1) / WK;          // blocks of a row; of a wave

    // Workgroups are dealt to the 8 XCDs round-robin, each with an L2 of its own: an XCD takes a contiguous run of
    // tiles, row tiles fastest, so that its workgroups share the activations of one token tile (2 x 4 MB at 8192
    // columns), which every one of them reads whole and, for the outliers, at random.
    const uint32_t nt = ga.tiles_n * ga.tiles_m, per = (nt + 7) / 8;
    const uint32_t t0 = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (t0 >= nt || blockIdx.x / 8 >= per) return;
    const uint32_t n0 = ga.row0 + t0 % ga.tiles_n * BN, m0 = t0 / ga.tiles_n * BM;

    // ---------------------------------------------------------------- A operands: this lane's rows
    // Lane (i, h) dequantises, of row i of every row block, one half (a group of 128 weights) of a block: 64, 48 or 32
    // bytes.  In turn p it makes the A operands of 32 weights, chunk s of them being step s's: nothing moves between lanes
    // and there is no A tile.  The copy of the activations has chunk s of turn p of half h at the block's 16 bytes 8 p + 2 s + h.
    // The index words come by loads straight into LDS, whole lines at a time, a block of 32 rows x 256 columns per wave, IBUF - 1
    // blocks ahead; only this wave reads them.  (As loads into registers their first use waited for every load under way, those
    // of the B tiles included, once per block: 28672 x 8192, 64 tokens 70 us as a product.)
    uint32_t row[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) row[rb] = min(n0 + (wn * RB + rb) * 32 + i, N - 1);
    Planes<BITS> P[RB];
    if constexpr (MODE == 0) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            uint32_t c[1 << (BITS - 1)];
            const uint32_t *cb = reinterpret_cast<const uint32_t *>(a.cb) + (size_t)row[rb] * (1 << (BITS - 1));
#pragma unroll
            for (int d = 0; d < (1 << (BITS - 1)); ++d) c[d] = cb[d];
            P[rb].set(c);
        }
    } else {
        // the library as planes: entry l at kBase + l * 2^BITS * 2, low bytes first; entry L: zeros
        for (uint32_t j = tid; j < (a.L + 1) * Planes<BITS>::ND; j += C::T) {
            const uint32_t l = j / Planes<BITS>::ND, d = j % Planes<BITS>::ND;
            const uint2 v = l < a.L ? *reinterpret_cast<const uint2 *>(a.cb + ((size_t)l << BITS) + 4 * d) : make_uint2(0u, 0u);
            const uint32_t o = lds0 + C::template kBase<BITS> + l * (2u << BITS) + d * 4;
            *(lds_u32_t *)(uintptr_t)o = __builtin_amdgcn_perm(v.y, v.x, 0x06040200u);
            *(lds_u32_t *)(uintptr_t)(o + Planes<BITS>::ND * 4) = __builtin_amdgcn_perm(v.y, v.x, 0x07050301u);
        }
    }

    float16_t acc[RB][TB], sum[RB][TB];                        // a block's chains; what becomes the results
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) sum[rb][tb] = float16_t{};
    float16_t deep[C::DEEP ? RB : 1][C::DEEP ? TB : 1];
#pragma unroll
    for (int rb = 0; rb < (C::DEEP ? RB : 1); ++rb)
#pragma unroll
        for (int tb = 0; tb < (C::DEEP ? TB : 1); ++tb) deep[rb][tb] = float16_t{};

    // ---------------------------------------------------------------- loads of the main loop
    // All of them go to LDS (load_to_lds) and nothing but the waits below waits for them.  Every block issues the same number
    // of loads in the same order (past the end: again the last block's), and every wait states how many may still be under way.
    const uint32_t rows = min(N - n0, (uint32_t)BN);
    const uint64_t base = (uint64_t)(uintptr_t)(a.idx + (size_t)n0 * wpr);
    const u32x4_t ri = {(uint32_t)base, (uint32_t)(base >> 32) & 0xFFFFu, rows * wpr * 4, 0x00020000u};
    // A row's 32 BITS bytes of a block are CPR chunks of 16.  With 8 or 4 of them a chunk's place is turned by the row, so that
    // the 16 lanes that read one chunk of 16 rows find them in different banks.
    constexpr uint32_t CPR = 2 * BITS;
    auto turned = [](uint32_t c, uint32_t r) -> uint32_t { return BITS == 4 ? c ^ (r >> 1 & 7u) : BITS == 2 ? c ^ (r >> 2 & 3u) : c; };
    uint32_t woff[BITS];
#pragma unroll
    for (int e = 0; e < BITS; ++e) {
        const uint32_t id = e * 64 + lane, r = id / CPR;
        woff[e] = (wn * RB * 32 + r) * (wpr * 4) + turned(id % CPR, r) * 16;
    }
    const uint32_t ring = lds0 + C::kTiles + wave * (C::IBUF * C::template kWordBlock<BITS>);
    uint32_t wload = 0;                                        // slot of the block being requested
    auto load_words = [&](uint32_t t) {                        // the wave's t-th block
        const uint32_t so = min(t * WK + wk, NB - 1) * (32 * BITS);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int e = 0; e < BITS; ++e)
                load_to_lds(ring + wload * C::template kWordBlock<BITS> + (rb * BITS + e) * 1024, woff[e] + so + rb * 32 * (wpr * 4), ri, 0);
        wload = wload + 1 == C::IBUF ? 0 : wload + 1;
    };
    constexpr int kWords = RB * BITS;                          // loads of a block's words
    static_assert((C::AHEAD - 1) * C::ND + kWords <= 63, "what vmcnt can say");
    // V2a: the ids of 64 groups of the tile's rows in LDS
    const uint32_t ids = lds0 + C::template kBase<BITS> + (MODE == 1 ? ((a.L + 1) * (2u << BITS) + 15) / 16 * 16 : 0u);
    auto load_ids = [&](uint32_t g0) {
        const uint8_t *src = a.gid + (size_t)n0 * G;
        for (uint32_t j = tid; j < rows * 16; j += C::T) {
            const uint32_t r = j / 16, g = g0 + j % 16 * 4;
            uint32_t v = 0;
            if (g + 3 < G) __builtin_memcpy(&v, src + (size_t)r * G + g, 4);
            else
#pragma unroll
                for (uint32_t b = 0; b < 4; ++b) v |= (g + b < G ? (uint32_t)src[(size_t)r * G + g + b] : 0u) << (8 * b);
            *(lds_u32_t *)(uintptr_t)(ids + j * 4) = v;
        }
    };
    const u32x4_t rx = {(uint32_t)(uintptr_t)ga.xp, (uint32_t)((uintptr_t)ga.xp >> 32) & 0xFFFFu, M * (NB * 512), 0x00020000u};
    uint32_t boff[C::ND];
#pragma unroll
    for (int e = 0; e < C::ND; ++e) {
        const uint32_t o = (wave * C::ND + e) * 1024 + lane * 16, r = o / C::RSB, p = (o % C::RSB / 16) ^ swz<CB>(r);
        boff[e] = min(m0 + r, M - 1) * (NB * 512) + p / (2 * C::SP) * 512 + p % (2 * C::SP) * 16;
    }
    uint32_t bload = 0;                                        // ring slot of the part being requested
    // Loads e0 .. e1 - 1 of a part.  They are spread over the steps: a wave that issues a part's loads at once stands in
    // front of its matrix instructions until the address unit has taken them all.
    auto load_b = [&](uint32_t q, int e0, int e1) {
        const uint32_t dst = lds0 + bload * C::kB + wave * (C::ND * 1024), x = min(q, 4 * C::U * NS - 1),
                       so = x / (4 * C::U) * (WK * 512) + x % (4 * C::U) * (C::SP * 32);
#pragma unroll
        for (int e = e0; e < e1; ++e)
            load_to_lds(dst + e * 1024, boff[e], rx, so);
        if (e1 == C::ND) bload = bload + 1 == C::NBUF ? 0 : bload + 1;
    };
    words_t<BITS> cw[RB], cn[RB];                              // the words of the turn whose A operands are being made; of the next
    uint32_t wcur = 0;                                         // slot of the block that cn is of
    uint32_t at_book[RB];                                      // V2a: where the codebooks of the wave's next block lie
    auto find_books = [&](uint32_t t) {                        // of the wave's t-th block
        if constexpr (MODE == 1) {
            const bool dead = 2 * (t * WK + wk) + h >= G;      // second half of the last block of a row with an odd number of groups
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const uint32_t id = *(lds_cu8_t *)(uintptr_t)(ids + (row[rb] - n0) * 64 + ((2 * (t * WK + wk) + h) & 63u));
                at_book[rb] = lds0 + C::template kBase<BITS> + (dead ? a.L : id) * (2u << BITS);
            }
        }
    };
    Planes<BITS> Pn[MODE == 1 ? RB : 1];
    auto read_books = [&] {
        if constexpr (MODE == 1) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if constexpr (BITS == 2) {
                    const u32x2_t v = *(lds_cu2_t *)(uintptr_t)at_book[rb];
                    Pn[rb].lo[0] = v[0]; Pn[rb].hi[0] = v[1];
                } else {
                    uint32_t v[2 * Planes<BITS>::ND];
#pragma unroll
                    for (int d = 0; d < Planes<BITS>::ND / 2; ++d) {
                        const u32x4_t q = *(lds_cu4_t *)(uintptr_t)(at_book[rb] + d * 16);
                        v[4 * d] = q[0]; v[4 * d + 1] = q[1]; v[4 * d + 2] = q[2]; v[4 * d + 3] = q[3];
                    }
#pragma unroll
                    for (int d = 0; d < Planes<BITS>::ND; ++d) { Pn[rb].lo[d] = v[d]; Pn[rb].hi[d] = v[Planes<BITS>::ND + d]; }
                }
            }
        }
    };
    auto next_books = [&](uint32_t t) {                        // from here on the A operands are the t-th block's
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if constexpr (MODE == 1) P[rb] = Pn[rb];
            else if (2 * (t * WK + wk) + h >= G)               // (such a block is the wave's last)
#pragma unroll
                for (int d = 0; d < Planes<BITS>::ND; ++d) P[rb].lo[d] = P[rb].hi[d] = 0u;
        }
    };
    auto read_words = [&](int p) {                             // turn p's words, as they are
        const uint32_t o = ring + wcur * C::template kWordBlock<BITS> + i * (32 * BITS);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const uint32_t w = o + rb * (1024 * BITS);
            if constexpr (BITS == 4) cn[rb] = *(lds_cu4_t *)(uintptr_t)(w + turned(4 * h + p, i) * 16);
            else if constexpr (BITS == 3) {
#pragma unroll
                for (int d = 0; d < 3; ++d) cn[rb][d] = *(lds_cu32_t *)(uintptr_t)(w + h * 48 + p * 12 + d * 4);
            } else cn[rb] = *(lds_cu2_t *)(uintptr_t)(w + turned(2 * h + p / 2, i) * 16 + p % 2 * 8);
        }
    };
    auto next_words = [&] {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            cw[rb] = cn[rb];
            arrange<BITS>(cw[rb]);
        }
    };

    // The outliers of the tile's rows (the term itself comes last): the rows' first entries and the first batch's entries are asked
    // for in front of the main loop, in vector loads: a scalar one is waited for with the next of any kind, a round trip to memory in front of
    // all other loads (4263 x 384, 145 tokens without outliers 13.1 / 12.6 us).
    constexpr int GL = BM / 8, RP = 64 / GL, RW = BN / NW;     // lanes of a row; rows of a wave at a time, in all
    static_assert((GL == 4 || GL == 8 || GL == 16) && RW % RP == 0 && RW < 62, "");
    const_i32_t *rp = (const_i32_t *)(uintptr_t)a.rp;
    int32_t ofirst = 0, olast = 0;
    auto tile_entries = [&] {
        ofirst = rp[min(n0, N)];
        olast = rp[min(n0 + BN, N)];
    };
    const uint32_t oo = lane % GL, orow = lane / GL;
    int32_t rpv = 0;                                           // lane r: first entry of row r; early: lanes 62 and 63: of the tile, of the next
    auto first_of = [&](uint32_t r) { return __builtin_amdgcn_ds_bpermute((int)(min(r, (uint32_t)RW) * 4), rpv); };
    int32_t oe = 0, oend = 0;                                  // this lane's row: first entry of the batch, end of the row
    uint32_t oc = 0, ov = 0;
    auto entries = [&] {                                       // (past the tile's entries: zeros)
        const int32_t n = a.col ? olast - ofirst : 0;
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc((void *)(a.col + ofirst), 0, n * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void *)(a.val + ofirst), 0, n * 2, 0x00020000);
        oc = __builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)(oe + (int32_t)oo - ofirst) * 4, 0, 0);
        ov = __builtin_amdgcn_raw_buffer_load_b16(rv, (uint32_t)(oe + (int32_t)oo - ofirst) * 2, 0, 0);
    };

    auto first_entries = [&] {
        if constexpr (EARLY) {
            ofirst = __builtin_amdgcn_readlane(rpv, 62);
            olast = __builtin_amdgcn_readlane(rpv, 63);
        } else rpv = a.rp[min(n0 + wave * RW + min(lane, (uint32_t)RW), N)];
        oe = first_of(orow);
        oend = first_of(orow + 1);
        entries();
    };

    // ---------------------------------------------------------------- prologue: as if the turns before the first had run
    u32x4_t af[4][RB];
    half8_t bf[2][TB];
    auto dequantise = [&](int s, int part) {                   // half of a step's A operand
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            uint32_t d0, d1;
            chunk_half<BITS>(P[rb], cw[rb], s, part, d0, d1);
            if constexpr (EARLY) asm volatile("" : "+v"(d0), "+v"(d1));     // (here and not in front of its use)
            af[s][rb][2 * part] = d0;
            af[s][rb][2 * part + 1] = d1;
        }
    };
    const uint32_t br = lds0 + i * C::RSB + (((wk * (2 * C::SP) + h) ^ swz<CB>(i)) * 16);
    auto operands = [&](int set, uint32_t buf, int s) {
        const uint32_t ba = (br + buf * C::kB) ^ (uint32_t)(s % C::SP * 32);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) bf[set][tb] = *(lds_ch8_t *)(uintptr_t)(ba + tb * (32 * C::RSB));
    };
    if constexpr (EARLY) rpv = a.rp[min(lane < 62 ? n0 + wave * RW + min(lane, (uint32_t)RW) : n0 + (lane - 62) * BN, N)];
#pragma unroll
    for (int b = 0; b < C::IBUF - 1; ++b) load_words(b);
#pragma unroll
    for (int q = 0; q < C::AHEAD; ++q) load_b(q, 0, C::ND);
    if constexpr (MODE == 1) load_ids(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if constexpr (EARLY) first_entries();                   // (older than every load that is waited for below)
    find_books(0);
    read_books();
    next_books(0);
    read_words(0);
    next_words();
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        dequantise(s, 0);
        dequantise(s, 1);
    }
    operands(0, 0, 0);

    // ---------------------------------------------------------------- main loop
    // A block is four turns of four steps.  In step s the B operands of step s + 1 are read, the A operands of the next
    // turn's step s - 1 are made (their registers were read by the step before) and the matrix instructions run, with the
    // other work of the step dealt out between them: an instruction of 32 x 32 x 16 keeps the matrix core for 32 clocks, in
    // which a wave's VALU instructions run, but one that follows it at once only waits, and so does the other wave of the SIMD,
    // which the barriers keep in step (figures: GemmTile::DEAL).  The barrier that opens the next part stands behind the first matrix instruction of a
    // part's last step; the loads that refill a ring slot follow the barrier behind its last reads.
    uint32_t bcur = 0;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[rb][tb] = float16_t{};
    auto add = [&] {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) sum[rb][tb] += acc[rb][tb];
    };
    auto fold = [&] {                                          // the sums so far into the third set
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) {
                deep[rb][tb] += sum[rb][tb];
                sum[rb][tb] = float16_t{};
            }
    };
    auto wait_part = [&](auto part) {
        // The part behind part x of a block, requested AHEAD parts ago.  Younger: the parts requested since, and a block's words if
        // they have been since its last load (they come in the second step of a block).
        constexpr int x = decltype(part)::value, from = x + 1 - C::AHEAD + (C::SP == 4 ? 1 : 0);           // first part whose words are younger
        constexpr bool words = from <= 0 || (from > x ? false : from % (4 * C::U) == 0);
        constexpr int kYounger = (C::AHEAD - 1) * C::ND + (words && from <= x ? kWords : 0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(kYounger) : "memory");
    };
    // In the compiler's order.
    auto compiled_block = [&](uint32_t t) {
        const bool on = WK == 1 || t * WK + wk < NB;           // (the last round of a row may have no block for this wave)
        for_each<16>([&](auto step) {
            constexpr int p = decltype(step)::value / 4, s = decltype(step)::value % 4;
            constexpr int x = p * C::U + s / C::SP;
            constexpr bool last = s % C::SP == C::SP - 1;
            const uint32_t bnext = bcur + 1 == C::NBUF ? 0 : bcur + 1;
            constexpr int set = s & 1;
            if constexpr (C::FINE && p == 2 && s == 0)
                if (ga.fine && on) {
                    add();
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int tb = 0; tb < TB; ++tb) acc[rb][tb] = float16_t{};
                }
            load_b(t * (4 * C::U) + x + C::AHEAD, s % C::SP * C::ND / C::SP, (s % C::SP + 1) * C::ND / C::SP);
            if constexpr (!last) operands(set ^ 1, bcur, s + 1);
            if constexpr (s == 0) {
                dequantise(3, 0);
                dequantise(3, 1);
            }
            if constexpr (s == 1) {
                if constexpr (p == 0) load_words(t + C::IBUF - 1);
                if constexpr (p == 3) {
                    wcur = wcur + 1 == C::IBUF ? 0 : wcur + 1;
                    find_books(t + 1);
                    read_books();
                    next_books(t + 1);
                }
                read_words((p + 1) % 4);
                next_words();
            }
            if constexpr (MODE == 1 && p == 1 && s == 0)
                if ((t + 1) * (2 * WK) % 64 == 0 && t + 1 < NS) load_ids((t + 1) * (2 * WK));
            if constexpr (last) {
                wait_part(std::integral_constant<int, x>{});
                operands(set ^ 1, bnext, (s + 1) % 4);
            }
            if constexpr (s > 0) {
                dequantise(s - 1, 0);
                dequantise(s - 1, 1);
            }
            if (on)
#pragma unroll
                for (int tb = 0; tb < TB; ++tb)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        acc[rb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, af[s][rb]), bf[set][tb], p + s == 0 ? float16_t{} : acc[rb][tb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (last) bcur = bnext;
        });
        if (on) add();
    };
    // MAYBE: the wave may have no such block (the last round of a row)
    auto block = [&](auto maybe, uint32_t t) {
        const bool on = !decltype(maybe)::value || t * WK + wk < NB;
        for_each<16>([&](auto step) {
            constexpr int p = decltype(step)::value / 4, s = decltype(step)::value % 4;        // turn, step in it
            constexpr int x = p * C::U + s / C::SP;            // part of the block
            constexpr bool last = s % C::SP == C::SP - 1;      // of the part
            const uint32_t bnext = bcur + 1 == C::NBUF ? 0 : bcur + 1;
            constexpr int set = s & 1;                         // where the step's operands are
            constexpr bool fresh = p + s == 0 || (C::FINE && p == 2 && s == 0);            // half blocks are chains of their own
            load_b(t * (4 * C::U) + x + C::AHEAD, s % C::SP * C::ND / C::SP, (s % C::SP + 1) * C::ND / C::SP);
            if constexpr (!last) operands(set ^ 1, bcur, s + 1);
            // the next turn's words and its books (older than the part that the last wait was for)
            if constexpr (p == 2 && s == 2 && EARLY) find_books(t + 1);
            if constexpr (s == (EARLY ? 0 : 1)) {
                if constexpr (p == 3) {
                    wcur = wcur + 1 == C::IBUF ? 0 : wcur + 1;
                    if constexpr (!EARLY) find_books(t + 1);
                    read_books();
                }
                read_words((p + 1) % 4);
            }
            if constexpr (p == 0 && s == 1) load_words(t + C::IBUF - 1);
            // the ids of the next 64 groups, behind the barrier that every wave passes after its last use of the old ones; another
            // barrier follows before their first use
            if constexpr (MODE == 1 && p == 1 && s == 0)
                if ((t + 1) * (2 * WK) % 64 == 0 && t + 1 < NS) load_ids((t + 1) * (2 * WK));
            for_each<TB>([&](auto token_block) {
                constexpr int tb = decltype(token_block)::value;
                if constexpr (fresh)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        asm volatile("" : "+v"(acc[rb][tb]));          // (the additions stay here)
                        sum[rb][tb] += acc[rb][tb];
                        acc[rb][tb] = float16_t{};
                        asm volatile("" : "+v"(sum[rb][tb]));
                    }
                if (on)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        acc[rb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, af[s][rb]), bf[set][tb], acc[rb][tb], 0, 0, 0);
                if constexpr (s == 1 && tb == 0) {
                    if constexpr (p == 3) next_books(t + 1);
                    next_words();
                }
                dequantise((s + 3) % 4, tb);
                if constexpr (TB == 1) dequantise((s + 3) % 4, 1);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (last && tb == 0) {
                    wait_part(std::integral_constant<int, x>{});
                    operands(set ^ 1, bnext, (s + 1) % 4);
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            if constexpr (C::DEEP && p + s == 0)
                if (ga.deep && t && t % 8 == 0) fold();
            if constexpr (last) bcur = bnext;
        });
    };
#pragma unroll 1
    for (uint32_t t = 0; t + (WK > 1 && DEAL) < NS; ++t)
        if constexpr (DEAL) block(std::false_type{}, t);
        else compiled_block(t);
    if constexpr (WK > 1 && DEAL) block(std::true_type{}, NS - 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // (loads to LDS that nobody waits for)
    if constexpr (DEAL) add();
    if constexpr (C::DEEP)
        if (ga.deep) {
            fold();
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) sum[rb][tb] = deep[rb][tb];
        }

    if constexpr (WK > 1) {
        // the other waves' sums of a block, added in their order; they may overwrite the tiles, which every wave has read
        lds_barrier();
        constexpr uint32_t kWave4 = kWave * 16, kBlock = RB * TB * 4 * kWave4;               // four registers of a wave; a wave's block
        const uint32_t at = lds0 + wn * kBlock + lane * 16;
        if (wk > 0) {
#pragma unroll
            for (int b = 0; b < RB * TB * 4; ++b) {
                const float16_t &v = sum[b / 4 % RB][b / 4 / RB];
                *(lds_f4_t *)(uintptr_t)(at + (wk - 1) * (C::WN * kBlock) + b * kWave4) =
                    float4_t{v[b % 4 * 4], v[b % 4 * 4 + 1], v[b % 4 * 4 + 2], v[b % 4 * 4 + 3]};
            }
        }
        lds_barrier();
        if (wk == 0)
#pragma unroll 1
        for (int w = 0; w < WK - 1; ++w)
#pragma unroll
            for (int b = 0; b < RB * TB * 4; ++b) {
                const float4_t x = *(lds_f4_t *)(uintptr_t)(at + w * (C::WN * kBlock) + b * kWave4);
                float16_t &v = sum[b / 4 % RB][b / 4 / RB];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[b % 4 * 4 + r] += x[r];
            }
    }

    // ---------------------------------------------------------------- the outlier term
    // Behind the product and not in front of it: the sums would otherwise be added to a term that is often larger than all
    // of theirs, and be rounded at its size (28672 columns, 0.3 % outliers: 2.0e-7 of the result instead of 1.0e-7).
    // Wave w owns rows RW w .. of the plane and takes RP of them at a time, GL = BM / 8 lanes each: lane o of a row sums the
    // tokens m0 + 8 o .. + 7 over the row's entries, whose activations are one contiguous read of 2 BM bytes.  Nothing is
    // added across lanes.  (With the lanes of a row's token dealt over its entries, every row paid a reduction and the walk
    // from row to row: 28672 x 8192, 2048 tokens 309 us of 1366 at 0.3 % outliers, 165 at 0.05 %; 4096 x 1024, 256 tokens 6.)
    // A row's entries are fetched GL at a time, one per lane, and handed to its lanes one by one (row_newbcast); a sum is
    // taken per GL entries and those are added up.
    if constexpr (!EARLY) tile_entries();
    if (a.col && ofirst < olast) {
        if constexpr (!EARLY) first_entries();
        lds_barrier();                                         // every wave is past its tiles (and sums)
        const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc((void *)ga.xt, 0, K * ga.MP * 2, 0x00020000);
        const uint32_t octet = min(m0 + 8 * oo, ga.MP - 8) * 2, plane = lds0 + wave * (RW * BM * 4) + orow * (BM * 4) + oo * 32;
        // lane k of every row's lanes to all of them
        auto deal = [&](auto k, uint32_t v) -> uint32_t {
            constexpr int kk = decltype(k)::value;
            if constexpr (GL == 4) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kk * 0x55, 0xf, 0xf, true);
            else if constexpr (GL == 16) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + kk, 0xf, 0xf, true);
            else
                return (uint32_t)__builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + kk, 0xf, 0xf, true),
                                                             (int)v, 0x158 + kk, 0xf, 0xc, false);
        };
        // A batch: GL entries of each of RP rows.  begin() asks for the next batch's entries, then for this one's activations;
        // finish() adds them.
        struct Batch {
            int32_t at, to;                                    // its first entry, the end of the row
            bool more;                                         // of any of the rows
            uint32_t row, val;
        };
        uint32_t r0 = 0;
        auto begin = [&](Batch &b, u32x4_t (&x)[GL]) {
            asm volatile("" : "+v"(oc), "+v"(ov));             // (waited for here, whatever the lane has)
            // an entry that is not there: a place past the copy, which reads as zeros, times zero
            const bool have = oe + (int32_t)oo < oend;
            const uint32_t off = have ? __umul24(oc, ga.MP * 2) : 0x80000000u;
            b.val = __builtin_bit_cast(uint32_t, half_bits_to_float((uint16_t)(have ? ov : 0u)));
            b.at = oe;
            b.to = oend;
            b.more = __builtin_amdgcn_ballot_w64(oe + GL < oend) != 0;
            b.row = r0;
            if (b.more) oe += GL;
            else {
                r0 += RP;
                oe = first_of(r0 + orow);
                oend = first_of(r0 + orow + 1);
            }
            entries();
            // (only the fours that some row has: all of them in any case, for the sake of the waits, is slower where rows have few
            // entries, 30636 x 128, 123 tokens 22.8 / 22.1 us, and no faster elsewhere, 4096 x 4096, 4 bits, 333 tokens 34.7 / 34.3)
            for_each<GL / 4>([&](auto q) {
                constexpr int k0 = 4 * decltype(q)::value;
                if (__builtin_amdgcn_ballot_w64(b.at + k0 < b.to))
                    for_each<4>([&](auto k) {
                        constexpr int kk = k0 + decltype(k)::value;
                        x[kk] = __builtin_amdgcn_raw_buffer_load_b128(rt, deal(std::integral_constant<int, kk>{}, off) + octet, 0, 0);
                    });
            });
        };
        float total[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        auto finish = [&](const Batch &b, const u32x4_t (&x)[GL]) {
            float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            for_each<GL / 4>([&](auto q) {
                constexpr int k0 = 4 * decltype(q)::value;
                if (__builtin_amdgcn_ballot_w64(b.at + k0 < b.to))
                    for_each<4>([&](auto k) {
                        constexpr int kk = k0 + decltype(k)::value;
                        const float w = __builtin_bit_cast(float, deal(std::integral_constant<int, kk>{}, b.val));
#pragma unroll
                        for (int t = 0; t < 8; ++t)
                            s[t] = fmaf(w, half_bits_to_float((uint16_t)(t & 1 ? x[kk][t / 2] >> 16 : x[kk][t / 2])), s[t]);
                    });
            });
#pragma unroll
            for (int t = 0; t < 8; ++t) total[t] += s[t];
            if (b.more) return;
            *(lds_f4_t *)(uintptr_t)(plane + b.row * (BM * 4)) = float4_t{total[0], total[1], total[2], total[3]};
            *(lds_f4_t *)(uintptr_t)(plane + b.row * (BM * 4) + 16) = float4_t{total[4], total[5], total[6], total[7]};
#pragma unroll
            for (int t = 0; t < 8; ++t) total[t] = 0.f;
        };
        auto last = [&](const Batch &b) { return !b.more && r0 >= (uint32_t)RW; };
        if constexpr (GL <= 8 && EARLY) {
            // two batches' activations under way (registers)
            Batch b0, b1;
            u32x4_t x0[GL], x1[GL];
            begin(b0, x0);
            for (;;) {
                if (last(b0)) { finish(b0, x0); break; }
                begin(b1, x1);
                finish(b0, x0);
                if (last(b1)) { finish(b1, x1); break; }
                begin(b0, x0);
                finish(b1, x1);
            }
        } else {
            for (;;) {
                Batch b;
                u32x4_t x[GL];
                begin(b, x);
                finish(b, x);
                if (last(b)) break;
            }
        }
        lds_barrier();
        if (wk == 0)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int tb = 0; tb < TB; ++tb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        sum[rb][tb][r] += *(lds_cf32_t *)(uintptr_t)(lds0 + ((wn * RB + rb) * 32 + 8 * (r / 4) + 4 * h + r % 4) * (BM * 4) + (32 * tb + i) * 4);
    }
    if (wk > 0) return;

    // ---------------------------------------------------------------- store: register r of a block is its row 8 (r / 4) + 4 h + r % 4
    const bool f32 = ga.y_f32 != 0, b16 = a.y_bf16 != 0;
    const bool quads = !f32 && a.y_stride % 4 == 0 && ((uintptr_t)a.y & 7) == 0;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        const uint32_t m = m0 + 32 * tb + i;
        if (m >= M) continue;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const uint32_t n = n0 + (wn * RB + rb) * 32 + 8 * r4 + 4 * h;
                const int64_t o = (int64_t)m * a.y_stride + n;
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = sum[rb][tb][4 * r4 + r];
                if (quads && n + 3 < N) {
                    uint16_t b[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) b[r] = b16 ? float_to_bf16_bits(v[r]) : __builtin_bit_cast(uint16_t, (_Float16)v[r]);
                    *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(a.y) + o) =
                        make_uint2((uint32_t)b[0] | ((uint32_t)b[1] << 16), (uint32_t)b[2] | ((uint32_t)b[3] << 16));
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (n + r < N) store_out(a.y, o + r, v[r], f32, b16);
                }
            }
    }
}

template <int BITS, int MODE, class C>
__global__ __launch_bounds__(C::T, C::kWavesPerSimd) void decode_gemm_kernel(GemmArgs ga)
{
    tile_product<BITS, MODE, C>(ga);
}

// Up to 32 tokens of many rows: the same product in tiles of 32 tokens (launch_wide_tiles).
template <int BITS, int MODE, class C>
__global__ __launch_bounds__(C::T, C::kWavesPerSimd) void decode_wide_tiles_kernel(GemmArgs ga)
{
    tile_product<BITS, MODE, C>(ga);
}

// The two copies of the activations.  Blocks [0, nb): xp, one thread per (token, run of 32 columns).  The rest: xt, a
// block per tile of 64 columns x 64 tokens, through LDS.  bf16 activations are converted to fp16 on the way.
template <int BITS>
__global__ __launch_bounds__(256) void relayout_x_gemm_kernel(const uint16_t *x, int64_t ldx, uint32_t M, uint32_t K, int bf16,
                                                              uint16_t *xp, uint16_t *xt, uint32_t MP, uint32_t nb)
{
    if (blockIdx.x < nb) {
        // run c of token m: half h, turn p of block B in the source's order is run 8 B + 4 h + p; the last block of a row
        // with an odd number of groups has zeros for its second half
        const uint32_t id = blockIdx.x * 256 + threadIdx.x, runs = (K + 255) / 256 * 8;
        if (id >= M * runs) return;
        const uint32_t m = id / runs, c = id - m * runs, hh = c / 4 % 2, p4 = c % 4;
        uint32_t w[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = 0u;
        if (c * 32 < K) {
            const uint4 *p = reinterpret_cast<const uint4 *>(x + (size_t)m * ldx + (size_t)c * 32);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint4 v = p[j];
                w[4 * j] = v.x; w[4 * j + 1] = v.y; w[4 * j + 2] = v.z; w[4 * j + 3] = v.w;
            }
            if (bf16) {
#pragma unroll
                for (int j = 0; j < 16; ++j) w[j] = bf16x2_to_f16x2(w[j]);
            }
        }
        auto at = [&](int s) { const int k = slot_k(BITS, s); return k & 1 ? w[k / 2] >> 16 : w[k / 2] & 0xFFFFu; };
        uint4 *o = reinterpret_cast<uint4 *>(xp + ((size_t)m * runs + c / 8 * 8) * 32) + 8 * p4 + hh;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t d[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) d[e] = at(8 * j + 2 * e) | (at(8 * j + 2 * e + 1) << 16);
            o[2 * j] = make_uint4(d[0], d[1], d[2], d[3]);
        }
        return;
    }
    __shared__ uint16_t tile[64][66];
    const uint32_t b = blockIdx.x - nb, tk = K / 64, k0 = b % tk * 64, m0 = b / tk * 64;
    const uint32_t c = threadIdx.x % 8, r = threadIdx.x / 8;   // column octet, token
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const uint32_t m = m0 + r + 32 * g;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (m < M) v = *reinterpret_cast<const uint4 *>(x + (size_t)m * ldx + k0 + 8 * c);
        if (bf16) v = make_uint4(bf16x2_to_f16x2(v.x), bf16x2_to_f16x2(v.y), bf16x2_to_f16x2(v.z), bf16x2_to_f16x2(v.w));
        uint32_t *d = reinterpret_cast<uint32_t *>(&tile[r + 32 * g][8 * c]);
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const uint32_t k = r + 32 * g;                         // now: token octet c, column k
        uint32_t d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = (uint32_t)tile[8 * c + 2 * e][k] | ((uint32_t)tile[8 * c + 2 * e + 1][k] << 16);
        if (m0 + 8 * c < MP) *reinterpret_cast<uint4 *>(xt + (size_t)(k0 + k) * MP + m0 + 8 * c) = make_uint4(d[0], d[1], d[2], d[3]);
    }
}

template <int BITS, int MODE, class C>
hipError_t launch_gemm_t(GemmArgs &ga, hipStream_t s)
{
    void (*kern)(GemmArgs);
    if constexpr (C::BM == 32) kern = decode_wide_tiles_kernel<BITS, MODE, C>;
    else kern = decode_gemm_kernel<BITS, MODE, C>;
    const int lds = C::template kBase<BITS> + (MODE == 1 ? ((int)((ga.a.L + 1) * (2u << BITS)) + 15) / 16 * 16 + C::kIds : 0);
    static_assert(C::template kBase<BITS> + (MODE == 1 ? (257 * (2 << BITS) + 15) / 16 * 16 + C::kIds : 0) <= 160 * 1024, "");
    ga.fine = ga.a.K <= kFineK || C::WK > 1;
    ga.deep = C::DEEP && ga.a.K > kDeepK;
    static std::atomic<int> configured[kMaxDevices];           // per device; idempotent attribute, benign race
    const int dev = current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    if (!configured[dev].load(std::memory_order_relaxed)) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (err != hipSuccess) return err;
        configured[dev].store(1, std::memory_order_relaxed);
    }
    ga.row0 = 0;
    ga.tiles_n = (ga.a.N + C::BN - 1) / C::BN;
    ga.tiles_m = (ga.M + C::BM - 1) / C::BM;
    const uint32_t per = (ga.tiles_n * ga.tiles_m + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(8 * per), dim3(C::T), lds, s, ga);
    return hipGetLastError();
}

// 128 rows x 64 tokens (four parts in the ring, three of them requested ahead: 4096 x 4096, 333 tokens, 3 bits 34 us with three, 32.7
// with four), x 32; 64 x 64, in parts of a whole turn where the index words leave LDS for three, 2 and 3 bits (with parts of half a
// turn the waves met twice as often, us without outliers 287 x 10880, 3 bits, 458 tokens 49.4 / 45.8, 1908 x 7168, 2 bits, 310
// 31.9 / 30.7, with 0.05 % 326 x 16896, 3 bits, 475 78.5 / 72.8).
template <int BITS, bool PLAIN = false>
using SmallTile = GemmTile<1, 2, 4, 2, 4, PLAIN ? 3 : 4, BITS == 4 ? 2 : 3, PLAIN>;
using LowTile = GemmTile<1, 1, 4, 2, 4, 5, 3>;
template <int BITS, bool PLAIN = false>
using TinyTile = std::conditional_t<BITS == 4, GemmTile<1, 2, 2, 4, 2, 4, 2, PLAIN>, GemmTile<1, 2, 2, 4, 4, 3, 2, PLAIN>>;

template <int BITS, int MODE>
hipError_t launch_gemm_m(GemmArgs &ga, hipStream_t s)
{
    // A round of tiles takes the same time for any number of them up to the 256 CUs, so the tile is as large as it can be
    // with few rounds.  Measured, 4 bits (2048 x 28672: 3 bits), us in tiles of 64 x 64 / 128 x 64 / 256 x 128 and their number:
    //   4096 x 4096, 256 tokens: 36 (256) / 51 (128) / 94 (32); 333: 60 (384) / 53 (192) / 94; 1024: 111 / 94 (512) / 97 (128);
    //   2048: 212 / 181 (1024) / 119 (256)
    //   8192 x 8192, 256 tokens: 95 (512) / 84 (256) / 155 (64); 512: 177 / 151 (512) / 157 (128); 700: 256 / 216 (704) / 169 (192)
    //   2048 x 28672, 512 tokens: 143 (256) / 237 (128) / 463 (32); 28672 x 8192, 512 tokens: 610 / 511 (1792) / 346 (448)
    using Large = GemmTile<1, 4, 8, 1, 4, 3, 2>;
    using Small = SmallTile<BITS>;
    using Small16 = GemmTile<1, 2, 4, 4, 2, 3, 2>;
    const uint64_t m = (ga.M + 63) / 64, small = (uint64_t)((ga.a.N + 127) / 128) * m;
    if ((uint64_t)((ga.a.N + 63) / 64) * m <= 256) {
        if (ga.a.K <= kPlainTinyK) return launch_gemm_t<BITS, MODE, TinyTile<BITS, true>>(ga, s);
        return launch_gemm_t<BITS, MODE, TinyTile<BITS>>(ga, s);
    }
    // (rows that ask for a third set of sums, in matrices that the 16-token kernel would cut into slices: see kDeepK)
    if (small > 512 && (ga.a.K <= kDeepK || ga.a.N >= 8192)) return launch_gemm_t<BITS, MODE, Large>(ga, s);
    // 2-bit weights leave registers for four waves to a SIMD, of which four share their rows and a quarter of K each
    // (4096 x 4096, 333 tokens: 42 us against 46 with two waves to a SIMD)
    if constexpr (BITS == 2)
        if (ga.a.K > kFineK) return launch_gemm_t<BITS, MODE, Small16>(ga, s);
    if (ga.a.K <= kPlainSmallK) return launch_gemm_t<BITS, MODE, SmallTile<BITS, true>>(ga, s);
    return launch_gemm_t<BITS, MODE, Small>(ga, s);
}

// What both kinds of launch begin with: the arguments and the copies of the activations, of cap halves each.
template <int BITS>
hipError_t prepare_gemm(GemmArgs &ga, const DecodeArgs &a, int M, bool y_f32, uint16_t *xp, uint16_t *xt, uint64_t cap, hipStream_t s)
{
    const uint32_t runs = (a.K + 255) / 256 * 8;
    ga.a = a;
    ga.M = (uint32_t)M;
    ga.MP = (ga.M + 7) / 8 * 8;
    if ((uint64_t)a.K * ga.MP > cap || (uint64_t)ga.M * runs * 32 > cap) return hipErrorInvalidValue;
    ga.xp = xp;
    ga.xt = xt;
    ga.y_f32 = (int)y_f32;
    const uint32_t nb = (uint32_t)(((uint64_t)ga.M * runs + 255) / 256), nt = a.col ? a.K / 64 * ((ga.M + 63) / 64) : 0u;
    hipLaunchKernelGGL(relayout_x_gemm_kernel<BITS>, dim3(nb + nt), dim3(256), 0, s, a.x, a.x_stride, ga.M, a.K, (int)a.x_bf16,
                       xp, xt, ga.MP, nb);
    return hipGetLastError();
}

template <int BITS>
hipError_t launch_gemm_b(int mode, const DecodeArgs &a, int M, bool y_f32, PromptCopies *xc, hipStream_t s)
{
    GemmArgs ga;
    hipError_t err = prepare_gemm<BITS>(ga, a, M, y_f32, xc->xb, xc->xt, kGemmHalves, s);
    if (err != hipSuccess) return err;
    return mode == 1 ? launch_gemm_m<BITS, 1>(ga, s) : launch_gemm_m<BITS, 0>(ga, s);
}

static_assert(kCopyHalves / 32 <= kDeepK, "the longest row with more than 16 tokens (wide_supports)");
template <int BITS, int MODE>
hipError_t launch_wide_tiles_m(GemmArgs &ga, hipStream_t s)
{
    if (ga.M <= 32) return launch_gemm_t<BITS, MODE, LowTile>(ga, s);
    return launch_gemm_t<BITS, MODE, SmallTile<BITS>>(ga, s);
}

template <int BITS>
hipError_t launch_wide_tiles_b(int mode, const DecodeArgs &a, int M, bool y_f32, XCopies *xc, hipStream_t s)
{
    GemmArgs ga;
    hipError_t err = prepare_gemm<BITS>(ga, a, M, y_f32, xc->xb, xc->xt, kCopyHalves, s);
    if (err != hipSuccess) return err;
    return mode == 1 ? launch_wide_tiles_m<BITS, 1>(ga, s) : launch_wide_tiles_m<BITS, 0>(ga, s);
}

}  // namespace

// 17 to 64 tokens of many rows, the 64-token kernel's, as one column of 128-row tiles: that kernel reads its activations from L2
// once per 32 rows and a lookup per pair of weights from LDS, which is most of its time once the matrix is large.  A round of tiles
// takes the same time for any number of them, so they have to fill most of the last one; more of it for a library, whose ids the tiles
// fetch through LDS and whose tables the other kernel builds once, most of all at 3 bits.  Always more than the line: at the half and at
// three quarters of a round the other kernel's own rounds, of 512 tiles of 32 rows, are full (16370 x 640, 36 tokens, 3 bits, library
// 14.1 us there, 17.9 in tiles; 24458 x 9856, 24, 4 bits 63 / 70).  us in the 64-token kernel / in tiles (cold weights, 0.05 to 1 %
// outliers), at 7664 shapes drawn near the lines and above, of which 6314 are above: 21 of these are more than 2.5 % slower in tiles, all but
// three in three rounds and more or within 3.1 % (7 % at most: 148979 x 2176, 53 tokens 144 / 154), the median 16 % faster:
//  - 28672 x 8192: 64 tokens, 3 bits, library 83 / 63, 4 bits 83 / 64; 32 tokens (tiles of 32), 3 bits 57 / 48, 17, 2 bits 46 / 39;
//  - one round: 17 to 48 tokens above three quarters 3 % slower at most, the median 11 to 15 % faster; more than 48 above five eighths
//    4 % slower at most, but libraries at 3 and 4 bits 10 % below three quarters (23810 x 2176, 49 30 / 33); rows of up to 1024 columns from
//    half a round on, where no library at 3 bits has more than 512 (16367 x 512, 59 14.3 / 15.6 at the half);
//  - several rounds: 4 bits, 17 to 32 tokens below fifteen sixteenths up to 8 % slower (146550 x 2176, 32 117 / 127), 33 to 48 tokens at 3
//    bits up to 10 % (115953 x 2176, 44 105 / 115), of a library 13 % (144207 x 1792, 43 115 / 130) and 6 % above that line; more than 48
//    tokens of a library below seven eighths 14 % (107614 x 1664, 56 95 / 109); rows of 640 to 1024 columns of a library below seven
//    eighths 15 % (72223 x 1024, 44 51 / 59), up to 512 columns 10 to 20 % faster there.
// What lies below the lines is given up for the sake of the slower ones: 4 % faster in tiles at the median.
bool prefer_wide_tiles(int bits, int mode, uint32_t N, uint32_t K, int M)
{
    const uint64_t m = (uint64_t)(M + 7) / 8 * 8, k = (uint64_t)(K + 255) / 256 * 256;
    if (mode > 1 || M < 17 || m * k > kCopyHalves) return false;
    const uint64_t tiles = ((uint64_t)N + 127) / 128, rounds = (tiles + 255) / 256;
    const bool lib = mode == 1, many = rounds > 1;
    uint64_t line;                                             // sixteenths of all rounds
    if (M > 32 && K <= 512) line = many ? 11 : 8;
    else if (M > 32 && K <= 1024) line = many ? (lib ? 14 : 12) : lib && bits == 3 ? 12 : 8;
    else if (M > 48) line = many ? (lib ? 14 : 13) : lib && bits >= 3 ? 12 : 10;
    else if (!many) line = 12;
    else if (M > 32) line = lib && bits == 3 ? 16 : bits == 3 || (lib && bits == 4) ? 15 : 14;
    else line = bits == 4 ? 15 : 14;
    return tiles > line * 16 * rounds;
}

hipError_t launch_wide_tiles(int bits, int mode, const DecodeArgs &a, int M, bool y_f32, XCopies *xc, hipStream_t s)
{
    if (!xc || mode < 0 || mode > 1) return hipErrorInvalidValue;
    if (bits == 4) return launch_wide_tiles_b<4>(mode, a, M, y_f32, xc, s);
    if (bits == 3) return launch_wide_tiles_b<3>(mode, a, M, y_f32, xc, s);
    return launch_wide_tiles_b<2>(mode, a, M, y_f32, xc, s);
}

// What the kernel takes: V2 and V2a at 2 to 4 bits, more than 64 tokens (which calls prefer it: prefer_gemm).  Rows up to 65536 columns (an outlier's column is kept in 16 bits;
// the copies of 256 tokens fit the workspace) and 128 rows and more: smaller matrices leave the chip to a few workgroups
// either way, and the 64-token kernel's 32-row tiles give them more.
bool gemm_supports(int bits, int mode, uint32_t L, uint32_t N, uint32_t K, int M)
{
    return bits >= 2 && bits <= 4 && (mode == 0 || (mode == 1 && L >= 1)) && M > 64 && N >= 128 && K % kGroup == 0 && K <= 65536;
}

int gemm_tokens(uint32_t K, int M)
{
    const uint32_t cap = (uint32_t)(kGemmHalves / ((K + 255) / 256 * 256)) & ~7u;
    return (uint32_t)M <= cap ? M : (int)(cap >= 256 ? cap & ~255u : cap);
}

// One pair of launches: the copies of the activations, the product.
hipError_t launch_decode_gemm(int bits, int mode, const DecodeArgs &a, int M, bool y_f32, PromptCopies *xc, hipStream_t s)
{
    if (!xc) return hipErrorInvalidValue;
    if (bits == 4) return launch_gemm_b<4>(mode, a, M, y_f32, xc, s);
    if (bits == 3) return launch_gemm_b<3>(mode, a, M, y_f32, xc, s);
    return launch_gemm_b<2>(mode, a, M, y_f32, xc, s);
}

}  // namespace xfp
