// General fused decode kernel: any K that is a multiple of 128, any N, every bit width of the paper's
// packing table (2 .. 6), and the only kernel for V2a matrices with a scale and a mid-point per group.
//
// One wave owns one output row at a time (no atomics, a fixed summation
// order).  The activation row is staged once per workgroup in LDS (paper
// section 5, activation-row caching), the codebook of the row (V2) or the
// whole library (V2a) sits in LDS next to it, each lane streams 32 indices
// per load, looks its codebook entries up in LDS and accumulates in fp32;
// the row's CSR outliers are folded in before the wave reduction.
#include "xfp_device.h"

#include <type_traits>
#include <utility>

namespace xfp {

constexpr int kRowsThreads = 256;
constexpr int kRowsWaves = kRowsThreads / kWave;

typedef __attribute__((address_space(3))) const uint16_t lds_entry_t;
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
}

// Entry of field F: the table (2^BITS entries, aligned to its size) is OR-ed into the field's address, an instruction less than added.
template <int BITS, int F>
__device__ __forceinline__ uint32_t entry(const LaneWords<BITS> &lw, uint32_t table)
{
    constexpr int bit = F * BITS, word = bit / 32, sh = bit % 32;
    uint32_t t;                                                           // the field at bit 1
    if constexpr (sh + BITS > 32) t = __builtin_amdgcn_alignbit(lw.w[word + 1], lw.w[word], sh - 1);
    else if constexpr (sh >= 1) t = lw.w[word] >> (sh - 1);
    else t = lw.w[word] << 1;
    return *(lds_entry_t *)(uintptr_t)((t & (2u * ((1u << BITS) - 1u))) | table);
}

// Eight of them: fields 8 C .. 8 C + 7.
template <int BITS, int C, int... Is>
__device__ __forceinline__ void eight_entries(const LaneWords<BITS> &lw, uint32_t table, uint32_t (&c)[8], std::integer_sequence<int, Is...>)
{
    ((c[Is] = entry<BITS, 8 * C + Is>(lw, table)), ...);
}

// A lane's words through bounds-checked buffer loads: past the end zeros, with no traffic.
template <int BITS>
__device__ __forceinline__ LaneWords<BITS> buffer_lane_words(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int kOnce = 2;                                              // non-temporal
    LaneWords<BITS> w;
    if constexpr (BITS == 2) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kOnce);
        w.w[0] = v.x; w.w[1] = v.y;
    } else if constexpr (BITS == 3) {
        const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(r, off, 0, kOnce);
        w.w[0] = v.x; w.w[1] = v.y; w.w[2] = v.z;
    } else {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kOnce);
        w.w[0] = v.x; w.w[1] = v.y; w.w[2] = v.z; w.w[3] = v.w;
        if constexpr (BITS == 5) w.w[4] = __builtin_amdgcn_raw_buffer_load_b32(r, off + 16, 0, kOnce);
        if constexpr (BITS == 6) {
            const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(r, off + 16, 0, kOnce);
            w.w[4] = q.x; w.w[5] = q.y;
        }
    }
    return w;
}

// 16-byte chunk c of the 32 activations of unit u, in LDS: turned by the unit, so that the 16 lanes that LDS serves together, which
// read one chunk of 16 neighbouring units, find it in 16 different places of the 64 banks (in plain order in four).
__device__ __forceinline__ uint32_t x_chunk(uint32_t u, uint32_t c) { return u * 4 + ((c + (u >> 2)) & 3u); }

// AFF (V2a only): every group carries a scale and a mid-point (paper section 3.4; no formula given, reading
// taken: entry * scale + mid).  By linearity a unit of 32 weights inside one group contributes
// scale * sum(x * entry) + mid * sum(x), both sums in fp32, one fused multiply-add on top.
//
// What bounds it at 5 and 6 bits is the chain of round trips of a wave that owns a row or two, so everything that does not depend on
// something else is asked for at once and ahead: codebook and row pointers of the next row, the index words two steps ahead, across
// rows, a row's outliers in front of its products.  Words and outliers come through buffer loads, which need no branch, so that every
// wait knows how many loads are younger than what it is for.  A step's 32 lookups are four runs of eight beside the run before: at
// 6 bits, in 64 registers, the compiler had made sixteen round trips to LDS of them, one behind the other.
// us with each behind the other / asked for ahead / as it is: 5 bits 8192 x 4096 9.2 / 9.0 / 8.4, 1000 x 20480 15.3 / 9.1 / 8.7,
// 2048 x 3072 5.6 / 4.7 / 4.3, 30000 x 640 15.1 / 13.3 / 12.0; 6 bits 7457 x 1152 5.8 / 6.5 / 5.4, 4974 x 7040 11.0 / 11.8 / 10.9,
// 1828 x 640, 4 tokens 5.5 / 6.2 / 5.3, 11008 x 8192 22.1 / 20.5 / 19.3.
template <int BITS, int MODE, bool YF32, bool AFF>
__global__ __launch_bounds__(kRowsThreads, AFF ? 4 : 8) void decode_rows_kernel(DecodeArgs a)
{
    extern __shared__ __align__(256) unsigned char smem[];                // (2 K bytes are a multiple of 256: the tables are aligned to their size)
    constexpr int ENT = 1 << BITS;
    _Float16 *xs = reinterpret_cast<_Float16 *>(smem);                    // K halves, in the order of x_chunk
    uint4 *xs4 = reinterpret_cast<uint4 *>(smem);
    _Float16 *tables = reinterpret_cast<_Float16 *>(smem + (size_t)a.K * 2);

    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t slot = blockIdx.y;
    const uint32_t e = a.eids ? (uint32_t)a.eids[slot] : 0u;
    const uint32_t N = a.N, K = a.K, G = K / kGroup;
    const uint32_t wpr = K / 32 * BITS;                                  // words per row
    const uint32_t *idx = a.idx + (size_t)e * N * wpr;
    const int32_t *rp = a.rp + (size_t)e * N;
    const uint16_t *x = a.x + (int64_t)slot * a.x_stride;
    const uint32_t row0 = blockIdx.x * a.rows_per_block, row1 = min(N, row0 + a.rows_per_block);
    uint32_t row = row0 + wave;
    const uint32_t units = K / kLaneWeights, steps = (units + kWave - 1) / kWave;

    // Requests.  Units that are not there: no words, the row's last id, results dropped; rows behind the wave's: none.
    auto codebook = [&](uint32_t r) -> uint32_t {
        if constexpr (MODE != 0) return 0u;
        return reinterpret_cast<const uint32_t *>(a.cb + ((size_t)e * N + r) * ENT)[min(lane, (uint32_t)ENT / 2 - 1)];
    };
    int32_t j0 = rp[min(row, row1 - 1)], j1 = rp[min(row, row1 - 1) + 1];
    uint32_t cbn = codebook(min(row, row1 - 1));
    constexpr int XB = 3;
    uint4 xv[XB];
#pragma unroll
    for (int b = 0; b < XB; ++b)
        if (b == 0 || (uint32_t)(b * kRowsThreads) < K / 8) xv[b] = reinterpret_cast<const uint4 *>(x)[min(tid + b * kRowsThreads, K / 8 - 1)];
    constexpr int P = 2;                                                  // steps ahead
    LaneWords<BITS> lw[P];
    uint32_t gid[P], gsc[P], gmd[P];
    uint32_t prow = row, pstep = 0;                                       // of the next request
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)(idx + (size_t)row0 * wpr), 0, (row1 - row0) * wpr * 4, 0x00020000);
    auto request = [&](int j) {
        const uint32_t u = pstep * kWave + lane;
        lw[j] = buffer_lane_words<BITS>(rw, u < units ? (prow - row0) * (wpr * 4) + u * (BITS * 4) : 0x80000000u);
        const size_t g = ((size_t)e * N + min(prow, row1 - 1)) * G + min(u, units - 1) / (kGroup / kLaneWeights);
        if constexpr (MODE == 1) gid[j] = a.gid[g];
        if constexpr (AFF) {
            gsc[j] = a.gscale[g];
            gmd[j] = a.gmid[g];
        }
        if (++pstep == steps) {
            pstep = 0;
            prow += kRowsWaves;
        }
    };
    request(0);
    if (prow < row1) request(1);

    // a1: stage the activation row.
    auto stage = [&](uint32_t i, uint4 v) {
        if (a.x_bf16) v = make_uint4(bf16x2_to_f16x2(v.x), bf16x2_to_f16x2(v.y), bf16x2_to_f16x2(v.z), bf16x2_to_f16x2(v.w));
        xs4[x_chunk(i >> 2, i & 3u)] = v;
    };
#pragma unroll
    for (int b = 0; b < XB; ++b)
        if (tid + b * kRowsThreads < K / 8) stage(tid + b * kRowsThreads, xv[b]);
    for (uint32_t i = tid + XB * kRowsThreads; i < K / 8; i += kRowsThreads) stage(i, reinterpret_cast<const uint4 *>(x)[i]);
    // a2: V2a library -> LDS once per workgroup.
    if constexpr (MODE == 1) {
        const uint16_t *lib = a.cb + (size_t)e * a.L * ENT;
        for (uint32_t i = tid; i < a.L * ENT; i += kRowsThreads)
            tables[i] = __builtin_bit_cast(_Float16, lib[i]);
    }
    lds_barrier();

    _Float16 *mytbl = tables + wave * ENT;                                // V2: per-wave table
    const uint32_t table0 = lds_address(tables);
    for (; row < row1; row += kRowsWaves) {
        if constexpr (MODE == 0) {
            __builtin_amdgcn_wave_barrier();
            if (lane < ENT / 2) reinterpret_cast<uint32_t *>(mytbl)[lane] = cbn;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        // a7, requests: the row's first 64 outliers; the next row's codebook and row pointers
        const int32_t jl = j0 + (int32_t)lane, jend = j1;
        const int32_t jfirst = __builtin_amdgcn_readfirstlane(j0), entries = max(__builtin_amdgcn_readfirstlane(j1) - jfirst, 0);
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc((void *)(a.col + jfirst), 0, entries * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void *)(a.val + jfirst), 0, entries * 2, 0x00020000);
        const uint32_t oc = __builtin_amdgcn_raw_buffer_load_b32(rc, lane * 4, 0, 0), ov = __builtin_amdgcn_raw_buffer_load_b16(rv, lane * 2, 0, 0);
        if (const uint32_t nrow = row + kRowsWaves; nrow < row1) {
            cbn = codebook(nrow);
            j0 = rp[nrow];
            j1 = rp[nrow + 1];
        }
        float acc = 0.f;
        // a3/a4: stream and depack; a5: gather; a6: multiply-accumulate.  One step, whose words are request j's.
        auto step = [&](uint32_t s, int j) {
            const uint32_t u = s * kWave + lane;
            const LaneWords<BITS> w = lw[j];
            const uint32_t id = MODE == 1 ? gid[j] : 0u;
            const float sc = AFF ? half_bits_to_float((uint16_t)gsc[j]) : 0.f, md = AFF ? half_bits_to_float((uint16_t)gmd[j]) : 0.f;
            if (prow < row1) request(j);
            if (u >= units) return;
            const uint32_t tbl = MODE == 1 ? table0 + id * (ENT * 2) : table0 + wave * (ENT * 2);
            const half2_t ones = {(_Float16)1.0f, (_Float16)1.0f};
            float au = 0.f, sum = 0.f;
            uint4 xq[2];
            uint32_t c[2][8];
            auto read = [&](auto quarter) {                               // eight activations and their entries
                constexpr int q = decltype(quarter)::value;
                xq[q & 1] = xs4[x_chunk(u, q)];
                eight_entries<BITS, q>(w, tbl, c[q & 1], std::make_integer_sequence<int, 8>{});
            };
            auto add = [&](auto quarter) {
                constexpr int q = decltype(quarter)::value;
                const uint32_t xw[4] = {xq[q & 1].x, xq[q & 1].y, xq[q & 1].z, xq[q & 1].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const half2_t pair = as_half2(c[q & 1][2 * i] | (c[q & 1][2 * i + 1] << 16));
                    if constexpr (AFF) {
                        au = dot2(pair, as_half2(xw[i]), au);
                        sum = dot2(ones, as_half2(xw[i]), sum);
                    } else {
                        acc = dot2(pair, as_half2(xw[i]), acc);
                    }
                }
            };
            const std::integral_constant<int, 0> q0; const std::integral_constant<int, 1> q1;
            const std::integral_constant<int, 2> q2; const std::integral_constant<int, 3> q3;
            read(q0);
            read(q1);
            add(q0);
            read(q2);
            add(q1);
            read(q3);
            add(q2);
            add(q3);
            if constexpr (AFF) acc += fmaf(sc, au, md * sum);
        };
        static_assert(P == 2, "the steps below");
        uint32_t s = 0;
        for (; s + 1 < steps; s += 2) {
            step(s, 0);
            step(s + 1, 1);
        }
        if (s < steps) {                                                  // an odd number of them: the requests change places
            step(s, 0);
            const LaneWords<BITS> t = lw[0];
            lw[0] = lw[1];
            lw[1] = t;
            if constexpr (MODE == 1) { const uint32_t v = gid[0]; gid[0] = gid[1]; gid[1] = v; }
            if constexpr (AFF) {
                const uint32_t v = gsc[0], w = gmd[0];
                gsc[0] = gsc[1]; gsc[1] = v;
                gmd[0] = gmd[1]; gmd[1] = w;
            }
        }
        // a7: outlier fold, CSR row owned by this wave.
        auto fold = [&](uint32_t k, uint32_t v) {
            acc = fmaf(half_bits_to_float((uint16_t)v), (float)xs[x_chunk(k >> 5, k >> 3 & 3u) * 8 + (k & 7u)], acc);
        };
        if (jl < jend) fold(oc, ov);
        for (int32_t j = jl + kWave; j < jend; j += kWave) fold((uint32_t)a.col[j], a.val[j]);
        // a8: reduce and store.
        acc = wave_sum(acc);
        if (lane == 0) store_y<YF32>(a.y, (int64_t)slot * a.y_stride + row, acc, a.y_bf16 != 0);
    }
}

template <int BITS, int MODE, bool YF32, bool AFF = false>
static hipError_t launch_rows_t(const DecodeArgs &a, int slots, hipStream_t s)
{
    size_t table_halves = MODE == 1 ? (size_t)a.L << BITS : (size_t)kRowsWaves << BITS;
    size_t smem = (size_t)a.K * 2 + table_halves * 2;
    dim3 grid((a.N + a.rows_per_block - 1) / a.rows_per_block, slots);
    auto kern = decode_rows_kernel<BITS, MODE, YF32, AFF>;
    if (smem > 48 * 1024) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL(kern, grid, dim3(kRowsThreads), smem, s, a);
    return hipGetLastError();
}

template <int BITS>
static hipError_t launch_rows_b(int mode, bool y_f32, const DecodeArgs &a, int slots, hipStream_t s)
{
    if (mode == 0)
        return y_f32 ? launch_rows_t<BITS, 0, true>(a, slots, s) : launch_rows_t<BITS, 0, false>(a, slots, s);
    if (a.gscale)
        return y_f32 ? launch_rows_t<BITS, 1, true, true>(a, slots, s) : launch_rows_t<BITS, 1, false, true>(a, slots, s);
    return y_f32 ? launch_rows_t<BITS, 1, true>(a, slots, s) : launch_rows_t<BITS, 1, false>(a, slots, s);
}

hipError_t launch_decode_rows(int bits, int mode, bool y_f32, const DecodeArgs &a, int slots,
                              hipStream_t s)
{
    switch (bits) {
    case 2: return launch_rows_b<2>(mode, y_f32, a, slots, s);
    case 3: return launch_rows_b<3>(mode, y_f32, a, slots, s);
    case 5: return launch_rows_b<5>(mode, y_f32, a, slots, s);
    case 6: return launch_rows_b<6>(mode, y_f32, a, slots, s);
    default: return launch_rows_b<4>(mode, y_f32, a, slots, s);
    }
}

}  // namespace xfp
