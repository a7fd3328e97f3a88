// The compression g = C y of Eq. (ylq) as a kernel of its own: G[m, n] = sum_c X[m, c] * C[n, c] with a
// short n range (k <= 64 phantom neurons), bf16 in, fp32 accumulate, bf16 out.
//
// As a tile of the general product it has few workgroups (one per 128 rows: 64 for an 8192-row batch)
// and every one of them walks the whole reduction range, so three quarters of the device wait for
// 14 us.  Here a workgroup owns 32 rows and all n; its eight wavefronts split the reduction range, then add their partial sums through LDS
// (thin_workgroup, as part of another kernel, feeds the MFMAs straight from global memory).  C (k x s, at most 128 KB) is
// read by every workgroup, from L2.
// What bounds it: the loads of operands in the MFMA's layout, 16 contiguous bytes of a row per lane.  On
// v_mfma_f32_16x16x32_bf16 an instruction covers 64 bytes of 16 rows, where v_mfma_f32_32x32x16_bf16 covers 32 bytes of 32,
// and up to 16 phantom neurons read half as much of C.  Us a step (32x32x16 : so): gradients of 64 ranks of 256 + 8, 4 layers at
// batch 512, 465 : 458; 8 ranks of 512 + 32 and 1024 + 64 in turn, 4 layers trained at 1024, 370 : 363.
// Wavefronts share the reduction in chunks of 32 (16 with the other form): where the shard is no multiple of 256 their partial sums are cut elsewhere, an other
// order of the same sum and no less exact, in which some values next to a rounding boundary of bf16 round the other way.
#pragma once
#include "common.h"
#include "elementwise.h"    // ClearList
#include "mfma_ring.h"

#include <type_traits>

namespace phantom {

constexpr int THIN_ROWS = 32;       // rows of X per workgroup
constexpr int THIN_MAX_N = 64;
constexpr int THIN_WAVES = 8;       // wavefronts per workgroup of the stand-alone kernel

typedef __bf16 thin_bf16x8 __attribute__((ext_vector_type(8)));
typedef float thin_f32x4 __attribute__((ext_vector_type(4)));

// One workgroup's share: rows [m0, m0 + 32) of group grp.  NF = number of 16-wide column blocks (N <= 16 NF);
// WAVES wavefronts split the reduction range (K is a multiple of 16) in chunks of 32; part: WAVES * NF * 512
// floats of LDS.  x_g, c_g, o_g: element offsets per group.
// M: end of the rows this call may read and store (the matrix's row count, or the end of a shorter share of a
// 32-row block: the MFMA rows beyond it repeat the last one and are dropped).
template <int NF, int WAVES>
__device__ __forceinline__ void thin_workgroup(const __bf16 *__restrict__ X, const __bf16 *__restrict__ C,
                                               __bf16 *__restrict__ G, int M, int N, int K, int64_t x_g, int64_t c_g,
                                               int64_t o_g, int m0, int grp, float *part)
{
    constexpr int MF = THIN_ROWS / 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const __bf16 *x = X + grp * x_g, *c = C + grp * c_g;
    __bf16 *out = G + grp * o_g;
    // [wavefront][row block][column block][accumulator][lane], turned such that a wavefront that reads whole rows meets every bank once
    auto part_at = [part](int w, int r, int f, int e, int l) -> float & { return part[(((w * MF + r) * NF + f) * 4 + e) * 64 + ((l + 16 * (f + NF * e)) & 63)]; };

    // this wavefront's share of the whole chunks; the last one takes the half that may be left
    const int chunks = K >> 5;
    const int c_lo = (int)((int64_t)chunks * wave / WAVES), c_hi = (int)((int64_t)chunks * (wave + 1) / WAVES);
    // MFMA operand of a lane: row (lane & 15), 8 consecutive reduction indices starting at 8 * (lane >> 4).
    // Rows past the end read the last row; what they produce is never stored.
    const int quarter = (lane >> 4) * 8;
    const __bf16 *xrow[MF], *crow[NF];
#pragma unroll
    for (int r = 0; r < MF; ++r) xrow[r] = x + (int64_t)min(m0 + r * 16 + (lane & 15), M - 1) * K + quarter;
#pragma unroll
    for (int f = 0; f < NF; ++f) crow[f] = c + (int64_t)min(f * 16 + (lane & 15), N - 1) * K + quarter;

    thin_f32x4 acc[MF][NF];
#pragma unroll
    for (int r = 0; r < MF; ++r)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[r][f] = thin_f32x4{0.f, 0.f, 0.f, 0.f};
    // four chunks' loads in flight together, then two, then one (a 1024-wide shard gives a wavefront exactly four)
    int ch = c_lo;
    auto batch = [&](auto count) {
        constexpr int U = decltype(count)::value;
        thin_bf16x8 a[MF][U], b[NF][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int r = 0; r < MF; ++r) a[r][u] = *(const thin_bf16x8 *)(xrow[r] + (ch + u) * 32);
#pragma unroll
            for (int f = 0; f < NF; ++f) b[f][u] = *(const thin_bf16x8 *)(crow[f] + (ch + u) * 32);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < MF; ++r)
#pragma unroll
                for (int f = 0; f < NF; ++f) acc[r][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r][u], b[f][u], acc[r][f], 0, 0, 0);
        ch += U;
    };
    while (ch + 4 <= c_hi) batch(std::integral_constant<int, 4>{});
    if (ch + 2 <= c_hi) batch(std::integral_constant<int, 2>{});
    if (ch < c_hi) batch(std::integral_constant<int, 1>{});
    if ((K & 16) && wave == WAVES - 1) {               // uniform: the upper 16 indices of the chunk do not exist
        const int at = quarter < 16 ? chunks * 32 : chunks * 32 - 16;      // (in bounds: read by their neighbours' lanes too)
        const auto half = [&](const __bf16 *row) {
            thin_bf16x8 v = *(const thin_bf16x8 *)(row + at);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = quarter < 16 ? v[i] : (__bf16)0.f;
            return v;
        };
        thin_bf16x8 b[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) b[f] = half(crow[f]);
#pragma unroll
        for (int r = 0; r < MF; ++r) {
            const thin_bf16x8 a = half(xrow[r]);
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[r][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[f], acc[r][f], 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < MF; ++r)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int e = 0; e < 4; ++e) part_at(wave, r, f, e, lane) = acc[r][f][e];
    __syncthreads();

    // accumulator e of lane l in blocks r, f is element (row 16 r + 4 (l >> 4) + e, column 16 f + (l & 15))
    for (int o = threadIdx.x; o < THIN_ROWS * NF * 16; o += WAVES * 64) {
        const int row = o / (NF * 16), col = o - row * (NF * 16);
        const int m = m0 + row;
        if (m >= M || col >= N) continue;
        const int r = row >> 4, f = col >> 4, e = row & 3, l = (col & 15) + 16 * ((row >> 2) & 3);
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) sum += part_at(w, r, f, e, l);
        out[(int64_t)m * N + col] = (__bf16)sum;
    }
}

// The kernel: workgroup (x, y) = rows [32 x, 32 x + 32) of group y, THIN_WAVES wavefronts; the sums of thin_workgroup in the same order.
// Neighbouring lanes of an operand in the MFMA's layout lie in different rows, and such loads run at a quarter of the rate (17 bytes a clock).  So a wavefront
// loads 64 bytes of 16 rows at a time to LDS that it alone reads, `ahead` chunks at once (all that it has, up to four), and no barrier comes before the sum over
// wavefronts.  Us a step, operands straight from memory : so: gradients of 8 ranks of 512 + 224 at batch 1024 208 :
// 205.5, of 64 of 256 + 504 at 512 433.5 : 431, unequal widths of 512 and 1024 trained at 1024 332.7 : 329.9.
// Rider: the kernel also clears buffers that later launches of a training step add into.
constexpr int THIN_AHEAD = 4;
constexpr int thin_chunk_bytes(int nf) { return (THIN_ROWS / 16 + nf) * 1024; }
// a wavefront's sums lie over its operands
constexpr int thin_region(int nf, int ahead) { return ahead * thin_chunk_bytes(nf) > nf * 2048 ? ahead * thin_chunk_bytes(nf) : nf * 2048; }

template <int NF>
__global__ __launch_bounds__(THIN_WAVES * 64) void thin_product_kernel(const __bf16 *__restrict__ X, const __bf16 *__restrict__ C,
                                                          __bf16 *__restrict__ G, int M, int N, int K,
                                                          int64_t x_g, int64_t c_g, int64_t o_g, int ahead,
                                                          ClearList clear)
{
    constexpr int MF = THIN_ROWS / 16, NL = MF + NF, CHUNK = thin_chunk_bytes(NF);
    extern __shared__ __attribute__((aligned(16))) unsigned char thin_lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), grp = blockIdx.y, m0 = blockIdx.x * THIN_ROWS;
    const int region = thin_region(NF, ahead);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LdsBytes)thin_lds + wave * region;
    // this wavefront's share of the whole chunks; the last one takes the half that may be left
    const int chunks = K >> 5, first = chunks * wave / THIN_WAVES;
    const int count = chunks * (wave + 1) / THIN_WAVES - first + (wave == THIN_WAVES - 1 && (K & 16) ? 1 : 0);
    // A load: lane l has row l / 4 and vector (l & 3) ^ (l >> 4) of a chunk, so that the operand reads of 16 rows at one vector fall on different banks.
    // Rows past the end read the last row; what they produce is never stored.  The half chunk that does not exist is read in the last half's place.
    const int row = lane >> 2, col = ((lane & 3) ^ (lane >> 4)) * 8;
    const __bf16 *xrow[MF], *crow[NF];
#pragma unroll
    for (int r = 0; r < MF; ++r) xrow[r] = X + grp * x_g + (int64_t)min(m0 + r * 16 + row, M - 1) * K;
#pragma unroll
    for (int f = 0; f < NF; ++f) crow[f] = C + grp * c_g + (int64_t)min(f * 16 + row, N - 1) * K;
    auto fetch = [&](int i, uint32_t to) {
        int c = (first + i) * 32 + col;
        c = c < K ? c : c - 16;
#pragma unroll
        for (int r = 0; r < MF; ++r) ring_load<0>(xrow[r] + c, to + r * 1024);
#pragma unroll
        for (int f = 0; f < NF; ++f) ring_load<0>(crow[f] + c, to + (MF + f) * 1024);
    };
    for (int i = 0; i < min(ahead, count); ++i) fetch(i, lds0 + i * CHUNK);            // uniform
    clear_rider(clear, (int)(blockIdx.y * gridDim.x + blockIdx.x), (int)(gridDim.x * gridDim.y), THIN_WAVES * 64);
    thin_f32x4 acc[MF][NF];
#pragma unroll
    for (int r = 0; r < MF; ++r)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[r][f] = thin_f32x4{0.f, 0.f, 0.f, 0.f};
    // operand of a lane: row (lane & 15), 8 consecutive reduction indices starting at 8 * (lane >> 4)
    const uint32_t at = (lane & 15) * 64 + (((lane >> 4) ^ ((lane >> 2) & 3)) << 4);
    uint32_t slot = lds0;
    for (int i = 0; i < count; ++i) {                  // uniform
        const int later = min(count - 1 - i, ahead - 1);
        // (The rider's stores count among the outstanding operations.  They are out by the second chunk, but counting from there on is slower: 8 ranks of 2048 + 32
        // at batch 1024 6.6 : 6.6 us a launch, of 4096 + 32 13.4 : 15.3, of 2048 + 64 9.6 : 9.8, 4 of 4096 + 16 at 2048 12.4 : 13.2.)
        if (clear.count) ring_own<0>();
        else ring_landed<NL, THIN_AHEAD - 1>(later);
        thin_bf16x8 a[MF], b[NF];
#pragma unroll
        for (int r = 0; r < MF; ++r) a[r] = *lds_at<const thin_bf16x8>(slot + at + r * 1024);
#pragma unroll
        for (int f = 0; f < NF; ++f) b[f] = *lds_at<const thin_bf16x8>(slot + at + (MF + f) * 1024);
        if ((first + i) * 32 + 32 > K && lane >= 32) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
#pragma unroll
                for (int r = 0; r < MF; ++r) a[r][u] = (__bf16)0.f;
#pragma unroll
                for (int f = 0; f < NF; ++f) b[f][u] = (__bf16)0.f;
            }
        }
#pragma unroll
        for (int r = 0; r < MF; ++r)
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[r][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r], b[f], acc[r][f], 0, 0, 0);
        if (i + ahead < count) {                       // uniform; the slot's operands are in registers
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fetch(i + ahead, slot);
        }
        slot = slot + CHUNK == lds0 + ahead * CHUNK ? lds0 : slot + CHUNK;
    }
    // [wavefront][row block][column block][accumulator][lane], turned such that a wavefront that reads whole rows meets every bank once
    float *const part = (float *)thin_lds;
    auto part_at = [part, region](int w, int r, int f, int e, int l) -> float & { return part[w * (region / 4) + ((r * NF + f) * 4 + e) * 64 + ((l + 16 * (f + NF * e)) & 63)]; };
#pragma unroll
    for (int r = 0; r < MF; ++r)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int e = 0; e < 4; ++e) part_at(wave, r, f, e, lane) = acc[r][f][e];
    __syncthreads();
    // accumulator e of lane l in blocks r, f is element (row 16 r + 4 (l >> 4) + e, column 16 f + (l & 15))
    __bf16 *const out = G + grp * o_g;
    for (int o = threadIdx.x; o < THIN_ROWS * NF * 16; o += THIN_WAVES * 64) {
        const int orow = o / (NF * 16), ocol = o - orow * (NF * 16);
        const int m = m0 + orow;
        if (m >= M || ocol >= N) continue;
        const int r = orow >> 4, f = ocol >> 4, e = orow & 3, l = (ocol & 15) + 16 * ((orow >> 2) & 3);
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < THIN_WAVES; ++w) sum += part_at(w, r, f, e, l);
        out[(int64_t)m * N + ocol] = (__bf16)sum;
    }
}

}  // namespace phantom
