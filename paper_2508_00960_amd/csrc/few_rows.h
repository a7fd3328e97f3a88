// A layer's forward products (Eq. (ylq): the update with the peers' part, and the compression beside it) for a batch of few rows, as
// inference at a serving batch has them: bf16, operands in 16-byte vectors, one rank.
//
// What bounds it.  The weights are read once and multiplied by a handful of rows, so a launch is a chain of latencies: parameters, one read of
// the operands, a few matrix instructions, the sum over wavefronts, the epilogue.  The tiles of gemm_flex.h walk the reduction in dependent steps with
// a barrier each, and 32 x 32 of them are too few to occupy the chip: 48 rows of 1024 + 448 make 72 workgroups that read 188 KB each.  Here a workgroup owns 16
// output columns and ROWS x 16 rows, its eight wavefronts split the reduction, and each requests up to few_ahead chunks of 32 reduction indices at
// once, to LDS that it alone reads: no barrier before the sum over wavefronts.  (Loads of operands in the matrix cores' layout, whose
// neighbouring lanes lie in different rows, run at a quarter of the rate.)
// Us a pass, 6 layers forward at batch 48 (gemm_flex.h : direct loads : so): 1024 + 448 46.4 : 38.8 : 36.3, 256 + 112 36.2 : 26.7 : 26.2, 1024 + 1792
// 67.0 : 57.2 : 54.4; a launch of nothing else is 4 of the 6 us a layer of the first.
#pragma once
#include "common.h"
#include "epilogue.h"
#include "mfma_ring.h"

namespace phantom {

constexpr int FEW_WAVES = 8, FEW_TILE = 16;
constexpr int few_ahead(int rows) { return rows == 1 ? 8 : rows == 2 ? 6 : 3; }        // chunks of a wavefront in flight
constexpr int few_lds_bytes(int rows) { return FEW_WAVES * few_ahead(rows) * (rows + 1) * 1024; }

// out(m, n) = sum_c A(m, c) B(n, c): both operands a head block [rows x split] and peers' segments of seg columns
struct FewProduct {
    const __bf16 *a0, *a1, *b0, *b1;
    void *out, *aux;
    const __bf16 *bias;      // NULL: neither bias nor activation
    int M, N, K, split, seg;
    uint32_t magic;          // ceil(2^32 / seg)
    int a_seg, b_seg;        // elements from a segment to the next
    int tiles_n, pitch;      // workgroups of a tile row, and that number rounded up to a multiple of 8: the workgroups that read the same
                             //   rows of B are on one XCD
    int act, aux_f32, aux_deriv;             // aux receives the pre-activation in bf16, or in float, or sigma' of it in float
};
struct FewBatch {
    FewProduct p[2];
    int first_wg;            // of the second product
    int count;
};

template <int ROWS>
__global__ __launch_bounds__(FEW_WAVES * 64) void few_rows_kernel(FewBatch batch)
{
    constexpr int AHEAD = few_ahead(ROWS), NL = ROWS + 1, CHUNK = NL * 1024;           // bytes of a chunk's operands
    extern __shared__ __attribute__((aligned(16))) unsigned char few_lds[];
    const bool second = batch.count > 1 && (int)blockIdx.x >= batch.first_wg;
    const FewProduct &P = second ? batch.p[1] : batch.p[0];
    const int id = (int)blockIdx.x - (second ? batch.first_wg : 0);
    const int tm = id / P.pitch, tn = id - tm * P.pitch;
    if (tn >= P.tiles_n) return;                       // uniform
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int m0 = tm * (ROWS * FEW_TILE), n0 = tn * FEW_TILE;
    // A load covers 64 bytes of 16 rows: lane l row l / 4 and vector (l & 3) ^ (l >> 4), so that the operand reads of 16 rows at one vector fall on
    // different banks.  Rows past the end repeat the last one and are not stored; reduction indices past the end are cleared below.
    // All element offsets fit 32 bits (checked on the host).
    const int row = lane >> 2, col = ((lane & 3) ^ (lane >> 4)) * 8, b_row = min(n0 + row, P.N - 1);
    int a_row[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) a_row[r] = min(m0 + r * FEW_TILE + row, P.M - 1);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)few_lds + wave * (AHEAD * CHUNK);

    const int chunks = (P.K + 31) >> 5;
    const int first = chunks * wave / FEW_WAVES, count = chunks * (wave + 1) / FEW_WAVES - first;
    auto fetch = [&](int i, uint32_t to) {             // chunk first + i
        const int c = min((first + i) * 32 + col, P.K - 8);
        const bool tail = c >= P.split;
        const uint32_t t = tail ? (uint32_t)(c - P.split) : 0u, seg = __umulhi(t, P.magic), w = t - seg * (uint32_t)P.seg;
        const uint32_t ld = tail ? P.seg : P.split;
        const __bf16 *a = (tail ? P.a1 : P.a0) + (tail ? seg * (uint32_t)P.a_seg + w : (uint32_t)c);
        const __bf16 *b = (tail ? P.b1 : P.b0) + (tail ? seg * (uint32_t)P.b_seg + w : (uint32_t)c);
        ring_load<0>(b + (uint32_t)b_row * ld, to);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) ring_load<0>(a + (uint32_t)a_row[r] * ld, to + 1024 + r * 1024);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (i < count) fetch(i, lds0 + i * CHUNK);     // uniform
    const int n = n0 + (lane & 15);
    f32x4 acc[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    // operand of a lane: row lane & 15, reduction indices 8 (lane >> 4) .. + 7 of the chunk
    const uint32_t at = (lane & 15) * 64 + (((lane >> 4) ^ ((lane >> 2) & 3)) << 4);
    uint32_t slot = lds0;
    for (int i = 0; i < count; ++i) {                  // uniform
        ring_landed<NL, AHEAD - 1>(count - 1 - i);
        bf16x8 b = *lds_at<const bf16x8>(slot + at), a[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) a[r] = *lds_at<const bf16x8>(slot + at + 1024 + r * 1024);
        if ((first + i + 1) * 32 > P.K && (first + i) * 32 + (lane >> 4) * 8 >= P.K) {
#pragma unroll
            for (int e = 0; e < 8; ++e) b[e] = (__bf16)0.f;
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int e = 0; e < 8; ++e) a[r][e] = (__bf16)0.f;
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r], b, acc[r], 0, 0, 0);
        if (i + AHEAD < count) {                       // uniform; the slot's operands are in registers
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fetch(i + AHEAD, slot);
        }
        slot = slot + CHUNK == lds0 + AHEAD * CHUNK ? lds0 : slot + CHUNK;
    }
    const float bias = P.bias ? (float)gload<__bf16>(P.bias + min(n, P.N - 1)) : 0.f;

    // accumulator e of lane l is element (row 4 (l >> 4) + e, column l & 15) of its block.  A wavefront's sums lie over its own operands.
    float *const part = (float *)few_lds;
    constexpr int PART = AHEAD * CHUNK / 4;            // floats from a wavefront's sums to the next one's
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[wave * PART + (r * 4 + e) * 64 + lane] = acc[r][e];
    __syncthreads();
#pragma unroll
    for (int o = 0; o < (ROWS * 4 + FEW_WAVES - 1) / FEW_WAVES; ++o) {
        const int q = o * FEW_WAVES + wave, m = m0 + (q >> 2) * FEW_TILE + 4 * (lane >> 4) + (q & 3);       // q: uniform per wavefront
        if (ROWS * 4 % FEW_WAVES && q >= ROWS * 4) break;
        if (m >= P.M || n >= P.N) continue;
        float x = 0.f;
#pragma unroll
        for (int w = 0; w < FEW_WAVES; ++w) x += part[w * PART + q * 64 + lane];
        const int64_t to = (int64_t)m * P.N + n;
        if (P.bias) {                                  // uniform
            const float pre = x + bias;
            float deriv = 1.f;
            x = pre;
            if (P.act == ACT_GELU) gelu_both(pre, x, deriv);
            else if (P.act == ACT_RELU) { x = pre > 0.f ? pre : 0.f; deriv = pre > 0.f ? 1.f : 0.f; }
            if (P.aux && (P.aux_deriv || P.aux_f32)) gstore<float>((float *)P.aux + to, P.aux_deriv ? deriv : pre);
            else if (P.aux) gstore<__bf16>((__bf16 *)P.aux + to, (__bf16)pre);
        }
        gstore<__bf16>((__bf16 *)P.out + to, (__bf16)x);
    }
}

}  // namespace phantom
