// A layer's forward products (Eq. (ylq): the update with the peers' part, and the compression beside it) for a batch of few rows, as
// inference at a serving batch has them: bf16, operands in 16-byte vectors, one rank.
//
// What bounds it.  The weights are read once and multiplied by a handful of rows, so a launch is a chain of latencies: parameters, one read of
// the operands, a few matrix instructions, the sum over wavefronts, the epilogue.  The tiles of gemm_flex.h walk the reduction in dependent steps with
// a barrier each, and 32 x 32 of them are too few to occupy the chip: 48 rows of 1024 + 448 make 72 workgroups that read 188 KB each.  Here a workgroup owns 16
// output columns and ROWS x 16 rows, and its eight wavefronts request their shares of the reduction, in chunks of 32 indices, at once.  (Loads of operands in
// the matrix cores' layout, whose neighbouring lanes lie in different rows, run at a quarter of the rate: so they go through LDS.)
//
// The sums are those of the tiles of gemm_flex.h that would take the same products, in the same order, so the same bits: a step's output does not depend on
// whether its last layer forms the output error, too, which those tiles do.  (v_mfma_f32_16x16x32_bf16 adds as two v_mfma_f32_32x32x16_bf16 in a row.)
// TEAMS = 8: every wavefront has the tiles of 64 indices of one of eight teams, loads up to few_ahead chunks ahead to LDS that it alone reads, and meets no
// barrier before the sum over wavefronts.  TEAMS = 2: reductions of less than 960 indices; all of it lies in LDS, and a wavefront per block of rows and
// team adds up every other tile from the last one down, the even and the odd quarters of a tile apart.
// Us a pass, 6 layers forward (gemm_flex.h : contiguous eighths of the reduction to eight wavefronts, other bits : so): 1024 + 448 at batch 48 47.2 : 37.5 : 37.1,
// at 128 50.4 : 48.7 : 47.5, 1024 + 1792 at 32 67.7 : 54.6 : 52.3, 256 + 112 at 48 39.4 : 26.4 : 26.3, 512 + 56 at 48 44.7 : 28.5 : 29.2; a launch of nothing
// else is 4 of the 6 to 8 us a layer of the first.
#pragma once
#include "common.h"
#include "epilogue.h"
#include "launch_rules.h"
#include "mfma_ring.h"

namespace phantom {

constexpr int FEW_WAVES = 8, FEW_TILE = 16;
constexpr int few_ahead(int rows) { return rows == 1 ? 8 : rows == 2 ? 6 : 3; }        // chunks of a wavefront in flight
constexpr int few_chunk_bytes(int rows) { return (rows + 1) * 1024; }
// chunks: of the launch's longest reduction (TEAMS = 2: behind them, the teams' sums)
constexpr int few_lds_bytes(int rows, int teams, int chunks)
{
    return teams == 8 ? FEW_WAVES * few_ahead(rows) * few_chunk_bytes(rows) : (chunks + 1) / 2 * 2 * few_chunk_bytes(rows) + 2 * rows * 1024;
}
static_assert(few_lds_bytes(4, 2, (FEW_SHORT - 1) / 32 + 1) <= 160 * 1024 && few_lds_bytes(2, 8, 0) <= 160 * 1024, "a compute unit's LDS");
static_assert(few_lds_bytes(4, 2, 24) == few_short_lds(4, 768), "as the rule has it");

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
    int chunks;              // of the longest reduction (TEAMS = 2)
};

template <int ROWS, int TEAMS>
__global__ __launch_bounds__(FEW_WAVES * 64) void few_rows_kernel(FewBatch batch)
{
    constexpr int AHEAD = few_ahead(ROWS), NL = ROWS + 1, CHUNK = few_chunk_bytes(ROWS);
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
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)few_lds;
    const int chunks = (P.K + 31) >> 5;
    auto fetch = [&](int chunk, uint32_t to) {
        const int c = min(chunk * 32 + col, P.K - 8);
        const bool tail = c >= P.split;
        const uint32_t t = tail ? (uint32_t)(c - P.split) : 0u, seg = __umulhi(t, P.magic), w = t - seg * (uint32_t)P.seg;
        const uint32_t ld = tail ? P.seg : P.split;
        const __bf16 *a = (tail ? P.a1 : P.a0) + (tail ? seg * (uint32_t)P.a_seg + w : (uint32_t)c);
        const __bf16 *b = (tail ? P.b1 : P.b0) + (tail ? seg * (uint32_t)P.b_seg + w : (uint32_t)c);
        ring_load<0>(b + (uint32_t)b_row * ld, to);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) ring_load<0>(a + (uint32_t)a_row[r] * ld, to + 1024 + r * 1024);
    };
    const int n = n0 + (lane & 15);
    // where vector v (8 reduction indices) of this lane's row lies in an operand of a chunk
    auto vector_at = [lane](int v) { return (uint32_t)((lane & 15) * 64 + ((v ^ ((lane >> 2) & 3)) << 4)); };
    auto clear = [](bf16x8 &v) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (__bf16)0.f;
    };
    float *part;                                       // sums: [team][block of rows][accumulator][lane], `pitch` floats from team to team
    int part_pitch;
    if constexpr (TEAMS == 8) {
        // this wavefront's chunks: 2 w and 2 w + 1, and every 16 further on
        const int count = (chunks >> 4) * 2 + max(0, min((chunks & 15) - 2 * wave, 2));
        auto chunk_of = [wave](int i) { return (i >> 1) * 16 + wave * 2 + (i & 1); };
        const uint32_t mine = lds0 + wave * (AHEAD * CHUNK);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
            if (i < count) fetch(chunk_of(i), mine + i * CHUNK);       // uniform
        f32x4 acc[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
        // operand of a lane: row lane & 15, reduction indices 8 (lane >> 4) .. + 7 of the chunk
        const uint32_t at = vector_at(lane >> 4);
        uint32_t slot = mine;
        for (int i = 0; i < count; ++i) {              // uniform
            ring_landed<NL, AHEAD - 1>(count - 1 - i);
            bf16x8 b = *lds_at<const bf16x8>(slot + at), a[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) a[r] = *lds_at<const bf16x8>(slot + at + 1024 + r * 1024);
            if (chunk_of(i) * 32 + 32 > P.K && chunk_of(i) * 32 + (lane >> 4) * 8 >= P.K) {
                clear(b);
#pragma unroll
                for (int r = 0; r < ROWS; ++r) clear(a[r]);
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r], b, acc[r], 0, 0, 0);
            if (i + AHEAD < count) {                   // uniform; the slot's operands are in registers
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                fetch(chunk_of(i + AHEAD), slot);
            }
            slot = slot + CHUNK == mine + AHEAD * CHUNK ? mine : slot + CHUNK;
        }
        part = (float *)few_lds;                       // over the wavefront's own operands
        part_pitch = AHEAD * CHUNK / 4;
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[wave * part_pitch + (r * 4 + e) * 64 + lane] = acc[r][e];
    } else {
#pragma unroll
        for (int i = 0; i < FEW_SHORT / 32 / FEW_WAVES + 1; ++i)
            if (const int c = wave + i * FEW_WAVES; c < chunks) fetch(c, lds0 + c * CHUNK);    // uniform
        part = (float *)(few_lds + (batch.chunks + 1) / 2 * 2 * CHUNK);
        part_pitch = ROWS * 256;
        ring_wait<0>();                                // everybody's operands
        const int team = wave & 1, r = wave >> 1, tiles = (chunks + 1) >> 1;
        if (r < ROWS) {                                // uniform
            f32x4 acc[2];                              // quarters 0 and 2 of a tile, quarters 1 and 3
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[h] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int tile = tiles - 1 - team; tile >= 0; tile -= 2) {                  // uniform
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int chunk = 2 * tile + (lane >> 5), v = 2 * h + ((lane >> 4) & 1);
                    const uint32_t at = lds0 + chunk * CHUNK + vector_at(v);
                    bf16x8 b = *lds_at<const bf16x8>(at), a = *lds_at<const bf16x8>(at + 1024 + r * 1024);
                    if (chunk * 32 + v * 8 >= P.K) { clear(a); clear(b); }
                    acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[h], 0, 0, 0);
                }
            }
            acc[0] += acc[1];
#pragma unroll
            for (int e = 0; e < 4; ++e) part[team * part_pitch + (r * 4 + e) * 64 + lane] = acc[0][e];
        }
    }
    const float bias = P.bias ? (float)gload<__bf16>(P.bias + min(n, P.N - 1)) : 0.f;

    // accumulator e of lane l is element (row 4 (l >> 4) + e, column l & 15) of its block
    __syncthreads();
#pragma unroll
    for (int o = 0; o < (ROWS * 4 + FEW_WAVES - 1) / FEW_WAVES; ++o) {
        const int q = o * FEW_WAVES + wave, m = m0 + (q >> 2) * FEW_TILE + 4 * (lane >> 4) + (q & 3);       // q: uniform per wavefront
        if (ROWS * 4 % FEW_WAVES && q >= ROWS * 4) break;
        if (m >= P.M || n >= P.N) continue;
        float x = part[q * 64 + lane];
#pragma unroll
        for (int t = 1; t < TEAMS; ++t) x += part[t * part_pitch + q * 64 + lane];
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
