// Which kernel a launch takes, where sizes alone decide it: plain arithmetic without HIP, so that a test can compile it by itself and see
// which kernels its cases reach.
#pragma once
#include <cstdint>

namespace phantom {

constexpr int F32_FEW_TERMS = 16, F32_FEW_GROUPS = 4;  // terms of a group; a team's groups, at most

// Does an fp32 launch run on gemm_flex_f32_few_kernel, and how many groups of 16 terms does each of its eight teams take?  0: no.  4 divides the
// widths and phantom widths; workgroups: the launch's tiles of 32 x 32, over all ranks held; longest: its longest reduction.
// Up to one workgroup to a compute unit with four groups (150 KB of LDS), two with one or two.  Trained, us a step, never : up to 128 workgroups : 256 : 512 with any
// number of groups: 4 layers of 8 ranks of 512 + 224 at batch 1024 (the compressions) 836 : 837 : 810 : 809; 3 of 8 of 128 + 112 at 256 121 : 118 : 92 : 90, of 4 of
// 256 + 96 at 256 155 : 139 : 116 : 107; 2 of 8 of 256 + 224 at 128 110 : 101 : 77 : 77, of 16 of 64 + 120 at 512 98 : 91 : 81 : 75, of 4 of 64 + 24 at 64 54.8 : 42.8 : 42.9 :
// 42.8; 4 of 4 of 96 + 72 at 333 164 : 150 : 118 : 118.  Up to 1024: 2 of 4 of 400 + 60 at 512 134.7 (512) : 198, of 16 of 256 + 120 at 256 114 : 164.
inline int f32_few_groups_for(int64_t workgroups, int64_t longest)
{
    if (longest > 8 * F32_FEW_TERMS * F32_FEW_GROUPS) return 0;
    const int groups = longest <= 8 * F32_FEW_TERMS ? 1 : longest <= 16 * F32_FEW_TERMS ? 2 : 4;
    return workgroups <= (groups <= 2 ? 512 : 256) ? groups : 0;
}

constexpr int FEW_SHORT = 960;                         // few_rows.h: reductions below it in two teams, ...
constexpr int64_t few_short_lds(int blocks, int64_t Kc) { return (Kc + 63) / 64 * 2 * (blocks + 1) * 1024 + 2 * blocks * 1024; }    // bytes of a workgroup's LDS, in two teams
inline bool few_rows_in_eight_teams(int64_t Kc) { return Kc >= FEW_SHORT || Kc == 512; }      // ... others, and this one, in eight (as the tiles of gemm_flex.h)

// Does a layer's forward pass (one rank, bf16, 8 divides the widths and phantom widths) run on the kernel for few rows (few_rows.h), and how many blocks
// of 16 rows does a workgroup take?  0: no.  Kc: the update's reduction; k = 0: dense.
// The fewest with which the launch is one round of workgroups, while a workgroup's operands (16 columns and those rows by the reduction) are
// not so long that gemm_flex.h, whose larger tiles read less, is the faster one.  With eight teams a workgroup has a compute unit for itself, and one round
// means 32 on every XCD, each of which takes every eighth column of either product: 1280 + 280 at batch 40 / 96 with 33 on some of them 55.8, 64.2 us; 43.2,
// 48.2 with one step more (gemm_flex.h 60.0, 62.6).  So does one with two teams and more than half of the LDS; but there the compression may be in a second
// round, where its reduction (the shard) is the shorter one.  gemm_flex.h : 4 blocks, us a layer forward, updates + compressions on the fullest XCD: 288 + 480 at batch 728
// (36 + 12) 7.97 : 9.28 (trained, 7 layers, 125 : 133.5), 392 + 240 at 542 (36 + 9) 8.03 : 9.23, 144 + 672 at 1078 (34 + 17) 8.91 : 11.45, 312 + 600 at 662 (33 + 11) 9.13 : 10.24, 536 + 24 at
// 408 (35 + 7) 7.67 : 8.13; 200 + 744 at 791 (26 + 13) 9.14 : 7.14, 288 + 392 at 637 (30 + 10) 7.97 : 7.77, 352 + 248 at 524 (27 + 9) 8.01 : 6.31; with a long one 704 + 120 at 257 (30 + 5)
// 8.16 : 8.31 (trained, 6 layers, 109.4 : 111.7), 496 + 56 at 493 (32 + 8) 7.68 : 7.78, and 400 + 120 at 476 (32 + 8), the line, 7.87 : 7.45.
// Measured, us, 6 layers forward (dense: 4), gemm_flex.h : 1 block : 2 : 4:
// 1024 + 448 at batch 48 / 96 / 128 46.4 : 36.7 : 39.8 : 43.3, 48.6 : 64.6 : 42.1 : 45.2, 49.2 : 84 : 63.7 : 46.7; 1024 + 1792 at 32 / 96 / 128 66.7 : 52.5 : 58.9 : 61.5,
// 67.9 : 95.9 : 59.9 : 64.8, 68.0 : 114 : 82.3 : 67.2; 512 + 960 at 96 / 192 48.6 : 36.8 : 39.6 : 43.5, 50.0 : 67.3 : 44.0 : 47.1; 512 + 3840 at 64 / 128 76.1 : 68.8 : 77.5 : 94.1,
// 76.3 : 79.8 : 78.6 : 93.1; 256 + 56 at 48 / 384 / 768 39.1 : 25.2 : 27.0 : 29.4, 40.7 : 27.9 : 27.4 : 30.2, 40.6 : 33.4 : 30.4 : 31.0; 512 + 336 at 96 51.6 : 31.9 : 33.4 : 36.6;
// 2048 + 224 at 32 / 48 60.0 : 81.0 : 55.7 : 55.8, 59.4 : 88.9 : 85.0 : 58.9; 2048 + 1024 at 32 63.5 : 94.6 : 69.7 : 71.4; dense 512 at 128 / 512 23.5 : 17.9 : 19.0 : 21.8, 24.0 : 44.9 :
// 29.3 : 23.3, 1024 at 64 / 128 / 256 26.5 : 22.3 : 23.5 : 26.3, 26.9 : 35.0 : 24.7 : 26.5, 29.0 : 64.2 : 40.7 : 28.1, 2048 at 32 35.0 : 32.7 : 34.0 : 34.8, 2560 at 16 33.7 : 36.8 : 37.2 : 39.3.
// Dense reductions of three and four times 512 load the eight teams of gemm_flex.h evenly, and with two blocks or more it is the faster one: 1472 / 1536 / 1600 at 64
// 31.7 : 28.7 (2 blocks), 28.2 : 28.8, 37.6 : 30.7; 1984 / 2048 39.6 : 34.7, 35.1 : 37.8.
inline int few_rows_blocks_for(int64_t B, int64_t so, int64_t k, int64_t Kc)
{
    const bool eight = few_rows_in_eight_teams(Kc);
    auto on_an_xcd = [](int64_t columns) { return (columns + 127) / 128; };            // workgroups of a row of them, at most
    auto workgroups = [=](int64_t columns) { return eight ? on_an_xcd(columns) * 8 : (columns + 15) / 16; };
    const int64_t rows = (B + 15) / 16, columns = workgroups(so) + workgroups(k);
    for (int blocks = 1; blocks <= 4; blocks *= 2) {
        const int64_t tall = (rows + blocks - 1) / blocks;
        if (tall * columns > 256) continue;
        if (!eight && few_short_lds(blocks, Kc) > 80 * 1024 && !(tall * (on_an_xcd(so) + on_an_xcd(k)) <= 32 || (tall * on_an_xcd(so) <= 32 && 5 * so <= 4 * Kc))) continue;
        if (k > 0) return (blocks + 1) * Kc <= 9000 ? blocks : 0;
        return (blocks + 1) * Kc <= 6144 && Kc <= 2048 && !(blocks > 1 && Kc > 1024 && Kc % 512 == 0) ? blocks : 0;
    }
    return 0;
}

}  // namespace phantom
