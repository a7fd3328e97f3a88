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

// Does a layer's forward pass (one rank, bf16, 8 divides the widths and phantom widths) run on the kernel for few rows (few_rows.h), and how many blocks
// of 16 rows does a workgroup take?  0: no.  Kc: the update's reduction; k = 0: dense.
// The fewest with which the launch is one round of workgroups, while a workgroup's operands (16 columns and those rows by the reduction) are
// not so long that gemm_flex.h, whose larger tiles read less, is the faster one.  Measured, us, 6 layers forward (dense: 4), gemm_flex.h : 1 block : 2 : 4:
// 1024 + 448 at batch 48 / 96 / 128 46.4 : 36.3 : 39.4 : 43.6, 48.5 : 64.6 : 41.6 : 45.8, 49.3 : 85 : 63.5 : 48.1; 1024 + 1792 at 32 / 96 / 128 67.1 : 54.4 : 61.3 : 64.8,
// 67.6 : 98.6 : 59.8 : 68.7, 67.9 : 116 : 81.4 : 72.0; 512 + 960 at 96 / 192 47.2 : 36.2 : 39.0 : 43.3, 48.7 : 67 : 42.8 : 47.9; 512 + 3840 at 64 / 128 75.8 : 70.5 : 81.9 : 103,
// 76.2 : 83.6 : 81.6 : 102; 256 + 48 at 384 / 768 36.3 : 37.9 : 26.6 : 27.4, 36.3 : 63.5 : 41.1 : 31.0; 1280 + 280 at 40 / 96 59.9 : 56.6 : 43.6 : 47.9, 62.3 : 83.5 : 64.1 : 50.4;
// 2048 + 224 at 32 / 48 59.8 : 80 : 54.5 : 56.7, 59.2 : 87 : 83 : 60.9; 2048 + 1024 at 32 63.1 : 91 : 64.3 : 67.9; dense 512 at 128 21.9 : 16.2 : 17.1 : 19.9, 1024 at 64 / 128
// 27.5 : 20.7 : 22.3 : 25.2, 27.8 : 35 : 23.6 : 25.8, 2048 at 32 / 64 / 128 34.8 : 31.4 : 33.1 : 34.7, 35.3 : 55 : 35.3 : 39.2, 36.0 : 103 : 62 : 41.8, 2560 at 16 34.0 : 36.5 : 37.1 : 39.3,
// 4096 at 16 44.2 : 49.0 : 50.9 : 55.9.
inline int few_rows_blocks_for(int64_t B, int64_t so, int64_t k, int64_t Kc)
{
    const int64_t rows = (B + 15) / 16, columns = (so + 15) / 16 + (k + 15) / 16;
    for (int blocks = 1; blocks <= 4; blocks *= 2)
        if ((rows + blocks - 1) / blocks * columns <= 256) return (blocks + 1) * Kc <= (k > 0 ? 9000 : 6144) && (k > 0 || Kc <= 2048) ? blocks : 0;
    return 0;
}

}  // namespace phantom
