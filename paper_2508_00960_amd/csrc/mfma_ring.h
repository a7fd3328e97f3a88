// The reduction loop of the 128 x 128 kernels (gemm_mfma.h) for operands in 16-byte vectors: a ring of LDS stages that
// direct-to-LDS loads fill, read by the matrix cores' operand loads.
//
// What bounds it.  A 128 x 128 x 64 step is 520 clocks of a compute unit's matrix cores; its 32 KB of operands take 570 clocks
// through the vector-memory path (57 bytes a clock, whether they end in registers or in LDS), its 64 KB of operand reads 260 (255
// bytes a clock).  All three run beside each other (570 clocks together); through registers (global -> registers -> LDS, two
// LDS stages) 420 clocks of LDS writes (78 bytes a clock) come on top, 690 together.  Operands that lie in L2: 660 to 830 clocks a
// step at 1.6 GHz, where the chip then runs (power), i.e. 0.43 us; through registers 0.55.  Operands from HBM: 0.57 to 0.67 us
// with either loop and with three, four or five stages: the step then waits for them.
// First stage, loop (clocks, at 2.3 GHz, before : now): layer update 1024 x 512 x 736 on 8 ranks 5000 + 15600 : 4050 + 12900; error
// compression 1024 x 224 x 512 5400 + 11950 : 3700 + 9500; 8 layers' weight gradients 1024 x 1984 x 4096 7900 + 102700 : 5500 + 94200.
// Passes (us): 4 x 4096, 8 ranks, gradients 247.7 : 233.6; widths 4096 / 8192 415 : 385; 6 layers of 1024, k 256, forward 359 : 352;
// 8 layers of 1024, k 64, trained at batch 4096 698 : 695; dense 4 x 4096 624 : 605.
//
// What stands between that and a step: whatever a wavefront waits for holds up its matrix instructions, and the two wavefronts of a SIMD wait for the same
// things.  All loads of a stage issued behind the barrier fill the queue of the vector-memory path for 570 clocks; four operand reads in a row, issued by
// eight wavefronts at once, return later than the four matrix instructions ahead of them end; every address worked out in between is an instruction the
// matrix cores wait for.  So a step is a straight piece of code: one operand read ahead of each matrix instruction, the loads of a regular shape one by one
// behind them, from a scalar base that moves by a constant for a run of tiles (RingCursor).  Bare products (us, operands and loads in bunches :
// so): 8192 x 1024 x 2816 in two-tile workgroups 50.8 : 44.6, x 5632 96 : 88; 4096 x 1024 x 1984 two teams to a tile 22.5 : 20.0; input-gradient layout 8192 x 1024 x
// 2048 39.3 : 33.5, 1024 x 4096 x 4096 41 : 35; weight gradients 8192 x 1024 over 4096 rows 71 : 60, 4096 x 4096 over 2048 in one-team workgroups 77 : 70.
// Matrix instructions alone take 61 of the 96.
// Steps (us, before : now): 6 layers of 1024 + 1792 forward at batch 8192 338 : 311, of 1024 + 28 165 : 159, 8 of 1024 + 960 with GELU trained at 4096 576 : 546,
// dense 4 x 4096 at 1024 501 : 479, gradients of 8 ranks of 512 + 224 at 1024 208 : 200.
//
// A stage holds one step of 64 of both operands.  The loads of a stage are issued RING - 1 steps before it is read, by all
// wavefronts that read it; each step has one barrier, placed before its last quarter of matrix instructions, and by then every
// wavefront has read its operands of the stage into registers, so that the freed slot is filled again right behind the barrier and the
// first operands of the next stage are read under the last quarter.
//
// LDS layout.  A wavefront's load instruction writes 64 consecutive vectors of 16 bytes: 8 rows of 64 reduction indices (LD_KC) or 4
// rows of 128 free indices (LD_KM), rows without padding.  The vectors of a row are permuted by the row's number, on the
// global side of the load, such that the operand reads fall on different banks:
//   LD_KC  vector v of row r sits at v ^ ((r >> 1) & 7): 16 rows at one v cover all 64 banks;
//   LD_KM  vector v of row r sits at v ^ 4 (r & 3) ^ 2 ((r >> 3) & 1): a transposing read takes 4 rows x 4 vectors.  (Rows of
//          64 free indices, half as long: 4 ((r >> 1) & 1) in the place of 4 (r & 3).)
//
// The loads are inline assembly: the compiler, which would wait for all of them before any LDS read, does not know about them, and
// every wait for them is written out (ring_wait).  Its own waits for other loads can only come out longer.
#pragma once
#include "common.h"
#include "epilogue.h"
#include "views.h"

#include <type_traits>

namespace phantom {

enum { LD_KC = 0, LD_KM = 1 };

constexpr int MT = 128;               // tile rows (m) and columns (n)
constexpr int KT = 64;                // reduction step
constexpr int RING_TILE = MT * KT * 2;       // bytes of one operand's tile in a stage

// Tile rows = free index r in [r0, r0 + TILE), columns = reduction index c in [c0, c0 + 64) (LD_KC), or rows = c, columns = r
// (LD_KM), staged by WAVES wavefronts: NV loads each.  TILE: 128, or 64 (gemm_flex.h).
template <int KIND, int WAVES, int TILE = MT>
struct RingCfg {
    static constexpr int PER_ROW = (KIND == LD_KC ? KT : TILE) / 8;   // vectors per row
    static constexpr int ROWS = KIND == LD_KC ? TILE : KT;
    static constexpr int NV = ROWS * PER_ROW / 64 / WAVES;
    static constexpr int ROW_STEP = 64 / PER_ROW * WAVES;             // from a wavefront's load to its next one (a multiple of 16:
    static_assert(NV >= 1 && ROW_STEP % 16 == 0, "");                 //   the permutation of the row's vectors stays the same)
};

template <int KIND, int TILE = MT> __device__ __forceinline__ int ring_swizzle(int row)
{
    if (KIND == LD_KC) return (row >> 1) & 7;
    return (TILE == MT ? 4 * (row & 3) : 4 * ((row >> 1) & 1)) ^ (2 * ((row >> 3) & 1));
}

// What a thread's loads of one operand share.  The reduction index may decide the region (LD_KC: head block / peer segments; LD_KM:
// head block / one tail block, [L ; C] stacked); otherwise the free index may (LD_KM, fixed per thread).
// All element offsets inside a group fit 32 bits (checked on the host).
struct RingOperand {
    const __bf16 *base0, *base1;
    int col, row0;           // this thread's vector column (elements) and first row inside the tile
    int c_lim;
    int c_decides, c_split, c_seg, c_skip;   // c_split: INT_MAX where c does not decide
    unsigned c_magic;        // ceil(2^32 / c_seg)
    int c_mult0, c_mult1, c_seg_stride;
    int r_region;            // LD_KM: region of the thread's fixed free index (-1: the reduction index decides)
    // "regular" shapes: a 64-wide step of the reduction index never straddles the head / tail boundary, and a peer segment either
    // holds whole steps or a whole number of segments fills a step (n/p a multiple of 64; k a divisor or a multiple of 64).
    // Then the region is the same for the whole workgroup in every step, a load takes a scalar base and one 32-bit offset per
    // thread, and a step's addresses cost a few scalar instructions.  Other shapes work out a 64-bit address per thread.
    bool regular;
    int col_seg, col_in_seg; // LD_KC regular, k < 64: segment and position of the thread's column inside a step
};

// off0[j], off1[j]: byte offsets of the thread's j-th vector that do not depend on the step, in region 0 and region 1.
// LD_KC: row * row stride, in region 0 with the vector's column.  LD_KM: fixed free-index offset + row * c stride.
// Rows (columns) past the end of the free index (r_axis, r_limit) read the last valid one; what they produce lands in outputs the
// epilogue never writes.  Fills in what of s does not come from the reduction index.
template <int KIND, int WAVES, int TILE>
__device__ __forceinline__ void ring_place(RingOperand &s, const Axis &r_axis, int r0, int r_limit, int wave, int lane,
                                           uint32_t (&off0)[RingCfg<KIND, WAVES, TILE>::NV], uint32_t (&off1)[RingCfg<KIND, WAVES, TILE>::NV])
{
    typedef RingCfg<KIND, WAVES, TILE> C;
    s.row0 = wave * (64 / C::PER_ROW) + lane / C::PER_ROW;
    s.col = ((lane % C::PER_ROW) ^ ring_swizzle<KIND, TILE>(s.row0)) * 8;
    s.r_region = -1;
    s.col_seg = 0; s.col_in_seg = s.col;
    if (KIND == LD_KC) {
        s.regular = !s.c_decides || (s.c_split % KT == 0 && (KT % s.c_seg == 0 || s.c_seg % KT == 0));
        if (s.regular && s.c_decides && s.c_seg < KT) {
            s.col_seg = (int)__umulhi((unsigned)s.col, s.c_magic);
            s.col_in_seg = s.col - s.col_seg * s.c_seg;
        }
#pragma unroll
        for (int j = 0; j < C::NV; ++j) {
            const unsigned r = (unsigned)min(r0 + s.row0 + j * C::ROW_STEP, r_limit - 1);
            off0[j] = (r * (unsigned)r_axis.mult0 + (unsigned)s.col) * 2u;
            off1[j] = r * (unsigned)r_axis.mult1 * 2u;
        }
    } else {
        // the region of the free index is the same for the whole tile unless the tile straddles the split
        const bool r_uniform = !r_axis.decides || r0 + TILE <= r_axis.split || r0 >= r_axis.split;
        s.regular = r_uniform && (!s.c_decides || s.c_split % KT == 0);
        const int r = min(r0 + s.col, r_limit - 8);
        const Loc lr = locate(r_axis, r, s.c_skip);
        s.r_region = lr.region;
        // one region for the whole kernel (the usual case): fold the choice into base0 / off0 / c_mult0
        const bool fold = s.regular && !s.c_decides && __builtin_amdgcn_readfirstlane(lr.region) > 0;
        if (fold) { s.base0 = s.base1; s.c_mult0 = s.c_mult1; }
#pragma unroll
        for (int j = 0; j < C::NV; ++j) {
            const unsigned cj = (unsigned)(s.row0 + j * C::ROW_STEP);
            off1[j] = ((unsigned)lr.off1 + cj * (unsigned)s.c_mult1) * 2u;
            off0[j] = fold ? off1[j] : ((unsigned)lr.off0 + cj * (unsigned)s.c_mult0) * 2u;
        }
    }
}

template <int KIND, int WAVES>
__device__ __forceinline__ RingOperand ring_init(const View &v, int g, int r0, int r_limit, int c_limit, int wave, int lane,
                                                 uint32_t (&off0)[RingCfg<KIND, WAVES>::NV], uint32_t (&off1)[RingCfg<KIND, WAVES>::NV])
{
    RingOperand s;
    s.base0 = (const __bf16 *)v.p0 + g * v.g0;
    s.base1 = (const __bf16 *)v.p1 + g * v.g1;
    s.c_lim = c_limit;
    s.c_decides = v.c.decides;
    s.c_split = v.c.decides ? v.c.split : 0x7fffffff;
    s.c_seg = v.c.seg; s.c_skip = v.skip0 + g * v.skip_g;
    s.c_magic = v.c.magic;                           // (never used with seg == 1: 8 divides seg)
    s.c_mult0 = (int)v.c.mult0; s.c_mult1 = (int)v.c.mult1; s.c_seg_stride = (int)v.c.seg_stride;
    ring_place<KIND, WAVES, MT>(s, v.r, r0, r_limit, wave, lane, off0, off1);
    return s;
}

// A value that is the same in every lane, in scalar registers (out of them, the compiler keeps some such values in vector registers).
__device__ __forceinline__ uint32_t ring_uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ const __bf16 *ring_uniform(const __bf16 *p)
{
    const uint64_t v = (uint64_t)(uintptr_t)p;
    return (const __bf16 *)(uintptr_t)((uint64_t)ring_uniform((uint32_t)(v >> 32)) << 32 | ring_uniform((uint32_t)v));
}

// 64 lanes x 16 bytes from base + off (bytes) of each lane to the LDS address lds_at + AHEAD (uniform) + 16 * lane.
// A base that a vector instruction brought to scalar registers (v_readfirstlane, the reload of a spilled one) must be five wait states old,
// which the compiler sees to for its own loads alone: the build looks for such a distance in the finished code (build.py,
// missing_wait_states) and fails on one.  A scalar move of the base inside the statement would do without the check; with one per load 8 layers
// of 1024 trained at batch 4096 took 703 us for 688, with one per step and operand layers of 1408 at 158 47.5 for 46.8.
// (The compiler reserves M0 and warns that it will not keep a value in it across the statements, which is what naming it is for.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int AHEAD> __device__ __forceinline__ void ring_load(const __bf16 *base, uint32_t off, uint32_t lds_at)
{
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(ring_uniform(lds_at)), "v"(off), "s"(ring_uniform(base)), "n"(AHEAD) : "memory", "scc", "m0");
}
template <int AHEAD> __device__ __forceinline__ void ring_load(const __bf16 *p, uint32_t lds_at)
{
    asm volatile("s_add_u32 m0, %0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(ring_uniform(lds_at)), "v"(p), "n"(AHEAD) : "memory", "scc", "m0");
}
#pragma clang diagnostic pop
// f(std::integral_constant<int, j>) for j = J .. N - 1
template <int N, int J = 0, typename F> __device__ __forceinline__ void ring_each(F &&f)
{
    if constexpr (J < N) {
        f(std::integral_constant<int, J>{});
        ring_each<N, J + 1>(static_cast<F &&>(f));
    }
}

// The loads of the tile whose reduction index starts at c0 (uniform), to the LDS address tile (uniform).  A step that reaches past the
// end of the reduction range reads the last valid index in the place of what lies behind it; ring_zero then clears those vectors.
// With one wavefront to a SIMD every instruction here is in the way of the loop: a step inside the head block of a regular shape, which is
// most of them, takes a base pointer and nothing else.
template <int KIND, int WAVES, int TILE = MT>
__device__ __forceinline__ void ring_fetch(const RingOperand &s, const uint32_t (&off0)[RingCfg<KIND, WAVES, TILE>::NV],
                                           const uint32_t (&off1)[RingCfg<KIND, WAVES, TILE>::NV], int c0, uint32_t tile, int wave)
{
    typedef RingCfg<KIND, WAVES, TILE> C;
    constexpr int STRIDE = WAVES * 1024;
    tile += wave * 1024;
    if (s.regular && c0 + KT <= s.c_lim) {             // uniform
        if (c0 < s.c_split) {
            const __bf16 *base = s.base0 + (KIND == LD_KC ? (unsigned)c0 : (unsigned)c0 * (unsigned)s.c_mult0);
            ring_each<C::NV>([&](auto j) { ring_load<j * STRIDE>(base, off0[j], tile); });
        } else if (KIND == LD_KC) {
            const unsigned t0 = (unsigned)(c0 - s.c_split);
            const unsigned i0 = __umulhi(t0, s.c_magic);          // first segment the step touches (scalar unit)
            const int rem = (int)(t0 - i0 * (unsigned)s.c_seg);   // 0 unless a segment holds several steps
            const int i = (int)i0 + s.col_seg;
            const int slot = i + (i >= s.c_skip ? 1 : 0);
            const unsigned add = (unsigned)(slot * s.c_seg_stride + rem + s.col_in_seg) * 2u;
            ring_each<C::NV>([&](auto j) { ring_load<j * STRIDE>(s.base1, off1[j] + add, tile); });
        } else {
            const __bf16 *base = s.base1 + (unsigned)(c0 - s.c_split) * (unsigned)s.c_mult1;
            ring_each<C::NV>([&](auto j) { ring_load<j * STRIDE>(base, off1[j], tile); });
        }
        return;
    }
    if (KIND == LD_KC) {
        const int c = max(0, min(c0 + s.col, s.c_lim - 8));
        const bool reg1 = c >= s.c_split;
        const unsigned t = reg1 ? (unsigned)(c - s.c_split) : 0u;
        const unsigned i = __umulhi(t, s.c_magic);
        const int w = (int)(t - i * (unsigned)s.c_seg);
        const int slot = (int)i + ((int)i >= s.c_skip ? 1 : 0);
        const int64_t base = (int64_t)(uintptr_t)(reg1 ? s.base1 : s.base0) + (int64_t)(reg1 ? slot * s.c_seg_stride + w : c - s.col) * 2;
        ring_each<C::NV>([&](auto j) {
            const uint32_t o0 = off0[j], o1 = off1[j];
            ring_load<j * STRIDE>((const __bf16 *)(uintptr_t)(base + (reg1 ? o1 : o0)), tile);
        });
    } else {
        ring_each<C::NV>([&](auto j) {
            const int cj = s.row0 + j * C::ROW_STEP, c = max(0, min(c0 + cj, s.c_lim - 1));
            const bool reg1 = s.c_decides ? c >= s.c_split : s.r_region > 0;
            const uint32_t o0 = off0[j], o1 = off1[j];
            const int64_t rows = reg1 ? (int64_t)(c - cj - (s.c_decides ? s.c_split : 0)) * s.c_mult1 : (int64_t)(c - cj) * s.c_mult0;
            ring_load<j * STRIDE>((const __bf16 *)(uintptr_t)((int64_t)(uintptr_t)(reg1 ? s.base1 : s.base0) + (reg1 ? o1 : o0) + rows * 2), tile);
        });
    }
}

// Where a regular shape's loads of full tiles come from, as the reduction range is walked down: a scalar base, and offsets of the thread that stay the
// same for a run of tiles, in which the base moves by the same amount from tile to tile.
template <int KIND, int WAVES, int TILE = MT>
struct RingCursor {
    const __bf16 *base;
    uint32_t off[RingCfg<KIND, WAVES, TILE>::NV];
    uint32_t step;           // bytes from a tile to the next lower one
    int left;                // lower tiles of the run
};

// the run that the tile whose reduction index starts at c0 (uniform) begins
template <int KIND, int WAVES, int TILE = MT>
__device__ __forceinline__ void ring_run(RingCursor<KIND, WAVES, TILE> &at, const RingOperand &s, const uint32_t (&off0)[RingCfg<KIND, WAVES, TILE>::NV],
                                             const uint32_t (&off1)[RingCfg<KIND, WAVES, TILE>::NV], int c0)
{
    typedef RingCfg<KIND, WAVES, TILE> C;
    if (c0 < s.c_split) {                              // uniform, like every branch here
        at.left = c0 >> 6;
        at.step = KIND == LD_KC ? KT * 2u : KT * 2u * (uint32_t)s.c_mult0;
        at.base = s.base0 + (KIND == LD_KC ? (unsigned)c0 : (unsigned)c0 * (unsigned)s.c_mult0);
#pragma unroll
        for (int j = 0; j < C::NV; ++j) at.off[j] = off0[j];
    } else if (KIND == LD_KC) {
        const unsigned t0 = (unsigned)(c0 - s.c_split);
        const int i0 = (int)__umulhi(t0, s.c_magic), rem = (int)t0 - i0 * s.c_seg;     // first segment the tile touches; 0 unless a segment holds several tiles
        const int i = i0 + s.col_seg, slot = i + (i >= s.c_skip ? 1 : 0);
        const unsigned add = (unsigned)(slot * s.c_seg_stride + rem + s.col_in_seg) * 2u;
#pragma unroll
        for (int j = 0; j < C::NV; ++j) at.off[j] = off1[j] + add;
        at.base = s.base1;
        // a run ends with its segment, or where segments that a tile holds lie on either side of the skipped slot
        if (s.c_seg > KT) {
            at.left = rem >> 6;
            at.step = KT * 2u;
        } else {
            const int held = (int)__umulhi(KT, s.c_magic);
            at.left = (i0 >= s.c_skip ? (i0 - s.c_skip) * s.c_seg : i0 + held <= s.c_skip ? i0 * s.c_seg : 0) >> 6;
            at.step = (uint32_t)(held * s.c_seg_stride) * 2u;
        }
    } else {
        at.left = (c0 - s.c_split) >> 6;
        at.step = KT * 2u * (uint32_t)s.c_mult1;
        at.base = s.base1 + (unsigned)(c0 - s.c_split) * (unsigned)s.c_mult1;
#pragma unroll
        for (int j = 0; j < C::NV; ++j) at.off[j] = off1[j];
    }
    // (scalar registers from here on: a base that the loop moved there ahead of each load would be too young for it, see ring_load)
    at.base = ring_uniform(at.base);
    at.step = ring_uniform(at.step);
}

typedef __attribute__((address_space(3))) unsigned char *LdsBytes;
template <typename V> __device__ __forceinline__ __attribute__((address_space(3))) V *lds_at(uint32_t at)
{
    return (__attribute__((address_space(3))) V *)(uintptr_t)at;
}

// Clears the thread's own vectors that lie past the end of the reduction range (its loads of the tile have landed).
template <int KIND, int WAVES, int TILE = MT>
__device__ __forceinline__ void ring_zero(const RingOperand &s, int c0, uint32_t tile, int wave, int lane)
{
    typedef RingCfg<KIND, WAVES, TILE> C;
#pragma unroll
    for (int j = 0; j < C::NV; ++j) {
        const int c = KIND == LD_KC ? c0 + s.col : c0 + s.row0 + j * C::ROW_STEP;
        if (c >= s.c_lim) *lds_at<u32x4>(tile + (j * WAVES + wave) * 1024 + lane * 16) = u32x4{0u, 0u, 0u, 0u};
    }
}

// Waits until at most N of this wavefront's vector-memory operations are outstanding.
template <int N> __device__ __forceinline__ void ring_own() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
// Waits until at most N of this wavefront's vector-memory operations and none of its LDS operations are outstanding, then for
// the workgroup's other wavefronts.
template <int N> __device__ __forceinline__ void ring_wait() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory"); }
// The same while the loads of `later` younger stages of NL loads each may be outstanding (uniform)
template <int NL, int MOST> __device__ __forceinline__ void ring_wait_stage(int later)
{
    if constexpr (MOST > 0) {
        if (later >= MOST) ring_wait<MOST * NL>();
        else ring_wait_stage<NL, MOST - 1>(later);
    } else {
        ring_wait<0>();
    }
}
template <int NL, int MOST> __device__ __forceinline__ void ring_landed(int later)
{
    if constexpr (MOST > 0) {
        if (later >= MOST) ring_own<MOST * NL>();
        else ring_landed<NL, MOST - 1>(later);
    } else {
        ring_own<0>();
    }
}

// A lane's place inside an operand tile for the matrix instructions' operand: rows rbase .. rbase + 31 and the first 16 reduction
// indices.  LD_KC: 32 rows further lie 4096 bytes further, sub-step kk is the XOR of kk << 5.  LD_KM: at(32 rows further) is the XOR of
// 64, sub-step kk lies 16 rows further.
template <int KIND, int TILE = MT> __device__ __forceinline__ int ring_lane_at(int rbase, int lane)
{
    if (KIND == LD_KC) {
        const int row = rbase + (lane & 31);
        return row * (KT * 2) + (((lane >> 5) ^ ring_swizzle<KIND>(row)) << 4);
    }
    const int krow = (lane >> 5) * 8 + ((lane & 15) >> 2), col = rbase + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    return krow * (TILE * 2) + (((col >> 3) ^ ring_swizzle<KIND, TILE>(krow)) << 4) + ((col >> 2) & 1) * 8;
}
// block: 0 or 1, 32 rows further; kk: sub-step of 16
template <int KIND, int TILE = MT> __device__ __forceinline__ bf16x8 ring_operand(uint32_t stage, int at, int block, int kk)
{
    if (KIND == LD_KC) return *lds_at<const bf16x8>(stage + (at ^ (kk << 5)) + block * 4096);
    const uint32_t p = stage + (at ^ (block << 6)) + kk * (16 * TILE * 2);
    union { struct { s16x4 a, b; } s; bf16x8 v; } u;
    u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_at<s16x4>(p));
    u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_at<s16x4>(p + 4 * TILE * 2));
    return u.v;
}

}  // namespace phantom
