// bf16 x bf16 -> fp32 tiled product on the CDNA4 matrix cores:
//   C(m, n) = sum_c A(m, c) * B(n, c),   A, B and C given as Views (views.h).
//
// One workgroup (512 threads = two teams of 4 wavefronts) owns a 128 x 128 tile of C and walks the
// reduction index in steps of 64 (see reduce_in_ring).  Within a team each wavefront owns a 64 x 64 quadrant = 2 x 2 MFMA tiles
// of v_mfma_f32_32x32x16_bf16, accumulators in registers (64 floats per lane).
//
// Two loader kinds, chosen per operand:
//   LD_KC  the reduction index is contiguous in memory (X, G, L, D in the forward; delta in dX).
//          A lane's MFMA operand is one 16-byte LDS read.
//   LD_KM  the free index is contiguous, the reduction index strides (L, C, D in dX and error
//          compression; delta, X, G in the weight gradients).  The MFMA
//          operand is built by two ds_read_b64_tr_b16 (the gfx950 transposing LDS read: within 16
//          lanes, lanes 4j..4j+3 supply row j of a 4 x 16 block, lane i receives column i).
// The peers' segments (G_i, D_i) are addressed in place through the View; VEC (8 or 4
// elements) is the widest vector that never straddles a segment boundary.
//
// VEC = 8: the stages of a ring in LDS are filled by direct-to-LDS loads (mfma_ring.h).
// VEC = 4: global -> registers -> LDS, two stages per team, padded rows ([128][64 + 8], [64][128 + 32]); the global loads of a
// step are issued two of the team's steps before the step is multiplied.  (A direct-to-LDS load has 4 or 16 bytes per lane.)
//
// Address arithmetic is kept off the vector ALU as far as possible (it competes with the MFMAs for
// issue slots): everything that depends only on the thread is computed once, everything that
// depends only on the reduction step is computed on the scalar unit.
//
// Workgroup ids are re-mapped so that the ids an XCD receives (id mod 8) form a contiguous range
// of tiles: neighbouring tiles share operand panels in that XCD's L2.
//
// An operand's tail block may also be a sum that is formed on read (SumOnRead, fetch_summed): the in-memory
// reduce-scatter of the backward pass as part of the input gradient's loader.
//
// Kernels in this file, all built on mfma_workgroup (one workgroup's work on one product):
//   gemm_mfma_kernel       one product, or two of the same operand layout and output type
//   gemm_mfma_uniform_kernel, gemm_mfma_table_kernel
//                          one rank: the weight + compressor gradients of all layers, with parameter blocks in the kernel
//                          arguments (layers of the same shapes) or in device memory
//   gemm_mfma_many_kernel  one rank: the compressions of all layers, more than 64 phantom neurons
//   gemm_mfma_tail_kernel  weight + compressor gradients with riders of other layouts (the error compression of
//                          the layer below, the loss)
//   gemm_mfma_fwd_kernel   a rank's layer update with the thin compression shared out over its workgroups
#pragma once
#include "common.h"
#include "elementwise.h"    // LossTail
#include "epilogue.h"
#include "mfma_ring.h"
#include "thin_product.h"   // thin_workgroup
#include "views.h"

namespace phantom {

constexpr int KC_PITCH = KT + 8;      // elements per LDS row, K-contiguous tile [128][72]
#ifndef PH_KM_PITCH
#define PH_KM_PITCH (MT + 32)
#endif
// elements per LDS row, K-major tile [64][160]: 80 words = 16 mod 64, so the four rows that 16 lanes of a
// transposing read touch start 16 banks apart and the next 16 lanes (16 columns = 8 banks further) fall between
// them; with 144 the two half-groups met on the same banks (SQ_LDS_BANK_CONFLICT: a quarter of the LDS cycles)
constexpr int KM_PITCH = PH_KM_PITCH;
constexpr int TILE_ELEMS = (MT * KC_PITCH > KT * KM_PITCH) ? MT * KC_PITCH : KT * KM_PITCH;   // one operand stage
constexpr int MFMA_THREADS = 512;       // two teams of four wavefronts
constexpr int MFMA_LDS_BYTES = 2 /*teams*/ * 2 /*stages*/ * 2 /*operands*/ * TILE_ELEMS * 2;

// How a workgroup's teams take output tiles (mfma_workgroup).  TILE_SHARED: both teams one tile, half of the sums
// each.  TILE_DUAL: two tiles, one above the other, with the B tile in common.  TILE_SOLO: one team only, one tile: half
// the threads and half the LDS, so that a compute unit holds two such workgroups.
enum { TILE_SHARED = 0, TILE_DUAL = 1, TILE_SOLO = 2 };
constexpr int mfma_threads(int mode) { return mode == TILE_SOLO ? MFMA_THREADS / 2 : MFMA_THREADS; }
constexpr int mfma_lds_bytes(int mode) { return mode == TILE_SOLO ? MFMA_LDS_BYTES / 2 : MFMA_LDS_BYTES; }

template <int VEC> struct VecOf;           // (vectors of 8 elements go from memory to LDS, mfma_ring.h)
template <> struct VecOf<4> { typedef u32x2 type; };

// a global-memory load that the compiler cannot mistake for a generic (flat) access
template <typename V>
__device__ __forceinline__ V load_global(const __bf16 *p)
{
    return *(const __attribute__((address_space(1))) V *)(uintptr_t)p;
}

// ---- staging one operand tile in 4-element vectors -------------------------------------
// KIND == LD_KC: tile rows = free index r in [r0, r0+128), columns = reduction index c in [c0, c0+64).
//                The reduction index may decide the region (head block / peer segments); r never does.
// KIND == LD_KM: tile rows = reduction index c in [c0, c0+64), columns = free index r in [r0, r0+128).
//                r may decide the region (fixed per thread); c may decide only between a head block
//                and ONE tail block ([L ; C] stacked along the reduction index).
// All element offsets inside a group fit 32 bits (checked on the host).
//
// No load is predicated (predication turns into divergent branches and makes the compiler wait for
// ALL outstanding loads instead of counting them).  Rows past the end of the free index read the
// last valid row; what they produce lands in outputs the epilogue never writes.  A tile that
// reaches past the end of the reduction range takes the slow path: indices are clamped to the last
// valid position and the store zeroes what was loaded for reduction indices >= c_lim.
// PART = 2: the 256 threads of a team stage only half of the tile's rows (the other team stages the
// other half of an operand tile that both teams read; see TILE_DUAL)
template <int KIND, int VEC, int PART = 1>
struct StageCfg {
    typedef typename VecOf<VEC>::type V;
    static constexpr int PER_ROW = (KIND == LD_KC ? KT : MT) / VEC;   // vectors per LDS row
    static constexpr int ROWS = KIND == LD_KC ? MT : KT;
    static constexpr int NV = ROWS * PER_ROW / 256 / PART;            // vectors per thread
    static_assert(NV >= 1 && NV * 256 * PART == ROWS * PER_ROW, "the team's threads tile its share of the rows");
    static constexpr int ROW_STEP = 256 / PER_ROW;
    static constexpr int PITCH = KIND == LD_KC ? KC_PITCH : KM_PITCH;
};

struct StageState {          // scalars only, so that it lives in registers
    const __bf16 *base0, *base1;
    int col, row0;           // this thread's vector column (elements) and first row inside the tile
    int c_lim;
    int c_decides, c_split, c_seg, c_skip;
    unsigned c_magic;        // ceil(2^32 / c_seg)
    int c_mult0, c_mult1, c_seg_stride;
    int r_region;            // LD_KM: region of the thread's fixed free index (-1: the reduction index decides).  PLAIN: folded into
                             // base0, off0 and c_mult0, which then differ from thread to thread
    // "regular" shapes: a 64-wide step of the reduction index never straddles the head / tail boundary,
    // and a peer segment either holds whole steps or a whole number of segments fills a step
    // (n/p a multiple of 64; k a divisor or a multiple of 64).  Then the region is the same for the
    // whole workgroup in every step and the addressing of a full tile is almost free.
    int regular;
    int col_seg, col_in_seg; // LD_KC regular, k < 64: segment and position of the thread's column inside a step
};

// off0[j], off1[j]: element offsets of the thread's j-th vector that do not depend on the step, in
// region 0 and region 1.  LD_KC: row * row stride.  LD_KM: fixed free-index offset + (row0 + j*ROW_STEP) * c stride.
// PLAIN (LD_KM only): the reduction index never decides, as the batch of a weight gradient.  The thread's columns stay in one region, so
// that every tile takes the fast path, also one that straddles the split: widths of which half are no multiples of 64 had such tiles
// in every launch, and these, on the general loop, took twice as long as the others.
template <int KIND, int VEC, int PART = 1, bool PLAIN = false>
__device__ __forceinline__ StageState stage_init(const View &v, int g, int r0, int r_limit, int c_limit, int tid,
                                                 int (&off0)[StageCfg<KIND, VEC, PART>::NV],
                                                 int (&off1)[StageCfg<KIND, VEC, PART>::NV], int row_shift = 0)
{
    typedef StageCfg<KIND, VEC, PART> C;
    StageState s;
    s.base0 = (const __bf16 *)v.p0 + g * v.g0;
    s.base1 = (const __bf16 *)v.p1 + g * v.g1;
    const int skip = v.skip0 + g * v.skip_g;
    s.col = (tid % C::PER_ROW) * VEC;
    s.row0 = tid / C::PER_ROW + row_shift;           // row_shift: first row of this team's share (PART = 2)
    s.c_lim = c_limit;
    s.c_decides = v.c.decides;
    s.c_split = v.c.decides ? v.c.split : 0x7fffffff;
    s.c_seg = v.c.seg; s.c_skip = skip;
    s.c_magic = v.c.magic;                           // the MFMA path never sees seg == 1 (VEC >= 2 divides seg)
    s.c_mult0 = (int)v.c.mult0; s.c_mult1 = (int)v.c.mult1; s.c_seg_stride = (int)v.c.seg_stride;
    s.r_region = -1;
    s.col_seg = 0; s.col_in_seg = s.col;
    if (KIND == LD_KC) {
        s.regular = !v.c.decides || (v.c.split % KT == 0 && (KT % v.c.seg == 0 || v.c.seg % KT == 0));
        if (s.regular && v.c.decides && v.c.seg < KT) {
            s.col_seg = (int)__umulhi((unsigned)s.col, v.c.magic);
            s.col_in_seg = s.col - s.col_seg * v.c.seg;
        }
#pragma unroll
        for (int j = 0; j < C::NV; ++j) {
            const int r = min(r0 + s.row0 + j * C::ROW_STEP, r_limit - 1);
            off0[j] = r * (int)v.r.mult0;
            off1[j] = r * (int)v.r.mult1;
        }
    } else {
        // the region of the free index is the same for the whole tile unless the tile straddles the split
        const bool r_uniform = !v.r.decides || r0 + MT <= v.r.split || r0 >= v.r.split;
        s.regular = r_uniform && (!v.c.decides || v.c.split % KT == 0);
        const int r = min(r0 + s.col, r_limit - VEC);
        const Loc lr = locate(v.r, r, skip);
        s.r_region = lr.region;
        if (PLAIN) {
            const bool tail = lr.region > 0;
            s.regular = 1;
            s.base0 = tail ? s.base1 + lr.off1 : s.base0 + lr.off0;
            s.c_mult0 = tail ? s.c_mult1 : s.c_mult0;
#pragma unroll
            for (int j = 0; j < C::NV; ++j) off0[j] = (s.row0 + j * C::ROW_STEP) * s.c_mult0;
            return s;
        }
        // one region for the whole kernel (the usual case): fold the choice into base0 / off0 / c_mult0
        const bool fold = s.regular && !v.c.decides && __builtin_amdgcn_readfirstlane(lr.region) > 0;
        if (fold) { s.base0 = s.base1; s.c_mult0 = s.c_mult1; }
#pragma unroll
        for (int j = 0; j < C::NV; ++j) {
            const int cj = s.row0 + j * C::ROW_STEP;
            off1[j] = (int)lr.off1 + (v.c.decides ? cj - s.c_split : cj) * s.c_mult1;
            off0[j] = fold ? off1[j] : (int)lr.off0 + cj * s.c_mult0;
        }
    }
    return s;
}

// issue the global loads of vectors J0 .. J1-1 of the tile whose reduction index starts at c0 (any shape).
// CAREFUL = false: the caller guarantees c0 + KT <= c_lim (a full interior tile).
template <int KIND, int VEC, bool CAREFUL, int PART = 1, bool PLAIN = false, int J0 = 0, int J1 = StageCfg<KIND, VEC, PART>::NV>
__device__ __forceinline__ void stage_fetch(const StageState &s, const int (&off0)[StageCfg<KIND, VEC, PART>::NV],
                                            const int (&off1)[StageCfg<KIND, VEC, PART>::NV],
                                            typename VecOf<VEC>::type (&regs)[StageCfg<KIND, VEC, PART>::NV], int c0)
{
    typedef StageCfg<KIND, VEC, PART> C;
    typedef typename C::V V;
    const bool interior = !CAREFUL || c0 + KT <= s.c_lim;   // uniform
    if (KIND == LD_KC) {
        const int c = interior ? c0 + s.col : max(0, min(c0 + s.col, s.c_lim - VEC));
        if (!s.c_decides) {                            // uniform: a plain operand
            const __bf16 *base = s.base0 + c;
#pragma unroll
            for (int j = J0; j < J1; ++j) regs[j] = load_global<V>(base + off0[j]);
        } else {
            const bool reg1 = c >= s.c_split;
            const unsigned t = reg1 ? (unsigned)(c - s.c_split) : 0u;
            const unsigned i = __umulhi(t, s.c_magic);
            const int w = (int)(t - i * (unsigned)s.c_seg);
            const int slot = (int)i + ((int)i >= s.c_skip ? 1 : 0);
            const int coff = reg1 ? slot * s.c_seg_stride + w : c;
            const __bf16 *base = (reg1 ? s.base1 : s.base0) + coff;
#pragma unroll
            for (int j = J0; j < J1; ++j) {
                const int o0 = off0[j], o1 = off1[j];
                regs[j] = load_global<V>(base + (reg1 ? o1 : o0));
            }
        }
    } else {
#pragma unroll
        for (int j = J0; j < J1; ++j) {
            const int cj = s.row0 + j * C::ROW_STEP;
            const int c = interior ? c0 + cj : max(0, min(c0 + cj, s.c_lim - 1));
            if (PLAIN) {
                regs[j] = load_global<V>(s.base0 + (int64_t)c * s.c_mult0);
                continue;
            }
            const bool reg1 = s.c_decides ? (c >= s.c_split) : (s.r_region > 0);
            const int o0 = off0[j], o1 = off1[j];
            const int off = reg1 ? o1 + (c - cj) * s.c_mult1 : o0 + (c - cj) * s.c_mult0;
            regs[j] = load_global<V>((reg1 ? s.base1 : s.base0) + off);
        }
    }
}

// whether stage_init would call the tile whose free index starts at r0 regular (same predicate, no state)
template <int KIND, bool PLAIN = false>
__device__ __forceinline__ bool tile_is_regular(const View &v, int r0)
{
    if (PLAIN) return true;
    if (KIND == LD_KC) return !v.c.decides || (v.c.split % KT == 0 && (KT % v.c.seg == 0 || v.c.seg % KT == 0));
    const bool r_uniform = !v.r.decides || r0 + MT <= v.r.split || r0 >= v.r.split;
    return r_uniform && (!v.c.decides || v.c.split % KT == 0);
}

// ---- the fast path: regular shapes, full interior tiles ----------------------------------
// What a step's loads share: a base pointer that is the same for the whole workgroup (it lives in
// scalar registers and the load takes it as its scalar base), which of the two offset arrays
// applies, and one 32-bit term added to every offset.  No branch, no clamp, no 64-bit vector math.
struct FastStep {
    const __bf16 *base;
    bool tail;          // uniform: offsets come from off1
    unsigned add;
};

template <int KIND, int VEC, bool PLAIN = false>
__device__ __forceinline__ FastStep fast_step_addr(const StageState &s, int c0 /* uniform, multiple of KT */)
{
    FastStep f;
    if (PLAIN) {
        f.base = s.base0 + (int64_t)c0 * s.c_mult0;    // (per thread)
        f.tail = false;
        f.add = 0;
        return f;
    }
    const bool head = c0 < s.c_split;                  // c_split = INT_MAX when c does not decide
    if (KIND == LD_KC) {
        const unsigned t0 = head ? 0u : (unsigned)(c0 - s.c_split);
        const unsigned i0 = __umulhi(t0, s.c_magic);   // first segment the step touches (scalar unit)
        const int rem = (int)(t0 - i0 * (unsigned)s.c_seg);   // 0 unless a segment holds several steps
        const int i = (int)i0 + s.col_seg;
        const int slot = i + (i >= s.c_skip ? 1 : 0);
        const int coff = slot * s.c_seg_stride + rem + s.col_in_seg;
        f.base = head ? s.base0 : s.base1;
        f.tail = !head;
        f.add = (unsigned)(head ? c0 + s.col : coff);
    } else {
        // stage_init left the free index's region folded into base0 / off0 / c_mult0 when c does not decide
        f.base = head ? s.base0 + (int64_t)c0 * s.c_mult0 : s.base1 + (int64_t)(c0 - s.c_split) * s.c_mult1;
        f.tail = !head;
        f.add = head ? 0u : (unsigned)(s.c_split * s.c_mult1);   // off1 holds (row - split) * stride: make it non-negative
    }
    return f;
}

template <int KIND, int VEC, int PART, int J0, int J1, bool PLAIN = false>
__device__ __forceinline__ void fast_fetch(const FastStep &f, const int (&off0)[StageCfg<KIND, VEC, PART>::NV],
                                           const int (&off1)[StageCfg<KIND, VEC, PART>::NV],
                                           typename VecOf<VEC>::type (&regs)[StageCfg<KIND, VEC, PART>::NV])
{
    typedef typename StageCfg<KIND, VEC, PART>::V V;
#pragma unroll
    for (int j = J0; j < J1; ++j) {
        if (PLAIN) {
            regs[j] = load_global<V>(f.base + (unsigned)off0[j]);
            continue;
        }
        const int o0 = off0[j], o1 = off1[j];          // values first: a conditional on the array elements themselves
        const unsigned off = (unsigned)(f.tail ? o1 : o0) + f.add;   // would select an address and force the arrays into memory
        regs[j] = *(const __attribute__((address_space(1))) V *)((uintptr_t)f.base + (uint64_t)off * 2u);
    }
}

// move vectors J0 .. J1-1 of the tile fetched for reduction start c0 into LDS; CAREFUL zeroes reduction indices >= c_lim
template <int KIND, int VEC, bool CAREFUL, int PART = 1, int J0 = 0, int J1 = StageCfg<KIND, VEC, PART>::NV>
__device__ __forceinline__ void stage_store(const StageState &s, const typename VecOf<VEC>::type (&regs)[StageCfg<KIND, VEC, PART>::NV],
                                            __bf16 *tile, int c0)
{
    typedef StageCfg<KIND, VEC, PART> C;
    typedef typename C::V V;
    __bf16 *dst = tile + s.row0 * C::PITCH + s.col;
#pragma unroll
    for (int j = J0; j < J1; ++j) {
        if (CAREFUL) {
            const int c = KIND == LD_KC ? c0 + s.col : c0 + s.row0 + j * C::ROW_STEP;
            const uint32_t keep = c < s.c_lim ? 0xffffffffu : 0u;
            *(V *)(dst + j * C::ROW_STEP * C::PITCH) = regs[j] & keep;
        } else {
            *(V *)(dst + j * C::ROW_STEP * C::PITCH) = regs[j];
        }
    }
}

// MFMA operand (rows rbase..rbase+31 of the tile, reduction sub-step ks of 16) for this lane
template <int KIND>
__device__ __forceinline__ bf16x8 lds_operand(const __bf16 *tile, int rbase, int ks, int lane)
{
    if (KIND == LD_KC) {
        return *(const bf16x8 *)(tile + (rbase + (lane & 31)) * KC_PITCH + ks * 16 + (lane >> 5) * 8);
    } else {
        const int krow = ks * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
        const int rcol = rbase + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
        const __bf16 *p = tile + krow * KM_PITCH + rcol;
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
        s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * KM_PITCH));
        union { struct { s16x4 a, b; } s; bf16x8 v; } u;
        u.s.a = lo; u.s.b = hi;
        return u.v;
    }
}

struct MfmaIn {          // what a product's reduction needs ...
    View a, b;
    SumOnRead rs;
    int M, N, K;
    int tiles_m, tiles_n;
    short ksplit;        // > 1: the reduction range is cut into ksplit pieces; their results are added
                         //   by the piece that finishes last (parts)
    short bursts;        // an operand's loads of a step together in regular shapes, too (see rows_off_lines in phantom_api.hip)
    int k_per_split;     // multiple of KT
    int total_wg;
    uint32_t magic_tiles, magic_band;        // div_by: tiles_m * tiles_n, RASTER rows of them
};
struct MfmaOut {         // ... and what its epilogue needs
    View o;              // the row index must not decide the region (true for every output here)
    Epilogue ep;
    float *parts;        // ksplit > 1 without atomics (float output, 8-element vectors, one group): room for ksplit
    unsigned *arrived;   //   tiles of 128 x 128 floats per output tile, and one word per output tile, zero on entry
                         //   and left zero (see epilogue_pieces_from_lds)
    SgdInPlace sgd;      // what the epilogue that finishes a float output tile does besides storing it
};
struct MfmaParams {
    MfmaIn in;
    MfmaOut out;
};
// tiles are walked in bands of mfma_raster tile rows (TILE_DUAL: pairs), down the band first: the workgroups that run
// together on one XCD then cover a near-square patch of C and share both operand panels in L2
constexpr int mfma_raster(bool dual) { return dual ? 4 : 8; }

// The vectors of a K-contiguous A tile (reduction start c0) that lie in the summed block: replaces what the loads of the stage (landed
// by then) left there.  A thread holds NV vectors of the same columns in rows row0 + j * ROW_STEP; the loads of seven
// senders are in flight together (with fewer senders the last one is read again and not added).  Sums in fp32 in
// the order of the senders, one rounding to bf16.
template <int WAVES>
__device__ __forceinline__ void fetch_summed(const SumOnRead &rs, int g, int r0, int r_limit, const RingOperand &s, int c0,
                                             uint32_t tile, int wave, int lane, bool write_out)
{
    typedef RingCfg<LD_KC, WAVES> C;
    constexpr int VEC = 8;
    const int c = c0 + s.col;
    if (c < s.c_split || c + VEC > s.c_lim) return;
    const int w = c - s.c_split;
    int64_t row_off[C::NV];
#pragma unroll
    for (int j = 0; j < C::NV; ++j) row_off[j] = (int64_t)min(r0 + s.row0 + j * C::ROW_STEP, r_limit - 1) * rs.k + w;
    float acc[C::NV][VEC];
#pragma unroll
    for (int j = 0; j < C::NV; ++j)
#pragma unroll
        for (int u = 0; u < VEC; ++u) acc[j][u] = 0.f;
    constexpr int AHEAD = 7;                 // the host allows at most 8 ranks: all senders in one batch
    const int senders = rs.p - 1;
    for (int a0 = 0; a0 < senders; a0 += AHEAD) {
        u32x4 v[AHEAD][C::NV];
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            const int i = min(a0 + a, senders - 1);            // the i-th sender other than g
            const int from = i < g ? i : i + 1;
            const int slot = g < from ? g : g - 1;
            const __bf16 *base = (const __bf16 *)rs.src + ((int64_t)from * (rs.p - 1) + slot) * rs.per_slot;
#pragma unroll
            for (int j = 0; j < C::NV; ++j) v[a][j] = load_global<u32x4>(base + row_off[j]);
        }
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            const float take = a0 + a < senders ? 1.f : 0.f;
#pragma unroll
            for (int j = 0; j < C::NV; ++j) {
                union { u32x4 v; __bf16 e[VEC]; } x;
                x.v = v[a][j];
#pragma unroll
                for (int u = 0; u < VEC; ++u) acc[j][u] = fmaf(take, (float)x.e[u], acc[j][u]);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // (the stage's own loads are older than the senders')
#pragma unroll
    for (int j = 0; j < C::NV; ++j) {
        union { u32x4 v; __bf16 e[VEC]; } x;
#pragma unroll
        for (int u = 0; u < VEC; ++u) x.e[u] = (__bf16)acc[j][u];
        *lds_at<u32x4>(tile + (j * WAVES + wave) * 1024 + lane * 16) = x.v;
        if (write_out) *(u32x4 *)((__bf16 *)rs.out + (int64_t)g * rs.per_slot + row_off[j]) = x.v;
    }
}

template <int KA, int KB>
__device__ __forceinline__ void mfma_tile(f32x16 (&acc)[2][2], const __bf16 *ta, const __bf16 *tb, int wm, int wn, int lane)
{
#pragma unroll
    for (int kk = 0; kk < KT / 16; ++kk) {
        bf16x8 av[2], bv[2];
        av[0] = lds_operand<KA>(ta, wm, kk, lane);
        av[1] = lds_operand<KA>(ta, wm + 32, kk, lane);
        bv[0] = lds_operand<KB>(tb, wn, kk, lane);
        bv[1] = lds_operand<KB>(tb, wn + 32, kk, lane);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv[j], av[i], acc[i][j], 0, 0, 0);   // B first: see acc_to_lds
    }
}

// One reduction step with everything interleaved: a quarter (16 of 64 reduction indices) of the
// MFMAs on the current LDS stage, then a quarter of the NEXT tile moved from registers to the other
// LDS stage, then a quarter of the loads of the tile after that into the registers just freed.  In
// this order the LDS writes (128 B/clk) and the global loads (64 B/clk through the vector L1, which
// for a 128 x 128 tile is as many cycles as the MFMAs themselves) run under the MFMAs instead of
// before them.
template <int KA, int KB, int VA, int VB, bool CAREFUL, int Q, int BP>
__device__ __forceinline__ void fused_quarter(f32x16 (&acc)[2][2], const __bf16 *ta, const __bf16 *tb, int wm, int wn, int lane,
                                              const StageState &sa, const int (&a_off0)[StageCfg<KA, VA>::NV],
                                              const int (&a_off1)[StageCfg<KA, VA>::NV],
                                              typename VecOf<VA>::type (&ra)[StageCfg<KA, VA>::NV], __bf16 *na,
                                              const StageState &sb, const int (&b_off0)[StageCfg<KB, VB, BP>::NV],
                                              const int (&b_off1)[StageCfg<KB, VB, BP>::NV],
                                              typename VecOf<VB>::type (&rb)[StageCfg<KB, VB, BP>::NV], __bf16 *nb,
                                              int c_store, int c_fetch)
{
    constexpr int NA = StageCfg<KA, VA>::NV, NB = StageCfg<KB, VB, BP>::NV;
    constexpr int A0 = Q * NA / 4, A1 = (Q + 1) * NA / 4, B0 = Q * NB / 4, B1 = (Q + 1) * NB / 4;   // this quarter's vectors
    bf16x8 av[2], bv[2];
    av[0] = lds_operand<KA>(ta, wm, Q, lane);
    av[1] = lds_operand<KA>(ta, wm + 32, Q, lane);
    bv[0] = lds_operand<KB>(tb, wn, Q, lane);
    bv[1] = lds_operand<KB>(tb, wn + 32, Q, lane);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv[j], av[i], acc[i][j], 0, 0, 0);   // B first: see acc_to_lds
    stage_store<KA, VA, CAREFUL, 1, A0, A1>(sa, ra, na, c_store);
    stage_store<KB, VB, CAREFUL, BP, B0, B1>(sb, rb, nb, c_store);
    stage_fetch<KA, VA, CAREFUL, 1, false, A0, A1>(sa, a_off0, a_off1, ra, c_fetch);
    stage_fetch<KB, VB, CAREFUL, BP, false, B0, B1>(sb, b_off0, b_off1, rb, c_fetch);
}

// One reduction step of the fast path.  Per quarter kk (16 of the 64 reduction indices):
//   - the LDS reads of the NEXT quarter's MFMA operands are issued first (two operand buffers), so
//     their latency runs under this quarter's MFMAs;
//   - the four MFMAs alternate with the other traffic of the quarter, which therefore issues while
//     the matrix pipe is busy: quarters 0..2 move the next tile from registers to the other LDS
//     stage, quarters 1..3 issue the global loads of the tile after that into the registers just
//     freed.
// The workgroup's barrier sits before quarter 3: by then every wavefront has finished reading the
// current stage (its last operands are in registers) and writing the next one, so quarter 3
// already reads the first operands of the next step and no barrier is needed at the step's end.
// On entry fr[0] holds the operands of quarter 0; on exit it holds those of the next step.
template <int KIND_A, int KIND_B>
__device__ __forceinline__ void read_operands(bf16x8 (&f)[4], const __bf16 *ta, const __bf16 *tb, int wm, int wn, int kk, int lane)
{
    f[0] = lds_operand<KIND_A>(ta, wm, kk, lane);
    f[1] = lds_operand<KIND_A>(ta, wm + 32, kk, lane);
    f[2] = lds_operand<KIND_B>(tb, wn, kk, lane);
    f[3] = lds_operand<KIND_B>(tb, wn + 32, kk, lane);
}

constexpr int part_lo(int n, int q) { return n * q / 3; }       // the q-th third of n vectors

// ---- the compression inside the update's reduction loop (one rank's forward) ----------------------------
// g = X C^T shares its A operand with the update: the rows of X that a workgroup stages for its tile are the rows the
// compression needs, over the first part [0, K) of the update's reduction range.  The 128 rows of a tile row and the
// N <= 64 phantom neurons make 4 x ceil(N / 32) blocks of 32 x 32; the workgroup of tile column tn takes block tn:
// it stages the block's 32 rows of C beside its B tile (4 KB per step, half a load more per wavefront), and in each team the
// one wavefront whose A fragment covers the block's rows issues one more MFMA per quarter of the step (a team has two) with the fragment it
// has read anyway.  No second pass over X, no partial sums between workgroups, and the work rides under a loop that
// the memory side bounds.  Conditions (host): 8-element vectors, regular shapes, a tile row has at
// least as many workgroups as blocks, one tile per workgroup (the two-tile loop has no registers left for it).
// For a single layer, as a layer call has it: 4.9 us of a launch (1024 + 960 at batch 4096, k 64), and a launch of its own takes 8.  A step of two layers
// or more compresses all of them behind the forward pass (compress_many_kernel): forward of 8 such layers 221 -> 199 us, of 2 55.3 -> 52.3.
constexpr int FOLD_TILE = 32 * KT * 2;           // bytes of a stage's C rows

struct FoldParams {
    const __bf16 *C;     // [N, K] per group
    __bf16 *G;           // [M, N] per group, M = the update's
    int64_t c_g, o_g;    // element offsets per group
    int N, K;
    int ncb;             // blocks per row of blocks = ceil(N / 32)
    int nblocks;         // 4 * ncb; 0: no folding
};

struct FoldState {
    bool on;             // the workgroup has a block (uniform)
    bool owner;          // this wavefront multiplies it (uniform per wavefront)
    bool own_hi;         // ... with the second of its two 32-row A fragments
    int limit;           // reduction indices below it belong to X (uniform)
    const __bf16 *base;  // row 0 of the block's C rows, reduction index 0 (uniform)
    uint32_t src_off;    // this thread's 16-byte vector of those rows: byte offset from base
    f32x16 acc;
};

template <int KA, int KB, int VA, int VB, int BP, bool DRAIN, bool PLAIN>
__device__ __forceinline__ void fast_step(f32x16 (&acc)[2][2], bf16x8 (&fr)[2][4], const __bf16 *ta, const __bf16 *tb,
                                          int wm, int wn, int lane,
                                          const StageState &sa, const int (&a_off0)[StageCfg<KA, VA>::NV],
                                          const int (&a_off1)[StageCfg<KA, VA>::NV],
                                          typename VecOf<VA>::type (&ra)[StageCfg<KA, VA>::NV], __bf16 *na,
                                          const StageState &sb, const int (&b_off0)[StageCfg<KB, VB, BP>::NV],
                                          const int (&b_off1)[StageCfg<KB, VB, BP>::NV],
                                          typename VecOf<VB>::type (&rb)[StageCfg<KB, VB, BP>::NV], __bf16 *nb, int c_fetch,
                                          bool do_mfma, bool do_store, bool do_fetch)
{
    constexpr int NA = StageCfg<KA, VA>::NV, NB = StageCfg<KB, VB, BP>::NV;
    // a tile that does not exist has no valid address: its step start is replaced by one that does
    const int c_safe = (DRAIN && !do_fetch) ? sa.c_lim - KT : c_fetch;
    const FastStep fa = fast_step_addr<KA, VA, PLAIN>(sa, c_safe), fb = fast_step_addr<KB, VB, PLAIN>(sb, c_safe);
#define PH_MFMA(buf, i, j) do { if (!DRAIN || do_mfma) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[buf][2 + j], fr[buf][i], acc[i][j], 0, 0, 0); } while (0)
#define PH_STORE_A(q) do { if (!DRAIN || do_store) stage_store<KA, VA, false, 1, part_lo(NA, q), part_lo(NA, q + 1)>(sa, ra, na, 0); } while (0)
#define PH_STORE_B(q) do { if (!DRAIN || do_store) stage_store<KB, VB, false, BP, part_lo(NB, q), part_lo(NB, q + 1)>(sb, rb, nb, 0); } while (0)
#define PH_FETCH_A(q) do { if (!DRAIN || do_fetch) fast_fetch<KA, VA, 1, part_lo(NA, q), part_lo(NA, q + 1), PLAIN>(fa, a_off0, a_off1, ra); } while (0)
#define PH_FETCH_B(q) do { if (!DRAIN || do_fetch) fast_fetch<KB, VB, BP, part_lo(NB, q), part_lo(NB, q + 1), PLAIN>(fb, b_off0, b_off1, rb); } while (0)
#define PH_PIN __builtin_amdgcn_sched_barrier(0)   /* the compiler's scheduler would regroup the sequence */
    // quarter 0
    PH_PIN; read_operands<KA, KB>(fr[1], ta, tb, wm, wn, 1, lane); PH_PIN;
    PH_MFMA(0, 0, 0); PH_STORE_A(0); PH_PIN;
    PH_MFMA(0, 0, 1); PH_STORE_B(0); PH_PIN;
    PH_MFMA(0, 1, 0); PH_MFMA(0, 1, 1); PH_PIN;
    // quarter 1
    read_operands<KA, KB>(fr[0], ta, tb, wm, wn, 2, lane); PH_PIN;
    PH_MFMA(1, 0, 0); PH_STORE_A(1); PH_PIN;
    PH_MFMA(1, 0, 1); PH_STORE_B(1); PH_PIN;
    PH_MFMA(1, 1, 0); PH_FETCH_A(0); PH_PIN;
    PH_MFMA(1, 1, 1); PH_FETCH_B(0); PH_PIN;
    // quarter 2
    read_operands<KA, KB>(fr[1], ta, tb, wm, wn, 3, lane); PH_PIN;
    PH_MFMA(0, 0, 0); PH_STORE_A(2); PH_PIN;
    PH_MFMA(0, 0, 1); PH_STORE_B(2); PH_PIN;
    PH_MFMA(0, 1, 0); PH_FETCH_A(1); PH_PIN;
    PH_MFMA(0, 1, 1); PH_FETCH_B(1); PH_PIN;
    __syncthreads();
    // quarter 3
    PH_PIN; read_operands<KA, KB>(fr[0], na, nb, wm, wn, 0, lane); PH_PIN;
    PH_MFMA(1, 0, 0); PH_FETCH_A(2); PH_PIN;
    PH_MFMA(1, 0, 1); PH_FETCH_B(2); PH_PIN;
    PH_MFMA(1, 1, 0); PH_MFMA(1, 1, 1); PH_PIN;
#undef PH_PIN
#undef PH_MFMA
#undef PH_STORE_A
#undef PH_STORE_B
#undef PH_FETCH_A
#undef PH_FETCH_B
}

// ---- epilogue ---------------------------------------------------------------------------
// The MFMA accumulator layout gives a lane one column and scattered rows: stored from registers,
// every store instruction would write two 64-byte pieces of 2-byte elements (measured: 12 us for
// the 8 MB of a 4096 x 1024 bf16 output, a third of the kernel).  Instead the finished fp32 tile
// goes to LDS and all 512 threads walk it row by row, VEC consecutive columns per thread: bias,
// activation (or its derivative) and every global access are then 16-byte vectors on full lines.
constexpr int CT_PITCH = MT + 4;                       // floats per row of an fp32 tile in LDS (132 = 4 mod 64: the 16-byte
                                                       // writes of 16 lanes in 16 different rows fall on 64 different banks)
constexpr int CT_ELEMS = MT * CT_PITCH;                // one tile per team
static_assert((2 * CT_ELEMS + MFMA_THREADS / 64) * 4 <= MFMA_LDS_BYTES, "both teams' fp32 tiles and one float per wavefront fit in the staging space");

// A wavefront's 64 x 64 block of accumulators -> its team's fp32 tile in LDS.
// The MFMAs are issued with the B operand first, i.e. they compute the transpose of each 32 x 32 block:
// a lane then holds, of block (i, j), row (lane & 31) and the columns 8*(e/4) + 4*(lane>>5) + e%4, so
// every group of four accumulators is 16 contiguous bytes of a row-major tile (one ds_write_b128;
// in the untransposed layout the same data would take four 4-byte writes).
__device__ __forceinline__ void acc_to_lds(float *ctile, const f32x16 (&acc)[2][2], int wm, int wn, int lane)
{
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                *(f32x4 *)(ctile + (wm + 32 * i + (lane & 31)) * CT_PITCH + wn + 32 * j + 8 * q + 4 * (lane >> 5)) = v;
            }
}

template <typename T, int VEC> struct PackOf { typedef T type __attribute__((ext_vector_type(VEC))); };

// What the epilogue reads from memory besides the tile.  It is requested before the tile is written to LDS (epilogue_request) and used
// behind it (epilogue_from_lds): the write and its barrier take as long as a load (1900 clocks).  Requested behind the barrier, one straight
// run of loads, it cost the layer update of 8 ranks of 512 5800 clocks of epilogue against 1900 for a plain store; pass by pass as
// the target and the master weights were, each waits a memory latency behind the stores of the one before (the last layer's update 12500).
// EPI: the only mode other than EPI_STORE that the kernel is built for (the first product's; the second
// product of a pair always stores plainly).  Building every mode into every kernel made the epilogue, which
// every workgroup runs exactly once and so fetches cold, long enough to cost each launch about 1 us.
template <int VEC, typename TOut, int MODE, int EPI>
struct EpilogueReads {
    typedef typename PackOf<__bf16, VEC>::type BfV;
    typedef typename PackOf<float, VEC>::type FlV;
    static constexpr int THREADS = MODE != TILE_SHARED ? 256 : MFMA_THREADS;    // one team per tile, or both
    static constexpr int PER_ROW = MT / VEC;           // vectors per tile row
    static constexpr int PASSES = MT * PER_ROW / THREADS, ROWS_PER_PASS = THREADS / PER_ROW;
    static_assert(THREADS % PER_ROW == 0, "a thread keeps its columns from pass to pass");
    static constexpr bool MSE = EPI == EPI_BIAS_ACT && sizeof(TOut) == 2;
    // The master weights of an update, which nothing else reads for the rest of the step: past the caches unless the whole step fits the last-level one
    // (step_fits_last_cache).  Kept, they push the operand tiles that other workgroups still share out of L2.
    static constexpr bool MASTERS = EPI == EPI_STORE && sizeof(TOut) == 4;
    // passes that are unrolled together and whose reads are in flight together, a group ahead of their use
    static constexpr int GROUP = EPI == EPI_DACT ? PASSES : MASTERS && MODE == TILE_DUAL ? 8 : MASTERS || MSE ? 4 : 2;
    static_assert(PASSES % GROUP == 0, "whole groups");
    union AuxU { FlV f; BfV h; unsigned bits; __device__ AuxU() {} };
    BfV bias;
    AuxU aux[EPI == EPI_DACT ? PASSES : 1];
    BfV target[MSE ? GROUP : 1];
    FlV masters[MASTERS ? GROUP : 1];

    // the target's and the master weights' vectors of passes i0 .. i0 + GROUP - 1
    // (addresses clamped into the tile's valid part instead of skipped: no branch per load.  Element offsets inside a group fit 32 bits.)
    __device__ __forceinline__ void group(const MfmaIn &P, const MfmaOut &Q, int g, int m0, int n0, int thread, int i0)
    {
        const int row = m0 + i0 * ROWS_PER_PASS + thread / PER_ROW, n = min(n0 + (thread % PER_ROW) * VEC, P.N - VEC);
        if constexpr (MSE) {
            const Epilogue &ep = Q.ep;
            if (ep.mode == EPI_BIAS_ACT && ep.mse_target) {    // uniform
                const __bf16 *base = (const __bf16 *)ep.mse_target + g * ep.aux_g;
#pragma unroll
                for (int h = 0; h < GROUP; ++h)
                    target[h] = gload<BfV>(base + ((uint32_t)min(row + h * ROWS_PER_PASS, P.M - 1) * (uint32_t)ep.aux_ld + (uint32_t)n));
            }
        }
        if constexpr (MASTERS) {
            if (Q.sgd.w0) {                                    // uniform
                const Loc lc = locate(Q.o.c, n, Q.o.skip0 + g * Q.o.skip_g);
                const float *base = lc.region > 0 ? Q.sgd.master1 + g * Q.o.g1 + lc.off1 : Q.sgd.master0 + g * Q.o.g0 + lc.off0;
                const uint32_t ld = (uint32_t)(lc.region > 0 ? Q.o.r.mult1 : Q.o.r.mult0);
                if (Q.sgd.past_caches) {                       // uniform
                    // (the statements keep the compiler from making one of the two loops, which would be without the hint)
                    asm volatile("; masters past the caches");
#pragma unroll
                    for (int h = 0; h < GROUP; ++h) masters[h] = gload_nt<FlV>(base + (uint32_t)min(row + h * ROWS_PER_PASS, P.M - 1) * ld);
                    asm volatile("; masters requested");
                } else {
#pragma unroll
                    for (int h = 0; h < GROUP; ++h) masters[h] = gload<FlV>(base + (uint32_t)min(row + h * ROWS_PER_PASS, P.M - 1) * ld);
                }
            }
        }
    }
};

template <int VEC, typename TOut, int MODE, int EPI>
__device__ __forceinline__ void epilogue_request(EpilogueReads<VEC, TOut, MODE, EPI> &R, const MfmaIn &P, const MfmaOut &Q, int g, int m0, int n0, int thread)
{
    typedef EpilogueReads<VEC, TOut, MODE, EPI> Reads;
    typedef typename Reads::BfV BfV;
    typedef typename Reads::FlV FlV;
    const Epilogue &ep = Q.ep;
#pragma unroll
    for (int u = 0; u < VEC; ++u) R.bias[u] = (__bf16)0.f;
    if (EPI == EPI_BIAS_ACT && ep.mode == EPI_BIAS_ACT) {
        const int n = n0 + (thread % Reads::PER_ROW) * VEC;
        if (n < P.N) R.bias = gload<BfV>((const __bf16 *)ep.bias + g * ep.bias_g + n);
    }
    if constexpr (EPI == EPI_DACT) {
        if (ep.mode == EPI_DACT && ep.aux) {
            // One straight run of loads per kind of aux: with the choice of kind and the bounds test inside the loop every pass was a
            // basic block of its own and the compiler waited for each pass's load before it issued the next one's.
            uint32_t at[Reads::PASSES];
#pragma unroll
            for (int i = 0; i < Reads::PASSES; ++i) {
                const int v = thread + i * Reads::THREADS;
                const int m = min(m0 + v / Reads::PER_ROW, P.M - 1), n = min(n0 + (v % Reads::PER_ROW) * VEC, P.N - VEC);
                at[i] = (uint32_t)m * (uint32_t)ep.aux_ld + (uint32_t)n;
            }
            const int64_t first = g * ep.aux_g;                // (of groups: a multiple of aux_ld, which VEC divides)
            if (ep.aux_bits) {                         // uniform
#pragma unroll
                for (int i = 0; i < Reads::PASSES; ++i) R.aux[i].bits = gload<uint8_t>((const uint8_t *)ep.aux + (first >> 3) + (at[i] >> 3));
            } else if (ep.aux_deriv) {
#pragma unroll
                for (int i = 0; i < Reads::PASSES; ++i) R.aux[i].f = gload_nt<FlV>((const float *)ep.aux + first + at[i]);   // read once
            } else {
#pragma unroll
                for (int i = 0; i < Reads::PASSES; ++i) R.aux[i].h = gload<BfV>((const __bf16 *)ep.aux + first + at[i]);
            }
        }
    }
    R.group(P, Q, g, m0, n0, thread, 0);
}

// rows [m0, m0+128) x columns [n0, n0+128) of the output = sum of the two teams' fp32 tiles in LDS, walked by
// all 512 threads; one team per tile: the tile at ctile alone, walked by the team's 256 threads (thread = 0..255)
// Nothing runs beside it where a workgroup has its compute unit for itself, and the vector instructions bound it: with every choice taken pass by
// pass, 64-bit products for every address, and sums and derivatives that nobody had asked for, they were some 120 for 8 elements; now 65.
// Clocks, before : now: ReLU forward, two tiles 7350 : 4270, one 4610 : 2840; GELU 11200 : 5500; input gradient with sigma' in bf16, two tiles
// 3670 : 1900, one 2470 : 1600.
// What a wavefront stores in one instruction has no gaps: 16 bytes per thread, so 8 columns of bf16 and 4 of floats.  With 8 floats to a thread an
// instruction wrote every other 16 bytes of its lines and the next one the rest, which the memory takes at half its rate.  Floats, halves : whole: GELU with
// sigma' kept, 4096 x 1024 outputs 28.5 : 24.9 us a launch (epilogue 11700 : 8000 clocks); gradients 4096 x 4096 over 512 rows 44.2 : 31.3.
// Passes, us, both steps: 8 layers of 1024 + 960 with GELU trained at batch 4096 631 : 587; gradients of 64 ranks of 256 + 16 at 512 467 : 454, 6 layers
// of 1024 + 28 forward at 8192 183 : 175.
enum { EPI_PIECEWISE, EPI_GELU, EPI_GELU_DERIV };      // EPI_BIAS_ACT: not GELU; GELU; GELU whose derivative is kept
template <int VEC, typename TOut, int MODE, int EPI, int ACT>
__device__ __forceinline__ void epilogue_from_lds(const MfmaIn &P, const MfmaOut &Q, int g, const float *ctile, int m0, int n0, int thread,
                                                  float *wave_sums, EpilogueReads<VEC, TOut, MODE, EPI> &R)
{
    typedef EpilogueReads<VEC, TOut, MODE, EPI> Reads;
    constexpr bool SOLO = MODE != TILE_SHARED;         // one team per tile
    constexpr int THREADS = Reads::THREADS, PER_ROW = Reads::PER_ROW, PASSES = Reads::PASSES, GROUP = Reads::GROUP, ROWS_PER_PASS = Reads::ROWS_PER_PASS;
    typedef typename PackOf<TOut, VEC>::type OutV;
    typedef typename Reads::BfV BfV;
    typedef typename Reads::FlV FlV;
    const Epilogue &ep = Q.ep;
    // A thread's columns stay the same; its row moves down ROWS_PER_PASS a pass, and its addresses by the same amount (element
    // offsets inside a group fit 32 bits).
    const int col = (thread % PER_ROW) * VEC, n = n0 + col, row0 = thread / PER_ROW;
    const int rows = n < P.N ? P.M - m0 - row0 : 0;    // pass i has a row of the output: i * ROWS_PER_PASS < rows
    const Loc ln = locate(Q.o.c, n, Q.o.skip0 + g * Q.o.skip_g);
    const bool tail = ln.region > 0;
    const int64_t out_first = tail ? g * Q.o.g1 + ln.off1 : g * Q.o.g0 + ln.off0;
    const uint32_t out_ld = (uint32_t)(tail ? Q.o.r.mult1 : Q.o.r.mult0);
    TOut *const out = (TOut *)(tail ? Q.o.p1 : Q.o.p0) + out_first;
    const uint32_t out_step = ROWS_PER_PASS * out_ld, aux_step = ROWS_PER_PASS * (uint32_t)ep.aux_ld;
    uint32_t out_at = (uint32_t)(m0 + row0) * out_ld, aux_at = (uint32_t)(m0 + row0) * (uint32_t)ep.aux_ld + (uint32_t)n;
    const int64_t aux_first = g * ep.aux_g;
    const float *ct = ctile + row0 * CT_PITCH + col;
    // (the last layer, which has the error, keeps no derivative)
    const bool mse = EPI == EPI_BIAS_ACT && ACT != EPI_GELU_DERIV && sizeof(TOut) == 2 && ep.mode == EPI_BIAS_ACT && ep.mse_target;      // uniform
    const bool sums = EPI != EPI_STORE && ep.colsum;                                                            // uniform
    float csum[VEC];                                   // this thread's share of the column sums (ep.colsum)
#pragma unroll
    for (int u = 0; u < VEC; ++u) csum[u] = 0.f;
    float sq_sum = 0.f;                                // ... and of the squared output error (ep.mse_target)
#pragma unroll 1
    for (int i0 = 0; i0 < PASSES; i0 += GROUP) {
        const Reads now = R;                           // the group's target and master weights; the next group's are requested
        if (i0 + GROUP < PASSES) R.group(P, Q, g, m0, n0, thread, i0 + GROUP);
        // Every choice below is the same for the whole workgroup and taken once for the group, not pass by pass: its passes then run as one
        // straight piece of code.  Rows past the output's end are computed like the others (from what the loaders repeat) and not stored.
        float x[GROUP][VEC], deriv[GROUP][VEC];        // deriv: sigma'(pre-activation)
        bool ok[GROUP];
#pragma unroll
        for (int h = 0; h < GROUP; ++h) {
            ok[h] = (i0 + h) * ROWS_PER_PASS < rows;
            const float *from = ct + (i0 + h) * ROWS_PER_PASS * CT_PITCH;
            const FlV c0 = *(const FlV *)from;
            if constexpr (SOLO) {
#pragma unroll
                for (int u = 0; u < VEC; ++u) x[h][u] = c0[u];
            } else {
                const FlV c1 = *(const FlV *)(from + CT_ELEMS);
#pragma unroll
                for (int u = 0; u < VEC; ++u) x[h][u] = c0[u] + c1[u];
            }
        }
        const auto store_aux = [&](const float (&v)[GROUP][VEC]) {             // in the storage type
#pragma unroll
            for (int h = 0; h < GROUP; ++h) {
                BfV a;
#pragma unroll
                for (int u = 0; u < VEC; ++u) a[u] = (__bf16)v[h][u];
                if (ok[h]) gstore<BfV>((__bf16 *)ep.aux + aux_first + (aux_at + h * aux_step), a);
            }
        };
        if (EPI == EPI_BIAS_ACT && ep.mode == EPI_BIAS_ACT) {
#pragma unroll
            for (int h = 0; h < GROUP; ++h)
#pragma unroll
                for (int u = 0; u < VEC; ++u) x[h][u] += (float)now.bias[u];
            if constexpr (ACT != EPI_PIECEWISE) {
                if (ACT == EPI_GELU && ep.aux) store_aux(x);
#pragma unroll
                for (int h = 0; h < GROUP; ++h)
#pragma unroll
                    for (int u = 0; u < VEC; ++u) {
                        const float pre = x[h][u];
                        gelu_both(pre, x[h][u], deriv[h][u]);
                    }
                if constexpr (ACT == EPI_GELU_DERIV) {
                    // written once, read once by the backward pass much later: a streaming store keeps it from
                    // pushing the operand panels that other workgroups still share out of L2
#pragma unroll
                    for (int h = 0; h < GROUP; ++h) {
                        FlV a;
#pragma unroll
                        for (int u = 0; u < VEC; ++u) a[u] = deriv[h][u];
                        if (ok[h]) gstore_nt<FlV>((float *)ep.aux + aux_first + (aux_at + h * aux_step), a);
                    }
                }
            } else {
                if (ep.aux && !ep.aux_bits) store_aux(x);
                if (ep.act == ACT_RELU) {
#pragma unroll
                    for (int h = 0; h < GROUP; ++h)
#pragma unroll
                        for (int u = 0; u < VEC; ++u) x[h][u] = __builtin_fmaxf(x[h][u], 0.f);      // (of a NaN: 0)
                }
            }
        } else if (EPI == EPI_DACT && ep.mode == EPI_DACT && ep.aux) {      // no aux: sigma' = 1, column sums only
            if (ep.aux_bits) {                         // one bit per element: ReLU' of the stored output
                if constexpr (VEC == 8) {
#pragma unroll
                    for (int h = 0; h < GROUP; ++h)
#pragma unroll
                        for (int u = 0; u < VEC; ++u) x[h][u] = (now.aux[EPI == EPI_DACT ? h : 0].bits >> u) & 1u ? x[h][u] : 0.f;
                }
            } else if (ep.aux_deriv) {                 // sigma' itself, float
#pragma unroll
                for (int h = 0; h < GROUP; ++h)
#pragma unroll
                    for (int u = 0; u < VEC; ++u) x[h][u] *= now.aux[EPI == EPI_DACT ? h : 0].f[u];
            } else {                                   // ReLU output in bf16
#pragma unroll
                for (int h = 0; h < GROUP; ++h)
#pragma unroll
                    for (int u = 0; u < VEC; ++u) x[h][u] = (float)now.aux[EPI == EPI_DACT ? h : 0].h[u] > 0.f ? x[h][u] : x[h][u] * 0.f;
            }
        }
        OutV o[GROUP];
#pragma unroll
        for (int h = 0; h < GROUP; ++h)
#pragma unroll
            for (int u = 0; u < VEC; ++u) o[h][u] = from_f32<TOut>(x[h][u]);
        bool store = true;
        if constexpr (EPI == EPI_STORE && sizeof(TOut) == 4) {
            if (Q.sgd.w0) {                            // uniform: Section VI's plain SGD on the finished gradient
                float *const masters = (tail ? Q.sgd.master1 : Q.sgd.master0) + out_first;
                __bf16 *const weights = (__bf16 *)(tail ? Q.sgd.w1 : Q.sgd.w0) + out_first;
                store = Q.sgd.keep_grad;
#pragma unroll
                for (int h = 0; h < GROUP; ++h) {
                    if (!ok[h]) continue;
                    float *const master = masters + (out_at + h * out_step);
                    const FlV before = now.masters[Reads::MASTERS ? h : 0];
                    FlV after;
                    BfV rounded;
#pragma unroll
                    for (int u = 0; u < VEC; ++u) {
                        after[u] = before[u] - Q.sgd.lr * x[h][u];
                        rounded[u] = (__bf16)after[u];
                    }
                    // (the master is next read a step later, by this epilogue; the bf16 copy by the next forward pass, which
                    // found it in the last-level cache before a streaming store put it out of there: 1.8 us per forward launch)
                    gstore_nt<FlV>(master, after);
                    gstore<BfV>(weights + (out_at + h * out_step), rounded);
                }
            }
        }
        if (store) {                                   // uniform
            // (outputs are written once and read by a later launch at the earliest: a streaming store leaves less for the
            // write-back at the end of the kernel; 0.4 % of configuration 4's step, 2-4 % of the forward-only and small ones)
#pragma unroll
            for (int h = 0; h < GROUP; ++h)
                if (ok[h]) gstore_nt<OutV>(out + (out_at + h * out_step), o[h]);
        }
        if constexpr (EPI == EPI_BIAS_ACT && VEC == 8) {
            if (ep.mode == EPI_BIAS_ACT && ep.aux && ep.aux_bits) {     // uniform
#pragma unroll
                for (int h = 0; h < GROUP; ++h) {
                    unsigned bits = 0;
#pragma unroll
                    for (int u = 0; u < VEC; ++u) bits |= ((float)o[h][u] > 0.f ? 1u : 0u) << u;
                    if (ok[h]) gstore<uint8_t>((uint8_t *)ep.aux + (aux_first >> 3) + ((aux_at + h * aux_step) >> 3), (uint8_t)bits);
                }
            }
        }
        if (mse) {
            // the MSE output error of Eq. (deltaL) from the output as stored, rounded once
#pragma unroll
            for (int h = 0; h < GROUP; ++h) {
                if (!ok[h]) continue;
                const BfV t = now.target[Reads::MSE ? h : 0];
                BfV dl;
#pragma unroll
                for (int u = 0; u < VEC; ++u) {
                    const float diff = (float)o[h][u] - (float)t[u];
                    sq_sum += diff * diff;
                    float e = diff * ep.mse_inv_b;
                    if (ACT != EPI_PIECEWISE) e *= deriv[h][u];
                    else if (ep.act == ACT_RELU) e *= x[h][u] > 0.f ? 1.f : 0.f;
                    dl[u] = (__bf16)e;
                    csum[u] += (float)dl[u];
                }
                gstore<BfV>((__bf16 *)ep.mse_delta + aux_first + (aux_at + h * aux_step), dl);
            }
        } else if (sums) {
#pragma unroll
            for (int h = 0; h < GROUP; ++h)
                if (ok[h]) {
#pragma unroll
                    for (int u = 0; u < VEC; ++u) csum[u] += (float)o[h][u];
                }
        }
        out_at += GROUP * out_step;
        aux_at += GROUP * aux_step;
    }
    if constexpr (EPI == EPI_STORE && sizeof(TOut) == 4) {
        if (Q.sgd.bias_master && n0 == 0 && thread < MT && m0 + thread < P.M) {
            const int64_t at = g * (int64_t)P.M + m0 + thread;
            const float nb = gload<float>(Q.sgd.bias_master + at) - Q.sgd.lr * gload<float>(Q.sgd.bias_grad + at);
            gstore<float>(Q.sgd.bias_master + at, nb);
            gstore<__bf16>((__bf16 *)Q.sgd.bias_w + at, (__bf16)nb);
        }
    }
    if (mse) {
        // the tile's share of sum (y - t)^2: wavefront sums, then one thread adds those of the tile's wavefronts
        // (wave_sums lies behind the fp32 tiles; nothing else uses it)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sq_sum += __shfl_down(sq_sum, off);
        const int wave_in_wg = (int)(threadIdx.x >> 6);
        if ((threadIdx.x & 63) == 0) wave_sums[wave_in_wg] = sq_sum;
        __syncthreads();
        if (thread == 0 && m0 < P.M) {
            constexpr int WAVES = THREADS / 64;
            const int first = SOLO ? (int)(threadIdx.x >> 6) : 0;
            float total = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) total += wave_sums[first + w];
            const int tiles_m = (P.M + MT - 1) / MT, tiles_n = (P.N + MT - 1) / MT;
            ep.mse_partial[(g * tiles_m + m0 / MT) * tiles_n + n0 / MT] = total;
        }
    }
    if (EPI != EPI_STORE && ep.colsum) {               // uniform
        // threads tid, tid + PER_ROW, ... hold partial sums of the same VEC columns: add them up through
        // LDS (over the fp32 tiles, once every thread has read its share), one atomic per column
        constexpr int SHARERS = THREADS / PER_ROW;
        float *red = const_cast<float *>(ctile);       // SOLO: each team reduces over its own tile
        __syncthreads();
#pragma unroll
        for (int u = 0; u < VEC; ++u) red[(thread / PER_ROW) * MT + (thread % PER_ROW) * VEC + u] = csum[u];
        __syncthreads();
        if (thread < MT && n0 + thread < P.N) {
            float t = 0.f;
#pragma unroll 8
            for (int r = 0; r < SHARERS; ++r) t += red[r * MT + thread];
            unsafeAtomicAdd(ep.colsum + g * ep.colsum_g + n0 + thread, t);
        }
    }
}

// The epilogue of one piece of a reduction that is cut into ksplit pieces without atomics (float output, plain store
// semantics, 4 columns per thread, all 512 threads).  Every piece writes its 128 x 128 result to its own slot of
// Q.parts and then counts itself in Q.arrived[tile]; the piece that finds all others counted adds the slots up in the
// order of the pieces (its own from registers), writes the output and leaves the word zero for the next launch.  The
// sum does not depend on which piece comes last, and no workgroup ever waits for another.
// The pieces may run on different XCDs, whose L2 caches do not see each other's lines.  What goes from one to the
// other therefore uses device-scope atomic stores and loads (8 bytes each; the cache policy writes them through to
// memory and reads them from there), as the counter does, so no cache has to be written back or invalidated as a whole:
// with such fences, one per wavefront, the launch took 130 us against 44 us for the uncut product.  Within a slot,
// thread t holds the 8-byte words t, t + 512, ...: every store and load instruction covers 4 KB without gaps.
__device__ __forceinline__ void epilogue_pieces_from_lds(const MfmaIn &P, const MfmaOut &Q, int tile, int ks, const float *ctile, unsigned *lds_word,
                                                         int m0, int n0, int thread)
{
    typedef unsigned long long u64;
    constexpr int VEC = 4, PER_ROW = MT / VEC, PASSES = MT * PER_ROW / MFMA_THREADS, WORDS = VEC / 2;
    constexpr int ROWS_PER_PASS = MFMA_THREADS / PER_ROW;
    constexpr int64_t SLOT = MT * MT / 2;              // 8-byte words per slot
    constexpr int GROUP = 2;                           // other pieces whose loads are in flight together
    union Two { u64 w; float f[2]; __device__ Two() {} };
    // passes whose rows all lie below the output's last row (the compressor gradient has k <= 64 rows) move nothing
    const int passes = min(PASSES, (P.M - m0 + ROWS_PER_PASS - 1) / ROWS_PER_PASS);      // uniform
    float x[PASSES][VEC];
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        const int v = thread + i * MFMA_THREADS;
        const int row = v / PER_ROW, col = (v % PER_ROW) * VEC;
        const f32x4 c0 = *(const f32x4 *)(ctile + row * CT_PITCH + col), c1 = *(const f32x4 *)(ctile + CT_ELEMS + row * CT_PITCH + col);
#pragma unroll
        for (int u = 0; u < VEC; ++u) x[i][u] = c0[u] + c1[u];
    }
    u64 *slots = (u64 *)Q.parts + (int64_t)tile * P.ksplit * SLOT;
    u64 *mine = slots + ks * SLOT + thread;
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        if (i >= passes) break;
#pragma unroll
        for (int c = 0; c < WORDS; ++c) {
            Two t;
            t.f[0] = x[i][2 * c]; t.f[1] = x[i][2 * c + 1];
            __hip_atomic_store(mine + (i * WORDS + c) * MFMA_THREADS, t.w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // written through before this piece counts itself
    __syncthreads();
    if (thread == 0) *lds_word = __hip_atomic_fetch_add(Q.arrived + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*lds_word + 1 != (unsigned)P.ksplit) return;   // uniform: another piece will finish the tile
    float t[PASSES][VEC];
#pragma unroll
    for (int i = 0; i < PASSES; ++i)
#pragma unroll
        for (int u = 0; u < VEC; ++u) t[i][u] = 0.f;
    for (int j0 = 0; j0 < P.ksplit; j0 += GROUP) {     // uniform
        Two got[GROUP][PASSES][WORDS];
#pragma unroll
        for (int jj = 0; jj < GROUP; ++jj) {
            const int j = j0 + jj;
            if (j >= P.ksplit || j == ks) continue;
            const u64 *theirs = slots + j * SLOT + thread;
#pragma unroll
            for (int i = 0; i < PASSES; ++i) {
                if (i >= passes) break;
#pragma unroll
                for (int c = 0; c < WORDS; ++c)
                    got[jj][i][c].w = __hip_atomic_load(theirs + (i * WORDS + c) * MFMA_THREADS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
#pragma unroll
        for (int jj = 0; jj < GROUP; ++jj) {
            const int j = j0 + jj;
            if (j >= P.ksplit) break;
#pragma unroll
            for (int i = 0; i < PASSES; ++i) {
                if (i >= passes) break;
#pragma unroll
                for (int c = 0; c < WORDS; ++c) {
                    t[i][2 * c] += j == ks ? x[i][2 * c] : got[jj][i][c].f[0];
                    t[i][2 * c + 1] += j == ks ? x[i][2 * c + 1] : got[jj][i][c].f[1];
                }
            }
        }
    }
    float *o0 = (float *)Q.o.p0, *o1 = (float *)Q.o.p1;
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        const int v = thread + i * MFMA_THREADS;
        const int m = m0 + v / PER_ROW, n = n0 + (v % PER_ROW) * VEC;
        if (m >= P.M || n >= P.N) continue;
        const Loc ln = locate(Q.o.c, n, Q.o.skip0);
        const int region = ln.region > 0 ? 1 : 0;
        const int64_t at = (region ? ln.off1 : ln.off0) + (int64_t)m * (region ? Q.o.r.mult1 : Q.o.r.mult0);
        float *dst = (region ? o1 : o0) + at;
        if (Q.sgd.w0) {                           // uniform: Section VI's plain SGD on the finished gradient
            float *master = (region ? Q.sgd.master1 : Q.sgd.master0) + at;
            __bf16 *w = (__bf16 *)(region ? Q.sgd.w1 : Q.sgd.w0) + at;
            const f32x4 before = gload_nt<f32x4>(master);
            f32x4 after;
            typename PackOf<__bf16, VEC>::type rounded;
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                after[u] = before[u] - Q.sgd.lr * t[i][u];
                rounded[u] = (__bf16)after[u];
            }
            gstore_nt<f32x4>(master, after);
            gstore<typename PackOf<__bf16, VEC>::type>(w, rounded);
            if (!Q.sgd.keep_grad) continue;
        }
        gstore_nt<f32x4>(dst, f32x4{t[i][0], t[i][1], t[i][2], t[i][3]});
    }
    if (thread == 0) __hip_atomic_store(Q.arrived + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

#ifdef PHANTOM_TIMELINE   // cycle stamps for the development micro-benchmark, never built into the library
// per workgroup 16 words at P.rs.out: slots 0..7 the core clock, 8..15 the 100 MHz wall clock at the same points
#define PH_PHASE(slot) do { __builtin_amdgcn_sched_barrier(0); if (threadIdx.x == 0 && P.rs.out) { \
        ((long long *)P.rs.out)[blockIdx.x * 16 + (slot)] = clock64(); ((long long *)P.rs.out)[blockIdx.x * 16 + 8 + (slot)] = wall_clock64(); } \
        __builtin_amdgcn_sched_barrier(0); } while (0)
#else
#define PH_PHASE(slot) do { } while (0)
#endif

// 512 threads = two teams of 4 wavefronts.  Both teams work on the SAME 128 x 128 tile of C, each on its half of every
// reduction step (VEC = 4: on alternate steps), so every SIMD holds two wavefronts whose LDS traffic and MFMAs interleave,
// without reading any operand twice.  At the end each team writes its partial fp32 tile to LDS and the epilogue adds the two.
// One launch may carry two independent products of the same operand layout and output type (the
// layer update with the compression, the error compression with the input gradient, the weight
// gradients with the compressor gradient): their workgroups run side by side instead of one thin
// launch waiting for the other.
struct MfmaRiders {      // what a launch of gemm_mfma_kernel may do on its way
    ClearList clear;     // forward layout: buffers that later launches of a training step add into
    LossTail tail;       // weight-gradient layout: the first workgroup finishes the loss (partial == NULL: nothing to do)
};
struct MfmaBatch {
    MfmaParams p[2];
    int count;
    int total_wg;
    int first_wg;        // = p[0].total_wg
    MfmaRiders ride;
};
static_assert(sizeof(MfmaBatch) <= 3840, "a batch travels as kernel arguments (4 KB with the hidden ones)");


// Reads the epilogue's part of the parameter block that starts at a byte offset of the kernel's argument.
struct OutFromArgs {
    size_t offset;
    __device__ __forceinline__ MfmaOut operator()() const { return args_at<MfmaOut>(offset + offsetof(MfmaParams, out)); }
};
// ... and the part that the reduction needs, with the epilogue's on its way to the scalar cache: first asked for behind the reduction, it took 700 clocks.
__device__ __forceinline__ MfmaIn in_from_args(size_t offset)
{
    touch_args<MfmaOut>(offset + offsetof(MfmaParams, out));
    return args_at<MfmaIn>(offset + offsetof(MfmaParams, in));
}

// DUAL: the two teams take two tiles that lie one above the other (rows m0 .. m0+127 and m0+128 .. m0+255)
// instead of the reduction of one tile.  They share the B tile (each team stages half of its
// rows), so per FLOP a quarter less goes through the vector-memory return path and into LDS, what
// bounds the loop beside the matrix cores; the price is half as many workgroups, so this is for launches with more tiles
// than compute units (the host decides).  Each team finishes its own tile: no sum in the epilogue.
// SOLO: a workgroup is one team with one tile, two workgroups to a compute unit.  The terms of a sum come in DUAL's order
// (the results are the same bits).  Nothing is shared, but one workgroup's epilogue runs beside the other's loop: for
// short reductions with a heavy epilogue (solo_tiles on the host).
// XCD-aware id: hardware deals workgroup ids round-robin over 8 XCDs; `first` (a multiple of 8) is the id of the
// first of `count` consecutive workgroups that share a list of tiles.  Workgroups of one XCD get neighbouring tiles.
__device__ __forceinline__ int xcd_order(int id, int first, int count)
{
    const int i = id - first, per = count >> 3;
    return i < per * 8 ? (i & 7) * per + (i >> 3) : i;
}

// The reduction of one workgroup: acc of each wavefront <- its 64 x 64 block of the team's tile (TILE_SHARED: the team's share of the
// sums), operands in 16-byte vectors (see mfma_ring.h).  tm, tn: the workgroup's tile; m0: first row of the team's tile.
// TILE_SHARED: both teams read every stage, team q the 32 reduction indices 32 q .. 32 q + 31 of each step.  TILE_DUAL: the teams'
// tiles share the B tile.  TILE_SOLO: two stages only, but another workgroup's loop runs beside this one's.
// The tiles of the reduction range are walked from the LAST one down: the only one that can be ragged (the end of the range), and
// the one that holds a summed block, then comes first, ahead of the loop.
// LEVELS: in the place of one running sum, those of 8 steps each (32 MFMAs) or of half the steps each, and the sum of those.
enum Levels { ONE_SUM, SUMS_OF_8, SUMS_OF_HALVES };
template <int KA, int KB, int MODE, bool FOLD, int LEVELS>
__device__ __forceinline__ void reduce_in_ring(const MfmaIn &P, int g, int m0, int n0, int tn, int k_begin, int k_end,
                                               f32x16 (&acc)[2][2], FoldState &fs, uint32_t lds0)
{
    constexpr bool DUAL = MODE == TILE_DUAL, SOLO = MODE == TILE_SOLO;
    constexpr int WAVES = SOLO ? 4 : 8, WA = DUAL ? 4 : WAVES;                  // wavefronts that stage the B tile, the A tile
    constexpr int B_AT = DUAL ? 2 * RING_TILE : RING_TILE, E_AT = B_AT + RING_TILE;
    constexpr int STAGE = E_AT + (FOLD ? FOLD_TILE : 0), RING = SOLO ? 2 : DUAL ? 3 : 4;
    static_assert(RING * STAGE <= mfma_lds_bytes(MODE), "the ring fits the LDS");
    typedef RingCfg<KA, WA> CA;
    typedef RingCfg<KB, WAVES> CB;
    constexpr int NL = CA::NV + CB::NV + (FOLD ? 1 : 0);                        // a wavefront's loads per stage
    constexpr int QUARTERS = MODE == TILE_SHARED ? 2 : 4;                       // 16 reduction indices each, per step

    const int lane = threadIdx.x & 63, wave8 = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int team = wave8 >> 2, wave = wave8 & 3, wave_a = DUAL ? wave : wave8;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const uint32_t a_at = DUAL ? team * RING_TILE : 0;
    uint32_t a_off0[CA::NV], a_off1[CA::NV], b_off0[CB::NV], b_off1[CB::NV];
    // a DUAL team whose tile lies below the last row still stages its half of B and keeps the barriers:
    // its loaders read the last valid row, its epilogue writes nothing
    const int a_m0 = min(m0, (P.M - 1) / MT * MT);
    const RingOperand sa = ring_init<KA, WA>(P.a, g, a_m0, P.M, k_end, wave_a, lane, a_off0, a_off1);
    const RingOperand sb = ring_init<KB, WAVES>(P.b, g, n0, P.N, k_end, wave8, lane, b_off0, b_off1);
    PH_PHASE(7);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    f32x16 sums[LEVELS ? 2 : 1][LEVELS ? 2 : 1];
    if constexpr (LEVELS) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) sums[i][j][e] = 0.f;
    }

    const int steps = (k_end - k_begin + KT - 1) / KT;
    auto c_of = [=](int i) { return k_begin + (steps - 1 - i) * KT; };          // tile processed in step i
    auto fetch_a = [&](int i, uint32_t stage) { ring_fetch<KA, WA>(sa, a_off0, a_off1, c_of(i), stage + a_at, wave_a); };
    auto fetch_b = [&](int i, uint32_t stage) {
        ring_fetch<KB, WAVES>(sb, b_off0, b_off1, c_of(i), stage + B_AT, wave8);
        if constexpr (FOLD) {
            // (always one load, so that every stage has the same number; behind X's part of the range it is not used)
            const int c0 = c_of(i);
            if (lane < 32) ring_load<0>(fs.base, fs.src_off + (unsigned)(fs.on && c0 < fs.limit ? c0 : 0) * 2u, stage + E_AT + wave8 * 512);
        }
    };
    PH_PHASE(1);
#pragma unroll
    for (int i = 0; i < RING; ++i)
        if (i < steps) { fetch_a(i, lds0 + i * STAGE); fetch_b(i, lds0 + i * STAGE); }     // uniform
    const int younger = min(steps, RING) - 1;          // stages in flight behind the first
    if constexpr (KA == LD_KC && KB == LD_KM) {        // the input gradient's layout
        // the summed block lies in the tile processed first (the host sees to it: it starts at a tile boundary
        // and is at most one tile long)
        if (P.rs.src && c_of(0) + KT > sa.c_split) fetch_summed<WA>(P.rs, g, a_m0, P.M, sa, c_of(0), lds0 + a_at, wave_a, lane, tn == 0);
    }
    if (c_of(0) + KT > k_end) {                        // uniform
        ring_landed<NL, RING - 1>(younger);
        ring_zero<KA, WA>(sa, c_of(0), lds0 + a_at, wave_a, lane);
        ring_zero<KB, WAVES>(sb, c_of(0), lds0 + B_AT, wave8, lane);
    }
    ring_wait_stage<NL, RING - 1>(younger);
    PH_PHASE(2);

    const int at_a = ring_lane_at<KA>(wm, lane), at_b = ring_lane_at<KB>(wn, lane);
    const int q0 = MODE == TILE_SHARED ? team * 2 : 0;
    bf16x8 fr[2][4];
    // One of the four operands of quarter q of a stage (f[0], f[1]: A's blocks of 32 rows, f[2], f[3]: B's), in the order in which the matrix instructions
    // want them.  One ahead of each matrix instruction of the quarter before: four together ahead of the four hold up each other and the loads' writes to LDS.
    auto read = [&](bf16x8 (&f)[4], uint32_t stage, int q, auto nth) {
        constexpr int W = (0x1320 >> 4 * decltype(nth)::value) & 15;
        if constexpr (W < 2) f[W] = ring_operand<KA>(stage + a_at, at_a, W, q0 + q);
        else f[W] = ring_operand<KB>(stage + B_AT, at_b, W - 2, q0 + q);
    };
#define PH_PIN __builtin_amdgcn_sched_barrier(0)   /* the compiler's scheduler would regroup the sequence */
#define PH_MFMA(buf, i, j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[buf][2 + j], fr[buf][i], acc[i][j], 0, 0, 0)   /* B first: see acc_to_lds */
    // (a branch, not a select between the two fragments: a select of array elements would move the array to memory)
#define PH_FOLD(buf) do { if (FOLD && e_mul) { \
        if (fs.own_hi) fs.acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fe[buf], fr[buf][1], fs.acc, 0, 0, 0); \
        else fs.acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fe[buf], fr[buf][0], fs.acc, 0, 0, 0); } } while (0)
    auto read_all = [&](bf16x8 (&f)[4], uint32_t stage, int q) { ring_each<4>([&](auto nth) { read(f, stage, q, nth); }); };
    read_all(fr[0], lds0, 0);
    if constexpr (FOLD || LEVELS != ONE_SUM) {
        // With a second set of sums, or the compression's, one loop with its conditions: three of them do not fit the registers (179 spilled; us a step, so : in
        // three: 4 layers of 2000 + 36 trained at batch 2048 384 : 585, 3 of 1024 + 700 at 4000 241 : 250).
        uint32_t cur = lds0, prev = lds0;
        for (int t = 0; t < steps; ++t) {                  // uniform; on entry fr[0] holds the operands of the step's first quarter
            const uint32_t next = cur + STAGE == lds0 + RING * STAGE ? lds0 : cur + STAGE;
            bf16x8 fe[2];                                  // the block's operands
            const bool e_mul = FOLD && fs.owner && c_of(t) < fs.limit;              // uniform per wavefront
            if constexpr (FOLD) {
                if (e_mul) {
                    const int at = ring_lane_at<LD_KC>(0, lane);
#pragma unroll
                    for (int q = 0; q < 2; ++q) fe[q] = ring_operand<LD_KC>(cur + E_AT, at, 0, q0 + q);
                }
            }
#pragma unroll
            for (int q = 0; q + 1 < QUARTERS; ++q) {
                PH_PIN; read_all(fr[(q + 1) & 1], cur, q + 1); PH_PIN;
                PH_MFMA(q & 1, 0, 0); PH_PIN;
                if (RING > 2 && q == 0 && t > 0 && t - 1 + RING < steps) fetch_b(t - 1 + RING, prev);
                PH_PIN; PH_MFMA(q & 1, 0, 1); PH_MFMA(q & 1, 1, 0); PH_MFMA(q & 1, 1, 1); PH_FOLD(0); PH_PIN;
            }
            ring_wait_stage<NL, RING - 2>(steps - 2 - t);  // the next stage has landed, and everybody has read this one
            if (t + 1 < steps) read_all(fr[0], next, 0);
            PH_PIN; PH_MFMA(1, 0, 0); PH_PIN;
            if (t + RING < steps) {
                fetch_a(t + RING, cur);                    // (the other operand's loads follow in the next step: half the burst)
                if (RING == 2) fetch_b(t + RING, cur);     // (... which waits for them itself with two stages)
            }
            PH_PIN; PH_MFMA(1, 0, 1); PH_MFMA(1, 1, 0); PH_MFMA(1, 1, 1); PH_FOLD(1); PH_PIN;
            if constexpr (LEVELS) {
                if (t + 1 == steps || (LEVELS == SUMS_OF_8 ? t % 8 == 7 : t + 1 == steps / 2)) {      // uniform
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
#pragma unroll
                            for (int e = 0; e < 16; ++e) { sums[i][j][e] += acc[i][j][e]; acc[i][j][e] = 0.f; }
                }
            }
            prev = cur;
            cur = next;
        }
    } else {
        // What goes on between two barriers is one piece of code: the last quarter of step t and the other quarters of step t + 1, and behind matrix instructions
        // of the latter (two stages: of the former, as the next barrier waits for them) the loads of the tile of step t + RING, to the slot that step t leaves.
        // Regular shapes: one by one, unless P.bursts.  Other shapes work out an address per load and issue an operand's together, half of them behind the barrier
        // and half in the next step.  A condition on each load, with one loop in the place of three, took 63.3 us where this takes 59.7 (weight gradients
        // 8192 x 1024 over 4096 rows).
        enum { NO_LOADS, BURSTS, ONE_BY_ONE };
        RingCursor<KA, WA> ca;
        RingCursor<KB, WAVES> cb;
        uint32_t cur = lds0, next = lds0;                  // slots of step t and step t + 1
        int t = 0;
        auto loads_behind = [&](auto kind, auto slot) {    // ... matrix instruction `slot` behind the barrier
            constexpr int KIND = decltype(kind)::value, S = decltype(slot)::value, SLOTS = RING == 2 ? 4 : 4 * QUARTERS;
            if constexpr (KIND == ONE_BY_ONE) {
                ring_each<NL>([&](auto load) {
                    constexpr int J = decltype(load)::value, JB = J - CA::NV;
                    if constexpr ((RING == 2 ? J * SLOTS / NL : 4 + J * (SLOTS - 4) / NL) == S) {
                        if constexpr (JB < 0) ring_load<J * WA * 1024>(ca.base, ca.off[J], cur + a_at + wave_a * 1024);
                        else ring_load<JB * WAVES * 1024>(cb.base, cb.off[JB], cur + B_AT + wave8 * 1024);
                    }
                });
            } else if constexpr (KIND == BURSTS) {
                if (S == 0) fetch_a(t + RING, cur);
                if (S == (RING == 2 ? 0 : 4)) fetch_b(t + RING, cur);
            }
        };
        auto last_quarter = [&](auto kind) {
            ring_each<4>([&](auto m) {
                constexpr int M = decltype(m)::value;
                PH_PIN; read(fr[0], next, 0, m); PH_PIN;
                PH_MFMA(1, M / 2, M % 2); PH_PIN;
                loads_behind(kind, m);
            });
        };
        // of step `step`, in slot `at`; fr[0] holds the operands of the first
        auto other_quarters = [&](auto kind, int step, uint32_t at) {
            ring_each<QUARTERS - 1>([&](auto quarter) {
                constexpr int q = decltype(quarter)::value;
                ring_each<4>([&](auto m) {
                    constexpr int M = decltype(m)::value;
                    PH_PIN; read(fr[(q + 1) & 1], at, q + 1, m); PH_PIN;
                    PH_MFMA(q & 1, M / 2, M % 2); PH_PIN;
                    if constexpr (RING > 2) loads_behind(kind, std::integral_constant<int, 4 + 4 * q + M>{});
                });
            });
        };
        auto between_barriers = [&](auto kind) {
            next = cur + STAGE == lds0 + RING * STAGE ? lds0 : cur + STAGE;
            last_quarter(kind);
            other_quarters(kind, t + 1, next);
            cur = next;
            ++t;
        };
        other_quarters(std::integral_constant<int, NO_LOADS>{}, 0, lds0);
        // (each barrier: the next stage has landed, and everybody has read this one)
        constexpr bool BURSTS_TOO = KA == KB && (KA == LD_KC || DUAL);         // (what the host sets it for)
        if (sa.regular && sb.regular && !(BURSTS_TOO && P.bursts)) {           // uniform
            while (t + RING < steps) {
                ring_run<KA, WA>(ca, sa, a_off0, a_off1, c_of(t + RING));
                ring_run<KB, WAVES>(cb, sb, b_off0, b_off1, c_of(t + RING));
                for (int run = min(min(ca.left, cb.left) + 1, steps - RING - t); run > 0; --run) {
                    ring_wait<(RING - 2) * NL>();
                    between_barriers(std::integral_constant<int, ONE_BY_ONE>{});
                    ca.base = (const __bf16 *)((uintptr_t)ca.base - ca.step);
                    cb.base = (const __bf16 *)((uintptr_t)cb.base - cb.step);
                }
            }
        } else {
            while (t + RING < steps) {
                ring_wait<(RING - 2) * NL>();
                between_barriers(std::integral_constant<int, BURSTS>{});
            }
        }
        while (t + 1 < steps) {
            ring_wait_stage<NL, RING - 2>(steps - 2 - t);
            between_barriers(std::integral_constant<int, NO_LOADS>{});
        }
        last_quarter(std::integral_constant<int, NO_LOADS>{});
    }
    if constexpr (LEVELS) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = sums[i][j];
    }
#undef PH_PIN
#undef PH_MFMA
#undef PH_FOLD
}

// The same for operands in 8-byte vectors, through registers: two stages per team, loads two of the team's steps ahead.
// TILE_SHARED: the teams take alternate steps.
template <int KA, int KB, int VA, int VB, int MODE>
__device__ __forceinline__ void reduce_in_registers(const MfmaIn &P, int g, int m0, int n0, int tm, int k_begin, int k_end,
                                                    f32x16 (&acc)[2][2], unsigned char *smem_raw)
{
    constexpr bool DUAL = MODE == TILE_DUAL, SOLO = MODE == TILE_SOLO;
    constexpr int BP = DUAL ? 2 : 1;                   // share of the B tile one team stages
    constexpr bool PLAIN = KA == LD_KM && KB == LD_KM; // (see stage_init)
    const int team = SOLO ? 0 : (int)threadIdx.x >> 8;
    const int team_u = __builtin_amdgcn_readfirstlane(team);
    const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    typedef StageCfg<KA, VA> SA;
    typedef StageCfg<KB, VB, BP> SB;
    int a_off0[SA::NV], a_off1[SA::NV], b_off0[SB::NV], b_off1[SB::NV];
    // a DUAL team whose tile lies below the last row still stages its half of B and keeps the barriers:
    // its loaders read the last valid row, its epilogue writes nothing
    const StageState sa = stage_init<KA, VA, 1, PLAIN>(P.a, g, min(m0, (P.M - 1) / MT * MT), P.M, k_end, tid, a_off0, a_off1);
    const StageState sb = stage_init<KB, VB, BP, PLAIN>(P.b, g, n0, P.N, k_end, tid, b_off0, b_off1,
                                                 DUAL ? team_u * (SB::ROWS / 2) : 0);
    PH_PHASE(7);
    typename SA::V ra0[SA::NV], ra1[SA::NV];
    typename SB::V rb0[SB::NV], rb1[SB::NV];
#define PH_FETCH(set, c0) do { stage_fetch<KA, VA, true, 1, PLAIN>(sa, a_off0, a_off1, ra##set, (c0)); \
                               stage_fetch<KB, VB, true, BP, PLAIN>(sb, b_off0, b_off1, rb##set, (c0)); } while (0)
#define PH_STORE(set, stage, c0) do { stage_store<KA, VA, true>(sa, ra##set, s##stage##a, (c0)); \
                                      stage_store<KB, VB, true, BP>(sb, rb##set, s##stage##b, (c0)); } while (0)

#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    PH_PHASE(1);

    // LDS: two stages per operand tile.  Two teams on one tile: each team has its own A and B stages
    // (8 tiles).  DUAL: own A stages, the B stages are common (6 tiles).
    __bf16 *smem = (__bf16 *)smem_raw;
    __bf16 *s0a, *s0b, *s1a, *s1b;
    if (DUAL) {
        s0a = smem + team * 2 * TILE_ELEMS; s1a = s0a + TILE_ELEMS;
        s0b = smem + 4 * TILE_ELEMS; s1b = s0b + TILE_ELEMS;
    } else {
        s0a = smem + team * 4 * TILE_ELEMS; s0b = s0a + TILE_ELEMS; s1a = s0a + 2 * TILE_ELEMS; s1b = s0a + 3 * TILE_ELEMS;
    }
    // The reduction range is cut into tiles of KT.  Two teams on one tile: team q takes the tiles q, q+2, ...;
    // DUAL: every team takes every tile.  Both teams pass the same number of barriers (`steps`).
    const int all_steps = (k_end - k_begin + KT - 1) / KT;
    const int steps = DUAL || SOLO ? all_steps : (all_steps + 1) >> 1;
    const int my_steps = DUAL || SOLO ? all_steps : (all_steps - team_u + 1) >> 1;      // tiles this team really has
    constexpr int KS = DUAL || SOLO ? KT : 2 * KT;
    const int kfirst = DUAL || SOLO ? k_begin : k_begin + team_u * KT;     // start of this team's first tile
    // Regular shapes walk their tiles from the LAST one down: the only tile that can be ragged (the end of the
    // reduction range) then comes first and is staged by the careful prologue; every later tile is a full
    // one and every step takes the fast path.  Other shapes walk upwards through the general loop.
    const bool regular = sa.regular && sb.regular &&
                         (!DUAL || tile_is_regular<KA, PLAIN>(P.a, min((tm * 2 + (1 - team_u)) * MT, (P.M - 1) / MT * MT)));
    int t = 0;
    if (PLAIN || regular) {                                         // uniform (in DUAL for both teams alike)
        const int c_last = kfirst + (my_steps - 1) * KS;            // start of the tile processed first
        auto c_of = [c_last](int i) { return c_last - i * KS; };    // tile processed in step i (i < my_steps)
        // only that first tile needs the careful loader (clamped indices, zeroed tail: some 30 vector instructions
        // per fetch and operand); a full one and the two tiles behind it take the loop's own addressing
#define PH_FETCH_FAST(set, c0) do { \
        const FastStep fa_ = fast_step_addr<KA, VA, PLAIN>(sa, (c0)), fb_ = fast_step_addr<KB, VB, PLAIN>(sb, (c0)); \
        fast_fetch<KA, VA, 1, 0, SA::NV, PLAIN>(fa_, a_off0, a_off1, ra##set); \
        fast_fetch<KB, VB, BP, 0, SB::NV, PLAIN>(fb_, b_off0, b_off1, rb##set); } while (0)
        const bool ragged_first = my_steps > 0 && c_of(0) + KT > k_end;     // the same for the whole team
        if (ragged_first) PH_FETCH(0, c_of(0));
        else if (my_steps > 0) PH_FETCH_FAST(0, c_of(0));
        if (my_steps > 1) PH_FETCH_FAST(1, c_of(1));
        if (ragged_first) {
            PH_STORE(0, 0, c_of(0));
        } else if (my_steps > 0) {
            stage_store<KA, VA, false>(sa, ra0, s0a, 0);
            stage_store<KB, VB, false, BP>(sb, rb0, s0b, 0);
        }
        if (my_steps > 2) PH_FETCH_FAST(0, c_of(2));
#undef PH_FETCH_FAST
        __syncthreads();
        PH_PHASE(2);
        // step i multiplies LDS stage i%2; on entry tile i+1 sits in register set (i+1)%2 and is moved to the other
        // stage (whose readers finished before the barrier inside step i-1), tile i+2 in the other set
        bf16x8 fr[2][4];
        read_operands<KA, KB>(fr[0], s0a, s0b, wm, wn, 0, lane);
        for (; t + 1 < steps && t + 4 < my_steps; t += 2) {          // everything these two steps touch exists
            fast_step<KA, KB, VA, VB, BP, false, PLAIN>(acc, fr, s0a, s0b, wm, wn, lane, sa, a_off0, a_off1, ra1, s1a, sb, b_off0, b_off1,
                                                       rb1, s1b, c_of(t + 3), true, true, true);
            fast_step<KA, KB, VA, VB, BP, false, PLAIN>(acc, fr, s1a, s1b, wm, wn, lane, sa, a_off0, a_off1, ra0, s0a, sb, b_off0, b_off1,
                                                       rb0, s0b, c_of(t + 4), true, true, true);
        }
        for (; t + 1 < steps; t += 2) {                              // the last steps: the pipeline runs empty
            fast_step<KA, KB, VA, VB, BP, true, PLAIN>(acc, fr, s0a, s0b, wm, wn, lane, sa, a_off0, a_off1, ra1, s1a, sb, b_off0, b_off1,
                                                      rb1, s1b, c_of(t + 3), t < my_steps, t + 1 < my_steps, t + 3 < my_steps);
            fast_step<KA, KB, VA, VB, BP, true, PLAIN>(acc, fr, s1a, s1b, wm, wn, lane, sa, a_off0, a_off1, ra0, s0a, sb, b_off0, b_off1,
                                                      rb0, s0b, c_of(t + 4), t + 1 < my_steps, t + 2 < my_steps, t + 4 < my_steps);
        }
        if (t < steps)
            fast_step<KA, KB, VA, VB, BP, true, PLAIN>(acc, fr, s0a, s0b, wm, wn, lane, sa, a_off0, a_off1, ra1, s1a, sb, b_off0, b_off1,
                                                      rb1, s1b, 0, t < my_steps, false, false);
    } else if constexpr (!PLAIN) {
        // prologue: tile 0 into LDS stage 0; tiles 1 and 2 on their way in register sets 1 and 0.  A tile past the
        // end of the range (the shorter team's last step) is stored as zeros.
        PH_FETCH(0, kfirst);
        PH_FETCH(1, kfirst + KS);
        PH_STORE(0, 0, kfirst);
        PH_FETCH(0, kfirst + 2 * KS);
        __syncthreads();
        PH_PHASE(2);
#define PH_STEP(set, cur, nxt, c_store, c_fetch) do { \
        fused_quarter<KA, KB, VA, VB, true, 0, BP>(acc, s##cur##a, s##cur##b, wm, wn, lane, sa, a_off0, a_off1, ra##set, s##nxt##a, sb, b_off0, b_off1, rb##set, s##nxt##b, (c_store), (c_fetch)); \
        fused_quarter<KA, KB, VA, VB, true, 1, BP>(acc, s##cur##a, s##cur##b, wm, wn, lane, sa, a_off0, a_off1, ra##set, s##nxt##a, sb, b_off0, b_off1, rb##set, s##nxt##b, (c_store), (c_fetch)); \
        fused_quarter<KA, KB, VA, VB, true, 2, BP>(acc, s##cur##a, s##cur##b, wm, wn, lane, sa, a_off0, a_off1, ra##set, s##nxt##a, sb, b_off0, b_off1, rb##set, s##nxt##b, (c_store), (c_fetch)); \
        fused_quarter<KA, KB, VA, VB, true, 3, BP>(acc, s##cur##a, s##cur##b, wm, wn, lane, sa, a_off0, a_off1, ra##set, s##nxt##a, sb, b_off0, b_off1, rb##set, s##nxt##b, (c_store), (c_fetch)); \
    } while (0)
        for (; t + 1 < steps; t += 2) {
            PH_STEP(1, 0, 1, kfirst + (t + 1) * KS, kfirst + (t + 3) * KS);
            __syncthreads();
            PH_STEP(0, 1, 0, kfirst + (t + 2) * KS, kfirst + (t + 4) * KS);
            __syncthreads();
        }
#undef PH_STEP
        if (t < steps) mfma_tile<KA, KB>(acc, s0a, s0b, wm, wn, lane);
    }
#undef PH_FETCH
#undef PH_STORE
}

// One workgroup's work: workgroup number wg (of P.total_wg, in tile order) of the product P.
// FOLD (the forward layout with 8-element vectors, regular shapes only): the workgroup also computes its block of
// the compression F (FoldParams).
// read_out(): the epilogue's part of the parameters, read behind the reduction.
template <int KA, int KB, int VA, int VB, typename TOut, int MODE, int EPI, bool FOLD = false, int LEVELS = ONE_SUM, typename ReadOut>
__device__ __forceinline__ void mfma_workgroup(const MfmaIn &P, int wg, ReadOut read_out, const FoldParams *Fp = nullptr)
{
    static_assert(!LEVELS || VA == 8, "on the ring only");
    static_assert(!FOLD || (KA == LD_KC && KB == LD_KC && VA == 8 && MODE == TILE_SHARED), "the compression rides with the forward product only");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    constexpr bool DUAL = MODE == TILE_DUAL, SOLO = MODE == TILE_SOLO;
    PH_PHASE(0);
    const int tiles = P.tiles_m * P.tiles_n;           // DUAL: tiles_m counts pairs of tile rows
    int rem = div_by(wg, tiles, P.magic_tiles);        // group * ksplit + piece
    const int g = P.ksplit > 1 ? rem / P.ksplit : rem, ks = rem - g * P.ksplit;
    rem = wg - rem * tiles;
    constexpr int RASTER_M = mfma_raster(DUAL);
    const int band = div_by(rem, RASTER_M * P.tiles_n, P.magic_band);
    const int in_band = rem - band * (RASTER_M * P.tiles_n);
    const int band_rows = min(P.tiles_m - band * RASTER_M, RASTER_M);
    const int tn = band_rows == RASTER_M ? in_band / RASTER_M : in_band / band_rows;
    const int tm = band * RASTER_M + (in_band - tn * band_rows);
    const int team = SOLO ? 0 : (int)threadIdx.x >> 8;
    const int team_u = __builtin_amdgcn_readfirstlane(team);
    const int m0 = DUAL ? (tm * 2 + team_u) * MT : tm * MT, n0 = tn * MT;
    const int k_begin = ks * P.k_per_split;
    const int k_end = min(P.K, k_begin + P.k_per_split);
    PH_PHASE(6);

    const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    // the compression's block of this workgroup: block tn of its tile row (block = 32 rows x 32 phantom neurons)
    FoldState fs;
    int e_rb = 0, e_cb = 0;
    fs.on = false; fs.owner = false;
    if constexpr (FOLD) {
        const FoldParams &F = *Fp;
        fs.on = tn < F.nblocks;
        e_rb = tn / F.ncb; e_cb = tn - e_rb * F.ncb;
        fs.owner = fs.on && __builtin_amdgcn_readfirstlane(wave) == (e_rb >> 1) * 2 + team_u;   // a wavefront with wm = 64 (rb / 2); the teams' on different SIMDs
        fs.own_hi = e_rb & 1;
        fs.limit = F.K;
        const int erow = (int)(threadIdx.x >> 6) * 4 + (lane >> 3);                    // half of a wavefront: 4 rows of 8 vectors
        fs.base = F.C + g * F.c_g + (int64_t)(e_cb * 32) * F.K;
        fs.src_off = (unsigned)(min(erow, F.N - 1 - e_cb * 32) * F.K + ((lane & 7) ^ ring_swizzle<LD_KC>(erow)) * 8) * 2u;
#pragma unroll
        for (int e = 0; e < 16; ++e) fs.acc[e] = 0.f;
    }
    f32x16 acc[2][2];
    if constexpr (VA == 8) reduce_in_ring<KA, KB, MODE, FOLD, LEVELS>(P, g, m0, n0, tn, k_begin, k_end, acc, fs, (uint32_t)(uintptr_t)(LdsBytes)smem_raw);
    else reduce_in_registers<KA, KB, VA, VB, MODE>(P, g, m0, n0, tm, k_begin, k_end, acc, smem_raw);
    const MfmaOut Q = read_out();
    __syncthreads();
    PH_PHASE(3);

    // each team writes its fp32 tile over the staging space (free after the barrier above).  Two teams
    // on one tile hold partial sums of it: the epilogue adds the two while reading.
    float *ctile = (float *)smem_raw;
    constexpr bool PIECES = MODE == TILE_SHARED && !FOLD && EPI == EPI_STORE && sizeof(TOut) == 4 && VA == 8;
    const int thread = DUAL || SOLO ? tid : (int)threadIdx.x;
    const bool piece = PIECES && Q.parts && P.ksplit > 1;            // uniform (one group: the host sees to that)
    auto finish = [&](auto vec, auto act) {
        EpilogueReads<decltype(vec)::value, TOut, MODE, EPI> reads;
        if (!piece) epilogue_request(reads, P, Q, g, m0, n0, thread);
        acc_to_lds(ctile + team * CT_ELEMS, acc, wm, wn, lane);
        __syncthreads();
        PH_PHASE(4);
        if constexpr (PIECES)
            if (piece) epilogue_pieces_from_lds(P, Q, rem, ks, ctile, (unsigned *)(ctile + 2 * CT_ELEMS), m0, n0, thread);
        if (!piece)
            epilogue_from_lds<decltype(vec)::value, TOut, MODE, EPI, decltype(act)::value>(P, Q, g, ctile + (DUAL || SOLO ? team * CT_ELEMS : 0), m0, n0, thread,
                                                                                            ctile + (SOLO ? 1 : 2) * CT_ELEMS, reads);
    };
    // 16 bytes per thread and store, see epilogue_from_lds (with 8 elements, GELU alone, whose derivative nobody wants, is 1 % faster than with 4)
    typedef std::integral_constant<int, sizeof(TOut) == 4 ? 4 : VA> Wide;
    typedef std::integral_constant<int, EPI_PIECEWISE> Piecewise;
    if constexpr (EPI == EPI_BIAS_ACT) {
        if (Q.ep.act != ACT_GELU) finish(Wide{}, Piecewise{});       // (uniform choices)
        else if (Q.ep.aux && Q.ep.aux_deriv) finish(std::integral_constant<int, 4>{}, std::integral_constant<int, EPI_GELU_DERIV>{});
        else finish(Wide{}, std::integral_constant<int, EPI_GELU>{});
    } else {
        finish(Wide{}, Piecewise{});
    }
    PH_PHASE(5);
    if constexpr (FOLD) {
        if (fs.on) {                                                 // uniform
            // the block of g: two teams on one tile hold partial sums of it (half of every step each): team 1's goes
            // through LDS to team 0's owner.  A lane holds row (lane & 31) of the block and the columns
            // 8 * (e / 4) + 4 * (lane >> 5) + e % 4 (B operand first, as in acc_to_lds).
            const FoldParams &F = *Fp;
            float *ex = (float *)smem_raw;
            if (!DUAL) {
                __syncthreads();                                     // the tile's epilogue is done with LDS
                if (fs.owner && team == 1) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) ex[e * 64 + lane] = fs.acc[e];
                }
                __syncthreads();
                if (fs.owner && team == 0) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) fs.acc[e] += ex[e * 64 + lane];
                }
            }
            if (fs.owner && (DUAL || team == 0)) {
                const int m = m0 + 32 * e_rb + (lane & 31);
                if (m < P.M) {
                    __bf16 *row = F.G + g * F.o_g + (int64_t)m * F.N;
                    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int c = 32 * e_cb + 8 * q + 4 * (lane >> 5);
                        if (c < F.N) {                               // N is a multiple of 8: four columns at a time stay inside
                            bf16x4 v = {(__bf16)fs.acc[4 * q], (__bf16)fs.acc[4 * q + 1], (__bf16)fs.acc[4 * q + 2], (__bf16)fs.acc[4 * q + 3]};
                            *(bf16x4 *)(row + c) = v;
                        }
                    }
                }
            }
        }
    }
}

template <int KA, int KB, int VA, int VB, typename TOut, bool PAIR, int MODE, int EPI>
__global__ __launch_bounds__(mfma_threads(MODE), MODE == TILE_SOLO ? 2 : 1) void gemm_mfma_kernel(MfmaBatch batch)
{
    // (launches of their own took 4.8 us: dense 4 x 4096 trained at batch 1024, which has both, 573 -> 563 us a step)
    if constexpr (EPI == EPI_BIAS_ACT) clear_rider(batch.ride.clear, (int)blockIdx.x, (int)gridDim.x, mfma_threads(MODE));
    if constexpr (sizeof(TOut) == 4) {
        if (blockIdx.x == 0 && batch.ride.tail.partial) {      // uniform
            extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
            finish_loss(batch.ride.tail, (float *)smem_raw);
            __syncthreads();
        }
    }
    int wg = xcd_order(blockIdx.x, 0, batch.total_wg);
    const bool second = PAIR && wg >= batch.first_wg;
    if (second) wg -= batch.first_wg;
    const size_t at = second ? offsetof(MfmaBatch, p[1]) : offsetof(MfmaBatch, p[0]);
    mfma_workgroup<KA, KB, VA, VB, TOut, MODE, EPI>(in_from_args(at), wg, OutFromArgs{at});
}

// Several independent products of one shape class in one launch: the compressions of all layers of one rank with more
// phantom neurons than thin_product.h takes.  One rank's g goes to the peers and nothing on the rank waits for it, so they
// go out together behind the forward pass: alone, a layer's fills half of the compute units (configuration 5, k = 256: 128
// tiles, 16.4 us a layer, 6 layers).
constexpr int MANY_PRODUCTS = 6;
struct MfmaMany {
    MfmaParams p[MANY_PRODUCTS];
    int count;
    int first_wg[MANY_PRODUCTS + 1];       // multiples of 8
};
static_assert(sizeof(MfmaMany) <= 3840, "travels as kernel arguments (4 KB with the hidden ones)");

template <int VEC, bool DUAL>
__global__ __launch_bounds__(512, 1) void gemm_mfma_many_kernel(MfmaMany many)
{
    int j = 0;
    while (j + 1 < many.count && (int)blockIdx.x >= many.first_wg[j + 1]) ++j;          // uniform
    const size_t at = offsetof(MfmaMany, p) + (size_t)j * sizeof(MfmaParams);
    const MfmaIn P = in_from_args(at);
    const int local = (int)blockIdx.x - many.first_wg[j];
    if (local >= P.total_wg) return;
    mfma_workgroup<LD_KC, LD_KC, VEC, VEC, __bf16, DUAL, EPI_STORE>(P, xcd_order(local, 0, P.total_wg), OutFromArgs{at});
}

// The last launch of a layer's backward pass, the weight + compressor gradients (tail[0], tail[1]: weight-gradient
// layout, float out; tail[1] may be empty: total_wg = 0), with up to two riders that need nothing it produces:
//  - head, all ranks on the device: the error compression of the layer below (input-gradient layout, storage
//    type out), which fills half of the device or less for a short while.  It runs in the workgroups
//    [0, head_wg) so that it is dispatched first and frees its compute units early.
//    One rank, first layer (no input gradient to share a launch with): the layer's own error compression.  Nothing
//    waits for it, so with more workgroups than compute units it goes out last (rotate) and fills in behind the
//    longer weight-gradient workgroups.
//  - the loss's final sum, one more workgroup.
// tail_first is a multiple of 8; workgroups in the gap do nothing.
struct MfmaTailBatch {
    MfmaParams head;
    MfmaParams tail[2];
    LossTail loss;
    int head_wg;         // = head.total_wg (0: no head)
    int tail_first;
    int tail_wg;         // = tail[0].total_wg + tail[1].total_wg
    int tail0_wg;        // = tail[0].total_wg
    int loss_first;      // the workgroup behind the tail's finishes the loss (loss.partial != NULL)
    int rotate;          // workgroup b does the work of number (b + rotate) mod the grid size: rotate = tail_first
                         //   sends the head's workgroups out last instead of first
    int dual;            // every product of the launch in two-tile workgroups (DUAL of mfma_workgroup): for a launch
                         //   that would otherwise not fit one workgroup per compute unit
};

template <int VEC>
__global__ __launch_bounds__(512, 1) void gemm_mfma_tail_kernel(MfmaTailBatch tb)
{
    int id = (int)blockIdx.x + tb.rotate;
    if (id >= (int)gridDim.x) id -= (int)gridDim.x;
    if (id < tb.tail_first) {                          // uniform, like every branch here
        if (id >= tb.head_wg) return;
        constexpr size_t at = offsetof(MfmaTailBatch, head);
        const MfmaIn P = in_from_args(at);
        if (tb.dual) mfma_workgroup<LD_KC, LD_KM, VEC, VEC, __bf16, true, EPI_STORE>(P, xcd_order(id, 0, tb.head_wg), OutFromArgs{at});
        else mfma_workgroup<LD_KC, LD_KM, VEC, VEC, __bf16, false, EPI_STORE>(P, xcd_order(id, 0, tb.head_wg), OutFromArgs{at});
    } else if (id < tb.loss_first) {
        // the XCD-aware order within each product
        int wg = id - tb.tail_first;
        const bool second = wg >= tb.tail0_wg;
        if (second) wg -= tb.tail0_wg;
        wg = xcd_order(wg, 0, second ? tb.tail_wg - tb.tail0_wg : tb.tail0_wg);
        const size_t at = second ? offsetof(MfmaTailBatch, tail[1]) : offsetof(MfmaTailBatch, tail[0]);
        const MfmaIn P = in_from_args(at);
        if (tb.dual) mfma_workgroup<LD_KM, LD_KM, VEC, VEC, float, true, EPI_STORE>(P, wg, OutFromArgs{at});
        else mfma_workgroup<LD_KM, LD_KM, VEC, VEC, float, false, EPI_STORE>(P, wg, OutFromArgs{at});
    } else {
        extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
        finish_loss(tb.loss, (float *)smem_raw);
    }
}

// One rank's weight and compressor gradients of ALL layers in one launch, at the end of the backward pass.
// They depend on nothing but each layer's delta and input, one layer's cover few of the 256 compute units with
// narrow shards (configuration 4: 128 + 8 tiles of 64 reduction steps), and a launch per layer ends when its
// slowest tile does; together they are 1088 tiles that the hardware deals out as compute units come free
// (8 launches of 41 us against one of 170 us).  The SGD update runs in the epilogues (SgdInPlace): every
// launch that reads the weights has finished by then.
// The products' parameter blocks do not fit the 4 KB of kernel arguments (16 blocks of some 600 bytes), so they sit in
// a table in device memory that small launches fill beforehand (table_upload_kernel).  Product j has the
// workgroups [first_wg[j], first_wg[j + 1]) (starts are multiples of 8; workgroups beyond a product's own do nothing).
constexpr int TABLE_PRODUCTS = 32;
constexpr int CHUNK_PRODUCTS = 5;          // parameter blocks per upload launch: kernel arguments hold 4 KB

struct ProductTable {
    int count;
    int first_wg[TABLE_PRODUCTS + 1];
    int wgs[TABLE_PRODUCTS];               // = p[j].total_wg
    int dual[TABLE_PRODUCTS];              // product j in two-tile workgroups (DUAL of mfma_workgroup)
    LossTail tail;                         // workgroup 0 finishes the loss first (partial == NULL: nothing to do)
    MfmaParams p[TABLE_PRODUCTS];
};

struct TableChunk {
    int at, n;                             // blocks p[0 .. n) go to the table's entries at .. at + n
    int count;                             // the table's count once every chunk is there
    int first_wg[CHUNK_PRODUCTS + 1];      // first_wg[at .. at + n]
    int wgs[CHUNK_PRODUCTS];
    int dual[CHUNK_PRODUCTS];
    LossTail tail;
    MfmaParams p[CHUNK_PRODUCTS];
};
static_assert(sizeof(TableChunk) + sizeof(void *) <= 3840, "a chunk travels as kernel arguments (4 KB with the hidden ones)");

// one workgroup of 256 threads copies a chunk from the kernel arguments into the table
__global__ __launch_bounds__(256) void table_upload_kernel(TableChunk c, ProductTable *table)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const uint32_t __attribute__((address_space(4))) *ArgWords;
    const ArgWords in = (ArgWords)((const char __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(TableChunk, p));
    uint32_t *out = (uint32_t *)(table->p + c.at);
    const int words = c.n * (int)(sizeof(MfmaParams) / 4);
    for (int i = (int)threadIdx.x; i < words; i += 256) out[i] = in[i];
#endif
    if ((int)threadIdx.x <= c.n) table->first_wg[c.at + threadIdx.x] = c.first_wg[threadIdx.x];
    if ((int)threadIdx.x < c.n) { table->wgs[c.at + threadIdx.x] = c.wgs[threadIdx.x]; table->dual[c.at + threadIdx.x] = c.dual[threadIdx.x]; }
    if (threadIdx.x == 0) { table->count = c.count; table->tail = c.tail; }
}

// Layers of the same shapes (the uniform network) need no table: their parameter blocks differ in pointers alone, and two
// blocks and every layer's pointers fit the kernel arguments.  (Two small launches less per step: 9 us.)
constexpr int UNIFORM_LAYERS = 12;
struct UniformInputs { const void *dw_a, *dw_b0, *dw_b1, *dc_a; };
struct UniformOutputs {
    void *dw_o0, *dw_o1, *dc_o0;
    float *l_master, *d_master, *c_master, *bias_master;
    void *l_w, *d_w, *c_w, *bias_w;
    const float *bias_grad;
};
struct UniformGradients {
    MfmaParams dw, dc;                     // any layer's blocks (dc.total_wg = 0: no compressor)
    int layers, dc_wg, dw_wg;              // workgroups per layer, multiples of 8
    int dw_dual;
    int64_t parts_layer, arrived_layer;    // floats / words from one layer's pieces to the next's
    LossTail tail;
    struct Pointers { UniformInputs in; UniformOutputs out; } at[UNIFORM_LAYERS];
};
static_assert(sizeof(UniformGradients) <= 3840, "travels as kernel arguments (4 KB with the hidden ones)");

// HALVES: the weight gradients' chains (a step on padded copies: the launches without copies, a layer each, have two teams on a tile and so two sums.
// 2-norm error against 64 bits at 2621 rows, 4 layers of 1152, k 4, two teams : one chain : halves, dL 1.61e-7 : 2.56e-7 : 1.61e-7, dD 1.33e-7 : 2.65e-7 : 1.35e-7;
// trained 300.6 : 189.5 : 190.8 us).
template <int VEC, bool SOLO, bool HALVES>
__global__ __launch_bounds__(SOLO ? 256 : 512, SOLO ? 2 : 1) void gemm_mfma_uniform_kernel(UniformGradients u)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int id = (int)blockIdx.x;
    if (id == 0 && u.tail.partial) {                            // uniform
        finish_loss(u.tail, (float *)smem_raw);
        __syncthreads();
    }
    const bool weights = id >= u.layers * u.dc_wg;
    const int i = weights ? id - u.layers * u.dc_wg : id, per = weights ? u.dw_wg : u.dc_wg;
    const int l = i / per, local = i - l * per;
    const size_t at = weights ? offsetof(UniformGradients, dw) : offsetof(UniformGradients, dc);
    MfmaIn P = in_from_args(at);
    if (local >= P.total_wg) return;
    // this layer's pointers, read where they are needed
    typedef UniformGradients::Pointers Pointers;
    const size_t layer = offsetof(UniformGradients, at) + (size_t)l * sizeof(Pointers);
    {
        const UniformInputs q = args_at<UniformInputs>(layer + offsetof(Pointers, in));
        P.a.p0 = const_cast<void *>(weights ? q.dw_a : q.dc_a);
        P.b.p0 = const_cast<void *>(q.dw_b0);
        if (weights) P.b.p1 = const_cast<void *>(q.dw_b1);
    }
    auto read_out = [=]() {
        MfmaOut Q = OutFromArgs{at}();
        const UniformOutputs q = args_at<UniformOutputs>(layer + offsetof(Pointers, out));
        if (weights) {
            Q.o.p0 = q.dw_o0; Q.o.p1 = q.dw_o1;
            Q.sgd.master0 = q.l_master; Q.sgd.master1 = q.d_master; Q.sgd.w0 = q.l_w; Q.sgd.w1 = q.d_w;
            Q.sgd.bias_master = q.bias_master; Q.sgd.bias_w = q.bias_w; Q.sgd.bias_grad = q.bias_grad;
        } else {
            Q.o.p0 = q.dc_o0;
            Q.sgd.master0 = q.c_master; Q.sgd.w0 = q.c_w;
            Q.parts += l * u.parts_layer; Q.arrived += l * u.arrived_layer;
        }
        return Q;
    };
    // One team has one set of sums: the compressor gradients, which two-tile launches cut into pieces of two teams each, take LEVELS.  2-norm error against 64
    // bits at 4096 rows, shard 512, k 64, pieces : one running sum : levels: 1.35e-7 : 3.95e-7 : 1.37e-7; 8 such layers trained 358.6 : 345.6 : 346.4 us.
    constexpr int WEIGHTS = HALVES ? SUMS_OF_HALVES : ONE_SUM;
    if constexpr (SOLO) {
        if (weights) mfma_workgroup<LD_KM, LD_KM, VEC, VEC, float, TILE_SOLO, EPI_STORE, false, WEIGHTS>(P, xcd_order(local, 0, P.total_wg), read_out);
        else mfma_workgroup<LD_KM, LD_KM, VEC, VEC, float, TILE_SOLO, EPI_STORE, false, SUMS_OF_8>(P, xcd_order(local, 0, P.total_wg), read_out);
    } else if (weights && u.dw_dual) mfma_workgroup<LD_KM, LD_KM, VEC, VEC, float, true, EPI_STORE, false, WEIGHTS>(P, xcd_order(local, 0, P.total_wg), read_out);
    else mfma_workgroup<LD_KM, LD_KM, VEC, VEC, float, false, EPI_STORE>(P, xcd_order(local, 0, P.total_wg), read_out);
}

#if defined(__HIP_DEVICE_COMPILE__)
// a part of the table, read where it is needed (see args_at)
template <typename Part>
__device__ __forceinline__ Part table_at(const Part __attribute__((address_space(4))) *p)
{
    constexpr int WORDS = sizeof(Part) / 4;
    union Words { Part p; uint32_t w[WORDS]; __device__ Words() {} };
    Words out;
    asm volatile("" : "+s"(p) :: "memory");
    typedef const uint32_t __attribute__((address_space(4))) *ArgWords;
#pragma unroll
    for (int i = 0; i < WORDS; ++i) out.w[i] = ((ArgWords)p)[i];
    return out.p;
}
#endif

template <int VEC, bool HALVES>
__global__ __launch_bounds__(512, 1) void gemm_mfma_table_kernel(const ProductTable *table)
{
#if defined(__HIP_DEVICE_COMPILE__)
    // read through the constant address space: the table is not written during this launch, and its entries are
    // the same for every lane (scalar loads)
    typedef const ProductTable __attribute__((address_space(4))) *TablePtr;
    const TablePtr t = (TablePtr)(uintptr_t)table;
    const int id = (int)blockIdx.x;
    if (id == 0 && t->tail.partial) {                           // uniform
        extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
        LossTail tail;
        tail.partial = t->tail.partial; tail.n = t->tail.n; tail.scale = t->tail.scale; tail.loss = t->tail.loss;
        finish_loss(tail, (float *)smem_raw);
        __syncthreads();
    }
    const int count = t->count;
    int j = 0;
    while (j + 1 < count && id >= t->first_wg[j + 1]) ++j;      // uniform
    const int local = id - t->first_wg[j], wgs = t->wgs[j];
    if (local >= wgs) return;
    const MfmaIn P = table_at<MfmaIn>(&t->p[j].in);
    auto read_out = [=]() { return table_at<MfmaOut>(&t->p[j].out); };
    if (t->dual[j]) mfma_workgroup<LD_KM, LD_KM, VEC, VEC, float, true, EPI_STORE, false, (HALVES ? SUMS_OF_HALVES : ONE_SUM)>(P, xcd_order(local, 0, wgs), read_out);
    else mfma_workgroup<LD_KM, LD_KM, VEC, VEC, float, false, EPI_STORE>(P, xcd_order(local, 0, wgs), read_out);
#endif
}

// One rank's forward of a layer in one launch: the layer update, and the thin compression g = C y (see
// thin_product.h), which in one-rank mode do not depend on each other (the peers' g are inputs).  Every
// workgroup takes one tile (or pair of tiles) of the update and then its share of the compression's rows:
// thin_rows consecutive rows (a multiple of 16), all 8 wavefronts splitting the reduction range.  The rows are
// read again right after the update streamed them through the same XCD's L2 (workgroup w's rows lie in the
// band of tile rows that its XCD works on), and no compute unit waits for a compression workgroup: as
// workgroups of their own in front of the update's, the compression's kept half of the device from the
// update for 9 us of a 38 us launch.  6 layers of 1024 + 448 at batch 8192, k 64: 233 us in launches of their own, 210 so.  (A share costs a chain of
// latencies, load -> multiply -> exchange -> store, about 5 us however short it is, and starting its loads
// ahead of the update's epilogue changed nothing.)  Steps of two layers or more with 8-element vectors do without: see compress_many_kernel, 6 such layers
// 223 -> 190 us.
struct MfmaFwdBatch {
    MfmaParams update;
    const __bf16 *X, *C;     // compression operands: X [M, K] per group, C [N, K] per group
    __bf16 *G;               // [M, N] per group
    int M, N, K;
    int64_t x_g, c_g, o_g;
    int update_wg;           // = update.total_wg
    int wg_per_group;        // workgroups of the update per group
    int thin_rows;           // rows of the compression per workgroup: wg_per_group * thin_rows >= M
    ClearList clear;
    FoldParams fold;         // FOLD kernels: the compression inside the update's loop instead (the fields above unused)
};

template <int VEC, bool DUAL, bool FOLD>
__global__ __launch_bounds__(512, 1) void gemm_mfma_fwd_kernel(MfmaFwdBatch fb)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int wg = xcd_order((int)blockIdx.x, 0, fb.update_wg);
    clear_rider(fb.clear, (int)blockIdx.x, (int)gridDim.x, MFMA_THREADS);
    constexpr size_t at = offsetof(MfmaFwdBatch, update);
    const MfmaIn update = in_from_args(at);
    if constexpr (FOLD) {
        // the compression rides inside the update's reduction loop (FoldParams)
        mfma_workgroup<LD_KC, LD_KC, VEC, VEC, __bf16, DUAL, EPI_BIAS_ACT, true>(update, wg, OutFromArgs{at}, &fb.fold);
    } else {
        mfma_workgroup<LD_KC, LD_KC, VEC, VEC, __bf16, DUAL, EPI_BIAS_ACT>(update, wg, OutFromArgs{at});
        const int grp = wg / fb.wg_per_group;
        const int first = (wg - grp * fb.wg_per_group) * fb.thin_rows;
        const int last = min(first + fb.thin_rows, fb.M);
        for (int m0 = first; m0 < last; m0 += THIN_ROWS) {           // uniform
            __syncthreads();                                         // the epilogue, or the block before, is done with LDS
            if (fb.N <= 32) thin_workgroup<2, 8>(fb.X, fb.C, fb.G, last, fb.N, fb.K, fb.x_g, fb.c_g, fb.o_g, m0, grp, (float *)smem_raw);
            else thin_workgroup<4, 8>(fb.X, fb.C, fb.G, last, fb.N, fb.K, fb.x_g, fb.c_g, fb.o_g, m0, grp, (float *)smem_raw);
        }
    }
}

}  // namespace phantom
