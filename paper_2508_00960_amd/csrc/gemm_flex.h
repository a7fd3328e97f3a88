// Products of any shape and either storage type on the matrix cores:
//   C(m, n) = sum_c A(m, c) * B(n, c)
// for the problems that the 128 x 128 kernels of gemm_mfma.h do not fit: fp32 storage, widths and phantom widths that
// are no multiples of their vectors, and launches with too few 128 x 128 tiles to fill the chip.
//
// Vectors.  Both operands are read 16 bytes at a time whatever their alignment (the memory pipe takes any address), and
// an index that is cut into a head and peer segments (views.h) is renumbered so that every piece starts on a vector:
// the head is padded to a multiple of V = 8 (bf16) or 4 (float), and so is every segment.  A vector then never straddles
// two pieces; one at the end of a piece holds fewer than V elements and its tail is masked to zero on the way to LDS
// (reduction index) or never stored (free index).  Such a vector is read beyond its piece, but never beyond the
// piece's last row: there the read starts earlier and the register is shifted.  Both operands of a product share the
// numbering.
//
// Tile and wavefronts.  A team of wavefronts owns a TM x TN tile (2 x 2 wavefronts, or one for a 32 x 32 tile) and
// TEAMS teams of a workgroup share the tile, taking alternate reduction steps; their sums are added in the order of
// the teams through LDS.  Every reduction step goes global -> registers (two steps ahead) -> LDS (two stages; one
// for a team of one wavefront, whose LDS accesses are in order anyway).
//
// fp32 runs on v_mfma_f32_32x32x2_f32: true fp32 products and sums, 256 FLOP per clock and compute unit, twice what
// single (unpacked) vector FMAs reach, and a lane's operand is one float, so LDS has an eighth of the bf16 kernel's
// traffic per cycle and the matrix pipe alone bounds the loop.  Sums in three levels (16 terms, 16 of those, the
// rest), terms in order: one running fp32 sum over a batch of some thousand rows drifts past 1e-5 of a weight gradient.
//
// FINE, bf16: sums in three levels there too (64 terms, 4 of those, the rest).  For problems with an odd width or phantom
// width, or a tensor beyond 2^31 elements; the others' sums are one running sum per team, as on the 128 x 128 kernels.
// Error of the weight gradients against 64 bits, one running sum : levels (2-norm, shard 201, k 13): batch 1030
// 1.3e-7 : 7.2e-8, 4096 4.0e-7 : 9.7e-8, 65536 1.7e-6 : 2.9e-7.  Time (us): 5 layers of 1153, k 9, trained at batch 4096
// 663 : 673, 3 layers of 751, k 11, at batch 1000 101 : 107.  The second accumulator takes the registers of one wavefront
// per SIMD; within those of four it spills (one rank's layer call of 64, shard 512, k 16: 44 -> 71 us).
// Such problems also take GELU and its derivative by erff rather than by the five-term formula of gelu_both: sigma' in float
// is then off by 3.0e-8 (rms over |a| < 3) instead of 6e-8 (4 layers of 1025, k 33, forward at batch 8192, with the levels: 329 -> 374 us).
#pragma once
#include "common.h"
#include "elementwise.h"
#include "epilogue.h"
#include "launch_rules.h"
#include "mfma_ring.h"

namespace phantom {

template <typename T> struct FlexType;
template <> struct FlexType<bf16_t> { static constexpr int V = 8; };     // elements per vector
template <> struct FlexType<float> { static constexpr int V = 4; };
// reduction step of a team of `team` threads
template <typename T> constexpr int flex_step(int team) { return sizeof(T) == 2 ? 64 : team == 64 ? 16 : 32; }

enum { FLEX_KC = 0, FLEX_KM = 1 };   // reduction index contiguous / free index contiguous in memory

struct FlexAxis {        // one index of a product, as the kernel numbers it
    int head, head_pad;  // length of the head block, and padded
    int seg, seg_pad;    // length of a peer segment, and padded; 0: there are none
    int total;           // padded length of the whole index
    uint32_t magic;      // ceil(2^32 / seg_pad)
};

struct FlexOperand {
    const void *p0, *p1; // head block, peer segments
    int64_t g0, g1;      // elements from one group to the next
    int64_t ld0, ld1;    // elements from one position of the strided index to the next, in each region
    int64_t seg_stride;
    int skip0, skip_g;   // slot skip0 + group * skip_g of the segments' buffer is passed over
    int tiny;            // one of the buffers may have fewer than V elements altogether
};

// A product's parameter block: what its reduction needs ...
struct FlexIn {
    FlexOperand a, b;
    FlexAxis k, n;       // reduction index, column index
    int M;
    int tiles_m, tiles_n, total_wg;
    uint32_t magic_tiles, magic_band, magic_last;      // div_by: tiles_m * tiles_n, FLEX_RASTER * tiles_n, rows of the last band
    int kind;            // 0: A along the reduction index (forward and input-gradient layouts); 1: weight-gradient layout
    int rowsum;          // FlexOut::rowsum is wanted
    SumOnRead rs;        // gemm_flex_f32_few_kernel: A's block dg_own is summed on read (src != nullptr)
};
// ... and what its epilogue needs
struct FlexOut {
    void *o0, *o1;       // output regions (the column index decides)
    int64_t o_g0, o_g1, o_ld0, o_ld1, o_seg_stride;
    Epilogue ep;
    SgdInPlace sgd;
    float *rowsum;       // weight-gradient layout, optional: [M] per group <- sums of A over the reduction index (Eq. (bpb))
};
struct FlexParams {
    FlexIn in;
    FlexOut out;
};

constexpr int FLEX_RASTER = 8;            // tile rows per band: tiles are walked in bands, down the band first (see gemm_mfma.h)
struct FlexTileAt { int g, tm, tn; };
// MAGIC: divides by the host's reciprocals: the kernels on the ring, and fp32 in 64 x 64 tiles (all 8 ranks of 512 trained, 980 -> 965 us,
// 974 with divisions).  Elsewhere the reduction leaves them no scalar registers (layers of 1024 at batch 48, 72 workgroups: 8.1 us a
// launch with divisions, 8.3 with reciprocals; ranks of 750 trained at batch 1000: 89.9 us a step, 90.9).
template <bool MAGIC> __device__ __forceinline__ FlexTileAt flex_tile_at(const FlexIn &P, int wg)
{
    FlexTileAt t;
    auto div = [](int n, int d, uint32_t magic) { return MAGIC ? div_by(n, d, magic) : n / d; };
    t.g = div(wg, P.tiles_m * P.tiles_n, P.magic_tiles);
    const int rem = wg - t.g * (P.tiles_m * P.tiles_n);
    const int band = div(rem, FLEX_RASTER * P.tiles_n, P.magic_band);
    const int in_band = rem - band * (FLEX_RASTER * P.tiles_n);
    const int band_rows = min(P.tiles_m - band * FLEX_RASTER, FLEX_RASTER);
    t.tn = MAGIC && band_rows == FLEX_RASTER ? in_band / FLEX_RASTER : div(in_band, band_rows, P.magic_last);
    t.tm = band * FLEX_RASTER + (in_band - t.tn * band_rows);
    return t;
}

constexpr int FLEX_MAX_PRODUCTS = 4;
struct FlexBatch {
    FlexParams p[FLEX_MAX_PRODUCTS];
    int count;
    int first_wg[FLEX_MAX_PRODUCTS];   // multiples of 8
    LossTail tail;       // the first workgroup also finishes the loss (partial == NULL: nothing to do)
};

static_assert(sizeof(FlexBatch) <= 3840, "a batch travels as kernel arguments (4 KB with the hidden ones)");

struct FlexLoc {         // where a position of an index lies
    int region;
    int64_t off;         // of the position inside its region, contiguous direction
    int in_piece;        // position inside the head or segment
    int len;             // length of that piece
};

// second ? b : a, on values: between members of a structure the compiler would choose an address instead and force the
// structure into memory
template <typename I> __device__ __forceinline__ I flex_pick(bool second, I a, I b) { return a ^ ((a ^ b) & -(I)second); }

__device__ __forceinline__ FlexLoc flex_locate(const FlexAxis &ax, int idx, int64_t seg_stride, int skip)
{
    FlexLoc l;
    const bool tail = idx >= ax.head_pad;
    const unsigned t = tail ? (unsigned)(idx - ax.head_pad) : 0u;
    unsigned i = flex_pick<unsigned>(ax.seg_pad <= 1, __umulhi(t, ax.magic), t);
    i -= i * (unsigned)ax.seg_pad > t ? 1u : 0u;       // the rounded-up reciprocal is at most one too high
    const int w = (int)(t - i * (unsigned)ax.seg_pad), slot = (int)i + ((int)i >= skip ? 1 : 0);
    l.region = tail ? 1 : 0;
    l.in_piece = flex_pick(tail, idx, w);
    l.len = flex_pick(tail, ax.head, ax.seg);
    l.off = flex_pick<int64_t>(tail, idx, (int64_t)slot * seg_stride + w);
    return l;
}

// 16 bytes at any element boundary
template <typename T> struct FlexVec;
template <> struct FlexVec<bf16_t> {
    typedef uint32_t Any __attribute__((ext_vector_type(4), aligned(2)));
    static __device__ __forceinline__ u32x4 keep(u32x4 v, int valid)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] &= valid >= 2 * i + 2 ? 0xffffffffu : valid == 2 * i + 1 ? 0xffffu : 0u;
        return v;
    }
    static __device__ __forceinline__ u32x4 shift(u32x4 v, int n)        // element u <- element u + n (0 behind the last)
    {
        v = n & 4 ? u32x4{v[2], v[3], 0u, 0u} : v;
        v = n & 2 ? u32x4{v[1], v[2], v[3], 0u} : v;
        const int bits = (n & 1) * 16;
        return u32x4{__builtin_amdgcn_alignbit(v[1], v[0], bits), __builtin_amdgcn_alignbit(v[2], v[1], bits),
                     __builtin_amdgcn_alignbit(v[3], v[2], bits), __builtin_amdgcn_alignbit(0u, v[3], bits)};
    }
};
template <> struct FlexVec<float> {
    typedef uint32_t Any __attribute__((ext_vector_type(4), aligned(4)));
    static __device__ __forceinline__ u32x4 keep(u32x4 v, int valid)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = i < valid ? v[i] : 0u;
        return v;
    }
    static __device__ __forceinline__ u32x4 shift(u32x4 v, int n)
    {
        v = n & 2 ? u32x4{v[2], v[3], 0u, 0u} : v;
        v = n & 1 ? u32x4{v[1], v[2], v[3], 0u} : v;
        return v;
    }
};
template <typename T> __device__ __forceinline__ u32x4 flex_load(const T *p)
{
    typedef typename FlexVec<T>::Any Any;
    return gload<Any>(p);
}

// How TT threads stage an operand tile of TF free positions x KT reduction positions.
// KC: LDS rows = free positions, 16 bytes of padding per row: 16 lanes of an operand read fall on all banks.  float: eight
//     reduction positions of a row are kept in the order 0 2 4 6 1 3 5 7, see flex_operand.
// KM: LDS rows = reduction positions.  bf16: four rows that a transposing read touches start 16 banks apart.
//     float: neighbouring rows (the two halves of a wavefront) start 32 banks apart.
template <typename T, int KIND, int TF, int TT>
struct FlexStage {
    static constexpr int V = FlexType<T>::V, KT = flex_step<T>(TT);
    static constexpr int PER_ROW = (KIND == FLEX_KC ? KT : TF) / V, ROWS = KIND == FLEX_KC ? TF : KT;
    static constexpr int NV = ROWS * PER_ROW / TT, ROW_STEP = TT / PER_ROW;
    static_assert(NV >= 1 && NV * TT == ROWS * PER_ROW, "the team's threads tile the stage");
    static constexpr int PITCH = KIND == FLEX_KC ? KT + V
                                 : TF == 32 ? 32 : TF + 32;
    static constexpr int ELEMS = ROWS * PITCH;
};

template <typename T, int KIND, int TF, int TT>
struct FlexLoader {
    typedef FlexStage<T, KIND, TF, TT> S;
    static constexpr int V = S::V, KT = S::KT;
    // KC: p0, p1 = the tile's first row in the two regions (uniform).  KM: this thread's free position in them.
    int64_t p0, p1, start0, start1;            // (addresses as numbers, see flex_pick); start: of the regions' buffers
    uint32_t off[S::NV];                       // plain tiles: byte offset of vector j from p0
    int64_t ld0, ld1, seg_stride;
    int row0[S::NV];                           // KC: element offset of row j in the head block, from p0;
    int row1[S::NV];                           //     in a segment, from p1
    int after[S::NV];                          //     rows behind row j
    int col, row, skip;
    int left;                                  // KM: elements from the vector's start to the end of its piece
    bool tiny;

    // f0: first free position; ax: the reduction index, fax: the free index
    __device__ __forceinline__ void init(const FlexOperand &op, const FlexAxis &ax, const FlexAxis &fax, int f0, int g, int tid)
    {
        constexpr int64_t E = sizeof(T);
        start0 = (int64_t)(uintptr_t)op.p0; start1 = (int64_t)(uintptr_t)op.p1;
        p0 = start0 + g * op.g0 * E; p1 = start1 + g * op.g1 * E;
        ld0 = op.ld0; ld1 = op.ld1; seg_stride = op.seg_stride; skip = op.skip0 + g * op.skip_g; tiny = op.tiny;
        col = (tid % S::PER_ROW) * V;
        row = tid / S::PER_ROW;
        if (KIND == FLEX_KC) {
            p0 += f0 * ld0 * E;
            p1 += f0 * ld1 * E;
#pragma unroll
            for (int j = 0; j < S::NV; ++j) {
                const int r = min(row + j * S::ROW_STEP, fax.head - 1 - f0);
                row0[j] = r * (int)ld0;
                row1[j] = r * (int)ld1;
                after[j] = fax.head - 1 - f0 - r;
                off[j] = (uint32_t)(row0[j] + col) * (uint32_t)E;
            }
        } else {
            const FlexLoc l = flex_locate(fax, min(f0 + col, fax.total - V), seg_stride, skip);
            left = l.len - l.in_piece;
            const bool folds = fax.seg_pad > 0 && l.region;      // the free index decides: this thread stays in region 1
            p0 = flex_pick(folds, p0, p1) + l.off * E;
            start0 = flex_pick(folds, start0, start1);
            ld0 = flex_pick(folds, ld0, ld1);
            p1 += l.off * E;
#pragma unroll
            for (int j = 0; j < S::NV; ++j) off[j] = (uint32_t)((row + j * S::ROW_STEP) * (int)ld0) * (uint32_t)E;
        }
    }

    // Is the tile that starts at c0 one whose vectors are all whole and inside (uniform)?  KC: it lies in the head block.
    // KM: so do V rows behind it.
    __device__ __forceinline__ bool plain(const FlexAxis &ax, int c0) const { return c0 + KT + (KIND == FLEX_KC ? 0 : V) <= ax.head; }

    struct Col {             // KC: what the vectors of a tile that is not plain share, this thread's reduction position
        int region, n, valid;            // n: elements from there to the end of the piece
        int64_t off;
    };
    struct At {              // vector j of such a tile
        int64_t p;
        int back;            // how many elements ahead of its place it is read, so that the read ends with the piece's last row
        int valid;           // elements that count
    };
    __device__ __forceinline__ Col column(const FlexAxis &ax, int c0) const
    {
        Col k{};
        if (KIND == FLEX_KC) {
            int c = c0 + col;
            asm volatile("" : "+v"(c));                // (opaque: hoisted out of the reduction loop it would hold registers there)
            const bool any = c < ax.total;
            const FlexLoc l = flex_locate(ax, any ? c : 0, seg_stride, skip);
            k.region = l.region; k.off = l.off; k.n = l.len - l.in_piece;
            k.valid = any ? min(V, k.n) : 0;
        }
        return k;
    }
    __device__ __forceinline__ At at(const FlexAxis &ax, const Col &k, int c0, int j) const
    {
        At a;
        int rest;            // elements from the vector's start to the end of the piece's last row (V and more are alike)
        bool tail;
        if (KIND == FLEX_KC) {
            tail = k.region;
            a.valid = k.valid;
            a.p = flex_pick(tail, p0, p1) + (k.off + flex_pick(tail, row0[j], row1[j])) * (int)sizeof(T);
            rest = min(after[j], V) * flex_pick(tail, min((int)ld0, V), min((int)ld1, V)) + k.n;
        } else {
            const int c = c0 + row + j * S::ROW_STEP;
            tail = ax.seg > 0 && c >= ax.head_pad;
            const int last = flex_pick(tail, ax.head, ax.seg) - 1, t = c - (tail ? ax.head_pad : 0), r = min(t, last);
            const int64_t ld = flex_pick(tail, ld0, ld1);
            a.valid = t <= last ? min(V, left) : 0;
            a.p = flex_pick(tail, p0, p1) + r * ld * (int)sizeof(T);
            rest = min(last - r, V) * min((int)ld, V) + left;
        }
        a.back = max(0, V - rest);
        if (tiny) {          // uniform
            // A buffer with fewer than V elements altogether is read from its start, which is 16-byte aligned: such a read
            // stays within the 16 bytes that the buffer begins.
            const int64_t before = (a.p - flex_pick(tail, start0, start1)) / (int)sizeof(T);
            a.back = before < a.back ? (int)before : a.back;
        }
        return a;
    }

    // Are the tile's vectors all whole, wherever they lie (uniform)?  Then nothing has to be shifted or masked.
    __device__ __forceinline__ bool whole(const FlexAxis &ax, int c0) const
    {
        return plain(ax, c0) || (KIND == FLEX_KC && ax.seg == ax.seg_pad && (ax.head == ax.head_pad || c0 >= ax.head_pad) && c0 + KT <= ax.total);
    }

    // The addresses are worked out in branches, the loads stand behind them: loads inside the branches would make the
    // compiler wait for all of them where it could count.
    __device__ __forceinline__ void fetch(const FlexAxis &ax, u32x4 (&regs)[S::NV], int c0) const
    {
        int64_t q[S::NV];
        if (plain(ax, c0)) {
            const int64_t p = p0 + (KIND == FLEX_KC ? c0 : c0 * ld0) * (int)sizeof(T);
#pragma unroll
            for (int j = 0; j < S::NV; ++j) q[j] = p + off[j];
        } else if (whole(ax, c0)) {                    // (a KC operand)
            const FlexLoc l = flex_locate(ax, c0 + col, seg_stride, skip);
            const int64_t p = flex_pick(l.region, p0, p1) + l.off * (int)sizeof(T);
#pragma unroll
            for (int j = 0; j < S::NV; ++j) q[j] = p + (int64_t)flex_pick(l.region, row0[j], row1[j]) * (int)sizeof(T);
        } else {
            const Col k = column(ax, c0);
#pragma unroll
            for (int j = 0; j < S::NV; ++j) {
                const At a = at(ax, k, c0, j);
                q[j] = a.p - a.back * (int)sizeof(T);
                __builtin_amdgcn_sched_barrier(0);     // one vector's arithmetic at a time: it takes many registers
            }
        }
#pragma unroll
        for (int j = 0; j < S::NV; ++j) asm volatile("" : "+v"(q[j]));
#pragma unroll
        for (int j = 0; j < S::NV; ++j) regs[j] = flex_load((const T *)(uintptr_t)q[j]);
    }

    __device__ __forceinline__ void store(const FlexAxis &ax, u32x4 (&regs)[S::NV], T *tile, int c0) const
    {
        if (!whole(ax, c0)) {                          // uniform
            const Col k = column(ax, c0);
#pragma unroll
            for (int j = 0; j < S::NV; ++j) {
                const At a = at(ax, k, c0, j);
                regs[j] = FlexVec<T>::keep(FlexVec<T>::shift(regs[j], a.back), a.valid);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (KIND == FLEX_KC && sizeof(T) == 4) {
            T *dst = tile + row * S::PITCH + (col & ~7) + ((col >> 1) & 2);
#pragma unroll
            for (int j = 0; j < S::NV; ++j) {
                *(u32x2 *)(dst + j * S::ROW_STEP * S::PITCH) = u32x2{regs[j][0], regs[j][2]};
                *(u32x2 *)(dst + j * S::ROW_STEP * S::PITCH + 4) = u32x2{regs[j][1], regs[j][3]};
            }
        } else {
            T *dst = tile + row * S::PITCH + col;
#pragma unroll
            for (int j = 0; j < S::NV; ++j) *(u32x4 *)(dst + j * S::ROW_STEP * S::PITCH) = regs[j];
        }
    }
};

// one reduction step of a wavefront's MI x NI blocks of 32 x 32 (B operand first: a lane then holds row (lane & 31) of a
// block and the columns 8 * (e / 4) + 4 * (lane >> 5) + e % 4)
template <int KIND, int PITCH>
__device__ __forceinline__ bf16x8 flex_operand(const bf16_t *tile, int rbase, int kk, int lane)
{
    if (KIND == FLEX_KC) return *(const bf16x8 *)(tile + (rbase + (lane & 31)) * PITCH + kk * 16 + (lane >> 5) * 8);
    const int krow = kk * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
    const int rcol = rbase + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    const bf16_t *p = tile + krow * PITCH + rcol;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    union { struct { s16x4 a, b; } s; bf16x8 v; } u;
    u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
    u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * PITCH));
    return u.v;
}
// float: the four reduction positions 8 kk + 2 t + (lane >> 5), t = 0..3, one per MFMA.  v_mfma_f32_32x32x2_f32 adds its
// two products one after the other, each with one rounding, so the terms are added in the order of the reduction index.
template <int KIND, int PITCH>
__device__ __forceinline__ f32x4 flex_operand(const float *tile, int rbase, int kk, int lane)
{
    if (KIND == FLEX_KC) return *(const f32x4 *)(tile + (rbase + (lane & 31)) * PITCH + kk * 8 + (lane >> 5) * 4);
    f32x4 v;
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = tile[(kk * 8 + 2 * t + (lane >> 5)) * PITCH + rbase + (lane & 31)];
    return v;
}

template <int MI, int NI> __device__ __forceinline__ void flex_add(f32x16 (&to)[MI][NI], const f32x16 (&part)[MI][NI])
{
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) to[i][j][e] += part[i][j][e];
}

// bf16: a reduction step added to acc, or (FIRST) on its own.
template <int KA, int KB, int PA, int PB, bool FIRST, int MI, int NI>
__device__ __forceinline__ void flex_multiply(f32x16 (&acc)[MI][NI], const bf16_t *ta, const bf16_t *tb, int wm, int wn, int lane)
{
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        bf16x8 av[MI], bv[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) av[i] = flex_operand<KA, PA>(ta, wm + 32 * i, kk, lane);
#pragma unroll
        for (int j = 0; j < NI; ++j) bv[j] = flex_operand<KB, PB>(tb, wn + 32 * j, kk, lane);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv[j], av[i], FIRST && kk == 0 ? zero : acc[i][j], 0, 0, 0);
    }
}
// fp32: adds every 16 terms of a reduction step (of KT) to mid.
template <int KA, int KB, int PA, int PB, int KT, int MI, int NI>
__device__ __forceinline__ void flex_multiply(f32x16 (&mid)[MI][NI], const float *ta, const float *tb, int wm, int wn, int lane)
{
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int part = 0; part < KT / 16; ++part) {
        f32x16 acc[MI][NI];
#pragma unroll
        for (int kk = 2 * part; kk < 2 * part + 2; ++kk) {
            f32x4 av[MI], bv[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) av[i] = flex_operand<KA, PA>(ta, wm + 32 * i, kk, lane);
#pragma unroll
            for (int j = 0; j < NI; ++j) bv[j] = flex_operand<KB, PB>(tb, wn + 32 * j, kk, lane);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[j][t], av[i][t], kk == 2 * part && t == 0 ? zero : acc[i][j], 0, 0, 0);
        }
        flex_add(mid, acc);
    }
}

// V consecutive elements to or from memory at any element boundary, the first `valid` of them
template <int V> struct FlexRow { float x[V]; };
template <typename E, int V> __device__ __forceinline__ FlexRow<V> flex_read(const E *p, int valid)
{
    typedef E Vec __attribute__((ext_vector_type(V), aligned(sizeof(E))));
    FlexRow<V> r;
    if (valid == V) {
        const Vec v = gload<Vec>(p);
#pragma unroll
        for (int u = 0; u < V; ++u) r.x[u] = (float)v[u];
    } else {
#pragma unroll
        for (int u = 0; u < V; ++u) r.x[u] = u < valid ? (float)gload<E>(p + u) : 0.f;
    }
    return r;
}
template <typename E, int V, bool NT = true> __device__ __forceinline__ void flex_write(E *p, const FlexRow<V> &r, int valid)
{
    typedef E Vec __attribute__((ext_vector_type(V), aligned(sizeof(E))));
    if (valid == V) {
        Vec v;
#pragma unroll
        for (int u = 0; u < V; ++u) v[u] = (E)r.x[u];
        if (NT) gstore_nt<Vec>(p, v);
        else gstore<Vec>(p, v);
    } else {
#pragma unroll
        for (int u = 0; u < V; ++u)
            if (u < valid) gstore<E>(p + u, (E)r.x[u]);
    }
}

template <int TM, int TN> struct FlexTileShape {       // a finished tile in LDS
    static constexpr int CPITCH = TN + 4, C_BYTES = TM * CPITCH * 4;
};
template <typename T, int TM, int TN, int TEAMS, bool FINE>
struct FlexShape {
    static constexpr int WM = TM >= 64 ? 2 : 1, WN = TN >= 64 ? 2 : 1;     // wavefronts of a team along each side
    static constexpr int MI = TM / 32 / WM, NI = TN / 32 / WN;             // 32 x 32 blocks per wavefront
    static constexpr int TT = 64 * WM * WN, THREADS = TT * TEAMS;
    static constexpr int STAGES = TT == 64 ? 1 : 2;
    static constexpr int SETS = 2;                     // reduction steps that the loads run ahead
    static constexpr bool LEVELS = sizeof(T) == 4 || FINE;                 // sums in three levels
    static constexpr int MIN_WAVES = TT == 64 || MI * NI > 1 ? 2 : LEVELS ? 3 : 4;      // wavefronts per SIMD that the registers have to allow

    static constexpr int CPITCH = FlexTileShape<TM, TN>::CPITCH, C_BYTES = FlexTileShape<TM, TN>::C_BYTES;
};
constexpr int flex_max(int a, int b) { return a > b ? a : b; }
template <typename T, int TM, int TN, int TEAMS, int KA, int KB>
constexpr int flex_lds_bytes()
{
    typedef FlexShape<T, TM, TN, TEAMS, false> F;
    return flex_max(TEAMS * F::STAGES * (FlexStage<T, KA, TM, F::TT>::ELEMS + FlexStage<T, KB, TN, F::TT>::ELEMS) * (int)sizeof(T),
                    TEAMS * F::C_BYTES + F::THREADS * 4 + 64);
}

// orders a wavefront's own LDS accesses for the compiler (the hardware keeps them in order)
__device__ __forceinline__ void flex_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// What the epilogue reads besides the tile, a vector per pass, requested before the tile is written to LDS (see EpilogueReads in
// gemm_mfma.h).  WHOLE: every vector is whole; else only the whole ones are requested, and the epilogue reads the others for itself.
// In the kernels without the ring, where a thread has one or two passes (us a step): all 4 ranks of 64 in fp32 at batch 32 56.4 -> 54.9,
// ranks of 750 trained at batch 1000 92.1 -> 90.6.
template <typename T, int PASSES> struct FlexAhead {
    static constexpr int V = FlexType<T>::V;
    typedef T VecT __attribute__((ext_vector_type(V), aligned(sizeof(T))));
    typedef float VecF __attribute__((ext_vector_type(V), aligned(4)));
    VecT bias;
    float row;               // the bias (or its master) that the row sums update
    union Pass { VecF f; VecT h; __device__ Pass() {} } pass[PASSES];      // sigma', activation or its argument, target, or (master) weights
};

template <typename T, int TM, int TN, int THREADS, bool WHOLE, bool ROWSUM, typename TOut, int EPI, int PASSES>
__device__ __forceinline__ void flex_request(FlexAhead<T, PASSES> &R, const FlexIn &P, const FlexOut &Q, int g, int tm, int tn, bool rows, int i0 = 0)
{
    typedef typename FlexAhead<T, PASSES>::VecT VecT;
    typedef typename FlexAhead<T, PASSES>::VecF VecF;
    constexpr int V = FlexType<T>::V, PER_ROW = TN / V;
    static_assert(THREADS % PER_ROW == 0, "a thread keeps its columns from pass to pass");
    const Epilogue &ep = Q.ep;
    const SgdInPlace &sgd = Q.sgd;
    // (addresses clamped into the tile's valid part)
    const int n = min(tn * TN + ((int)threadIdx.x % PER_ROW) * V, P.n.total - V);
    const int m0 = tm * TM + (int)threadIdx.x / PER_ROW;
    auto row = [&](int i) { return (int64_t)min(m0 + (i0 + i) * (THREADS / PER_ROW), P.M - 1); };
    const FlexLoc l = flex_locate(P.n, n, Q.o_seg_stride, NO_SKIP);
    const bool whole = WHOLE || l.len - l.in_piece >= V;
    if constexpr (ROWSUM) {
        const int m = tm * TM + (int)threadIdx.x;
        if (rows && i0 == 0 && sgd.bias_w && (int)threadIdx.x < TM && m < P.M)
            R.row = gload<float>((sizeof(T) == 2 ? sgd.bias_master : (float *)sgd.bias_w) + (int64_t)g * P.M + m);
    }
    if (!whole || (TM * PER_ROW < THREADS && (int)threadIdx.x >= TM * PER_ROW)) return;
    if constexpr (EPI == EPI_BIAS_ACT) {
        if (ep.mode == EPI_BIAS_ACT) {                 // uniform, like every branch below
            R.bias = gload<VecT>((const T *)ep.bias + g * ep.bias_g + n);
            if (ep.mse_target) {
#pragma unroll
                for (int i = 0; i < PASSES; ++i) R.pass[i].h = gload<VecT>((const T *)ep.mse_target + g * ep.aux_g + row(i) * ep.aux_ld + n);
            }
        }
    } else if constexpr (EPI == EPI_DACT) {
        if (ep.mode == EPI_DACT && ep.aux) {
            if (ep.aux_deriv || ep.aux_f32) {
#pragma unroll
                for (int i = 0; i < PASSES; ++i) R.pass[i].f = gload<VecF>((const float *)ep.aux + g * ep.aux_g + row(i) * ep.aux_ld + n);
            } else {
#pragma unroll
                for (int i = 0; i < PASSES; ++i) R.pass[i].h = gload<VecT>((const T *)ep.aux + g * ep.aux_g + row(i) * ep.aux_ld + n);
            }
        }
    } else {
        if (sgd.w0) {
            float *const m0_ = sizeof(T) == 2 ? sgd.master0 : (float *)sgd.w0, *const m1_ = sizeof(T) == 2 ? sgd.master1 : (float *)sgd.w1;
            const float *base = l.region ? m1_ + g * Q.o_g1 + l.off : m0_ + g * Q.o_g0 + l.off;
            const int64_t ld = flex_pick<int64_t>(l.region, Q.o_ld0, Q.o_ld1);
#pragma unroll
            for (int i = 0; i < PASSES; ++i) R.pass[i].f = gload<VecF>(base + row(i) * ld);
        }
    }
}

// The requested vectors are here, for every thread.  Threads without an element of the output would else leave with loads under way, and
// where one kernel holds several products' code the compiler waited for these registers inside the next product's reduction loop, which
// waits for the ring's loads as well (one rank's 1720 + 480 wide layer backward, 1160 workgroups: 33 us, 37 with it).
template <typename T, int PASSES> __device__ __forceinline__ void flex_arrived(FlexAhead<T, PASSES> &R)
{
#pragma unroll
    for (int i = 0; i < PASSES; ++i)
#pragma unroll
        for (int u = 0; u < FlexAhead<T, PASSES>::V; ++u) asm volatile("" : "+v"(R.pass[i].f[u]));
    asm volatile("" : "+v"(R.row));
}

// What a workgroup of THREADS threads does with its finished tile: TEAMS partial sums of it at ctile (C_BYTES apart), and with rows the
// parts of A's row sums in extra (THREADS floats).  AHEAD: the passes whose reads are in R (WHOLE as there), the first ones of the tile; the next ones'
// are requested as R's are used.  0: none, it reads for itself.
template <typename T, int TM, int TN, int TEAMS, int THREADS, bool FINE, bool WHOLE, bool ROWSUM, typename TOut, int EPI, int AHEAD>
__device__ __forceinline__ void flex_epilogue(const FlexIn &P, const FlexOut &Q, int g, int tm, int tn, const float *ctile, float *extra, bool rows,
                                              FlexAhead<T, (AHEAD > 0 ? AHEAD : 1)> &R)
{
    typedef FlexTileShape<TM, TN> F;
    constexpr int V = FlexType<T>::V;
    const int m0 = tm * TM, n0 = tn * TN;
    const Epilogue &ep = Q.ep;
    const SgdInPlace &sgd = Q.sgd;
    if constexpr (ROWSUM) {
        if (rows && (int)threadIdx.x < TM && m0 + (int)threadIdx.x < P.M) {
            float t = 0.f;
            // bf16, eight parts a row and more: four at a time.  Not on the ring, whose epilogue has less to wait for (us a pass, in turn : four at a time:
            // 3 layers of 750 + 70 with GELU trained at batch 1000, without the ring, 89.9 : 89.4; a layer's calls of 512 + 1008 at 2048, on it, 35.7 : 35.9).
            if constexpr (THREADS >= 8 * TM && sizeof(T) == 2 && !WHOLE) {
#pragma unroll
                for (int r = threadIdx.x; r < THREADS; r += 4 * TM) t += (extra[r] + extra[r + TM]) + (extra[r + 2 * TM] + extra[r + 3 * TM]);
            } else {
#pragma unroll 4
                for (int r = threadIdx.x; r < THREADS; r += TM) t += extra[r];      // parts of a team, then the next team
            }
            const int64_t at = (int64_t)g * P.M + m0 + threadIdx.x;
            gstore<float>(Q.rowsum + at, t);
            if (sgd.bias_w) {
                if constexpr (sizeof(T) == 2) {
                    const float nb = (AHEAD > 0 ? R.row : gload<float>(sgd.bias_master + at)) - sgd.lr * t;
                    gstore<float>(sgd.bias_master + at, nb);
                    gstore<bf16_t>((bf16_t *)sgd.bias_w + at, (bf16_t)nb);
                } else {
                    float *w = (float *)sgd.bias_w + at;
                    gstore<float>(w, (AHEAD > 0 ? R.row : gload<float>(w)) - sgd.lr * t);
                }
            }
        }
    }
    constexpr int PER_ROW = TN / V;
    float sq_sum = 0.f;
    // a vector that was read ahead, as floats; the others are read now
    auto ready = [](auto vec) {
        FlexRow<V> r;
#pragma unroll
        for (int u = 0; u < V; ++u) r.x[u] = (float)vec[u];
        return r;
    };
    constexpr int GROUP = AHEAD > 0 ? AHEAD : 1, PASSES = (TM * PER_ROW + THREADS - 1) / THREADS;
    static_assert(PASSES % GROUP == 0, "whole groups");
#pragma unroll 1
    for (int i0 = 0; i0 < PASSES; i0 += GROUP) {
    const FlexAhead<T, GROUP> now = R;
    if constexpr (AHEAD > 0 && PASSES > GROUP) {
        if (i0 + GROUP < PASSES) flex_request<T, TM, TN, THREADS, WHOLE, ROWSUM, TOut, EPI>(R, P, Q, g, tm, tn, rows, i0 + GROUP);
    }
#pragma unroll
    for (int h = 0; h < GROUP; ++h) {
        const int v = (int)threadIdx.x + (i0 + h) * THREADS;
        if (TM * PER_ROW % THREADS && v >= TM * PER_ROW) break;
        const int row = v / PER_ROW, col = (v % PER_ROW) * V, m = m0 + row, n = n0 + col;
        if (m >= P.M || n >= P.n.total) continue;
        const FlexLoc l = flex_locate(P.n, n, Q.o_seg_stride, NO_SKIP);
        const int valid = WHOLE ? V : min(V, l.len - l.in_piece);
        const bool have = AHEAD > 0 && valid == V;     // (WHOLE: known to the compiler)
        const typename FlexAhead<T, GROUP>::Pass &read = now.pass[h];
        FlexRow<V> x;
#pragma unroll
        for (int h = 0; h < V / 4; ++h) {
            f32x4 t = *(const f32x4 *)(ctile + row * F::CPITCH + col + 4 * h);
#pragma unroll
            for (int q = 1; q < TEAMS; ++q) t += *(const f32x4 *)(ctile + q * (F::C_BYTES / 4) + row * F::CPITCH + col + 4 * h);
#pragma unroll
            for (int u = 0; u < 4; ++u) x.x[4 * h + u] = t[u];
        }
        const int64_t aux_at = g * ep.aux_g + (int64_t)m * ep.aux_ld + n;      // (such outputs are plain: n is the column)
        FlexRow<V> deriv;
        if (EPI == EPI_BIAS_ACT && ep.mode == EPI_BIAS_ACT) {
            FlexRow<V> bias;
            if (have) bias = ready(now.bias);
            else bias = flex_read<T, V>((const T *)ep.bias + g * ep.bias_g + n, valid);
            FlexRow<V> pre;
#pragma unroll
            for (int u = 0; u < V; ++u) { x.x[u] += bias.x[u]; pre.x[u] = x.x[u]; }
            if constexpr (sizeof(T) == 2) {
                if (ep.act == ACT_GELU) {              // uniform
#pragma unroll
                    for (int u = 0; u < V; ++u) {
                        if constexpr (FINE) { x.x[u] = act_apply(ACT_GELU, pre.x[u]); deriv.x[u] = act_deriv(ACT_GELU, pre.x[u]); }
                        else gelu_both(pre.x[u], x.x[u], deriv.x[u]);
                    }
                } else {
                    piecewise_both(ep.act, x.x, deriv.x);
                }
            } else {
#pragma unroll
                for (int u = 0; u < V; ++u) { x.x[u] = act_apply(ep.act, pre.x[u]); deriv.x[u] = 1.f; }
            }
            if (sizeof(T) == 4 && (ep.aux_deriv || ep.mse_target)) {       // uniform
#pragma unroll
                for (int u = 0; u < V; ++u) deriv.x[u] = act_deriv(ep.act, pre.x[u]);
            }
            if (ep.aux) {                              // uniform
                if (ep.aux_deriv) flex_write<float, V>((float *)ep.aux + aux_at, deriv, valid);
                else if (ep.aux_f32) flex_write<float, V>((float *)ep.aux + aux_at, pre, valid);
                else flex_write<T, V>((T *)ep.aux + aux_at, pre, valid);
            }
        } else if (EPI == EPI_DACT && ep.mode == EPI_DACT && ep.aux) {
            if (ep.aux_deriv) {
                FlexRow<V> a;
                if (have) a = ready(read.f);
                else a = flex_read<float, V>((const float *)ep.aux + aux_at, valid);
#pragma unroll
                for (int u = 0; u < V; ++u) x.x[u] *= a.x[u];
            } else {
                FlexRow<V> a;
                if (have && ep.aux_f32) a = ready(read.f);
                else if (have) a = ready(read.h);
                else a = ep.aux_f32 ? flex_read<float, V>((const float *)ep.aux + aux_at, valid) : flex_read<T, V>((const T *)ep.aux + aux_at, valid);
#pragma unroll
                for (int u = 0; u < V; ++u) x.x[u] *= sizeof(T) == 2 ? (a.x[u] > 0.f ? 1.f : 0.f) : act_deriv(ep.act, a.x[u]);   // (bf16: ReLU output)
            }
        }
        const int64_t o_at = l.region ? g * Q.o_g1 + (int64_t)m * Q.o_ld1 + l.off : g * Q.o_g0 + (int64_t)m * Q.o_ld0 + l.off;
        if constexpr (EPI == EPI_STORE && sizeof(TOut) == 4) {
            if (sgd.w0) {                              // uniform
                void *const w0 = sgd.w0, *const w1 = sgd.w1;
                void *const w = l.region ? w1 : w0;
                if constexpr (sizeof(T) == 2) {
                    float *const m0 = sgd.master0, *const m1 = sgd.master1;
                    float *const master = (l.region ? m1 : m0) + o_at;
                    FlexRow<V> mv;
                    if (have) mv = ready(read.f);
                    else mv = flex_read<float, V>(master, valid);
#pragma unroll
                    for (int u = 0; u < V; ++u) mv.x[u] -= sgd.lr * x.x[u];
                    flex_write<float, V>(master, mv, valid);
                    flex_write<bf16_t, V, false>((bf16_t *)w + o_at, mv, valid);
                } else {
                    FlexRow<V> wv;
                    if (have) wv = ready(read.f);
                    else wv = flex_read<float, V>((const float *)w + o_at, valid);
#pragma unroll
                    for (int u = 0; u < V; ++u) wv.x[u] -= sgd.lr * x.x[u];
                    flex_write<float, V, false>((float *)w + o_at, wv, valid);
                }
                if (!sgd.keep_grad) continue;
            }
        }
        void *const o0 = Q.o0, *const o1 = Q.o1;
        flex_write<TOut, V>((TOut *)(l.region ? o1 : o0) + o_at, x, valid);
        if (EPI == EPI_BIAS_ACT && ep.mode == EPI_BIAS_ACT && ep.mse_target) {         // uniform
            // the MSE output error of Eq. (deltaL) from the output as stored, rounded once
            FlexRow<V> t;
            if (have) t = ready(read.h);
            else t = flex_read<T, V>((const T *)ep.mse_target + aux_at, valid);
            FlexRow<V> dl;
#pragma unroll
            for (int u = 0; u < V; ++u) {
                const float diff = (float)(T)x.x[u] - t.x[u];
                if (u < valid) sq_sum += diff * diff;
                dl.x[u] = diff * ep.mse_inv_b;
                if (ep.act != ACT_IDENTITY) dl.x[u] *= deriv.x[u];
            }
            flex_write<T, V, false>((T *)ep.mse_delta + aux_at, dl, valid);
        }
    }
    }
    if (EPI == EPI_BIAS_ACT && ep.mode == EPI_BIAS_ACT && ep.mse_target) {             // uniform
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sq_sum += __shfl_down(sq_sum, off);
        if ((threadIdx.x & 63) == 0) extra[threadIdx.x >> 6] = sq_sum;
        __syncthreads();
        if (threadIdx.x == 0) {
            float total = 0.f;
#pragma unroll
            for (int w = 0; w < THREADS / 64; ++w) total += extra[w];
            ep.mse_partial[(g * P.tiles_m + tm) * P.tiles_n + tn] = total;
        }
    }
}

// One workgroup's work on the product P: workgroup number wg of P.total_wg.
template <typename T, int TM, int TN, int TEAMS, bool FINE, int KA, int KB, typename TOut, int EPI>
__device__ __forceinline__ void flex_workgroup(const FlexIn &P, int product, int wg, unsigned char *lds)
{
    typedef FlexShape<T, TM, TN, TEAMS, FINE> F;
    typedef FlexLoader<T, KA, TM, F::TT> LA;
    typedef FlexLoader<T, KB, TN, F::TT> LB;
    constexpr int KT = flex_step<T>(F::TT), V = FlexType<T>::V, MI = F::MI, NI = F::NI;
    constexpr bool ROWSUM = KA == FLEX_KM && KB == FLEX_KM;

    const FlexTileAt at = flex_tile_at<sizeof(T) == 4 && TM == 64>(P, wg);
    const int g = at.g, tm = at.tm, tn = at.tn;
    const int m0 = tm * TM, n0 = tn * TN;

    const int team = TEAMS > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / F::TT) : 0;
    const int tid = (int)threadIdx.x - team * F::TT, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave / F::WN) * MI * 32, wn = (wave % F::WN) * NI * 32;

    const FlexAxis &ka = P.k;
    FlexAxis ma{};                                     // the row index: never cut
    ma.head = P.M; ma.head_pad = (P.M + V - 1) / V * V; ma.total = ma.head_pad;
    LA la;
    LB lb;
    la.init(P.a, ka, ma, m0, g, tid);
    lb.init(P.b, ka, P.n, n0, g, tid);

    f32x16 acc[MI][NI], mid[MI][NI];                   // the sums; with levels: the third level's, and the second's
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) { acc[i][j][e] = 0.f; mid[i][j][e] = 0.f; }
    const bool rows = ROWSUM && P.rowsum && n0 == 0;   // uniform
    float row_acc = 0.f, row_mid = 0.f;
    int in_mid = 0;                                    // sixteenths of a second-level sum (256 terms) in mid

    T *stage0 = (T *)lds + team * F::STAGES * (LA::S::ELEMS + LB::S::ELEMS);
    const int steps = (ka.total + KT - 1) / KT, loops = (steps + TEAMS - 1) / TEAMS;
    auto c_of = [=](int i) { return (i * TEAMS + team) * KT; };
    constexpr int SETS = F::SETS;
    u32x4 ra[SETS][LA::S::NV], rb[SETS][LB::S::NV];
#pragma unroll
    for (int d = 0; d < SETS; ++d) { la.fetch(ka, ra[d], c_of(d)); lb.fetch(ka, rb[d], c_of(d)); }
    // step i: LDS stage d = i % 2, register set d % SETS
    auto step = [&](int d, int i, bool last) {
        T *ta = stage0 + (F::STAGES == 2 ? d : 0) * (LA::S::ELEMS + LB::S::ELEMS), *tb = ta + LA::S::ELEMS;
        const int c0 = c_of(i);
        u32x4 (&ma_)[LA::S::NV] = ra[d % SETS];
        u32x4 (&mb_)[LB::S::NV] = rb[d % SETS];
        la.store(ka, ma_, ta, c0);
        lb.store(ka, mb_, tb, c0);
        if (!last) {
            la.fetch(ka, ma_, c_of(i + SETS));
            lb.fetch(ka, mb_, c_of(i + SETS));
        }
        if constexpr (F::TT > 64) __syncthreads();
        else flex_wave_sync();
        if constexpr (sizeof(T) == 4) {
            flex_multiply<KA, KB, LA::S::PITCH, LB::S::PITCH, KT>(mid, ta, tb, wm, wn, lane);
        } else if constexpr (F::LEVELS) {
            f32x16 part[MI][NI];
            flex_multiply<KA, KB, LA::S::PITCH, LB::S::PITCH, true>(part, ta, tb, wm, wn, lane);
            flex_add(mid, part);
        } else {
            flex_multiply<KA, KB, LA::S::PITCH, LB::S::PITCH, false>(acc, ta, tb, wm, wn, lane);
        }
        if constexpr (ROWSUM) {
            if (rows) {
                constexpr int PARTS = F::TT / TM;
                const int part = tid / TM;
                float t = 0.f;
#pragma unroll 8
                for (int r = 0; r < KT / PARTS; ++r) t += (float)ta[(part + r * PARTS) * LA::S::PITCH + tid % TM];
                row_mid += t;
            }
        }
        if constexpr (F::LEVELS) {
            in_mid += sizeof(T) == 4 ? KT / 16 : 4;
            if (in_mid == 16) {                        // uniform
                flex_add(acc, mid);
#pragma unroll
                for (int a = 0; a < MI; ++a)
#pragma unroll
                    for (int b = 0; b < NI; ++b)
#pragma unroll
                        for (int e = 0; e < 16; ++e) mid[a][b][e] = 0.f;
                in_mid = 0;
                if (sizeof(T) == 4) { row_acc += row_mid; row_mid = 0.f; }
            }
            if (sizeof(T) == 2 && (i & 63) == 63) { row_acc += row_mid; row_mid = 0.f; }      // (a step's 16 terms, 64 of those, the rest)
        }
        if constexpr (F::TT == 64) flex_wave_sync();
    };
    // (two whole steps per pass, no way out in between: the compiler counts the loads in flight)
    int i = 0;
    for (; i + 1 < loops; i += 2) {
        step(0, i, false);
        step(1, i + 1, false);
    }
    if (i < loops) step(0, i, true);
    row_acc += row_mid;
    if constexpr (F::LEVELS) flex_add(acc, mid);
    FlexOut Q;
    const size_t q_at = offsetof(FlexBatch, p) + (size_t)product * sizeof(FlexParams) + offsetof(FlexParams, out);
    // Reads ahead of the epilogue, its passes unrolled.  Not the FINE forward epilogue of a 64 x 64 tile: erff and expf, inlined for every pass of
    // a loop that runs once, are fetched cold (all 8 ranks of 405 at batch 615 with GELU, 560 workgroups: 24.6 us a launch, 23.4 without; 16 ranks
    // of 133 trained at batch 534 253.1 : 247.2 us a step).  Nor two passes of the input-gradient layout, whose launches carry the error
    // compression: it stores cut vectors element by element and reads nothing (gradients of 32 ranks of 256 + 22 at batch 663 527.8 : 512.8,
    // 64 ranks of 234 + 8 trained at 1532 1775 : 1766; 3 layers of 750 + 10 trained at 1000 lose, 90.1 : 91.2).
    constexpr int PASSES = (TM * TN / V + F::THREADS - 1) / F::THREADS;
    constexpr bool DEARER = (FINE && EPI == EPI_BIAS_ACT && TM == 64) || (PASSES == 2 && EPI == EPI_DACT);
    constexpr int AHEAD = PASSES <= 2 && !DEARER ? PASSES : 0;
    FlexAhead<T, (AHEAD > 0 ? AHEAD : 1)> ahead;
    if constexpr (AHEAD > 0) Q = args_at<FlexOut>(q_at);
    if constexpr (AHEAD > 0) flex_request<T, TM, TN, F::THREADS, false, ROWSUM, TOut, EPI>(ahead, P, Q, g, tm, tn, rows);
    __syncthreads();

    // the finished tile goes through LDS, so that every global access of the epilogue is a run of whole rows
    float *ctile = (float *)lds;
    float *extra = (float *)(lds + TEAMS * F::C_BYTES);   // THREADS floats
    {
        float *mine = ctile + team * (F::C_BYTES / 4);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                    *(f32x4 *)(mine + (wm + 32 * i + (lane & 31)) * F::CPITCH + wn + 32 * j + 8 * q + 4 * (lane >> 5)) = v;
                }
    }
    if (rows) extra[threadIdx.x] = row_acc;
    __syncthreads();
    if constexpr (AHEAD > 0) flex_arrived(ahead);
    else Q = args_at<FlexOut>(q_at);
    flex_epilogue<T, TM, TN, TEAMS, F::THREADS, FINE, false, ROWSUM, TOut, EPI, AHEAD>(P, Q, g, tm, tn, ctile, extra, rows, ahead);
}

// ---- fp32 in whole vectors ------------------------------------------------------------------------------------------------
// Where 4 divides the widths and phantom widths: the sums of flex_workgroup, term by term in the same order, so the same bits.
// What bounds it: v_mfma_f32_32x32x2_f32 and the vector ALU do not run beside each other, whichever wavefronts they come from (8 ranks of
// 512 + 32 at batch 1024, update: 94000 clocks of matrix instructions a SIMD; with 145, 100 and 64 other vector instructions a wavefront and step,
// whose own four clocks each make 53000, 37000 and 23000, the compute units were busy for 160000, 150000 and 140000).  So a step keeps little more
// than the 32 additions of its sums: loads take a scalar base and offsets that stay, LDS addresses stay too.
// Both operands lie in LDS as rows of 32 reduction indices per free index, so that an operand read is 16 bytes for either kind, unpadded: of each
// eight reduction positions first the even ones (one 16-byte unit), then the odd (see flex_operand); unit u of row r sits at u ^ flex_f32_swizzle(r),
// where 16 rows' reads cover all 64 banks.  A thread has two vectors that differ by one free index (FLEX_KC) or by two
// reduction indices (FLEX_KM), so that what it writes are pairs of words.
// 32 KB of stages and 128 registers: four workgroups of 64 x 64 to a compute unit.
// Trained (us, flex_workgroup : so): 4 layers of 8 ranks of 512 + 32 at batch 1024 952 : 842, 2 of 8 of 512 + 64 at 300 296 : 264, 2 of 16 of 256 + 32 at 400
// 261 : 237, 3 of 4 of 256 + 8 at 1024 224 : 218.
constexpr int F32_KT = 32, F32_ROW = F32_KT * 4, F32_TILE = 64 * F32_ROW, F32_STAGE = 2 * F32_TILE;       // bytes
constexpr int F32_LDS_BYTES = flex_max(2 * F32_STAGE, FlexTileShape<64, 64>::C_BYTES + 256 * 4 + 64);
__device__ __forceinline__ int flex_f32_swizzle(int row) { return ((row >> 1) & 7) ^ ((row >> 4) & 1); }

// CUT: FLEX_KM, the reduction index may be cut (FLEX_KC: it may).
template <int KIND, bool CUT>
struct FlexF32Loader {
    const char *base0, *base1;                 // uniform
    uint32_t off0[2], off1[2];                 // bytes, of the thread's vectors in region 0 and 1 at reduction start 0 (FLEX_KM: of the first)
    uint32_t free_off;                         // FLEX_KM: bytes, of the thread's free position
    bool own1;                                 // FLEX_KM: the tile straddles the cut, and the thread's free position lies in region 1
    uint32_t ld0, ld1;                         // bytes
    int c;                                     // reduction index of the first vector inside a step (FLEX_KM: the second's is two higher)
    int seg, seg_stride, skip, split, lim, plain_lim;      // split: start of region 1 (or none); plain_lim: end of the steps in region 0
    uint32_t magic;
    int col_seg, col_in_seg;                   // FLEX_KC, a step holds several segments: the thread's
    bool regular;                              // FLEX_KC: steps do not straddle the cut, and segments hold steps or steps segments
    uint32_t even, odd;                        // LDS bytes of what it writes

    __device__ __forceinline__ void init(const FlexOperand &op, const FlexAxis &ax, const FlexAxis &fax, int f0, int g, int tid)
    {
        base0 = (const char *)op.p0 + g * op.g0 * 4;
        base1 = (const char *)op.p1 + g * op.g1 * 4;
        seg = ax.seg; seg_stride = (int)op.seg_stride; skip = op.skip0 + g * op.skip_g; magic = ax.magic;
        split = ax.seg > 0 ? ax.head : 0x7fffffff;
        lim = ax.seg > 0 ? ax.total : ax.head;
        plain_lim = min(split, lim);
        ld0 = (uint32_t)op.ld0 * 4u; ld1 = (uint32_t)op.ld1 * 4u;
        int row, unit, word;
        if (KIND == FLEX_KC) {
            const int col = c = (tid & 7) * 4;
            row = (tid >> 3) * 2; unit = col >> 3 << 1; word = (col & 4) >> 1;
            regular = seg <= 0 || (split % F32_KT == 0 && (F32_KT % seg == 0 || seg % F32_KT == 0));
            col_seg = 0; col_in_seg = col;
            if (regular && seg > 0 && seg < F32_KT) {
                col_seg = col / seg;
                col_in_seg = col - col_seg * seg;
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t r = (uint32_t)min(f0 + row + j, fax.head - 1);
                off0[j] = r * ld0 + (uint32_t)col * 4u;
                off1[j] = r * ld1;
            }
        } else {
            // reduction indices 8 (pair / 4) + 4 (pair / 2 % 2) + pair % 2 and two further; half a wavefront writes for 8 rows of 128 bytes, 4 pairs each
            const int pair = (tid >> 6) * 4 + (tid >> 3 & 3);
            row = ((tid & 7) + (tid >> 5 & 1) * 8) * 4; unit = (pair >> 2) * 2 + (pair & 1); word = pair & 2;
            const FlexLoc l = flex_locate(fax, min(f0 + row, fax.total - 4), seg_stride, skip);
            const bool straddles = fax.seg > 0 && f0 < fax.head && f0 + 64 > fax.head, tail = fax.seg > 0 && f0 >= fax.head;      // uniform
            if (tail) { base0 = base1; ld0 = ld1; }
            if (straddles) plain_lim = 0;
            own1 = straddles && l.region;
            free_off = (uint32_t)l.off * 4u;
            c = (pair >> 2) * 8 + (pair & 2) * 2 + (pair & 1);
            off0[0] = (uint32_t)c * ld0 + free_off;
            off1[0] = (uint32_t)c * ld1 + free_off;
        }
        even = (uint32_t)(row * F32_ROW + ((unit ^ flex_f32_swizzle(row)) << 4) + word * 4);
        odd = even ^ 16u;
    }

    // (The comments in assembly keep the branches' loads apart: the compiler would join them behind the branches, where their addresses are 64-bit
    // vector values.)
    __device__ __forceinline__ void fetch(u32x4 (&regs)[2], int c0 /* uniform */) const
    {
        if (c0 + F32_KT <= plain_lim) {                // uniform, like every branch here
            const char *base = base0 + (KIND == FLEX_KC ? (uint64_t)((uint32_t)c0 * 4u) : (uint64_t)(uint32_t)c0 * ld0);
#pragma unroll
            for (int j = 0; j < 2; ++j) regs[j] = KIND == FLEX_KC ? gload<u32x4>(base + off0[j]) : gload<u32x4>(base + (uint64_t)(2 * j) * ld0 + off0[0]);
            asm volatile("; region 0");
        } else if (KIND == FLEX_KC && regular && c0 + F32_KT <= lim) {
            const uint32_t t0 = (uint32_t)(c0 - split);
            uint32_t i0 = __umulhi(t0, magic);
            i0 -= i0 * (uint32_t)seg > t0 ? 1u : 0u;
            const int rem = (int)(t0 - i0 * (uint32_t)seg);
            const char *base = base1;
            uint32_t add = (uint32_t)c * 4u;
            if (seg >= F32_KT) {
                const int slot = (int)i0 + ((int)i0 >= skip ? 1 : 0);
                base += ((int64_t)slot * seg_stride + rem) * 4;
            } else {
                const int i = (int)i0 + col_seg, slot = i + (i >= skip ? 1 : 0);
                add = (uint32_t)(slot * seg_stride + col_in_seg) * 4u;
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) regs[j] = gload<u32x4>(base + (off1[j] + add));
            asm volatile("; segments");
        } else if (KIND == FLEX_KC) {
            const int at = min(c0 + c, lim - 4);
            const bool tail = at >= split;
            const uint32_t t = tail ? (uint32_t)(at - split) : 0u;
            uint32_t i = __umulhi(t, magic);
            i -= i * (uint32_t)seg > t ? 1u : 0u;
            const int slot = (int)i + ((int)i >= skip ? 1 : 0);
            const int64_t from = tail ? ((int64_t)slot * seg_stride + (int)(t - i * (uint32_t)seg)) * 4 : (int64_t)(at - c) * 4;
            const int64_t base = (int64_t)(uintptr_t)(tail ? base1 : base0) + from;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t o0 = off0[j], o1 = off1[j];
                regs[j] = gload<u32x4>((const char *)(uintptr_t)(base + (tail ? o1 : o0)));
            }
            asm volatile("; any");
        } else if (CUT && c0 >= split && c0 + F32_KT <= lim) {
            const char *base = base1 + (uint64_t)(uint32_t)(c0 - split) * ld1;
#pragma unroll
            for (int j = 0; j < 2; ++j) regs[j] = gload<u32x4>(base + (uint64_t)(2 * j) * ld1 + off1[0]);
            asm volatile("; region 1");
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int at = min(c0 + c + 2 * j, lim - 1);
                const bool tail = CUT && at >= split;
                const char *base = tail || own1 ? base1 : base0;
                regs[j] = gload<u32x4>(base + ((int64_t)(tail ? at - split : at) * (tail || own1 ? ld1 : ld0) + free_off));
            }
            asm volatile("; any");
        }
    }

    // zeros in the place of what lies behind the end
    __device__ __forceinline__ void settle(u32x4 (&regs)[2], int c0) const
    {
        if (c0 + F32_KT > lim) {                       // uniform
#pragma unroll
            for (int j = 0; j < 2; ++j) regs[j] = c0 + c + (KIND == FLEX_KC ? 0 : 2 * j) < lim ? regs[j] : u32x4{0u, 0u, 0u, 0u};
        }
    }

    // (inline assembly: from the stores the compiler makes 8-byte ones, and moves words together for them.  It does not count these on
    // their way: flex_f32_barrier.)
    __device__ __forceinline__ void put(const u32x4 (&regs)[2], uint32_t tile) const
    {
        const uint32_t e = tile + even, o = tile + odd;
#define PH_PAIR(at, x, y, row) asm volatile("ds_write2_b32 %0, %1, %2 offset0:%3 offset1:%4" :: "v"(at), "v"(x), "v"(y), "n"((row) * (F32_ROW / 4)), "n"((row) * (F32_ROW / 4) + 1) : "memory")
        if (KIND == FLEX_KC) {                         // row's words 0 2 | 1 3
            PH_PAIR(e, regs[0][0], regs[0][2], 0);
            PH_PAIR(o, regs[0][1], regs[0][3], 0);
            PH_PAIR(e, regs[1][0], regs[1][2], 1);
            PH_PAIR(o, regs[1][1], regs[1][3], 1);
        } else {                                       // (rows 2 and 3 of four have the swizzle's next value)
            PH_PAIR(e, regs[0][0], regs[1][0], 0);
            PH_PAIR(e, regs[0][1], regs[1][1], 1);
            PH_PAIR(o, regs[0][2], regs[1][2], 2);
            PH_PAIR(o, regs[0][3], regs[1][3], 3);
        }
#undef PH_PAIR
    }
};
__device__ __forceinline__ void flex_f32_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// SETS: steps that the loads run ahead.  2, and a step's operand reads ahead of its matrix instructions: for launches whose few workgroups wait for
// them (the registers of two workgroups to a compute unit).
template <int SETS, int KA, int KB, int EPI>
__device__ __forceinline__ void flex_f32_workgroup(const FlexIn &P, int product, int wg, unsigned char *lds)
{
    constexpr int TILE = 64, THREADS = 256, KT = F32_KT;
    constexpr bool ROWSUM = KA == FLEX_KM && KB == FLEX_KM;
    typedef FlexTileShape<TILE, TILE> C;

    const FlexTileAt at = flex_tile_at<true>(P, wg);
    const int g = at.g, tm = at.tm, tn = at.tn;
    const int m0 = tm * TILE, n0 = tn * TILE;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    FlexAxis ma{};                                     // the row index: never cut
    ma.head = P.M; ma.head_pad = (P.M + 3) / 4 * 4; ma.total = ma.head_pad;
    FlexF32Loader<KA, false> la;
    FlexF32Loader<KB, !ROWSUM> lb;
    la.init(P.a, P.k, ma, m0, g, tid);
    lb.init(P.b, P.k, P.n, n0, g, tid);

    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc = zero;                                 // the third level's sums
    const bool rows = ROWSUM && P.rowsum && n0 == 0;   // uniform
    float row_acc = 0.f, row_mid = 0.f;                // of column tid % 64 of A
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LdsBytes)lds;
    const int steps = (la.lim + KT - 1) / KT;
    // the operands of the reduction positions 0 .. 7; 8 kk further at the XOR of kk << 5
    auto place = [&](int rbase) {
        const int row = rbase + (lane & 31);
        return (uint32_t)(row * F32_ROW + (((lane >> 5) ^ flex_f32_swizzle(row)) << 4));
    };
    uint32_t at_a[KT / 8], at_b[KT / 8];
#pragma unroll
    for (int kk = 0; kk < KT / 8; ++kk) { at_a[kk] = lds0 + (place(wm) ^ (kk << 5)); at_b[kk] = lds0 + (place(wn) ^ (kk << 5)); }
    u32x4 ra[SETS][2], rb[SETS][2];
#pragma unroll
    for (int d = 0; d < SETS; ++d)
        if (d < steps) {                               // uniform
            la.fetch(ra[d], d * KT);
            lb.fetch(rb[d], d * KT);
        }
    auto step = [&](auto stage, int i, f32x16 &mid) {
        constexpr int AT = decltype(stage)::value * F32_STAGE, SET = decltype(stage)::value % SETS;
        la.settle(ra[SET], i * KT);
        lb.settle(rb[SET], i * KT);
        la.put(ra[SET], lds0 + AT);
        lb.put(rb[SET], lds0 + AT + F32_TILE);
        if (i + SETS < steps) {                        // uniform
            la.fetch(ra[SET], (i + SETS) * KT);
            lb.fetch(rb[SET], (i + SETS) * KT);
        }
        flex_f32_barrier();                            // (the stage's readers of two steps ago have passed the barrier between)
        f32x4 av[KT / 8], bv[KT / 8];
        auto read = [&](int kk) { av[kk] = *lds_at<const f32x4>(at_a[kk] + AT); bv[kk] = *lds_at<const f32x4>(at_b[kk] + AT + F32_TILE); };
        if constexpr (SETS == 2) {
#pragma unroll
            for (int kk = 0; kk < KT / 8; ++kk) read(kk);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int part = 0; part < KT / 16; ++part) {
            f32x16 sum;
#pragma unroll
            for (int kk = 2 * part; kk < 2 * part + 2; ++kk) {
                if constexpr (SETS == 1) read(kk);
#pragma unroll
                for (int t = 0; t < 4; ++t) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[kk][t], av[kk][t], kk == 2 * part && t == 0 ? zero : sum, 0, 0, 0);
            }
            mid += sum;
        }
        if constexpr (ROWSUM) {
            if (rows) {
                float t = 0.f;
#pragma unroll
                for (int r = 0; r < KT / 4; ++r) {
                    const int c = wave + r * 4, unit = (c >> 3) * 2 + (c & 1);
                    t += *lds_at<const float>(lds0 + AT + lane * F32_ROW + ((unit ^ flex_f32_swizzle(lane)) << 4) + ((c & 7) >> 1) * 4);
                }
                row_mid += t;
            }
        }
    };
    // (two loops: with the second level's end in one, the compiler made it 48 selects in every step)
#pragma unroll 1
    for (int i0 = 0; i0 < steps; i0 += 8) {            // a second-level sum holds 256 terms
        f32x16 mid = zero;
        row_mid = 0.f;
        const int end = min(i0 + 8, steps);
#pragma unroll 1
        for (int i = i0; i < end; i += 2) {
            step(std::integral_constant<int, 0>{}, i, mid);
            if (i + 1 < end) step(std::integral_constant<int, 1>{}, i + 1, mid);
        }
        acc += mid;
        row_acc += row_mid;
    }

    const FlexOut Q = args_at<FlexOut>(offsetof(FlexBatch, p) + (size_t)product * sizeof(FlexParams) + offsetof(FlexParams, out));
    constexpr int AHEAD = EPI == EPI_BIAS_ACT ? 1 : 4;
    FlexAhead<float, AHEAD> ahead;
    flex_request<float, TILE, TILE, THREADS, true, ROWSUM, float, EPI>(ahead, P, Q, g, tm, tn, rows);
    __syncthreads();
    float *const ctile = (float *)lds;
    float *const extra = (float *)(lds + C::C_BYTES);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 v = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        *(f32x4 *)(ctile + (wm + (lane & 31)) * C::CPITCH + wn + 8 * q + 4 * (lane >> 5)) = v;
    }
    if (rows) extra[tid] = row_acc;
    __syncthreads();
    flex_arrived(ahead);
    flex_epilogue<float, TILE, TILE, 1, THREADS, false, true, ROWSUM, float, EPI, AHEAD>(P, Q, g, tm, tn, ctile, extra, rows, ahead);
}

// ---- fp32 in whole vectors, few tiles and short reductions ------------------------------------------------------------------
// Where 4 divides the widths and phantom widths, 32 x 32 tiles whose eight teams of one wavefront take one, two or four groups of 16 terms each: the sums of
// flex_workgroup, group by group in the same order, so the same bits.
// What bounds it: a launch of 8 to 40 workgroups is a chain of latencies (parameters, one read of the operands, eight matrix instructions, the epilogue) and of
// instructions that are fetched cold.  So nothing is in a loop, what the epilogue reads is requested with the operands, and a wavefront stages what it
// alone reads: one barrier, ahead of the epilogue.
// 2 layers of 4 ranks of 64 + 24 trained at batch 32, ten launches (us a step, flex_workgroup : so): 54.9 : 44.4.
constexpr int F32_FEW_KC = F32_FEW_TERMS + 4, F32_FEW_KM = 32;                          // floats per LDS row
constexpr int F32_FEW_STAGE = 2 * 32 * F32_FEW_KC * 4;                                  // bytes of a group's two operands
// A team's region: the tiles of its groups' sums, its operands over the last one's place
constexpr int f32_few_region(int groups) { return (groups - 1) * FlexTileShape<32, 32>::C_BYTES + F32_FEW_STAGE; }
constexpr int f32_few_lds(int groups) { return 8 * f32_few_region(groups) + 512 * 4 + 64; }

// All ranks on the device, at most 8: dg_own is summed on read by the launch that needs it first, the senders in the order in which reduce_scatter_kernel
// adds them, and stored by the workgroups of tile column 0 for the launches behind it (the same step, with two launches for the sums : without, 44.4 : 42.4).
__device__ __forceinline__ u32x4 f32_few_sum(const SumOnRead &rs, int g, int64_t at /* element of the rank's dg_own */)
{
    constexpr int MOST = 7;                            // (the host allows at most 8 ranks)
    f32x4 v[MOST];
#pragma unroll
    for (int a = 0; a < MOST; ++a) {
        const int i = min(a, rs.p - 2), from = i < g ? i : i + 1, slot = g < from ? g : g - 1;      // the i-th sender other than g
        v[a] = gload<f32x4>((const float *)rs.src + ((int64_t)from * (rs.p - 1) + slot) * rs.per_slot + at);
    }
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int a = 0; a < MOST; ++a)
        if (a < rs.p - 1) sum += v[a];                 // uniform
    union { f32x4 f; u32x4 u; } r;
    r.f = sum;
    return r.u;
}

// 32 free positions from f0 on x 16 reduction positions from c0 on, two vectors a lane.  Free positions past the end repeat the last ones (nothing is
// stored of them), reduction positions past the end are zeros.
// rs: NULL, or where the operand's block dg_own comes from (KC: what lies behind the cut of the reduction index; KM: all of it); keep: store it, too.
template <int KIND>
__device__ __forceinline__ void f32_few_fetch(u32x4 (&v)[2], const FlexOperand &op, const FlexAxis &ax, const FlexAxis &fax, int f0, int c0, int g, int lane,
                                              const SumOnRead *rs = nullptr, bool keep = false)
{
    const float *p0 = (const float *)op.p0 + g * op.g0, *p1 = (const float *)op.p1 + g * op.g1;
    const int skip = op.skip0 + g * op.skip_g, end = ax.seg > 0 ? ax.total : ax.head;
    const float *at[2];
    bool in[2], summed[2] = {false, false}, store[2] = {false, false};
    int64_t own[2] = {0, 0};
    const bool sums = rs && rs->src;                   // uniform
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (KIND == FLEX_KC) {
            const int c = c0 + (lane & 3) * 4, r = min(f0 + (lane >> 2) + 16 * j, fax.head - 1);
            in[j] = c < end;
            const FlexLoc l = flex_locate(ax, in[j] ? c : 0, op.seg_stride, skip);
            at[j] = (l.region ? p1 + r * op.ld1 : p0 + r * op.ld0) + l.off;
            summed[j] = sums && in[j] && l.region;
            store[j] = keep && summed[j] && f0 + (lane >> 2) + 16 * j < fax.head;
            own[j] = r * op.ld1 + l.off;
        } else {
            int c = c0 + (lane >> 3) + 8 * j;
            in[j] = c < end;
            c = in[j] ? c : 0;
            const FlexLoc l = flex_locate(fax, min(f0 + (lane & 7) * 4, fax.total - 4), op.seg_stride, skip);
            const bool below = ax.seg > 0 && c >= ax.head, tail = below || (fax.seg > 0 && l.region);       // (one of the two indices is cut)
            at[j] = (tail ? p1 + (int64_t)(c - (below ? ax.head : 0)) * op.ld1 : p0 + (int64_t)c * op.ld0) + l.off;
            summed[j] = sums && in[j];
            store[j] = keep && summed[j] && f0 + (lane & 7) * 4 < fax.head;
            own[j] = (int64_t)c * op.ld0 + l.off;
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (summed[j]) v[j] = f32_few_sum(*rs, g, own[j]);
        else v[j] = gload<u32x4>(at[j]);
        if (store[j]) gstore<u32x4>((float *)rs->out + (int64_t)g * rs->per_slot + own[j], v[j]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int u = 0; u < 4; ++u) v[j][u] = in[j] ? v[j][u] : 0u;
}
// ... to LDS, as flex_operand reads it
template <int KIND>
__device__ __forceinline__ void f32_few_store(const u32x4 (&v)[2], float *tile, int lane)
{
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (KIND == FLEX_KC) {
            const int col = (lane & 3) * 4;
            float *to = tile + ((lane >> 2) + 16 * j) * F32_FEW_KC + (col & ~7) + ((col >> 1) & 2);
            *(u32x2 *)to = u32x2{v[j][0], v[j][2]};
            *(u32x2 *)(to + 4) = u32x2{v[j][1], v[j][3]};
        } else {
            *(u32x4 *)(tile + ((lane >> 3) + 8 * j) * F32_FEW_KM + (lane & 7) * 4) = v[j];
        }
    }
}

template <int GROUPS, int KA, int KB, int EPI>
__device__ __forceinline__ void flex_f32_few_workgroup(const FlexIn &P, int product, int wg, unsigned char *lds)
{
    typedef FlexTileShape<32, 32> F;
    constexpr bool ROWSUM = KA == FLEX_KM && KB == FLEX_KM;
    constexpr int PA = KA == FLEX_KC ? F32_FEW_KC : F32_FEW_KM, PB = KB == FLEX_KC ? F32_FEW_KC : F32_FEW_KM;
    const FlexTileAt at = flex_tile_at<true>(P, wg);
    const int g = at.g, tm = at.tm, tn = at.tn;
    const int lane = threadIdx.x & 63, team = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    FlexAxis ma{};                                     // the row index: never cut
    ma.head = P.M; ma.head_pad = ma.total = (P.M + 3) & ~3;
    const bool rows = ROWSUM && P.rowsum && tn == 0;   // uniform
    u32x4 va[GROUPS][2], vb[GROUPS][2];
#pragma unroll
    for (int i = 0; i < GROUPS; ++i) {
        const int c0 = (team * GROUPS + i) * F32_FEW_TERMS;
        f32_few_fetch<KA>(va[i], P.a, P.k, ma, tm * 32, c0, g, lane, &P.rs, tn == 0);
        f32_few_fetch<KB>(vb[i], P.b, P.k, P.n, tn * 32, c0, g, lane);
    }
    const FlexOut Q = args_at<FlexOut>(offsetof(FlexBatch, p) + (size_t)product * sizeof(FlexParams) + offsetof(FlexParams, out));
    FlexAhead<float, 1> ahead;
    flex_request<float, 32, 32, 512, true, ROWSUM, float, EPI>(ahead, P, Q, g, tm, tn, rows);
    constexpr int REGION = f32_few_region(GROUPS);
    unsigned char *const mine = lds + team * REGION;
    float *const ta = (float *)(mine + (GROUPS - 1) * F::C_BYTES), *const tb = ta + 32 * F32_FEW_KC;
    float *const extra = (float *)(lds + 8 * REGION);
    float row_acc = 0.f;
#pragma unroll
    for (int i = 0; i < GROUPS; ++i) {
        f32_few_store<KA>(va[i], ta, lane);
        f32_few_store<KB>(vb[i], tb, lane);
        flex_wave_sync();
        f32x16 sum[1][1];
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[0][0][e] = 0.f;
        flex_multiply<KA, KB, PA, PB, F32_FEW_TERMS>(sum, ta, tb, 0, 0, lane);
        if (rows) {
            float t = 0.f;
#pragma unroll
            for (int r = 0; r < F32_FEW_TERMS / 2; ++r) t += ta[((lane >> 5) + 2 * r) * F32_FEW_KM + (lane & 31)];
            row_acc += t;
        }
        flex_wave_sync();
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *(f32x4 *)((float *)(mine + i * F::C_BYTES) + (lane & 31) * F::CPITCH + 8 * q + 4 * (lane >> 5)) =
                f32x4{sum[0][0][4 * q], sum[0][0][4 * q + 1], sum[0][0][4 * q + 2], sum[0][0][4 * q + 3]};
        flex_wave_sync();
    }
    if (rows) extra[threadIdx.x] = row_acc;
    __syncthreads();
    flex_arrived(ahead);
    // the groups' sums, 16 of them to a second-level sum, over the first one's place (read again by the same thread alone)
    float *const ctile = (float *)lds;
    if (threadIdx.x < 256) {
        const int word = ((int)threadIdx.x >> 3) * F::CPITCH + ((int)threadIdx.x & 7) * 4;
        f32x4 total = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int h = 0; h < (8 * GROUPS + 15) / 16; ++h) {
            f32x4 mid = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 16 * h; j < 16 * h + 16 && j < 8 * GROUPS; ++j) mid += *(const f32x4 *)((const float *)(lds + j / GROUPS * REGION + j % GROUPS * F::C_BYTES) + word);
            total += mid;
        }
        *(f32x4 *)(ctile + word) = total;
    }
    flex_epilogue<float, 32, 32, 1, 512, false, true, ROWSUM, float, EPI, 1>(P, Q, g, tm, tn, ctile, extra, rows, ahead);
}

// ---- bf16 in 16-byte vectors: the ring of mfma_ring.h ----------------------------------------------------------------
// Problems whose widths and phantom widths 8 divides need neither the renumbering nor masked vectors.  A workgroup owns a 64 x 64 tile, each
// wavefront of a team a quadrant of it; two teams share it as in the kernel above, each with every other tile of the reduction range in stages
// of its own.  (Half of every step each, in common stages, has twice the barriers and half the bytes under way: one rank's layer of 1904,
// 224 tiles of 31 steps with operands that no cache holds, 18.2 us forward, 14.6 so, 15.7 the kernel above.)
// What bounds it: a step costs a wavefront a chain of instructions (operand reads, barrier, the loads' addresses, 2 or 4 matrix
// instructions), no pipe is busy; so a step of the loop above, 300 to 500 vector and scalar instructions, became one of about 60, and three
// workgroups of one team fill a compute unit (48 KB of stages each).  Two stages, or four to eight and fewer workgroups, are slower; so is a
// K-split with the whole tile per wavefront, whose four sums cost more to add than its fewer operand reads save.  Two teams: four stages
// each (128 KB) where no compute unit gets a second workgroup, two where one may.
// Passes (us, the kernel above : this one): one rank's layer of 64 44.9 : 35.7; layer of 1024, batch 1024, 36.0 : 30.4; 3 layers of 1024
// trained at batch 1000 107 : 99, of 2048 231 : 204; 4 layers of 1024 forward at batch 2048 71 : 60; 8 layers of 1720 + 480
// trained at batch 266 (two teams) 419 : 381, of 832 + 96 at 424 205 : 164.
constexpr int FLEX_RING_TILE = 64;

template <int KIND, int WAVES, int TILE>
__device__ __forceinline__ RingOperand flex_ring_init(const FlexOperand &op, const FlexAxis &k, int k_len, const FlexAxis &free, int free_len, int g, int r0,
                                                      int wave, int lane, uint32_t (&off0)[RingCfg<KIND, WAVES, TILE>::NV],
                                                      uint32_t (&off1)[RingCfg<KIND, WAVES, TILE>::NV])
{
    RingOperand s;
    s.base0 = (const __bf16 *)op.p0 + g * op.g0;
    s.base1 = (const __bf16 *)op.p1 + g * op.g1;
    s.c_lim = k_len;
    s.c_decides = k.seg > 0;
    s.c_split = k.seg > 0 ? k.head : 0x7fffffff;
    s.c_seg = k.seg; s.c_skip = op.skip0 + g * op.skip_g;
    s.c_magic = k.magic;
    s.c_mult0 = KIND == LD_KC ? 1 : (int)op.ld0; s.c_mult1 = KIND == LD_KC ? 1 : (int)op.ld1; s.c_seg_stride = (int)op.seg_stride;
    Axis r;
    r.decides = KIND == LD_KM && free.seg > 0;
    r.split = free.head; r.seg = free.seg > 0 ? free.seg : 1; r.magic = free.magic;
    r.mult0 = KIND == LD_KC ? op.ld0 : 1; r.mult1 = KIND == LD_KC ? op.ld1 : 1; r.seg_stride = op.seg_stride;
    ring_place<KIND, WAVES, TILE>(s, r, r0, free_len, wave, lane, off0, off1);
    return s;
}

// read_out(): the epilogue's part of the parameters, read behind the reduction.
template <int TEAMS, int RING, int KA, int KB, typename TOut, int EPI, typename ReadOut>
__device__ __forceinline__ void flex_ring_workgroup(const FlexIn &P, ReadOut read_out, int wg, unsigned char *lds)
{
    constexpr int TILE = FLEX_RING_TILE, WAVES = 4 * TEAMS;
    constexpr int A_BYTES = TILE * KT * 2, STAGE = 2 * A_BYTES;
    typedef RingCfg<KA, 4, TILE> CA;                   // a team loads its own tiles of the reduction range
    typedef RingCfg<KB, 4, TILE> CB;
    typedef FlexTileShape<TILE, TILE> F;
    constexpr int NL = CA::NV + CB::NV;
    constexpr bool ROWSUM = KA == LD_KM && KB == LD_KM;

    const FlexTileAt at = flex_tile_at<true>(P, wg);
    const int g = at.g, tm = at.tm, tn = at.tn;
    const int m0 = tm * TILE, n0 = tn * TILE;

    const int lane = threadIdx.x & 63, team = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    const int wave = __builtin_amdgcn_readfirstlane(((int)threadIdx.x >> 6) & 3);
    const int wm = wave >> 1, wn = wave & 1;     // the wavefront's quadrant
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LdsBytes)lds + team * RING * STAGE;
    FlexAxis ma{};                                     // the row index: never cut
    ma.head = P.M;
    const int k_len = P.k.seg > 0 ? P.k.total : P.k.head;          // (total pads a plain index, the batch, to whole vectors)
    uint32_t a_off0[CA::NV], a_off1[CA::NV], b_off0[CB::NV], b_off1[CB::NV];
    const RingOperand sa = flex_ring_init<KA, 4, TILE>(P.a, P.k, k_len, ma, P.M, g, m0, wave, lane, a_off0, a_off1);
    const RingOperand sb = flex_ring_init<KB, 4, TILE>(P.b, P.k, k_len, P.n, P.n.total, g, n0, wave, lane, b_off0, b_off1);

    // the tiles of the reduction range, from the last one down (see reduce_in_ring in gemm_mfma.h)
    const int tiles = (k_len + KT - 1) / KT;
    const int loops = (tiles + TEAMS - 1) / TEAMS, steps = TEAMS == 1 ? tiles : (tiles + 1 - team) >> 1;   // all teams', and this one's
    auto c_of = [=](int i) { return (tiles - 1 - team - TEAMS * i) * KT; };
    auto fetch = [&](int i, uint32_t stage) {
        ring_fetch<KA, 4, TILE>(sa, a_off0, a_off1, c_of(i), stage, wave);
        ring_fetch<KB, 4, TILE>(sb, b_off0, b_off1, c_of(i), stage + A_BYTES, wave);
    };
#pragma unroll
    for (int i = 0; i < RING; ++i)
        if (i < steps) fetch(i, lds0 + i * STAGE);     // uniform
    f32x16 acc[2];                                     // two sums: half of every step each
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[h][e] = 0.f;
    const int younger = min(steps, RING) - 1;
    if (steps > 0 && c_of(0) + KT > k_len) {           // uniform
        ring_landed<NL, RING - 1>(younger);
        ring_zero<KA, 4, TILE>(sa, c_of(0), lds0, wave, lane);
        ring_zero<KB, 4, TILE>(sb, c_of(0), lds0 + A_BYTES, wave, lane);
    }
    ring_wait_stage<NL, RING - 1>(younger);

    const int at_a = ring_lane_at<KA, TILE>(0, lane), at_b = ring_lane_at<KB, TILE>(0, lane);
    const bool rows = ROWSUM && P.rowsum && n0 == 0;   // uniform
    float row_acc = 0.f;                               // column threadIdx.x % 64 of A, rows wave + 4 i of every stage
    uint32_t cur = lds0;
    for (int t = 0; t < loops; ++t) {                  // uniform
        const uint32_t next = cur + STAGE == lds0 + RING * STAGE ? lds0 : cur + STAGE;
        // (all of the step's operands, then the barrier: reading them a step ahead into a second set of registers gains nothing)
        const bool mine = TEAMS == 1 || t < steps;     // uniform
        bf16x8 av[4], bv[4];
        if (mine) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                av[q] = ring_operand<KA, TILE>(cur, at_a, wm, q);
                bv[q] = ring_operand<KB, TILE>(cur + A_BYTES, at_b, wn, q);
            }
            if constexpr (ROWSUM) {
                if (rows) {
                    float sum = 0.f;
#pragma unroll
                    for (int i = 0; i < KT / 4; ++i) {
                        const int r = i * 4 + wave;
                        sum += (float)*lds_at<const __bf16>(cur + r * (TILE * 2) + ((((lane >> 3) ^ ring_swizzle<LD_KM, TILE>(r)) << 4) | ((lane & 7) << 1)));
                    }
                    row_acc += sum;
                }
            }
        }
        ring_wait_stage<NL, RING - 2>(steps - 2 - t);  // the next stage has landed, and everybody has read this one
        if (t + RING < steps) fetch(t + RING, cur);
        __builtin_amdgcn_sched_barrier(0);
        if (mine) {
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv[q], av[q], acc[q % 2], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        cur = next;
    }
    __syncthreads();

    const FlexOut Q = read_out();
    constexpr int PASSES = TILE * TILE / 8 / (WAVES * 64);
    FlexAhead<bf16_t, PASSES> ahead;
    flex_request<bf16_t, TILE, TILE, WAVES * 64, true, ROWSUM, TOut, EPI>(ahead, P, Q, g, tm, tn, rows);
    acc[0] += acc[1];
    float *ctile = (float *)lds;
    float *extra = (float *)(lds + TEAMS * F::C_BYTES);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 v = {acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]};
        *(f32x4 *)(ctile + team * (F::C_BYTES / 4) + (32 * wm + (lane & 31)) * F::CPITCH + 32 * wn + 8 * q + 4 * (lane >> 5)) = v;
    }
    if (rows) extra[threadIdx.x] = row_acc;
    __syncthreads();
    flex_arrived(ahead);
    flex_epilogue<bf16_t, TILE, TILE, TEAMS, WAVES * 64, false, true, ROWSUM, TOut, EPI, PASSES>(P, Q, g, tm, tn, ctile, extra, rows, ahead);
}
template <int TEAMS, int RING> constexpr int flex_ring_lds()
{
    return flex_max(TEAMS * RING * 2 * FLEX_RING_TILE * KT * 2,
                    TEAMS * FlexTileShape<FLEX_RING_TILE, FLEX_RING_TILE>::C_BYTES + 4 * TEAMS * 64 * 4 + 64);
}

__device__ __forceinline__ int flex_xcd_order(int i, int count)     // see xcd_order in gemm_mfma.h
{
    const int per = count >> 3;
    return i < per * 8 ? (i & 7) * per + (i >> 3) : i;
}

// FORWARD: products in the forward layout (bias + activation, or plain store).  Otherwise: products in the input-gradient
// layout (sigma' or plain store, kind 0) and in the weight-gradient layout (kind 1, float out), in any mix.
template <typename T, int TM, int TN, int TEAMS, bool FORWARD, bool FINE>
__global__ __launch_bounds__((FlexShape<T, TM, TN, TEAMS, FINE>::THREADS), (FlexShape<T, TM, TN, TEAMS, FINE>::MIN_WAVES)) void gemm_flex_kernel(FlexBatch batch)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    if (batch.tail.partial && blockIdx.x == 0) {       // uniform
        finish_loss(batch.tail, (float *)smem_raw);
        __syncthreads();
    }
    int j = 0;
    while (j + 1 < batch.count && (int)blockIdx.x >= batch.first_wg[j + 1]) ++j;       // uniform
    const int local = (int)blockIdx.x - batch.first_wg[j];
    const FlexIn P = args_at<FlexIn>(offsetof(FlexBatch, p) + (size_t)j * sizeof(FlexParams) + offsetof(FlexParams, in));
    if (local >= P.total_wg) return;
    const int wg = flex_xcd_order(local, P.total_wg);
    if constexpr (FORWARD) flex_workgroup<T, TM, TN, TEAMS, FINE, FLEX_KC, FLEX_KC, T, EPI_BIAS_ACT>(P, j, wg, smem_raw);
    else if (P.kind == 0) flex_workgroup<T, TM, TN, TEAMS, FINE, FLEX_KC, FLEX_KM, T, EPI_DACT>(P, j, wg, smem_raw);
    else flex_workgroup<T, TM, TN, TEAMS, FINE, FLEX_KM, FLEX_KM, float, EPI_STORE>(P, j, wg, smem_raw);
}

template <bool FORWARD, bool MANY>
__global__ __launch_bounds__(256, MANY ? 4 : 2) void gemm_flex_f32_kernel(FlexBatch batch)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    if (batch.tail.partial && blockIdx.x == 0) {       // uniform
        finish_loss(batch.tail, (float *)smem_raw);
        __syncthreads();
    }
    int j = 0;
    while (j + 1 < batch.count && (int)blockIdx.x >= batch.first_wg[j + 1]) ++j;       // uniform
    const int local = (int)blockIdx.x - batch.first_wg[j];
    const FlexIn P = args_at<FlexIn>(offsetof(FlexBatch, p) + (size_t)j * sizeof(FlexParams) + offsetof(FlexParams, in));
    if (local >= P.total_wg) return;
    const int wg = flex_xcd_order(local, P.total_wg);
    if constexpr (FORWARD) flex_f32_workgroup<(MANY ? 1 : 2), FLEX_KC, FLEX_KC, EPI_BIAS_ACT>(P, j, wg, smem_raw);
    else if (P.kind == 0) flex_f32_workgroup<(MANY ? 1 : 2), FLEX_KC, FLEX_KM, EPI_DACT>(P, j, wg, smem_raw);
    else flex_f32_workgroup<(MANY ? 1 : 2), FLEX_KM, FLEX_KM, EPI_STORE>(P, j, wg, smem_raw);
}

template <bool FORWARD, int GROUPS>
__global__ __launch_bounds__(512) void gemm_flex_f32_few_kernel(FlexBatch batch)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    if (batch.tail.partial && blockIdx.x == 0) {       // uniform
        finish_loss(batch.tail, (float *)smem_raw);
        __syncthreads();
    }
    int j = 0;
    while (j + 1 < batch.count && (int)blockIdx.x >= batch.first_wg[j + 1]) ++j;       // uniform
    const int local = (int)blockIdx.x - batch.first_wg[j];
    const FlexIn P = args_at<FlexIn>(offsetof(FlexBatch, p) + (size_t)j * sizeof(FlexParams) + offsetof(FlexParams, in));
    if (local >= P.total_wg) return;
    const int wg = flex_xcd_order(local, P.total_wg);
    if constexpr (FORWARD) flex_f32_few_workgroup<GROUPS, FLEX_KC, FLEX_KC, EPI_BIAS_ACT>(P, j, wg, smem_raw);
    else if (P.kind == 0) flex_f32_few_workgroup<GROUPS, FLEX_KC, FLEX_KM, EPI_DACT>(P, j, wg, smem_raw);
    else flex_f32_few_workgroup<GROUPS, FLEX_KM, FLEX_KM, EPI_STORE>(P, j, wg, smem_raw);
}

template <int TEAMS, int RING, bool FORWARD>
__global__ __launch_bounds__(TEAMS * 256, TEAMS == 1 ? 3 : 2) void gemm_flex_ring_kernel(FlexBatch batch)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    if (batch.tail.partial && blockIdx.x == 0) {       // uniform
        finish_loss(batch.tail, (float *)smem_raw);
        __syncthreads();
    }
    int j = 0;
    while (j + 1 < batch.count && (int)blockIdx.x >= batch.first_wg[j + 1]) ++j;       // uniform
    const int local = (int)blockIdx.x - batch.first_wg[j];
    const FlexIn P = args_at<FlexIn>(offsetof(FlexBatch, p) + (size_t)j * sizeof(FlexParams) + offsetof(FlexParams, in));
    if (local >= P.total_wg) return;
    const int wg = flex_xcd_order(local, P.total_wg);
    auto out = [=]() { return args_at<FlexOut>(offsetof(FlexBatch, p) + (size_t)j * sizeof(FlexParams) + offsetof(FlexParams, out)); };
    if constexpr (FORWARD) flex_ring_workgroup<TEAMS, RING, LD_KC, LD_KC, bf16_t, EPI_BIAS_ACT>(P, out, wg, smem_raw);
    else if (P.kind == 0) flex_ring_workgroup<TEAMS, RING, LD_KC, LD_KM, bf16_t, EPI_DACT>(P, out, wg, smem_raw);
    else flex_ring_workgroup<TEAMS, RING, LD_KM, LD_KM, float, EPI_STORE>(P, out, wg, smem_raw);
}

// One rank's compressions g = C y of several layers with at most 64 phantom neurons (8 divides them and the widths) in one launch, behind the
// forward pass: nothing on the rank waits for them.  A tile of 64 rows streams its rows of X once; the launch is bound by that, 64 MB for 8 layers
// of 1024 at batch 4096.
constexpr int COMPRESS_LAYERS = 32;
struct CompressMany {
    struct Layer {
        const void *X, *C;   // [M, K], [N, K]
        void *G;             // [M, N]
        int M, N, K;
        uint32_t magic_tiles, magic_last;      // see FlexIn
    } at[COMPRESS_LAYERS];
    int count;
    int first_wg[COMPRESS_LAYERS + 1];         // multiples of 8
};
static_assert(sizeof(CompressMany) <= 3840, "travels as kernel arguments (4 KB with the hidden ones)");

__global__ __launch_bounds__(256, 3) void compress_many_kernel(CompressMany many)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    int j = 0;
    while (j + 1 < many.count && (int)blockIdx.x >= many.first_wg[j + 1]) ++j;         // uniform
    const int local = (int)blockIdx.x - many.first_wg[j];
    const CompressMany::Layer l = args_at<CompressMany::Layer>(offsetof(CompressMany, at) + (size_t)j * sizeof(CompressMany::Layer));
    FlexIn P{};
    P.M = l.M;
    P.tiles_m = (l.M + FLEX_RING_TILE - 1) / FLEX_RING_TILE; P.tiles_n = 1; P.total_wg = P.tiles_m;
    if (local >= P.total_wg) return;
    P.magic_tiles = l.magic_tiles; P.magic_band = div_magic(FLEX_RASTER); P.magic_last = l.magic_last;
    P.a.p0 = l.X; P.b.p0 = l.C;
    P.a.ld0 = P.b.ld0 = l.K;
    P.a.skip0 = P.b.skip0 = NO_SKIP;
    P.k.head = P.k.head_pad = P.k.total = l.K;
    P.n.head = P.n.head_pad = P.n.total = l.N;
    auto out = [=]() {
        FlexOut Q{};
        Q.o0 = l.G; Q.o_ld0 = l.N;
        Q.ep.mode = EPI_STORE;
        return Q;
    };
    flex_ring_workgroup<1, 3, LD_KC, LD_KC, bf16_t, EPI_STORE>(P, out, flex_xcd_order(local, P.total_wg), smem_raw);
}

}  // namespace phantom
