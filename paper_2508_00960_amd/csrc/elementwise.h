// Memory-bound helpers of the phantom layer: local error, bias gradient,
// in-memory reduce-scatter, the loss's final sum.
#pragma once
#include "common.h"

namespace phantom {

// delta = dY * sigma'(S)   (Eq. (deltaL); the sigma' factor of Eq. (backprop)), 16 bytes per thread and pass.
// S is the pre-activation (any activation) or, for ReLU, the layer output.
// GELU is a kernel of its own: its erff and expf, inlined for every element, are what a launch of a few microseconds fetches cold.  2048 x 512 in bf16, ReLU,
// with GELU's code beside it : without, 35.8 : 35.5 us for a layer's forward and backward call (512 + 1008).
template <typename T, bool GELU>
__global__ __launch_bounds__(256) void delta_kernel(const T *__restrict__ dY, const T *__restrict__ S,
                                                   T *__restrict__ delta, int64_t count)
{
    constexpr int VEC = 16 / (int)sizeof(T), ACT = GELU ? ACT_GELU : ACT_RELU;
    typedef T TV __attribute__((ext_vector_type(VEC)));
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = first; i < count / VEC; i += stride) {
        TV d = ((const TV *)dY)[i];
        const TV s = ((const TV *)S)[i];
#pragma unroll
        for (int u = 0; u < VEC; ++u) d[u] = from_f32<T>(to_f32((T)d[u]) * act_deriv(ACT, to_f32((T)s[u])));
        ((TV *)delta)[i] = d;
    }
    for (int64_t i = count / VEC * VEC + first; i < count; i += stride)
        delta[i] = from_f32<T>(to_f32(dY[i]) * act_deriv(ACT, to_f32(S[i])));
}

// The loss of a step is left as partial sums (one per tile of
// the last layer's product); a launch of its own for adding up to 1024 of them costs 4 us, so the first
// memory-bound kernel that follows in the stream carries the sum as a rider: one of its workgroups (all
// 256 threads) calls finish_loss, which adds the partial sums in a fixed order into loss = scale * sum.
struct LossTail {
    const float *partial;    // NULL: nothing to do
    int n;
    float scale;
    float *loss;
};

// lred: 256 floats of LDS that nothing else uses meanwhile
__device__ __forceinline__ void finish_loss(const LossTail &t, float *lred)
{
    // 256 threads do the work; a larger workgroup's other threads only keep the barriers company
    const int me = threadIdx.x;
    if (me < 256) {
        float acc = 0.f;
        for (int i = me; i < t.n; i += 256) acc += t.partial[i];
        lred[me] = acc;
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (me < w) lred[me] += lred[me + w];
        __syncthreads();
    }
    if (me == 0) *t.loss = lred[0] * t.scale;
}

__global__ __launch_bounds__(256) void loss_kernel(LossTail t)
{
    __shared__ float lred[256];
    finish_loss(t, lred);
}

// Column sums of delta [rows x cols] (Eq. (bpb): dLoss/db = sum over the batch of delta).  One workgroup
// owns CSUM_COLS columns of one group and rows [chunk*rows_per_chunk, ...): 16-byte loads, row lanes x
// column lanes, one LDS reduction at the end.  With one chunk the result is stored (deterministic);
// with several chunks (few columns, many rows) each adds its part atomically into the cleared output.
// Rider (step only): workgroup (0,0,0) also finishes the loss (see LossTail).
constexpr int CSUM_COLS = 128;
template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(const T *__restrict__ delta, float *__restrict__ out, int rows, int cols,
                                                    int rows_per_chunk, LossTail tail)
{
    constexpr int VEC = 16 / (int)sizeof(T);            // elements per 16-byte load
    constexpr int CL = CSUM_COLS / VEC;                 // column lanes
    constexpr int RL = 256 / CL;                        // row lanes
    __shared__ float red[RL][CSUM_COLS + 1];
    const int g = blockIdx.y;
    const int cl = threadIdx.x % CL, rl = threadIdx.x / CL;
    const int col = blockIdx.x * CSUM_COLS + cl * VEC;
    const T *d = delta + (int64_t)g * rows * cols;
    const int r_begin = blockIdx.z * rows_per_chunk;
    const int r_end = min(rows, r_begin + rows_per_chunk);
    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
    if (col + VEC <= cols && (cols % VEC) == 0) {
        for (int r = r_begin + rl; r < r_end; r += RL) {
            const uint4 raw = *(const uint4 *)(d + (int64_t)r * cols + col);
            const T *e = (const T *)&raw;
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] += to_f32(e[v]);
        }
    } else {
        for (int r = r_begin + rl; r < r_end; r += RL)
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                if (col + v < cols) acc[v] += to_f32(d[(int64_t)r * cols + col + v]);
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) red[rl][cl * VEC + v] = acc[v];
    __syncthreads();
    if (threadIdx.x < CSUM_COLS) {
        const int c = blockIdx.x * CSUM_COLS + threadIdx.x;
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < RL; ++r) sum += red[r][threadIdx.x];
        if (c < cols) {
            if (gridDim.z == 1) out[(int64_t)g * cols + c] = sum;
            else unsafeAtomicAdd(out + (int64_t)g * cols + c, sum);
        }
    }
    __shared__ float lred[256];
    if (tail.partial && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) finish_loss(tail, lred);      // uniform
}

// In-memory Reduce-Scatter of Algorithm 1's backward: dg_own[i] = sum_{j != i} dG_send[j][slot of i on j].
// dG_send [p, p-1, B*k], dg_own [p, B*k]; on holder j, source i sits in slot i (i < j) or i-1 (i > j).
// A workgroup owns 32 * VEC consecutive elements of one receiver: thread = (element vector, sender lane);
// sender lane g adds the senders g, g + 8, g + 16, ... in fp32, the eight partial sums are added in lane
// order through LDS (a fixed order, whatever p is).  With one thread walking all p-1 senders the kernel
// was bound by the latency of its own loads (33 MB in 24 us at p = 64).  Workgroup (0,0) may carry the
// loss rider (LossTail).
constexpr int RS_LANES = 8;
template <typename T, int VEC>
__global__ __launch_bounds__(256) void reduce_scatter_kernel(const T *__restrict__ dG_send, T *__restrict__ dg_own,
                                                            int p, int64_t per_slot, LossTail tail)
{
    typedef T TV __attribute__((ext_vector_type(VEC)));
    // part[lane][u * 40 + ev]: element u of vector ev.  A wavefront writes 32 consecutive words per sender lane, its
    // two sender lanes 32 banks apart; the 64 threads of a wavefront read 8 u-rows x 8 vectors, and the rows start
    // 40 words = 8 banks mod 64 apart in a permuted order (with rows of 32 * VEC + 1 words indexed [ev * VEC + u]
    // the writes met each bank four times: SQ_LDS_BANK_CONFLICT 448 cycles per workgroup, now 64)
    constexpr int RS_U_PITCH = 40, RS_LANE_PITCH = VEC * RS_U_PITCH + 32;
    __shared__ float part[RS_LANES * RS_LANE_PITCH];
    const int ev = threadIdx.x & 31, lane = threadIdx.x >> 5;
    const int64_t e = ((int64_t)blockIdx.x * 32 + ev) * VEC;
    const int i = blockIdx.y;
    float acc[VEC];
#pragma unroll
    for (int u = 0; u < VEC; ++u) acc[u] = 0.f;
    if (e < per_slot) {
        for (int j = lane; j < p; j += RS_LANES) {
            if (j == i) continue;
            const int slot = i < j ? i : i - 1;
            const T *src = dG_send + ((int64_t)j * (p - 1) + slot) * per_slot + e;
            if constexpr (VEC > 1) {
                const TV v = *(const TV *)src;
#pragma unroll
                for (int u = 0; u < VEC; ++u) acc[u] += to_f32((T)v[u]);
            } else {
                acc[0] += to_f32(src[0]);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < VEC; ++u) part[lane * RS_LANE_PITCH + u * RS_U_PITCH + ev] = acc[u];
    __syncthreads();
    // 256 threads, 32 * VEC elements: thread t finishes elements t, t + 256, ...
    for (int c = threadIdx.x; c < 32 * VEC; c += 256) {
        const int64_t at = (int64_t)blockIdx.x * 32 * VEC + c;
        if (at >= per_slot) continue;
        float sum = 0.f;
#pragma unroll
        for (int g = 0; g < RS_LANES; ++g) sum += part[g * RS_LANE_PITCH + (c % VEC) * RS_U_PITCH + c / VEC];
        dg_own[(int64_t)i * per_slot + at] = from_f32<T>(sum);
    }
    __shared__ float lred[256];
    if (tail.partial && blockIdx.x == 0 && blockIdx.y == 0) finish_loss(tail, lred);      // uniform; rider, see LossTail
}

// Buffers that a step adds into (bias gradients, counters), cleared by a launch that runs anyway before the first of them
// is added to, or by one launch of their own.
constexpr int CLEAR_MAX = 8;
struct ClearList {
    int count;               // 0: nothing to do
    int n[CLEAR_MAX];        // floats
    float *p[CLEAR_MAX];
};
// workgroup `job` of `jobs`, of `threads` threads
__device__ __forceinline__ void clear_rider(const ClearList &c, int job, int jobs, int threads)
{
    if (c.count == 0) return;                          // uniform
#pragma unroll 1
    for (int i = 0; i < c.count; ++i)
        for (int z = job * threads + (int)threadIdx.x; z < c.n[i]; z += jobs * threads) c.p[i][z] = 0.f;
}
__global__ __launch_bounds__(256) void clear_kernel(ClearList c) { clear_rider(c, (int)blockIdx.x, (int)gridDim.x, 256); }

__global__ __launch_bounds__(256) void fill_zero_kernel(float *__restrict__ dst, int64_t count)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) dst[i] = 0.f;
}

template <typename T>
__global__ __launch_bounds__(256) void copy_kernel(const T *__restrict__ src, T *__restrict__ dst, int64_t count)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) dst[i] = src[i];
}

// Copies of bf16 matrices (or of float ones, as twice the columns) whose rows of `len` elements become rows of `plen`, a multiple of 8, with zeros behind
// them: 16 bytes per thread.
// len is even, so that every row starts on a word.  Bound by the launch: 9 MB for 6 layers of 7 peers' G [8192, 4] and D [1024, 4] to 8.
constexpr int PAD_ENTRIES = 112;
struct PadList {
    struct Entry {
        const void *src;
        void *dst;
        int vectors, len, plen, first_block;
    } at[PAD_ENTRIES];
    int count;
};
static_assert(sizeof(PadList) <= 3840, "travels as kernel arguments (4 KB with the hidden ones)");

__global__ __launch_bounds__(256) void pad_kernel(PadList list)
{
    int j = 0;
    while (j + 1 < list.count && (int)blockIdx.x >= list.at[j + 1].first_block) ++j;      // uniform
    const PadList::Entry e = list.at[j];
    const int v = ((int)blockIdx.x - e.first_block) * 256 + (int)threadIdx.x;
    if (v >= e.vectors) return;
    const int per_row = e.plen / 8, row = v / per_row, col = (v - row * per_row) * 8;
    typedef uint32_t Words __attribute__((ext_vector_type(4)));
    typedef uint32_t AnyWords __attribute__((ext_vector_type(4), aligned(4)));
    const uint32_t *src = (const uint32_t *)e.src + ((int64_t)row * e.len + col) / 2;
    Words x;
    if (col + 8 <= e.len) {
        x = *(const AnyWords *)src;
    } else {
#pragma unroll
        for (int h = 0; h < 4; ++h) x[h] = col + 2 * h < e.len ? src[h] : 0u;
    }
    ((Words *)e.dst)[v] = x;
}

// Back from rows of `plen` floats with `len` (even) that count: out <- the gradient (NULL: not wanted), master <- the updated fp32 weights and
// w <- the same in bf16 (master == NULL: no update).  Two elements per thread.
struct UnpadList {
    struct Entry {
        const float *grad;
        float *out;
        const float *updated;
        float *master;
        void *w;
        int pairs, len, plen, first_block;
    } at[PAD_ENTRIES / 2];
    int count;
};
static_assert(sizeof(UnpadList) <= 3840, "travels as kernel arguments (4 KB with the hidden ones)");

__global__ __launch_bounds__(256) void unpad_kernel(UnpadList list)
{
    int j = 0;
    while (j + 1 < list.count && (int)blockIdx.x >= list.at[j + 1].first_block) ++j;      // uniform
    const UnpadList::Entry e = list.at[j];
    const int v = ((int)blockIdx.x - e.first_block) * 256 + (int)threadIdx.x;
    if (v >= e.pairs) return;
    typedef float F2 __attribute__((ext_vector_type(2)));
    typedef bf16_t B2 __attribute__((ext_vector_type(2)));
    const int per_row = e.len / 2, row = v / per_row, col = (v - row * per_row) * 2;
    const int64_t from = (int64_t)row * e.plen + col;
    if (e.master) {                                    // uniform
        const F2 m = *(const F2 *)(e.updated + from);
        ((F2 *)e.master)[v] = m;
        ((B2 *)e.w)[v] = B2{(bf16_t)m[0], (bf16_t)m[1]};
    }
    if (e.out) ((F2 *)e.out)[v] = *(const F2 *)(e.grad + from);      // uniform
}

// dst [rows, len] <- the first len columns of src [rows, plen]
template <typename T>
__global__ __launch_bounds__(256) void unpad_copy_kernel(const T *src, T *dst, int64_t rows, int len, int plen)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rows * len; i += stride) dst[i] = src[i / len * plen + i % len];
}

}  // namespace phantom
