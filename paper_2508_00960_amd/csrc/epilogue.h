// What a product does with its output tile besides storing it, shared by the product kernels.
#pragma once
#include "common.h"
#include "views.h"

namespace phantom {

enum { EPI_STORE = 0, EPI_BIAS_ACT = 1, EPI_DACT = 2 };

struct Epilogue {
    int32_t mode;
    int32_t act;
    const void *bias;    // EPI_BIAS_ACT: [N] per group, storage type
    int64_t bias_g;
    void *aux;           // EPI_BIAS_ACT: optional pre-activation out; EPI_DACT: pre-activation (or ReLU output) in
                         //   (gemm_mfma_kernel: NULL = multiply by nothing, for the column sums alone)
    int64_t aux_ld;      //   plain row-major [M x N]
    int64_t aux_g;
    int32_t aux_f32;     // aux holds float instead of the storage type
    int32_t aux_deriv;   // aux holds sigma'(pre-activation), in float, instead of the pre-activation:
                         //   EPI_BIAS_ACT writes it, EPI_DACT multiplies by it as it stands
    float *colsum;       // gemm_mfma_kernel only, optional: the column sums of the stored output (as rounded to
    int64_t colsum_g;    //   the output type) are ADDED to colsum[N] per group; the caller zeroes it first
    // EPI_BIAS_ACT, optional (mse_target != NULL): the layer is the last one and the MSE output
    // error is formed on the way out (Eq. (deltaL)): with y the output as stored and t = mse_target (laid out
    // like aux: aux_ld, aux_g, storage type), mse_delta <- ((y - t) * mse_inv_b) * sigma'(pre-activation)
    // (sigma' of the pre-activation in float for GELU, from y for ReLU), colsum
    // then receives the column sums of mse_delta instead of y's, and mse_partial[tile] <- sum over the
    // tile of (y - t)^2, tile = (group * tile rows + tile row) * tile columns + tile column.
    const void *mse_target;
    void *mse_delta;
    float *mse_partial;
    float mse_inv_b;
    int32_t aux_bits;    // gemm_mfma_kernel, 8-element vectors, ReLU only: aux holds ONE BIT per element, (stored output > 0), i.e.
                         //   ReLU' as the backward pass reads it off the stored output, in an eighth of the bytes:
                         //   EPI_BIAS_ACT writes it (bit u of byte (g*aux_g + m*aux_ld + n) / 8 = column n + u),
                         //   EPI_DACT keeps or zeroes each element by it
};

// SGD inside the epilogue that finishes a weight gradient (Section VI's plain SGD): the parameters that the gradient
// belongs to, laid out like the output's two regions.  w0 == nullptr: none.
struct SgdInPlace {
    float *master0, *master1;    // bf16 storage: fp32 master copies: master -= lr * gradient.  NULL with fp32 storage.
    void *w0, *w1;               // bf16: compute copies, w = bf16(master).  fp32: w -= lr * gradient
    float lr;
    short keep_grad;             // also store the gradient (the caller wants to see it)
    short past_caches;           // gemm_mfma kernels: read the masters past the caches (step_fits_last_cache)
    float *bias_master;          // weight gradients only: the layer's bias [M], likewise
    void *bias_w;                //   NULL: none
    const float *bias_grad;      // gemm_mfma kernels: its finished gradient (Eq. (bpb): column sums of delta, left by earlier
                                 //   launches); the tiles of the first tile column update the rows they cover
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Global loads and stores that the compiler cannot mistake for generic ones: the pointers come out of parameter
// blocks, and flat instructions also count as LDS operations (every wait for an LDS read then waits for all of
// them).  _nt: streaming (read or written once).
template <typename V> __device__ __forceinline__ V gload(const void *p) { return *(const __attribute__((address_space(1))) V *)(uintptr_t)p; }
template <typename V> __device__ __forceinline__ V gload_nt(const void *p)
{
    return __builtin_nontemporal_load((const __attribute__((address_space(1))) V *)(uintptr_t)p);
}
template <typename V> __device__ __forceinline__ void gstore(void *p, const V &v) { *(__attribute__((address_space(1))) V *)(uintptr_t)p = v; }
template <typename V> __device__ __forceinline__ void gstore_nt(void *p, const V &v)
{
    __builtin_nontemporal_store(v, (__attribute__((address_space(1))) V *)(uintptr_t)p);
}

}  // namespace phantom
