// C ABI of libphantom.so: argument checks, workspace layout, and the sequence of
// kernel launches that makes up each operator of the phantom layer.
// Declarations and the meaning of every argument: include/phantom.h.
#include "../../include/phantom.h"

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "common.h"
#include "elementwise.h"
#include "few_rows.h"
#include "gemm_flex.h"
#include "gemm_mfma.h"
#include "launch_rules.h"
#include "lds_reserve.h"
#include "thin_product.h"
#include "views.h"

using namespace phantom;

namespace {

thread_local char g_err[512];

ph_status fail(ph_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

// The body of a C entry point: the lists that a call keeps of its layers may not fit the host's memory, and an exception must
// not leave a C function.
template <typename F>
ph_status without_exceptions(F &&body)
{
    try {
        return body();
    } catch (const std::bad_alloc &) {
        return fail(PH_ERR_LAUNCH, "out of host memory");
    } catch (const std::exception &e) {
        return fail(PH_ERR_LAUNCH, "internal error: %s", e.what());
    }
}

#define PH_TRY(expr) do { ph_status st__ = (expr); if (st__ != PH_OK) return st__; } while (0)

// Measurement switches (force one of two launch schedules that the library otherwise chooses between by
// its own model) exist only in a library built with -DPHANTOM_TUNING_ENV; a production build reads no
// environment variable.
inline const char *tuning_env(const char *name)
{
#ifdef PHANTOM_TUNING_ENV
    return getenv(name);
#else
    (void)name;
    return nullptr;
#endif
}

// One layer's shapes on this GPU.  si / so: inputs / outputs of the layer held by one rank (equal unless
// the problem gives per-layer widths).
struct Geo {
    int64_t p, k, B, si, so, q, Kc;
    int64_t k_given;  // the caller's phantom width: k, or less where the step runs on padded copies (padded_geos)
    int groups;       // ranks held on this GPU: 1 or p
    bool all;         // all-ranks mode
    int act, dtype, rank, layers;
    size_t esz;       // bytes per element of the storage type
    int vec;          // bf16: widest vector (8 or 4 elements) dividing si, so and k; 0: the kernels of gemm_flex.h only
    bool fine;        // bf16: ... in their FINE form
    bool whole;       // fp32: 4 divides si, so and k, and 32 bits hold a byte offset inside a rank's share of a tensor (FlexF32Loader)
};

// Checks the problem and fills in the shapes of layer `layer` (0-based).
ph_status make_geo(const ph_problem *pr, Geo &g, int layer = 0)
{
    if (!pr) return fail(PH_ERR_INVALID_ARG, "problem is NULL");
    if (pr->p < 1) return fail(PH_ERR_INVALID_ARG, "p = %lld must be >= 1", (long long)pr->p);
    if (pr->batch < 1) return fail(PH_ERR_INVALID_ARG, "batch = %lld must be >= 1", (long long)pr->batch);
    if (pr->act < PH_ACT_IDENTITY || pr->act > PH_ACT_GELU) return fail(PH_ERR_INVALID_ARG, "unknown activation %d", pr->act);
    if (pr->dtype != PH_F32 && pr->dtype != PH_BF16) return fail(PH_ERR_INVALID_ARG, "unknown dtype %d", pr->dtype);
    if (pr->rank < -1 || pr->rank >= pr->p) return fail(PH_ERR_INVALID_ARG, "rank = %d must lie in [-1, p)", pr->rank);
    if (pr->layers < 1) return fail(PH_ERR_INVALID_ARG, "layers = %d must be >= 1", pr->layers);
    if (layer < 0 || layer >= pr->layers) return fail(PH_ERR_INVALID_ARG, "layer %d of %d", layer, pr->layers);
    int64_t n_in = pr->n, n_out = pr->n, k = pr->k;
    if (pr->widths) {
        if (pr->p > 1 && !pr->ks) return fail(PH_ERR_INVALID_ARG, "widths without ks");
        n_in = pr->widths[layer]; n_out = pr->widths[layer + 1];
        if (pr->ks) k = pr->ks[layer];
    } else if (pr->ks) {
        return fail(PH_ERR_INVALID_ARG, "ks without widths");
    }
    if (n_in < 1 || n_in % pr->p || n_out < 1 || n_out % pr->p)
        return fail(PH_ERR_INVALID_ARG, "layer %d: widths %lld -> %lld must be positive multiples of p = %lld", layer,
                    (long long)n_in, (long long)n_out, (long long)pr->p);
    const int64_t si = n_in / pr->p, so = n_out / pr->p;
    if (pr->p > 1 && (k < 1 || k > std::max(si, so)))
        return fail(PH_ERR_INVALID_ARG, "layer %d: k = %lld must lie in [1, n/p = %lld]", layer, (long long)k,
                    (long long)std::max(si, so));
    g.p = pr->p; g.B = pr->batch; g.si = si; g.so = so; g.q = pr->p - 1;
    g.k = g.k_given = g.q > 0 ? k : 0;
    g.Kc = si + g.q * g.k;
    g.all = pr->rank < 0;
    g.groups = g.all ? (int)pr->p : 1;
    g.act = pr->act; g.dtype = pr->dtype; g.rank = pr->rank; g.layers = pr->layers;
    g.esz = pr->dtype == PH_BF16 ? 2 : 4;
    g.vec = 0;
    g.fine = pr->dtype == PH_BF16 && ((si | so | g.k) & 1);
    if (pr->dtype == PH_BF16) {
        for (int v = 8; v >= 4 && !g.vec; v >>= 1)
            if (si % v == 0 && so % v == 0 && (g.q == 0 || g.k % v == 0)) g.vec = v;
    }
    // The matrix-core kernels address an operand with 32-bit element offsets inside one rank's share of a tensor:
    // a problem with a larger tensor goes through the kernels with 64-bit offsets like one whose widths
    // allow no vector loads (gemm_flex.h).
    {
        const int64_t wide = std::max(si, so), slots = g.all ? g.p : g.q;
        const int64_t largest = std::max({g.B * wide, slots * g.B * g.k, so * si, slots * so * g.k, g.k * si});
        g.whole = pr->dtype == PH_F32 && si % 4 == 0 && so % 4 == 0 && g.k % 4 == 0 && largest < (int64_t)1 << 30 && g.q * g.k * g.k < (int64_t)1 << 32;
        if (largest > 0x7fffffff) {
            g.vec = 0;
            g.fine = pr->dtype == PH_BF16;
        }
        // they also divide a position among the peers' segments by k with a multiply (Axis::magic), exact while
        // position * k < 2^32
        if (g.q * g.k * g.k >= (int64_t)1 << 32) g.vec = 0;
    }
    // index arithmetic inside the kernels uses 32-bit row/column numbers and a 3-D grid
    if (g.B > (1 << 22) || si > (1 << 22) || so > (1 << 22) || g.Kc > (1 << 24) || so + g.q * g.k > (1 << 24) || g.p > 65535)
        return fail(PH_ERR_UNSUPPORTED, "problem too large for 32-bit tile indices (batch, n/p <= 2^22, n/p+(p-1)k <= 2^24)");
    // ... and numbers its 128 x 128 output tiles with 32 bits, over all ranks held: the largest product of the layer
    {
        auto t = [](int64_t x) { return (x + 127) / 128; };
        const int64_t tiles = std::max({t(g.B) * t(so), t(g.B) * t(si), t(g.B) * t(std::max<int64_t>(g.q * g.k, 1)),
                                        t(so) * t(g.Kc), t(std::max<int64_t>(g.k, 1)) * t(si)}) * g.groups;
        if (tiles * 8 > 0x7fffffff)
            return fail(PH_ERR_UNSUPPORTED, "layer %d: %lld output tiles in one product, more than the kernels number", layer,
                        (long long)tiles);
    }
    return PH_OK;
}

// every layer's shapes (a uniform problem: `layers` copies of the same)
ph_status make_geos(const ph_problem *pr, std::vector<Geo> &geos)
{
    Geo first;
    PH_TRY(make_geo(pr, first, 0));
    geos.assign((size_t)pr->layers, first);
    for (int l = 1; l < pr->layers; ++l) PH_TRY(make_geo(pr, geos[(size_t)l], l));
    return PH_OK;
}

ph_status need(const void *p, const char *name)
{
    if (!p) return fail(PH_ERR_INVALID_ARG, "%s is NULL", name);
    if ((uintptr_t)p & 15) return fail(PH_ERR_INVALID_ARG, "%s is not 16-byte aligned", name);
    return PH_OK;
}
ph_status optional(const void *p, const char *name)
{
    if (p && ((uintptr_t)p & 15)) return fail(PH_ERR_INVALID_ARG, "%s is not 16-byte aligned", name);
    return PH_OK;
}

// Do the `na` bytes at a and the `nb` bytes at b share any?
bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    return a && b && (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

ph_status check_launch(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PH_ERR_LAUNCH, "%s: %s", what, hipGetErrorString(e));
    return PH_OK;
}

// ---- optional per-launch timing (phantom_profile_begin / _end) ----------------------------
struct ProfRec {
    const char *name;
    int64_t M, N, K;
    int groups;
    int64_t M2, N2, K2;   // second to fourth product of a launch that carries several (0 if none)
    int64_t M3, N3, K3;
    int64_t M4, N4, K4;
};
struct Profiler {
    bool on = false;
    std::vector<hipEvent_t> ev;      // 2 per record: start, stop
    std::vector<ProfRec> recs;
    size_t cap = 0;
    bool calibrated = false;
};
thread_local Profiler g_prof;
constexpr int PROF_CALIBRATION_LAUNCHES = 32;
const char *const PROF_EMPTY_NAME = "(empty launch)";

// Brackets one kernel launch with a pair of events on its stream while profiling is on.
struct ProfScope {
    hipStream_t st;
    long idx = -1;
    ProfScope(const char *name, int64_t M, int64_t N, int64_t K, int groups, hipStream_t s, int64_t M2 = 0,
              int64_t N2 = 0, int64_t K2 = 0, int64_t M3 = 0, int64_t N3 = 0, int64_t K3 = 0, int64_t M4 = 0, int64_t N4 = 0,
              int64_t K4 = 0) : st(s)
    {
        if (!g_prof.on) return;
        if (!g_prof.calibrated) {
            // What an event pair reads around a kernel that does nothing: the part of every figure
            // below that is launch and time-stamp latency rather than execution.  Reported as an
            // entry of its own so that the caller can subtract it.
            g_prof.calibrated = true;
            for (int i = 0; i < PROF_CALIBRATION_LAUNCHES && g_prof.recs.size() < g_prof.cap; ++i) {
                const long at = (long)g_prof.recs.size();
                g_prof.recs.push_back(ProfRec{PROF_EMPTY_NAME, 0, 0, 0, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0});
                (void)hipEventRecord(g_prof.ev[2 * at], st);
                hipLaunchKernelGGL(fill_zero_kernel, dim3(256), dim3(256), 0, st, (float *)nullptr, (int64_t)0);
                (void)hipEventRecord(g_prof.ev[2 * at + 1], st);
            }
        }
        if (g_prof.recs.size() >= g_prof.cap) return;
        idx = (long)g_prof.recs.size();
        g_prof.recs.push_back(ProfRec{name, M, N, K, groups, M2, N2, K2, M3, N3, K3, M4, N4, K4});
        (void)hipEventRecord(g_prof.ev[2 * idx], st);
    }
    ~ProfScope()
    {
        if (idx >= 0) (void)hipEventRecord(g_prof.ev[2 * idx + 1], st);
    }
};

// ---- workspace ---------------------------------------------------------------
struct Arena {
    char *base;
    size_t used;
    void *take(size_t bytes)
    {
        size_t at = (used + 255) & ~(size_t)255;
        used = at + bytes;
        return base ? base + at : nullptr;
    }
};

struct BwdWs {
    void *delta;        // [groups, B, so] storage type
};

BwdWs carve_bwd(Arena &a, const Geo &g)
{
    BwdWs w;
    w.delta = a.take((size_t)g.groups * g.B * g.so * g.esz);
    return w;
}

struct StepWs {
    std::vector<void *> Y, A, G;
    std::vector<void *> relu_bits;                  // per layer, or NULL: one bit per element of y_l (y_l > 0), see relu_bits_ok
    void *dYa, *dYb, *dG_send, *dg_own;
    float *dLw[2], *dCw[2], *dDw[2];                // two sets, used by alternate layers: a layer's update may still read
                                                    //   its gradients while the layer below writes its own
    float *dbias, *mse_partial;                     // dbias: one block, layer l's [groups, so_l] at dbias_at[l]
    std::vector<int64_t> dbias_at;                  // float offsets into dbias; dbias_at[layers] = the block's length
    unsigned *arrived;                              // one word per cut tile (cut_tiles) right behind the dbias block: cleared with
                                                    //   it at the start of a step, left zero by every launch that uses them
    int64_t arrived_words;
    float *parts;                                   // deferred weight gradients (one rank): the pieces' results of the cut
    ProductTable *table;                            //   compressor gradients, the launch's parameter table (DEFER_SMALL), and
    std::vector<void *> delta_of;                   //   every layer's delta [B, so_l]
    BwdWs bwd;
};

// ReLU in bf16 storage: what the backward pass needs of layer l is the sign of its stored output alone.  Where the
// update of layer l and the input gradient of layer l + 1 (whose epilogue multiplies by sigma'_l) both run on the
// matrix cores with 8-element vectors, the update leaves one bit per element and the input gradient reads
// that instead of the bf16 output: an eighth of the bytes (configuration 2: 8.4 MB -> 0.5 MB per launch).
bool relu_bits_ok(const std::vector<Geo> &geos, size_t l)
{
    return l + 1 < geos.size() && geos[l].act == PH_ACT_RELU && geos[l].dtype == PH_BF16 && geos[l].vec == 8 &&
           geos[l + 1].vec == 8;
}

inline int64_t tiles_of(int64_t M, int64_t N) { return ((M + MT - 1) / MT) * ((N + MT - 1) / MT); }

bool use_flex(const std::vector<Geo> &geos, bool backward, bool single_call = false);

bool all_alike(const std::vector<Geo> &geos)
{
    return std::all_of(geos.begin(), geos.end(), [&](const Geo &g) { return g.si == geos[0].si && g.so == geos[0].so && g.k == geos[0].k; });
}

// One rank's backward pass over two or more layers keeps every layer's delta and runs all weight + compressor
// gradients in one launch at its end (gemm_mfma_uniform_kernel, gemm_mfma_table_kernel): bf16 with 8-element vectors.
// A layer with at most 256 weight-gradient tiles would leave compute units idle in a launch of its own.  Larger ones (layers alike): within one
// launch a tile's epilogue runs beside others' loops to the end, where each layer's own launch ended with all its compute units in the update.
// Us a step, a launch per layer : one: 4 layers of 4096 trained at batch 1024 575 : 539, 3 of 3072 with GELU at 1500 425 : 384, 3 of 2048 + 192 at 2048
// 304 : 263, at 4096 475 : 413, 2 of 4096 at 4096 712 : 703.  Their deltas then lie where a launch per layer has its buffers (carve_step), so that
// no step needs more workspace for it; where they do not fit there, each layer keeps its launch.
// (All ranks on the device: the weight gradients' launches carry the next error compression and the update on the compute units they leave
// idle, and putting them off made configuration 2 slower, 0.272 against 0.260 ms; a single layer has nothing to gain.)
enum Deferral { DEFER_NONE, DEFER_SMALL, DEFER_LARGE };
Deferral deferred_weight_gradients(const std::vector<Geo> &geos)
{
    const size_t L = geos.size();
    if (L < 2 || 2 * L > (size_t)TABLE_PRODUCTS) return DEFER_NONE;
    bool large = false;
    for (const Geo &g : geos) {
        if (g.all || g.dtype != PH_BF16 || g.vec != 8) return DEFER_NONE;
        large = large || tiles_of(g.so, g.Kc) > 256;
    }
    if (!large) return DEFER_SMALL;
    const Geo &g = geos[0];
    if (L > (size_t)UNIFORM_LAYERS || !all_alike(geos) || use_flex(geos, true)) return DEFER_NONE;
    const int64_t delta = (g.B * g.so * (int64_t)g.esz + 255) & ~(int64_t)255, beside = 4 * (g.so * g.Kc + g.k * g.si);
    return ((int64_t)L - 3) * delta <= beside ? DEFER_LARGE : DEFER_NONE;
}

// The compressor gradient [k, si] of a layer has few tiles with a long reduction (configuration 4: 8 tiles of 64
// steps, half of their rows empty).  In that launch they are cut along the batch into pieces of at least 16 steps,
// at most 4, which go out first and add up without atomics (MfmaParams::parts).
int compressor_gradient_pieces(const Geo &g)
{
    const int64_t ksteps = (g.B + KT - 1) / KT;
    return (int)std::max<int64_t>(1, std::min<int64_t>(ksteps / 16, 4));
}

// Output tiles of that launch whose reduction is cut (MfmaParams::arrived has a word for each).
int64_t cut_tiles(const std::vector<Geo> &geos)
{
    int64_t tiles = 0;
    if (deferred_weight_gradients(geos) != DEFER_SMALL) return 0;
    for (const Geo &g : geos)
        if (g.q > 0 && compressor_gradient_pieces(g) > 1) tiles += tiles_of(g.k, g.si);
    return tiles;
}

// geos: every layer's shapes.  Buffers that are reused from layer to layer take the largest layer's size.
// forward: only what a forward step uses.
StepWs carve_step(Arena &a, const std::vector<Geo> &geos, bool forward = false)
{
    StepWs w{};
    for (size_t l = 0; l < geos.size(); ++l)
        w.relu_bits.push_back(!forward && relu_bits_ok(geos, l) ? a.take((size_t)geos[l].groups * geos[l].B * geos[l].so / 8) : nullptr);
    const Geo &g0 = geos[0];
    size_t act_max = 0, k_max = 0, lw_max = 0, cw_max = 0, dw_max = 0;
    int64_t dbias_total = 0;
    for (const Geo &g : geos) {
        const size_t act_bytes = (size_t)g.groups * g.B * g.so * g.esz;
        w.Y.push_back(a.take(act_bytes));
        // GELU keeps per layer but the last, in float: fp32 storage, the pre-activation; bf16 storage, sigma'(pre-activation)
        w.A.push_back(!forward && g.act == PH_ACT_GELU && w.Y.size() < geos.size() ? a.take((size_t)g.groups * g.B * g.so * sizeof(float)) : nullptr);
        w.G.push_back(g.q > 0 ? a.take((size_t)g.groups * g.B * g.k * g.esz) : nullptr);   // all-ranks: [p,B,k]; one-rank: [B,k]
        act_max = std::max(act_max, (size_t)std::max(g.si, g.so));
        k_max = std::max(k_max, (size_t)g.k);
        lw_max = std::max(lw_max, (size_t)(g.so * g.si));
        cw_max = std::max(cw_max, (size_t)(g.k * g.si));
        dw_max = std::max(dw_max, (size_t)(g.q * g.so * g.k));
        w.dbias_at.push_back(dbias_total);
        dbias_total += ((int64_t)g.groups * g.so + 3) & ~(int64_t)3;   // every layer's block starts 16-byte aligned
    }
    w.dbias_at.push_back(dbias_total);
    if (forward) return w;
    const size_t groups = (size_t)g0.groups, B = (size_t)g0.B;
    w.dYa = a.take(groups * B * act_max * g0.esz);
    w.dYb = a.take(groups * B * act_max * g0.esz);
    w.dG_send = g0.q > 0 ? a.take(groups * g0.q * B * k_max * g0.esz) : nullptr;
    w.dg_own = g0.q > 0 ? a.take(groups * B * k_max * g0.esz) : nullptr;
    size_t second = 0;                                 // where the second set starts
    for (int set = 0; set < 2; ++set) {
        second = (a.used + 255) & ~(size_t)255;
        w.dLw[set] = (float *)a.take(groups * lw_max * 4);
        w.dCw[set] = (float *)a.take(groups * cw_max * 4 + 16);
        w.dDw[set] = (float *)a.take(groups * dw_max * 4 + 16);
    }
    const Deferral deferral = deferred_weight_gradients(geos);
    w.arrived_words = cut_tiles(geos);
    w.dbias = (float *)a.take((size_t)(dbias_total + w.arrived_words) * 4);
    w.arrived = w.dbias ? (unsigned *)(w.dbias + dbias_total) : nullptr;
    if (deferral == DEFER_SMALL) {
        size_t slots = 0;
        for (const Geo &g : geos) {
            w.delta_of.push_back(a.take((size_t)g.B * g.so * g.esz));
            if (g.q > 0) slots += (size_t)tiles_of(g.k, g.si) * compressor_gradient_pieces(g);
        }
        w.parts = (float *)a.take(std::max<size_t>(slots, 1) * MT * MT * sizeof(float));
        w.table = (ProductTable *)a.take(sizeof(ProductTable));
    }
    // one partial sum of the loss per output tile of the last layer, at the smallest tile (32 x 32)
    const Geo &gL = geos.back();
    w.mse_partial = (float *)a.take((size_t)((gL.B + 31) / 32) * (size_t)((gL.so + 31) / 32 * g0.groups) * sizeof(float));
    w.bwd.delta = a.take(groups * B * act_max * g0.esz);
    if (deferral == DEFER_LARGE) {
        Arena beside{a.base, second};                  // (the gradients of all layers that nobody wants lie in the first set)
        for (size_t l = 0; l < geos.size(); ++l)
            w.delta_of.push_back(l == 0 ? w.dYa : l == 1 ? w.dYb : l == 2 ? w.bwd.delta : beside.take(B * (size_t)g0.so * g0.esz));
    }
    return w;
}

// ---- one product ---------------------------------------------------------------
inline unsigned blocks_for(int64_t count, int per_block = 256, int cap = 8192)
{
    int64_t b = (count + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

// Does this bf16 problem run on the kernels of gemm_flex.h rather than the 128 x 128 ones?  Widths or phantom widths that
// no 8- or 4-element vector divides always do.  Otherwise where a layer's output has so few 128 x 128 tiles that they leave
// compute units idle: 64 x 64 tiles then spread over four times as many workgroups, and the backward pass has fewer launches.
// Measured (us, 128 x 128 kernels : these; 8-element vectors; p = 8, k = 32 unless stated):
//   forward, 4 layers of 1024 at 128 / 160 / 192 / 256 tiles 66 : 58, 67 : 68, 67 : 90, 90 : 104; of 512 at 128 / 256 53 : 44, 70 : 78;
//   dense 4096 at 128 / 192 162 : 149, 158 : 207;
//   trained, 3 layers of 1024 at 128 tiles (batch 2000) 142 : 134, at 192 159 : 190; of 2048 at 128 241 : 203, at 192 262 : 281; dense 4096
//   at 64 / 128 382 : 293, 398 : 366.  With a batch much longer than the layer is wide the weight gradients have few tiles and a long
//   reduction: 512 wide, batch 3000 / 4096 (96 / 128 tiles) 125 : 124, 135 : 147;
//   a layer's backward call saves two launches more where the tiles are cheap: forward + backward of 1024 at 256 / 384 / 512 tiles 93 : 76,
//   119 : 106, 153 : 135; of 512 at 256 118 : 88; of 2048 at 128 / 192 / 512 78 : 68, 85 : 91, 184 : 197; 64 ranks, 1024 wide, k 64 (reduction
//   5056) at 256 190 : 220;
//   all ranks on the device, whose 128 x 128 launches carry the next layer's error compression and sum the reduce-scatter on read; lines in tiles of
//   64 x 64, of which a compute unit holds three.  A pass with a backward part up to 768: 8 ranks of 256 + 32 at 256 / 512 / 768 tiles (batch 512 /
//   1024 / 1536) 152 : 122, 190 : 167, 216 : 187; of 512 + 32 at 512 / 768 185 : 170, 215 : 200; 16 of 128 + 32 at 768 183 : 174; 32 of 128 + 16 at
//   640 / 768 217 : 212, 234 : 235; 64 of 128 + 8 at 512 / 768 224 : 220, 285 : 286; a layer's backward call of 8 of 512 + 32 at 768 48 : 39.  Less the
//   longer the peers' part is against the shard, which smaller tiles read more often: 32 of 128 + 24 at 768 210 : 226, 16 of 128 + 64 236 : 247,
//   64 of 128 + 16 243 : 269, 64 of 64 + 8 at 384 180 : 162, 32 of 128 + 32 at 512 / 768 190 : 193, 227 : 254; 64 of 64 + 16 at 320 213 : 201, of 128 + 32
//   at 256 / 512 268 : 232, 323 : 335, + 64 at 512 548 : 637.
//   Forward alone up to 768 where the peers' part is at most twice the shard: 4 layers of 8 ranks of 256 + 32 at 512 / 768 59 : 56, 64.4 : 62.4, of 512 + 32 69 :
//   60, 70.8 : 66.9 (with GELU 81 : 72), 2 of 2048 + 32 at 768 140 : 132, 16 of 128 + 16 57.6 : 59.8 (with GELU 67.5 : 65.4); beyond, up to 512: 32 of 128 + 16 at
//   512 / 768 63 : 58, 65.8 : 69.8, 64 of 128 + 8 74.8 : 70, 77 : 87.5.  With more than 32 phantom neurons the compression has two column blocks
//   there, or no kernel of its own: 8 of 256 + 40 at 640 72.5 : 70, 4 of 1024 + 64 at 768 103 : 88, 8 of 512 + 128 107 : 97, 32 of 128 + 64 at 640
//   117 : 115, but 64 of 128 + 48 at 640 164 : 179.
// All of these were measured before the 128 x 128 kernels' loop was rewritten.  With the present one (128 x 128 : these) they are right where tiles are few
// (trained, 3 layers of 1024 at 64 / 96 tiles 109 : 93, 116 : 112; dense 4096 at 64 376 : 348; a layer's calls of 1024 at 128 53 : 44; 8 ranks of 256 + 32 at 256 / 512 / 768
// small tiles 142 : 121, 169 : 164, 191 : 186), and lie too far out near the lines: 3 layers of 1024 trained at 128 123 : 130, of 2048 174 : 192, dense 4096 403 : 458; 4 of
// 1024 forward at 128 53 : 57; 32 ranks of 128 + 16 trained at 768 218 : 233, + 32 at 512 175 : 194, 64 of 128 + 16 at 512 196 : 214; all ranks forward at 768 8 of 256 + 32 58 : 64,
// of 512 + 32 64 : 70, 4 of 1024 + 64 85 : 92, 32 of 128 + 64 at 640 97 : 118; their layer forward calls 15 : 17.5.
// 4-element vectors, which take the renumbering kernel, keep the lines that were measured for it: 96 and 128 tiles, 192 for a layer's call.
bool use_flex(const std::vector<Geo> &geos, bool backward, bool single_call)
{
    int64_t tiles = 0;
    bool wide = true, narrow = true, ring = true, all_fit = true;
    for (const Geo &g : geos) {
        if (g.vec == 0) return true;
        tiles = std::max(tiles, tiles_of(g.B, g.so) * g.groups);
        ring = ring && g.vec == 8;
        wide = wide && g.B <= (ring ? 2 : 1) * g.so;
        narrow = narrow && g.so <= 1024 && g.Kc <= 2048;
        const int64_t peers = g.q * g.k, small = ((g.B + 63) / 64) * ((g.so + 63) / 64) * g.groups;
        all_fit = all_fit && small <= (backward ? (peers <= 4 * g.so ? 768 : peers <= 8 * g.so ? 512 : 384)
                                                : peers <= 2 * g.so || (g.k > 32 && peers <= 16 * g.so) ? 768 : 512);
    }
    static const char *force = tuning_env("PHANTOM_FLEX");
    if (force) return force[0] == '1';
    if (geos[0].all) return ring && all_fit;
    if (single_call && !ring) return tiles <= 192;
    if (single_call) return tiles <= (backward && narrow ? 512 : 128);
    return tiles <= (!backward || wide ? 128 : 96);
}

// How a product is to be run on the 128 x 128 kernels: loader kinds of the two operands and the vector width the
// problem allows.
struct GemmPlan {
    int ka, kb;
    int vec;
};

struct Product {
    View a, b, o;
    Epilogue ep;
    int64_t M, N, K;
    SumOnRead rs;        // the tail block of a (gemm_flex_f32_few_kernel, weight-gradient layout: all of it) is summed on read (src != nullptr; kernels that do it only)
    SgdInPlace sgd;      // weight gradients: the update applied by the epilogue that finishes them (w0 == nullptr: none)
    float *rowsum;       // gemm_flex kernels, weight gradients: receives the bias gradient (MfmaParams has no such thing)
    bool km;             // gemm_flex kernels: weight-gradient layout (both operands along their free index), float out
};

ph_status reserve_lds(LdsReserved &reserved, const void *kernel, int bytes, const char *what)
{
    const hipError_t e = reserved.reserve(kernel, bytes);
    return e == hipSuccess ? PH_OK : fail(PH_ERR_LAUNCH, "%s: cannot reserve %d bytes of LDS: %s", what, bytes, hipGetErrorString(e));
}

template <int KA, int KB, int VEC, typename TOut, bool PAIR, int MODE, int EPI>
ph_status launch_mfma_kernel(const MfmaBatch &batch, hipStream_t st, const char *what)
{
    auto kern = gemm_mfma_kernel<KA, KB, VEC, VEC, TOut, PAIR, MODE, EPI>;
    constexpr int LDS = mfma_lds_bytes(MODE);
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)kern, LDS, what));
    hipLaunchKernelGGL(kern, dim3((unsigned)batch.total_wg), dim3(mfma_threads(MODE)), LDS, st, batch);
    return check_launch(what);
}

template <int KA, int KB, int VEC, typename TOut, int EPI>
ph_status launch_mfma_inst(const MfmaBatch &batch, int mode, hipStream_t st, const char *what)
{
    if constexpr (KB == LD_KM) {
        if (mode == TILE_SOLO) {
            if (batch.count == 2) return launch_mfma_kernel<KA, KB, VEC, TOut, true, TILE_SOLO, EPI>(batch, st, what);
            return launch_mfma_kernel<KA, KB, VEC, TOut, false, TILE_SOLO, EPI>(batch, st, what);
        }
    }
    if (mode == TILE_DUAL) {
        if (batch.count == 2) return launch_mfma_kernel<KA, KB, VEC, TOut, true, TILE_DUAL, EPI>(batch, st, what);
        return launch_mfma_kernel<KA, KB, VEC, TOut, false, TILE_DUAL, EPI>(batch, st, what);
    }
    if (batch.count == 2) return launch_mfma_kernel<KA, KB, VEC, TOut, true, TILE_SHARED, EPI>(batch, st, what);
    return launch_mfma_kernel<KA, KB, VEC, TOut, false, TILE_SHARED, EPI>(batch, st, what);
}

// EPI: the epilogue mode the kernel is built for besides the plain store (see epilogue_from_lds)
template <int KA, int KB, typename TOut, int EPI>
ph_status launch_mfma_vec(const MfmaBatch &batch, int vec, int mode, hipStream_t st, const char *what)
{
    if (vec == 8) return launch_mfma_inst<KA, KB, 8, TOut, EPI>(batch, mode, st, what);
    return launch_mfma_inst<KA, KB, 4, TOut, EPI>(batch, mode, st, what);
}

// Do rows of an operand's head block start off the cache lines of 128 bytes?  (Those that hold less than one: no.)  A step's 128 bytes of a row then lie in two
// lines, each of which the next step needs again, and loads that are spread over a step find the second one gone more often than loads in a burst.
// Us a launch, one by one : in bursts: forward 1000 x 3000 x 3000 35.0 : 33.3, 1500 x 2040 x 2040 26.4 : 24.4, 4000 x 2040 x 2040 42.9 : 42.3, 2000 x 3000 x 3000 53.5 :
// 54.0; the gradients of two layers of 2040 over 4000 rows, two tiles to a workgroup, 81.9 : 77.6, of 2024 over 8000 146.8 : 139.6.
// Not the input gradient (2000 x 3000 x 3000 41.8 : 45.1), nor other gradients (one layer of 3000 over 4000 rows 103 : 111, two in one-tile workgroups 197.6 :
// 200, of 2040 over 1500 40.1 : 39.9).  Rows on lines: 4000 x 4096 x 4096 forward 61 : 64.
bool rows_off_lines(const Product &pr)
{
    static const char *force = tuning_env("PHANTOM_BURSTS");           // =0 / 1 (for measurements)
    if (force) return force[0] == '1';
    auto off = [](const View &v) {
        const int64_t row = std::max(v.r.mult0, v.c.mult0);        // (one of the two is 1)
        return row % 64 != 0 && row >= 64;
    };
    return off(pr.a) || off(pr.b);
}

MfmaParams mfma_params(const Product &pr, int groups, int ksplit, bool dual)
{
    MfmaParams params{};
    MfmaIn &P = params.in;
    P.a = pr.a; P.b = pr.b; P.rs = pr.rs;
    params.out.o = pr.o; params.out.ep = pr.ep; params.out.sgd = pr.sgd;
    P.M = (int)pr.M; P.N = (int)pr.N; P.K = (int)pr.K;
    const int mt = dual ? 2 * MT : MT;               // rows of C per workgroup
    P.tiles_m = (int)((pr.M + mt - 1) / mt);
    P.tiles_n = (int)((pr.N + MT - 1) / MT);
    const int ksteps = (int)((pr.K + KT - 1) / KT);
    const int steps_per = (ksteps + ksplit - 1) / ksplit;
    P.ksplit = (short)((ksteps + steps_per - 1) / steps_per);
    P.bursts = pr.a.c.mult0 == 1 && pr.b.c.mult0 == 1 && rows_off_lines(pr);           // (forward layout)
    P.k_per_split = steps_per * KT;
    P.total_wg = P.tiles_m * P.tiles_n * groups * P.ksplit;
    P.magic_tiles = div_magic(P.tiles_m * P.tiles_n); P.magic_band = div_magic(mfma_raster(dual) * P.tiles_n);
    return params;
}

// More tiles than compute units: two workgroups of one tile each per compute unit (TILE_SOLO), or one of two tiles that
// share their B operand (TILE_DUAL)?  All workgroups of a round are in the same phase, so the memory idles during DUAL's
// loop and the matrix cores during its epilogue; SOLO's overlap, for a third more bytes staged.  It wins where the loop is
// short against the epilogue.  Step times (us, no launch in SOLO : every launch that can be : this rule):
//   weight gradients with the update (10 to 14 bytes of weights per element), reduction 256 to 1536 long: 32 ranks of 1024 at batch
//   256 470 : 400 : 402, 64 ranks of 256 at 512 541 : 510 : 510, 64 ranks of 128 at 1024 808 : 703 : 702, dense 4 x 4096 at 1024
//   589 : 565 : 564 and at 1536 769 : 767 : 755; longer: dense at 2048 863 : 864 : 863, at 4096 1539 : 1568 : 1534;
//   gradients alone: 64 ranks of 256 at 512 449 : 436 : 437, dense at 1024 528 : 495 : 495.  Not caught by it: 8 ranks of 1024 with GELU, gradients
//   at 2048, 871 : 850 : 872.
//   Those are from before the loop was rewritten.  With the present one, no launch in SOLO : every launch that can be : this rule: 32 ranks of 1024 trained at 256
//   368 : 350 : 347, 64 of 128 at 1024 721 : 655 : 656, 64 of 256 at 512 482 : 486 : 486 and its gradients 436 : 436 : 436, at 2048 with GELU 1542 : 1561 : 1517,
//   8 ranks of 1024 with GELU 803 : 808 : 803, 8 of unequal widths 333 : 330 : 330.
// The forward layout lost at 760 already (488 : 498, operands through registers).
template <typename TOut>
bool solo_tiles(const GemmPlan &plan, const Product *prods, int count)
{
    int64_t K = 0;
    for (int i = 0; i < count; ++i) K = std::max(K, prods[i].K);
    static const char *force = tuning_env("PHANTOM_SOLO");         // =0 / 1 (for measurements)
    if (force) return force[0] == '1' && plan.kb == LD_KM;
    if (std::is_same<TOut, float>::value) return K <= 1536;
    return plan.kb == LD_KM && K <= (prods[0].ep.mode == EPI_DACT ? 768 : 256);
}

// bf16 operands on the matrix cores: one product, or two of the same layout side by side in one launch
template <typename TOut>
ph_status launch_mfma(const GemmPlan &plan, const Product *prods, int count, int groups, const MfmaRiders &ride, hipStream_t st, const char *what)
{
    const Product &first = prods[0];
    const int64_t tiles = tiles_of(first.M, first.N) * groups;
    if (tiles * 8 > 0x7fffffff) return fail(PH_ERR_LAUNCH, "%s: internal error, too many tiles (make_geo admits none such)", what);
    // More tiles than compute units: the launch would run in rounds.  Then two tiles, one above the other,
    // go to one workgroup (its teams share the B tile): fewer bytes staged per FLOP and half the rounds.
    // PHANTOM_DUAL=0 / 1 forces the choice (for measurements).
    bool dual = tiles + (count == 2 ? tiles_of(prods[1].M, prods[1].N) * groups : 0) > 256;
    static const char *force = tuning_env("PHANTOM_DUAL");
    if (force) dual = force[0] == '1';
    const int tile_mode = !dual ? TILE_SHARED : solo_tiles<TOut>(plan, prods, count) ? TILE_SOLO : TILE_DUAL;
    dual = tile_mode == TILE_DUAL;
    MfmaBatch batch{};
    batch.count = count;
    batch.p[0] = mfma_params(first, groups, 1, dual);
    batch.total_wg = batch.p[0].in.total_wg;
    batch.first_wg = batch.p[0].in.total_wg;
    batch.ride = ride;
    if (count == 2) {
        batch.p[1] = mfma_params(prods[1], groups, 1, dual);
        batch.total_wg += batch.p[1].in.total_wg;
    }
    const Product &second = prods[count - 1];
    ProfScope prof(what, first.M, first.N, first.K, groups, st, count == 2 ? second.M : 0, count == 2 ? second.N : 0,
                   count == 2 ? second.K : 0);
    // The kernels that exist: the forward layout (both operands read along the reduction index) with the
    // bias + activation epilogue, the input-gradient layout with the sigma' epilogue, each also with the plain
    // store alone, in the storage type; the weight-gradient layout with the plain store in float.  The
    // second product of a pair always stores plainly.
    const int mode = first.ep.mode;
    if (count == 2 && second.ep.mode != EPI_STORE) return fail(PH_ERR_LAUNCH, "%s: internal error, the second product of a pair must store plainly", what);
    if constexpr (std::is_same<TOut, float>::value) {
        if (plan.ka == LD_KM && plan.kb == LD_KM && mode == EPI_STORE)
            return launch_mfma_vec<LD_KM, LD_KM, float, EPI_STORE>(batch, plan.vec, tile_mode, st, what);
    } else {
        if (plan.ka == LD_KC && plan.kb == LD_KC) {
            if (mode == EPI_BIAS_ACT) return launch_mfma_vec<LD_KC, LD_KC, TOut, EPI_BIAS_ACT>(batch, plan.vec, tile_mode, st, what);
            if (mode == EPI_STORE) return launch_mfma_vec<LD_KC, LD_KC, TOut, EPI_STORE>(batch, plan.vec, tile_mode, st, what);
        }
        if (plan.ka == LD_KC && plan.kb == LD_KM) {
            if (mode == EPI_DACT) return launch_mfma_vec<LD_KC, LD_KM, TOut, EPI_DACT>(batch, plan.vec, tile_mode, st, what);
            if (mode == EPI_STORE) return launch_mfma_vec<LD_KC, LD_KM, TOut, EPI_STORE>(batch, plan.vec, tile_mode, st, what);
        }
    }
    return fail(PH_ERR_LAUNCH, "%s: internal error, no kernel for this operand layout, output type and epilogue", what);
}

// The weight + compressor gradients (tail0, tail1; tail1 may be empty) with their riders in one launch: the
// error compression of the layer below (head, may be NULL) and the loss's final sum (loss.partial may be NULL): see
// MfmaTailBatch.
template <int VEC>
ph_status launch_tail_kernel(const MfmaTailBatch &tb, unsigned total_wg, hipStream_t st, const char *what)
{
    auto kern = gemm_mfma_tail_kernel<VEC>;
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)kern, MFMA_LDS_BYTES, what));
    hipLaunchKernelGGL(kern, dim3(total_wg), dim3(MFMA_THREADS), MFMA_LDS_BYTES, st, tb);
    return check_launch(what);
}

ph_status launch_tail(const Product *head, const Product &tail0, const Product &tail1, const LossTail &loss, int groups, int vec, hipStream_t st, const char *what, bool head_last = false)
{
    MfmaTailBatch tb{};
    const bool two = tail1.M > 0 && tail1.N > 0;
    // More tiles than compute units with the head's: in two-tile workgroups if the launch then fits one round
    // (PHANTOM_TAIL_DUAL=0 / 1 forces the choice, for measurements)
    auto wgs = [&](bool dual) {
        int64_t n = (head ? (int64_t)mfma_params(*head, groups, 1, dual).in.total_wg : 0) + mfma_params(tail0, groups, 1, dual).in.total_wg;
        if (two) n += mfma_params(tail1, groups, 1, dual).in.total_wg;
        return n;
    };
    bool dual = head && !head_last && wgs(false) > 256 && wgs(true) <= 256;
    static const char *dual_force = tuning_env("PHANTOM_TAIL_DUAL");
    if (dual_force) dual = dual_force[0] == '1';
    tb.dual = dual;
    if (head) tb.head = mfma_params(*head, groups, 1, dual);
    tb.head_wg = head ? tb.head.in.total_wg : 0;
    tb.tail_first = (tb.head_wg + 7) & ~7;
    tb.tail[0] = mfma_params(tail0, groups, 1, dual);
    tb.tail_wg = tb.tail[0].in.total_wg;
    tb.tail0_wg = tb.tail[0].in.total_wg;
    if (two) {
        tb.tail[1] = mfma_params(tail1, groups, 1, dual);
        tb.tail_wg += tb.tail[1].in.total_wg;
    }
    tb.loss_first = tb.tail_first + tb.tail_wg;
    tb.loss = loss;
    ProfScope prof(what, tail0.M, tail0.N, tail0.K, groups, st, two ? tail1.M : 0, two ? tail1.N : 0, two ? tail1.K : 0,
                   head ? head->M : 0, head ? head->N : 0, head ? head->K : 0);
    const unsigned total = (unsigned)(tb.loss_first + (loss.partial ? 1 : 0));
    tb.rotate = (head && head_last) ? tb.tail_first : 0;
    return vec == 8 ? launch_tail_kernel<8>(tb, total, st, what) : launch_tail_kernel<4>(tb, total, st, what);
}

// The weight-gradient-layout products `prods` (float out, 8-element vectors, one group each; at most TABLE_PRODUCTS)
// in one launch through a parameter table in device memory: see gemm_mfma_table_kernel.  upload_product_table
// fills the table (small launches, any time before); launch_product_table runs the products.
// splits[j] > 1 cuts product j's reduction into pieces (parts, arrived: room for all of them, see MfmaParams);
// A product's sgd.w0 != NULL puts the SGD update into its epilogue.  tail: the launch's first workgroup finishes
// the loss.  *grid: the launch's size.
ph_status upload_product_table(const std::vector<Product> &prods, const std::vector<int> &splits,
                               ProductTable *table, float *parts, unsigned *arrived, const LossTail &tail, hipStream_t st, int *grid)
{
    const char *what = "parameter table";
    if (prods.size() > (size_t)TABLE_PRODUCTS) return fail(PH_ERR_LAUNCH, "%s: internal error, more products than the table holds", what);
    size_t slot = 0, word = 0;
    std::vector<MfmaParams> blocks;
    std::vector<int> first, duals;
    int64_t all_tiles = 0;
    for (const Product &pr : prods) all_tiles += tiles_of(pr.M, pr.N);
    const bool many_tiles = all_tiles > 256;
    int next = 0;
    for (size_t j = 0; j < prods.size(); ++j) {
        const Product &pr = prods[j];
        if (tiles_of(pr.M, pr.N) * 8 > 0x7fffffff) return fail(PH_ERR_LAUNCH, "%s: internal error, too many tiles (make_geo admits none such)", what);
        // with more than 256 tiles in the launch, the uncut products run in two-tile workgroups like a launch of their own
        const bool dual = splits[j] == 1 && many_tiles;
        MfmaParams P = mfma_params(pr, 1, splits[j], dual);
        duals.push_back(dual ? 1 : 0);
        const int64_t tiles = tiles_of(pr.M, pr.N);
        if (P.in.ksplit > 1) {
            P.out.parts = parts + slot * MT * MT; P.out.arrived = arrived + word;
            slot += (size_t)tiles * splits[j]; word += (size_t)tiles;
        }
        first.push_back(next);
        next += (P.in.total_wg + 7) & ~7;
        blocks.push_back(P);
    }
    first.push_back(next);
    const int count = (int)blocks.size();
    for (int at = 0; at < count; at += CHUNK_PRODUCTS) {
        TableChunk c{};
        c.at = at; c.n = std::min(CHUNK_PRODUCTS, count - at); c.count = count; c.tail = tail;
        for (int i = 0; i < c.n; ++i) { c.p[i] = blocks[(size_t)(at + i)]; c.wgs[i] = blocks[(size_t)(at + i)].in.total_wg; c.dual[i] = duals[(size_t)(at + i)]; }
        for (int i = 0; i <= c.n; ++i) c.first_wg[i] = first[(size_t)(at + i)];
        ProfScope prof(what, 0, (int64_t)c.n * (int64_t)(sizeof(MfmaParams) / 4), 0, 1, st);
        hipLaunchKernelGGL(table_upload_kernel, dim3(1), dim3(256), 0, st, c, table);
        PH_TRY(check_launch(what));
    }
    *grid = next;
    return PH_OK;
}

// prof_a, prof_b, prof_groups: the profile entry's two shapes and how many products of each the table holds (exact
// when all layers have the same shapes); HALVES: see gemm_mfma_uniform_kernel
template <bool HALVES>
ph_status launch_product_table(const ProductTable *table, int grid, hipStream_t st, const char *what, const Product &prof_a,
                               const Product &prof_b, int prof_groups)
{
    auto kern = gemm_mfma_table_kernel<8, HALVES>;
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)kern, MFMA_LDS_BYTES, what));
    ProfScope prof(what, prof_a.M, prof_a.N, prof_a.K, prof_groups, st, prof_b.M, prof_b.N, prof_b.K);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(MFMA_THREADS), MFMA_LDS_BYTES, st, table);
    return check_launch(what);
}

template <bool SOLO, bool HALVES>
ph_status launch_uniform_kernel(const UniformGradients &u, const Product &dw, const Product &dc, hipStream_t st, const char *what)
{
    auto kern = gemm_mfma_uniform_kernel<8, SOLO, HALVES>;
    constexpr int MODE = SOLO ? TILE_SOLO : TILE_DUAL, LDS = mfma_lds_bytes(MODE);
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)kern, LDS, what));
    ProfScope prof(what, dw.M, dw.N, dw.K, u.layers, st, dc.M, dc.N, dc.K);
    hipLaunchKernelGGL(kern, dim3((unsigned)(u.layers * (u.dc_wg + u.dw_wg))), dim3(mfma_threads(MODE)), LDS, st, u);
    return check_launch(what);
}

// The same launch for layers of one shape, without a table (dw, dc: by layer; without compressors the dc have no rows).
// More tiles than compute units: one tile to a workgroup, two workgroups to a compute unit (TILE_SOLO), where that takes no more rounds of
// the chip than two tiles to a workgroup, whose compressor gradients are cut and start the launch: there the epilogues of the first
// round run beside the second's loops.  Us a step, two tiles : SOLO: 3 layers of 3072 with GELU trained at batch 1500 367 : 363, 8 of 512 + 960 at 4096 329 : 321 (their
// gradients 325 : 319), 4 of 1024 + 224 at 4096 233 : 228.  A round more: 8 of 1024 + 960 at 4096 (1088 tiles) 622 : 651, at 2560 426 : 439.  Not with whole rounds of two tiles a
// workgroup and long reductions, where loops are most of the time: 2 of 4096 at 3500 / 4096 565 : 587, 614 : 646, 4 of them at 4096 1396 : 1451, 2 and 4 of 2048 183 : 190, 389 : 398.
// The loop with single loads moved the line: up to 3072 rows and with rounds that are not whole, two tiles are now the faster one for dense 4096 (4 layers at 1024 / 2048 482 : 486,
// 747 : 764, two at 3072 525 : 541) and 3 of 2048 + 192 at 2048 / 4096 (242 : 247, 378 : 387), as fast for 4 of 2048 and 6 of 1024 + 448.
ph_status launch_uniform_gradients(const std::vector<Product> &dw, const std::vector<Product> &dc, int pieces, float *parts,
                                   unsigned *arrived, const LossTail &tail, bool halves, hipStream_t st, const char *what)
{
    const int L = (int)dw.size();
    const bool two = dc[0].M > 0;
    UniformGradients u{};
    int64_t tiles = tiles_of(dw[0].M, dw[0].N) * L;
    if (two) tiles += tiles_of(dc[0].M, dc[0].N) * L;
    const int64_t pairs = ((dw[0].M + 2 * MT - 1) / (2 * MT)) * ((dw[0].N + MT - 1) / MT) * L;
    bool solo = tiles > 256 && (tiles + 511) / 512 <= (pairs + 255) / 256 && (dw[0].K <= 3072 || pairs % 256 != 0);
    static const char *force = tuning_env("PHANTOM_UNIFORM_SOLO");         // =0 / 1 (for measurements)
    if (force) solo = force[0] == '1';
    if (solo) pieces = 1;                              // (whole, with sums in levels: gemm_mfma_uniform_kernel)
    u.dw_dual = tiles > 256 && !solo;
    u.dw = mfma_params(dw[0], 1, 1, u.dw_dual);
    u.dw.in.bursts = u.dw_dual && rows_off_lines(dw[0]);
    u.dw_wg = (u.dw.in.total_wg + 7) & ~7;
    if (two) {
        u.dc = mfma_params(dc[0], 1, pieces, false);
        u.dc_wg = (u.dc.in.total_wg + 7) & ~7;
        const int64_t t = tiles_of(dc[0].M, dc[0].N);
        if (u.dc.in.ksplit > 1) {
            u.dc.out.parts = parts; u.dc.out.arrived = arrived;
            u.parts_layer = t * pieces * MT * MT; u.arrived_layer = t;
        }
    }
    u.layers = L;
    u.tail = tail;
    for (int l = 0; l < L; ++l) {
        const Product &w = dw[(size_t)l], &c = dc[(size_t)l];
        u.at[l].in = {w.a.p0, w.b.p0, w.b.p1, c.a.p0};
        u.at[l].out = {w.o.p0, w.o.p1, c.o.p0, w.sgd.master0, w.sgd.master1, c.sgd.master0, w.sgd.bias_master, w.sgd.w0, w.sgd.w1, c.sgd.w0,
                       w.sgd.bias_w, w.sgd.bias_grad};
    }
    if (halves) return solo ? launch_uniform_kernel<true, true>(u, dw[0], dc[0], st, what) : launch_uniform_kernel<false, true>(u, dw[0], dc[0], st, what);
    return solo ? launch_uniform_kernel<true, false>(u, dw[0], dc[0], st, what) : launch_uniform_kernel<false, false>(u, dw[0], dc[0], st, what);
}

// Up to MANY_PRODUCTS products of the forward layout with a plain store, in one launch.
template <int VEC, bool DUAL>
ph_status launch_many_kernel(const MfmaMany &many, hipStream_t st, const char *what)
{
    auto kern = gemm_mfma_many_kernel<VEC, DUAL>;
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)kern, MFMA_LDS_BYTES, what));
    hipLaunchKernelGGL(kern, dim3((unsigned)many.first_wg[many.count]), dim3(MFMA_THREADS), MFMA_LDS_BYTES, st, many);
    return check_launch(what);
}

ph_status launch_many(const std::vector<Product> &prods, int vec, hipStream_t st, const char *what)
{
    for (size_t at = 0; at < prods.size(); at += MANY_PRODUCTS) {
        MfmaMany many{};
        many.count = (int)std::min<size_t>(MANY_PRODUCTS, prods.size() - at);
        int64_t tiles = 0;
        for (int i = 0; i < many.count; ++i) tiles += tiles_of(prods[at + i].M, prods[at + i].N);
        const bool dual = tiles > 256;                 // as for any launch
        for (int i = 0; i < many.count; ++i) {
            many.p[i] = mfma_params(prods[at + i], 1, 1, dual);
            many.first_wg[i + 1] = many.first_wg[i] + ((many.p[i].in.total_wg + 7) & ~7);
        }
        ProfScope prof(what, prods[at].M, prods[at].N, prods[at].K, many.count, st);
        if (vec == 8) PH_TRY(dual ? (launch_many_kernel<8, true>(many, st, what)) : (launch_many_kernel<8, false>(many, st, what)));
        else PH_TRY(dual ? (launch_many_kernel<4, true>(many, st, what)) : (launch_many_kernel<4, false>(many, st, what)));
    }
    return PH_OK;
}

// One rank's thin compression and layer update in one launch: see MfmaFwdBatch.
template <int VEC, bool DUAL, bool FOLD = false>
ph_status launch_fwd_kernel(const MfmaFwdBatch &fb, unsigned total_wg, hipStream_t st, const char *what)
{
    auto kern = gemm_mfma_fwd_kernel<VEC, DUAL, FOLD>;
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)kern, MFMA_LDS_BYTES, what));
    hipLaunchKernelGGL(kern, dim3(total_wg), dim3(MFMA_THREADS), MFMA_LDS_BYTES, st, fb);
    return check_launch(what);
}

ph_status launch_fwd_pair(const Product &update, const Product &compress, int groups, int vec, const ClearList &clear, hipStream_t st,
                          const char *what)
{
    const int64_t tiles = tiles_of(update.M, update.N) * groups;
    if (tiles * 8 > 0x7fffffff) return fail(PH_ERR_LAUNCH, "%s: internal error, too many tiles (make_geo admits none such)", what);
    const bool dual = tiles > 256;                     // as for a launch of the update alone
    MfmaFwdBatch fb{};
    fb.clear = clear;
    fb.update = mfma_params(update, groups, 1, dual);
    fb.X = (const __bf16 *)compress.a.p0; fb.C = (const __bf16 *)compress.b.p0; fb.G = (__bf16 *)compress.o.p0;
    fb.M = (int)compress.M; fb.N = (int)compress.N; fb.K = (int)compress.K;
    fb.x_g = compress.a.g0; fb.c_g = compress.b.g0; fb.o_g = compress.o.g0;
    fb.update_wg = fb.update.in.total_wg;
    fb.wg_per_group = fb.update.in.total_wg / groups;
    fb.thin_rows = (int)(((compress.M + fb.wg_per_group - 1) / fb.wg_per_group + 15) / 16 * 16);
    const unsigned total = (unsigned)fb.update.in.total_wg;
    ProfScope prof(what, update.M, update.N, update.K, groups, st, compress.M, compress.N, compress.K);
    // The compression inside the update's reduction loop (FoldParams): 16-byte vectors, shapes that take the loop's
    // fast path (widths multiples of 64; the phantom width a divisor of 64), and a tile row with at least as many
    // workgroups as the compression has 32 x 32 blocks per 128 rows.
    const int64_t si = compress.K, k = compress.N;
    const int ncb = (int)((k + 31) / 32);
    // One tile per workgroup only: with two tiles per workgroup (more than 256 tiles) the loop has no registers to
    // spare, and the share behind the epilogue measured as fast or faster (6 layers of 1024 + 112 at batch 8192, operands through
    // registers: 0.195 against 0.221 ms).
    if (!dual && vec == 8 && si % KT == 0 && KT % k == 0 && 4 * ncb <= fb.update.in.tiles_n && update.a.c.decides && update.a.c.split == si) {
        fb.fold.C = fb.C; fb.fold.G = fb.G; fb.fold.c_g = fb.c_g; fb.fold.o_g = fb.o_g;
        fb.fold.N = (int)k; fb.fold.K = (int)si; fb.fold.ncb = ncb; fb.fold.nblocks = 4 * ncb;
        return launch_fwd_kernel<8, false, true>(fb, total, st, what);
    }
    if (vec == 8) return dual ? launch_fwd_kernel<8, true>(fb, total, st, what) : launch_fwd_kernel<8, false>(fb, total, st, what);
    return dual ? launch_fwd_kernel<4, true>(fb, total, st, what) : launch_fwd_kernel<4, false>(fb, total, st, what);
}

// Runs one product, or two independent ones of the same kind (names: `what` for the pair, `what_first` / `what_second`
// when they run as launches of their own).  ride: taken along by the first launch.
template <typename TIn, typename TOut>
ph_status launch_products(const GemmPlan &plan, const Product *prods_in, int count_in, int groups, hipStream_t st,
                          const char *what, const char *what_first = nullptr, const char *what_second = nullptr, const MfmaRiders &ride = MfmaRiders{})
{
    Product prods[2];
    const char *names[2];
    int count = 0;
    for (int i = 0; i < count_in; ++i)
        if (prods_in[i].M > 0 && prods_in[i].N > 0) {
            names[count] = i == 0 ? (what_first ? what_first : what) : (what_second ? what_second : what);
            prods[count++] = prods_in[i];
        }
    if (count == 0 || groups <= 0) return PH_OK;
    // Two products share a launch when the launch-time model below says the pair is faster.  A
    // workgroup occupies a whole compute unit, so up to 256 tiles run at once (fixed cost ~8.6 us +
    // 0.5 us per 64 of the reduction length); above that, workgroups take two tiles each (~9.5 us +
    // 0.76 us per 64) and run in rounds of 256.  Separate launches pay ~2.5 us for the extra launch.
    // (Its figures are those of operands through registers; its choices with the ring, us, apart : together : by the model: 8 layers of 1024 + 64 trained
    // at batch 4096 697 : 677 : 676, 3 of 1024 + 256 321 : 344 : 321, gradients of 64 ranks of 256 + 8 at 512 471 : 437 : 431, of 16 of 512 + 32 at
    // 1024 298 : 293 : 298.)
    // PHANTOM_PAIR=0 / 1 forces the choice (for measurements).
    bool pair = count == 2;
    if (pair) {
        auto tiles_of = [&](const Product &pr) { return ((pr.M + MT - 1) / MT) * ((pr.N + MT - 1) / MT) * groups; };
        auto launch_us = [](int64_t tiles, int64_t K) {
            const double steps = (double)((K + KT - 1) / KT);
            if (tiles <= 256) return 8.6 + 0.5 * steps;
            return (double)(((tiles + 1) / 2 + 255) / 256) * (9.5 + 0.76 * steps);
        };
        const int64_t t0 = tiles_of(prods[0]), t1 = tiles_of(prods[1]);
        const double together = launch_us(t0 + t1, std::max(prods[0].K, prods[1].K));
        const double apart = launch_us(t0, prods[0].K) + launch_us(t1, prods[1].K) + 2.5;
        pair = together < apart;
        static const char *force = tuning_env("PHANTOM_PAIR");
        if (force) pair = force[0] == '1';
    }
    if (pair || count == 1) return launch_mfma<TOut>(plan, prods, count, groups, ride, st, count == 2 ? what : names[0]);
    GemmPlan single = plan;
    PH_TRY(launch_mfma<TOut>(single, &prods[0], 1, groups, ride, st, names[0]));
    return launch_mfma<TOut>(single, &prods[1], 1, groups, MfmaRiders{}, st, names[1]);
}

// ---- products of any shape and storage type (gemm_flex.h) ------------------------------------
FlexAxis flex_axis(const Axis &ax, int64_t length, int V)
{
    auto pad = [V](int64_t x) { return (int)((x + V - 1) / V * V); };
    FlexAxis f{};
    f.head = ax.decides ? ax.split : (int)length;
    f.head_pad = pad(f.head);
    f.total = f.head_pad;
    if (ax.decides && length > ax.split) {
        f.seg = ax.seg; f.seg_pad = pad(ax.seg);
        f.magic = (uint32_t)((0x100000000ull + (uint32_t)f.seg_pad - 1) / (uint32_t)f.seg_pad);
        f.total += (int)((length - ax.split) / ax.seg) * f.seg_pad;
    }
    return f;
}

// k, free: the operand's reduction index and free index
FlexOperand flex_operand_of(const View &v, bool km, const FlexAxis &k, const FlexAxis &free, int V)
{
    FlexOperand o{};
    const Axis &strided = km ? v.c : v.r, &contiguous = km ? v.r : v.c;
    o.p0 = v.p0; o.p1 = v.p1; o.g0 = v.g0; o.g1 = v.g1;
    o.ld0 = strided.mult0; o.ld1 = strided.mult1;
    o.seg_stride = contiguous.seg_stride;
    o.skip0 = v.skip0; o.skip_g = v.skip_g;
    // rows times length of the head block and of one segment
    const FlexAxis &c = km ? free : k, &r = km ? k : free;
    auto small = [V](int64_t rows, int64_t len) { return rows * len > 0 && rows * len < V; };
    o.tiny = small(r.head, c.head) || ((c.seg > 0 || r.seg > 0) && small(r.seg > 0 ? r.seg : r.head, c.seg > 0 ? c.seg : c.head));
    return o;
}

// Tile of a launch, by how many tiles of 64 x 64 it has.  More than one per compute unit: 64 x 64 with one team of four
// wavefronts, several workgroups per unit.  Fewer: two teams that share the reduction (a lone workgroup otherwise spends
// half of a step waiting).  Very few: 32 x 32 and eight teams of one wavefront.  Measured with each tile throughout (us,
// 64 x 64 one team : two : 32 x 32): forward and backward call of 1024 wide at batch 1024 37 : 44 : 110, 3 layers of 512 trained at
// batch 1000 88 : 76 : 153, 6 layers of 1024 forward at batch 512 84 : 74 : 117 and at batch 48 80 : 70 : 48.
// 8-element vectors, whose 64 x 64 tiles run on the ring, take 32 x 32 ones where they fit one round of workgroups and the reduction is so long that
// eight teams gain more than the renumbering costs: 960 forward, or 512, which eight teams have in one whole step each (ring : 32 x 32; 6 layers): dense
// 384 / 512 / 640 / 896 / 960 / 1024 wide at batch 64 35.4 : 39.3, 38.2 : 31.4, 41.3 : 47.9, 45.5 : 46.6, 47 : 46.1, 48 : 39.9, 512 at batch 512 39 : 32.6; 512 + 448
// at 64 47.3 : 45.7, 1024 + 448 at 192 57 : 51, at 256 57 : 79, 2048 + 448 at 64 / 128 52 : 40, 52 : 64; all 8 ranks of 512 + 32 (the compression) at 512 66 : 61.
// Backward, where the launch ends with its weight gradients, beyond 768 and at most 96 tiles of 32 x 32 (3 layers trained): dense 64 wide at batch
// 512 / 1024 / 2048 / 8192 41.7 : 42.7, 49 : 49.5, 64.2 : 59.7, 156 : 118, 256 wide at 1024 / 4096 52.4 : 52.6, 100 : 85 (at most 24 tiles of 64 x 64: 101), 512 + 56 at
// 8192 168 : 150; 128 + 16 at batch 64, whatever its tiles, 56 : 74.  Eight teams are eight partial sums, two of the ring's four: error of the weight
// gradients against 64 bits (2-norm), dense 256 at 256 / 768 / 1000 / 4096 rows 4.7e-8 : 4.9e-8, 6.7e-8 : 6.9e-8, 7.2e-8 : 6.7e-8, 1.0e-7 : 7.3e-8.
// fp32 adds its terms in the order of the reduction index (gemm_flex.h) and so has one team, except where eight teams
// take one group of 16 terms each, the first level of its sums.
enum FlexTile { FLEX_64, FLEX_64_2, FLEX_32_8 };
constexpr int FLEX_FEW = 24;      // bf16 without the ring: up to so many tiles of 64 x 64 run as 32 x 32 ones with eight teams

template <typename T>
FlexTile flex_tile_for(const Product *prods, int count, int groups, bool forward, bool ring)
{
    int64_t tiles = 0, small = 0, longest = 0;         // of 64 x 64, of 32 x 32
    for (int i = 0; i < count; ++i) {
        tiles += ((prods[i].M + 63) / 64) * ((prods[i].N + 63) / 64) * groups;
        small += ((prods[i].M + 31) / 32) * ((prods[i].N + 31) / 32) * groups;
        const int64_t pad = prods[i].km ? 0 : ((prods[i].K - prods[i].a.c.split) / std::max(prods[i].a.c.seg, 1) + 1) * (FlexType<T>::V - 1);
        longest = std::max(longest, prods[i].K + (prods[i].a.c.decides && !ring ? pad : 0));      // (at most; the numbering pads pieces to vectors)
    }
    static const char *force = tuning_env("PHANTOM_FLEX_TILE");
    const int forced = force ? atoi(force) : -1;
    if (forced >= FLEX_64 && forced <= FLEX_32_8 && !(sizeof(T) == 4 && forced == FLEX_64_2)) return (FlexTile)forced;      // (fp32 has no kernel with two teams)
    if (sizeof(T) == 4) return tiles <= 128 && longest <= 8 * 16 ? FLEX_32_8 : FLEX_64;
    const bool few = !ring ? tiles <= FLEX_FEW : forward ? small <= 256 && (longest >= 960 || longest == 8 * 64) : small <= 96 && longest > 768;
    return tiles > 256 ? FLEX_64 : few ? FLEX_32_8 : FLEX_64_2;
}

template <typename T, int TM, int TN, int TEAMS, bool FORWARD, bool FINE>
ph_status launch_flex_kernel(const FlexBatch &batch, unsigned total_wg, hipStream_t st, const char *what)
{
    auto kern = gemm_flex_kernel<T, TM, TN, TEAMS, FORWARD, FINE>;
    constexpr int LDS = FORWARD ? flex_lds_bytes<T, TM, TN, TEAMS, FLEX_KC, FLEX_KC>()
                                : flex_max(flex_lds_bytes<T, TM, TN, TEAMS, FLEX_KC, FLEX_KM>(), flex_lds_bytes<T, TM, TN, TEAMS, FLEX_KM, FLEX_KM>());
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)kern, LDS, what));
    hipLaunchKernelGGL(kern, dim3(total_wg), dim3(FlexShape<T, TM, TN, TEAMS, FINE>::THREADS), LDS, st, batch);
    return check_launch(what);
}

template <bool FORWARD, bool MANY>
ph_status launch_flex_f32(const FlexBatch &batch, unsigned total_wg, hipStream_t st, const char *what)
{
    constexpr int LDS = F32_LDS_BYTES;
    static_assert(4 * LDS <= 160 * 1024, "four workgroups share a compute unit");
    hipLaunchKernelGGL((gemm_flex_f32_kernel<FORWARD, MANY>), dim3(total_wg), dim3(256), LDS, st, batch);
    return check_launch(what);
}

template <bool FORWARD, int GROUPS>
ph_status launch_flex_f32_few(const FlexBatch &batch, unsigned total_wg, hipStream_t st, const char *what)
{
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)(gemm_flex_f32_few_kernel<FORWARD, GROUPS>), f32_few_lds(GROUPS), what));
    hipLaunchKernelGGL((gemm_flex_f32_few_kernel<FORWARD, GROUPS>), dim3(total_wg), dim3(512), f32_few_lds(GROUPS), st, batch);
    return check_launch(what);
}

template <typename T, bool FORWARD, bool FINE>
ph_status launch_flex_tile(const FlexBatch &batch, FlexTile tile, unsigned total_wg, hipStream_t st, const char *what)
{
    if (tile == FLEX_64) return launch_flex_kernel<T, 64, 64, 1, FORWARD, FINE>(batch, total_wg, st, what);
    if constexpr (sizeof(T) == 2)
        if (tile == FLEX_64_2) return launch_flex_kernel<T, 64, 64, 2, FORWARD, FINE>(batch, total_wg, st, what);
    return launch_flex_kernel<T, 32, 32, 8, FORWARD, FINE>(batch, total_wg, st, what);
}

template <int TEAMS, int RING, bool FORWARD>
ph_status launch_flex_ring(const FlexBatch &batch, unsigned total_wg, hipStream_t st, const char *what)
{
    auto kern = gemm_flex_ring_kernel<TEAMS, RING, FORWARD>;
    constexpr int LDS = flex_ring_lds<TEAMS, RING>();
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)kern, LDS, what));
    hipLaunchKernelGGL(kern, dim3(total_wg), dim3(TEAMS * 256), LDS, st, batch);
    return check_launch(what);
}

// The groups of 16 terms of an fp32 launch on gemm_flex_f32_few_kernel, or 0 (f32_few_groups_for).  Empty products count for nothing.
int f32_few_groups(const Product *prods, int count, const Geo &g)
{
    if (g.dtype != PH_F32 || !g.whole) return 0;
    int64_t small = 0, longest = 0;
    for (int i = 0; i < count; ++i) {
        if (prods[i].M <= 0 || prods[i].N <= 0) continue;
        small += ((prods[i].M + 31) / 32) * ((prods[i].N + 31) / 32) * g.groups;
        longest = std::max(longest, prods[i].K);
    }
    const int groups = f32_few_groups_for(small, longest);
    static const char *force[] = {tuning_env("PHANTOM_F32_FEW1"), tuning_env("PHANTOM_F32_FEW2"), tuning_env("PHANTOM_F32_FEW4")};     // workgroups, at most (for measurements)
    if (const char *most = force[f32_few_groups_for(0, longest) / 2]) return small <= atoi(most) ? f32_few_groups_for(0, longest) : 0;
    return groups;
}

// Up to FLEX_MAX_PRODUCTS independent products in one launch.  forward: all in the forward layout; else any mix of the
// input-gradient and the weight-gradient (Product::km) layout.  Empty products are left out.  tail: finished by the
// launch's first workgroup.
// mse_tiles: receives the number of tiles of the first product (one partial sum of the loss each).
template <typename T>
ph_status launch_flex(const Product *prods_in, int count_in, bool forward, const Geo &g, const LossTail &tail, hipStream_t st,
                      const char *what, int *mse_tiles = nullptr)
{
    Product prods[FLEX_MAX_PRODUCTS];
    int count = 0;
    for (int i = 0; i < count_in; ++i)
        if (prods_in[i].M > 0 && prods_in[i].N > 0) prods[count++] = prods_in[i];
    const int groups = g.groups;
    if (count == 0 || groups <= 0) return PH_OK;
    const int few = f32_few_groups(prods, count, g);
    const FlexTile tile = few > 0 ? FLEX_32_8 : flex_tile_for<T>(prods, count, groups, forward, g.vec == 8);
    const int t = tile == FLEX_32_8 ? 32 : 64;
    constexpr int V = FlexType<T>::V;
    FlexBatch batch{};
    batch.count = count;
    batch.tail = tail;
    int next = 0;
    for (int i = 0; i < count; ++i) {
        const Product &pr = prods[i];
        FlexIn &P = batch.p[i].in;
        FlexOut &Q = batch.p[i].out;
        P.kind = pr.km ? 1 : 0;
        Q.o0 = pr.o.p0; Q.o1 = pr.o.p1; Q.o_g0 = pr.o.g0; Q.o_g1 = pr.o.g1;
        Q.o_ld0 = pr.o.r.mult0; Q.o_ld1 = pr.o.r.mult1; Q.o_seg_stride = pr.o.c.seg_stride;
        Q.ep = pr.ep; Q.sgd = pr.sgd; Q.rowsum = pr.rowsum; P.rowsum = pr.rowsum != nullptr;
        P.k = flex_axis(pr.km ? Axis{} : pr.a.c, pr.K, V);
        P.n = flex_axis(pr.o.c, pr.N, V);
        P.M = (int)pr.M;
        P.rs = pr.rs;
        FlexAxis rows{};
        rows.head = P.M;
        P.a = flex_operand_of(pr.a, pr.km, P.k, rows, V);
        P.b = flex_operand_of(pr.b, !forward, P.k, P.n, V);
        P.tiles_m = (int)((pr.M + t - 1) / t);
        P.tiles_n = (P.n.total + t - 1) / t;
        P.total_wg = P.tiles_m * P.tiles_n * groups;
        P.magic_tiles = div_magic(P.tiles_m * P.tiles_n); P.magic_band = div_magic(FLEX_RASTER * P.tiles_n);
        P.magic_last = div_magic(P.tiles_m % FLEX_RASTER);
        if (i == 0 && mse_tiles) *mse_tiles = P.total_wg;
        batch.first_wg[i] = next;
        next += (P.total_wg + 7) & ~7;
    }
    auto dim = [&](int i, int64_t Product::*d) { return i < count ? prods[i].*d : (int64_t)0; };
    ProfScope prof(what, prods[0].M, prods[0].N, prods[0].K, groups, st, dim(1, &Product::M), dim(1, &Product::N), dim(1, &Product::K),
                   dim(2, &Product::M), dim(2, &Product::N), dim(2, &Product::K), dim(3, &Product::M), dim(3, &Product::N), dim(3, &Product::K));
    const unsigned total = (unsigned)next;
    // Sums of up to 128 terms per team need no levels (300 rows, two teams: 7.1e-8 with one running sum, 7.5e-8 in levels)
    const int teams = tile == FLEX_64 ? 1 : tile == FLEX_64_2 ? 2 : 8;
    bool fine = g.fine && prods[0].ep.mode == EPI_BIAS_ACT && prods[0].ep.act == ACT_GELU;
    for (int i = 0; i < count; ++i) fine = fine || (g.fine && prods[i].K > 128 * teams);
    if constexpr (sizeof(T) == 2)
        if (g.vec == 8 && tile != FLEX_32_8) {
            // Two teams also where few tiles have a long reduction and hold up the rest (us, one team : two): one rank's layer of 64, 256 + 32
            // tiles (1520 and 512 long) forward 14.8 : 13.7, 200 + 768 tiles (2048 and 512) backward 24.4 : 21.2.  Otherwise one team: layers
            // of 2048 trained at batch 1000 203 : 224; 4 layers of 1024 forward at batch 2048 60.1 : 70.0.
            int64_t longest = 0, tiles = 0;
            for (int i = 0; i < count; ++i) longest = std::max(longest, prods[i].K);
            for (int i = 0; i < count; ++i)
                if (2 * prods[i].K >= longest) tiles += batch.p[i].in.total_wg;
            static const char *force = tuning_env("PHANTOM_FLEX_RING");
            // Four stages per team, one workgroup per compute unit, while none gets a second; else two stages (one rank's layer of 1720, 1160
            // workgroups backward: 31.9 us; 36 with four stages in common, 33.4 the kernel without the ring).
            if (force ? force[0] == '2' : tile == FLEX_64_2 || tiles <= 256) {
                if (total <= 256) return forward ? launch_flex_ring<2, 4, true>(batch, total, st, what) : launch_flex_ring<2, 4, false>(batch, total, st, what);
                return forward ? launch_flex_ring<2, 2, true>(batch, total, st, what) : launch_flex_ring<2, 2, false>(batch, total, st, what);
            }
            return forward ? launch_flex_ring<1, 3, true>(batch, total, st, what) : launch_flex_ring<1, 3, false>(batch, total, st, what);
        }
    if constexpr (sizeof(T) == 4)
        if (few > 0) {
            if (few == 1) return forward ? launch_flex_f32_few<true, 1>(batch, total, st, what) : launch_flex_f32_few<false, 1>(batch, total, st, what);
            if (few == 2) return forward ? launch_flex_f32_few<true, 2>(batch, total, st, what) : launch_flex_f32_few<false, 2>(batch, total, st, what);
            return forward ? launch_flex_f32_few<true, 4>(batch, total, st, what) : launch_flex_f32_few<false, 4>(batch, total, st, what);
        }
    if constexpr (sizeof(T) == 4)
        if (tile == FLEX_64 && g.whole) {
            // Up to two workgroups to a compute unit the launch waits for loads and operand reads, not for the matrix pipe (us a step of this kernel with
            // neither far ahead : so): 3 layers of 4 ranks of 256 + 8 trained at batch 1024, 256 to 384 workgroups, 251 : 218, of 4 of 400 + 20 at 700 302 : 277.
            static const char *force = tuning_env("PHANTOM_F32_MANY");     // =0 / 1 (for measurements)
            if (force ? force[0] == '1' : total > 512) return forward ? launch_flex_f32<true, true>(batch, total, st, what) : launch_flex_f32<false, true>(batch, total, st, what);
            return forward ? launch_flex_f32<true, false>(batch, total, st, what) : launch_flex_f32<false, false>(batch, total, st, what);
        }
    if constexpr (sizeof(T) == 2)
        if (fine) return forward ? launch_flex_tile<T, true, true>(batch, tile, total, st, what) : launch_flex_tile<T, false, true>(batch, tile, total, st, what);
    return forward ? launch_flex_tile<T, true, false>(batch, tile, total, st, what) : launch_flex_tile<T, false, false>(batch, tile, total, st, what);
}

// The compressions of several layers of one rank in one launch (compress_many_kernel).
ph_status launch_compressions(const std::vector<Product> &prods, hipStream_t st, const char *what)
{
    for (size_t at = 0; at < prods.size(); at += COMPRESS_LAYERS) {
        CompressMany many{};
        many.count = (int)std::min<size_t>(COMPRESS_LAYERS, prods.size() - at);
        for (int i = 0; i < many.count; ++i) {
            const Product &pr = prods[at + i];
            const int tiles = (int)((pr.M + FLEX_RING_TILE - 1) / FLEX_RING_TILE);
            many.at[i] = {pr.a.p0, pr.b.p0, pr.o.p0, (int)pr.M, (int)pr.N, (int)pr.K, div_magic(tiles), div_magic(tiles % FLEX_RASTER)};
            many.first_wg[i + 1] = many.first_wg[i] + ((tiles + 7) & ~7);
        }
        ProfScope prof(what, prods[at].M, prods[at].N, prods[at].K, many.count, st);
        hipLaunchKernelGGL(compress_many_kernel, dim3((unsigned)many.first_wg[many.count]), dim3(256), (flex_ring_lds<1, 3>()), st, many);
        PH_TRY(check_launch(what));
    }
    return PH_OK;
}

Epilogue epi_store()
{
    Epilogue e{};
    e.mode = EPI_STORE;
    return e;
}

// ---- forward of one layer (Eq. (ylq)) ------------------------------------------------
struct FwdArgs {
    const void *X, *Lw, *Cw, *Dw, *bias, *G;
    void *Y, *g_own, *A_save;
    bool apart;   // one rank, layer call: g_own lies over G, so the compression waits for the update, which reads G
    bool a_f32;   // step only: A_save is float
    bool a_deriv; // step only: A_save receives sigma'(A), in float, instead of A
    bool a_bits;  // step only, ReLU: A_save receives one bit per element (stored output > 0)
    const struct OutputError *mse;   // step only, last layer: form the MSE output error in the update's epilogue
    ClearList *clear;                // step only: buffers to clear; a launch that can do it on its way empties the list
    std::vector<Product> *later;     // step only, one rank: takes a compression that would leave compute units idle (launch_many, or
                                     //   launch_compressions where it is thin)
};

// What the last layer's update needs to leave the output error of the MSE loss behind (Epilogue::mse_*).
struct OutputError {
    const void *target;      // [groups, B, s] storage type
    void *delta;             // [groups, B, s] storage type
    float *partial;          // one partial sum of squares per tile of the update
    float inv_b;
    float *dbias;            // [groups, s], receives the column sums of delta (zero on entry)
};

// A list of buffers to clear, in a launch of its own.
ph_status launch_clear(ClearList &list, hipStream_t st)
{
    if (list.count == 0) return PH_OK;
    int64_t n = 0;
    for (int i = 0; i < list.count; ++i) n += list.n[i];
    ProfScope prof("clear bias gradients", 0, n, 0, 1, st);
    hipLaunchKernelGGL(clear_kernel, dim3(blocks_for(n)), dim3(256), 0, st, list);
    list = ClearList{};
    return check_launch("clear bias gradients");
}

// The products of a layer's forward pass (Eq. (ylq)).
struct FwdProducts {
    Product update, compress;
};

FwdProducts make_fwd_products(const Geo &g, const FwdArgs &f)
{
    const int64_t B = g.B, si = g.si, so = g.so, k = g.k, q = g.q;
    FwdProducts pr{};
    // compression g = C y: [B, si] x [k, si]^T -> [B, k]
    pr.compress = Product{view_plain(f.X, si, B * si), view_plain(f.Cw, si, k * si), view_plain(f.g_own, k, B * k), epi_store(),
                          q > 0 ? B : 0, k, si};
    // local update + decompression + remote update + bias + activation: one product over the
    // concatenated reduction index [y | g_1 .. g_{p-1}] . [L | D_1 .. D_{p-1}]^T
    const void *gathered = g.all ? f.g_own : f.G;
    Product &update = pr.update;
    update.a = q > 0 ? view_rowseg(f.X, si, (int)si, B * si, gathered, (int)k, B * k, 0, g.all ? 0 : NO_SKIP, g.all ? 1 : 0)
                     : view_plain(f.X, si, B * si);
    update.b = q > 0 ? view_rowseg(f.Lw, si, (int)si, so * si, f.Dw, (int)k, so * k, q * so * k) : view_plain(f.Lw, si, so * si);
    update.o = view_plain(f.Y, so, B * so);
    update.ep.mode = EPI_BIAS_ACT; update.ep.act = g.act; update.ep.bias = f.bias; update.ep.bias_g = so;
    update.ep.aux = f.A_save; update.ep.aux_ld = so; update.ep.aux_g = B * so; update.ep.aux_f32 = f.a_f32; update.ep.aux_deriv = f.a_deriv; update.ep.aux_bits = f.a_bits;
    update.M = B; update.N = so; update.K = g.Kc;
    if (f.mse) {
        update.ep.mse_target = f.mse->target; update.ep.mse_delta = f.mse->delta; update.ep.mse_partial = f.mse->partial;
        update.ep.mse_inv_b = f.mse->inv_b;
        update.ep.colsum = f.mse->dbias; update.ep.colsum_g = so;
    }
    return pr;
}

// Blocks of 16 rows to a workgroup of a layer's forward pass on the kernel for few rows (few_rows.h), or 0 (few_rows_blocks_for).
int few_rows_blocks(const Geo &g, const FwdArgs &f)
{
    if (g.all || g.vec != 8 || f.apart || f.mse || f.a_bits) return 0;
    static const char *force = tuning_env("PHANTOM_FEW");              // =0, 1, 2 or 4 (for measurements)
    if (force) return atoi(force);
    return few_rows_blocks_for(g.B, g.so, g.k, g.Kc);
}

template <int ROWS, int TEAMS>
ph_status launch_few_rows_kernel(const FewBatch &batch, unsigned total_wg, hipStream_t st, const char *what)
{
    constexpr int MOST = few_lds_bytes(ROWS, TEAMS, (FEW_SHORT + 31) / 32);
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)(few_rows_kernel<ROWS, TEAMS>), MOST, what));
    hipLaunchKernelGGL((few_rows_kernel<ROWS, TEAMS>), dim3(total_wg), dim3(FEW_WAVES * 64), few_lds_bytes(ROWS, TEAMS, batch.chunks), st, batch);
    return check_launch(what);
}

// teams: those of the tiles of gemm_flex.h that these products would have
ph_status launch_few_rows(const Geo &g, const FwdProducts &pr, int blocks, int teams, hipStream_t st)
{
    FewBatch batch{};
    int next = 0;
    for (const Product *p : {&pr.update, &pr.compress}) {
        if (p->M == 0 || p->N == 0) continue;
        FewProduct &P = batch.p[batch.count];
        const bool cut = p->a.c.decides;
        P.a0 = (const __bf16 *)p->a.p0; P.a1 = (const __bf16 *)p->a.p1; P.b0 = (const __bf16 *)p->b.p0; P.b1 = (const __bf16 *)p->b.p1;
        P.out = p->o.p0; P.M = (int)p->M; P.N = (int)p->N; P.K = (int)p->K;
        P.split = (int)g.si; P.seg = cut ? p->a.c.seg : 8; P.magic = div_magic(P.seg);
        P.a_seg = (int)p->a.c.seg_stride; P.b_seg = (int)p->b.c.seg_stride;
        if (p->ep.mode == EPI_BIAS_ACT) {
            P.bias = (const __bf16 *)p->ep.bias; P.act = p->ep.act;
            P.aux = p->ep.aux; P.aux_f32 = p->ep.aux_f32; P.aux_deriv = p->ep.aux_deriv;
        }
        P.tiles_n = (P.N + FEW_TILE - 1) / FEW_TILE; P.pitch = (P.tiles_n + 7) & ~7;
        if (batch.count == 1) batch.first_wg = next;
        batch.chunks = std::max(batch.chunks, (P.K + 31) / 32);
        next += (P.M + blocks * FEW_TILE - 1) / (blocks * FEW_TILE) * P.pitch;
        ++batch.count;
    }
    const char *what = batch.count == 2 ? "layer update + compression" : "layer update";
    ProfScope prof(what, pr.update.M, pr.update.N, pr.update.K, 1, st, pr.compress.M, pr.compress.N, pr.compress.K);
    const unsigned total = (unsigned)next;
    if (teams == 8)
        return blocks == 1 ? launch_few_rows_kernel<1, 8>(batch, total, st, what) : blocks == 2 ? launch_few_rows_kernel<2, 8>(batch, total, st, what)
                           : launch_few_rows_kernel<4, 8>(batch, total, st, what);
    return blocks == 1 ? launch_few_rows_kernel<1, 2>(batch, total, st, what) : blocks == 2 ? launch_few_rows_kernel<2, 2>(batch, total, st, what)
                       : launch_few_rows_kernel<4, 2>(batch, total, st, what);
}

// Forward through gemm_flex.h.  mse_tiles: with f.mse, the number of partial sums of the loss it leaves.
template <typename T>
ph_status flex_fwd(const Geo &g, const FwdArgs &f, hipStream_t st, int *mse_tiles = nullptr)
{
    const FwdProducts pr = make_fwd_products(g, f);
    if (g.all) {
        // every rank reads the other ranks' g: the compression of all ranks has to finish first
        PH_TRY((launch_flex<T>(&pr.compress, 1, true, g, LossTail{}, st, "compression")));
        return launch_flex<T>(&pr.update, 1, true, g, LossTail{}, st, "layer update", mse_tiles);
    }
    const Product both[2] = {pr.update, pr.compress};
    if constexpr (sizeof(T) == 2)
        if (const int blocks = few_rows_blocks(g, f)) {
            // (a dense layer has no compression: its product has no rows)
            const FlexTile tile = flex_tile_for<T>(both, 2, 1, true, true);
            if (tile == FLEX_32_8 || (tile == FLEX_64_2 && g.Kc < FEW_SHORT)) return launch_few_rows(g, pr, blocks, tile == FLEX_32_8 ? 8 : 2, st);
        }
    if (f.apart) {
        PH_TRY((launch_flex<T>(&pr.update, 1, true, g, LossTail{}, st, "layer update")));
        return launch_flex<T>(&pr.compress, 1, true, g, LossTail{}, st, "compression");
    }
    return launch_flex<T>(both, 2, true, g, LossTail{}, st, g.q > 0 ? "layer update + compression" : "layer update", mse_tiles);
}

template <int NF>
ph_status launch_thin_product(dim3 grid, const FwdArgs &f, int64_t B, int64_t k, int64_t si, const ClearList &clear, hipStream_t st)
{
    static LdsReserved reserved;
    PH_TRY(reserve_lds(reserved, (const void *)(thin_product_kernel<NF>), THIN_WAVES * thin_region(NF, NF == 4 ? 3 : THIN_AHEAD), "compression"));
    // all chunks of 32 that a wavefront may have, up to four (three of 64 phantom neurons: 144 KB of LDS)
    const int most = NF == 4 ? 3 : THIN_AHEAD, ahead = (int)std::max<int64_t>(1, std::min<int64_t>(most, (si / 16 + 2 * THIN_WAVES - 1) / (2 * THIN_WAVES)));
    hipLaunchKernelGGL(thin_product_kernel<NF>, grid, dim3(THIN_WAVES * 64), THIN_WAVES * thin_region(NF, ahead), st, (const __bf16 *)f.X, (const __bf16 *)f.Cw,
                       (__bf16 *)f.g_own, (int)B, (int)k, (int)si, B * si, k * si, B * k, ahead, clear);
    return check_launch("compression");
}

ph_status fwd_impl(const Geo &g, const FwdArgs &f, hipStream_t st)
{
    typedef bf16_t T;
    const int64_t B = g.B, si = g.si, so = g.so, k = g.k, q = g.q;
    const GemmPlan plan{LD_KC, LD_KC, g.vec};
    FwdProducts prods = make_fwd_products(g, f);
    const Product &update = prods.update, &compress = prods.compress;
    auto take_clear = [&]() {
        ClearList c{};
        if (f.clear) std::swap(c, *f.clear);
        return c;
    };
    // A compression with few phantom neurons has a kernel of its own (32 rows per workgroup instead of 128)
    const bool thin = q > 0 && k <= THIN_MAX_N && si % 16 == 0 && g.vec > 0;
    auto launch_thin = [&]() -> ph_status {
        ProfScope prof("compression", B, k, si, g.groups, st);
        dim3 grid((unsigned)((B + THIN_ROWS - 1) / THIN_ROWS), (unsigned)g.groups);
        if (k <= 16) return launch_thin_product<1>(grid, f, B, k, si, take_clear(), st);
        return k <= 32 ? launch_thin_product<2>(grid, f, B, k, si, take_clear(), st) : launch_thin_product<4>(grid, f, B, k, si, take_clear(), st);
    };
    // (this layer's update adds into the buffers itself if it is the last one)
    if (f.clear && f.mse && !(g.all && thin)) PH_TRY(launch_clear(*f.clear, st));
    if (g.all) {
        // every rank reads the other ranks' g: the compression of all ranks has to finish first
        if (thin) PH_TRY(launch_thin());
        else PH_TRY((launch_products<T, T>(plan, &compress, 1, g.groups, st, "compression")));
        return launch_products<T, T>(plan, &update, 1, g.groups, st, "layer update");
    }
    if (f.apart) {
        PH_TRY((launch_products<T, T>(plan, &update, 1, g.groups, st, "layer update")));
        return thin ? launch_thin() : launch_products<T, T>(plan, &compress, 1, g.groups, st, "compression");
    }
    // one rank: the peers' g are inputs, so the rank's own compression runs beside the update when the two
    // fit the device together
    const int64_t tiles_both = (tiles_of(B, so) + tiles_of(B, k)) * g.groups;
    const auto riders = [&]() { MfmaRiders r{}; r.clear = take_clear(); return r; };
    if (thin && tiles_both > 256) {
        static const char *force = tuning_env("PHANTOM_FWD_PAIR");         // =0: with the update (for measurements)
        if (f.later && g.vec == 8 && !(force && force[0] == '0')) {
            f.later->push_back(compress);
            return launch_products<T, T>(plan, &update, 1, g.groups, st, "layer update", nullptr, nullptr, riders());
        }
        return launch_fwd_pair(update, compress, g.groups, g.vec, take_clear(), st, "layer update + thin compression");
    }
    if (f.later && q > 0 && k > THIN_MAX_N) {
        f.later->push_back(compress);
        return launch_products<T, T>(plan, &update, 1, g.groups, st, "layer update", nullptr, nullptr, riders());
    }
    Product both[2] = {update, compress};
    return launch_products<T, T>(plan, both, 2, g.groups, st, "layer update + compression", "layer update", "compression", riders());
}

// ---- backward of one layer (Eq. (deltaL), (backprop), (bpb)-(bpD)) ---------------------------
struct BwdArgs {
    const void *dY, *X, *S, *Lw, *Cw, *Dw, *G;
    void *dg_own;
    void *dX;
    float *dLw, *dCw, *dDw, *dbias;
    void *dG_send;
    const void *delta_ready;   // step only: delta already formed (dY, S unused)
    bool dx_S_f32;             // step only: dx_S holds float
    bool dx_S_deriv;           // step only: dx_S holds sigma' itself, in float
    bool dx_S_bits;            // step only, ReLU: dx_S holds one bit per element (the layer below's stored output > 0)
    const void *dx_S;          // step only: multiply dX by sigma'(dx_S) on the way out, which makes it the
                               //   previous layer's delta with a single rounding (Eq. (backprop))
    float *dx_colsum;          // step only: zeroed [groups, s]; the input-gradient product adds the column sums
                               //   of what it stores, i.e. the layer below's bias gradient (Eq. (bpb))
    bool dbias_ready;          // step only: dbias already holds the column sums of delta
    bool send_done;            // step only: this layer's error compression was launched by the layer above (below)
    const void *below_Dw;      // step only, all ranks: D of the layer below; its error compression (dX -> dG_send)
    const Geo *below_g;        //   (that layer's shapes)
    bool *below_done;          //   may then ride with this layer's weight gradients; *below_done says whether it did
    SgdInPlace sgd_w, sgd_c;   // step only: the update of L, D, the bias / of C in the epilogues that finish their gradients
    LossTail *loss_tail;       // step only, last layer: the first memory-bound kernel of this backward finishes
                               //   the loss as a rider and clears loss_tail->partial; left alone if there is none
    void *tap_dG_send;         // step only, optional: copies of this layer's dG_send / (all ranks) dg_own, taken right
    void *tap_dg_own;          //   after the launch that finishes each
    bool defer;                // step only: the weight + compressor gradients are not launched here (the step runs all
                               //   layers' in one launch at the end of the backward pass)
};

// copy of a tensor (count elements of the storage type), for a tap of the step or an output that lies over an input
template <typename T>
ph_status tap_copy(void *dst, const void *src, int64_t count, hipStream_t st)
{
    if (!dst || !src || count <= 0) return PH_OK;
    hipLaunchKernelGGL((copy_kernel<T>), dim3(blocks_for(count)), dim3(256), 0, st, (const T *)src, (T *)dst, count);
    return check_launch("copy");
}

// copy of a step's tensor with rows of g.k elements into the caller's, with rows of g.k_given
template <typename T>
ph_status tap_rows(const Geo &g, void *dst, const void *src, int64_t rows, hipStream_t st)
{
    if (g.k == g.k_given) return tap_copy<T>(dst, src, rows * g.k, st);
    if (!dst || !src || rows <= 0) return PH_OK;
    hipLaunchKernelGGL((unpad_copy_kernel<T>), dim3(blocks_for(rows * g.k_given)), dim3(256), 0, st, (const T *)src, (T *)dst, rows, (int)g.k_given, (int)g.k);
    return check_launch("copy");
}

// error compression: dG_send[i] = delta . D_i   ([B, so] x [so, k] for every peer, one product over N = q*k);
// w_out, kk: the output width and phantom width of the layer whose delta (dl) and D these are
Product error_compression_product(int64_t B, int64_t q, void *dG_send, const void *dl, const void *Dw, int64_t w_out, int64_t kk)
{
    Product send{};
    send.a = view_plain(dl, w_out, B * w_out);
    send.b.p0 = nullptr; send.b.p1 = const_cast<void *>(Dw); send.b.g0 = 0; send.b.g1 = q * w_out * kk;
    send.b.r = axis_seg(0, (int)kk, 0, 1, w_out * kk); send.b.c = axis_plain(0, kk);
    send.b.skip0 = NO_SKIP; send.b.skip_g = 0;
    send.o.p0 = nullptr; send.o.p1 = dG_send; send.o.g0 = 0; send.o.g1 = q * B * kk;
    send.o.r = axis_plain(0, kk); send.o.c = axis_seg(0, (int)kk, 0, 1, B * kk);
    send.o.skip0 = NO_SKIP; send.o.skip_g = 0;
    send.ep = epi_store();
    send.M = q > 0 ? B : 0; send.N = q * kk; send.K = w_out;
    return send;
}

// The four products of a layer's backward pass (Eq. (backprop), (bpL)-(bpD)) from its local error delta.
struct BwdProducts {
    Product send, dx, dw, dc;
};

BwdProducts make_bwd_products(const Geo &g, const BwdArgs &b, const void *delta)
{
    const int64_t B = g.B, si = g.si, so = g.so, k = g.k, q = g.q;
    BwdProducts pr{};
    pr.send = error_compression_product(B, q, b.dG_send, delta, b.Dw, so, k);

    // dX = delta . L + dg_own . C: reduction index = [delta | dg_own] against [L ; C]
    Product &dx = pr.dx;
    dx.a = q > 0 ? view_rowseg(delta, so, (int)so, B * so, b.dg_own, (int)k, 0, B * k) : view_plain(delta, so, B * so);
    dx.b = q > 0 ? view_colstack(b.Lw, si, (int)so, so * si, b.Cw, si, (int)k, k * si) : view_plain_t(b.Lw, si, so * si);
    dx.o = view_plain(b.dX, si, B * si);
    dx.ep = epi_store();
    if (b.dx_S && g.act != PH_ACT_IDENTITY) {
        dx.ep.mode = EPI_DACT; dx.ep.act = g.act; dx.ep.aux = const_cast<void *>(b.dx_S); dx.ep.aux_ld = si;
        dx.ep.aux_g = B * si; dx.ep.aux_f32 = b.dx_S_f32; dx.ep.aux_deriv = b.dx_S_deriv; dx.ep.aux_bits = b.dx_S_bits;
    } else if (b.dx_colsum) {
        dx.ep.mode = EPI_DACT; dx.ep.act = g.act; dx.ep.aux = nullptr;      // identity: column sums only
    }
    dx.ep.colsum = b.dx_colsum; dx.ep.colsum_g = si;
    dx.M = b.dX ? B : 0; dx.N = si; dx.K = so + k;

    // weight gradients: [dL | dD_1 .. dD_{p-1}] = delta^T . [X | G_1 .. G_{p-1}], and dC = dg_own^T . X beside it
    Product &dw = pr.dw;
    dw.a = view_plain_t(delta, so, B * so);
    dw.b = q > 0 ? view_rowseg_t(b.X, si, (int)si, B * si, b.G, (int)k, B * k, 0, g.all ? 0 : NO_SKIP, g.all ? 1 : 0)
                 : view_plain_t(b.X, si, B * si);
    dw.o.p0 = b.dLw; dw.o.p1 = b.dDw; dw.o.g0 = so * si; dw.o.g1 = q * so * k;
    dw.o.r = axis_plain(si, k);
    dw.o.c = q > 0 ? axis_seg((int)si, (int)k, 1, 1, so * k) : axis_plain(1, 0);
    dw.o.skip0 = NO_SKIP; dw.o.skip_g = 0;
    dw.ep = epi_store();
    dw.M = so; dw.N = g.Kc; dw.K = B;
    pr.dc = Product{view_plain_t(b.dg_own, k, B * k), view_plain_t(b.X, si, B * si), view_plain(b.dCw, si, k * si), epi_store(),
                    q > 0 ? k : 0, si, B};
    dw.sgd = b.sgd_w;
    pr.dc.sgd = b.sgd_c;
    return pr;
}

// In-memory reduce-scatter: dg_own of every rank from what all ranks sent; tail: finished by its first workgroup.
template <typename T>
ph_status launch_reduce_scatter(const Geo &g, const void *dG_send, void *dg_own, const LossTail &tail, hipStream_t st)
{
    const int64_t per_slot = g.B * g.k;
    constexpr int RS_VEC = 16 / (int)sizeof(T);
    const bool wide = per_slot % RS_VEC == 0 && (((uintptr_t)dG_send | (uintptr_t)dg_own) & 15) == 0;
    const int64_t per_wg = 32 * (wide ? RS_VEC : 1);
    dim3 grid((unsigned)((per_slot + per_wg - 1) / per_wg), (unsigned)g.p);
    ProfScope prof("reduce-scatter", 0, per_slot * g.p * (g.p - 1), 0, 1, st);
    if (wide)
        hipLaunchKernelGGL((reduce_scatter_kernel<T, RS_VEC>), grid, dim3(256), 0, st, (const T *)dG_send, (T *)dg_own, (int)g.p, per_slot, tail);
    else
        hipLaunchKernelGGL((reduce_scatter_kernel<T, 1>), grid, dim3(256), 0, st, (const T *)dG_send, (T *)dg_own, (int)g.p, per_slot, tail);
    return check_launch("reduce-scatter");
}

// Does an output of a layer's backward call lie over dY?
bool gradient_overlaps_dY(const Geo &g, const BwdArgs &b)
{
    const size_t held = (size_t)g.groups;
    auto hits = [&](const void *p, size_t bytes) { return overlap(b.dY, held * g.B * g.so * g.esz, p, bytes); };
    bool any = hits(b.dX, held * g.B * g.si * g.esz) || hits(b.dLw, held * g.so * g.si * 4) || hits(b.dbias, held * g.so * 4);
    if (g.q > 0)
        any = any || hits(b.dCw, held * g.k * g.si * 4) || hits(b.dDw, held * g.q * g.so * g.k * 4) ||
              hits(b.dG_send, held * g.q * g.B * g.k * g.esz) || (g.all && hits(b.dg_own, held * g.B * g.k * g.esz));
    return any;
}

// delta = dY * sigma'(S); with the identity, dY itself and no launch, or a copy of it if an output lies over it
template <typename T>
ph_status local_error(const Geo &g, const BwdArgs &b, void *buffer, const void **delta, hipStream_t st)
{
    const int64_t count = (int64_t)g.groups * g.B * g.so;
    if (g.act == PH_ACT_IDENTITY) {
        const bool copy = gradient_overlaps_dY(g, b);
        *delta = copy ? buffer : b.dY;
        return copy ? tap_copy<T>(buffer, b.dY, count, st) : PH_OK;
    }
    ProfScope prof("local error", 0, count, 0, 1, st);
    auto kern = g.act == PH_ACT_GELU ? delta_kernel<T, true> : delta_kernel<T, false>;
    hipLaunchKernelGGL(kern, dim3(blocks_for(count, 256 * 16 / (int)sizeof(T))), dim3(256), 0, st,
                       (const T *)b.dY, (const T *)b.S, (T *)buffer, count);
    *delta = buffer;
    return check_launch("local error");
}

// A layer's backward call through gemm_flex.h: everything that needs the local error alone goes out together.
template <typename T>
ph_status flex_layer_bwd(const Geo &g, const BwdArgs &b, const BwdWs &w, hipStream_t st)
{
    const void *delta = nullptr;
    PH_TRY(local_error<T>(g, b, w.delta, &delta, st));
    BwdProducts pr = make_bwd_products(g, b, delta);
    pr.dw.km = pr.dc.km = true;
    pr.dw.rowsum = b.dbias;
    if (g.all && g.q > 0) {
        PH_TRY((launch_flex<T>(&pr.send, 1, false, g, LossTail{}, st, "error compression")));
        PH_TRY(launch_reduce_scatter<T>(g, b.dG_send, b.dg_own, LossTail{}, st));
        const Product rest[3] = {pr.dw, pr.dc, pr.dx};
        return launch_flex<T>(rest, 3, false, g, LossTail{}, st, "weight + compressor + input gradients");
    }
    const Product every[4] = {pr.dw, pr.dc, pr.dx, pr.send};
    return launch_flex<T>(every, 4, false, g, LossTail{}, st, "gradients | error compression");
}

ph_status bwd_impl(const Geo &g, const BwdArgs &b, const BwdWs &w, hipStream_t st)
{
    typedef bf16_t T;
    const int64_t B = g.B, so = g.so, k = g.k, q = g.q;
    const int64_t act_count = (int64_t)g.groups * B * so;

    // local error delta = dY * sigma'
    const void *delta = b.delta_ready;
    if (!delta) PH_TRY(local_error<T>(g, b, w.delta, &delta, st));

    // the loss rider goes to the first launch that can carry it
    auto take_tail = [&]() {
        LossTail t{};
        if (b.loss_tail) { t = *b.loss_tail; b.loss_tail->partial = nullptr; }
        return t;
    };

    // bias gradient: column sums of delta
    {
        const int strips = (int)((so + CSUM_COLS - 1) / CSUM_COLS);
        // enough workgroups to pull the whole tensor at memory speed: split the rows when the strips are few
        int chunks = (int)std::max<int64_t>(1, std::min<int64_t>(256 / ((int64_t)strips * g.groups), B / 128));
        const int rows_per_chunk = (int)((B + chunks - 1) / chunks);
        chunks = (int)((B + rows_per_chunk - 1) / rows_per_chunk);
        if (chunks > 1 && !b.dbias_ready) {
            ProfScope prof("clear bias gradient", 0, (int64_t)g.groups * so, 0, 1, st);
            hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks_for((int64_t)g.groups * so)), dim3(256), 0, st, b.dbias,
                               (int64_t)g.groups * so);
            PH_TRY(check_launch("clear bias gradient"));
        }
        if (!b.dbias_ready) {
            dim3 grid((unsigned)strips, (unsigned)g.groups, (unsigned)chunks);
            ProfScope prof("bias gradient", 0, act_count, 0, 1, st);
            hipLaunchKernelGGL((colsum_kernel<T>), grid, dim3(256), 0, st, (const T *)delta, b.dbias, (int)B, (int)so,
                               rows_per_chunk, take_tail());
            PH_TRY(check_launch("bias gradient"));
        }
    }

    BwdProducts pr = make_bwd_products(g, b, delta);
    const Product &send = pr.send, &dw = pr.dw, &dc = pr.dc;
    Product &dx = pr.dx;
    auto error_compression = [&](const void *dl, const void *Dw, int64_t w_out, int64_t kk) {
        return error_compression_product(B, q, b.dG_send, dl, Dw, w_out, kk);
    };
    // Riders of the weight-gradient launch (MfmaTailBatch) exist on the matrix-core path for launches of at most one
    // tile per compute unit.  PHANTOM_TAIL=0 switches them off (for measurements).
    const int64_t tail_tiles = (tiles_of(dw.M, dw.N) + tiles_of(dc.M, dc.N)) * g.groups;
    static const char *tail_force = tuning_env("PHANTOM_TAIL");
    const bool riders = tail_tiles <= 256 && !(tail_force && tail_force[0] == '0');
    // One rank, no input gradient wanted (the first layer): this layer's error compression has no launch to share
    // with the input gradient and nothing waits for it, so it rides with the weight gradients.
    // (not with an update in the epilogues: it would write the D that the error compression reads)
    const bool send_rides = riders && !g.all && !b.dX && q > 0 && !b.defer && !b.sgd_w.w0;

    const GemmPlan plan_x{LD_KC, LD_KM, g.vec};
    const int64_t send_rows = (int64_t)g.groups * q * B;
    if (g.all) {
        // the input gradient needs dg_own, which is the sum of what all ranks send: three launches
        if (!b.send_done) PH_TRY((launch_products<T, T>(plan_x, &send, 1, g.groups, st, "error compression")));
        PH_TRY(tap_rows<T>(g, b.tap_dG_send, b.dG_send, send_rows, st));
        // Reduce-scatter as a sum on read: the input gradient's loader sums the p-1 senders' slices while it stages
        // the one reduction tile that holds dg_own, and writes dg_own out for the compressor gradient.  Conditions:
        // the block starts on a tile boundary of the reduction index and fits one tile (so a multiple of 64,
        // k a divisor of 64), 16-byte vectors, and at most 8 ranks: a thread has the loads of seven senders
        // in flight at a time, and with 16 ranks the step got 0.4 % slower instead of 1.8 % faster.  PHANTOM_RS_ON_READ=0 keeps the kernel of its own (for measurements).
        static const char *rs_force = tuning_env("PHANTOM_RS_ON_READ");
        const bool sum_on_read = g.vec == 8 && q > 0 && b.dX && g.p <= 8 && k <= KT &&
                                 KT % k == 0 && so % KT == 0 && !(rs_force && rs_force[0] == '0');
        if (sum_on_read) {
            dx.rs.src = b.dG_send; dx.rs.out = b.dg_own;
            dx.rs.per_slot = B * k; dx.rs.p = (int)g.p; dx.rs.k = (int)k;
        } else if (q > 0) {
            PH_TRY(launch_reduce_scatter<T>(g, b.dG_send, b.dg_own, take_tail(), st));
        }
        PH_TRY((launch_products<T, T>(plan_x, &dx, 1, g.groups, st, "input gradient")));
        PH_TRY(tap_copy<T>(b.tap_dg_own, b.dg_own, (int64_t)g.groups * B * k, st));
    } else if (!send_rides) {
        Product both[2] = {dx, send};
        PH_TRY((launch_products<T, T>(plan_x, both, 2, g.groups, st, "input gradient + error compression",
                                      "input gradient", "error compression")));
        PH_TRY(tap_rows<T>(g, b.tap_dG_send, b.dG_send, send_rows, st));
    }

    if (b.below_done) *b.below_done = false;
    if (b.defer) return PH_OK;
    if (riders) {
        // The layer below starts its backward with an error compression that fills half of the device or less
        // for a short while: it comes along when it leaves at least half of the compute units to the weight
        // gradients from the start (they take over the rest as it finishes).
        Product below{};
        bool with_head = false;
        int64_t used = tail_tiles;
        int vec = g.vec;
        if (send_rides) {
            below = send;
            with_head = true;
            used += (tiles_of(below.M, below.N) * g.groups + 7) & ~(int64_t)7;
        } else if (b.below_Dw && b.below_g && b.below_g->vec > 0 && b.dX && g.all && q > 0) {
            below = error_compression(b.dX, b.below_Dw, b.below_g->so, b.below_g->k);
            vec = std::min(vec, b.below_g->vec);
            with_head = tiles_of(below.M, below.N) * g.groups <= 128;
        }
        // a loss that no kernel has finished yet: one more workgroup does it
        const bool with_loss = b.loss_tail && b.loss_tail->partial;
        if (with_head || with_loss) {
            const LossTail tail = with_loss ? take_tail() : LossTail{};
            PH_TRY(launch_tail(with_head ? &below : nullptr, dw, dc, tail, g.groups, vec, st,
                               send_rides  ? "weight + compressor gradients | error compression"
                               : with_head ? "weight + compressor gradients | error compression below"
                                           : "weight + compressor gradients | loss",
                               send_rides && used > 256));
            if (b.below_done) *b.below_done = with_head && !send_rides;
            if (send_rides) PH_TRY(tap_rows<T>(g, b.tap_dG_send, b.dG_send, send_rows, st));
            return PH_OK;
        }
    }
    MfmaRiders ride{};
    ride.tail = take_tail();
    Product grads[2] = {dw, dc};
    // (send_rides never gets here: its launch above carries the error compression)
    return launch_products<T, float>(GemmPlan{LD_KM, LD_KM, g.vec}, grads, q > 0 ? 2 : 1, g.groups, st,
                                     "weight + compressor gradients", "weight gradients", "compressor gradient", ride);
}

ph_status check_fwd_args(const Geo &g, const FwdArgs &f)
{
    PH_TRY(need(f.X, "X")); PH_TRY(need(f.Lw, "Lw")); PH_TRY(need(f.bias, "bias")); PH_TRY(need(f.Y, "Y"));
    PH_TRY(optional(f.A_save, "A_save"));
    if (g.q > 0) {
        PH_TRY(need(f.Cw, "Cw")); PH_TRY(need(f.Dw, "Dw")); PH_TRY(need(f.g_own, "g_own"));
        if (!g.all) PH_TRY(need(f.G, "G"));
    }
    return PH_OK;
}

ph_status check_bwd_args(const Geo &g, const BwdArgs &b)
{
    PH_TRY(need(b.dY, "dY")); PH_TRY(need(b.X, "X")); PH_TRY(need(b.Lw, "Lw"));
    if (g.act != PH_ACT_IDENTITY) PH_TRY(need(b.S, "A_or_Y"));
    PH_TRY(optional(b.dX, "dX"));
    PH_TRY(need(b.dLw, "dLw")); PH_TRY(need(b.dbias, "dbias"));
    if (g.q > 0) {
        PH_TRY(need(b.Cw, "Cw")); PH_TRY(need(b.Dw, "Dw")); PH_TRY(need(b.G, "G")); PH_TRY(need(b.dg_own, "dg_own"));
        PH_TRY(need(b.dCw, "dCw")); PH_TRY(need(b.dDw, "dDw")); PH_TRY(need(b.dG_send, "dG_send"));
    }
    return PH_OK;
}

ph_status check_ws(void *ws, size_t have, size_t want)
{
    if (want == 0) return PH_OK;
    if (!ws) return fail(PH_ERR_WORKSPACE, "workspace is NULL, %zu bytes needed", want);
    if ((uintptr_t)ws & 255) return fail(PH_ERR_WORKSPACE, "workspace is not 256-byte aligned");
    if (have < want) return fail(PH_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", have, want);
    return PH_OK;
}

// The update of layer l in the epilogues that finish its gradients (Section VI: plain SGD), `weights` (L, D and the bias) or
// C; keep: the gradients are stored too.
SgdInPlace sgd_of(const ph_step_args &a, int l, int64_t q, bool weights, const float *bias_grad, bool past_caches = false)
{
    auto at = [l](auto *const *arr) { return arr ? arr[l] : nullptr; };
    SgdInPlace s{};
    s.lr = a.lr;
    s.past_caches = past_caches;
    if (weights) {
        s.master0 = at(a.Lw_master); s.w0 = a.Lw[l];
        s.master1 = q ? at(a.Dw_master) : nullptr; s.w1 = q ? a.Dw[l] : nullptr;
        s.keep_grad = a.dLw || a.dDw;
        s.bias_master = at(a.bias_master); s.bias_w = a.bias[l]; s.bias_grad = bias_grad;
    } else if (q) {
        s.master0 = at(a.Cw_master); s.w0 = a.Cw[l];
        s.keep_grad = a.dCw != nullptr;
    }
    return s;
}

// Copies of the layers' forward results for the taps of the step.
template <typename T>
ph_status forward_taps(const std::vector<Geo> &geos, const ph_step_args &a, const StepWs &w, hipStream_t st)
{
    if (!a.taps) return PH_OK;
    for (size_t l = 0; l < geos.size(); ++l) {
        const Geo &g = geos[l];
        if (a.taps->Y) PH_TRY(tap_copy<T>(a.taps->Y[l], w.Y[l], (int64_t)g.groups * g.B * g.so, st));
        if (a.taps->g_own && g.q) PH_TRY(tap_rows<T>(g, a.taps->g_own[l], w.G[l], (int64_t)g.groups * g.B, st));
    }
    return PH_OK;
}

// One step through gemm_flex.h.  The weight + compressor gradients of a layer (with the update in their epilogues: by then
// nothing reads that layer's weights any more) go out with the first launch of the layer below, so that a layer's
// backward pass is one launch with one rank and three with all ranks on the device.
template <typename T>
ph_status flex_step(const std::vector<Geo> &geos, const ph_step_args &a, const StepWs &w, hipStream_t st)
{
    Geo g = geos.back();              // what does not depend on the layer is read from the last one
    for (const Geo &x : geos) {                                // (a backward launch carries products of two layers)
        g.fine = g.fine || x.fine;
        g.vec = std::min(g.vec, x.vec);
        g.whole = g.whole && x.whole;
    }
    const int L = g.layers;
    const int64_t B = g.B, q = g.q;
    const bool train = a.mode != PH_STEP_FORWARD, update = a.mode == PH_STEP_TRAIN;
    const bool gelu = g.act == PH_ACT_GELU, save_deriv = gelu && std::is_same<T, bf16_t>::value;
    // delta_l is read until the launch after the next one is out: three buffers in turn
    void *const deltas[3] = {w.dYa, w.dYb, w.bwd.delta};
    auto delta_of = [&](int l) { return deltas[l % 3]; };
    auto dbias_of = [&](int l) { return a.dbias ? a.dbias[l] : w.dbias + w.dbias_at[(size_t)l]; };

    OutputError oe{a.T, delta_of(L - 1), w.mse_partial, 1.0f / (float)B, nullptr};
    int mse_tiles = 0;
    for (int l = 0; l < L; ++l) {
        FwdArgs f{};
        f.X = l > 0 ? w.Y[(size_t)l - 1] : a.X0;
        f.Lw = a.Lw[l]; f.Cw = q ? a.Cw[l] : nullptr; f.Dw = q ? a.Dw[l] : nullptr; f.bias = a.bias[l];
        f.G = (q && !g.all) ? a.G[l] : nullptr;
        // (nobody reads the last layer's: its update forms delta_L itself)
        f.Y = w.Y[(size_t)l]; f.g_own = w.G[(size_t)l]; f.A_save = train && l < L - 1 ? w.A[(size_t)l] : nullptr;
        f.a_f32 = !save_deriv; f.a_deriv = save_deriv;
        f.mse = train && l == L - 1 ? &oe : nullptr;
        PH_TRY(flex_fwd<T>(geos[(size_t)l], f, st, f.mse ? &mse_tiles : nullptr));
    }
    PH_TRY(forward_taps<T>(geos, a, w, st));
    if (!train) return PH_OK;
    if (a.taps && a.taps->delta) PH_TRY(tap_copy<T>(a.taps->delta[L - 1], delta_of(L - 1), (int64_t)g.groups * B * g.so, st));

    LossTail tail{w.mse_partial, mse_tiles, 0.5f / (float)B, a.loss};
    std::vector<Product> next;        // the next launch's products
    auto go = [&](const char *what) -> ph_status {
        bool any = false;
        for (const Product &pr : next) any = any || (pr.M > 0 && pr.N > 0);
        if (!any) { next.clear(); return PH_OK; }
        PH_TRY((launch_flex<T>(next.data(), (int)next.size(), false, g, tail, st, what)));
        tail.partial = nullptr;
        next.clear();
        return PH_OK;
    };
    for (int l = L - 1; l >= 0; --l) {
        const Geo &gl = geos[(size_t)l];
        BwdArgs b{};
        b.X = l > 0 ? w.Y[(size_t)l - 1] : a.X0;
        b.Lw = a.Lw[l]; b.Cw = q ? a.Cw[l] : nullptr; b.Dw = q ? a.Dw[l] : nullptr;
        b.G = q ? (g.all ? w.G[(size_t)l] : a.G[l]) : nullptr;
        b.dg_own = q ? (g.all ? w.dg_own : const_cast<void *>(a.dg_own[l])) : nullptr;
        b.dX = l > 0 ? delta_of(l - 1) : nullptr;
        b.dx_S = l > 0 ? (gelu ? w.A[(size_t)l - 1] : w.Y[(size_t)l - 1]) : nullptr;
        b.dx_S_f32 = gelu && !save_deriv; b.dx_S_deriv = save_deriv;
        b.dLw = a.dLw ? a.dLw[l] : w.dLw[l & 1];
        b.dCw = q ? (a.dCw ? a.dCw[l] : w.dCw[l & 1]) : nullptr;
        b.dDw = q ? (a.dDw ? a.dDw[l] : w.dDw[l & 1]) : nullptr;
        b.dbias = dbias_of(l);
        b.dG_send = w.dG_send;
        if (update) {
            b.sgd_w = sgd_of(a, l, q, true, b.dbias);
            b.sgd_c = sgd_of(a, l, q, false, nullptr);
        }
        BwdProducts pr = make_bwd_products(gl, b, delta_of(l));
        pr.dw.km = pr.dc.km = true;
        pr.dw.rowsum = b.dbias;
        const int64_t send_rows = (int64_t)g.groups * q * B;
        void *tap_send = (a.taps && a.taps->dG_send && q) ? a.taps->dG_send[l] : nullptr;
        if (g.all && q > 0) {
            next.push_back(pr.send);
            PH_TRY(go("error compression | gradients above"));
            PH_TRY(tap_rows<T>(gl, tap_send, b.dG_send, send_rows, st));
            // the launch that needs dg_own first sums it on read where it can: the input gradient, or (first layer) the compressor gradient's
            const SumOnRead sum{b.dG_send, b.dg_own, B * gl.k, (int)g.p, (int)gl.k};
            const Product last[2] = {pr.dw, pr.dc};
            const bool on_read = sizeof(T) == 4 && g.p <= 8 && (l > 0 ? f32_few_groups(&pr.dx, 1, g) : f32_few_groups(last, 2, g)) > 0;
            if (on_read) (l > 0 ? pr.dx : pr.dc).rs = sum;
            else PH_TRY(launch_reduce_scatter<T>(gl, b.dG_send, b.dg_own, LossTail{}, st));
            next.push_back(pr.dx);
            PH_TRY(go("input gradient"));
            if (on_read && l == 0) {
                next.push_back(pr.dw);
                next.push_back(pr.dc);
                PH_TRY(go("weight + compressor gradients"));
            }
            PH_TRY(tap_copy<T>(a.taps && a.taps->dg_own ? a.taps->dg_own[l] : nullptr, b.dg_own, (int64_t)g.groups * B * gl.k, st));
            if (on_read && l == 0) break;
        } else {
            next.push_back(pr.dx);
            next.push_back(pr.send);
            // (Dense, first layer: there is neither, and its gradients go out with the second layer's, as the launches that read the weights are out.  With peers the
            // error compression reads D, which the gradients' launch updates.  Trained, us a step, in a launch of their own : so: 3 x 751 at batch 1000 94.4 :
            // 86.2, 2 x 2048 at 256 63.6 : 59.0, 4 x 1024 at 512 83.3 : 79.3, 3 x 512 at 4000 95.9 : 96.1.)
            if (l > 0 || q > 0) PH_TRY(go("input gradient + error compression | gradients above"));
            PH_TRY(tap_rows<T>(gl, tap_send, b.dG_send, send_rows, st));
        }
        if (a.taps && a.taps->delta && l > 0) PH_TRY(tap_copy<T>(a.taps->delta[l - 1], b.dX, (int64_t)g.groups * B * gl.si, st));
        next.push_back(pr.dw);
        next.push_back(pr.dc);
    }
    return go("weight + compressor gradients");
}

// Do a bf16 training step's tensors (weights, masters, activations, what the peers send and get) fit the last-level cache of 256 MB?  Repeated steps then
// find their masters there, and streaming reads would give that up.
// Trained, us a step, masters past the caches : kept.  Smaller steps: dense 4096 at batch 1024 (128 MB) 103.8 : 95.8, two (240 MB) 228.9 : 220.4, 3 of 3072 (210 MB)
// 248.0 : 242.5, 6 of 1024 + 448 at 4096 (190 MB) 376.2 : 372.0, 8 ranks of 1024 + 224, two layers at 1024 (220 MB), 203.9 : 197.0; larger: 4 of 3072 at
// 1024 (276 MB) 337.7 : 351.0, 8 ranks of 512 / 1024 (262 MB) 329.4 : 337.0, 4 of 4096 485 : 530, 8 of 1024 + 960 with GELU at 4096 (430 MB) 594 : 598;
// 6 of 2048 at 2048 (256 MB) 387.3 : 389.2.
bool step_fits_last_cache(const std::vector<Geo> &geos)
{
    static const char *force = tuning_env("PHANTOM_KEEP_MASTERS");     // =0 / 1 (for measurements)
    if (force) return force[0] == '1';
    int64_t bytes = 0, send = 0;
    for (const Geo &g : geos) {
        const int64_t act = g.B * g.so, peers = g.q * g.B * g.k, e = (int64_t)g.esz;
        bytes += g.groups * ((g.so * g.Kc + g.k * g.si) * (e + 4) + 2 * act * e + g.B * g.k * e);
        if (g.act == PH_ACT_GELU && &g != &geos.back()) bytes += g.groups * act * 4;
        if (!g.all) bytes += (peers + g.B * g.k) * e;
        send = std::max(send, g.groups * peers * e);
    }
    const Geo &first = geos.front(), &last = geos.back();
    bytes += send + first.groups * first.B * (first.si + last.so) * (int64_t)first.esz;
    return bytes <= (int64_t)256 << 20;
}

// One bf16 step on the 128 x 128 kernels of gemm_mfma.h.
ph_status step_impl(const std::vector<Geo> &geos, const ph_step_args &a, const StepWs &w, hipStream_t st)
{
    typedef bf16_t T;
    const Geo &g = geos.back();       // the last layer; what does not depend on the layer is read from it
    const int L = g.layers;
    const int64_t B = g.B, q = g.q;
    const int64_t act_count = (int64_t)g.groups * B * g.so;      // elements of the network output

    // What the backward pass needs of a layer's pre-activation A is sigma'(A) alone.  ReLU reads it off the
    // layer's output.  GELU has the forward epilogue, which evaluates erf and exp for
    // sigma(A) anyway, store sigma'(A) in float: the bytes of an fp32 A and no second evaluation in the
    // input-gradient epilogue.  (Any coarser grid for that factor moves delta across bf16 rounding
    // boundaries often enough to show after a few layers.)
    const bool save_deriv = g.act == PH_ACT_GELU;

    // Bias gradients (Eq. (bpb)) are column sums of delta: the product that writes a layer's delta (the input gradient
    // of the layer above; for the last layer its own update, see below) adds them up on its way out, so every
    // layer's bias gradient has a buffer of its own that is zeroed once for the whole step.
    const bool train = a.mode != PH_STEP_FORWARD, update = a.mode == PH_STEP_TRAIN, past_caches = update && !step_fits_last_cache(geos);
    auto dbias_of = [&](int l) { return a.dbias ? a.dbias[l] : w.dbias + w.dbias_at[(size_t)l]; };
    // What the step adds into is cleared by its first forward launch that can do it on the way, else by one of its own (the
    // words for cut reductions lie right behind the workspace's block and are cleared with it).
    ClearList clear{};
    if (train) {
        auto add = [&](void *p, int64_t n) { clear.p[clear.count] = (float *)p; clear.n[clear.count++] = (int)n; };
        if (a.dbias) {
            for (int l = 0; l < L; ++l) {
                if (clear.count == CLEAR_MAX - 1) PH_TRY(launch_clear(clear, st));
                add(a.dbias[l], (int64_t)g.groups * geos[(size_t)l].so);
            }
            if (w.arrived_words > 0) add(w.arrived, w.arrived_words);
        } else {
            add(w.dbias, w.dbias_at[(size_t)L] + w.arrived_words);
        }
    }

    // The output error of the MSE loss (Eq. (deltaL)) is elementwise in the last layer's output, so
    // that layer's update forms it in its epilogue, together with the last bias gradient and one partial
    // sum of the loss per tile: two launches less than a kernel for the error and one for the column sums.
    const int64_t out_tiles = tiles_of(B, g.so) * g.groups;
    // (one rank with deferred weight gradients keeps every layer's delta: the last layer's goes to its own buffer)
    const Deferral deferral = train ? deferred_weight_gradients(geos) : DEFER_NONE;
    const bool deferred = deferral != DEFER_NONE;
    void *delta_top = deferred ? w.delta_of[(size_t)L - 1] : w.dYa;
    OutputError oe{a.T, delta_top, w.mse_partial, 1.0f / (float)B, dbias_of(L - 1)};

    // Deferred weight gradients: the products of all layers are known from the buffers alone.  Their launch comes at the
    // end of the backward pass (layers of different shapes: its parameter table goes up now, ahead of the
    // forward pass): the compressor gradients first (few
    // tiles with half of their rows empty, cut into pieces), then the weight gradients' tiles, which fill the compute
    // units as those come free; the SGD update of L, C, D and the bias in the epilogues, the loss by the first workgroup.
    int table_grid = 0;
    std::vector<Product> all_dw, all_dc;               // by layer
    const bool uniform = L <= UNIFORM_LAYERS && all_alike(geos);
    const LossTail table_tail{w.mse_partial, (int)out_tiles, 0.5f / (float)B, a.loss};
    if (deferred) {
        for (int l = 0; l < L; ++l) {
            BwdArgs b{};
            b.X = l > 0 ? w.Y[l - 1] : a.X0;
            b.G = q ? a.G[l] : nullptr;
            b.dg_own = q ? const_cast<void *>(a.dg_own[l]) : nullptr;
            // (gradients that the caller does not want: a training step has the update in the epilogues and stores
            // none; a step without update stores every layer's in the same place, where nobody reads them)
            b.dLw = a.dLw ? a.dLw[l] : w.dLw[0];
            b.dCw = q ? (a.dCw ? a.dCw[l] : w.dCw[0]) : nullptr;
            b.dDw = q ? (a.dDw ? a.dDw[l] : w.dDw[0]) : nullptr;
            if (update) {
                b.sgd_w = sgd_of(a, l, q, true, dbias_of(l), past_caches);
                b.sgd_c = sgd_of(a, l, q, false, nullptr, past_caches);
            }
            const BwdProducts all = make_bwd_products(geos[(size_t)l], b, w.delta_of[(size_t)l]);
            all_dw.push_back(all.dw);
            all_dc.push_back(all.dc);
        }
        if (!uniform) {
            std::vector<Product> later;
            std::vector<int> splits;
            for (int l = L - 1; l >= 0; --l)
                if (all_dc[(size_t)l].M > 0) { later.push_back(all_dc[(size_t)l]); splits.push_back(compressor_gradient_pieces(geos[(size_t)l])); }
            for (int l = L - 1; l >= 0; --l) { later.push_back(all_dw[(size_t)l]); splits.push_back(1); }
            PH_TRY(upload_product_table(later, splits, w.table, w.parts, w.arrived, table_tail, st, &table_grid));
        }
    }

    // forward through every layer; y_l stays in the storage type between layers
    std::vector<Product> later;
    for (int l = 0; l < L; ++l) {
        const bool bits = train && w.relu_bits[(size_t)l] != nullptr;
        FwdArgs f{l > 0 ? w.Y[(size_t)l - 1] : a.X0, a.Lw[l], q ? a.Cw[l] : nullptr, q ? a.Dw[l] : nullptr, a.bias[l],
                  (q && !g.all) ? a.G[l] : nullptr, w.Y[l], w.G[l], bits ? w.relu_bits[(size_t)l] : train && l < L - 1 ? w.A[l] : nullptr,      // (the last layer's update forms delta_L itself)
                  false, !save_deriv && !bits, save_deriv, bits, (train && l == L - 1) ? &oe : nullptr, &clear, g.all || L == 1 ? nullptr : &later};
        PH_TRY(fwd_impl(geos[(size_t)l], f, st));
    }
    std::vector<Product> thin;
    later.erase(std::remove_if(later.begin(), later.end(), [&](const Product &pr) { if (pr.N <= THIN_MAX_N) thin.push_back(pr); return pr.N <= THIN_MAX_N; }), later.end());
    if (!later.empty()) {
        int vec = 8;
        for (const Geo &x : geos) vec = std::min(vec, x.vec);
        PH_TRY(launch_many(later, vec, st, "compressions of all layers"));
    }
    if (!thin.empty()) PH_TRY(launch_compressions(thin, st, "compressions of all layers"));
    PH_TRY(forward_taps<T>(geos, a, w, st));
    if (!train) return PH_OK;

    // The loss is the sum of partial sums that the output-error computation leaves; the first memory-bound
    // kernel after it adds them up as a rider (LossTail), a kernel of its own if there is none.
    LossTail loss_tail{w.mse_partial, (int)out_tiles, 0.5f / (float)B, a.loss};
    if (a.taps && a.taps->delta) PH_TRY(tap_copy<T>(a.taps->delta[L - 1], delta_top, act_count, st));   // delta_L, Eq. (deltaL)

    void *dY = w.dYa, *dX = w.dYb;    // delta of the current layer / of the layer below
    bool send_done = false;           // the current layer's error compression went out with the layer above
    for (int l = L - 1; l >= 0; --l) {
        BwdArgs b{};
        b.send_done = send_done;
        b.below_Dw = (g.all && q > 0 && l > 0) ? a.Dw[l - 1] : nullptr;
        b.below_g = l > 0 ? &geos[(size_t)l - 1] : nullptr;
        b.below_done = &send_done;
        b.dbias_ready = true;         // the product that wrote this layer's delta took the column sums
        b.loss_tail = &loss_tail;
        b.dx_colsum = l > 0 ? dbias_of(l - 1) : nullptr;
        if (deferred) { dY = w.delta_of[(size_t)l]; dX = l > 0 ? w.delta_of[(size_t)l - 1] : nullptr; b.defer = true; b.loss_tail = nullptr; }
        b.delta_ready = dY; b.X = l > 0 ? w.Y[(size_t)l - 1] : a.X0;
        b.dx_S_bits = l > 0 && w.relu_bits[(size_t)l - 1] != nullptr;
        b.dx_S = l > 0 ? (b.dx_S_bits ? w.relu_bits[(size_t)l - 1] : save_deriv ? w.A[l - 1] : w.Y[l - 1]) : nullptr;
        b.dx_S_deriv = save_deriv;
        b.Lw = a.Lw[l]; b.Cw = q ? a.Cw[l] : nullptr; b.Dw = q ? a.Dw[l] : nullptr;
        b.G = q ? (g.all ? w.G[l] : a.G[l]) : nullptr;
        b.dg_own = q ? (g.all ? w.dg_own : const_cast<void *>(a.dg_own[l])) : nullptr;
        b.dX = l > 0 ? dX : nullptr;
        b.dLw = a.dLw ? a.dLw[l] : w.dLw[l & 1];
        b.dCw = q ? (a.dCw ? a.dCw[l] : w.dCw[l & 1]) : nullptr;
        b.dDw = q ? (a.dDw ? a.dDw[l] : w.dDw[l & 1]) : nullptr;
        b.dbias = dbias_of(l);
        b.dG_send = w.dG_send;
        // SGD on this layer in the epilogues of its gradients: every launch that reads its weights is out by then
        if (update && !deferred) {
            b.sgd_w = sgd_of(a, l, q, true, b.dbias, past_caches);
            b.sgd_c = sgd_of(a, l, q, false, nullptr, past_caches);
        }
        const Geo &gl = geos[(size_t)l];
        if (a.taps) {
            b.tap_dG_send = (a.taps->dG_send && q) ? a.taps->dG_send[l] : nullptr;
            b.tap_dg_own = (a.taps->dg_own && q && g.all) ? a.taps->dg_own[l] : nullptr;
        }
        PH_TRY(bwd_impl(gl, b, w.bwd, st));
        // what the input gradient's epilogue left in dX is delta_{l-1} (Eq. (backprop), sigma' applied)
        if (a.taps && a.taps->delta && l > 0) PH_TRY(tap_copy<T>(a.taps->delta[l - 1], dX, (int64_t)g.groups * B * gl.si, st));
        if (deferred) continue;
        std::swap(dY, dX);
        if (loss_tail.partial) {                       // no kernel of this layer's backward could carry the rider
            ProfScope prof("loss", 0, loss_tail.n, 0, 1, st);
            hipLaunchKernelGGL(loss_kernel, dim3(1), dim3(256), 0, st, loss_tail);
            PH_TRY(check_launch("loss"));
            loss_tail.partial = nullptr;
        }
    }
    if (deferred) {
        const char *what = update ? "weight + compressor gradients of all layers + SGD | loss" : "weight + compressor gradients of all layers | loss";
        const bool copies = std::any_of(geos.begin(), geos.end(), [](const Geo &x) { return x.k != x.k_given; });      // (step_on_padded)
        if (uniform) PH_TRY(launch_uniform_gradients(all_dw, all_dc, deferral == DEFER_SMALL ? compressor_gradient_pieces(g) : 1, w.parts, w.arrived, table_tail, copies, st, what));
        else PH_TRY((copies ? launch_product_table<true> : launch_product_table<false>)(w.table, table_grid, st, what, all_dw.back(), all_dc.back(), L));
    }
    return PH_OK;
}

// ---- one rank's step on padded phantom widths --------------------------------------------------------
// Phantom widths that 8 does not divide cost 8-byte vectors through registers (4 divides them), or the renumbering kernels of gemm_flex.h.  One rank's
// bf16 step whose widths 8 divides therefore runs on copies of D, C, G and dg_own in which every phantom width is rounded up to a multiple
// of 8, the rest zeros: one launch ahead of the step, and in training one behind it that takes the gradients and the updated weights of D
// and C from their padded places.  The zeros meet zeros in every product that leaves the rank or the layer, also where a tensor holds
// infinities.  (All ranks on the device would read each other's padded g, zeros times what may be infinite; odd phantom widths keep the levels of sums
// that the FINE kernels give them.)
// The layers' shapes on padded copies; empty where a step cannot run on them.  (The launch ahead of the step names its tensors in the kernel arguments, six a
// layer in training: a step of more than 18 layers runs on the caller's tensors.)
std::vector<Geo> padded_geos(const ph_problem *prob, const std::vector<Geo> &geos)
{
    std::vector<Geo> out;
    auto up = [](int64_t k) { return (k + 7) & ~(int64_t)7; };
    bool any = false;
    for (const Geo &g : geos) {
        if (g.all || g.q == 0 || g.dtype != PH_BF16 || g.fine || g.si % 8 || g.so % 8) return out;
        any = any || g.k % 8;
    }
    if (!any || geos.size() > (size_t)PAD_ENTRIES / 6) return out;
    std::vector<int64_t> ks;
    for (const Geo &g : geos) ks.push_back(up(g.k));
    ph_problem padded = *prob;
    padded.k = up(prob->k);
    if (prob->widths) padded.ks = ks.data();
    char message[sizeof g_err];                        // (the caller's last error stays what it was)
    memcpy(message, g_err, sizeof g_err);
    if (make_geos(&padded, out) != PH_OK) {
        memcpy(g_err, message, sizeof g_err);
        out.clear();
    }
    for (size_t l = 0; l < out.size(); ++l) {
        out[l].k_given = geos[l].k;
        if (out[l].vec != 8 || out[l].k * out[l].si >= (int64_t)1 << 29) { out.clear(); break; }      // (PadList counts a C's elements in 32 bits)
    }
    return out;
}

// Are they worth the launches?  Where the 128 x 128 kernels then run, or the peers' part is long, which the renumbering kernels go through vector by vector,
// or the step is.  Measured (us, on the caller's tensors : on copies).  128 x 128 kernels: 6 layers of 1024 forward at batch 8192, k 4 198 : 169, k 10 275 :
// 169; 2 of 1024 + 3750 at 2000 214 : 92; 8 of 1024 + 28 trained at 4096 828 : 554, 4 of 1024 + 750 with GELU 495 : 348, 3 of 2048 + 300 at 2048 391 :
// 307.  Sums of the peers' parts over the layers: 8 ranks of 256 + 100 forward at 1500, 2 layers (1400) 31 : 26, 16 of 1024 + 100 at 128 (6000)
// 113 : 59, 32 of 512 + 18 trained at 512, 4 layers (2232) 121 : 97, 16 of 256 + 36 at 600, 3 layers (1620) 77 : 72, 32 of 256 + 10 at 256, 4 layers
// (1240) 77.6 : 77.6, 8 of 1024 + 20 at 300, 2 layers (280) 59 : 61.5.  Steps of 64 x 64 tiles (a backward pass counts twice): 6 layers of 1024 + 84 forward at
// 2048 (53000) 101 : 91, 4 of 1024 + 28 trained at 1024 (50000) 132 : 125; 4 of 512 + 28 forward at 1024 (4300) 32.8 : 35.5, 3 of 2048 + 108 at 256 (12900)
// 39.9 : 46.3.
// Where a layer's forward launch on the caller's tensors has so few tiles that eight teams share each (flex_tile_for), they share the peers' part as well, and less of it
// counts; training also moves D's masters, by the shard.  Forward, 2 and 4 layers at batch 64: 256 + 1054 21.3 : 21.6, 42.6 : 40.2, 128 + 1550 27.6 : 25.0, 55.3 : 46.8; 3 of 512 +
// 620 28.2 : 31.1.  Trained: 128 + 1054 46.8 : 43.9, 83.7 : 75.5, 256 + 1550 52.2 : 52.7, 95.1 : 92.6, 256 + 2646 67.2 : 61.4, 129.8 : 104.4, 512 + 1638 (2) 56.2 : 63.4, 512 + 3276 (2)
// 76.3 : 78.2; 3 of 512 + 620 at 128 64.0 : 71.0 (at 192, past that line, 86.0 : 71.6), 4 of 1024 + 378 at 64 100.9 : 114.7 (at 96 126.0 : 112.9).
// (The forward ones are older than the kernel for few rows, which copies may run on and the caller's tensors may not: 2 of 256 + 1054 21.2 : 18.1, 3 of 512 + 620 28.2 : 24.8.)
bool padding_pays(const std::vector<Geo> &padded, bool train)
{
    if (padded.empty()) return false;
    static const char *force = tuning_env("PHANTOM_PAD");              // =0 / 1 (for measurements)
    if (force) return force[0] == '1';
    int64_t peers = 0, steps = 0;
    for (const Geo &g : padded) {
        const int64_t own = g.q * g.k_given, small = ((g.B + 63) / 64) * ((g.so + 63) / 64 + (g.k_given + 63) / 64);
        const int64_t lost = small > FLEX_FEW ? 0 : train ? 4 * g.so : 550;
        if (own <= lost) continue;
        peers += own - lost;
        steps += ((g.B + 63) / 64) * ((g.so + 63) / 64) * ((g.Kc + 63) / 64);
    }
    return !use_flex(padded, train) || peers >= 1280 || steps * (train ? 3 : 1) >= 30000;
}

struct PadWs {
    std::vector<void *> G, C, D, dg;               // per layer, NULL where the caller's tensors are used
    std::vector<float *> dC, dD, mC, mD;           // (masters: mC, mD)
};

PadWs carve_pad(Arena &a, const std::vector<Geo> &padded, bool forward)
{
    PadWs w;
    for (const Geo &g : padded) {
        const bool on = g.k != g.k_given;
        auto take = [&](int64_t elems, size_t size) { return on && elems > 0 ? a.take((size_t)elems * size) : nullptr; };
        const int64_t train = forward ? 0 : 1;
        w.G.push_back(take(g.q * g.B * g.k, g.esz));
        w.C.push_back(take(g.k * g.si, g.esz));
        w.D.push_back(take(g.q * g.so * g.k, g.esz));
        w.dg.push_back(take(train * g.B * g.k, g.esz));
        w.dC.push_back((float *)take(train * g.k * g.si, 4));
        w.dD.push_back((float *)take(train * g.q * g.so * g.k, 4));
        w.mC.push_back((float *)take(train * g.k * g.si, 4));
        w.mD.push_back((float *)take(train * g.q * g.so * g.k, 4));
    }
    return w;
}

size_t step_ws_bytes(const std::vector<Geo> &geos)
{
    Arena a{nullptr, 0};
    carve_step(a, geos);
    return a.used;
}

// Bytes of workspace of a step on padded copies; 0: it runs on the caller's tensors, as it does with less workspace than that.
size_t padded_ws_bytes(const std::vector<Geo> &padded, bool forward)
{
    if (!padding_pays(padded, !forward)) return 0;
    Arena a{nullptr, 0};
    carve_step(a, padded, forward);
    carve_pad(a, padded, forward);
    return a.used;
}

ph_status step_on_padded(const std::vector<Geo> &geos, const ph_step_args &given, const StepWs &w, const PadWs &x, hipStream_t st)
{
    const size_t L = geos.size();
    const bool train = given.mode != PH_STEP_FORWARD, update = given.mode == PH_STEP_TRAIN;
    std::vector<void *> Cw, Dw;
    std::vector<const void *> G, dg;
    std::vector<float *> dC, dD, mC, mD;
    PadList in{};
    int blocks = 0;
    // rows of `len` 2-byte elements (a float counts as two)
    auto pad = [&](const void *src, void *dst, int64_t rows, int64_t len, int64_t plen) {
        PadList::Entry &e = in.at[in.count++];
        e = {src, dst, (int)(rows * (plen / 8)), (int)len, (int)plen, blocks};
        blocks += (e.vectors + 255) / 256;
    };
    for (size_t l = 0; l < L; ++l) {
        const Geo &g = geos[l];
        const bool on = g.k != g.k_given;
        Cw.push_back(on ? x.C[l] : given.Cw[l]);
        Dw.push_back(on ? x.D[l] : given.Dw[l]);
        G.push_back(on ? x.G[l] : given.G[l]);
        if (train) dg.push_back(on ? x.dg[l] : given.dg_own[l]);
        if (given.dCw) dC.push_back(on ? x.dC[l] : given.dCw[l]);
        if (given.dDw) dD.push_back(on ? x.dD[l] : given.dDw[l]);
        if (update) mC.push_back(on ? x.mC[l] : given.Cw_master[l]);
        if (update) mD.push_back(on ? x.mD[l] : given.Dw_master[l]);
        if (!on) continue;
        pad(given.G[l], x.G[l], g.q * g.B, g.k_given, g.k);
        pad(given.Dw[l], x.D[l], g.q * g.so, g.k_given, g.k);
        pad(given.Cw[l], x.C[l], 1, g.k_given * g.si, g.k * g.si);
        if (train) pad(given.dg_own[l], x.dg[l], g.B, g.k_given, g.k);
        if (update) pad(given.Dw_master[l], x.mD[l], g.q * g.so, 2 * g.k_given, 2 * g.k);
        if (update) pad(given.Cw_master[l], x.mC[l], 1, 2 * g.k_given * g.si, 2 * g.k * g.si);
    }
    {
        ProfScope prof("pad", 0, (int64_t)blocks * 2048, 0, 1, st);
        hipLaunchKernelGGL(pad_kernel, dim3((unsigned)blocks), dim3(256), 0, st, in);
        PH_TRY(check_launch("pad"));
    }
    auto arr = [](auto &v) { return v.empty() ? nullptr : v.data(); };
    ph_step_args a = given;
    a.Cw = Cw.data(); a.Dw = Dw.data(); a.G = G.data(); a.dg_own = arr(dg);
    a.dCw = arr(dC); a.dDw = arr(dD);
    a.Cw_master = arr(mC); a.Dw_master = arr(mD);
    PH_TRY(use_flex(geos, train) ? flex_step<bf16_t>(geos, a, w, st) : step_impl(geos, a, w, st));
    UnpadList out{};
    blocks = 0;
    auto unpad = [&](const float *grad, float *keep, const float *from, float *master, void *weight, int64_t rows, int64_t len, int64_t plen) {
        if (!keep && !update) return;
        UnpadList::Entry &e = out.at[out.count++];
        e = {grad, keep, from, master, weight, (int)(rows * (len / 2)), (int)len, (int)plen, blocks};
        blocks += (e.pairs + 255) / 256;
    };
    for (size_t l = 0; train && l < L; ++l) {
        const Geo &g = geos[l];
        if (g.k == g.k_given) continue;
        unpad(x.dD[l], given.dDw ? given.dDw[l] : nullptr, x.mD[l], update ? given.Dw_master[l] : nullptr, given.Dw[l], g.q * g.so, g.k_given, g.k);
        unpad(x.dC[l], given.dCw ? given.dCw[l] : nullptr, x.mC[l], update ? given.Cw_master[l] : nullptr, given.Cw[l], 1, g.k_given * g.si, g.k * g.si);
    }
    if (out.count == 0) return PH_OK;
    ProfScope prof("D and C from padded rows", 0, (int64_t)blocks * 512, 0, 1, st);
    hipLaunchKernelGGL(unpad_kernel, dim3((unsigned)blocks), dim3(256), 0, st, out);
    return check_launch("D and C from padded rows");
}

ph_status check_ptr_array(const void *const *arr, int L, const char *name)
{
    if (!arr) return fail(PH_ERR_INVALID_ARG, "%s (host array of device pointers) is NULL", name);
    for (int l = 0; l < L; ++l) {
        char nm[64];
        snprintf(nm, sizeof nm, "%s[%d]", name, l);
        PH_TRY(need(arr[l], nm));
    }
    return PH_OK;
}

}  // namespace

extern "C" {

int32_t phantom_abi_version(void) { return 4; }

ph_status phantom_profile_begin(int32_t max_launches)
{
    return without_exceptions([&]() -> ph_status {
        if (max_launches < 1) return fail(PH_ERR_INVALID_ARG, "max_launches = %d must be >= 1", max_launches);
        if (g_prof.on) return fail(PH_ERR_INVALID_ARG, "profiling is already on");
        max_launches += PROF_CALIBRATION_LAUNCHES;
        while (g_prof.ev.size() < (size_t)max_launches * 2) {
            hipEvent_t e;
            hipError_t err = hipEventCreate(&e);
            if (err != hipSuccess) return fail(PH_ERR_LAUNCH, "hipEventCreate: %s", hipGetErrorString(err));
            g_prof.ev.push_back(e);
        }
        g_prof.recs.clear();
        g_prof.cap = (size_t)max_launches;
        g_prof.calibrated = false;
        g_prof.on = true;
        return PH_OK;
    });
}

ph_status phantom_profile_end(ph_profile_entry *entries, int32_t capacity, int32_t *count)
{
    if (!g_prof.on) return fail(PH_ERR_INVALID_ARG, "profiling is not on");
    g_prof.on = false;
    if (!count || (capacity > 0 && !entries)) return fail(PH_ERR_INVALID_ARG, "entries / count is NULL");
    int32_t used = 0;
    for (size_t i = 0; i < g_prof.recs.size(); ++i) {
        const ProfRec &r = g_prof.recs[i];
        hipError_t err = hipEventSynchronize(g_prof.ev[2 * i + 1]);
        float ms = 0.f;
        if (err == hipSuccess) err = hipEventElapsedTime(&ms, g_prof.ev[2 * i], g_prof.ev[2 * i + 1]);
        if (err != hipSuccess) return fail(PH_ERR_LAUNCH, "profile event %zu: %s", i, hipGetErrorString(err));
        int32_t at = -1;
        for (int32_t j = 0; j < used && at < 0; ++j)
            if (!strncmp(entries[j].name, r.name, sizeof entries[j].name - 1) && entries[j].M == r.M &&
                entries[j].N == r.N && entries[j].K == r.K && entries[j].groups == r.groups && entries[j].M2 == r.M2 &&
                entries[j].N2 == r.N2 && entries[j].K2 == r.K2 && entries[j].M3 == r.M3 && entries[j].N3 == r.N3 &&
                entries[j].K3 == r.K3 && entries[j].M4 == r.M4 && entries[j].N4 == r.N4 && entries[j].K4 == r.K4)
                at = j;
        if (at < 0) {
            if (used >= capacity) continue;
            at = used++;
            memset(&entries[at], 0, sizeof entries[at]);
            strncpy(entries[at].name, r.name, sizeof entries[at].name - 1);
            entries[at].M = r.M; entries[at].N = r.N; entries[at].K = r.K; entries[at].groups = r.groups;
            entries[at].M2 = r.M2; entries[at].N2 = r.N2; entries[at].K2 = r.K2;
            entries[at].M3 = r.M3; entries[at].N3 = r.N3; entries[at].K3 = r.K3;
            entries[at].M4 = r.M4; entries[at].N4 = r.N4; entries[at].K4 = r.K4;
        }
        entries[at].calls += 1;
        entries[at].total_ms += ms;
    }
    *count = used;
    return PH_OK;
}

const char *phantom_last_error(void) { return g_err; }

ph_status phantom_workspace_bytes(const ph_problem *prob, size_t *bytes)
{
    return without_exceptions([&]() -> ph_status {
        std::vector<Geo> geos;
        PH_TRY(make_geos(prob, geos));
        if (!bytes) return fail(PH_ERR_INVALID_ARG, "bytes is NULL");
        // the step's layout contains the backward's; a layer's forward needs none
        const std::vector<Geo> padded = padded_geos(prob, geos);
        *bytes = std::max({step_ws_bytes(geos), padded_ws_bytes(padded, false), padded_ws_bytes(padded, true)}) + 256;
        return PH_OK;
    });
}

ph_status phantom_layer_fwd(const ph_problem *prob, const void *X, const void *Lw, const void *Cw, const void *Dw,
                            const void *bias, const void *G, void *Y, void *g_own, void *A_save,
                            void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return without_exceptions([&]() -> ph_status {
        (void)workspace; (void)workspace_bytes;
        Geo g;
        PH_TRY(make_geo(prob, g));
        FwdArgs f{};
        f.X = X; f.Lw = Lw; f.Cw = Cw; f.Dw = Dw; f.bias = bias; f.G = G; f.Y = Y; f.g_own = g_own; f.A_save = A_save;
        PH_TRY(check_fwd_args(g, f));
        f.apart = !g.all && g.q > 0 && overlap(g_own, (size_t)(g.B * g.k) * g.esz, G, (size_t)(g.q * g.B * g.k) * g.esz);
        hipStream_t st = (hipStream_t)hip_stream;
        if (g.dtype == PH_F32) return flex_fwd<float>(g, f, st);
        return use_flex({g}, false, true) ? flex_fwd<bf16_t>(g, f, st) : fwd_impl(g, f, st);
    });
}

ph_status phantom_layer_bwd(const ph_problem *prob, const void *dY, const void *X, const void *A_or_Y,
                            const void *Lw, const void *Cw, const void *Dw, const void *G, void *dg_own,
                            void *dX, float *dLw, float *dCw, float *dDw, float *dbias, void *dG_send,
                            void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return without_exceptions([&]() -> ph_status {
        Geo g;
        PH_TRY(make_geo(prob, g));
        BwdArgs b{};
        b.dY = dY; b.X = X; b.S = A_or_Y; b.Lw = Lw; b.Cw = Cw; b.Dw = Dw; b.G = G; b.dg_own = dg_own; b.dX = dX;
        b.dLw = dLw; b.dCw = dCw; b.dDw = dDw; b.dbias = dbias; b.dG_send = dG_send;
        PH_TRY(check_bwd_args(g, b));
        Arena sizing{nullptr, 0};
        carve_bwd(sizing, g);
        PH_TRY(check_ws(workspace, workspace_bytes, sizing.used));
        Arena a{(char *)workspace, 0};
        BwdWs w = carve_bwd(a, g);
        hipStream_t st = (hipStream_t)hip_stream;
        if (g.dtype == PH_F32) return flex_layer_bwd<float>(g, b, w, st);
        return use_flex({g}, true, true) ? flex_layer_bwd<bf16_t>(g, b, w, st) : bwd_impl(g, b, w, st);
    });
}

}  // extern "C"

namespace {

// The argument checks of a step, all made before any GPU call; `ws_need`: the least bytes of workspace it takes.
ph_status check_step_args(const ph_problem *prob, const ph_step_args *args, std::vector<Geo> &geos, size_t &ws_need)
{
    PH_TRY(make_geos(prob, geos));
    const Geo &g = geos[0];
    if (!args) return fail(PH_ERR_INVALID_ARG, "args is NULL");
    const int L = g.layers;
    if (args->mode < PH_STEP_TRAIN || args->mode > PH_STEP_NO_UPDATE) return fail(PH_ERR_INVALID_ARG, "unknown step mode %d", args->mode);
    const bool train = args->mode != PH_STEP_FORWARD;
    const bool update = args->mode == PH_STEP_TRAIN;
    PH_TRY(need(args->X0, "X0"));
    PH_TRY(check_ptr_array((const void *const *)args->Lw, L, "Lw"));
    PH_TRY(check_ptr_array((const void *const *)args->bias, L, "bias"));
    if (g.q > 0) {
        PH_TRY(check_ptr_array((const void *const *)args->Cw, L, "Cw"));
        PH_TRY(check_ptr_array((const void *const *)args->Dw, L, "Dw"));
        if (!g.all) {
            PH_TRY(check_ptr_array(args->G, L, "G"));
            if (train) PH_TRY(check_ptr_array(args->dg_own, L, "dg_own"));
        }
    }
    PH_TRY(optional(args->Y_out, "Y_out"));
    if (train) {
        PH_TRY(need(args->T, "T"));
        if (!args->loss) return fail(PH_ERR_INVALID_ARG, "loss is NULL");
        if (g.dtype == PH_BF16 && update) {
            PH_TRY(check_ptr_array((const void *const *)args->Lw_master, L, "Lw_master"));
            PH_TRY(check_ptr_array((const void *const *)args->bias_master, L, "bias_master"));
            if (g.q > 0) {
                PH_TRY(check_ptr_array((const void *const *)args->Cw_master, L, "Cw_master"));
                PH_TRY(check_ptr_array((const void *const *)args->Dw_master, L, "Dw_master"));
            }
        }
        if (args->dLw) PH_TRY(check_ptr_array((const void *const *)args->dLw, L, "dLw"));
        if (args->dbias) PH_TRY(check_ptr_array((const void *const *)args->dbias, L, "dbias"));
        if (g.q > 0 && args->dCw) PH_TRY(check_ptr_array((const void *const *)args->dCw, L, "dCw"));
        if (g.q > 0 && args->dDw) PH_TRY(check_ptr_array((const void *const *)args->dDw, L, "dDw"));
    }
    if (args->taps) {
        const ph_step_taps &t = *args->taps;
        const struct { void *const *arr; const char *name; } taps[] = {
            {t.Y, "taps.Y"}, {t.g_own, "taps.g_own"}, {t.delta, "taps.delta"}, {t.dG_send, "taps.dG_send"}, {t.dg_own, "taps.dg_own"}};
        for (const auto &tp : taps)
            for (int l = 0; tp.arr && l < L; ++l) {
                char nm[64];
                snprintf(nm, sizeof nm, "%s[%d]", tp.name, l);
                PH_TRY(optional(tp.arr[l], nm));
            }
    }
    ws_need = step_ws_bytes(geos);
    return PH_OK;
}

// Does Y_out share memory with anything that the step reads: its input, the target, the peers' buffers, the weights?
bool output_overlaps_input(const std::vector<Geo> &geos, const ph_step_args &a)
{
    const Geo &last = geos.back();
    const size_t out_bytes = (size_t)last.groups * last.B * last.so * last.esz;
    auto hits = [&](const void *p, size_t elems) { return overlap(a.Y_out, out_bytes, p, elems * last.esz); };
    const bool train = a.mode != PH_STEP_FORWARD;
    bool any = hits(a.X0, (size_t)geos[0].groups * geos[0].B * geos[0].si) || (train && hits(a.T, out_bytes / last.esz));
    for (size_t l = 0; l < geos.size(); ++l) {
        const Geo &g = geos[l];
        const size_t held = (size_t)g.groups;
        any = any || hits(a.Lw[l], held * g.so * g.si) || hits(a.bias[l], held * g.so);
        if (g.q == 0) continue;
        any = any || hits(a.Cw[l], held * g.k * g.si) || hits(a.Dw[l], held * g.q * g.so * g.k);
        if (!g.all) any = any || hits(a.G[l], (size_t)g.q * g.B * g.k) || (train && hits(a.dg_own[l], (size_t)g.B * g.k));
    }
    return any;
}

// ws_bytes: with less than the padded copies need the step runs on the caller's tensors (include/phantom.h says so).
ph_status run_step(const ph_problem *prob, const std::vector<Geo> &geos, const ph_step_args *args, void *workspace, size_t ws_bytes, void *hip_stream)
{
    const bool forward = args->mode == PH_STEP_FORWARD;
    std::vector<Geo> padded = padded_geos(prob, geos);
    const size_t with_copies = padded_ws_bytes(padded, forward);
    if (with_copies == 0 || with_copies > ws_bytes) padded.clear();
    Arena a{(char *)workspace, 0};
    StepWs w = padded.empty() ? carve_step(a, geos) : carve_step(a, padded, forward);
    hipStream_t st = (hipStream_t)hip_stream;
    // The last layer writes the network output where the caller wants it, unless other workgroups or later launches still
    // read what lies there: then it writes the workspace, and the output is copied when the step is over.
    const bool copy = args->Y_out && output_overlaps_input(geos, *args);
    if (args->Y_out && !copy) w.Y.back() = args->Y_out;
    if (!padded.empty()) PH_TRY(step_on_padded(padded, *args, w, carve_pad(a, padded, forward), st));
    else if (geos[0].dtype == PH_F32) PH_TRY(flex_step<float>(geos, *args, w, st));
    else PH_TRY(use_flex(geos, args->mode != PH_STEP_FORWARD) ? flex_step<bf16_t>(geos, *args, w, st) : step_impl(geos, *args, w, st));
    if (!copy) return PH_OK;
    const Geo &last = geos.back();
    const int64_t count = (int64_t)last.groups * last.B * last.so;
    return last.dtype == PH_F32 ? tap_copy<float>(args->Y_out, w.Y.back(), count, st) : tap_copy<bf16_t>(args->Y_out, w.Y.back(), count, st);
}

// ---- the step for callers that cannot allocate -------------------------------------------------
// Its workspace is this array: device memory that every GPU the library runs on holds from the moment the
// code object is loaded there until the process ends.  In host code the array's name is only a handle:
// the address a kernel can use comes from hipGetSymbolAddress, once per device, with that device current.
constexpr size_t STATIC_WS_BYTES = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_WS_BYTES];

constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES];      // per device; written once under g_scratch_lock
std::mutex g_scratch_lock;

ph_status scratch_of_current_device(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(PH_ERR_LAUNCH, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(PH_ERR_UNSUPPORTED, "device index %d beyond %d", dev, MAX_DEVICES);
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return fail(PH_ERR_LAUNCH, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return PH_OK;
}

}  // namespace

extern "C" {

ph_status phantom_ffn_step(const ph_problem *prob, const ph_step_args *args, void *workspace, size_t workspace_bytes,
                           void *hip_stream)
{
    return without_exceptions([&]() -> ph_status {
        std::vector<Geo> geos;
        size_t ws_need = 0;
        PH_TRY(check_step_args(prob, args, geos, ws_need));
        PH_TRY(check_ws(workspace, workspace_bytes, ws_need));
        return run_step(prob, geos, args, workspace, workspace_bytes, hip_stream);
    });
}

size_t phantom_static_workspace_bytes(void) { return STATIC_WS_BYTES; }

ph_status phantom_ffn_step_static(const ph_problem *prob, const ph_step_args *args, void *hip_stream)
{
    return without_exceptions([&]() -> ph_status {
        std::vector<Geo> geos;
        size_t ws_need = 0;
        PH_TRY(check_step_args(prob, args, geos, ws_need));
        if (ws_need > STATIC_WS_BYTES)
            return fail(PH_ERR_WORKSPACE, "the step needs %zu bytes of workspace, the library's own scratch array holds %zu: "
                                          "use phantom_ffn_step with a workspace of the caller's", ws_need, STATIC_WS_BYTES);
        void *ws = nullptr;
        PH_TRY(scratch_of_current_device(&ws));
        return run_step(prob, geos, args, ws, STATIC_WS_BYTES, hip_stream);
    });
}

}  // extern "C"
