// Internal declarations of libchym (gfx950).  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/chym.h"

namespace chym {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(4))) double f64x4;

// Value of an OCP E4M3 (e4m3fn) byte: sign, 4 exponent bits (bias 7), 3
// mantissa bits; exponent field 0 holds the subnormals m * 2^-9; 0x7f and
// 0xff are NaN (the format has no infinities).
__device__ __forceinline__ float e4m3_value(uint32_t b) {
    const uint32_t mag = b & 0x7fu;
    float v;
    if (mag == 0x7fu)
        v = __builtin_nanf("");
    else if (mag < 8u)
        v = (float)mag * 0x1p-9f;
    else
        v = __uint_as_float((((mag >> 3) + 120u) << 23) | ((mag & 7u) << 20));
    return (b & 0x80u) ? -v : v;
}

// Nearest E4M3 code of a (|a| <= 448 assumed), ties to even; sign from the
// float's sign bit.
__device__ __forceinline__ uint32_t e4m3_code(float v) {
    const uint32_t bits = __float_as_uint(v);
    const uint32_t sign = (bits >> 24) & 0x80u;
    const float a = fabsf(v);
    uint32_t code;
    if (a < 0x1p-6f) {
        // subnormal spacing 2^-9; a * 512 is exact, rintf rounds to even
        code = (uint32_t)rintf(a * 512.0f);  // 8 is the smallest normal, 0x08
    } else {
        const uint32_t ab = __float_as_uint(a);
        int e = (int)(ab >> 23) - 127;
        const uint32_t mant = ab & 0x7fffffu;
        uint32_t m3 = mant >> 20;
        const uint32_t rest = mant & 0xfffffu;
        if (rest > 0x80000u || (rest == 0x80000u && (m3 & 1u))) ++m3;
        if (m3 == 8u) {
            m3 = 0u;
            ++e;
        }
        code = ((uint32_t)(e + 7) << 3) | m3;
    }
    return sign | code;
}

// Least e with amax <= 448 * 2^e (0 for amax = 0): the power-of-two row
// scale that puts a row's largest magnitude at the top E4M3 binade.
__device__ __forceinline__ int e4m3_row_exponent(float amax) {
    if (!(amax > 0.0f)) return 0;
    int k;
    frexpf(amax, &k);  // amax = f 2^k, f in [0.5, 1)
    int e = k - 9;     // 448 * 2^(k - 9) = 0.875 * 2^k: the answer is e or e + 1
    if (amax > ldexpf(448.0f, e)) ++e;
    if (amax <= ldexpf(448.0f, e - 1)) --e;
    return e;
}

// Sparse (ELL) couplings, int32 [n + 1][2 w]: row 0 = {n, w, ...}; row p + 1
// = w columns, then w float32 couplings (bit patterns).
struct EllView {
    const int *rows;
    int w;
    __device__ __forceinline__ const int *row(int p) const { return rows + (size_t)(p + 1) * 2 * w; }
};
// A header that does not describe an n-row matrix reads as no couplings.
__device__ __forceinline__ EllView ell_view(const void *j, int n) {
    const int *h = reinterpret_cast<const int *>(j);
    return EllView{h, (h[0] == n && h[1] > 0) ? h[1] : 0};
}

// Coupling J_pq of an n x n matrix stored as j_dtype, as float (exact for
// every storage type but float32 input, where it is the stored value).
__device__ __forceinline__ float coupling(const void *j, int j_dtype, int n, int p, int q) {
    const size_t i = (size_t)p * n + q;
    switch (j_dtype) {
        case CHYM_J_I8: return (float)reinterpret_cast<const int8_t *>(j)[i];
        case CHYM_J_F32: return reinterpret_cast<const float *>(j)[i];
        case CHYM_J_BF16: return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(j)[i] << 16);
        default: {
            const uint8_t *b = reinterpret_cast<const uint8_t *>(j);
            const uint32_t e = b[(size_t)n * n + p];
            if (e == 0xffu) return __builtin_nanf("");
            return ldexpf(e4m3_value(b[i]), (int)e - 127);
        }
    }
}

// The couplings J[p][q .. q+3], all inside the n x n matrix, as float: one load
// of 4, 8 or 16 bytes at the element alignment.
__device__ __forceinline__ void coupling4_inside(const void *j, int j_dtype, int n, int p, int q, float (&v)[4]) {
    const size_t i = (size_t)p * n + q;
    switch (j_dtype) {
        case CHYM_J_I8: {
            uint32_t b;
            __builtin_memcpy(&b, reinterpret_cast<const int8_t *>(j) + i, 4);
#pragma unroll
            for (int s = 0; s < 4; ++s) v[s] = (float)(int8_t)(b >> (8 * s));
            break;
        }
        case CHYM_J_F32: {
            __builtin_memcpy(v, reinterpret_cast<const float *>(j) + i, 16);
            break;
        }
        case CHYM_J_BF16: {
            uint32_t b[2];
            __builtin_memcpy(b, reinterpret_cast<const uint16_t *>(j) + i, 8);
#pragma unroll
            for (int s = 0; s < 4; ++s) v[s] = __uint_as_float((s & 1) ? b[s >> 1] & 0xffff0000u : b[s >> 1] << 16);
            break;
        }
        default: {
            const uint8_t *j8 = reinterpret_cast<const uint8_t *>(j);
            const uint32_t e = j8[(size_t)n * n + p];
            uint32_t b;
            __builtin_memcpy(&b, j8 + i, 4);
#pragma unroll
            for (int s = 0; s < 4; ++s)
                v[s] = e == 0xffu ? __builtin_nanf("") : ldexpf(e4m3_value((b >> (8 * s)) & 0xffu), (int)e - 127);
        }
    }
}

// The same with 0 outside the matrix; the last columns of a row are read one
// by one.
__device__ __forceinline__ void coupling4(const void *j, int j_dtype, int n, int p, int q, float (&v)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = 0.0f;
    if (p >= n || q >= n) return;
    if (q + 3 < n) {
        coupling4_inside(j, j_dtype, n, p, q, v);
        return;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (q + s < n) v[s] = coupling(j, j_dtype, n, p, q + s);
}

// Largest row-tile count (16 rows per tile) of the register-resident
// integrator for d components, xs state terms and js J terms (0 if none).
int resident_tile_limit(int d, int xs, int js);

// Values read from a table in memory at an index that is the same in the whole
// wavefront: in scalar registers, and a pointer known to point to global
// memory.  Without the latter its accesses are flat ones, which count as LDS
// accesses too: a wait for LDS also waits for them, and they for it (400 steps
// of the team integrator at N = 75, D = 4, float couplings: 0.85 ms per solve
// with flat accesses, 0.66 without).
__device__ __forceinline__ int in_wave(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float in_wave(float v) { return __int_as_float(in_wave(__float_as_int(v))); }
template <typename T>
__device__ __forceinline__ T *in_wave(T *p) {
    const uint64_t v = (uint64_t)p;
    const uint64_t u = (uint64_t)(uint32_t)in_wave((int)(v >> 32)) << 32 | (uint32_t)in_wave((int)v);
    return (T *)(__attribute__((address_space(1))) T *)u;
}

// Arguments of one integration launch (one problem, one replica block).
struct IntegArgs {
    const void *j;
    const float *pump;
    float *x;
    const float *alpha;
    int32_t n, d, r, steps, start_step, j_dtype;
    float eps, btil, eta, dt;
    // round-trip map form only: kappa L of the medium, and the constant part
    // (1 - loss)(1 - b) of the per-round-trip factor
    float kl, c0;
};

__device__ __forceinline__ IntegArgs in_wave(const IntegArgs &t) {
    IntegArgs a;
    a.j = in_wave(t.j);
    a.pump = in_wave(t.pump);
    a.x = in_wave(t.x);
    a.alpha = in_wave(t.alpha);
    a.n = in_wave(t.n);
    a.d = in_wave(t.d);
    a.r = in_wave(t.r);
    a.steps = in_wave(t.steps);
    a.start_step = in_wave(t.start_step);
    a.j_dtype = in_wave(t.j_dtype);
    a.eps = in_wave(t.eps);
    a.btil = in_wave(t.btil);
    a.eta = in_wave(t.eta);
    a.dt = in_wave(t.dt);
    a.kl = in_wave(t.kl);
    a.c0 = in_wave(t.c0);
    return a;
}

// The most blocks of one launch: HIP takes fewer than 2^32 threads in a
// dimension, and cuts a larger grid short without an error.
constexpr int max_blocks(int threads) { return (int)((1ll << 31) / threads); }

// Host-side launcher of the resident integrator for one (tiles, d, xs, js)
// variant; returns hipSuccess or the launch error.
hipError_t launch_integrate(int tiles, int d, int xs, int js, int waves_per_block,
                            const IntegArgs &a, hipStream_t stream, bool *supported);
// The round-trip map form (single coupling term only) runs up to this many row
// tiles.
constexpr int kMapMaxTiles = 7;
bool integrate_variant_exists(int tiles, int d, int xs, int js);
// Team integrator (a problem's row tiles spread over the wavefronts of a
// block): the layout to take for `blocks` packed blocks, that is `waves` groups
// of 16 replicas, on a GPU of cus compute units, or kTeamNone where another
// integrator is faster.  tuned: the other integrator is a plan that the
// autotuner chose (a register-resident variant's; else the default one).
constexpr int kTeamNone = 0;
constexpr int kTeamPack = 1;   // 16 columns per block
constexpr int kTeamPlane = 2;  // 16 replicas x d planes per block
int team_layout(int tiles, int d, int xs, int js, int64_t blocks, int64_t waves, bool map, bool tuned, int cus);
// Replicas per block of a layout (0 for kTeamNone).
int team_block_replicas(int layout, int d);
// Rough time of one step of a batch's item, in us.
double dense_step_us(int n, int xs, int js, bool slab);
double sparse_step_us(int n, int lrb);
// One problem (items = NULL, `blocks` of its replica blocks), or n blocks'
// items (task, replica block) of many problems of one shape.
hipError_t launch_integrate_team(int layout, int tiles, int d, int xs, int js, bool map, int blocks,
                                 const IntegArgs &one, const IntegArgs *tasks, const int2 *items, hipStream_t stream);
// Persistent kernel kinds: J gathered into each wavefront's registers, work
// items of 16 replicas; or J staged in LDS per block, work items of
// 16 * waves_per_block replicas.
constexpr int kKernelRegJ = 0;
constexpr int kKernelLdsJ = 1;   // two wavefronts per SIMD
constexpr int kKernelLdsJ1 = 2;  // one wavefront per SIMD
constexpr int kKernelPipe = 3;   // one wavefront per SIMD, update and split interleaved with the products
constexpr int kKernelLdsJ3 = 4;  // three wavefronts per SIMD
// Whether a persistent kernel of this kind is built for the shape (the
// pipelined kind exists for some shapes only).
bool persistent_kind_exists(int tiles, int d, int xs, int js, int kind);
hipError_t persistent_occupancy(int tiles, int d, int xs, int js, int kind, int waves_per_block, int *blocks_per_cu);
hipError_t launch_zero_counters(int *counters, int n, hipStream_t stream);
// FP8 (E4M3 + per-row power-of-two) packing of a float32 coupling matrix.
hipError_t launch_quantize_fp8(int n, const float *j, uint8_t *out, hipStream_t stream);
// Sparse (ELL) couplings: whether the gather integrator takes n and d, its
// replicas per block (log2) where r replicas run on cus compute units, and its
// launch.
bool ell_takes(int n, int d);
int ell_lrb(int n, int d, int64_t r, int cus);
hipError_t launch_integrate_ell(const IntegArgs &a, int cus, hipStream_t stream);
// LDS bytes of one block; the persistent form over many problems of one d
// (items: task, 8 x replica block + log2 of its replicas), launched with the
// largest LDS size of its items.
size_t ell_lds_bytes(int n, int d, int lrb);
hipError_t ell_persistent_occupancy(int d, size_t lds, int *blocks_per_cu);
hipError_t launch_integrate_ell_persistent(int d, int blocks, size_t lds, const IntegArgs *tasks, const int2 *items,
                                           int n_items, int *counter, hipStream_t stream);
// Synthetic timing problem for the autotuner.
hipError_t launch_fill_probe(void *j, int j_dtype, int n, float *pump, int r, float *alpha, int na,
                             hipStream_t stream);
hipError_t launch_fill_state(float *x, size_t nx, hipStream_t stream);
hipError_t launch_split3(const float *x, int64_t n, uint16_t *hi, uint16_t *mid, uint16_t *lo, hipStream_t stream);
// Persistent launch over a work list: items[i] = (task index, replica slab).
hipError_t launch_integrate_persistent(int tiles, int d, int xs, int js, int kind, int waves_per_block, int blocks,
                                       const IntegArgs *tasks, const int2 *items, int n_items, int *counter,
                                       hipStream_t stream);

// Per-task arguments of the batched scoring kernels.
struct ScoreArgs {
    const float *x;
    const void *j;
    uint64_t *spins;
    int32_t *e_i32;
    double *e_f64;
    double *e_hs;
    double *extra;
    uint8_t *diverged;
    int32_t n, d, r, j_dtype;
};

__device__ __forceinline__ ScoreArgs in_wave(const ScoreArgs &t) {
    ScoreArgs a;
    a.x = in_wave(t.x);
    a.j = in_wave(t.j);
    a.spins = in_wave(t.spins);
    a.e_i32 = in_wave(t.e_i32);
    a.e_f64 = in_wave(t.e_f64);
    a.e_hs = in_wave(t.e_hs);
    a.extra = in_wave(t.extra);
    a.diverged = in_wave(t.diverged);
    a.n = in_wave(t.n);
    a.d = in_wave(t.d);
    a.r = in_wave(t.r);
    a.j_dtype = in_wave(t.j_dtype);
    return a;
}

// LDS one block needs for a task's float64 energies: the Ising energy of
// couplings other than int8 (0 where it needs none), the hyperspin energy.
size_t ising_score_lds(int n, int j_dtype);
size_t hs_score_lds(int n, int d, int j_dtype);
// Readout, Ising energy and hyperspin energy of every replica of every task
// (first = replica prefix table, first[n_tasks] = total_replicas); ising_lds
// and hs_lds: the largest of the above over the tasks that want the energy.
hipError_t launch_score_batched(const ScoreArgs *tasks, const int64_t *first, int n_tasks, int64_t total_replicas,
                                size_t ising_lds, size_t hs_lds, bool any_readout, bool any_ising, bool any_hs,
                                int cus, hipStream_t stream);

// Streamed-J slab integrator (large n).  Tiles of 16 rows; kSlabMaxLds
// bounds the LDS operand area of one column slab (beyond it the float32 form
// holds one component at a time and makes d passes over J per step).
constexpr size_t kSlabMaxLds = 159 * 1024;  // 160 KiB per CU, less room for static LDS
// Blocks of eight or sixteen wavefronts (kSlabWaves8, kSlabWaves16); the
// sixteen-wavefront shapes are built for the bf16 form, up to 32 tiles (64
// at d <= 2).
constexpr int kSlabWaves8 = 8;
constexpr int kSlabWaves16 = 16;
int slab_tpw_for(int tiles, int waves);
size_t slab_lds_bytes(int tiles, int d, int xs);
size_t slab_jfrag_bytes(int tiles, int js);
bool slab_variant_exists(int tiles, int d, int xs, int js);  // the eight-wavefront shape
bool slab_shape_exists(int tiles, int d, int xs, int js, int waves);
// narrow: couplings in one term may be staged as E2M1 or E4M3 codes (else
// bf16), in quads, for the packed streamed-J integrator.
hipError_t launch_stage_jfrag(const IntegArgs &a, int js, bool narrow, void *out, hipStream_t stream);
// Stages the couplings of the tasks list[0 .. n) of a batch (all with js
// coupling terms) into stages[task], ncps[task] chunks each, narrow ones in
// quads or not; tasks, list, ncps and stages are device arrays.
hipError_t launch_stage_batched(int js, bool quads, const IntegArgs *tasks, const int *list, int n, const int *ncps,
                                unsigned char *const *stages, hipStream_t stream);
hipError_t launch_integrate_slab(int tiles, int d, int xs, int js, int waves, const IntegArgs &a, const void *jfrag,
                                 hipStream_t stream);
hipError_t slab_occupancy(int tiles, int d, int xs, int js, int waves, size_t lds, int *blocks_per_cu);
hipError_t launch_integrate_slab_persistent(int tiles, int d, int xs, int js, int waves, size_t lds, int blocks,
                                            const IntegArgs *tasks, const int2 *items, int n_items, int *counter,
                                            const void *const *jfs, const int *ncps, hipStream_t stream);

// Packed streamed-J integrator (16 columns per block), for launches of few
// replicas: whether it takes `blocks` packed blocks on cus compute units
// (narrow: the couplings are stored in eight bits; batch: in one batch group),
// and the launches: of one problem staged at `stage`, and of items of many
// problems of any D with one shape (row tiles per wavefront), lds the largest
// spack_lds among them.
bool spack_takes(int tiles, int d, int xs, int js, bool narrow, int64_t blocks, bool batch, int cus);
int spack_shape(int tiles);
size_t spack_lds(int tiles, int xs);
hipError_t launch_integrate_spack(int tiles, int d, int xs, int js, int blocks, const IntegArgs &a, const void *stage,
                                  hipStream_t stream);
hipError_t launch_integrate_spack_batch(int shape, int xs, int js, size_t lds, int blocks, const IntegArgs *tasks,
                                        const int2 *items, const void *const *stages, hipStream_t stream);

// Learned early restart: trajectory features and the MLP.
hipError_t launch_features(int n, int d, int r, const void *j, int j_dtype, const float *x, uint64_t *prev,
                           float *feat, int feat_stride, int feat_off, hipStream_t stream);
hipError_t launch_sign_words(int n, int d, int r, const float *x, uint64_t *words, hipStream_t stream);
hipError_t launch_standardize(int groups, int group, const float *in, float *out, hipStream_t stream);
hipError_t launch_select_top(int groups, int group, int keep, const float *score, int32_t *idx, hipStream_t stream);
hipError_t launch_gather_replicas(int n, int d, int r_src, const float *x_src, const float *pump_src, int m,
                                  const int32_t *idx, float *x_dst, float *pump_dst, hipStream_t stream);
int mlp_param_count();
size_t mlp_backward_scratch_floats(int batch);
hipError_t launch_mlp_forward(int batch, const float *feat, const void *wb, float *logit, float *h1, float *h2,
                              hipStream_t stream);
hipError_t launch_mlp_backward(int batch, const float *feat, const float *label, const void *wb, const float *logit,
                               const float *h1, const float *h2, float *scratch, float *grad, float *loss,
                               hipStream_t stream);
hipError_t launch_mlp_adam(float *wm, void *wb, float *m, float *v, const float *grad, float lr, float b1, float b2,
                           float eps, int t, hipStream_t stream);
hipError_t launch_to_bf16(const float *src, void *dst, int n, hipStream_t stream);

hipError_t launch_readout(int n, int d, int r, const float *x, uint64_t *spins, double *extra,
                          uint8_t *diverged, hipStream_t stream);
hipError_t launch_ising_energy(int n, int r, const void *j, int j_dtype, const uint64_t *spins,
                               int32_t *e_i32, double *e_f64, hipStream_t stream);
hipError_t launch_hs_energy(int n, int d, int r, const void *j, int j_dtype, const float *x,
                            double *e_hs, hipStream_t stream);

}  // namespace chym
