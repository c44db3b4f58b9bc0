// Host-side dispatch of the register-resident integrator variants.
#include <algorithm>

#include "integrate_slab.h"
#include "integrate_spack.h"

namespace chym {

typedef KernelSet KernelFn;

static KernelFn lookup(int tiles, int d, int xs, int js) {
#define CHYM_PICK(D, XS, JS) \
    if (d == D && xs == XS && js == JS) return lookup_resident_##D##_##XS##_##JS(tiles);
    CHYM_PICK(1, 3, 1) CHYM_PICK(1, 1, 1) CHYM_PICK(1, 3, 3)
    CHYM_PICK(2, 3, 1) CHYM_PICK(2, 1, 1) CHYM_PICK(2, 3, 3)
    CHYM_PICK(3, 3, 1) CHYM_PICK(3, 1, 1) CHYM_PICK(3, 3, 3)
    CHYM_PICK(4, 3, 1) CHYM_PICK(4, 1, 1) CHYM_PICK(4, 3, 3)
#undef CHYM_PICK
    return KernelSet{nullptr, nullptr, nullptr, nullptr, 0, nullptr, nullptr};
}

int resident_tile_limit(int d, int xs, int js) {
    return (d >= 1 && d <= 4) ? resident_max_tiles(d, xs, js) : 0;
}

// ------------------------------------------------------------ slab kernels
static SlabKernels lookup_slab_shape(int tpw, int waves, int d, int xs, int js, bool cp) {
#define CHYM_PICK(D, XS, JS) \
    if (d == D && xs == XS && js == JS) return lookup_slab_##D##_##XS##_##JS(tpw, waves, cp);
    CHYM_PICK(1, 3, 1) CHYM_PICK(1, 1, 1) CHYM_PICK(1, 3, 3)
    CHYM_PICK(2, 3, 1) CHYM_PICK(2, 1, 1) CHYM_PICK(2, 3, 3)
    CHYM_PICK(3, 3, 1) CHYM_PICK(3, 1, 1) CHYM_PICK(3, 3, 3)
    CHYM_PICK(4, 3, 1) CHYM_PICK(4, 1, 1) CHYM_PICK(4, 3, 3)
#undef CHYM_PICK
    return SlabKernels{nullptr, nullptr, 0};
}

// Tiles per wavefront of the slab kernel for a tile count and block size
// (eight or sixteen wavefronts); 0 when no shape holds that many tiles.
int slab_tpw_for(int tiles, int waves) {
    const int per = (tiles + waves - 1) / waves;
    if (waves == 8) return per <= 4 ? 4 : (per <= 8 ? 8 : 0);
    if (waves == 16) return per <= 1 ? 1 : (per <= 2 ? 2 : (per <= 4 ? 4 : 0));
    return 0;
}

// The float32 form takes component passes where the operand of all d
// components exceeds the LDS budget (the bf16 form's always fits).
static bool slab_component_passes(int tiles, int d, int xs) {
    return xs == 3 && d > 1 && (size_t)((tiles + 1) / 2) * d * xs * 64 * sizeof(bf16x8) > kSlabMaxLds;
}

static SlabKernels lookup_slab(int tiles, int d, int xs, int js, int waves) {
    const int tpw = slab_tpw_for(tiles, waves);
    if (tpw == 0) return SlabKernels{nullptr, nullptr, 0};
    return lookup_slab_shape(tpw, waves, d, xs, js, slab_component_passes(tiles, d, xs));
}

size_t slab_lds_bytes(int tiles, int d, int xs) {
    const int dp = slab_component_passes(tiles, d, xs) ? 1 : d;
    return (size_t)((tiles + 1) / 2) * dp * xs * 64 * sizeof(bf16x8);
}

// The fragments, plus kSlabRingChunks chunks of padding: the streamed-J
// kernel's prefetch ring refills unconditionally, so around the last tile it
// loads (and discards) up to that many chunks past the staged data.  Their
// offsets travel in the scalar operand of the buffer load, which the range
// check of the buffer resource does not cover; the padding keeps those loads
// inside the workspace.
size_t slab_jfrag_bytes(int tiles, int js) {
    return stage_frag_offset(tiles) + ((size_t)tiles * ((tiles + 1) / 2) + kSlabRingChunks) * js * 64 * sizeof(bf16x8);
}

bool slab_variant_exists(int tiles, int d, int xs, int js) { return slab_shape_exists(tiles, d, xs, js, 8); }

bool slab_shape_exists(int tiles, int d, int xs, int js, int waves) {
    return slab_lds_bytes(tiles, d, xs) <= kSlabMaxLds && lookup_slab(tiles, d, xs, js, waves).single != nullptr;
}

// Decides the staging format of the couplings, checked element by element:
// E2M1 codes when every coupling is -1, 0 or +1; else E4M3 bytes when every
// row is a set of E4M3 values times one power of two (the row scale, chosen
// as in the FP8 quantizer; FP8 storage always qualifies); else bf16.  A launch
// sets the header's flags, then blocks of four rows, one per wavefront, clear
// them and write the row scales.  (One block per task that walked all its rows
// took 586 us for 75 tasks of N = 50 - 800; now 17 us.)
__device__ __forceinline__ void stage_prep_row(const IntegArgs &a, int p, unsigned char *__restrict__ stage) {
    int *flags = reinterpret_cast<int *>(stage);
    float *scale = reinterpret_cast<float *>(stage + kStageHeader);
    const int lane = threadIdx.x & 63;
    const int n = a.n;
    bool ok = true, pm1 = true;
    float sc = 1.0f;
    if (p < n) {
        if (a.j_dtype == CHYM_J_FP8) {
            const uint32_t e = reinterpret_cast<const uint8_t *>(a.j)[(size_t)n * n + p];
            sc = e == 0xffu ? __builtin_nanf("") : ldexpf(1.0f, (int)e - 127);
            for (int q = lane; q < n; q += 64) {
                const float v = coupling(a.j, a.j_dtype, n, p, q);
                if (!(v == 0.0f || v == 1.0f || v == -1.0f)) pm1 = false;
            }
        } else {
            float amax = 0.0f;
            bool fin = true;
            for (int q = lane; q < n; q += 64) {
                const float v = coupling(a.j, a.j_dtype, n, p, q);
                fin = fin && __builtin_isfinite(v);
                amax = fmaxf(amax, fabsf(v));
                if (!(v == 0.0f || v == 1.0f || v == -1.0f)) pm1 = false;
            }
            for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
            const int e = e4m3_row_exponent(amax);
            if (!__all(fin) || e < -126 || e > 127) {
                ok = false;
            } else {
                sc = ldexpf(1.0f, e);
                for (int q = lane; q < n; q += 64) {
                    const float v = coupling(a.j, a.j_dtype, n, p, q);
                    if (ldexpf(e4m3_value(e4m3_code(ldexpf(v, -e))), e) != v) ok = false;
                }
            }
        }
    }
    ok = __all(ok);
    pm1 = __all(pm1);
    if (lane == 0) {
        scale[p] = sc;
        if (!pm1) atomicAnd(&flags[0], 0);
        if (!ok) atomicAnd(&flags[1], 0);
    }
}

// Header flags of n stagings: both set (the row pass clears what does not
// hold), or both clear (bf16 fragments).
__global__ void k_stage_header(const int *__restrict__ list, int n, unsigned char *const *__restrict__ stages,
                               unsigned char *__restrict__ one, int value) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int *flags = reinterpret_cast<int *>(one ? one : stages[list[i]]);
    flags[0] = value;
    flags[1] = value;
}

__global__ __launch_bounds__(256) void k_stage_prep(IntegArgs a, unsigned char *__restrict__ stage) {
    const int p = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (p < (a.n + 15) / 16 * 16) stage_prep_row(a, p, stage);
}

// The same for the tasks list[0 .. n) of a batch, bpt blocks each.
__global__ __launch_bounds__(256) void k_stage_prep_batched(const IntegArgs *__restrict__ tasks,
                                                            const int *__restrict__ list, int bpt,
                                                            unsigned char *const *__restrict__ stages) {
    const int t = list[blockIdx.x / bpt];
    const IntegArgs a = in_wave(tasks[t]);
    const int rows = (a.n + 15) / 16 * 16;
    for (int p = (blockIdx.x % bpt) * 4 + (threadIdx.x >> 6); p < rows; p += 4 * bpt) stage_prep_row(a, p, in_wave(stages[t]));
}

constexpr int kStageBlocksPerTask = 32;  // 128 rows at a time; 8192 threads share a task's fragment slots

hipError_t launch_stage_batched(int js, bool quads, const IntegArgs *tasks, const int *list, int n, const int *ncps,
                                unsigned char *const *stages, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    if (js == 3) {
        hipLaunchKernelGGL(k_stage_jfrag_batched<3>, dim3(n * kStageBlocksPerTask), dim3(256), 0, stream, tasks, list,
                           kStageBlocksPerTask, ncps, quads, stages);
    } else {
        hipLaunchKernelGGL(k_stage_header, dim3((n + 255) / 256), dim3(256), 0, stream, list, n, stages,
                           (unsigned char *)nullptr, 1);
        hipLaunchKernelGGL(k_stage_prep_batched, dim3(n * kStageBlocksPerTask), dim3(256), 0, stream, tasks, list,
                           kStageBlocksPerTask, stages);
        hipLaunchKernelGGL(k_stage_jfrag_batched<1>, dim3(n * kStageBlocksPerTask), dim3(256), 0, stream, tasks, list,
                           kStageBlocksPerTask, ncps, quads, stages);
    }
    return hipGetLastError();
}

hipError_t launch_stage_jfrag(const IntegArgs &a, int js, bool narrow, void *out, hipStream_t stream) {
    const bool quads = narrow;  // the packed kernel alone takes the narrow formats of a single problem
    const int nt = (a.n + 15) / 16;
    const int ncp = (nt + 1) / 2;
    const int total = nt * ncp * 64;
    const int grid = (total + 255) / 256;
    unsigned char *stage = reinterpret_cast<unsigned char *>(out);
    if (js == 3) {
        hipLaunchKernelGGL(k_stage_jfrag<3>, dim3(grid), dim3(256), 0, stream, a, ncp, quads, stage);
    } else {
        hipLaunchKernelGGL(k_stage_header, dim3(1), dim3(64), 0, stream, (const int *)nullptr, 1,
                           (unsigned char *const *)nullptr, stage, narrow ? 1 : 0);
        if (narrow) hipLaunchKernelGGL(k_stage_prep, dim3(nt * 4), dim3(256), 0, stream, a, stage);
        hipLaunchKernelGGL(k_stage_jfrag<1>, dim3(grid), dim3(256), 0, stream, a, ncp, quads, stage);
    }
    return hipGetLastError();
}

static hipError_t slab_prepare(const void *fn, size_t lds) {
    if (lds <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

hipError_t launch_integrate_slab(int tiles, int d, int xs, int js, int waves, const IntegArgs &a, const void *jfrag,
                                 hipStream_t stream) {
    SlabKernels k = lookup_slab(tiles, d, xs, js, waves);
    if (!k.single) return hipErrorInvalidDeviceFunction;
    const size_t lds = slab_lds_bytes(tiles, d, xs);
    hipError_t e = slab_prepare(reinterpret_cast<const void *>(k.single), lds);
    if (e != hipSuccess) return e;
    const int blocks = (a.r + 15) / 16;
    hipLaunchKernelGGL(k.single, dim3(blocks), dim3(64 * k.waves), lds, stream, a,
                       reinterpret_cast<const unsigned char *>(jfrag),
                       (tiles + 1) / 2);
    return hipGetLastError();
}

hipError_t slab_occupancy(int tiles, int d, int xs, int js, int waves, size_t lds, int *blocks_per_cu) {
    *blocks_per_cu = 0;
    SlabKernels k = lookup_slab(tiles, d, xs, js, waves);
    if (!k.persistent) return hipErrorInvalidDeviceFunction;
    hipError_t e = slab_prepare(reinterpret_cast<const void *>(k.persistent), lds);
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k.persistent, 64 * k.waves, lds);
}

hipError_t launch_integrate_slab_persistent(int tiles, int d, int xs, int js, int waves, size_t lds, int blocks,
                                            const IntegArgs *tasks, const int2 *items, int n_items, int *counter,
                                            const void *const *jfs, const int *ncps, hipStream_t stream) {
    SlabKernels k = lookup_slab(tiles, d, xs, js, waves);
    if (!k.persistent) return hipErrorInvalidDeviceFunction;
    hipError_t e = slab_prepare(reinterpret_cast<const void *>(k.persistent), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k.persistent, dim3(blocks), dim3(64 * k.waves), lds, stream, tasks, items, n_items, counter,
                       reinterpret_cast<const unsigned char *const *>(jfs), ncps);
    return hipGetLastError();
}

// ------------------------------------------------------------ team kernels
static TeamFn lookup_team(int tiles, int d, int xs, int js, bool pack, bool map) {
    if (tiles < 1 || tiles > kTeamMaxTiles) return nullptr;
    switch (d) {
        case 1: return lookup_team_1(tiles, xs, js, pack, map);
        case 2: return lookup_team_2(tiles, xs, js, pack, map);
        case 3: return lookup_team_3(tiles, xs, js, pack, map);
        case 4: return lookup_team_4(tiles, xs, js, pack, map);
        default: return nullptr;
    }
}

// Which integrator for r replicas.  Measured per step (us), +-1 couplings,
// 256 CUs; "wave" is one wavefront per 16 replicas (the register-resident
// kernel, 1024 SIMDs hold 16384 replicas), "slab" the streamed-J kernel:
//   N = 100, D = 3, f32    16 replicas: packed 0.52, plane 1.24, wave 3.18
//                          2048: 0.88, 1.33, 3.25    8192: 2.8, 2.1, 3.3
//                          16384: 5.3, 4.1, 3.7      20000: 6.8, 5.2, 6.8
//   N = 100, D = 2, f32    2048: 0.54, 0.97, 2.38    16384: 2.50, 2.69, 2.54
//   N = 100, D = 4, f32    2048: 0.93, 1.66, 4.23    8192: 2.96, 3.43, 4.37
//   N = 200, D = 3, bf16   1024: packed 0.63, plane 1.09, slab 1.44
//                          20000: 11.6, 6.1, 8.2
// Packed blocks have the shortest step, and are the fastest up to two of them
// on a CU (four with two chunks, eight with one, and twice as many for the map,
// whose steps hold more vector work).  Beyond that the plane layout is faster
// where the packed one idles a column (D = 3) or where the quad sums weigh more
// than the operand exchange (bf16); otherwise packed blocks stay level with it,
// and no plane kernel is built.  Against one wavefront per 16 replicas both
// lose once those fill the SIMDs: the wave's time goes up in steps of 16384
// replicas, the team's in proportion, so the line is drawn at 0.9 of a full
// step (0.7 with three wavefronts on four SIMDs; 0.6 of the first against a
// tuned plan, which overlaps two or three wavefronts per SIMD at full load).
// The map takes the team at every size: the medium's gain is vector work, which
// one wavefront per SIMD cannot overlap with its products (N = 100, D = 3,
// 65536 replicas: 28.2 us a step, plane 23.4).  Against the streamed-J kernel
// both layouts win at every replica count, except where the plane layout's
// operand does not fit LDS twice (float32 at D = 4 beyond 12 tiles) and J is
// one term: there packed blocks are 5-10% slower beyond two to a CU.
int team_layout(int tiles, int d, int xs, int js, int64_t blocks, int64_t waves, bool map, bool tuned, int cus) {
    if (!lookup_team(tiles, d, xs, js, true, map)) return kTeamNone;
    const int nc = (tiles + 1) / 2;
    const bool wave = map ? tiles <= kMapMaxTiles : tiles <= resident_tile_limit(d, xs, js);
    // D = 1, N <= 32: the same work in the same single wavefront, in blocks of one
    // or, in the register-resident kernel, of four.  With one state term blocks of
    // one are faster at every count (400 steps, 4096 replicas: N = 16 36 against 54
    // us, N = 32 52 against 62; 16384: 38 and 54, 55 and 64; 131072: 135 and 150,
    // 269 and 285); with three they are no faster where it matters most, N = 32 and
    // one wavefront per SIMD (104 against 94 us; 87 against 92 below).
    if (nc == 1 && d == 1 && xs == 3 && !map) return kTeamNone;
    if (wave && !map && (nc > 1 || tuned)) {
        const int64_t full = (int64_t)4 * cus;
        const int64_t steps = tuned ? 1 : (waves + full - 1) / full;
        if (10 * waves > (tuned ? 6 : nc == 3 ? 7 : 9) * steps * full) return kTeamNone;
    }
    const int64_t per_cu = (blocks + cus - 1) / cus;
    if (per_cu <= (nc == 1 ? 8 : nc == 2 ? 4 : 2) * (map ? 2 : 1)) return kTeamPack;
    if (!wave && js == 1 && team_lds_bytes(nc, d, xs, false) > kSlabMaxLds) return kTeamNone;
    return lookup_team(tiles, d, xs, js, false, map) ? kTeamPlane : kTeamPack;
}

// From what was measured at N = 100 to 800: 0.3 us, and 2.2e-5 n^2 on the slab
// kernel, 1e-5 n^2 on the other dense ones, twice and four times that for three
// state terms with one and three coupling terms.
double dense_step_us(int n, int xs, int js, bool slab) {
    const double terms = js == 3 ? 4.0 : xs == 3 ? 2.0 : 1.0;
    return 0.3 + terms * (slab ? 2.2e-5 : 1e-5) * n * n;
}

// The gather integrator's step goes with the block's units, n for each of its
// 2^lrb replicas (N = 800, four replicas 0.9 us, N = 200, D = 1, two 0.23 us).
// Measured on 3-regular rows: the width of a task's rows lies in its couplings,
// in device memory, and wide rows take longer (20% rows at N = 200: 13 us).
double sparse_step_us(int n, int lrb) { return 0.2 + 2.5e-4 * ((int64_t)n << lrb); }

int team_block_replicas(int layout, int d) { return layout == kTeamNone ? 0 : team_replicas(d, layout == kTeamPack); }

hipError_t launch_integrate_team(int layout, int tiles, int d, int xs, int js, bool map, int blocks,
                                 const IntegArgs &one, const IntegArgs *tasks, const int2 *items, hipStream_t stream) {
    const bool pack = layout == kTeamPack;
    TeamFn fn = lookup_team(tiles, d, xs, js, pack, map);
    if (!fn) return hipErrorInvalidDeviceFunction;
    const int nc = (tiles + 1) / 2;
    const size_t lds = team_lds_bytes(nc, d, xs, pack);
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const int threads = 64 * team_waves(nc, team_tiles(tiles, xs, pack));
    for (int first = 0; first < blocks; first += max_blocks(threads))
        hipLaunchKernelGGL(fn, dim3(std::min(blocks - first, max_blocks(threads))), dim3(threads), lds, stream, one, first,
                           tasks, items ? items + first : nullptr);
    return hipGetLastError();
}

// ------------------------------------------------- packed streamed-J kernels
static SpackFn lookup_spack(int tpw, int d, int xs, int js) {
    switch (d) {
        case 1: return lookup_spack_1(tpw, xs, js);
        case 2: return lookup_spack_2(tpw, xs, js);
        case 3: return lookup_spack_3(tpw, xs, js);
        case 4: return lookup_spack_4(tpw, xs, js);
        default: return nullptr;
    }
}

int spack_shape(int tiles) { return spack_tiles_per_wave(tiles); }
size_t spack_lds(int tiles, int xs) { return spack_lds_bytes((tiles + 1) / 2, xs); }

// Where the packed kernel is faster than the slab kernel (one problem, slab
// time / packed time, at N = 260, 512, 800, 1000; +-1 couplings are "narrow"):
//                                packed blocks per CU    0.25 - 1            2
//   three state terms, D = 4, narrow          1.9 - 2.1, 3.9 - 4.5,    1.0, 2.1,
//                                             4.1 - 5.2, 4.0 - 5.0     2.1, 2.1
//   the same, D = 2                           1.4 - 1.6, 1.6 - 1.7,    0.8, 0.9,
//                                             1.8 - 2.0, 2.0 - 2.2     1.0, 1.1
//   three coupling terms, D = 4               1.3 - 1.6, 2.9 - 3.7,    0.7, 1.5,
//                                             2.9 - 3.6, 3.4 - 4.0     1.4, 1.7
//   the same, D = 1                           1.0 - 1.1, 1.0, 0.9 - 1.0, 0.9 - 1.0
//   one state term, D = 4, narrow             1.0 - 1.1, 1.8 - 2.0,    0.7, 1.1,
//                                             1.9 - 2.2, 1.9 - 2.3     1.0, 1.1
//   the same, bf16 couplings                  0.8, 1.1 - 1.2, 1.0 - 1.3, 1.0 - 1.3
//   the same, D = 1                           0.95, 1.0, 1.0, 0.95
// A block streams all of J either way, so with D = 1 or one state term, where
// the slab's products are no more than that stream costs, only narrow
// couplings gain.  Up to three blocks per CU, one after another, pay where the
// slab kernel passes over J once per component (three state terms, D >= 3,
// more than 32 tiles).
bool spack_takes(int tiles, int d, int xs, int js, bool narrow, int64_t blocks, bool batch, int cus) {
    if (!lookup_spack(spack_shape(tiles), d, xs, js)) return false;
    if (blocks > cus) {
        if (batch || xs != 3 || d < 3 || tiles <= 32) return false;
        return blocks <= (d == 4 && js == 1 ? 3 : 2) * (int64_t)cus;
    }
    if (js == 3) return d > 1;
    if (narrow) return xs == 3 || d < 3 || tiles >= 24;
    return xs == 3 ? d > 1 : d == 4 && tiles >= 24 && 2 * blocks <= cus;
}

hipError_t launch_integrate_spack(int tiles, int d, int xs, int js, int blocks, const IntegArgs &a, const void *stage,
                                  hipStream_t stream) {
    SpackFn fn = lookup_spack(spack_shape(tiles), d, xs, js);
    if (!fn) return hipErrorInvalidDeviceFunction;
    const size_t lds = spack_lds(tiles, xs);
    hipError_t e = slab_prepare(reinterpret_cast<const void *>(fn), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(64 * kSpackWaves), lds, stream, a,
                       reinterpret_cast<const unsigned char *>(stage));
    return hipGetLastError();
}

hipError_t launch_integrate_spack_batch(int shape, int xs, int js, size_t lds, int blocks, const IntegArgs *tasks,
                                        const int2 *items, const void *const *stages, hipStream_t stream) {
    SpackBatchFn fn = js == 3 ? lookup_spack_batch_3_3(shape)
                      : xs == 3 ? lookup_spack_batch_3_1(shape)
                                : lookup_spack_batch_1_1(shape);
    if (!fn) return hipErrorInvalidDeviceFunction;
    hipError_t e = slab_prepare(reinterpret_cast<const void *>(fn), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(64 * kSpackWaves), lds, stream, tasks, items,
                       reinterpret_cast<const unsigned char *const *>(stages));
    return hipGetLastError();
}

// Synthetic problem for timing runs: J = +-1 by a hash of (p, q) (symmetric,
// zero diagonal), pump 1.2, alpha 1.
__device__ __forceinline__ uint32_t mix32(uint32_t v) {
    v ^= v >> 16;
    v *= 0x7feb352dU;
    v ^= v >> 15;
    v *= 0x846ca68bU;
    v ^= v >> 16;
    return v;
}

__global__ void k_fill_probe(void *j, int j_dtype, int n, float *pump, int r, float *alpha, int na) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t nn = (size_t)n * n;
    if (i < nn) {
        const int p = (int)(i / n), q = (int)(i % n);
        const int lo = p < q ? p : q, hi = p < q ? q : p;
        const float v = p == q ? 0.0f : ((mix32((uint32_t)(lo * 65537 + hi)) & 1) ? 1.0f : -1.0f);
        if (j_dtype == CHYM_J_I8) reinterpret_cast<int8_t *>(j)[i] = (int8_t)v;
        else reinterpret_cast<float *>(j)[i] = v;
    }
    if (i < (size_t)r) pump[i] = 1.2f;
    if (i < (size_t)na) alpha[i] = 1.0f;
}

__global__ void k_fill_state(float *x, size_t nx) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nx; i += (size_t)gridDim.x * blockDim.x)
        x[i] = ((float)(mix32((uint32_t)i) & 0xffff) - 32768.0f) * 3e-8f;
}

hipError_t launch_fill_probe(void *j, int j_dtype, int n, float *pump, int r, float *alpha, int na,
                             hipStream_t stream) {
    size_t m = (size_t)n * n;
    if ((size_t)r > m) m = r;
    if ((size_t)na > m) m = na;
    hipLaunchKernelGGL(k_fill_probe, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, stream, j, j_dtype, n, pump,
                       r, alpha, na);
    return hipGetLastError();
}

hipError_t launch_fill_state(float *x, size_t nx, hipStream_t stream) {
    hipLaunchKernelGGL(k_fill_state, dim3(2048), dim3(256), 0, stream, x, nx);
    return hipGetLastError();
}

// Eight consecutive values per thread through the kernels' own split.
__global__ void k_split3(const float *x, int64_t n8, bf16x8 *hi, bf16x8 *mid, bf16x8 *lo) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n8) return;
    float v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = x[i * 8 + s];
    XSplit<3> out;
    split8<3>(v, out);
    hi[i] = out.t[0];
    mid[i] = out.t[1];
    lo[i] = out.t[2];
}

hipError_t launch_split3(const float *x, int64_t n, uint16_t *hi, uint16_t *mid, uint16_t *lo, hipStream_t stream) {
    const int64_t n8 = n / 8;
    if (n8 == 0) return hipSuccess;
    hipLaunchKernelGGL(k_split3, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, stream, x, n8,
                       reinterpret_cast<bf16x8 *>(hi), reinterpret_cast<bf16x8 *>(mid), reinterpret_cast<bf16x8 *>(lo));
    return hipGetLastError();
}

__global__ void k_zero_counters(int *c, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) c[i] = 0;
}

hipError_t launch_integrate(int tiles, int d, int xs, int js, int waves_per_block, const IntegArgs &a,
                            hipStream_t stream, bool *supported) {
    KernelFn fn = lookup(tiles, d, xs, js);
    *supported = fn.single != nullptr;
    if (!fn.single) return hipSuccess;
    const int reps_per_block = 16 * waves_per_block;
    const int blocks = (a.r + reps_per_block - 1) / reps_per_block;
    hipLaunchKernelGGL(fn.single, dim3(blocks), dim3(64 * waves_per_block), 0, stream, a);
    return hipGetLastError();
}

bool integrate_variant_exists(int tiles, int d, int xs, int js) { return lookup(tiles, d, xs, js).single != nullptr; }

static void (*lds_kernel(const KernelFn &fn, int kind))(const IntegArgs *, const int2 *, int, int *) {
    switch (kind) {
        case kKernelPipe: return fn.persistent_pipe;
        case kKernelLdsJ1: return fn.persistent_lds1;
        case kKernelLdsJ3: return fn.persistent_lds3;
        default: return fn.persistent_lds;
    }
}

static bool uses_lds(int kind) {
    return kind == kKernelLdsJ || kind == kKernelLdsJ1 || kind == kKernelPipe || kind == kKernelLdsJ3;
}

bool persistent_kind_exists(int tiles, int d, int xs, int js, int kind) {
    KernelFn fn = lookup(tiles, d, xs, js);
    if (!fn.persistent) return false;
    return uses_lds(kind) ? lds_kernel(fn, kind) != nullptr : true;
}

static hipError_t prepare_lds(const KernelFn &fn, int kind) {
    if (fn.lds_bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(lds_kernel(fn, kind)),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)fn.lds_bytes);
}

hipError_t persistent_occupancy(int tiles, int d, int xs, int js, int kind, int waves_per_block, int *blocks_per_cu) {
    KernelFn fn = lookup(tiles, d, xs, js);
    *blocks_per_cu = 0;
    if (!fn.persistent) return hipErrorInvalidDeviceFunction;
    if (uses_lds(kind)) {
        if (!lds_kernel(fn, kind)) return hipErrorInvalidDeviceFunction;
        hipError_t e = prepare_lds(fn, kind);
        if (e != hipSuccess) return e;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, lds_kernel(fn, kind), 64 * waves_per_block,
                                                            fn.lds_bytes);
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn.persistent, 64 * waves_per_block, 0);
}

hipError_t launch_zero_counters(int *counters, int n, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_counters, dim3((n + 255) / 256), dim3(256), 0, stream, counters, n);
    return hipGetLastError();
}

hipError_t launch_integrate_persistent(int tiles, int d, int xs, int js, int kind, int waves_per_block, int blocks,
                                       const IntegArgs *tasks, const int2 *items, int n_items, int *counter,
                                       hipStream_t stream) {
    KernelFn fn = lookup(tiles, d, xs, js);
    if (!fn.persistent) return hipErrorInvalidDeviceFunction;
    if (uses_lds(kind)) {
        if (!lds_kernel(fn, kind)) return hipErrorInvalidDeviceFunction;
        hipError_t e = prepare_lds(fn, kind);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(lds_kernel(fn, kind), dim3(blocks), dim3(64 * waves_per_block), fn.lds_bytes, stream,
                           tasks, items, n_items, counter);
    } else {
        hipLaunchKernelGGL(fn.persistent, dim3(blocks), dim3(64 * waves_per_block), 0, stream, tasks, items, n_items,
                           counter);
    }
    return hipGetLastError();
}

}  // namespace chym
