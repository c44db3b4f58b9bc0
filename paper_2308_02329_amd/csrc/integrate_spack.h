// Packed streamed-J CHYM integrator for gfx950: the streamed-J kernel's problem
// (large N, J read from L2 every step) for launches with few column slabs.
//
// A slab of the streamed-J kernel is 16 replicas x D planes, so a launch of R
// replicas fills R / 16 CUs and a step takes D times the products of 16
// columns.  Here a block has 16 columns in all, a replica taking 1, 2, 4, 4
// adjacent lanes for D = 1, 2, 3, 4 as in the team integrator's packed layout:
// up to four times the blocks, each with a D-th of the products.  Every block
// reads all of J every step, from L2 at 64 bytes per cycle and CU, so J is
// staged as E2M1 or E4M3 codes where it is exact in them, for single problems
// too: at N = 1000, D = 4 a step of one block per CU takes 14.0 us with three
// state terms and +-1 couplings (10 us of it the products, 3.4 us the widening
// of the codes, which hardly overlap), 16.3 us with bf16 couplings (the read of
// J), where the slab kernel takes 71 us; with one state term 8.5 and 15.2 us
// for the slab kernel's 20.  Beyond a few blocks per CU the slabs, which share
// the read among more columns, are faster again.
//
// Eight wavefronts own the row tiles round-robin, their state and all their
// accumulators in registers, so that the operand is read from LDS once per
// wavefront and step.  Two LDS operand buffers alternate where both fit, with
// one barrier per step; else one buffer and two barriers.  K-chunk order, term
// order and update arithmetic are those of the other integrators: results are
// bit-identical.
#pragma once

#include "integrate_slab.h"
#include "integrate_team.h"

namespace chym {

constexpr int kSpackWaves = 8;

// Largest operand of one buffer is 96 KiB (N = 1024, three terms).
__host__ __device__ constexpr size_t spack_buffer_bytes(int ncp, int xs) { return (size_t)ncp * xs * 64 * sizeof(bf16x8); }
// The read ahead goes one chunk past the last.
__host__ __device__ constexpr bool spack_two_buffers(int ncp, int xs) {
    return spack_buffer_bytes(2 * ncp + 1, xs) <= kSlabMaxLds;
}
__host__ __device__ constexpr size_t spack_lds_bytes(int ncp, int xs) {
    return spack_buffer_bytes((spack_two_buffers(ncp, xs) ? 2 : 1) * ncp + 1, xs);
}

// Integrates the replicas rep0 .. of problem a; stage, FMT, ncp and lb as for
// integrate_slab, the staging in quads.  Called by all eight wavefronts of the
// block; contains block barriers.
template <int D, int XS, int JS, int TPW, int FMT>
__device__ __forceinline__ void integrate_spack(const IntegArgs &a, int rep0, const unsigned char *__restrict__ stage,
                                                int ncp, bf16x8 *lb) {
    typedef __attribute__((ext_vector_type(4))) int i4;
    constexpr int W = kSpackWaves;
    constexpr int LPR = team_lanes(D);
    // tiles accumulated together: all, or half of them where the three-term
    // fragments of all would not fit the registers
    constexpr int GS = JS == 3 && TPW > 4 ? (TPW + 1) / 2 : TPW;
    constexpr int NG = (TPW + GS - 1) / GS;
    constexpr int CPQ = stage_quad_chunks(FMT);
    const int n = a.n;
    const int r = a.r;
    const int nt = (n + 15) / 16;
    const int ncq = (ncp + CPQ - 1) / CPQ;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4;
    const int rep = rep0 + (lane & 15) / LPR;
    const int mul = (lane & 15) % LPR;
    const bool valid = rep < r && mul < D;
    const int buf = ncp * XS * 64;
    const bool two = spack_two_buffers(ncp, XS);

    constexpr int QB = JS * 1024;  // bytes of a quad
    const __amdgpu_buffer_rsrc_t jres = buffer_over(stage + stage_frag_offset(nt), (uint32_t)(nt * ncq * QB));
    const int jvoff = lane * 16;
    const __amdgpu_buffer_rsrc_t sres = buffer_over(stage + kStageHeader, (uint32_t)(nt * 64));
    // tile k of this wavefront; past the last: its first, whose products are not used
    auto tile = [&](int k) __attribute__((always_inline)) { return k < TPW && w + W * k < nt ? w + W * k : w; };

    for (int i = threadIdx.x; i < buf * (two ? 2 : 1); i += blockDim.x) lb[i] = bf16x8{};
    __syncthreads();

    float x[TPW][4];
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
        const int I = w + W * k;
        float v4[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int p = 16 * I + 4 * g + v;
            x[k][v] = valid && p < n ? a.x[((size_t)p * r + rep) * D + mul] : 0.0f;
            v4[v] = x[k][v];
        }
        if (I < nt) slab_write_comp<XS>(v4, I, (I >> 1) * XS * 64 + lane, lb);
    }

    i4 cur[GS][JS];  // the quad of J in use
    float sc[FMT == kStageE4M3 ? TPW : 1];
    if constexpr (FMT == kStageE4M3) {
#pragma unroll
        for (int k = 0; k < TPW; ++k)  // the lane's A row is 16 I + (lane & 15)
            sc[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sres, (lane & 15) * 4, tile(k) * 64, 0));
    }
    auto fetch = [&](i4 (&to)[GS][JS], int grp, int cq) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < GS; ++i)
#pragma unroll
            for (int t = 0; t < JS; ++t)
                to[i][t] = __builtin_amdgcn_raw_buffer_load_b128(jres, jvoff, (tile(GS * grp + i) * ncq + cq) * QB + t * 1024, 0);
    };
    fetch(cur, 0, 0);
    __syncthreads();

    const float base = valid ? fmaf(a.dt, a.pump[rep] - 1.0f, 1.0f) : 0.0f;
    const float nbd = -(a.dt * a.btil);
    const float ned = -(a.dt * a.eta);
    const float dte = a.dt * a.eps;
    constexpr int NP = JS == 1 ? XS : 6;
    constexpr int pj[6] = {JS == 1 ? 0 : 2, JS == 1 ? 0 : 1, 0, JS == 1 ? 0 : 1, 0, 0};
    constexpr int px[6] = {JS == 1 ? XS - 1 : 0, JS == 1 ? (XS > 1 ? XS - 2 : 0) : 1, JS == 1 ? 0 : 2, 0, 1, 0};
    const float *al = a.alpha + (size_t)a.start_step * D + (mul < D ? mul : 0);
    float an = al[0];

    for (int k = 0; k < a.steps; ++k) {
        const float ga = dte * an;
        an = al[(size_t)(k + 1 < a.steps ? k + 1 : k) * D];
        const bf16x8 *lr = lb + (two && (k & 1) ? buf : 0) + lane;
        // local part of the update in the state's place, as in the team kernel
#pragma unroll
        for (int kk = 0; kk < TPW; ++kk)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float x2 = x[kk][v] * x[kk][v];
                x[kk][v] = x[kk][v] * fmaf(ned, x2, fmaf(nbd, quad_norm<D>(x2), base));
                asm volatile("" : "+v"(x[kk][v]));  // or it would be formed after the products, its parts kept meanwhile
            }
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) {
            f32x4 acc[GS];
#pragma unroll
            for (int i = 0; i < GS; ++i) acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            // the operand of the next chunk is read while this one's products run
            bf16x8 bn[XS];
#pragma unroll
            for (int t = 0; t < XS; ++t) bn[t] = lr[t * 64];
            // chunk c, the s-th of the quad in use
            auto chunk = [&](int s, int c) __attribute__((always_inline)) {
                bf16x8 af[GS][JS], bx[XS];
#pragma unroll
                for (int t = 0; t < XS; ++t) {
                    bx[t] = bn[t];
                    bn[t] = lr[((c + 1) * XS + t) * 64];
                }
#pragma unroll
                for (int i = 0; i < GS; ++i) {
                    if constexpr (FMT == kStageE4M3)
                        af[i][0] = fp8_fragment(uint2{(uint32_t)cur[i][0][2 * s], (uint32_t)cur[i][0][2 * s + 1]},
                                                sc[GS * grp + i < TPW ? GS * grp + i : 0]);
                    else if constexpr (FMT == kStageE2M1)
                        af[i][0] = fp4_fragment((uint32_t)cur[i][0][s]);
                    else {
#pragma unroll
                        for (int t = 0; t < JS; ++t) af[i][t] = __builtin_bit_cast(bf16x8, cur[i][t]);
                    }
                }
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int i = 0; i < GS; ++i)
                        if (GS * grp + i < TPW)
                            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i][pj[p]], bx[px[p]], acc[i], 0, 0, 0);
                // the next operand's reads first, then between any two products
                // the widening of a fragment needed soon
                __builtin_amdgcn_sched_group_barrier(0x100, XS, 0);
#pragma unroll
                for (int i = 0; i < GS * NP; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if (CPQ > 1) __builtin_amdgcn_sched_group_barrier(0x002, (4 + NP - 1) / NP, 0);
                }
            };
            // The next quad (past the end, the next group's or step's first) is
            // loaded while this one is used, and moved into its place after.
            i4 nxt[GS][JS];
            int cq = 0;
            for (; (cq + 1) * CPQ <= ncp; ++cq) {
                const bool in = cq + 1 < ncq;
                fetch(nxt, in ? grp : (grp + 1) % NG, in ? cq + 1 : 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < CPQ; ++s) chunk(s, cq * CPQ + s);
#pragma unroll
                for (int i = 0; i < GS; ++i)
#pragma unroll
                    for (int t = 0; t < JS; ++t) cur[i][t] = nxt[i][t];
            }
            if (CPQ > 1 && cq < ncq) {
                fetch(nxt, (grp + 1) % NG, 0);
                __builtin_amdgcn_sched_barrier(0);
                chunk(0, cq * CPQ);
#pragma unroll
                for (int s = 1; s + 1 < CPQ; ++s)
                    if (cq * CPQ + s < ncp) chunk(s, cq * CPQ + s);
#pragma unroll
                for (int i = 0; i < GS; ++i)
#pragma unroll
                    for (int t = 0; t < JS; ++t) cur[i][t] = nxt[i][t];
            }
#pragma unroll
            for (int i = 0; i < GS; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (GS * grp + i < TPW) x[GS * grp + i][v] = fmaf(ga, acc[i][v], x[GS * grp + i][v]);
        }
        if (!two) __syncthreads();  // every wavefront is done reading the operand
        bf16x8 *lw = lb + (two && !(k & 1) ? buf : 0);
#pragma unroll
        for (int kk = 0; kk < TPW; ++kk) {
            const int I = w + W * kk;
            if (I < nt) slab_write_comp<XS>(x[kk], I, (I >> 1) * XS * 64 + lane, lw);
        }
        __syncthreads();
    }

    int row = 4 * g;  // opaque, or the addresses of the loads would be kept in registers over the steps
    asm volatile("" : "+v"(row));
#pragma unroll
    for (int k = 0; k < TPW; ++k)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int p = 16 * (w + W * k) + row + v;
            if (valid && p < n) a.x[((size_t)p * r + rep) * D + mul] = x[k][v];
        }
}

// Integrates one replica block in the format of its staging (uniform; narrow
// formats exist for single-term couplings).
template <int D, int XS, int JS, int TPW>
__device__ __forceinline__ void spack_run(const IntegArgs &a, int block, const unsigned char *__restrict__ stage,
                                          bf16x8 *lb) {
    const int ncp = ((a.n + 15) / 16 + 1) / 2;
    const int rep0 = block * team_replicas(D, true);
    if constexpr (JS == 1) {
        const int fmt = __builtin_amdgcn_readfirstlane(stage_format(stage));
        if (fmt == kStageE2M1) {
            integrate_spack<D, XS, JS, TPW, kStageE2M1>(a, rep0, stage, ncp, lb);
            return;
        }
        if (fmt == kStageE4M3) {
            integrate_spack<D, XS, JS, TPW, kStageE4M3>(a, rep0, stage, ncp, lb);
            return;
        }
    }
    integrate_spack<D, XS, JS, TPW, kStageBf16>(a, rep0, stage, ncp, lb);
}

template <int D, int XS, int JS, int TPW>
__global__ __launch_bounds__(64 * kSpackWaves) __attribute__((amdgpu_waves_per_eu(2)))
void k_integrate_spack(IntegArgs a, const unsigned char *__restrict__ stage) {
    extern __shared__ __align__(16) unsigned char smem[];
    spack_run<D, XS, JS, TPW>(a, blockIdx.x, stage, reinterpret_cast<bf16x8 *>(smem));
}

// Many problems: block b integrates item b, (task, replica block).  One launch
// takes all D: a launch runs few blocks, for long, and only a few launches run
// side by side.
template <int XS, int JS, int TPW>
__global__ __launch_bounds__(64 * kSpackWaves) __attribute__((amdgpu_waves_per_eu(2)))
void k_integrate_spack_batch(const IntegArgs *__restrict__ tasks, const int2 *__restrict__ items,
                             const unsigned char *const *__restrict__ stages) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 wi = items[blockIdx.x];
    const IntegArgs a = in_wave(tasks[wi.x]);
    const unsigned char *stage = in_wave(stages[wi.x]);
    bf16x8 *lb = reinterpret_cast<bf16x8 *>(smem);
    switch (a.d) {
        case 1: return spack_run<1, XS, JS, TPW>(a, wi.y, stage, lb);
        case 2: return spack_run<2, XS, JS, TPW>(a, wi.y, stage, lb);
        case 3: return spack_run<3, XS, JS, TPW>(a, wi.y, stage, lb);
        case 4: return spack_run<4, XS, JS, TPW>(a, wi.y, stage, lb);
    }
}

typedef void (*SpackFn)(IntegArgs, const unsigned char *);
typedef void (*SpackBatchFn)(const IntegArgs *, const int2 *, const unsigned char *const *);

// Beyond the team integrator's sizes: 17 .. 64 row tiles, three to eight per
// wavefront.  (A wavefront computes all its tiles' places: at N = 800, 50 tiles,
// seven places take 6.2 us a step where eight take 7.1, one state term, D = 4.)
constexpr int kSpackMinTiles = kTeamMaxTiles + 1;

inline int spack_tiles_per_wave(int tiles) {
    if (tiles < kSpackMinTiles || tiles > 64) return 0;
    return (tiles + kSpackWaves - 1) / kSpackWaves;
}

template <int D, int XS, int JS>
SpackFn spack_lookup_tiles(int tpw) {
    switch (tpw) {
        case 3: return k_integrate_spack<D, XS, JS, 3>;
        case 4: return k_integrate_spack<D, XS, JS, 4>;
        case 5: return k_integrate_spack<D, XS, JS, 5>;
        case 6: return k_integrate_spack<D, XS, JS, 6>;
        case 7: return k_integrate_spack<D, XS, JS, 7>;
        case 8: return k_integrate_spack<D, XS, JS, 8>;
        default: return nullptr;
    }
}

template <int D>
SpackFn spack_lookup(int tpw, int xs, int js) {
    if (js == 3) return spack_lookup_tiles<D, 3, 3>(tpw);
    return xs == 3 ? spack_lookup_tiles<D, 3, 1>(tpw) : spack_lookup_tiles<D, 1, 1>(tpw);
}

template <int XS, int JS>
SpackBatchFn spack_batch_lookup(int tpw) {
    switch (tpw) {
        case 3: return k_integrate_spack_batch<XS, JS, 3>;
        case 4: return k_integrate_spack_batch<XS, JS, 4>;
        case 5: return k_integrate_spack_batch<XS, JS, 5>;
        case 6: return k_integrate_spack_batch<XS, JS, 6>;
        case 7: return k_integrate_spack_batch<XS, JS, 7>;
        case 8: return k_integrate_spack_batch<XS, JS, 8>;
        default: return nullptr;
    }
}

// One translation unit per D instantiates its kernels, one per number of terms
// those of batches.
SpackFn lookup_spack_1(int tpw, int xs, int js);
SpackFn lookup_spack_2(int tpw, int xs, int js);
SpackFn lookup_spack_3(int tpw, int xs, int js);
SpackFn lookup_spack_4(int tpw, int xs, int js);
SpackBatchFn lookup_spack_batch_1_1(int tpw);
SpackBatchFn lookup_spack_batch_3_1(int tpw);
SpackBatchFn lookup_spack_batch_3_3(int tpw);

}  // namespace chym
