// Team CHYM integrator for gfx950: the row tiles of one problem spread over
// the wavefronts of a block, for launches too small to fill the chip with one
// wavefront per 16 replicas.
//
// In the register-resident kernel one wavefront carries all N rows of 16
// replicas, so a step is a serial chain through every product and every
// update of the problem, and a call of R replicas occupies R/16 of the 1024
// SIMDs.  Here wavefront w of a block of NC = ceil(N / 32) owns K-chunk w, the
// rows 32 w .. 32 w + 31 (row tiles 2w and 2w+1): their state, and the
// J fragments of those two tiles for every chunk, stay in its registers for
// the whole run (8 NC registers per coupling term), and the state's bf16
// operand goes through LDS.  The 8 values a lane owns are exactly its slots of
// the operand fragment of chunk w, so a step writes one 16-byte fragment per
// term and plane.  Two LDS operand buffers alternate: a step reads one and
// writes the other, with one barrier between steps.  A block of one wavefront
// (N <= 32) uses its own registers and neither LDS nor barriers.
//
// Columns of a block, two layouts:
//   PACK   16 columns in all: a replica takes LPR = 1, 2, 4, 4 adjacent lanes
//          for D = 1, 2, 3, 4 (one lane of four idle at D = 3), so a block
//          holds 16 / LPR replicas and a call has up to four times the blocks;
//          the norm is summed over the quad's lanes with DPP operands, in
//          component order;
//   plane  16 replicas x D planes, as in the other kernels: the norm is
//          in-lane and no column idles.
//
// K-chunk order, term order and update arithmetic are those of the other
// integrators, so the results are bit-identical.
#pragma once

#include "integrate_kernel.h"

namespace chym {

// Lanes of a replica in the packed layout.
__host__ __device__ constexpr int team_lanes(int d) { return d <= 2 ? d : 4; }
// Row tiles of a wavefront.
__host__ __device__ constexpr int team_tiles(int tiles, int xs, bool pack) {
    return tiles == 1 ? 1 : pack && (tiles == 3 || tiles == 4 || (xs == 1 && tiles > 4 && tiles <= 8)) ? 1 : 2;
}
// Wavefronts of a block.
__host__ __device__ constexpr int team_waves(int nc, int tw) { return nc == 1 ? 1 : (2 * nc + tw - 1) / tw; }
// Replicas of a block.
__host__ __device__ constexpr int team_replicas(int d, bool pack) { return pack ? 16 / team_lanes(d) : 16; }
// LDS bytes of a block: two operand buffers (none for a single wavefront).
__host__ __device__ constexpr size_t team_lds_bytes(int nc, int d, int xs, bool pack) {
    return nc == 1 ? 0 : (size_t)2 * nc * (pack ? 1 : d) * xs * 64 * sizeof(bf16x8);
}

// Chunks of the operand read from LDS ahead of their products (P planes, XS
// terms, NC chunks in all): a read takes longer than the products of a packed
// chunk (two per term, 16 cycles each), and the compiler would otherwise sink
// every read to its first use and wait for each.
constexpr int team_ahead(int p, int xs, int nc) {
    const int a = p == 1 ? (nc * xs <= 12 ? nc : (xs == 3 ? 4 : 6)) : (p * xs >= 6 ? 1 : 2);
    return a < nc ? a : nc;
}

template <int CTRL>
__device__ __forceinline__ float dpp_quad(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// sum over the components of a replica, in component order, from the square
// each of its lanes holds
template <int D>
__device__ __forceinline__ float quad_norm(float x2) {
    if constexpr (D == 1) return x2;
    if constexpr (D == 2) return x2 + dpp_quad<0xb1>(x2);  // the other lane of the pair; addition commutes
    float s = dpp_quad<0x00>(x2) + dpp_quad<0x55>(x2);
    s = s + dpp_quad<0xaa>(x2);
    if constexpr (D == 4) s = s + dpp_quad<0xff>(x2);
    return s;
}

// Gain of the nonlinear medium for a field of amplitude A under pump h:
// K = P / (P cosh(kl P) - h sinh(kl P)), P = sqrt(h^2 + A^2), written as
// 2 P e / ((P + h) + (P - h) e^2) with e = exp(kl P).  For h >= 0, with
// P - h = A^2 / s and both terms multiplied by s = P + h, this is
// 2 P e s / (s^2 + A^2 e^2), which has no cancellation and needs one reciprocal.
// For h < 0 the same with s = P + |h| and e = exp(-kl P) (P + h = A^2 / s, then
// both sides times e^-2).  ha = |h|, kl2 = kl log2(e) with the sign of h, tiny =
// 2^-60.  The square root, reciprocal and exponential are the hardware's (each
// within about 1 ulp).  Below s = 2^-60 the squares leave the normal floats (at h = 0 the
// reciprocal would overflow from |A| = 4e-20 down) and the gain is 1 to within
// 2^-60 kl.  A select rather than a branch at the end lets the rows of a lane
// run side by side (N = 14, D = 1, 16384 replicas: 0.38 us a step, 0.60 with
// branches).
__device__ __forceinline__ float nlm_gain(float A, float ha, float kl2, float tiny) {
    const float A2 = A * A;
    const float P = __builtin_amdgcn_sqrtf(fmaf(ha, ha, A2));
    const float s = P + ha;
    const float e = __builtin_amdgcn_exp2f(kl2 * P);
    const float den = fmaf(A2, e * e, s * s);
    const float k = (2.0f * P * e * s) * __builtin_amdgcn_rcpf(den);
    return s > tiny ? k : 1.0f;
}

// Writes the operand terms of one tile and plane (the lane's four rows, v) into
// the tile's half of the fragments f[64 t], t < XS.
template <int XS>
__device__ __forceinline__ void team_write_half(const float (&v)[4], int I, bf16x8 *f) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    const float v8[8] = {v[0], v[1], v[2], v[3], 0.0f, 0.0f, 0.0f, 0.0f};
    XSplit<XS> s;
    split8<XS>(v8, s);
#pragma unroll
    for (int t = 0; t < XS; ++t)
        reinterpret_cast<bf16x4 *>(f + 64 * t)[I & 1] = __builtin_shufflevector(s.t[t], s.t[t], 0, 1, 2, 3);
}

// Integrates the replicas rep0 .. rep0 + team_replicas(D, PACK) - 1 of problem
// a; called by all wavefronts of the block.  MAP: the round-trip map of Eq. (2)
// instead of its continuous limit: every amplitude first passes the medium
// (A <- K(A) A, pump h = pump[replica]), then the same update runs with the
// map's coefficients, which the host puts in eps, btil, eta and c0 (dt = 1).
template <int D, int XS, int JS, int NC, int TW, bool PACK, bool MAP>
__device__ __forceinline__ void integrate_team(const IntegArgs &a, int rep0, bf16x8 *lb) {
    constexpr int P = PACK ? 1 : D;                  // column planes
    constexpr int LPR = PACK ? team_lanes(D) : 1;    // lanes of a replica
    constexpr bool ONE = NC == 1;                    // one wavefront: no exchange
    constexpr int BUF = NC * P * XS * 64;            // fragments of one operand buffer
    constexpr int NP = JS == 1 ? XS : 6;
    constexpr int pj[6] = {JS == 1 ? 0 : 2, JS == 1 ? 0 : 1, 0, JS == 1 ? 0 : 1, 0, 0};
    constexpr int px[6] = {JS == 1 ? XS - 1 : 0, JS == 1 ? (XS > 1 ? XS - 2 : 0) : 1, JS == 1 ? 0 : 2, 0, 1, 0};
    const int n = a.n;
    const int r = a.r;
    const int nt = (n + 15) / 16;
    const int lane = threadIdx.x & 63;
    const int w = ONE ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4;
    const int rep = rep0 + (lane & 15) / LPR;
    const int mul = (lane & 15) % LPR;  // packed: the lane's component
    const bool valid = rep < r && mul < D;

    bf16x8 jr[TW][NC][JS];
#pragma unroll
    for (int i = 0; i < TW; ++i) {
#pragma unroll
        for (int c = 0; c < NC; ++c) j_fragment<JS>(a, TW * w + i, c, lane, jr[i][c]);
        __builtin_amdgcn_sched_barrier(0);  // one tile's loads in flight: all of them would set the register count
    }

    float x[TW][P][4];
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int p = 16 * (TW * w + i) + 4 * g + v;
            const bool ok = valid && p < n;
#pragma unroll
            for (int mu = 0; mu < P; ++mu) x[i][mu][v] = ok ? a.x[((size_t)p * r + rep) * D + mu + mul] : 0.0f;
        }

    const float base = valid ? (MAP ? a.c0 : fmaf(a.dt, a.pump[rep] - 1.0f, 1.0f)) : 0.0f;
    const float hmap = (MAP && valid) ? a.pump[rep] : 0.0f;
    const float kl2 = (hmap < 0.0f ? -a.kl : a.kl) * 1.44269504088896340736f;  // kl log2(e), with the sign of h
    float tiny = 0x1p-60f;
    if constexpr (MAP) asm("" : "+s"(tiny));  // in a register: as a literal it makes each compare 8 bytes long
    const float nbd = -(a.dt * a.btil);
    const float ned = -(a.dt * a.eta);
    const float dte = a.dt * a.eps;

    // the annealing weights are read one step ahead
    const float *al = a.alpha + (size_t)a.start_step * D + (mul < D ? mul : 0);
    float an[P];
#pragma unroll
    for (int mu = 0; mu < P; ++mu) an[mu] = al[mu];

    // The operand terms of the wavefront's tiles, to LDS buffer buf (kept in
    // registers by a block of one wavefront): whole 16-byte fragments where a
    // wavefront owns both tiles of a chunk, else the tile's 8-byte half.
    // The tile past the last of an odd count reads as zero even where an
    // infinite amplitude has made its products NaN, as in the other kernels:
    // by a select here (packed), or by leaving it out of the update (plane,
    // where D selects per row cost more than a wave-uniform branch: 0.61
    // against 0.71 us a step at N = 100, D = 3, bf16).
    XSplit<XS> own[ONE ? P : 1];
    auto value = [&](int i, int mu, int v) __attribute__((always_inline)) {
        return !PACK || TW * w + i < nt ? x[i][mu][v] : 0.0f;
    };
    auto operand = [&](int buf) __attribute__((always_inline)) {
        if constexpr (MAP) {
#pragma unroll
            for (int i = 0; i < TW; ++i)
#pragma unroll
                for (int mu = 0; mu < P; ++mu)
#pragma unroll
                    for (int v = 0; v < 4; ++v) x[i][mu][v] = nlm_gain(x[i][mu][v], fabsf(hmap), kl2, tiny) * x[i][mu][v];
        }
        if constexpr (ONE || TW % 2 == 0) {
#pragma unroll
            for (int i = 0; i < TW; i += 2)
#pragma unroll
                for (int mu = 0; mu < P; ++mu) {
                    float v8[8];
#pragma unroll
                    for (int s = 0; s < 8; ++s) v8[s] = i + (s >> 2) < TW ? value(i + (s >> 2) < TW ? i + (s >> 2) : i, mu, s & 3) : 0.0f;
                    XSplit<XS> f;
                    split8<XS>(v8, f);
                    if constexpr (ONE) {
                        own[mu] = f;
                    } else {
                        const int c = (TW * w + i) >> 1;
                        if (TW == 2 || c < NC) {
#pragma unroll
                            for (int t = 0; t < XS; ++t) lb[buf * BUF + ((c * P + mu) * XS + t) * 64 + lane] = f.t[t];
                        }
                    }
                }
        } else {
#pragma unroll
            for (int i = 0; i < TW; ++i) {
                const int I = TW * w + i;
                if (I < 2 * NC) {
#pragma unroll
                    for (int mu = 0; mu < P; ++mu) {
                        const float v4[4] = {value(i, mu, 0), value(i, mu, 1), value(i, mu, 2), value(i, mu, 3)};
                        team_write_half<XS>(v4, I, lb + buf * BUF + ((I >> 1) * P + mu) * XS * 64 + lane);
                    }
                }
            }
        }
    };
    // The local part of the update in x's place, y = x (1 + dt (r-1) -
    // dt btil S - dt eta x^2) as in integrate_group: x itself is not needed
    // again once the operand is written.
    auto local_part = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float x2[P];
#pragma unroll
                for (int mu = 0; mu < P; ++mu) x2[mu] = x[i][mu][v] * x[i][mu][v];
                float S = PACK ? quad_norm<D>(x2[0]) : x2[0];
#pragma unroll
                for (int mu = 1; mu < P; ++mu) S = S + x2[mu];
                const float cc = fmaf(nbd, S, base);
#pragma unroll
                for (int mu = 0; mu < P; ++mu) x[i][mu][v] = x[i][mu][v] * fmaf(ned, x2[mu], cc);
            }
    };
    operand(0);
    if constexpr (!ONE) __syncthreads();

    constexpr int AHEAD = team_ahead(P, XS, NC);
    const int steps = a.steps;
    for (int k = 0; k < steps; ++k) {
        float ga[P];
        const size_t kn = (size_t)(k + 1 < steps ? k + 1 : k) * D;
#pragma unroll
        for (int mu = 0; mu < P; ++mu) {
            ga[mu] = dte * an[mu];
            an[mu] = al[kn + mu];
        }
        f32x4 acc[TW][P];
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int mu = 0; mu < P; ++mu) acc[i][mu] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        const bf16x8 *lr = lb + (k & 1) * BUF + lane;
        bf16x8 bx[NC][P][XS];
        auto read_chunk = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int mu = 0; mu < P; ++mu)
#pragma unroll
                for (int q = 0; q < XS; ++q) {
                    const int t = JS == 1 ? XS - 1 - q : q;  // in the order the products take them
                    if constexpr (!ONE) bx[c][mu][t] = lr[((c * P + mu) * XS + t) * 64];
                    else bx[c][mu][t] = own[mu].t[t];
                }
        };
#pragma unroll
        for (int c = 0; c < NC && c < AHEAD; ++c) read_chunk(c);
        if constexpr (!ONE) __builtin_amdgcn_sched_barrier(0x00f);  // LDS reads stay above; other instructions may move
        local_part();
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c + AHEAD < NC) {
                read_chunk(c + AHEAD);
                __builtin_amdgcn_sched_barrier(0x00f);
            }
#pragma unroll
            for (int q = 0; q < NP; ++q)
#pragma unroll
                for (int i = 0; i < TW; ++i)
#pragma unroll
                    for (int mu = 0; mu < P; ++mu)
                        acc[i][mu] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(jr[i][c][pj[q]], bx[c][mu][px[q]],
                                                                            acc[i][mu], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < TW; ++i) {
            if (!PACK && TW * w + i >= nt) continue;
#pragma unroll
            for (int mu = 0; mu < P; ++mu)
#pragma unroll
                for (int v = 0; v < 4; ++v) x[i][mu][v] = fmaf(ga[mu], acc[i][mu][v], x[i][mu][v]);
        }
        // A block of one wavefront forms it after the last step too: without the
        // branch a step is one piece, which the compiler orders as a whole, the
        // weight's load at its head.  With it the load went to the step's end, and its
        // time lay on the chain of a step, the more the more blocks a CU had (400
        // steps, N = 16, bf16, D = 1, 4096 replicas: 40 us with the branch, 36 without;
        // 16384: 54, 38; D = 4, 512: 74, 48; float32 form, N = 32, D = 3, 512: 128,
        // 102.  From three wavefronts per SIMD on it gains nothing, N = 32, D = 1,
        // bf16 loses 7% there: 250, 269 us at 131072).
        if ((ONE && !MAP) || k + 1 < steps) {
            operand((k + 1) & 1);
            if constexpr (!ONE) __syncthreads();
        }
    }

#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int p = 16 * (TW * w + i) + 4 * g + v;
            if (valid && p < n) {
#pragma unroll
                for (int mu = 0; mu < P; ++mu) a.x[((size_t)p * r + rep) * D + mu + mul] = x[i][mu][v];
            }
        }
}

// Wavefronts per SIMD the registers are limited for: an estimate of what the
// step loop holds (J fragments, state and accumulators, the operand fragments
// read ahead), rounded down to a budget of 512 / WPE registers; two at least,
// which also keeps the accumulators in ordinary registers.  Six variants hold
// more than their budget and spill: 2, 24 and 40 registers with float couplings
// at D = 3 (plane, NC = 6 to 8), 6 at D = 2 (plane, one state term, NC = 8) and 4
// in the packed layout with one state term, NC = 6, D = 2 to 4.  They are faster
// than the streamed-J kernel all the same (200 steps, 4096 replicas: float
// couplings, D = 3, N = 192 815 against 1074 us, N = 256 1290 against 1440; one
// state term, N = 190, D = 4 282 against 293).
template <int D, int XS, int JS, int NC, int TW, bool PACK>
constexpr int team_wpe() {
    constexpr int P = PACK ? 1 : D;
    constexpr int ahead = team_ahead(P, XS, NC);
    constexpr int need = 4 * TW * NC * JS + 8 * TW * P + 4 * P * XS * (ahead < NC ? ahead + 1 : NC) + 36;
    return need <= 128 ? 4 : need <= 168 ? 3 : 2;
}

// One problem (items = NULL): block b integrates its replicas from
// (first + b) * team_replicas on.  Many problems of one shape: block b integrates
// item b, (task, replica block); the host lists the longest tasks first, and the
// hardware hands the blocks out in that order.
template <int D, int XS, int JS, int NC, int TW, bool PACK, bool MAP, int WPE = team_wpe<D, XS, JS, NC, TW, PACK>()>
__global__ __launch_bounds__(64 * team_waves(NC, TW)) __attribute__((amdgpu_waves_per_eu(WPE)))
void k_integrate_team(IntegArgs one, int first, const IntegArgs *__restrict__ tasks, const int2 *__restrict__ items) {
    extern __shared__ __align__(16) unsigned char smem[];
    int2 w = int2{0, first + (int)blockIdx.x};
    if (items) w = items[blockIdx.x];
    const IntegArgs a = in_wave(items ? tasks[w.x] : one);
    integrate_team<D, XS, JS, NC, TW, PACK, MAP>(a, w.y * team_replicas(D, PACK), reinterpret_cast<bf16x8 *>(smem));
}

// Largest row-tile count of the team kernels (N <= 256).
constexpr int kTeamMaxTiles = 16;

typedef void (*TeamFn)(IntegArgs, int, const IntegArgs *, const int2 *);

// The plane layout's operand of all D components must fit LDS twice; D = 1
// has the packed layout only (they coincide), and so have three state terms with
// D = 2 and 4 beyond one chunk, where team_layout never takes the other.
template <int D, int XS, int JS, int NC, int TW, bool MAP, bool PACK>
constexpr TeamFn team_fn() {
    if constexpr (MAP && (JS != 1 || 2 * NC > kMapMaxTiles + 1)) return nullptr;
    else if constexpr (!PACK && (D == 1 || (XS == 3 && D != 3 && NC > 1) || team_lds_bytes(NC, D, XS, false) > kSlabMaxLds))
        return nullptr;
    else return k_integrate_team<D, XS, JS, NC, TW, PACK, MAP>;
}

template <int D, int XS, int JS, bool MAP>
TeamFn team_lookup_tiles(int tiles, bool pack) {
    if (tiles == 1) return pack ? team_fn<D, XS, JS, 1, 1, MAP, true>() : team_fn<D, XS, JS, 1, 1, MAP, false>();
    switch ((tiles + 1) / 2) {
#define CHYM_NC(NC) \
        case NC: return pack ? team_fn<D, XS, JS, NC, team_tiles(2 * NC, XS, true), MAP, true>() \
                             : team_fn<D, XS, JS, NC, team_tiles(2 * NC, XS, false), MAP, false>();
        CHYM_NC(1) CHYM_NC(2) CHYM_NC(3) CHYM_NC(4) CHYM_NC(5) CHYM_NC(6) CHYM_NC(7) CHYM_NC(8)
#undef CHYM_NC
        default: return nullptr;
    }
}

template <int D>
TeamFn team_lookup(int tiles, int xs, int js, bool pack, bool map) {
    if (map)
        return js != 1 ? nullptr : xs == 3 ? team_lookup_tiles<D, 3, 1, true>(tiles, pack)
                                           : team_lookup_tiles<D, 1, 1, true>(tiles, pack);
    if (js == 3) return team_lookup_tiles<D, 3, 3, false>(tiles, pack);
    return xs == 3 ? team_lookup_tiles<D, 3, 1, false>(tiles, pack) : team_lookup_tiles<D, 1, 1, false>(tiles, pack);
}

// One translation unit per D instantiates its kernels.
TeamFn lookup_team_1(int tiles, int xs, int js, bool pack, bool map);
TeamFn lookup_team_2(int tiles, int xs, int js, bool pack, bool map);
TeamFn lookup_team_3(int tiles, int xs, int js, bool pack, bool map);
TeamFn lookup_team_4(int tiles, int xs, int js, bool pack, bool map);

}  // namespace chym
