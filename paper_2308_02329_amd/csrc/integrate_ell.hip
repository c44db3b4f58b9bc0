// Sparse-coupling (ELL) CHYM integrator for gfx950.
//
// For graphs with few couplings per row (3-regular: 3; the paper's 20%
// Erdos-Renyi graphs: ~0.2 N) the dense matrix-core contraction does N/w
// times the necessary work.  Here a block owns rb replicas of one problem
// (a power of two, at most as many as let the double-buffered state fit in LDS)
// for the whole run: the state x[p][replica][mu] lives in LDS, each step
// every (row, replica) unit gathers its w couplings (G_mu = sum_k val x_col)
// in float32 from the current buffer and writes the Euler update of Eq. (2)'s
// continuous limit into the other buffer; one block barrier per step.
// Units are ordered row-major with the replica fastest, so the lanes of a
// wavefront read the same coupling row (broadcast) and contiguous state.
//
// What bounds a step of a full chip is the LDS: w + 1 accesses of 16 bytes
// (D = 3, 4) per unit, at about 90 bytes per cycle (N = 800, 3-regular, D = 3,
// 4096 replicas: 1.26 us a step of 3200 units before, 0.93 us now).  With fewer
// replicas the blocks take fewer of them each, and a step is a few latencies
// (N = 200, D = 1, 328 replicas: 0.77 us before, 0.23 us now).
//
// A missing coupling (column out of range) points to a slot of zeros behind
// the state, with value -0.0: it adds -0.0, which changes no sum, so no test
// of the column stands between the loads of a row.
//
// Short rows (w <= kEllRegW, e.g. 3-regular graphs) with few units per thread
// (<= kEllUnits): a thread keeps its units' rows and own state in registers for
// the whole run.  Longer rows are read each step, from
// LDS if they fit the block's row budget (each coupling as the byte offset of
// its column's state and its value), else from global memory, several
// couplings at a time either way (N = 200, 20%, D = 3, 4096 replicas: 34 us a
// step one at a time from global memory, 13 us now).  A persistent form takes (task, replica
// block) items of many problems from a counter.
#include <type_traits>

#include "chym_internal.h"

namespace chym {

constexpr size_t kEllMaxLds = 159 * 1024;
constexpr size_t kEllRowBudget = 32 * 1024;  // LDS for the coupling rows, at least
constexpr int kEllThreads = 1024;
constexpr int kEllRegW = 3;   // rows in registers: at most this many couplings
constexpr int kEllUnits = 4;  // and this many (row, replica) units per thread
constexpr int kEllMaxLrb = 4;

// Floats per (row, replica) unit in LDS: d, with d = 3 padded to 4, so that
// a unit is one 4-, 8- or 16-byte access and the lanes of a wavefront, which
// read consecutive units of a row, touch consecutive banks.
__host__ __device__ constexpr int ell_unit_floats(int d) { return d == 3 ? 4 : d; }

// LDS of a block without its rows: two buffers of the state and a slot of
// zeros, the pumps.
__host__ __device__ constexpr size_t ell_state_bytes(int n, int d, int lrb) {
    return 2 * (((size_t)n << lrb) + 1) * ell_unit_floats(d) * sizeof(float) + 16 * sizeof(float);
}

// Most replicas per block (log2): what the LDS holds (the slots of zeros, 32
// bytes at most, are of the KiB that kEllMaxLds leaves), and at most kEllUnits
// units per thread (so that short rows take the register path at every size);
// -1: n is too large.
static int ell_max_lrb(int n, int d) {
    for (int l = kEllMaxLrb; l >= 0; --l)
        if (2 * ((size_t)n << l) * ell_unit_floats(d) * sizeof(float) + kEllRowBudget + 64 <= kEllMaxLds &&
            (l == 0 || ((size_t)n << l) <= (size_t)kEllUnits * kEllThreads))
            return l;
    return -1;
}

bool ell_takes(int n, int d) { return ell_max_lrb(n, d) >= 0; }

// The time of a launch goes with the rounds of blocks, and that of a block's
// step with its units and what a step takes without any: 0.2 us, as long as
// 700 units.
int ell_lrb(int n, int d, int64_t r, int cus) {
    int best = ell_max_lrb(n, d);
    auto time = [&](int l) { return ((((r + (1 << l) - 1) >> l) + cus - 1) / cus) * (700 + ((int64_t)n << l)); };
    for (int l = best - 1; l >= 0; --l)
        if (time(l) < time(best)) best = l;
    return best;
}

size_t ell_lds_bytes(int n, int d, int lrb) { return ell_state_bytes(n, d, lrb) + kEllRowBudget; }

// The D values of unit u of an LDS state buffer, as one access.
template <int D>
__device__ __forceinline__ void ell_get(const float *buf, size_t u, float (&v)[D]) {
    if constexpr (D == 1) {
        v[0] = buf[u];
    } else if constexpr (D == 2) {
        const float2 t = reinterpret_cast<const float2 *>(buf)[u];
        v[0] = t.x;
        v[1] = t.y;
    } else {
        const float4 t = reinterpret_cast<const float4 *>(buf)[u];
        v[0] = t.x;
        v[1] = t.y;
        v[2] = t.z;
        if constexpr (D == 4) v[3] = t.w;
    }
}

// A neighbour's state, the padding of d = 3 with it: three floats out of four
// are read by a slower instruction (N = 800, 3-regular, 4096 replicas: 1.21 us a
// step with it for D = 3, 1.06 us for D = 4).  ell_use comes where the state
// is used.
template <int D>
__device__ __forceinline__ void ell_gather(const float *buf, float (&v)[ell_unit_floats(D)]) {
    ell_get<ell_unit_floats(D)>(buf, 0, v);
}
template <int D>
__device__ __forceinline__ void ell_use(float (&v)[ell_unit_floats(D)]) {
    if constexpr (D == 3) asm volatile("" : "+v"(v[3]));
}

template <int D>
__device__ __forceinline__ void ell_put(float *buf, size_t u, const float (&v)[D]) {
    if constexpr (D == 1) {
        buf[u] = v[0];
    } else if constexpr (D == 2) {
        reinterpret_cast<float2 *>(buf)[u] = float2{v[0], v[1]};
    } else {
        reinterpret_cast<float4 *>(buf)[u] = float4{v[0], v[1], v[2], D == 4 ? v[D - 1] : 0.0f};
    }
}

// The update of one unit from its state xv and coupling sum G: xv becomes the
// new state.
template <int D>
__device__ __forceinline__ void ell_local(float (&xv)[D], float base, float nbd, float ned) {
    float x2[D];
#pragma unroll
    for (int mu = 0; mu < D; ++mu) x2[mu] = xv[mu] * xv[mu];
    float S = x2[0];
#pragma unroll
    for (int mu = 1; mu < D; ++mu) S = S + x2[mu];
    const float cc = fmaf(nbd, S, base);
#pragma unroll
    for (int mu = 0; mu < D; ++mu) xv[mu] = xv[mu] * fmaf(ned, x2[mu], cc);
}

// Integrates replicas rep0 .. rep0 + 2^lrb - 1 of problem a; called by all
// threads of the block (block barriers inside).  The block size is a multiple
// of 2^lrb, so all units of a thread belong to one replica.  row_budget: LDS
// bytes for the rows; REGS: the short-row form.
template <int D, bool REGS>
__device__ __forceinline__ void ell_block(const IntegArgs &a, int rep0, int lrb, size_t row_budget, float *sm) {
    const int n = a.n;
    const int r = a.r;
    const int rb = 1 << lrb;
    const int units = n << lrb;
    constexpr int UF = ell_unit_floats(D);
    constexpr int UB = UF * (int)sizeof(float);
    constexpr int U = REGS ? kEllUnits : 1;
    const int buf = (units + 1) * UB;            // bytes of a state buffer; its last slot is zero
    float *pl = sm + 2 * (size_t)(units + 1) * UF;  // pumps of the block's replicas [16]
    int *rl = reinterpret_cast<int *>(pl + 16);  // couplings [n][w], offsets and values, if they fit
    const EllView e = ell_view(a.j, n);
    const int w = e.w;
    const bool staged = !REGS && (size_t)n * 2 * w * sizeof(int) <= row_budget;
    const int jr = threadIdx.x & (rb - 1);
    // offset of column q's state of this thread's replica
    auto offset = [&](int q) __attribute__((always_inline)) {
        return (unsigned)q < (unsigned)n ? ((q << lrb) + jr) * UB : units * UB;
    };
    auto value = [&](int q, int v) __attribute__((always_inline)) {
        return __int_as_float((unsigned)q < (unsigned)n ? v : (int)0x80000000);
    };
    auto at = [&](int bytes) __attribute__((always_inline)) {
        return reinterpret_cast<float *>(reinterpret_cast<char *>(sm) + bytes);
    };
    if (staged) {
        for (int i = threadIdx.x; i < n * w; i += blockDim.x) {
            const int *row = e.row(i / w) + i % w;
            const int q = row[0];
            rl[2 * i] = (unsigned)q < (unsigned)n ? (q << lrb) * UB : units * UB;
            rl[2 * i + 1] = __float_as_int(value(q, row[w]));
        }
    }
    if (threadIdx.x < rb) pl[threadIdx.x] = rep0 + (int)threadIdx.x < r ? a.pump[rep0 + threadIdx.x] : 1.0f;
    if (threadIdx.x < UF) *at(units * UB + 4 * threadIdx.x) = *at(buf + units * UB + 4 * threadIdx.x) = 0.0f;
    for (int u = threadIdx.x; u < units; u += blockDim.x) {
        float v[D];
#pragma unroll
        for (int mu = 0; mu < D; ++mu) v[mu] = rep0 + jr < r ? a.x[((size_t)(u >> lrb) * r + rep0 + jr) * D + mu] : 0.0f;
        ell_put<D>(sm, u, v);
    }
    __syncthreads();

    // unit i of this thread is u = threadIdx.x + i blockDim.x
    const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63);
    auto mine = [&](int i) __attribute__((always_inline)) { return (int)threadIdx.x + i * (int)blockDim.x; };
    auto some = [&](int i) __attribute__((always_inline)) { return wave0 + i * (int)blockDim.x < units; };  // wave-uniform
    // the register path's units past the last read the zeros and store nothing
    float xv[U][D];
    int nq[U][kEllRegW];
    float nv[U][kEllRegW];
    if constexpr (REGS) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            ell_get<D>(sm, min(mine(i), units), xv[i]);
#pragma unroll
            for (int kk = 0; kk < kEllRegW; ++kk) {
                const bool has = mine(i) < units && kk < w;
                const int *row = e.row(has ? mine(i) >> lrb : -1);
                const int q = has ? row[kk] : -1;
                nq[i][kk] = offset(q);
                nv[i][kk] = value(q, has ? row[w + kk] : 0);
            }
        }
    }

    const float nbd = -(a.dt * a.btil);
    const float ned = -(a.dt * a.eta);
    const float dte = a.dt * a.eps;
    const float base = rep0 + jr < r ? fmaf(a.dt, pl[jr] - 1.0f, 1.0f) : 0.0f;  // 1 + dt (r_i - 1)
    const float *al = a.alpha + (size_t)a.start_step * D;
    float an[D];
#pragma unroll
    for (int mu = 0; mu < D; ++mu) an[mu] = al[mu];

    int from = 0, to = buf;
    for (int k = 0; k < a.steps; ++k) {
        // the annealing weights of the next step are read meanwhile
        float ga[D];
        const size_t kn = (size_t)(k + 1 < a.steps ? k + 1 : k) * D;
#pragma unroll
        for (int mu = 0; mu < D; ++mu) {
            ga[mu] = dte * an[mu];
            an[mu] = al[kn + mu];
        }
        if constexpr (REGS) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                if (!some(i)) break;
                float xq[kEllRegW][UF];
#pragma unroll
                for (int kk = 0; kk < kEllRegW; ++kk) ell_gather<D>(at(nq[i][kk] + from), xq[kk]);
                ell_local<D>(xv[i], base, nbd, ned);
#pragma unroll
                for (int kk = 0; kk < kEllRegW; ++kk) ell_use<D>(xq[kk]);
#pragma unroll
                for (int mu = 0; mu < D; ++mu) {
                    float G = 0.0f;
#pragma unroll
                    for (int kk = 0; kk < kEllRegW; ++kk) G = fmaf(nv[i][kk], xq[kk][mu], G);
                    xv[i][mu] = fmaf(ga[mu], G, xv[i][mu]);
                }
                if (mine(i) < units) ell_put<D>(at(mine(i) * UB + to), 0, xv[i]);
            }
        } else {
            for (int u = threadIdx.x; u < units; u += blockDim.x) {
                const int p = u >> lrb;
                float x[D], G[D];
                ell_get<D>(at(u * UB + from), 0, x);
#pragma unroll
                for (int mu = 0; mu < D; ++mu) G[mu] = 0.0f;
                // C couplings from kk on
                auto couplings = [&](auto count, int kk) __attribute__((always_inline)) {
                    constexpr int C = decltype(count)::value;
                    int off[C];
                    float v[C], xq[C][UF];
                    if (staged) {
                        const int2 *row = reinterpret_cast<const int2 *>(rl) + (size_t)p * w + kk;
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            off[c] = min(row[c].x + jr * UB, units * UB);
                            v[c] = __int_as_float(row[c].y);
                        }
                    } else {
                        const int *row = e.row(p) + kk;
#pragma unroll
                        for (int c = 0; c < C; ++c) off[c] = row[c];
#pragma unroll
                        for (int c = 0; c < C; ++c) v[c] = __int_as_float(row[w + c]);
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            v[c] = value(off[c], __float_as_int(v[c]));
                            off[c] = offset(off[c]);
                        }
                    }
#pragma unroll
                    for (int c = 0; c < C; ++c) ell_gather<D>(at(off[c] + from), xq[c]);
#pragma unroll
                    for (int c = 0; c < C; ++c) ell_use<D>(xq[c]);
#pragma unroll
                    for (int c = 0; c < C; ++c)
#pragma unroll
                        for (int mu = 0; mu < D; ++mu) G[mu] = fmaf(v[c], xq[c][mu], G[mu]);
                };
                int kk = 0;
                for (; kk + 8 <= w; kk += 8) couplings(std::integral_constant<int, 8>{}, kk);
                if (w & 4) {
                    couplings(std::integral_constant<int, 4>{}, kk);
                    kk += 4;
                }
                for (; kk < w; ++kk) couplings(std::integral_constant<int, 1>{}, kk);
                ell_local<D>(x, base, nbd, ned);
#pragma unroll
                for (int mu = 0; mu < D; ++mu) x[mu] = fmaf(ga[mu], G[mu], x[mu]);
                ell_put<D>(at(u * UB + to), 0, x);
            }
        }
        __syncthreads();
        const int t = from;
        from = to;
        to = t;
    }

    if (rep0 + jr >= r) return;
    for (int u = threadIdx.x; u < units; u += blockDim.x) {
        float v[D];
        ell_get<D>(at(u * UB + from), 0, v);
#pragma unroll
        for (int mu = 0; mu < D; ++mu) a.x[((size_t)(u >> lrb) * r + rep0 + jr) * D + mu] = v[mu];
    }
}

template <int D>
__device__ __forceinline__ void ell_run(const IntegArgs &a, int block, int lrb, size_t row_budget, float *sm) {
    const bool regs = in_wave(ell_view(a.j, a.n).w) <= kEllRegW && a.n << lrb <= kEllUnits * (int)blockDim.x;
    if (regs) ell_block<D, true>(a, block << lrb, lrb, row_budget, sm);
    else ell_block<D, false>(a, block << lrb, lrb, row_budget, sm);
}

template <int D>
__global__ __launch_bounds__(kEllThreads) void k_integrate_ell(IntegArgs a, int lrb, int row_budget) {
    extern __shared__ __align__(16) float sm[];
    ell_run<D>(a, blockIdx.x, lrb, row_budget, sm);
}

// Many problems of one D: blocks pop items, (task, 8 x replica block + log2 of
// its replicas), from the counter (zero at launch) until n_items are taken.
template <int D>
__global__ __launch_bounds__(kEllThreads) void k_integrate_ell_persistent(const IntegArgs *__restrict__ tasks,
                                                                          const int2 *__restrict__ items,
                                                                          int n_items, int *__restrict__ counter) {
    extern __shared__ __align__(16) float sm[];
    __shared__ int s_item;
    for (;;) {
        __syncthreads();  // the previous item's LDS use is over
        if (threadIdx.x == 0) s_item = atomicAdd(counter, 1);
        __syncthreads();
        const int it = s_item;
        if (it >= n_items) break;
        const int2 w = items[in_wave(it)];
        const IntegArgs a = in_wave(tasks[w.x]);
        ell_run<D>(a, w.y >> 3, w.y & 7, kEllRowBudget, sm);
    }
}

hipError_t launch_integrate_ell(const IntegArgs &a, int cus, hipStream_t stream) {
    if (!ell_takes(a.n, a.d)) return hipErrorInvalidValue;
    const int lrb = ell_lrb(a.n, a.d, a.r, cus);
    const int blocks = (int)(((int64_t)a.r + (1 << lrb) - 1) >> lrb);
    const int units = a.n << lrb;
    const int threads = units >= kEllThreads ? kEllThreads : (units + 63) / 64 * 64;
    const size_t state = ell_state_bytes(a.n, a.d, lrb);
    // with at most one block per compute unit the rows may have all of its LDS
    const size_t lds = blocks <= cus || 2 * (state + kEllRowBudget) > kEllMaxLds ? kEllMaxLds : state + kEllRowBudget;
    void (*fn)(IntegArgs, int, int) = a.d == 1 ? k_integrate_ell<1>
                                      : a.d == 2 ? k_integrate_ell<2>
                                      : a.d == 3 ? k_integrate_ell<3>
                                                 : k_integrate_ell<4>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(threads), lds, stream, a, lrb, (int)(lds - state));
    return hipGetLastError();
}

typedef void (*EllPersistentFn)(const IntegArgs *, const int2 *, int, int *);

static EllPersistentFn ell_persistent_fn(int d) {
    return d == 1 ? k_integrate_ell_persistent<1>
           : d == 2 ? k_integrate_ell_persistent<2>
           : d == 3 ? k_integrate_ell_persistent<3>
                    : k_integrate_ell_persistent<4>;
}

static hipError_t ell_persistent_prepare(EllPersistentFn fn, size_t lds) {
    if (lds <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds);
}

hipError_t ell_persistent_occupancy(int d, size_t lds, int *blocks_per_cu) {
    EllPersistentFn fn = ell_persistent_fn(d);
    *blocks_per_cu = 0;
    hipError_t e = ell_persistent_prepare(fn, lds);
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, kEllThreads, lds);
}

hipError_t launch_integrate_ell_persistent(int d, int blocks, size_t lds, const IntegArgs *tasks, const int2 *items,
                                           int n_items, int *counter, hipStream_t stream) {
    EllPersistentFn fn = ell_persistent_fn(d);
    hipError_t e = ell_persistent_prepare(fn, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(kEllThreads), lds, stream, tasks, items, n_items, counter);
    return hipGetLastError();
}

}  // namespace chym
