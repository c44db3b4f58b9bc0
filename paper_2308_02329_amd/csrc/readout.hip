// Readout and scoring kernels: sign readout of the Ising spins, exact Ising
// energy, and the float64 hyperspin energy of Eq. (3).
#include <algorithm>

#include "chym_internal.h"

namespace chym {

// Readout of up to 64 replicas of one problem by a block of nw <= 16
// wavefronts, one replica per lane (lane of every wavefront the same; lanes
// with mine = false read and write nothing): packs the spin bits (sigma_p = +1
// iff x_{p,1} >= 0), and finds the largest share of the extra components and
// the divergence flag.  A wavefront takes 16 rows at a time, so that a row's
// components are read by consecutive lanes and 16 rows are in flight; its 16
// bits go to LDS, where four make a spin word.  One thread per replica walked
// the rows one after the other and was bound by their latency (N = 200, D = 3,
// 20000 replicas: 120 us; now 12 us, 3.9 TB/s; N = 100, 2000 replicas: 59 and
// 5.6).  Called by all threads of the block; contains block barriers.
struct ReadoutLds {
    uint16_t bits[16][64];
    float share[16][64];
    uint8_t bad[16][64];
};

// One wavefront's 16 rows from p0 on: their bits, and the running share and
// flag.  Eight rows' loads are issued before the first use (rows past n read
// row n-1).
template <int D>
__device__ __forceinline__ uint32_t readout_rows(int n, int r, int rep, int p0, const float *__restrict__ x, float &m,
                                                 int &bad) {
    uint32_t bits = 0;
#pragma unroll 1
    for (int h = 0; h < 16; h += 8) {
        float v[8][D];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float *xp = x + ((size_t)min(p0 + h + i, n - 1) * r + rep) * D;
#pragma unroll
            for (int mu = 0; mu < D; ++mu) v[i][mu] = xp[mu];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (v[i][0] >= 0.0f && p0 + h + i < n) bits |= 1u << (h + i);
            float tot = 0.0f, ext = 0.0f;
#pragma unroll
            for (int mu = 0; mu < D; ++mu) {
                const float v2 = v[i][mu] * v[i][mu];
                tot = tot + v2;
                if (mu > 0) ext = ext + v2;
                if (!isfinite(v[i][mu]) || fabsf(v[i][mu]) > 1e3f) bad = 1;
            }
            if (tot > 0.0f && ext / tot > m) m = ext / tot;
        }
    }
    return bits;
}

template <int D>
__device__ __forceinline__ void readout_block(int n, int r, int rep, bool mine, int nw, const float *__restrict__ x,
                                              uint64_t *__restrict__ spins, double *__restrict__ extra,
                                              uint8_t *__restrict__ diverged, ReadoutLds &sm) {
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int w = (n + 63) >> 6;
    const int segs = (n + 15) >> 4;
    float m = 0.0f;  // float32: the share needs no more (its reference runs in float64, rtol 1e-6)
    int bad = 0;
    for (int s0 = 0; s0 < segs; s0 += 16) {
        __syncthreads();  // the previous words, or the previous call's results, have been read
        for (int s = s0 + wv; s < s0 + 16; s += nw)
            sm.bits[s - s0][lane] = mine && s < segs ? (uint16_t)readout_rows<D>(n, r, rep, 16 * s, x, m, bad) : 0;
        __syncthreads();
        if (spins && mine) {
            for (int k = wv; k < 4; k += nw) {
                const int wd = (s0 >> 2) + k;
                if (wd < w)
                    spins[(size_t)rep * w + wd] = (uint64_t)sm.bits[4 * k][lane] | (uint64_t)sm.bits[4 * k + 1][lane] << 16 |
                                                  (uint64_t)sm.bits[4 * k + 2][lane] << 32 |
                                                  (uint64_t)sm.bits[4 * k + 3][lane] << 48;
            }
        }
    }
    sm.share[wv][lane] = m;
    sm.bad[wv][lane] = (uint8_t)bad;
    __syncthreads();
    if (wv == 0 && mine) {
        for (int k = 1; k < nw; ++k) {
            m = fmaxf(m, sm.share[k][lane]);
            bad |= sm.bad[k][lane];
        }
        if (extra) extra[rep] = (double)m;
        if (diverged) diverged[rep] = (uint8_t)bad;
    }
}

__device__ __forceinline__ void readout_any(int n, int d, int r, int rep, bool mine, int nw, const float *__restrict__ x,
                            uint64_t *__restrict__ spins, double *__restrict__ extra,
                            uint8_t *__restrict__ diverged, ReadoutLds &sm) {
    switch (d) {
        case 1: readout_block<1>(n, r, rep, mine, nw, x, spins, extra, diverged, sm); break;
        case 2: readout_block<2>(n, r, rep, mine, nw, x, spins, extra, diverged, sm); break;
        case 3: readout_block<3>(n, r, rep, mine, nw, x, spins, extra, diverged, sm); break;
        default: readout_block<4>(n, r, rep, mine, nw, x, spins, extra, diverged, sm); break;
    }
}

__global__ __launch_bounds__(1024) void k_readout(int n, int d, int r, int first, const float *__restrict__ x,
                                                  uint64_t *__restrict__ spins, double *__restrict__ extra,
                                                  uint8_t *__restrict__ diverged) {
    __shared__ ReadoutLds sm;
    const int rep = first + blockIdx.x * 64 + (threadIdx.x & 63);
    readout_any(n, d, r, rep, rep < r, blockDim.x >> 6, x, spins, extra, diverged, sm);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ int spin_of(const uint64_t *s, int p) {
    return ((s[p >> 6] >> (p & 63)) & 1ull) ? 1 : -1;
}

// Ising energy of one replica by one wavefront, for sparse rows and for dense
// couplings beyond the block kernels' sizes (float64 of the stored values):
// E = -sum_q sigma_q sum_p J_pq sigma_p.
__device__ void ising_one(int n, int rep, const void *__restrict__ j, int j_dtype, const uint64_t *__restrict__ spins,
                          double *__restrict__ e_f64) {
    const int lane = threadIdx.x & 63;
    const int w = (n + 63) >> 6;
    const uint64_t *s = spins + (size_t)rep * w;
    double acc = 0.0;
    if (j_dtype == CHYM_J_ELL) {
        // lanes own rows p: E = -sum_p sigma_p sum_k val[p][k] sigma_{col[p][k]}
        const EllView e = ell_view(j, n);
        for (int p = lane; p < n; p += 64) {
            const int *row = e.row(p);
            double h = 0.0;
            for (int k = 0; k < e.w; ++k) {
                const int q = row[k];
                if ((unsigned)q < (unsigned)n) h += (double)__int_as_float(row[e.w + k]) * (double)spin_of(s, q);
            }
            acc += (double)spin_of(s, p) * h;
        }
    } else {
        // lanes own columns q (coalesced reads of each row of J)
        for (int q = lane; q < n; q += 64) {
            double h = 0.0;
            for (int p = 0; p < n; ++p) h += (double)coupling(j, j_dtype, n, p, q) * (double)spin_of(s, p);
            acc += (double)spin_of(s, q) * h;
        }
    }
    acc = wave_sum(acc);
    if (lane == 0 && e_f64) e_f64[rep] = -acc;
}

// 16 columns q0 .. q0+15 of row p of int8 couplings, 0 outside the matrix: one
// load where its 16 bytes lie inside the matrix's storage (past the row's end
// they are the next row's, and masked).
__device__ __forceinline__ i32x4 int8_row16(const int8_t *__restrict__ J, int n, int p, int q0) {
    const int left = p < n ? n - q0 : 0;
    const size_t i = (size_t)p * n + q0;
    const bool whole = i + 16 <= (size_t)n * n;
    i32x4 v = {0, 0, 0, 0};
    if (left > 0 && whole) __builtin_memcpy(&v, J + i, 16);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int b = left - 4 * k;  // bytes of the row in dword k
        v[k] = b >= 4 ? v[k] : (b <= 0 ? 0 : v[k] & (int)((1u << (8 * b)) - 1u));
    }
    if (left > 0 && !whole) {
#pragma unroll
        for (int s = 0; s < 16; ++s)
            if (s < left) v[s >> 2] |= (int)((uint32_t)(uint8_t)J[i + s] << (8 * (s & 3)));
    }
    return v;
}

// Exact Ising energies of cnt <= 16 replicas of one problem with int8
// couplings by a block of four wavefronts.  G = J S runs on
// v_mfma_i32_16x16x64_i8 with the spins (+-1 bytes, expanded from the words)
// as the B operand; wavefront w takes row tiles w, w+4, ..., each lane
// multiplies its rows of G by their spins, and the sums meet in LDS.  All
// integer, so any order gives the same energy.  The per-replica walk over the
// rows that this replaces was bound by its chain of row reads (N = 200, 20000
// replicas: 180 us; now 12 us).  Called by all threads of the block; contains
// block barriers.
__device__ __forceinline__ void ising_block_i8(int n, int rep0, int cnt, const int8_t *__restrict__ J,
                               const uint64_t *__restrict__ spins, int32_t *__restrict__ e_i32,
                               double *__restrict__ e_f64, int (&red)[4][16]) {
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int col = lane & 15, g = lane >> 4;
    const int w = (n + 63) >> 6;
    const int nt = (n + 15) >> 4;
    const uint64_t *s = spins + (size_t)(rep0 + (col < cnt ? col : 0)) * w;
    int acc = 0;
    for (int I = wv; I < nt; I += 4) {
        i32x4 G = {0, 0, 0, 0};
        // four chunks' loads in flight (chunks past the last are zero)
        for (int c0 = 0; c0 < w; c0 += 4) {
            i32x4 A[4];
            uint32_t b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                A[u] = int8_row16(J, n, 16 * I + col, 64 * (c0 + u) + 16 * g);
                b[u] = (uint32_t)(s[min(c0 + u, w - 1)] >> (16 * g)) & 0xffffu;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                i32x4 B;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    // four bits to four bytes: 0/1, then +1 for a set bit, -1 for a clear one
                    const uint32_t one = (((b[u] >> (4 * k)) & 0xfu) * 0x00204081u) & 0x01010101u;
                    B[k] = (int)(((one ^ 0x01010101u) * 0xffu) | 0x01010101u);
                }
                G = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[u], B, G, 0, 0, 0);
            }
        }
        const uint32_t sp = (uint32_t)(s[I >> 2] >> (16 * (I & 3) + 4 * g));
#pragma unroll
        for (int v = 0; v < 4; ++v) acc += ((sp >> v) & 1u) ? G[v] : -G[v];  // rows past n: G = 0
    }
    acc += __shfl_xor(acc, 16, 64);
    acc += __shfl_xor(acc, 32, 64);
    __syncthreads();  // the previous call's sums have been read
    if (g == 0) red[wv][col] = acc;
    __syncthreads();
    if (threadIdx.x < (unsigned)cnt) {
        const int sum = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
        if (e_i32) e_i32[rep0 + threadIdx.x] = -sum;
        if (e_f64) e_f64[rep0 + threadIdx.x] = -(double)sum;
    }
}

// Rows of the unit vectors U of quad_block: 128 bytes, and 64 bytes more after
// every four, so that the four lane groups of a read, four rows apart, touch
// all banks.
__device__ __forceinline__ int quad_row(int p) { return p * 16 + (p >> 2) * 8; }

size_t quad_lds_bytes(int n) { return sizeof(double) * (size_t)((n + 15) / 16) * 16 * 18; }

// The quadratic form of quad_block for one replica (u: its first column of U)
// by one wavefront, lanes owning columns q, pair by pair: an infinite coupling
// times the dot product of its pair is infinite, while the components' parts of
// it may have both signs.  NaN if a vector is not finite.
__device__ __forceinline__ double quad_walk(int n, int d, const void *__restrict__ j, int j_dtype, const double *u) {
    const int lane = threadIdx.x & 63;
    bool finite = true;
    for (int q = lane; q < n; q += 64)
        for (int mu = 0; mu < d; ++mu) finite = finite && isfinite(u[quad_row(q) + mu]);
    if (!__all(finite)) return __builtin_nan("");
    double acc = 0.0;
#pragma unroll 1
    for (int q = lane; q < n; q += 64) {
        double h = 0.0;
#pragma unroll 1
        for (int p = 0; p < n; ++p) {
            double dot = 0.0;
            for (int mu = 0; mu < d; ++mu) dot = dot + u[quad_row(p) + mu] * u[quad_row(q) + mu];
            h = h + (double)coupling(j, j_dtype, n, p, q) * dot;
        }
        acc += h;
    }
    return -wave_sum(acc);
}

// Quadratic form -sum_{p,q} J_pq u_p . u_q in float64 of cnt replicas of one
// problem by a block of four wavefronts: the hyperspin energy with the unit
// vectors u_p = x_p / |x_p| (0 for a zero hyperspin), or, with x = NULL, the
// Ising energy with u_p = sigma_p (d = 1).  The vectors of 16 / d replicas fill
// the 16 columns of U [n][16] in LDS (formed once per block), and G = J U runs
// on v_mfma_f64_16x16x4_f64: each lane reads four consecutive couplings and
// feeds them to four products, whose K index k of lane group g is the column
// 4 g + u, and reads U in the same order; wavefront w takes row tiles w, w+4,
// ....  The float64 vector code that this replaces formed the dot products of
// every pair per replica with J read from L2 by every wavefront (N = 100,
// D = 3, 2000 replicas: 41 us; now 14 us).  Called by all threads of the block;
// contains block barriers.
__device__ __forceinline__ void quad_block(int n, int d, int r, int rep0, int cnt, const void *__restrict__ j, int j_dtype,
                           const float *__restrict__ x, const uint64_t *__restrict__ spins, double *__restrict__ out,
                           double *u, double (&red)[4][16]) {
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int col = lane & 15, g = lane >> 4;
    const int nt = (n + 15) >> 4;
    const int w = (n + 63) >> 6;
    __syncthreads();  // the previous call's reads are done
    // one thread per hyperspin; q = cnt stands for the columns without a replica
    const int used = cnt * d;
    for (int i = threadIdx.x; i < nt * 16 * (cnt + 1); i += blockDim.x) {
        const int p = i / (cnt + 1), q = i - p * (cnt + 1);
        double *up = u + quad_row(p);
        if (q == cnt) {
            for (int c = used; c < 16; ++c) up[c] = 0.0;
        } else if (p >= n) {
            for (int mu = 0; mu < d; ++mu) up[q * d + mu] = 0.0;
        } else if (x) {
            const float *xp = x + ((size_t)p * r + rep0 + q) * d;
            float v[4];
            double s = 0.0;
            for (int mu = 0; mu < d; ++mu) {
                v[mu] = xp[mu];
                s = s + (double)v[mu] * (double)v[mu];
            }
            const double nrm = sqrt(s);
            // divided, not multiplied by a reciprocal: at d = 1 exactly +-1 (0 if NaN too)
            for (int mu = 0; mu < d; ++mu) up[q * d + mu] = nrm > 0.0 ? (double)v[mu] / nrm : 0.0;
        } else {
            up[q] = (double)spin_of(spins + (size_t)(rep0 + q) * w, p);
        }
    }
    __syncthreads();
    double sum = 0.0;
    for (int I = wv; I < nt; I += 4) {
        f64x4 G = {0.0, 0.0, 0.0, 0.0};
        // whole chunks four at a time, their loads in flight together (rows past
        // n read row n-1: their products meet zero rows of U), then the rest
        const int p = 16 * I + col, pc = min(p, n - 1);
        int c = 0;
        for (; 16 * (c + 4) <= n; c += 4) {
            float jv[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) coupling4_inside(j, j_dtype, n, pc, 16 * (c + k) + 4 * g, jv[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double *ub = u + quad_row(16 * (c + k) + 4 * g) + col;
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    G = __builtin_amdgcn_mfma_f64_16x16x4f64((double)jv[k][s], ub[16 * s], G, 0, 0, 0);
            }
        }
        for (; c < nt; ++c) {
            float jv[4];
            coupling4(j, j_dtype, n, p, 16 * c + 4 * g, jv);
            const double *ub = u + quad_row(16 * c + 4 * g) + col;
#pragma unroll
            for (int s = 0; s < 4; ++s) G = __builtin_amdgcn_mfma_f64_16x16x4f64((double)jv[s], ub[16 * s], G, 0, 0, 0);
        }
        // lane (col, g) of the result holds rows g, g + 4, g + 8, g + 12; those past n
        // are left out, 0 times an infinite coupling is not 0
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int pv = 16 * I + g + 4 * v;
            sum = pv < n ? fma(u[quad_row(pv) + col], G[v], sum) : sum;
        }
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if (g == 0) red[wv][col] = sum;
    __syncthreads();
    if (wv == 0) {
        double e = 0.0;
        for (int mu = 0; mu < d && lane < cnt; ++mu) {
            const int c = lane * d + mu;
            e += (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
        }
        e = -e;
        uint64_t redo = d > 1 ? __ballot(e != e) : 0ull;
        for (; __builtin_expect(redo != 0ull, 0); redo &= redo - 1) {
            const int q = __ffsll((unsigned long long)redo) - 1;
            const double v = quad_walk(n, d, j, j_dtype, u + q * d);
            if (lane == q) e = v;
        }
        if (lane < cnt) out[rep0 + lane] = e;
    }
}

// Sizes the block kernels take: int8 Ising energies at every n, the float64
// forms while U fits LDS.
constexpr int kQuadMaxN = 1024;
constexpr int kEnergyThreads = 256;

__global__ __launch_bounds__(kEnergyThreads) void k_ising_energy_i8(int n, int r, const int8_t *__restrict__ J,
                                                                    const uint64_t *__restrict__ spins,
                                                                    int32_t *__restrict__ e_i32,
                                                                    double *__restrict__ e_f64) {
    __shared__ int red[4][16];
    const int rep0 = blockIdx.x * 16;
    ising_block_i8(n, rep0, min(16, r - rep0), J, spins, e_i32, e_f64, red);
}

__global__ __launch_bounds__(kEnergyThreads) void k_quad(int n, int d, int r, int first, const void *__restrict__ j, int j_dtype,
                                                         const float *__restrict__ x,
                                                         const uint64_t *__restrict__ spins,
                                                         double *__restrict__ out) {
    extern __shared__ double u[];
    __shared__ double red[4][16];
    const int rp = 16 / d;
    const int rep0 = first + blockIdx.x * rp;
    quad_block(n, d, r, rep0, min(rp, r - rep0), j, j_dtype, x, spins, out, u, red);
}

// One replica per wavefront (sparse rows; dense beyond kQuadMaxN).
__global__ __launch_bounds__(kEnergyThreads) void k_ising_energy(int n, int r, const void *__restrict__ j, int j_dtype,
                                                                 const uint64_t *__restrict__ spins,
                                                                 double *__restrict__ e_f64) {
    const int rep = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (rep >= r) return;
    ising_one(n, rep, j, j_dtype, spins, e_f64);
}

// Unit vectors u_p = x_p / |x_p| (0 for a zero hyperspin) of one replica in
// float64 by one wavefront, to its private LDS area u [n][d].
__device__ __forceinline__ void hs_units(int n, int d, int r, int rep, const float *__restrict__ x, double *u) {
    const int lane = threadIdx.x & 63;
    for (int q = lane; q < n; q += 64) {
        const float *xq = x + ((size_t)q * r + rep) * d;
        double s = 0.0;
        for (int mu = 0; mu < d; ++mu) {
            const double v = (double)xq[mu];
            s = s + v * v;
        }
        const double nrm = sqrt(s);
        for (int mu = 0; mu < d; ++mu) u[q * d + mu] = nrm > 0.0 ? (double)xq[mu] / nrm : 0.0;
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Hyperspin energy of one replica by one wavefront (sparse rows; dense beyond
// kQuadMaxN other than int8): E_hs = -sum_q sum_p J_pq (u_p . u_q) with lanes
// owning columns q.
__device__ void hs_one(int n, int d, int r, int rep, const void *__restrict__ j, int j_dtype,
                       const float *__restrict__ x, double *__restrict__ e_hs, double *u) {
    const int lane = threadIdx.x & 63;
    hs_units(n, d, r, rep, x, u);
    double acc = 0.0;
    if (j_dtype == CHYM_J_ELL) {
        const EllView e = ell_view(j, n);
        for (int p = lane; p < n; p += 64) {
            const int *row = e.row(p);
            double h = 0.0;
            for (int k = 0; k < e.w; ++k) {
                const int q = row[k];
                if ((unsigned)q >= (unsigned)n) continue;
                double dot = 0.0;
                for (int mu = 0; mu < d; ++mu) dot = dot + u[p * d + mu] * u[q * d + mu];
                h = h + (double)__int_as_float(row[e.w + k]) * dot;
            }
            acc += h;
        }
    } else {
        for (int q = lane; q < n; q += 64) {
            double h = 0.0;
            for (int p = 0; p < n; ++p) {
                double dot = 0.0;
                for (int mu = 0; mu < d; ++mu) dot = dot + u[p * d + mu] * u[q * d + mu];
                const double jv = (double)coupling(j, j_dtype, n, p, q);
                h = h + jv * dot;
            }
            acc += h;
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) e_hs[rep] = -acc;
}

__global__ __launch_bounds__(64) void k_hs_energy(int n, int d, int r, const void *__restrict__ j, int j_dtype,
                                                  const float *__restrict__ x, double *__restrict__ e_hs) {
    extern __shared__ double u[];  // [n][d]
    const int rep = blockIdx.x;
    if (rep >= r) return;
    hs_one(n, d, r, rep, j, j_dtype, x, e_hs, u);
}

// The same for int8 couplings beyond kQuadMaxN.  Four rows at a time into four
// partial sums: with one sum and the storage looked up for each coupling the
// chain of its additions sets the time (N = 1500, D = 2, 512 replicas: 12.4 ms;
// so 2.3 ms).
template <int D>
__global__ __launch_bounds__(64) void k_hs_energy_i8(int n, int r, const int8_t *__restrict__ J,
                                                     const float *__restrict__ x, double *__restrict__ e_hs) {
    extern __shared__ double u[];  // [n][D]
    const int lane = threadIdx.x;
    const int rep = blockIdx.x;
    if (rep >= r) return;
    hs_units(n, D, r, rep, x, u);
    double acc = 0.0;
#pragma unroll 1
    for (int q = lane; q < n; q += 64) {
        double uq[D];
#pragma unroll
        for (int mu = 0; mu < D; ++mu) uq[mu] = u[q * D + mu];
        double h[4] = {0.0, 0.0, 0.0, 0.0};
        auto row = [&](int p, double &sum) {
            double dot = 0.0;
#pragma unroll
            for (int mu = 0; mu < D; ++mu) dot = fma(u[p * D + mu], uq[mu], dot);
            sum = fma((double)J[(size_t)p * n + q], dot, sum);
        };
        int p = 0;
#pragma unroll 1
        for (; p + 4 <= n; p += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) row(p + i, h[i]);
        }
#pragma unroll 1
        for (; p < n; ++p) row(p, h[0]);
        acc += (h[0] + h[1]) + (h[2] + h[3]);
    }
    acc = wave_sum(acc);
    if (lane == 0) e_hs[rep] = -acc;
}

// ------------------------------------------------------- batched scoring
// Global replica index g of a batch maps to (task, replica) through the
// prefix table first[t] = sum of r over tasks < t (first[n_tasks] = total).
__device__ __forceinline__ int task_of(const int64_t *__restrict__ first, int n_tasks, int64_t g) {
    int lo = 0, hi = n_tasks - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Blocks take 64 consecutive global replicas at a time and walk the tasks they
// belong to (block-uniform control flow).
__global__ __launch_bounds__(1024) void k_readout_batched(const ScoreArgs *__restrict__ t,
                                                          const int64_t *__restrict__ first, int n_tasks) {
    __shared__ ReadoutLds sm;
    const int64_t total = first[n_tasks];
    for (int64_t b0 = (int64_t)blockIdx.x * 64; b0 < total; b0 += (int64_t)gridDim.x * 64) {
        const int64_t b1 = min(b0 + 64, total);
        const int64_t g = b0 + (threadIdx.x & 63);
        for (int k = task_of(first, n_tasks, b0); k < n_tasks && first[k] < b1; ++k) {
            const ScoreArgs a = in_wave(t[k]);
            if (first[k + 1] <= b0 || first[k + 1] == first[k] || (!a.spins && !a.extra && !a.diverged)) continue;
            const bool mine = g >= first[k] && g < first[k + 1] && g < b1;
            readout_any(a.n, a.d, a.r, mine ? (int)(g - first[k]) : 0, mine, blockDim.x >> 6, a.x, a.spins, a.extra,
                          a.diverged, sm);
        }
    }
}

// Whether a task's float64 energies come from the block kernel.
__host__ __device__ constexpr bool quad_takes(int n, int j_dtype) { return j_dtype != CHYM_J_ELL && n <= kQuadMaxN; }

// Global replicas a block takes at a time: one group of int8 energies, or a
// few column groups of the quadratic form (16, 8, 5 or 4 replicas each).
constexpr int kIsingBlockReplicas = 16;
constexpr int kHsBlockReplicas = 40;

__global__ __launch_bounds__(kEnergyThreads) void k_ising_batched(const ScoreArgs *__restrict__ t,
                                                                  const int64_t *__restrict__ first, int n_tasks) {
    extern __shared__ double u_all[];
    __shared__ double red[4][16];
    const int64_t total = first[n_tasks];
    const int wave = threadIdx.x >> 6;
    for (int64_t b0 = (int64_t)blockIdx.x * kIsingBlockReplicas; b0 < total;
         b0 += (int64_t)gridDim.x * kIsingBlockReplicas) {
        const int64_t b1 = min(b0 + kIsingBlockReplicas, total);
        for (int k = task_of(first, n_tasks, b0); k < n_tasks && first[k] < b1; ++k) {
            const ScoreArgs a = in_wave(t[k]);
            if (!a.e_i32 && !a.e_f64) continue;
            const int64_t s0 = max(first[k], b0), s1 = min(first[k + 1], b1);
            if (s1 <= s0) continue;
            const int rep0 = (int)(s0 - first[k]), cnt = (int)(s1 - s0);
            if (a.j_dtype == CHYM_J_I8) {
                ising_block_i8(a.n, rep0, cnt, reinterpret_cast<const int8_t *>(a.j), a.spins, a.e_i32, a.e_f64,
                               *reinterpret_cast<int(*)[4][16]>(&red));
            } else if (quad_takes(a.n, a.j_dtype)) {
                quad_block(a.n, 1, a.r, rep0, cnt, a.j, a.j_dtype, nullptr, a.spins, a.e_f64, u_all, red);
            } else {
                for (int i = wave; i < cnt; i += kEnergyThreads / 64)
                    ising_one(a.n, rep0 + i, a.j, a.j_dtype, a.spins, a.e_f64);
            }
        }
    }
}

// lds: bytes of u_all; the tasks that run one replica per wavefront use as
// many wavefronts as its [n][d] areas allow.
__global__ __launch_bounds__(kEnergyThreads) void k_hs_batched(const ScoreArgs *__restrict__ t,
                                                               const int64_t *__restrict__ first, int n_tasks,
                                                               int lds) {
    extern __shared__ double u_all[];
    __shared__ double red[4][16];
    const int64_t total = first[n_tasks];
    const int wave = threadIdx.x >> 6;
    for (int64_t b0 = (int64_t)blockIdx.x * kHsBlockReplicas; b0 < total; b0 += (int64_t)gridDim.x * kHsBlockReplicas) {
        const int64_t b1 = min(b0 + kHsBlockReplicas, total);
        for (int k = task_of(first, n_tasks, b0); k < n_tasks && first[k] < b1; ++k) {
            const ScoreArgs a = in_wave(t[k]);
            if (!a.e_hs) continue;
            const int64_t s0 = max(first[k], b0), s1 = min(first[k + 1], b1);
            if (s1 <= s0) continue;
            const int rep0 = (int)(s0 - first[k]), cnt = (int)(s1 - s0);
            if (quad_takes(a.n, a.j_dtype)) {
                const int rp = 16 / a.d;
                for (int i = 0; i < cnt; i += rp)
                    quad_block(a.n, a.d, a.r, rep0 + i, min(rp, cnt - i), a.j, a.j_dtype, a.x, nullptr, a.e_hs, u_all,
                               red);
            } else {
                const int nd = a.n * a.d;
                const int nw = min(kEnergyThreads / 64, lds / (int)(sizeof(double) * nd));
                __syncthreads();  // the previous task's reads are done
                if (wave < nw) {
                    for (int i = wave; i < cnt; i += nw) {
                        hs_one(a.n, a.d, a.r, rep0 + i, a.j, a.j_dtype, a.x, a.e_hs, u_all + (size_t)wave * nd);
                        __builtin_amdgcn_wave_barrier();  // u is rewritten by the next replica
                    }
                }
            }
        }
    }
}

hipError_t launch_readout(int n, int d, int r, const float *x, uint64_t *spins, double *extra, uint8_t *diverged,
                          hipStream_t stream) {
    const int waves = std::min(16, (n + 15) / 16);  // 16 rows each
    const int blocks = (r + 63) / 64;
    for (int b = 0; b < blocks; b += max_blocks(64 * waves))
        hipLaunchKernelGGL(k_readout, dim3(std::min(blocks - b, max_blocks(64 * waves))), dim3(64 * waves), 0, stream, n, d, r,
                           64 * b, x, spins, extra, diverged);
    return hipGetLastError();
}

template <typename F>
static hipError_t allow_lds(F fn, size_t lds) {
    if (lds <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

static hipError_t launch_quad(int n, int d, int r, const void *j, int j_dtype, const float *x, const uint64_t *spins,
                              double *out, hipStream_t stream) {
    const size_t lds = quad_lds_bytes(n);
    hipError_t e = allow_lds(k_quad, lds);
    if (e != hipSuccess) return e;
    const int rp = 16 / d;
    const int64_t blocks = ((int64_t)r + rp - 1) / rp;
    for (int64_t b = 0; b < blocks; b += max_blocks(kEnergyThreads))
        hipLaunchKernelGGL(k_quad, dim3((unsigned)std::min<int64_t>(blocks - b, max_blocks(kEnergyThreads))),
                           dim3(kEnergyThreads), lds, stream, n, d, r, (int)(b * rp), j, j_dtype, x, spins, out);
    return hipGetLastError();
}

hipError_t launch_ising_energy(int n, int r, const void *j, int j_dtype, const uint64_t *spins, int32_t *e_i32,
                               double *e_f64, hipStream_t stream) {
    if (j_dtype == CHYM_J_I8) {
        const int part = 16 * max_blocks(kEnergyThreads);
        for (int r0 = 0; r0 < r; r0 += part) {
            const int k = std::min(r - r0, part);
            hipLaunchKernelGGL(k_ising_energy_i8, dim3((k + 15) / 16), dim3(kEnergyThreads), 0, stream, n, k,
                               reinterpret_cast<const int8_t *>(j), spins + (size_t)r0 * ((n + 63) / 64),
                               e_i32 ? e_i32 + r0 : nullptr, e_f64 ? e_f64 + r0 : nullptr);
            if (k == r - r0) break;  // r0 + part may pass the largest int
        }
    } else if (quad_takes(n, j_dtype)) {
        return launch_quad(n, 1, r, j, j_dtype, nullptr, spins, e_f64, stream);
    } else {
        const int waves = kEnergyThreads / 64;
        hipLaunchKernelGGL(k_ising_energy, dim3((r + waves - 1) / waves), dim3(kEnergyThreads), 0, stream, n, r, j,
                           j_dtype, spins, e_f64);
    }
    return hipGetLastError();
}

hipError_t launch_hs_energy(int n, int d, int r, const void *j, int j_dtype, const float *x, double *e_hs,
                            hipStream_t stream) {
    if (quad_takes(n, j_dtype)) return launch_quad(n, d, r, j, j_dtype, x, nullptr, e_hs, stream);
    const size_t lds = sizeof(double) * (size_t)n * d;
    if (j_dtype == CHYM_J_I8) {
        auto *fn = d == 1 ? k_hs_energy_i8<1> : d == 2 ? k_hs_energy_i8<2> : d == 3 ? k_hs_energy_i8<3> : k_hs_energy_i8<4>;
        hipLaunchKernelGGL(fn, dim3(r), dim3(64), lds, stream, n, r, reinterpret_cast<const int8_t *>(j), x, e_hs);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_hs_energy, dim3(r), dim3(64), lds, stream, n, d, r, j, j_dtype, x, e_hs);
    return hipGetLastError();
}

size_t ising_score_lds(int n, int j_dtype) {
    return j_dtype != CHYM_J_I8 && quad_takes(n, j_dtype) ? quad_lds_bytes(n) : 0;
}

size_t hs_score_lds(int n, int d, int j_dtype) {
    if (quad_takes(n, j_dtype)) return quad_lds_bytes(n);
    const size_t nd = sizeof(double) * (size_t)n * d;  // at most 64 KiB
    return nd * (size_t)std::min(4, std::max(1, (int)(64 * 1024 / nd)));
}

hipError_t launch_score_batched(const ScoreArgs *tasks, const int64_t *first, int n_tasks, int64_t total_replicas,
                                size_t ising_lds, size_t hs_lds, bool any_readout, bool any_ising, bool any_hs,
                                int cus, hipStream_t stream) {
    if (total_replicas <= 0) return hipSuccess;
    const int64_t grid_cap = 16 * (cus > 0 ? cus : 256);
    auto grid = [&](int per) { return dim3((unsigned)std::min<int64_t>((total_replicas + per - 1) / per, grid_cap)); };
    if (any_readout) {
        hipLaunchKernelGGL(k_readout_batched, grid(64), dim3(1024), 0, stream, tasks, first, n_tasks);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (any_ising) {
        hipError_t e = allow_lds(k_ising_batched, ising_lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_ising_batched, grid(kIsingBlockReplicas), dim3(kEnergyThreads), ising_lds, stream, tasks,
                           first, n_tasks);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (any_hs) {
        hipError_t e = allow_lds(k_hs_batched, hs_lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_hs_batched, grid(kHsBlockReplicas), dim3(kEnergyThreads), hs_lds, stream, tasks, first,
                           n_tasks, (int)hs_lds);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace chym
