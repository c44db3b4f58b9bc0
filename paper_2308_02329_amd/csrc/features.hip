// Trajectory features for the learned early restart, the per-batch
// standardization, top-k selection and replica gather that the restart loop
// needs, and the small MLP that maps the features to a success logit.
//
// Features (per replica, at one checkpoint), all about the first component,
// the one the anneal keeps and the readout reads: its Rayleigh quotient per
// spin -(x_1^T J x_1) / (n x_1^T x_1), the Ising energy per spin of the
// current sign readout, the first component's share of the squared norm
// sum_p x_{p,1}^2 / sum_{p,mu} x_{p,mu}^2, and the fraction of spins whose
// sign flipped since the previous checkpoint.  Runs of one problem and pump
// reach the same hyperspin configuration up to a rotation, so quantities
// invariant under rotations (the hyperspin energy, the norms) do not tell
// them apart; the first component's orientation does.  float32 sums in a fixed
// order.
//
// MLP: 32 -> 128 -> 128 -> 1, ReLU, sigmoid output, binary cross-entropy.
// Weights are kept as float32 master copies (updated by Adam) and as a bf16
// copy that the forward and backward passes use.  The two hidden layers run
// on the matrix cores in bf16 with float32 accumulation: a layer's input
// (the features, then the first layer's activations) is rounded to bf16
// (nearest even), its bias added in float32; the output layer is a float32
// dot product.  The backward pass differentiates that network (the
// weight gradients use the rounded layer inputs) in float32.
#include <algorithm>

#include "chym_internal.h"

namespace chym {

constexpr int kFeat = CHYM_FEATURES;  // feature columns per replica

template <typename T>
__device__ __forceinline__ T wsum(T v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Features of RB replicas (consecutive, lanes) by a block of RB * 16 threads.
// The per-replica wavefront that this replaces read the state with a stride of
// a whole row between lanes and J once per replica (N = 200, D = 3, 20000
// replicas: 632 us a checkpoint; now 58 us).
//
// Every sum keeps its order: it runs over the 64 classes q mod 64, each class
// in ascending q, then over the classes by halving (32, 16, .. 1).
//   1. Threads (replica, 4 classes) read the state, consecutive replicas in
//      consecutive lanes, and sum the squares per class; the first components
//      go to LDS.
//   2. Sign words and flips from the first components.
//   3. G_q = sum_p J_pq x_{p,1} and h_q = sum_p J_pq sigma_p for 16 columns q x
//      16 replicas at a time on v_mfma_f32_16x16x4_f32, whose result is the
//      chain of four fused multiply-adds in ascending p (checked bit for bit
//      on the chip, denormals included), so that G and h round as a loop of
//      fmaf over p.  With int8 couplings h is a sum of integers below 2^24,
//      the same in any arithmetic, and comes from the int8 products, at a
//      sixteenth of the time.  Wavefront w takes the column tiles of one residue
//      mod 4 and the replica group w / 4: its classes 16 (I mod 4) + 4 g + v are
//      the rows of its results.
constexpr int kFeatThreads = 16;  // threads per replica
constexpr int kFeatUnroll = 8;    // products in flight

// LDS floats: first components [rows][RB] (rows: n up to whole unrolls), two
// class sums [64][RB], flips [RB].
__host__ __device__ constexpr int feat_rows(int n) { return (n + 4 * kFeatUnroll - 1) / (4 * kFeatUnroll) * (4 * kFeatUnroll); }
constexpr size_t feat_lds(int n, int rb) { return sizeof(float) * (size_t)rb * (feat_rows(n) + 2 * 64 + 1); }

template <int JT>
__device__ __forceinline__ float feat_coupling(const void *__restrict__ j, int n, int p, int q) {
    return coupling(j, JT, n, p, q);  // the storage type is a constant here
}

template <int RB>
__device__ __forceinline__ void class_tree(float *ca, float *cb) {
    const int rep = threadIdx.x % RB, c = threadIdx.x / RB;
    for (int off = 32; off > 0; off >>= 1) {
        __syncthreads();
        for (int k = c; k < off; k += kFeatThreads) {
            ca[k * RB + rep] += ca[(k + off) * RB + rep];
            cb[k * RB + rep] += cb[(k + off) * RB + rep];
        }
    }
    __syncthreads();
}

// The couplings a[m] = J[p0 + 4 m + g][q0 + col] of an int8 matrix, zero outside
// it: the four lanes of a quad read four bytes of four rows each, a row in
// one read, and take their column's byte from each other's (a byte read per
// lane and row takes the address unit four times as long: 67 us a checkpoint
// of the above against 58).
__device__ __forceinline__ void feat_rows_i8(int n, const int8_t *__restrict__ j, int p0, int g, int q0, int col,
                                             float (&a)[kFeatUnroll]) {
    const int lane4 = col & 3;
    const int qa = q0 + col - lane4;  // the quad's first column
#pragma unroll
    for (int t = 0; t < kFeatUnroll; t += 4) {
        const int p = p0 + 4 * (t + lane4) + g;
        uint32_t own = 0u;
        if (p < n) {
            const int8_t *row = j + (size_t)p * n + qa;
            if (qa + 4 <= n) {
                __builtin_memcpy(&own, row, 4);
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (qa + c < n) own |= (uint32_t)(uint8_t)row[c] << (8 * c);
            }
        }
        const uint32_t s[4] = {(uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0x00, 0xf, 0xf, true),
                               (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0x55, 0xf, 0xf, true),
                               (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xaa, 0xf, 0xf, true),
                               (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xff, 0xf, 0xf, true)};
#pragma unroll
        for (int m = 0; m < 4; ++m) a[t + m] = (float)((int32_t)(s[m] << (24 - 8 * lane4)) >> 24);
    }
}

template <int RB, int JT>
__device__ __forceinline__ void feat_products(int n, const void *__restrict__ j, const float *sx, float *ca, float *cb) {
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int col = lane & 15, g = lane >> 4;
    const int nt = (n + 15) >> 4;
    const int rep = 16 * (w >> 2) + col;
    // the classes of most tiles go to other SIMDs for the other replicas and blocks
    const int cls = (w + 2 * (w >> 2) + blockIdx.x) & 3;
    constexpr bool INT = JT == CHYM_J_I8;
    float quad[4] = {0.0f, 0.0f, 0.0f, 0.0f}, eis[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int I = cls; I < nt; I += 4) {
        const int q = 16 * I + col;
        f32x4 G = {0.0f, 0.0f, 0.0f, 0.0f}, H = {0.0f, 0.0f, 0.0f, 0.0f};
        i32x4 HI = {0, 0, 0, 0};
        for (int p0 = 0; p0 < n; p0 += 4 * kFeatUnroll) {
            float a[kFeatUnroll], b[kFeatUnroll];
            if constexpr (INT) feat_rows_i8(n, reinterpret_cast<const int8_t *>(j), p0, g, 16 * I, col, a);
#pragma unroll
            for (int m = 0; m < kFeatUnroll; ++m) {
                const int p = p0 + 4 * m + g;
                if constexpr (!INT) {
                    const float v = feat_coupling<JT>(j, n, min(p, n - 1), min(q, n - 1));
                    a[m] = p < n && q < n ? v : 0.0f;
                }
                b[m] = sx[p * RB + rep];
            }
#pragma unroll
            for (int m = 0; m < kFeatUnroll; ++m) {
                G = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[m], G, 0, 0, 0);
                if constexpr (!INT)
                    H = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[m] >= 0.0f ? 1.0f : -1.0f, H, 0, 0, 0);
            }
            if constexpr (INT) {
                // the row p0 + 4 m + g in byte m of lane group g, on both sides
                uint32_t pa[2] = {0u, 0u}, pb[2] = {0u, 0u};
#pragma unroll
                for (int m = 0; m < kFeatUnroll; ++m) {
                    pa[m >> 2] |= ((uint32_t)(int)a[m] & 0xffu) << (8 * (m & 3));
                    pb[m >> 2] |= (b[m] >= 0.0f ? 0x01u : 0xffu) << (8 * (m & 3));
                }
                HI = __builtin_amdgcn_mfma_i32_16x16x32_i8((long)((uint64_t)pa[1] << 32 | pa[0]),
                                                           (long)((uint64_t)pb[1] << 32 | pb[0]), HI, 0, 0, 0);
            }
        }
        if constexpr (INT) H = f32x4{(float)HI[0], (float)HI[1], (float)HI[2], (float)HI[3]};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int qr = 16 * I + 4 * g + v;
            if (qr < n) {
                const float xq = sx[qr * RB + rep];
                quad[v] = fmaf(xq, G[v], quad[v]);
                eis[v] = fmaf(xq >= 0.0f ? 1.0f : -1.0f, H[v], eis[v]);
            }
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        ca[(16 * cls + 4 * g + v) * RB + rep] = quad[v];
        cb[(16 * cls + 4 * g + v) * RB + rep] = eis[v];
    }
}

template <int RB>
__global__ __launch_bounds__(RB *kFeatThreads) void k_features(int n, int d, int r, const void *__restrict__ j,
                                                               int j_dtype, const float *__restrict__ x,
                                                               uint64_t *__restrict__ prev, float *__restrict__ feat,
                                                               int feat_stride, int feat_off) {
    extern __shared__ float shf[];
    float *sx = shf;                          // [rows][RB]
    float *ca = sx + (size_t)feat_rows(n) * RB;  // [64][RB]
    float *cb = ca + 64 * RB;                 // [64][RB]
    int *fl = reinterpret_cast<int *>(cb + 64 * RB);  // [RB]
    const int lr = threadIdx.x % RB, part = threadIdx.x / RB;
    const int rep = blockIdx.x * RB + lr;
    const int rr = min(rep, r - 1);  // replicas past the last: computed, not written
    const int w = (n + 63) >> 6;
    {
        float s1[4] = {0.0f, 0.0f, 0.0f, 0.0f}, sall[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int q0 = 4 * part; q0 < n; q0 += 64) {
            float v[4][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float *xq = x + ((size_t)min(q0 + c, n - 1) * r + rr) * d;
#pragma unroll
                for (int mu = 0; mu < 4; ++mu) v[c][mu] = mu < d ? xq[mu] : 0.0f;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (q0 + c >= n) break;
                float s = 0.0f;
                for (int mu = 0; mu < d; ++mu) s = fmaf(v[c][mu], v[c][mu], s);
                sall[c] += s;
                s1[c] = fmaf(v[c][0], v[c][0], s1[c]);
                sx[(q0 + c) * RB + lr] = v[c][0];
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            ca[(4 * part + c) * RB + lr] = s1[c];
            cb[(4 * part + c) * RB + lr] = sall[c];
        }
        for (int q = n + part; q < feat_rows(n); q += kFeatThreads) sx[q * RB + lr] = 0.0f;
        if (part == 0) fl[lr] = 0;
    }
    class_tree<RB>(ca, cb);
    const float s1 = ca[lr], sall = cb[lr];
    // sign words, one per thread
    for (int wd = part; wd < w; wd += kFeatThreads) {
        uint64_t bits = 0;
        const int qn = min(64, n - 64 * wd);
        for (int i = 0; i < qn; ++i) bits |= (uint64_t)(sx[(64 * wd + i) * RB + lr] >= 0.0f) << i;
        if (rep < r) {
            uint64_t *old = prev + (size_t)rep * w + wd;
            const uint64_t mask = qn == 64 ? ~0ull : (1ull << qn) - 1ull;
            atomicAdd(&fl[lr], __popcll((*old ^ bits) & mask));
            *old = bits;
        }
    }
    __syncthreads();  // the sums have been read before they are written again
    switch (j_dtype) {
        case CHYM_J_I8: feat_products<RB, CHYM_J_I8>(n, j, sx, ca, cb); break;
        case CHYM_J_F32: feat_products<RB, CHYM_J_F32>(n, j, sx, ca, cb); break;
        case CHYM_J_BF16: feat_products<RB, CHYM_J_BF16>(n, j, sx, ca, cb); break;
        default: feat_products<RB, CHYM_J_FP8>(n, j, sx, ca, cb); break;
    }
    class_tree<RB>(ca, cb);
    if (part == 0 && rep < r) {
        float *f = feat + (size_t)rep * feat_stride + feat_off;
        f[0] = s1 > 0.0f ? -ca[lr] / ((float)n * s1) : 0.0f;
        f[1] = -cb[lr] / (float)n;
        f[2] = sall > 0.0f ? s1 / sall : 0.0f;
        f[3] = (float)fl[lr] / (float)n;
    }
}

// One replica per wavefront, for sizes whose first components of 16 replicas do
// not fit LDS.  LDS: the first components x_{p,1} [n] and the signs as +-1 [n].
__global__ __launch_bounds__(64) void k_features_one(int n, int d, int r, const void *__restrict__ j, int j_dtype,
                                                 const float *__restrict__ x, uint64_t *__restrict__ prev,
                                                 float *__restrict__ feat, int feat_stride, int feat_off) {
    extern __shared__ float shf[];
    float *x1 = shf;       // [n]
    float *sg = shf + n;   // [n]
    const int lane = threadIdx.x;
    const int rep = blockIdx.x;
    if (rep >= r) return;
    const int w = (n + 63) >> 6;
    float s1 = 0.0f, sall = 0.0f;
    int flips = 0;
    for (int q = lane; q < n; q += 64) {
        const float *xq = x + ((size_t)q * r + rep) * d;
        float s = 0.0f;
        for (int mu = 0; mu < d; ++mu) s = fmaf(xq[mu], xq[mu], s);
        sall += s;
        s1 = fmaf(xq[0], xq[0], s1);
        x1[q] = xq[0];
        const bool up = xq[0] >= 0.0f;
        sg[q] = up ? 1.0f : -1.0f;
        const bool was = (prev[(size_t)rep * w + (q >> 6)] >> (q & 63)) & 1ull;
        flips += (up != was);
    }
    __syncthreads();
    // column sums: G_q = sum_p J_pq x_{p,1}, h_q = sum_p J_pq sigma_p, so that
    // x_1^T J x_1 = sum_q x_{q,1} G_q and sigma^T J sigma = sum_q sigma_q h_q
    float quad = 0.0f, eis = 0.0f;
    for (int q = lane; q < n; q += 64) {
        float gq = 0.0f, hq = 0.0f;
        for (int p = 0; p < n; ++p) {
            const float jv = coupling(j, j_dtype, n, p, q);
            gq = fmaf(jv, x1[p], gq);
            hq = fmaf(jv, sg[p], hq);
        }
        quad = fmaf(x1[q], gq, quad);
        eis = fmaf(sg[q], hq, eis);
    }
    quad = wsum(quad);
    eis = wsum(eis);
    s1 = wsum(s1);
    sall = wsum(sall);
    flips = wsum(flips);
    // new sign words (one per 64 spins, built by the lanes that own them)
    __syncthreads();
    for (int wd = 0; wd < w; ++wd) {
        const int q = wd * 64 + lane;
        const bool up = q < n && sg[q] > 0.0f;
        const uint64_t bits = __ballot(up);
        if (lane == 0) prev[(size_t)rep * w + wd] = bits;
    }
    if (lane == 0) {
        float *f = feat + (size_t)rep * feat_stride + feat_off;
        f[0] = s1 > 0.0f ? -quad / ((float)n * s1) : 0.0f;
        f[1] = -eis / (float)n;
        f[2] = sall > 0.0f ? s1 / sall : 0.0f;
        f[3] = (float)flips / (float)n;
    }
}

// Standardizes every feature column within each group of `group`
// consecutive replicas (one pump's batch of runs): (f - mean) / sd, with the
// mean and the population standard deviation of the group, 0 where sd = 0.
// Sums in a fixed order: 256 strided partial sums per column, then a tree.  A
// block takes four columns of one group (1024 threads: 256 partial sums x 4
// columns, 16 bytes of a row per wavefront quarter); one block per group with
// its columns in turn left most of the chip idle (20 groups of 1000: 132 us;
// now 7.4 us).
constexpr int kStdCols = 4;

__global__ __launch_bounds__(256 * kStdCols) void k_standardize(int group, const float *__restrict__ in,
                                                                float *__restrict__ out) {
    __shared__ float red[256][kStdCols];
    const int t = threadIdx.x / kStdCols, cc = threadIdx.x % kStdCols;
    const size_t base = (size_t)blockIdx.x * group * kFeat + blockIdx.y * kStdCols + cc;
    auto tree = [&](float v) {
        red[t][cc] = v;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (t < h) red[t][cc] += red[t + h][cc];
            __syncthreads();
        }
        const float s = red[0][cc];
        __syncthreads();
        return s;
    };
    float sum = 0.0f;
    for (int i = t; i < group; i += 256) sum += in[base + (size_t)i * kFeat];
    const float mean = tree(sum) / (float)group;
    float ss = 0.0f;
    for (int i = t; i < group; i += 256) {
        const float v = in[base + (size_t)i * kFeat] - mean;
        ss = fmaf(v, v, ss);
    }
    const float sd = sqrtf(tree(ss) / (float)group);
    for (int i = t; i < group; i += 256) {
        const float v = in[base + (size_t)i * kFeat];
        out[base + (size_t)i * kFeat] = sd > 0.0f ? (v - mean) / sd : 0.0f;
    }
}

// Order-preserving map of a float to an unsigned key (NaN lowest).
__device__ __forceinline__ uint32_t score_key(float v) {
    if (v != v) return 0u;
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Exclusive prefix count of pred over the block in thread order, and the total.
template <int B>
__device__ __forceinline__ int block_scan(bool pred, int *red, int *total) {
    const uint64_t m = __ballot(pred);
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    if (ln == 0) red[wv] = __popcll(m);
    __syncthreads();
    int before = 0, tot = 0;
    for (int i = 0; i < B / 64; ++i) {
        if (i < wv) before += red[i];
        tot += red[i];
    }
    __syncthreads();
    *total = tot;
    return before + __popcll(m & ((ln == 0) ? 0ull : (~0ull >> (64 - ln))));
}

// For each group of `group` consecutive scores, the indices of its `keep`
// highest scores (equal scores: the lower index first; NaN lowest), written
// in ascending order to idx[g * keep ...] as global replica indices.  One
// block per group: a radix search over the four bytes of the keys, highest
// first (a histogram of the byte among the keys that match the bytes found so
// far, then the byte that holds the keep-th largest key), then one ordered
// pass writes the indices.  Four passes over the scores in place of a
// bisection's 32 (20 groups of 1000: 21 us; now 6.6 us).
__global__ __launch_bounds__(1024) void k_select_top(int group, int keep, const float *__restrict__ score,
                                                     int32_t *__restrict__ idx) {
    __shared__ int red[16];
    __shared__ int hist[256];
    __shared__ int found[2];  // the byte, and how many keys lie above it
    const size_t base = (size_t)blockIdx.x * group;
    uint32_t t = 0u;  // bytes found so far
    int eq_left = keep;  // keys still to keep among those that match them
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (threadIdx.x < 256) hist[threadIdx.x] = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < group; i += 1024) {
            const uint32_t k = score_key(score[base + i]);
            if (shift == 24 || (k >> (shift + 8)) == (t >> (shift + 8))) atomicAdd(&hist[(k >> shift) & 0xffu], 1);
        }
        __syncthreads();
        if (threadIdx.x < 64) {
            // lane l holds bytes 255 - 4l .. 252 - 4l: counts above its first
            int c[4], sum = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = hist[255 - 4 * (int)threadIdx.x - u];
                sum += c[u];
            }
            int above = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(above, off, 64);
                if ((int)threadIdx.x >= off) above += o;
            }
            above -= sum;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (above < eq_left && above + c[u] >= eq_left) {  // one lane and byte
                    found[0] = 255 - 4 * (int)threadIdx.x - u;
                    found[1] = above;
                }
                above += c[u];
            }
        }
        __syncthreads();
        t |= (uint32_t)found[0] << shift;
        eq_left -= found[1];
    }
    int out = 0;
    for (int i0 = 0; i0 < group; i0 += 1024) {
        const int i = i0 + threadIdx.x;
        const uint32_t k = i < group ? score_key(score[base + i]) : 0u;
        int eq_tot = 0;
        const int eq_before = block_scan<1024>(i < group && k == t, red, &eq_tot);
        const bool take = i < group && (k > t || (k == t && eq_before < eq_left));
        int tot = 0;
        const int pos = block_scan<1024>(take, red, &tot);
        if (take) idx[(size_t)blockIdx.x * keep + out + pos] = (int32_t)(base + i);
        out += tot;
        eq_left -= eq_tot < eq_left ? eq_tot : eq_left;
    }
}

// x_dst[p][j][mu] = x_src[p][idx[j]][mu] and pump_dst[j] = pump_src[idx[j]].
__global__ __launch_bounds__(256) void k_gather_replicas(int n, int d, int r_src, const float *__restrict__ x_src,
                                                         const float *__restrict__ pump_src, int m,
                                                         const int32_t *__restrict__ idx, float *__restrict__ x_dst,
                                                         float *__restrict__ pump_dst) {
    const size_t tot = (size_t)n * m * d;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < tot; e += (size_t)gridDim.x * blockDim.x) {
        const int mu = (int)(e % d);
        const size_t jq = e / d;
        const int jr = (int)(jq % m);
        const size_t p = jq / m;
        x_dst[e] = x_src[(p * r_src + idx[jr]) * d + mu];
        if (p == 0 && mu == 0 && pump_dst) pump_dst[jr] = pump_src[idx[jr]];
    }
}

hipError_t launch_features(int n, int d, int r, const void *j, int j_dtype, const float *x, uint64_t *prev,
                           float *feat, int feat_stride, int feat_off, hipStream_t stream) {
    // 32 replicas per block while their first components fit LDS (n <= 1120), then
    // 16 (n <= 2400), then one replica per wavefront
    constexpr size_t kMax = 159 * 1024;
    if (feat_lds(n, 16) > kMax) {
        hipLaunchKernelGGL(k_features_one, dim3(r), dim3(64), sizeof(float) * 2 * (size_t)n, stream, n, d, r, j, j_dtype,
                           x, prev, feat, feat_stride, feat_off);
        return hipGetLastError();
    }
    const bool wide = feat_lds(n, 32) <= kMax;
    const int rb = wide ? 32 : 16;
    const size_t lds = feat_lds(n, rb);
    auto *fn = wide ? k_features<32> : k_features<16>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fn, dim3((r + rb - 1) / rb), dim3(rb * kFeatThreads), lds, stream, n, d, r, j, j_dtype, x, prev,
                       feat, feat_stride, feat_off);
    return hipGetLastError();
}

// Sign words of the initial state (the reference of the first checkpoint): the
// readout's spin words.
hipError_t launch_sign_words(int n, int d, int r, const float *x, uint64_t *words, hipStream_t stream) {
    return launch_readout(n, d, r, x, words, nullptr, nullptr, stream);
}

hipError_t launch_standardize(int groups, int group, const float *in, float *out, hipStream_t stream) {
    if (groups <= 0) return hipSuccess;
    for (int g = 0; g < groups; g += max_blocks(256 * kStdCols)) {
        const size_t at = (size_t)g * group * kFeat;
        hipLaunchKernelGGL(k_standardize, dim3(std::min(groups - g, max_blocks(256 * kStdCols)), kFeat / kStdCols),
                           dim3(256 * kStdCols), 0, stream, group, in + at, out + at);
    }
    return hipGetLastError();
}

hipError_t launch_select_top(int groups, int group, int keep, const float *score, int32_t *idx, hipStream_t stream) {
    if (groups <= 0 || keep <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_select_top, dim3(groups), dim3(1024), 0, stream, group, keep, score, idx);
    return hipGetLastError();
}

hipError_t launch_gather_replicas(int n, int d, int r_src, const float *x_src, const float *pump_src, int m,
                                  const int32_t *idx, float *x_dst, float *pump_dst, hipStream_t stream) {
    if (m <= 0) return hipSuccess;
    const size_t tot = (size_t)n * m * d;
    const unsigned blocks = (unsigned)std::min<size_t>((tot + 255) / 256, 65536);
    hipLaunchKernelGGL(k_gather_replicas, dim3(blocks), dim3(256), 0, stream, n, d, r_src, x_src, pump_src, m, idx,
                       x_dst, pump_dst);
    return hipGetLastError();
}

// ------------------------------------------------------------------ MLP
// Parameter block layout (float32 master and bf16 copy use the same order):
//   W1 [H1][F], b1 [H1], W2 [H2][H1], b2 [H2], w3 [H2], b3 [1]
constexpr int kF = 32, kH1 = 128, kH2 = 128;
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kH1 * kF;
constexpr int kOffW2 = kOffB1 + kH1;
constexpr int kOffB2 = kOffW2 + kH2 * kH1;
constexpr int kOffW3 = kOffB2 + kH2;
constexpr int kOffB3 = kOffW3 + kH2;
constexpr int kParams = kOffB3 + 1;
static_assert(kParams == CHYM_MLP_PARAMS && kF == CHYM_FEATURES, "parameter block must match chym.h");

__device__ __forceinline__ float bf(const __bf16 *w, int i) { return (float)w[i]; }

typedef __attribute__((ext_vector_type(2))) float mlp_f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 mlp_bf16x2;
typedef __attribute__((ext_vector_type(4))) __bf16 mlp_bf16x4;

__device__ __forceinline__ mlp_bf16x2 mlp_pack(float a, float b) {
    return __builtin_convertvector((mlp_f32x2){a, b}, mlp_bf16x2);
}

__device__ __forceinline__ bf16x8 mlp_join(mlp_bf16x2 a, mlp_bf16x2 b, mlp_bf16x2 c, mlp_bf16x2 d) {
    const mlp_bf16x4 lo = __builtin_shufflevector(a, b, 0, 1, 2, 3);
    const mlp_bf16x4 hi = __builtin_shufflevector(c, d, 0, 1, 2, 3);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ mlp_bf16x4 mlp_load4(const __bf16 *p) { return *reinterpret_cast<const mlp_bf16x4 *>(p); }

// Forward pass on the matrix cores, one wavefront per 16 samples (the batch
// tail padded with zero features, its outputs not written).  Both hidden
// layers are computed transposed, H^T = W X^T, with v_mfma_f32_16x16x32_bf16:
// the weights are the A operand (16 units x 32 inputs per fragment), the
// layer input the B operand (32 inputs x 16 samples), and lane (j, g) of a
// 16 x 16 result holds units 4 g + v of sample j.  The second layer's K
// chunk c is the rows lane (j, g) already holds in result tiles 2c and 2c+1
// (slot s: unit 32 c + 16 (s >> 2) + 4 g + (s & 3)), with W2's columns read in
// that order, so its B operand comes from the lane's own registers.  The
// weights are staged in LDS once per block, whose wavefronts take groups of 16
// samples in turn: read from L2 by every wavefront, 64 eight-byte loads per
// lane over rows 256 bytes apart set the time (8192 samples: 15.5 us, 20000:
// 20; now 10.7 and 9.7).
// Writes the logit, and h1 (the rounded first-layer activations, the second
// layer's input) and h2 when given, [batch][128] each.
constexpr int kW2Row = kH1 + 8;  // elements of a W2 row in LDS: 16 rows of a fragment start on different banks

__global__ __launch_bounds__(256) void k_mlp_forward(int batch, const float *__restrict__ feat,
                                                     const __bf16 *__restrict__ wg, float *__restrict__ logit,
                                                     float *__restrict__ h1, float *__restrict__ h2) {
    __shared__ __align__(16) __bf16 sw1[kH1 * kF];
    __shared__ __align__(16) __bf16 sw2[kH2 * kW2Row];
    __shared__ __align__(16) __bf16 sb[3 * kH1];  // b1, b2, w3
    for (int i = threadIdx.x; i < kH1 * kF / 8; i += blockDim.x)
        reinterpret_cast<bf16x8 *>(sw1)[i] = reinterpret_cast<const bf16x8 *>(wg + kOffW1)[i];
    for (int i = threadIdx.x; i < kH2 * kH1 / 8; i += blockDim.x)
        *reinterpret_cast<bf16x8 *>(sw2 + (i / (kH1 / 8)) * kW2Row + (i % (kH1 / 8)) * 8) =
            reinterpret_cast<const bf16x8 *>(wg + kOffW2)[i];
    for (int i = threadIdx.x; i < kH1; i += blockDim.x) {
        sb[i] = wg[kOffB1 + i];
        sb[kH1 + i] = wg[kOffB2 + i];
        sb[2 * kH1 + i] = wg[kOffW3 + i];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int j = lane & 15, g = lane >> 4;
    const int waves = gridDim.x * (blockDim.x >> 6);
    for (int s0 = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 16; s0 < batch; s0 += 16 * waves) {
        asm volatile("" ::: "memory");  // the weights stay in LDS, read again for every group
        const int smp = s0 + j;
        const bool ok = smp < batch;
        // layer 1: B operand = features 8 g .. 8 g + 7 of sample j, rounded to bf16
        bf16x8 bx;
        {
            float v[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) v[s] = ok ? feat[(size_t)smp * kF + 8 * g + s] : 0.0f;
            bx = mlp_join(mlp_pack(v[0], v[1]), mlp_pack(v[2], v[3]), mlp_pack(v[4], v[5]), mlp_pack(v[6], v[7]));
        }
        f32x4 a1[8];
#pragma unroll
        for (int I = 0; I < 8; ++I) {
            const mlp_bf16x4 b = mlp_load4(sb + 16 * I + 4 * g);
            a1[I] = f32x4{(float)b[0], (float)b[1], (float)b[2], (float)b[3]};
            // A fragment: W1 row 16 I + j, inputs 8 g .. 8 g + 7
            const bf16x8 aw = *reinterpret_cast<const bf16x8 *>(sw1 + (16 * I + j) * kF + 8 * g);
            a1[I] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw, bx, a1[I], 0, 0, 0);
        }
        // ReLU, then the rounded activations (the second layer's input)
        mlp_bf16x2 hp[8][2];
#pragma unroll
        for (int I = 0; I < 8; ++I) {
            float r[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) r[v] = a1[I][v] > 0.0f ? a1[I][v] : 0.0f;
            hp[I][0] = mlp_pack(r[0], r[1]);
            hp[I][1] = mlp_pack(r[2], r[3]);
            if (h1 && ok) {
                float4 o;
                o.x = (float)hp[I][0][0];
                o.y = (float)hp[I][0][1];
                o.z = (float)hp[I][1][0];
                o.w = (float)hp[I][1][1];
                *reinterpret_cast<float4 *>(h1 + (size_t)smp * kH1 + 16 * I + 4 * g) = o;
            }
        }
        // layer 2
        f32x4 a2[8];
#pragma unroll
        for (int I = 0; I < 8; ++I) {
            const mlp_bf16x4 b = mlp_load4(sb + kH1 + 16 * I + 4 * g);
            a2[I] = f32x4{(float)b[0], (float)b[1], (float)b[2], (float)b[3]};
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bf16x8 bh = mlp_join(hp[2 * c][0], hp[2 * c][1], hp[2 * c + 1][0], hp[2 * c + 1][1]);
#pragma unroll
            for (int I = 0; I < 8; ++I) {
                const __bf16 *row = sw2 + (16 * I + j) * kW2Row + 32 * c + 4 * g;
                const mlp_bf16x4 lo = mlp_load4(row), hi = mlp_load4(row + 16);
                const bf16x8 aw = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                a2[I] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw, bh, a2[I], 0, 0, 0);
            }
        }
        // ReLU and the output layer: float32 dot with w3 over the lane's units,
        // then over the four lanes of the sample
        float part = 0.0f;
#pragma unroll
        for (int I = 0; I < 8; ++I) {
            const mlp_bf16x4 w3 = mlp_load4(sb + 2 * kH1 + 16 * I + 4 * g);
            float r[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                r[v] = a2[I][v] > 0.0f ? a2[I][v] : 0.0f;
                part = fmaf((float)w3[v], r[v], part);
            }
            if (h2 && ok) *reinterpret_cast<float4 *>(h2 + (size_t)smp * kH2 + 16 * I + 4 * g) = float4{r[0], r[1], r[2], r[3]};
        }
        part += __shfl_xor(part, 16, 64);
        part += __shfl_xor(part, 32, 64);
        if (g == 0 && ok) logit[smp] = (float)wg[kOffB3] + part;
    }
}

// Backward pass of the mean binary cross-entropy over the batch, in two
// deterministic stages:
//  1. k_mlp_backward, blocks of four wavefronts that take chunks of 32 samples
//     in turn: dz = (sigmoid(z) - y) / B, d2 = dz w3 [h2 > 0],
//     d1 = (W2^T d2) [h1 > 0] and the loss terms, then the chunk's weight
//     gradients (sums over its samples of outer products), held in registers
//     over a block's chunks and written once as the block's partial gradient;
//  2. k_mlp_reduce: the partials summed over blocks in block order.
// All products run on v_mfma_f32_16x16x4_f32 (float32 operands and sums).  The
// three kernels that this replaces kept one sample per thread with rows 512
// bytes apart, and wrote a partial gradient per 16 samples (batch 8192: 137 us,
// 38 us and 122 us to sum the 512 partials; now 21 us and 8.8 us, of which the
// matrix products take 5).
constexpr int kBS = 32;          // samples of a chunk
constexpr int kBBlocks = 256;    // partial gradients at most
constexpr int kBRow = kH1 + 16;  // floats of an LDS row: the four rows of a product's lanes on different banks
constexpr int kXRow = kF + 16;

__global__ __launch_bounds__(256) void k_mlp_backward(int batch, const float *__restrict__ feat,
                                                      const float *__restrict__ label,
                                                      const __bf16 *__restrict__ wb,
                                                      const float *__restrict__ logit, const float *__restrict__ h1,
                                                      const float *__restrict__ h2, float *__restrict__ partial,
                                                      float *__restrict__ loss) {
    __shared__ __align__(16) float sd2[kBS * kBRow], sh1[kBS * kBRow], sd1[kBS * kBRow], sx[kBS * kXRow];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int col = lane & 15, g = lane >> 4;
    // loads: eight samples at a time, four of a row's 128 values per thread
    const int ls = threadIdx.x >> 5, lc = (threadIdx.x & 31) * 4;
    float w3[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) w3[u] = bf(wb, kOffW3 + lc + u);
    // A operand of d1: W2^T, rows i of the wavefront's two tiles, k = o; step
    // (m, u) takes o = 16 m + 4 g + u
    float wt[2][8][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int u = 0; u < 4; ++u) wt[t][m][u] = bf(wb, kOffW2 + (16 * m + 4 * g + u) * kH1 + 16 * (2 * w + t) + col);

    f32x4 gw2[2][8], gw1[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int k = 0; k < 8; ++k) gw2[t][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 2; ++k) gw1[t][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    float gb1[2][4] = {}, gw3[4] = {}, gb2[4] = {}, gb3 = 0.0f;

    for (int s0 = blockIdx.x * kBS; s0 < batch; s0 += gridDim.x * kBS) {
        __syncthreads();  // the previous chunk's products have read LDS
#pragma unroll
        for (int k = 0; k < kBS / 8; ++k) {
            const int s = 8 * k + ls;
            const bool ok = s0 + s < batch;
            const size_t row = (size_t)(ok ? s0 + s : 0);
            float4 a1 = *reinterpret_cast<const float4 *>(h1 + row * kH1 + lc);
            float4 a2 = *reinterpret_cast<const float4 *>(h2 + row * kH2 + lc);
            const float z = logit[row], y = label[row];
            const float p = 1.0f / (1.0f + expf(-z));
            const float dz = ok ? (p - y) / (float)batch : 0.0f;
            if (!ok) a1 = a2 = float4{0.0f, 0.0f, 0.0f, 0.0f};
            if (lc == 0 && ok) {
                loss[row] = (z > 0.0f ? z + log1pf(expf(-z)) : log1pf(expf(z))) - y * z;
                gb3 += dz;
            }
            const float v[4] = {a2.x, a2.y, a2.z, a2.w};
            float d2[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                d2[u] = v[u] > 0.0f ? dz * w3[u] : 0.0f;
                gw3[u] = fmaf(dz, v[u], gw3[u]);
                gb2[u] += d2[u];
            }
            *reinterpret_cast<float4 *>(sd2 + s * kBRow + lc) = float4{d2[0], d2[1], d2[2], d2[3]};
            *reinterpret_cast<float4 *>(sh1 + s * kBRow + lc) = a1;
        }
        {
            // the first layer's input as the forward pass rounds it
            const int s = threadIdx.x >> 3, c = (threadIdx.x & 7) * 4;
            float4 v = float4{0.0f, 0.0f, 0.0f, 0.0f};
            if (s0 + s < batch) v = *reinterpret_cast<const float4 *>(feat + (size_t)(s0 + s) * kF + c);
            *reinterpret_cast<float4 *>(sx + s * kXRow + c) =
                float4{(float)(__bf16)v.x, (float)(__bf16)v.y, (float)(__bf16)v.z, (float)(__bf16)v.w};
        }
        __syncthreads();
        // d1 for the wavefront's rows i of tiles 2w, 2w+1 and all samples
        f32x4 acc[2][kBS / 16];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < kBS / 16; ++q) acc[t][q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int m = 0; m < 8; ++m) {
#pragma unroll
            for (int q = 0; q < kBS / 16; ++q) {
                const f32x4 b = *reinterpret_cast<const f32x4 *>(sd2 + (16 * q + col) * kBRow + 16 * m + 4 * g);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[t][m][u], b[u], acc[t][q], 0, 0, 0);
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < kBS / 16; ++q) {
                const int at = (16 * q + col) * kBRow + 16 * (2 * w + t) + 4 * g;
                const f32x4 a1 = *reinterpret_cast<const f32x4 *>(sh1 + at);
                f32x4 d;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    d[v] = a1[v] > 0.0f ? acc[t][q][v] : 0.0f;
                    gb1[t][v] += d[v];
                }
                *reinterpret_cast<f32x4 *>(sd1 + at) = d;
            }
        __syncthreads();
        // weight gradients: rows o of tiles 2w, 2w+1, k = sample
#pragma unroll
        for (int m = 0; m < kBS / 4; ++m) {
            const int r = 4 * m + g;
            float a2[2], a1[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                a2[t] = sd2[r * kBRow + 16 * (2 * w + t) + col];
                a1[t] = sd1[r * kBRow + 16 * (2 * w + t) + col];
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float b = sh1[r * kBRow + 16 * k + col];
#pragma unroll
                for (int t = 0; t < 2; ++t) gw2[t][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[t], b, gw2[t][k], 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float b = sx[r * kXRow + 16 * k + col];
#pragma unroll
                for (int t = 0; t < 2; ++t) gw1[t][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[t], b, gw1[t][k], 0, 0, 0);
            }
        }
    }

    float *out = partial + (size_t)blockIdx.x * kParams;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int o = 16 * (2 * w + t) + 4 * g + v;
#pragma unroll
            for (int k = 0; k < 8; ++k) out[kOffW2 + o * kH1 + 16 * k + col] = gw2[t][k][v];
#pragma unroll
            for (int k = 0; k < 2; ++k) out[kOffW1 + o * kF + 16 * k + col] = gw1[t][k][v];
            float b = gb1[t][v];
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) b += __shfl_xor(b, off, 64);
            if (col == 0) out[kOffB1 + o] = b;
        }
    // the loading threads' sums: eight sample rows per column
    __syncthreads();
    *reinterpret_cast<float4 *>(sd2 + ls * kBRow + lc) = float4{gw3[0], gw3[1], gw3[2], gw3[3]};
    *reinterpret_cast<float4 *>(sh1 + ls * kBRow + lc) = float4{gb2[0], gb2[1], gb2[2], gb2[3]};
    if (lc == 0) sx[ls] = gb3;
    __syncthreads();
    if (threadIdx.x < kH2) {
        float a = 0.0f, b = 0.0f;
        for (int s = 0; s < 8; ++s) {
            a += sd2[s * kBRow + threadIdx.x];
            b += sh1[s * kBRow + threadIdx.x];
        }
        out[kOffW3 + threadIdx.x] = a;
        out[kOffB2 + threadIdx.x] = b;
    }
    if (threadIdx.x == 0) {
        float a = 0.0f;
        for (int s = 0; s < 8; ++s) a += sx[s];
        out[kOffB3] = a;
    }
}

// 64 parameters per block, four threads each (every fourth partial, then their
// four sums in order).
__global__ __launch_bounds__(256) void k_mlp_reduce(int blocks, const float *__restrict__ partial,
                                                    float *__restrict__ grad) {
    __shared__ float red[4][64];
    const int c = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + c;
    float acc = 0.0f;
    if (i < kParams) {
        int b = part;
        for (; b + 28 < blocks; b += 32) {  // eight in flight
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(b + 4 * u) * kParams + i];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += v[u];
        }
        for (; b < blocks; b += 4) acc += partial[(size_t)b * kParams + i];
    }
    red[part][c] = acc;
    __syncthreads();
    if (part == 0 && i < kParams) grad[i] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
}

// Adam (Kingma & Ba) on the float32 master weights; refreshes the bf16 copy.
__global__ __launch_bounds__(256) void k_mlp_adam(float *__restrict__ wm, __bf16 *__restrict__ wb,
                                                  float *__restrict__ m, float *__restrict__ v,
                                                  const float *__restrict__ grad, float lr, float b1, float b2,
                                                  float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kParams) return;
    const float gi = grad[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1, vh = vi / c2;
    const float wi = wm[i] - lr * mh / (sqrtf(vh) + eps);
    wm[i] = wi;
    wb[i] = (__bf16)wi;
}

__global__ __launch_bounds__(256) void k_to_bf16(const float *__restrict__ src, __bf16 *__restrict__ dst, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (__bf16)src[i];
}

int mlp_param_count() { return kParams; }

constexpr int kForwardBlocks = 768;  // three blocks (42 KB of weights each) on every CU

hipError_t launch_mlp_forward(int batch, const float *feat, const void *wb, float *logit, float *h1, float *h2,
                              hipStream_t stream) {
    if (batch <= 0) return hipSuccess;
    const int waves = (batch + 15) / 16;  // 16 samples per wavefront, 4 wavefronts per block
    hipLaunchKernelGGL(k_mlp_forward, dim3(std::min((waves + 3) / 4, kForwardBlocks)), dim3(256), 0, stream, batch, feat,
                       reinterpret_cast<const __bf16 *>(wb), logit, h1, h2);
    return hipGetLastError();
}

// Backward scratch: a partial gradient per block of the backward kernel.  The
// size that callers were always asked for (one partial gradient per 16 samples
// and three activations per sample) holds them.
size_t mlp_backward_scratch_floats(int batch) {
    return (size_t)batch * (1 + kH1 + kH2) + (size_t)((batch + 15) / 16) * kParams;
}

hipError_t launch_mlp_backward(int batch, const float *feat, const float *label, const void *wb, const float *logit,
                               const float *h1, const float *h2, float *scratch, float *grad, float *loss,
                               hipStream_t stream) {
    if (batch <= 0) return hipSuccess;
    const int blocks = std::min((batch + kBS - 1) / kBS, kBBlocks);
    hipLaunchKernelGGL(k_mlp_backward, dim3(blocks), dim3(256), 0, stream, batch, feat, label,
                       reinterpret_cast<const __bf16 *>(wb), logit, h1, h2, scratch, loss);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_reduce, dim3((kParams + 63) / 64), dim3(256), 0, stream, blocks, scratch, grad);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float *wm, void *wb, float *m, float *v, const float *grad, float lr, float b1, float b2,
                           float eps, int t, hipStream_t stream) {
    const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_mlp_adam, dim3((kParams + 255) / 256), dim3(256), 0, stream, wm,
                       reinterpret_cast<__bf16 *>(wb), m, v, grad, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float *src, void *dst, int n, hipStream_t stream) {
    hipLaunchKernelGGL(k_to_bf16, dim3((n + 255) / 256), dim3(256), 0, stream, src, reinterpret_cast<__bf16 *>(dst),
                       n);
    return hipGetLastError();
}

}  // namespace chym
