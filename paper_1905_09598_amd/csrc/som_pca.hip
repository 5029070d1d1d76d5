// Principal components of the data and the linear initialisation of a map
// (paper Sec. 6D, Fig. 2): the prototypes start as a regular grid in the
// plane through the data mean spanned by the two largest principal
// components, and the map size follows from the two largest variances.
//
// On the device:
//   1. column means (fp64 partial sums over row chunks, summed in a fixed
//      order);
//   2. the covariance C = (1/n) sum_i (x_i - mu)(x_i - mu)^T on the fp32
//      matrix cores (v_mfma_f32_16x16x4_f32), one 64 x 64 tile per
//      workgroup, upper tiles only, mirrored on the store;
//   3. subspace iteration with kPcaBlock vectors: Y = C V over the chip, each
//      workgroup also leaving its rows' parts of the 8 x 8 products V^T Y,
//      Y^T Y and V^T V (fp64); one small workgroup adds them and finds the
//      8 x 8 matrix R that makes Y R orthonormal (Cholesky of Y^T Y in fp64),
//      which the next step applies as it reads Y.  Every 8th step that
//      workgroup also does the Rayleigh-Ritz step (Jacobi eigen-pairs Q of
//      V^T Y) and the residuals |y_a - theta_a v_a| of the top two Ritz pairs,
//      |Y q - theta V q|^2 = q'(Y^T Y)q - 2 theta q'(V^T Y)q + theta^2
//      q'(V^T V)q;
//   4. the grid itself.
// A step thus reads C once and has no pass of its own over the long vectors:
// on one workgroup, the Rayleigh-Ritz step and modified Gram-Schmidt over
// vectors of 2000 took 384 us a step, ten times the product with C; a step now
// takes 14 us for the product and 5 (27 with the Ritz pairs) for the rest, and
// the initialisation of a 20 x 20 map from 2000 x 2000 samples 0.84 ms instead
// of 8.1.
#include "som_internal.h"

#include <math.h>

namespace som {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kMeanChunks = 64;
constexpr int kCovTile = 64;
constexpr int kCovK = 32;
constexpr int kCovPitch = kCovTile + 16;  // the four rows of an operand read hit all 64 banks
constexpr int kMatvecRows = 8;      // rows of C per workgroup (2 per wave)
constexpr int kMatvecChunk = 1024;  // columns of V staged in LDS at a time
constexpr int kOrthThreads = 1024;
constexpr int kProducts = 3 * kPcaBlock * kPcaBlock;  // V^T Y, Y^T Y, V^T V

__global__ __launch_bounds__(256) void col_partial_kernel(const float *X, int64_t n, int32_t d,
                                                          double *part) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int chunk = blockIdx.y;
    if (j >= d) return;
    const int64_t r0 = n * chunk / kMeanChunks, r1 = n * (chunk + 1) / kMeanChunks;
    double s = 0.0;
    for (int64_t i = r0; i < r1; ++i) s += (double)X[i * d + j];
    part[(int64_t)chunk * d + j] = s;
}

__global__ __launch_bounds__(256) void col_mean_kernel(const double *part, int64_t n, int32_t d,
                                                       float *mean) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= d) return;
    double s = 0.0;
    for (int c = 0; c < kMeanChunks; ++c) s += part[(int64_t)c * d + j];
    mean[j] = (float)(s / (double)n);
}

// Upper tile t of the nt x nt tile grid, row-major over ti <= tj.
__device__ inline void upper_tile(int t, int nt, int &ti, int &tj) {
    int i = 0, left = t;
    while (left >= nt - i) {
        left -= nt - i;
        ++i;
    }
    ti = i;
    tj = i + left;
}

// Each slab of kCovK samples is loaded into registers while the one before it
// is multiplied (loads clamped into X, what lies outside zeroed as it goes to
// LDS): without that the kernel waited for memory once per slab (254 us at
// n = d = 2000, now 139).  VEC4: whole aligned float4s of a row.
template <bool VEC4>
__global__ __launch_bounds__(256) void covariance_kernel(const float *X, int64_t n, int32_t d,
                                                         const float *mean, float *C) {
    __shared__ __align__(16) float As[kCovK][kCovPitch];
    __shared__ __align__(16) float Bs[kCovK][kCovPitch];
    const int nt = (d + kCovTile - 1) / kCovTile;
    int ti, tj;
    upper_tile(blockIdx.x, nt, ti, tj);
    const int i0 = ti * kCovTile, j0 = tj * kCovTile;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
    const int l16 = lane & 15, lk = lane >> 4;
    f4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f4{0.f, 0.f, 0.f, 0.f};
    // staging: rows sr and sr + 16 of a slab, columns sc .. sc + 3 of both tiles
    const int sc = 4 * (tid & 15), sr = tid >> 4;
    const auto load4 = [&](const float *x, int c) {
        f4 v;
        if (VEC4) {
            v = *reinterpret_cast<const f4 *>(x + (c < d ? c : d - 4));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = x[c + e < d ? c + e : d - 1];
        }
        return v;
    };
    const f4 mi = load4(mean, i0 + sc), mj = load4(mean, j0 + sc);
    f4 va[2], vb[2];
    const auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int64_t k = k0 + sr + 16 * r;
            const float *x = X + (k < n ? k : n - 1) * d;
            va[r] = load4(x, i0 + sc);
            vb[r] = load4(x, j0 + sc);
        }
    };
    fetch(0);
    for (int64_t k0 = 0; k0 < n; k0 += kCovK) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const bool in = k0 + sr + 16 * r < n;
            f4 a = va[r] - mi, b = vb[r] - mj;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = in && i0 + sc + e < d ? a[e] : 0.f;
                b[e] = in && j0 + sc + e < d ? b[e] : 0.f;
            }
            *reinterpret_cast<f4 *>(&As[sr + 16 * r][sc]) = a;
            *reinterpret_cast<f4 *>(&Bs[sr + 16 * r][sc]) = b;
        }
        __syncthreads();
        if (k0 + kCovK < n) fetch(k0 + kCovK);
#pragma unroll
        for (int ks = 0; ks < kCovK; ks += 4) {
            float a[2], b[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                a[u] = As[ks + lk][wm + 16 * u + l16];
                b[u] = Bs[ks + lk][wn + 16 * u + l16];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v)
                    acc[u][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], b[v], acc[u][v], 0, 0, 0);
        }
    }
    // acc[u][v][e]: row i0 + wm + 16u + 4 lk + e, column j0 + wn + 16v + l16
    const float inv_n = (float)(1.0 / (double)n);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = i0 + wm + 16 * u + 4 * lk + e, j = j0 + wn + 16 * v + l16;
                if (i < d && j < d) {
                    const float c = acc[u][v][e] * inv_n;
                    C[(int64_t)i * d + j] = c;
                    if (ti != tj) C[(int64_t)j * d + i] = c;
                }
            }
}

// Column-major P-vectors of row j times R: out[a] = sum_b in[b] R[b][a], one
// rounding.
__device__ inline void times_r(const float *in, int64_t d, int64_t j, const double *R,
                               float (&out)[kPcaBlock]) {
    constexpr int P = kPcaBlock;
    double v[P];
#pragma unroll
    for (int b = 0; b < P; ++b) v[b] = (double)in[b * d + j];
#pragma unroll
    for (int a = 0; a < P; ++a) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < P; ++b) s = fma(v[b], R[b * P + a], s);
        out[a] = (float)s;
    }
}

// V = Yin R and Y = C V for kMatvecRows rows of C per workgroup (Yin, Y: d x
// kPcaBlock, column-major), and the rows' parts of V^T Y, Y^T Y and V^T V into
// part[workgroup].  Bound by reading C (16 MB at d = 2000): 8 rows a workgroup,
// so that 250 of them share it.
__global__ __launch_bounds__(256) void matvec_kernel(const float *C, int32_t d, const float *Yin,
                                                     const double *R, float *Y, double *part) {
    constexpr int P = kPcaBlock;
    constexpr int RW = kMatvecRows / 4;  // rows per wave
    __shared__ float vs[kMatvecChunk * P];
    __shared__ double rs[P * P];
    __shared__ float vr[kMatvecRows][P], yr[kMatvecRows][P];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * kMatvecRows + wave * RW;
    if (tid < P * P) rs[tid] = R[tid];
    __syncthreads();
    if (tid < kMatvecRows) {
        const int64_t row = (int64_t)blockIdx.x * kMatvecRows + tid;
        float v[P];
        times_r(Yin, d, row < d ? row : d - 1, rs, v);
#pragma unroll
        for (int a = 0; a < P; ++a) vr[tid][a] = row < d ? v[a] : 0.f;
    }
    float acc[RW][P];
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int a = 0; a < P; ++a) acc[r][a] = 0.f;
    for (int c0 = 0; c0 < d; c0 += kMatvecChunk) {
        const int cn = d - c0 < kMatvecChunk ? d - c0 : kMatvecChunk;
        __syncthreads();
        for (int j = tid; j < cn; j += 256) {
            float v[P];
            times_r(Yin, d, c0 + j, rs, v);
#pragma unroll
            for (int a = 0; a < P; ++a) vs[j * P + a] = v[a];
        }
        __syncthreads();
#pragma unroll 4
        for (int j = lane; j < cn; j += 64) {
            float vv[P];
#pragma unroll
            for (int a = 0; a < P; ++a) vv[a] = vs[j * P + a];
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const int64_t row = r0 + r < d ? r0 + r : d - 1;  // clamped; unused past d
                const float c = C[row * d + c0 + j];
#pragma unroll
                for (int a = 0; a < P; ++a) acc[r][a] = fmaf(c, vv[a], acc[r][a]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int a = 0; a < P; ++a) {
            float s = acc[r][a];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
            acc[r][a] = s;
        }
    if (lane == 0)
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int64_t row = r0 + r;
#pragma unroll
            for (int a = 0; a < P; ++a) {
                yr[wave * RW + r][a] = row < d ? acc[r][a] : 0.f;
                if (row < d) Y[(int64_t)a * d + row] = acc[r][a];
            }
        }
    __syncthreads();
    if (tid < kProducts) {
        const int kind = tid / (P * P), a = tid / P % P, b = tid % P;
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < kMatvecRows; ++r)
            s += (double)(kind == 1 ? yr[r][a] : vr[r][a]) * (double)(kind == 2 ? vr[r][b] : yr[r][b]);
        part[(int64_t)blockIdx.x * kProducts + tid] = s;
    }
}

// Jacobi eigen-decomposition of the symmetric P x P matrix H in LDS by the
// first 4 P lanes of one wave: H <- diag, Q <- eigenvectors (columns).  A sweep
// is P - 1 rounds of P / 2 disjoint rotations (the circle method); lane (r, k)
// applies rotation r to column pair entries k, then to row pair entries k.
__device__ inline void jacobi_eigen(double (&H)[kPcaBlock][kPcaBlock],
                                    double (&Q)[kPcaBlock][kPcaBlock]) {
    constexpr int P = kPcaBlock;
    const int lane = threadIdx.x & 63, r = lane / P, k = lane % P;
    const bool mine = lane < P * P / 2;
    double scale = 0.0;  // squared norm: rotations keep it
    for (int e = 0; e < P * P; ++e) scale += H[e / P][e % P] * H[e / P][e % P];
    for (int sweep = 0; sweep < 60; ++sweep) {
        double off = 0.0;
        for (int i = 0; i < P; ++i)
            for (int j = i + 1; j < P; ++j) off += H[i][j] * H[i][j];
        if (!(off > 1e-30 * scale)) break;
        for (int round = 0; round < P - 1; ++round) {
            // pair r: (P - 1, round) or (round + r, round - r) modulo P - 1
            int p = 0, q = 0;
            double c = 1.0, s = 0.0;
            if (mine) {
                p = r == 0 ? P - 1 : (round + r) % (P - 1);
                q = r == 0 ? round : (round + P - 1 - r) % (P - 1);
                if (p > q) {
                    const int t = p;
                    p = q;
                    q = t;
                }
                const double apq = H[p][q];
                if (apq != 0.0) {
                    const double theta = (H[q][q] - H[p][p]) / (2.0 * apq);
                    const double t =
                        (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                    c = 1.0 / sqrt(t * t + 1.0);
                    s = t * c;
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (mine) {
                const double hp = H[k][p], hq = H[k][q], vp = Q[k][p], vq = Q[k][q];
                H[k][p] = c * hp - s * hq;
                H[k][q] = s * hp + c * hq;
                Q[k][p] = c * vp - s * vq;
                Q[k][q] = s * vp + c * vq;
            }
            __builtin_amdgcn_wave_barrier();
            if (mine) {
                const double hp = H[p][k], hq = H[q][k];
                H[p][k] = c * hp - s * hq;
                H[q][k] = s * hp + c * hq;
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// One workgroup: adds the `parts` rows of products (in a fixed order) and leaves
// R for the next step.  With `ritz` it first rotates to the Ritz basis and sets
// stats: theta_0, theta_1, residual_0, residual_1; with `last` R is the Ritz
// rotation alone (of the step's own V).  A direction below 3e-7 of the largest
// (the rank of the data, or noise) gets a zero column.
constexpr int kSmallThreads = 1024;
__global__ __launch_bounds__(kSmallThreads) void orthonormal_kernel(const double *part, int parts,
                                                                   double *R, double *stats,
                                                                   int ritz, int last) {
    constexpr int P = kPcaBlock, kGroups = kSmallThreads / kProducts;
    __shared__ double sums[kGroups][kProducts];
    __shared__ double prod[3][P][P], Qs[P][P], Hs[P][P], Es[P][P], theta[P];
    const int tid = threadIdx.x, grp = tid / kProducts, e = tid % kProducts;
    if (grp < kGroups) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        int k = grp;
        for (; k + 3 * kGroups < parts; k += 4 * kGroups)
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] += part[(int64_t)(k + q * kGroups) * kProducts + e];
        for (; k < parts; k += kGroups) s[0] += part[(int64_t)k * kProducts + e];
        sums[grp][e] = (s[0] + s[1]) + (s[2] + s[3]);
    }
    __syncthreads();
    if (tid < kProducts) {
        double s = sums[0][tid];
        for (int g = 1; g < kGroups; ++g) s += sums[g][tid];
        prod[tid / (P * P)][tid / P % P][tid % P] = s;
    }
    if (tid < P * P) Qs[tid / P][tid % P] = tid / P == tid % P ? 1.0 : 0.0;
    __syncthreads();
    if (ritz) {
        if (tid < P * P)
            Hs[tid / P][tid % P] =
                0.5 * (prod[0][tid / P][tid % P] + prod[0][tid % P][tid / P]);
        if (tid < P * P) Es[tid / P][tid % P] = tid / P == tid % P ? 1.0 : 0.0;
        __syncthreads();
        if (tid < 64) jacobi_eigen(Hs, Es);
        __syncthreads();
        if (tid < P) {  // Ritz values in descending order: column tid's place
            const double own = Hs[tid][tid];
            int place = 0;
            for (int i = 0; i < P; ++i)
                place += Hs[i][i] > own || (Hs[i][i] == own && i < tid) ? 1 : 0;
            for (int i = 0; i < P; ++i) Qs[i][place] = Es[i][tid];
            theta[place] = own;
        }
        __syncthreads();
        if (tid < 2) {
            const double th = theta[tid];
            double r2 = 0.0;
            for (int i = 0; i < P; ++i)
                for (int j = 0; j < P; ++j)
                    r2 += Qs[i][tid] * Qs[j][tid] *
                          (prod[1][i][j] - 2.0 * th * prod[0][i][j] + th * th * prod[2][i][j]);
            stats[tid] = th;
            stats[2 + tid] = sqrt(fmax(r2, 0.0));
        }
    }
    __syncthreads();
    if (last) {
        if (tid < P * P) R[tid] = Qs[tid / P][tid % P];
        return;
    }
    // S = Q^T (Y^T Y) Q (in place of V^T V), then S = U^T U and R = Q U^-1
    if (tid < P * P) {
        const int a = tid / P, b = tid % P;
        double s = 0.0;
        for (int i = 0; i < P; ++i)
            for (int j = 0; j < P; ++j) s += Qs[i][a] * prod[1][i][j] * Qs[j][b];
        prod[2][a][b] = s;
    }
    __syncthreads();
    if (tid < P) {
        // lane r: row r of Q U^-1, its column k once U's row k is known; every
        // lane factors S itself
        double U[P][P], out[P], top = 0.0;
#pragma unroll
        for (int k = 0; k < P; ++k) top = fmax(top, prod[2][k][k]);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            double pivot = prod[2][k][k];
#pragma unroll
            for (int i = 0; i < k; ++i) pivot -= U[i][k] * U[i][k];
            const double inv = pivot > 1e-13 * top ? 1.0 / sqrt(pivot) : 0.0;
#pragma unroll
            for (int j = k; j < P; ++j) {
                double s = prod[2][k][j];
#pragma unroll
                for (int i = 0; i < k; ++i) s -= U[i][k] * U[i][j];
                U[k][j] = s * inv;
            }
            double o = Qs[tid][k];
#pragma unroll
            for (int i = 0; i < k; ++i) o -= out[i] * U[i][k];
            out[k] = o * inv;
        }
#pragma unroll
        for (int k = 0; k < P; ++k) R[tid * P + k] = out[k];
    }
}

// V = A R1 and then V R2, column-major (the Ritz vectors of a step's own V).
__global__ __launch_bounds__(256) void ritz_vectors_kernel(const float *A, const double *R1,
                                                           const double *R2, int32_t d,
                                                           float *V) {
    constexpr int P = kPcaBlock;
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= d) return;
    float v[P];
    times_r(A, d, j, R1, v);
#pragma unroll
    for (int a = 0; a < P; ++a) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < P; ++b) s = fma((double)v[b], R2[b * P + a], s);
        V[(int64_t)a * d + j] = (float)s;
    }
}

// The products of a starting basis with itself (its Y is itself), as one part
// per 256 rows.
__global__ __launch_bounds__(256) void start_products_kernel(const float *V, int32_t d,
                                                             double *part) {
    constexpr int P = kPcaBlock;
    const int64_t j0 = (int64_t)blockIdx.x * 256;
    const int tid = threadIdx.x;
    if (tid >= kProducts) return;
    const int a = tid / P % P, b = tid % P;
    double s = 0.0;
    const int64_t j1 = j0 + 256 < d ? j0 + 256 : d;
#pragma unroll 8
    for (int64_t j = j0; j < j1; ++j)
        s += (double)V[(int64_t)a * d + j] * (double)V[(int64_t)b * d + j];
    part[(int64_t)blockIdx.x * kProducts + tid] = s;
}

// Starting basis: SplitMix64 values in [-1/2, 1/2).
__global__ void start_basis_kernel(float *V, int64_t count, uint64_t seed) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    uint64_t z = seed + (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    V[i] = (float)((double)(z >> 40) * (1.0 / 16777216.0) - 0.5);
}

// Sum over the workgroup's threads, in a fixed order, to every thread.
__device__ inline double block_sum(double v, double (&red)[kOrthThreads / 64]) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = red[0];
    for (int w = 1; w < kOrthThreads / 64; ++w) s += red[w];
    return s;
}

// Smallest key of the workgroup's threads, to every thread.
__device__ inline unsigned long long block_min(unsigned long long k,
                                               unsigned long long (&best)[kOrthThreads / 64]) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long other = __shfl_xor(k, o, 64);
        k = other < k ? other : k;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) best[threadIdx.x >> 6] = k;
    __syncthreads();
    unsigned long long m = best[0];
    for (int w = 1; w < kOrthThreads / 64; ++w) m = best[w] < m ? best[w] : m;
    return m;
}

// One workgroup: the two Ritz vectors as unit vectors at a right angle (any such
// pair has the eigenvalue 0 where the data have no variance).  A direction that
// vanished in the iteration (data of rank 1, a single sample) is zero until here:
// v1 becomes the first axis, v2 the axis on which v1 is smallest less its part
// along v1.  Vectors within 1e-3 of that already stay as they are.  Then the sign
// convention: the component of largest magnitude (lowest index on ties) of each
// is made positive.
__global__ __launch_bounds__(kOrthThreads) void finish_vectors_kernel(float *V, int32_t d) {
    __shared__ unsigned long long best[kOrthThreads / 64];
    __shared__ double red[kOrthThreads / 64];
    const int tid = threadIdx.x;
    float *v1 = V;
    for (int a = 0; a < 2 && a < d; ++a) {
        float *v = V + (int64_t)a * d;
        double sq = 0.0, dot = 0.0;
        for (int64_t j = tid; j < d; j += kOrthThreads) {
            sq = fma((double)v[j], (double)v[j], sq);
            if (a > 0) dot = fma((double)v[j], (double)v1[j], dot);
        }
        sq = block_sum(sq, red);
        dot = block_sum(dot, red);
        if (!(sq == sq) || (fabs(sq - 1.0) <= 1e-3 && fabs(dot) <= 1e-3)) continue;
        const double left = sq - dot * dot;
        if (left > 1e-6) {
            const double inv = 1.0 / sqrt(left);
            for (int64_t j = tid; j < d; j += kOrthThreads)
                v[j] = (float)(((double)v[j] - (a > 0 ? dot * (double)v1[j] : 0.0)) * inv);
        } else {
            unsigned long long k = ~0ull;  // (|v1| bits, index)
            for (int64_t j = tid; j < d; j += kOrthThreads) {
                const unsigned mag = a > 0 ? __float_as_uint(fabsf(v1[j])) : 0u;
                const unsigned long long key = ((unsigned long long)mag << 32) | (unsigned)j;
                k = key < k ? key : k;
            }
            const int64_t axis = (int64_t)(unsigned)block_min(k, best);
            const double on = a > 0 ? (double)v1[axis] : 0.0, inv = 1.0 / sqrt(1.0 - on * on);
            for (int64_t j = tid; j < d; j += kOrthThreads)
                v[j] = (float)(((j == axis ? 1.0 : 0.0) - (a > 0 ? on * (double)v1[j] : 0.0)) * inv);
        }
        __syncthreads();
    }
    for (int a = 0; a < 2; ++a) {
        float *v = V + (int64_t)a * d;
        unsigned long long k = ~0ull;  // (~|v| bits, index): the minimum is the largest |v|
        for (int64_t j = tid; j < d; j += kOrthThreads) {
            const unsigned mag = __float_as_uint(fabsf(v[j]));
            const unsigned long long key = ((unsigned long long)(~mag) << 32) | (unsigned)j;
            k = key < k ? key : k;
        }
        const int64_t j = (int64_t)(unsigned)block_min(k, best);
        const bool flip = v[j] < 0.f;
        __syncthreads();
        if (flip)
            for (int64_t i = tid; i < d; i += kOrthThreads) v[i] = -v[i];
        __syncthreads();
    }
}

__global__ void linear_init_kernel(float *W, int64_t ld, int32_t rows, int32_t cols, int32_t d,
                                   const float *mean, const float *v1, const float *v2, float s1,
                                   float s2) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)rows * cols * ld;
    if (e >= total) return;
    const int64_t u = e / ld, j = e - u * ld;
    if (j >= d) {
        W[e] = 0.f;
        return;
    }
    const int r = (int)(u / cols), c = (int)(u - (int64_t)r * cols);
    const float a = cols > 1 ? (float)(2.0 * c / (cols - 1) - 1.0) : 0.f;
    const float b = rows > 1 ? (float)(2.0 * r / (rows - 1) - 1.0) : 0.f;
    W[e] = fmaf(b * s2, v2[j], fmaf(a * s1, v1[j], mean[j]));
}

}  // namespace

// Work buffer: C (d x d), two sets of iteration vectors (d x kPcaBlock each),
// then at an even float offset the doubles: the column partials (kMeanChunks x
// d; the step's products afterwards) and two 8 x 8 matrices.
static size_t pca_part_offset(int32_t d) {
    const size_t dd = (size_t)d;
    return (dd * dd + 2 * dd * kPcaBlock + 1) & ~(size_t)1;
}
static size_t pca_part_doubles(int32_t d) {
    const size_t dd = (size_t)d, blocks = (dd + kMatvecRows - 1) / kMatvecRows;
    const size_t products = blocks * kProducts, columns = dd * kMeanChunks;
    return products > columns ? products : columns;
}

size_t pca_work_floats(int32_t d) {
    return pca_part_offset(d) + 2 * (pca_part_doubles(d) + 2 * kPcaBlock * kPcaBlock);
}

hipError_t pca_top2(const float *X, int64_t n, int32_t d, float *work, float *mean, double *stats,
                    int max_iters, double tol, hipStream_t s, double *lambda, int *iters) {
    float *C = work;
    // the step's input (V = in R) and output vectors, swapped after each step
    float *in = C + (size_t)d * d, *out = in + (size_t)d * kPcaBlock;
    float *const vectors = in;
    double *part = reinterpret_cast<double *>(work + pca_part_offset(d));
    double *R = part + pca_part_doubles(d), *Q = R + kPcaBlock * kPcaBlock;
    const unsigned col_blocks = (unsigned)((d + 255) / 256);
    col_partial_kernel<<<dim3(col_blocks, kMeanChunks), dim3(256), 0, s>>>(X, n, d, part);
    col_mean_kernel<<<dim3(col_blocks), dim3(256), 0, s>>>(part, n, d, mean);
    const int nt = (d + kCovTile - 1) / kCovTile;
    const bool vec4 = d % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
    (vec4 ? covariance_kernel<true> : covariance_kernel<false>)
        <<<dim3((unsigned)(nt * (nt + 1) / 2)), dim3(256), 0, s>>>(X, n, d, mean, C);
    const int64_t vcount = (int64_t)d * kPcaBlock;
    start_basis_kernel<<<dim3((unsigned)((vcount + 255) / 256)), dim3(256), 0, s>>>(
        in, vcount, 0x5043412d494e4954ull);
    start_products_kernel<<<dim3(col_blocks), dim3(256), 0, s>>>(in, d, part);
    orthonormal_kernel<<<dim3(1), dim3(kSmallThreads), 0, s>>>(part, (int)col_blocks, R, stats, 0,
                                                              0);
    const unsigned mv_blocks = (unsigned)((d + kMatvecRows - 1) / kMatvecRows);
    double h[4] = {0, 0, 0, 0};
    hipError_t e;
    int it = 0;
    for (;;) {
        matvec_kernel<<<dim3(mv_blocks), dim3(256), 0, s>>>(C, d, in, R, out, part);
        ++it;
        const bool check = (it % 8) == 0 || it >= max_iters;
        orthonormal_kernel<<<dim3(1), dim3(kSmallThreads), 0, s>>>(part, (int)mv_blocks, R, stats,
                                                                  check, 0);
        float *t = in;
        in = out;
        out = t;
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (!check) continue;
        e = hipMemcpyAsync(h, stats, sizeof(h), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        const double scale = h[0] > 0.0 ? h[0] : 1.0;
        if ((h[2] <= tol * scale && h[3] <= tol * scale) || it >= max_iters) break;
    }
    // final Rayleigh-Ritz pair of the next basis in `vectors` (columns 0, 1),
    // unit vectors with their signs fixed
    matvec_kernel<<<dim3(mv_blocks), dim3(256), 0, s>>>(C, d, in, R, out, part);
    orthonormal_kernel<<<dim3(1), dim3(kSmallThreads), 0, s>>>(part, (int)mv_blocks, Q, stats, 1,
                                                              1);
    ritz_vectors_kernel<<<dim3(col_blocks), dim3(256), 0, s>>>(in, R, Q, d, out);
    if (out != vectors) {
        e = hipMemcpyAsync(vectors, out, (size_t)vcount * sizeof(float), hipMemcpyDeviceToDevice,
                           s);
        if (e != hipSuccess) return e;
    }
    finish_vectors_kernel<<<dim3(1), dim3(kOrthThreads), 0, s>>>(vectors, d);
    e = hipMemcpyAsync(h, stats, sizeof(h), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    lambda[0] = h[0] > 0.0 ? h[0] : 0.0;
    lambda[1] = h[1] > 0.0 ? h[1] : 0.0;
    if (iters) *iters = it;
    return hipGetLastError();
}

const float *pca_vectors(const float *work, int32_t d) { return work + (size_t)d * d; }

hipError_t launch_linear_init(float *W, int64_t ld, int32_t rows, int32_t cols, int32_t d,
                              const float *mean, const float *v1, const float *v2, double lambda1,
                              double lambda2, hipStream_t s) {
    const int64_t total = (int64_t)rows * cols * ld;
    linear_init_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>(
        W, ld, rows, cols, d, mean, v1, v2, (float)sqrt(lambda1), (float)sqrt(lambda2));
    return hipGetLastError();
}

}  // namespace som
