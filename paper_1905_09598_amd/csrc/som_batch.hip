// Batch-map training: Kohonen's batch rule, the SOM variant that Sec. 4
// attributes to earlier GPU SOMs ([25], [26]), beside the paper's online
// rule.  One epoch assigns every sample to its BMU (the batched MFMA BMU of
// som_eval.hip) and then sets
//     w_u = sum_c h(u, c) S_c / sum_c h(u, c) n_c,
// S_c and n_c being the sum and the number of the samples whose BMU is c,
// h the Gaussian of Eq. (1) without the learning rate.  A unit whose
// denominator is 0 keeps its prototype.
//
// The lattice Gaussian factors over the two lattice axes: with a = 1 (RECT)
// or 3/4 (HEX, the square of its row pitch sqrt(3)/2) and the column offset
// o = (parity(u) - parity(c)) / 2 of HEX's shifted odd rows (0 for RECT),
//     h(u, c) = exp(-a dr^2 / (2 sigma^2)) exp(-(dc + o)^2 / (2 sigma^2)),
// so the N x N product is a blur along the columns (one table per offset)
// followed by a blur along the rows, O(N d (rows + cols)) instead of
// O(N^2 d).  Everything after the BMU is fp64; the count n_c rides along
// as column d of S.
#include "som_internal.h"

#include <math.h>

#include <algorithm>

namespace som {
namespace {

constexpr int kUnitsPerWG = 64;   // units of a list and of a batch_sums workgroup
constexpr int kColsPerWG = 128;   // ... and its columns
constexpr int kListThreads = 1024;

// Lists of the samples of each group of 64 units, in increasing sample index:
// list[first[grp]] .. = (sample, unit of the group), first[grp + 1] the end.
// One workgroup per group, two passes over the BMUs (how many belong to earlier
// groups, then its own, compacted by ballots).  Without the lists every
// workgroup of the sums walked all BMUs, 256 at a time with three barriers
// each: 1.39 ms at 30,000 samples x 2048 on 10,000 units, now 0.03 for the lists
// and 0.46 for the sums.
__global__ __launch_bounds__(kListThreads) void batch_lists_kernel(const int32_t *bmu, int64_t n,
                                                                   int32_t groups, int2 *list,
                                                                   int64_t *first) {
    __shared__ int wave_count[kListThreads / 64];
    __shared__ unsigned long long before;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, grp = blockIdx.x;
    const int u0 = grp * kUnitsPerWG;
    if (t == 0) before = 0;
    __syncthreads();
    unsigned long long less = 0;
#pragma unroll 4
    for (int64_t i = t; i < n; i += kListThreads) less += bmu[i] < u0 ? 1 : 0;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) less += __shfl_xor(less, o, 64);
    if (lane == 0) atomicAdd(&before, less);
    __syncthreads();
    int64_t at = (int64_t)before;
    if (t == 0) {
        first[grp] = at;
        if (grp == groups - 1) first[groups] = n;
    }
    for (int64_t i0 = 0; i0 < n; i0 += kListThreads) {
        const int64_t i = i0 + t;
        const int c = i < n ? bmu[i] - u0 : -1;
        const bool mine = c >= 0 && c < kUnitsPerWG;
        const unsigned long long m = __ballot(mine);
        if (lane == 0) wave_count[wave] = __builtin_popcountll(m);
        __syncthreads();
        int base = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kListThreads / 64; ++w) {
            const int k = wave_count[w];
            base += w < wave ? k : 0;
            total += k;
        }
        if (mine)
            list[at + base + __builtin_popcountll(m & ((1ull << lane) - 1ull))] =
                make_int2((int)i, c);
        at += total;
        __syncthreads();
    }
}

// S[u][j] (u < N, j <= d, row pitch dp) = sum of X[i][j] over the samples
// i with BMU u, in increasing i; S[u][d] = their number.  Workgroup (x, y)
// owns units 64 x .. and columns 128 y ..: it walks its group's list and adds
// the rows into fp64 accumulators in LDS (one column per thread), eight rows
// in flight.
__global__ __launch_bounds__(kColsPerWG) void batch_sums_kernel(const int2 *list,
                                                                const int64_t *first,
                                                                const float *X, int32_t d,
                                                                int32_t N, double *S,
                                                                int64_t dp) {
    __shared__ double acc[kUnitsPerWG][kColsPerWG];
    const int t = threadIdx.x;
    const int u0 = blockIdx.x * kUnitsPerWG;
    const int64_t j = (int64_t)blockIdx.y * kColsPerWG + t;
    const int64_t jj = j < d ? j : d - 1;
    for (int r = 0; r < kUnitsPerWG; ++r) acc[r][t] = 0.0;
    const int64_t k0 = first[blockIdx.x], k1 = first[blockIdx.x + 1];
    for (int64_t k = k0; k < k1; k += 8) {  // in increasing sample index
        int2 e[8];
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) e[q] = list[k + q < k1 ? k + q : k];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = X[(int64_t)e[q].x * d + jj];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (k + q < k1) acc[e[q].y][t] += j < d ? (double)v[q] : (j == d ? 1.0 : 0.0);
    }
    if (j < dp)
        for (int r = 0; r < kUnitsPerWG && u0 + r < N; ++r) S[(int64_t)(u0 + r) * dp + j] = acc[r][t];
}

// Factor tables of the lattice Gaussian at radius sigma:
//   Hr[ru][rc]     = exp(-a (ru - rc)^2 / (2 sigma^2)),
//   Hc[o][cu][cc]  = exp(-(cu - cc + off_o)^2 / (2 sigma^2)), off = 0, +1/2, -1/2
// (a = 1 and one offset for RECT; a = 3/4 and three for HEX); sigma = 0
// gives the Kronecker delta, sigma = inf all ones.
__global__ void batch_tables_kernel(int32_t rows, int32_t cols, int32_t topology, double sigma,
                                    double *Hr, double *Hc) {
    const int64_t nr = (int64_t)rows * rows, nc = (int64_t)cols * cols;
    const int planes = topology == 1 ? 3 : 1;
    const double a = topology == 1 ? 0.75 : 1.0;
    const double off[3] = {0.0, 0.5, -0.5};
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nr + planes * nc;
         e += (int64_t)gridDim.x * blockDim.x) {
        double g;
        if (e < nr) {
            const double dr = (double)(e / rows) - (double)(e % rows);
            g = a * dr * dr;
        } else {
            const int64_t k = e - nr, o = k / nc, q = k % nc;
            const double dx = (double)(q / cols) - (double)(q % cols) + off[o];
            g = dx * dx;
        }
        double h;
        if (sigma == 0.0)
            h = g == 0.0 ? 1.0 : 0.0;
        else if (isinf(sigma))
            h = 1.0;
        else
            h = exp(-g / (2.0 * sigma * sigma));
        if (e < nr)
            Hr[e] = h;
        else
            Hc[e - nr] = h;
    }
}

// Column blur: T[o][r][cu][j] = sum_cc Hc[o][cu][cc] S[r][cc][j].  Workgroup
// (x, y, z): lattice row r = x / ceil(cols/64) with output columns
// 64 (x % ceil(cols/64)) .., columns 256 y .. of j, offset plane z.  Thread
// t: j = t % 64 + 64 q (q < 4), outputs cu = cu0 + t / 64 + 4 k (k < 16).  S and
// Hc are staged through LDS 16 lattice columns at a time.  Four columns a
// thread use each factor read from LDS four times: with one column the LDS
// bound both passes (1.33 and 0.89 ms on 100 x 100 units of 2048, now 0.37 and
// 0.35).
constexpr int kBlurCols = 256, kBlurStage = 16;
__global__ __launch_bounds__(256) void batch_col_pass_kernel(const double *S, const double *Hc,
                                                             double *T, int32_t rows,
                                                             int32_t cols, int64_t dp) {
    __shared__ double ls[kBlurStage][kBlurCols];
    __shared__ double lh[64][kBlurStage + 1];
    const int t = threadIdx.x, jl = t & 63, g = t >> 6;
    const int cblocks = (cols + 63) / 64;
    const int r = blockIdx.x / cblocks, cu0 = (blockIdx.x % cblocks) * 64;
    const int64_t j0 = (int64_t)blockIdx.y * kBlurCols;
    const int o = blockIdx.z;
    const double *hc = Hc + (int64_t)o * cols * cols;
    double acc[16][4];
#pragma unroll
    for (int k = 0; k < 16; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[k][q] = 0.0;
    for (int cc0 = 0; cc0 < cols; cc0 += kBlurStage) {
#pragma unroll
        for (int e = 0; e < kBlurStage; ++e) {
            const int cc = cc0 + e;
            const int64_t jj = j0 + t;
            ls[e][t] = (cc < cols && jj < dp) ? S[((int64_t)r * cols + cc) * dp + jj] : 0.0;
        }
        for (int e = t; e < 64 * kBlurStage; e += 256) {
            const int cu = cu0 + e / kBlurStage, cc = cc0 + e % kBlurStage;
            lh[e / kBlurStage][e % kBlurStage] =
                (cu < cols && cc < cols) ? hc[(int64_t)cu * cols + cc] : 0.0;
        }
        __syncthreads();
        for (int c = 0; c < kBlurStage; ++c) {
            double s[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] = ls[c][jl + 64 * q];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const double h = lh[g + 4 * k][c];
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[k][q] = fma(h, s[q], acc[k][q]);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t j = j0 + jl + 64 * q;
        if (j >= dp) continue;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int cu = cu0 + g + 4 * k;
            if (cu < cols) T[(((int64_t)o * rows + r) * cols + cu) * dp + j] = acc[k][q];
        }
    }
}

// Row blur: O[ru][cu][j] = sum_rc Hr[ru][rc] T[o(ru, rc)][rc][cu][j], where
// the HEX offset plane o follows the rows' parities (0 equal, 1 for an odd
// ru over an even rc, 2 the other way).  Workgroup (x, y): lattice column
// cu = x / ceil(rows/64) with output rows 64 (x % ceil(rows/64)) .., columns
// 256 y .. of j.  Thread t: j = t % 64 + 64 q, outputs ru = ru0 + t / 64 + 4 k;
// the parity of ru is the same for all of a thread's k, so with three planes
// each row of T is staged twice, for even and for odd ru (PLANES 2).
template <int PLANES>
__global__ __launch_bounds__(256) void batch_row_pass_kernel(const double *T, const double *Hr,
                                                             double *O, int32_t rows,
                                                             int32_t cols, int64_t dp) {
    __shared__ double lt[PLANES][kBlurStage][kBlurCols];
    __shared__ double lh[64][kBlurStage + 1];
    const int t = threadIdx.x, jl = t & 63, g = t >> 6;
    const int rblocks = (rows + 63) / 64;
    const int cu = blockIdx.x / rblocks, ru0 = (blockIdx.x % rblocks) * 64;
    const int64_t j0 = (int64_t)blockIdx.y * kBlurCols;
    const int mine = PLANES == 1 ? 0 : (ru0 + g) & 1;
    double acc[16][4];
#pragma unroll
    for (int k = 0; k < 16; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[k][q] = 0.0;
    for (int rc0 = 0; rc0 < rows; rc0 += kBlurStage) {
#pragma unroll
        for (int e = 0; e < PLANES * kBlurStage; ++e) {
            const int pu = e / kBlurStage, rc = rc0 + e % kBlurStage, pc = rc & 1;
            const int o = PLANES == 1 ? 0 : (pu == pc ? 0 : (pu ? 1 : 2));
            const int64_t jj = j0 + t;
            lt[pu][e % kBlurStage][t] =
                (rc < rows && jj < dp) ? T[(((int64_t)o * rows + rc) * cols + cu) * dp + jj] : 0.0;
        }
        for (int e = t; e < 64 * kBlurStage; e += 256) {
            const int ru = ru0 + e / kBlurStage, rc = rc0 + e % kBlurStage;
            lh[e / kBlurStage][e % kBlurStage] =
                (ru < rows && rc < rows) ? Hr[(int64_t)ru * rows + rc] : 0.0;
        }
        __syncthreads();
        for (int c = 0; c < kBlurStage; ++c) {
            double v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = lt[mine][c][jl + 64 * q];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const double h = lh[g + 4 * k][c];
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[k][q] = fma(h, v[q], acc[k][q]);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t j = j0 + jl + 64 * q;
        if (j >= dp) continue;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int ru = ru0 + g + 4 * k;
            if (ru < rows) O[((int64_t)ru * cols + cu) * dp + j] = acc[k][q];
        }
    }
}

// W[u][j] = fp32(O[u][j] / O[u][d]) where the denominator is positive.
__global__ void batch_finish_kernel(const double *O, float *W, int64_t ld, int32_t N, int32_t d,
                                    int64_t dp) {
    const int64_t total = (int64_t)N * d;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t u = e / d, j = e - u * d;
        const double den = O[u * dp + d];
        if (den > 0.0) W[u * ld + j] = (float)(O[u * dp + j] / den);
    }
}

}  // namespace

// Doubles of the blurs' arrays; the sample lists lie in the arrays that the
// blurs write after them where they fit, and behind everything otherwise.
static int64_t batch_array_doubles(int64_t rows, int64_t cols, int64_t d, int planes) {
    return rows * cols * (d + 1) * (2 + planes) + rows * rows + planes * cols * cols;
}

size_t batch_work_doubles(int32_t rows, int32_t cols, int32_t d, int32_t topology, int64_t n) {
    const int64_t N = (int64_t)rows * cols, groups = (N + kUnitsPerWG - 1) / kUnitsPerWG;
    const int planes = topology == 1 ? 3 : 1;
    const int64_t lists = n + groups + 1;  // (an int2 or an int64 each)
    const int64_t spare = N * ((int64_t)d + 1) * planes;
    return (size_t)(batch_array_doubles(rows, cols, d, planes) + (lists <= spare ? 0 : lists));
}

hipError_t launch_batch_epoch(const BatchArgs &b, hipStream_t s) {
    const int64_t N = (int64_t)b.rows * b.cols, dp = (int64_t)b.d + 1;
    const int planes = b.topology == 1 ? 3 : 1;
    const int64_t groups = (N + kUnitsPerWG - 1) / kUnitsPerWG;
    const int64_t sum_cols = (dp + kColsPerWG - 1) / kColsPerWG;
    if (b.rows < 1 || b.cols < 1 || (dp + 63) / 64 > 65535) return hipErrorInvalidValue;
    double *S = b.work, *T = S + N * dp, *O = T + planes * N * dp;
    double *Hr = O + N * dp, *Hc = Hr + (int64_t)b.rows * b.rows;
    double *at = b.n + groups + 1 <= planes * N * dp
                     ? T
                     : b.work + batch_array_doubles(b.rows, b.cols, b.d, planes);
    int64_t *first = reinterpret_cast<int64_t *>(at);
    int2 *list = reinterpret_cast<int2 *>(at + groups + 1);
    batch_lists_kernel<<<dim3((unsigned)groups), dim3(kListThreads), 0, s>>>(
        b.bmu, b.n, (int32_t)groups, list, first);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    batch_sums_kernel<<<dim3((unsigned)groups, (unsigned)sum_cols), dim3(kColsPerWG), 0, s>>>(
        list, first, b.X, b.d, (int32_t)N, S, dp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int64_t tab = (int64_t)b.rows * b.rows + (int64_t)planes * b.cols * b.cols;
    batch_tables_kernel<<<dim3((unsigned)std::min<int64_t>((tab + 255) / 256, 4096)), dim3(256), 0,
                          s>>>(b.rows, b.cols, b.topology, b.sigma, Hr, Hc);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const unsigned blur = (unsigned)((dp + kBlurCols - 1) / kBlurCols);
    batch_col_pass_kernel<<<dim3((unsigned)(b.rows * ((b.cols + 63) / 64)), blur,
                              (unsigned)planes),
                         dim3(256), 0, s>>>(S, Hc, T, b.rows, b.cols, dp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    (planes == 1 ? batch_row_pass_kernel<1> : batch_row_pass_kernel<2>)
        <<<dim3((unsigned)(b.cols * ((b.rows + 63) / 64)), blur), dim3(256), 0, s>>>(
            T, Hr, O, b.rows, b.cols, dp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    batch_finish_kernel<<<dim3((unsigned)std::min<int64_t>((N * b.d + 255) / 256, 65536)), dim3(256),
                          0, s>>>(O, b.W, b.ld, (int32_t)N, b.d, dp);
    return hipGetLastError();
}

}  // namespace som
