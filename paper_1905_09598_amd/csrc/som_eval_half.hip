// The batched BMU's products X W^T for large calls, on the fp16 matrix
// instructions (v_mfma_f32_16x16x32_f16, fp32 accumulation) at fp32 precision:
// every operand is split into two halves, x 2^k = hi + lo + e with |e| <=
// max(2^-23 |x 2^k|, 2^-25) (hi the nearest fp16, lo the fp16 nearest to the
// rest, k a power of two per row that puts its largest magnitude just below
// 2^15), and a product is hi hi' + hi lo' + lo hi'.  What is left out, lo lo' and
// e, is at most 2^-21.4 of a term at random signs, below the rounding of an fp32
// sum of 32 terms and more (kMinCols).  Three instructions of 16 cycles replace
// eight of 32.
//
// Measured at 100,000 samples x 10,000 units x 2048: the whole evaluation 12.3
// ms, 332 TFLOP/s of fp32 products, against 40.2 ms and 102 TFLOP/s on the fp32
// instructions (som_eval.hip).  Root mean square error of a score over |x| |w|
// against fp64, the fp32 kernel with fp32 norms before and here (norms summed
// in fp64): Gaussian mixtures of d = 64, 500, 2048, 10000 7.1e-8, 1.55e-7,
// 3.0e-7, 6.6e-7 and 5.7e-8, 1.0e-7, 1.9e-7, 4.3e-7; TF-IDF rows 4.2e-8, 3.8e-8,
// 3.6e-8, 5.2e-8 and 3.5e-8, 2.8e-8, 3.0e-8, 2.7e-8.
#include "som_candidates.h"

#include <math.h>

#include <algorithm>

namespace som {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

// A workgroup's tile: 256 samples x 128 units on 8 waves (4 x 2) of 64 x 64,
// d in slabs of 32.  Operands are stored in the order the instructions read
// them: per 16 rows and 32 columns one block of 1 KB (hi) and one (lo), 16 bytes
// (8 columns) per lane, lane 16 g + i holding columns 8 g .. of row i; so a slab
// goes from memory straight into LDS (1 KB per wave and load) and is read
// back without bank conflicts.  64 x 64 per wave keeps the LDS at 64 KB per
// 768 matrix cycles of the four SIMDs, half of what it can deliver.
constexpr int kHM = 256, kHN = 128, kHK = 32;
constexpr int kHThreads = 512;
constexpr int kBlockHalves = 2 * 16 * kHK;                 // hi and lo of 16 rows
constexpr int kSlabHalves = (kHM + kHN) / 16 * kBlockHalves;
constexpr float kRowLo = 0x1p-40f, kRowHi = 0x1p40f;       // row maxima that are split

// 16 rows per workgroup: each row's scale, then its halves.  A row that holds
// a NaN or an infinity or a magnitude above 2^40, and a sample (not small_ok)
// whose largest one is below 2^-40, is stored as zeros with scale -1 and raises
// *bad: its products are formed in fp32 (bmu_unsplit_kernel).  A prototype that
// small keeps the scale of 2^-40: its halves are then exact to 2^-79, far below a
// rounding of the distance to a sample that is not as small.
// scale[row] = 2^-k; rows past `rows` are zero.  Bound by memory: the rows are
// read twice, the second time from L2, and written once.  The first `ablocks`
// workgroups take a's rows, the others b's: the prototypes and the first samples
// in one launch.
template <bool VEC4>
__global__ __launch_bounds__(256) void split_rows_kernel(SplitRows a, SplitRows b, int ablocks,
                                                         int32_t d, int32_t slabs) {
    __shared__ float mul[16];
    const int t = threadIdx.x, r = t >> 4, c0 = t & 15;
    const bool first = (int)blockIdx.x < ablocks;
    const int64_t block = first ? blockIdx.x : blockIdx.x - ablocks;
    const float *X = first ? a.X : b.X;
    const int64_t rows = first ? a.rows : b.rows, ld = first ? a.ld : b.ld;
    float *scale = first ? a.scale : b.scale;
    int32_t *bad = first ? a.bad : b.bad;
    const bool small_ok = first ? a.small_ok : b.small_ok;
    const int64_t row0 = block * 16;
    const auto load4 = [&](const float *x, int c) {
        f4 v;
        if (VEC4) {
            v = *reinterpret_cast<const f4 *>(x + (c < d ? c : d - 4));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = x[c + e < d ? c + e : d - 1];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = c + e < d ? v[e] : 0.f;
        return v;
    };
    {
        const int64_t row = row0 + r < rows ? row0 + r : rows - 1;
        const float *x = X + row * ld;
        unsigned top = 0;  // bits of the largest magnitude (a NaN's are the largest)
#pragma unroll 4
        for (int c = 4 * c0; c < d; c += 64) {
            const f4 v = load4(x, c);
#pragma unroll
            for (int e = 0; e < 4; ++e) top = max(top, __float_as_uint(v[e]) & 0x7fffffffu);
        }
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) top = max(top, (unsigned)__shfl_xor((int)top, o, 64));
        if (c0 == 0) {
            const float big = __uint_as_float(top);
            const bool fine = big <= kRowHi && (big >= kRowLo || top == 0 || small_ok);
            // 2^14 <= big 2^k < 2^15
            const int k = top == 0 ? 0 : 14 - (max((int)(top >> 23), 127 - 40) - 127);
            mul[r] = fine ? ldexpf(1.f, k) : 0.f;
            if (row0 + r < rows) {
                scale[row0 + r] = fine ? ldexpf(1.f, -k) : -1.f;
                if (!fine) atomicOr(bad, 1);
            }
        }
    }
    __syncthreads();
    const int lane = t & 63, wave = t >> 6, i = lane & 15, g = lane >> 4;
    const int64_t row = row0 + i < rows ? row0 + i : rows - 1;
    const float m = row0 + i < rows ? mul[i] : 0.f;
    const float *x = X + row * ld;
    _Float16 *out = static_cast<_Float16 *>(first ? a.out : b.out);
    h8 *to = reinterpret_cast<h8 *>(out + block * slabs * kBlockHalves);
    for (int s = wave; s < slabs; s += 4) {
        const int c = s * kHK + 8 * g;
        const f4 a = load4(x, c), b = load4(x, c + 4);
        h8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = m == 0.f ? 0.f : (e < 4 ? a[e & 3] : b[e & 3]) * m;
            hi[e] = (_Float16)v;
            lo[e] = (_Float16)(v - (float)hi[e]);
        }
        to[(int64_t)s * 128 + lane] = hi;
        to[(int64_t)s * 128 + 64 + lane] = lo;
    }
}

typedef const __attribute__((address_space(1))) void *GlobalPtr;
typedef __attribute__((address_space(3))) void *LdsPtr;

// acc[a][b] = products over slabs [s0, s1) of units 16 a + 4 g .. (of the
// wave's 64) with sample 16 b + i (of its 64), in the rows' scaled units.
// Slab s + 1 is loaded into the other LDS buffer while slab s is multiplied;
// one barrier a slab.
__device__ inline void half_products(const EvalArgs &a, int64_t stile, int64_t utile, int s0,
                                     int s1, _Float16 *lds, f4 (&acc)[4][4]) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wsamp = wave & 3, wunit = wave >> 2;
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[x][y] = f4{0.f, 0.f, 0.f, 0.f};
    // 48 KB a slab: the first 16 blocks the samples', then 8 of the units'; each
    // wave brings 3 blocks (2 samples', 1 units')
    const _Float16 *xs = a.xhalf + (stile * (kHM / 16) + 2 * wave) * a.slabs * kBlockHalves;
    const _Float16 *ws = a.whalf + (utile * (kHN / 16) + wave) * a.slabs * kBlockHalves;
    const auto load = [&](int s, int buf) {
        _Float16 *to = lds + buf * kSlabHalves;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const _Float16 *from = b < 2 ? xs + ((int64_t)b * a.slabs + s) * kBlockHalves
                                         : ws + (int64_t)s * kBlockHalves;
            _Float16 *dst = to + (b < 2 ? 2 * wave + b : kHM / 16 + wave) * kBlockHalves;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                __builtin_amdgcn_global_load_lds((GlobalPtr)(from + h * 512 + lane * 8),
                                                 (LdsPtr)(dst + h * 512), 16, 0, 0);
        }
    };
    load(s0, 0);
    for (int s = s0; s < s1; ++s) {
        const int buf = (s - s0) & 1;
        __builtin_amdgcn_s_waitcnt(0x0F70);  // this wave's loads of slab s are in LDS
        __syncthreads();                     // and everyone's; slab s - 1 is no longer read
        if (s + 1 < s1) load(s + 1, buf ^ 1);
        const h8 *from = reinterpret_cast<const h8 *>(lds + buf * kSlabHalves);
        h8 uh[4], ul[4], xh[4], xl[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int ub = kHM / 16 + wunit * 4 + t, xb = wsamp * 4 + t;
            uh[t] = from[ub * 128 + lane];
            ul[t] = from[ub * 128 + 64 + lane];
            xh[t] = from[xb * 128 + lane];
            xl[t] = from[xb * 128 + 64 + lane];
        }
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                        p == 1 ? ul[x] : uh[x], p == 2 ? xl[y] : xh[y], acc[x][y], 0, 0, 0);
    }
    __syncthreads();  // the buffers are free again
}

// Whether a workgroup's products are all formed in fp32 instead: a prototype
// has no halves, or none of the tile's samples has.
__device__ inline bool all_unsplit(const EvalArgs &a, int64_t s0) {
    if (a.bad[0] != 0) return true;
    if (a.bad[1] == 0) return false;
    const int64_t smp = s0 + threadIdx.x;
    return !__syncthreads_or((int)threadIdx.x < kHM && smp < a.n && a.xscale[smp] >= 0.f);
}

// Fused form: sample tile blockIdx.x, unit group blockIdx.y walked tile by
// tile; per sample the kCand best (score, unit) pairs of the group.
__global__ __launch_bounds__(kHThreads, 2) void half_candidates_kernel(EvalArgs a) {
    extern __shared__ __align__(16) _Float16 lds[];
    if (all_unsplit(a, (int64_t)blockIdx.x * kHM)) return;
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wsamp = wave & 3, wunit = wave >> 2;
    const int64_t s0 = (int64_t)blockIdx.x * kHM;
    const int grp = blockIdx.y, u_begin = grp * a.group_units;
    const int u_end = u_begin + a.group_units < a.N ? u_begin + a.group_units : a.N;
    float ts[4][kCand], sx2[4];
    int tu[4][kCand];
#pragma unroll
    for (int y = 0; y < 4; ++y) {
        const int64_t smp = s0 + wsamp * 64 + 16 * y + i;
        sx2[y] = 2.f * a.xscale[smp < a.n ? smp : a.n - 1];
#pragma unroll
        for (int c = 0; c < kCand; ++c) { ts[y][c] = INFINITY; tu[y][c] = -1; }
    }
    for (int u0 = u_begin; u0 < u_end; u0 += kHN) {
        f4 acc[4][4];
        half_products(a, blockIdx.x, u0 / kHN, 0, a.slabs, lds, acc);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int u = u0 + wunit * 64 + 16 * x + 4 * g + v;
                if (u >= u_end) continue;
                const float wn = a.wnorm[u], sw = a.wscale[u];
#pragma unroll
                for (int y = 0; y < 4; ++y)
                    insert_top(ts[y], tu[y], fmaf(-sx2[y] * sw, acc[x][y][v], wn), u);
            }
    }
    // merge the 8 partial lists of each sample (2 unit waves x 4 lane groups)
    int2 *ls = reinterpret_cast<int2 *>(lds);  // [kHM][8][kCand]
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
        for (int c = 0; c < kCand; ++c)
            ls[((wsamp * 64 + 16 * y + i) * 8 + wunit * 4 + g) * kCand + c] =
                make_int2(__float_as_int(ts[y][c]), tu[y][c]);
    __syncthreads();
    const int t = threadIdx.x;
    if (t < kHM && s0 + t < a.n) {
        float ms[kCand];
        int mu[kCand];
#pragma unroll
        for (int c = 0; c < kCand; ++c) { ms[c] = INFINITY; mu[c] = -1; }
        for (int e = 0; e < 8 * kCand; ++e) {
            const int2 p = ls[t * 8 * kCand + e];
            if (p.y >= 0) insert_top(ms, mu, __int_as_float(p.x), p.y);
        }
        int2 *out = reinterpret_cast<int2 *>(a.cand) + ((s0 + t) * a.ugroups + grp) * kCand;
#pragma unroll
        for (int c = 0; c < kCand; ++c) out[c] = make_int2(__float_as_int(ms[c]), mu[c]);
    }
}

// Split form: the products of one tile over slabs [z split, (z + 1) split),
// sample-major as the fp32 kernel writes them.
__global__ __launch_bounds__(kHThreads, 2) void half_partial_kernel(EvalArgs a) {
    extern __shared__ __align__(16) _Float16 lds[];
    if (all_unsplit(a, (int64_t)blockIdx.x * kHM)) return;
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wsamp = wave & 3, wunit = wave >> 2;
    const int z = blockIdx.z, s0 = z * (a.split_len / kHK);
    const int s1 = s0 + a.split_len / kHK < a.slabs ? s0 + a.split_len / kHK : a.slabs;
    f4 acc[4][4];
    half_products(a, blockIdx.x, blockIdx.y, s0, s1, lds, acc);
    const int64_t np = (int64_t)a.tiles_u * kHN;
    float sw[4][4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int u = blockIdx.y * kHN + wunit * 64 + 16 * x + 4 * g + v;
            sw[x][v] = a.wscale[u < a.N ? u : a.N - 1];
        }
#pragma unroll
    for (int y = 0; y < 4; ++y) {
        const int64_t smp = (int64_t)blockIdx.x * kHM + wsamp * 64 + 16 * y + i;
        if (smp >= a.n) continue;
        const float sx = a.xscale[smp];
        f4 *row = reinterpret_cast<f4 *>(a.part + ((int64_t)z * a.n + smp) * np +
                                         blockIdx.y * kHN + wunit * 64 + 4 * g);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            f4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[x][y][e] * (sx * sw[x][e]);
            row[4 * x] = v;
        }
    }
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
constexpr size_t kHalfLds = 2 * (size_t)kSlabHalves * sizeof(_Float16);
// Microseconds of one slab of a tile on a workgroup (1.2 on few tiles, where the
// line lies; up to 1.7 with every compute unit busy, where the halves take a third
// of the fp32 products' time), of one workgroup's start and finish, and of the
// two extra launches; the rows are split at about 3 TB/s.  The line against the
// fp32 kernels lies where these add up to less than those kernels' measured
// 4.3 us per slice.  Evaluations on either side, fp32 and halves in
// microseconds: 23,395 samples of 303 on 12 x 32 units 219 and 164, 17,406 of 71
// on 15 x 34 172 and 125, 1,307 of 186 on 52 x 100 120 and 90; at 2,000 of 2,000
// on 20 x 20 units the fp32 kernel (46 us) stays.
constexpr double kSlabUs = 1.2, kTileUs = 3.0, kLaunchUs = 3.0;
constexpr int64_t kChunkBytes = 256 << 20;  // samples split at a time
// A sum of fewer terms has fewer roundings than the halves leave out.  Root mean
// square error of a score over |x| |w| against fp64 (emulated, norms summed in
// fp64 on both sides), fp32 products and halves: Gaussian rows of 2, 4, 8, 16, 24
// and 32 columns 9.2e-8 and 1.5e-7, 7.0e-8 and 1.0e-7, 6.0e-8 and 7.7e-8, 5.7e-8
// and 6.2e-8, 5.4e-8 and 5.3e-8, 5.4e-8 and 5.1e-8; clusters of 16, 24, 32 and 64
// columns 6.3e-8 and 6.8e-8, 7.4e-8 and 6.2e-8, 7.8e-8 and 6.0e-8, 9.3e-8 and
// 5.6e-8.
constexpr int kMinCols = 32;

}  // namespace

int64_t half_rows_halves(int64_t rows, int32_t d, int tile) {
    return ceil_div(rows, tile) * (tile / 16) * ceil_div(d, kHK) * kBlockHalves;
}

int64_t half_lists_bytes(const HalfPlan &plan, int64_t rows, int32_t N) {
    return plan.splits > 1 ? plan.splits * rows * ceil_div(N, kHN) * kHN * (int64_t)sizeof(float)
                           : rows * plan.ugroups * kCand * (int64_t)sizeof(int2);
}

bool plan_bmu_half(EvalArgs *a, int num_cus, uint64_t max_bytes, double fp32_us, HalfPlan *plan) {
    // Few tiles of 256 x 128 leave the chip idle while a workgroup walks a long
    // row, and the times above are those of a busier one; calls of fewer than 2^20
    // sample-unit pairs stay on the fp32 products.  Microseconds of a search with
    // the fp32 products and with halves, below that line: 9 samples of 12000 floats
    // on 25 units 52 and 160, 1500 of 2000 on 400 58 and 69, 100 of 2048 on 10,000
    // 131 and 151, 2600 of 2000 on 400 79 and 77, 400 of 10000 on 2500 292 and 241;
    // above it, halves by the times above: 2700 of 2000 on 400 101 and 77, 200 and
    // 255 of 2048 on 10,000 184 and 155, 187 and 157, 420 of 10000 on 2500 294 and
    // 243, 2700 of 12000 on 400 366 and 326, 1307 of 186 on 5200 70 and 59; fp32 by
    // them: 45,000 of 12000 on 25 1326 and 2833, 20,000 of 2000 on 100 156 and 205,
    // 100 of 512 on 65,536 140 and 172.
    const bool asked = isinf(fp32_us);
    if (!asked && (a->d < kMinCols || a->n * (int64_t)a->N < (int64_t)1 << 20)) return false;
    const int64_t slabs = ceil_div(a->d, kHK), tiles_u = ceil_div(a->N, kHN);
    const int64_t row_bytes = slabs * kHK * 4;
    // one buffer holds the halves, the scales (4 bytes a row) and the lists, at
    // least those of one unit group
    const uint64_t w_bytes = (uint64_t)half_rows_halves(a->N, a->d, kHN) * 2 + 4 * (uint64_t)a->N +
                             2048;
    if (w_bytes > max_bytes) return false;
    const uint64_t left = std::min<uint64_t>(max_bytes - w_bytes, INT64_MAX);
    int64_t chunk = std::min<int64_t>(kChunkBytes / row_bytes, (int64_t)left / (row_bytes + 4 + kCand * 8)) /
                    kHM * kHM;
    if (chunk < kHM) return false;
    // equal chunks: a short last one would leave most of the chip idle
    const int64_t chunks = ceil_div(a->n, chunk);
    chunk = ceil_div(ceil_div(a->n, chunks), kHM) * kHM;
    const int64_t tiles_s = chunk / kHM;
    const uint64_t lists_max = left - (uint64_t)chunk * (row_bytes + 4);
    double best = 1e300;
    for (int64_t tpg = tiles_u; tpg >= 1; --tpg) {
        const int64_t g = ceil_div(tiles_u, tpg);
        if ((uint64_t)chunk * g * kCand * 8 > lists_max) break;
        const double us = ceil_div(tiles_s * g, num_cus) * (tpg * (slabs * kSlabUs + 1.0) + kTileUs) +
                          (double)chunk * g * kCand * 1e-5;
        if (us < best) {
            best = us;
            plan->splits = 1;
            plan->split_len = (int32_t)(slabs * kHK);
            plan->ugroups = (int32_t)g;
            plan->group_units = (int32_t)(tpg * kHN);
        }
    }
    for (int64_t S = 2; S <= 16 && S <= slabs; ++S) {
        const int64_t len = ceil_div(slabs, S), Se = ceil_div(slabs, len);
        const uint64_t part = (uint64_t)Se * chunk * tiles_u * kHN * 4;
        if (Se != S || part > lists_max) continue;
        const double us = ceil_div(tiles_s * tiles_u * Se, num_cus) * (len * kSlabUs + kTileUs) +
                          2.0 * (double)part / 5e6;
        if (us < best) {
            best = us;
            plan->splits = (int32_t)Se;
            plan->split_len = (int32_t)(len * kHK);
            plan->ugroups = 0;
            plan->group_units = 0;
        }
    }
    if (best >= 1e300) return false;
    plan->chunk = chunk;
    plan->slabs = (int32_t)slabs;
    const double rows_us = ((double)a->n + a->N) * row_bytes * 2 / 3e6;
    return (double)chunks * (best + kLaunchUs) + rows_us + kLaunchUs < fp32_us;
}

hipError_t launch_split_rows(const SplitRows *first, const SplitRows &second, int32_t d,
                             hipStream_t s) {
    const auto blocks = [](const SplitRows &r) { return ceil_div(r.rows, r.tile) * (r.tile / 16); };
    const auto vec4 = [d](const SplitRows &r) {
        return d % 4 == 0 && r.ld % 4 == 0 && reinterpret_cast<uintptr_t>(r.X) % 16 == 0;
    };
    if (first && vec4(*first) != vec4(second)) {
        const hipError_t e = launch_split_rows(nullptr, *first, d, s);
        if (e != hipSuccess) return e;
        first = nullptr;
    }
    const int ablocks = first ? (int)blocks(*first) : 0;
    (vec4(second) ? split_rows_kernel<true> : split_rows_kernel<false>)
        <<<dim3((unsigned)(ablocks + blocks(second))), dim3(256), 0, s>>>(
            first ? *first : second, second, ablocks, d, (int32_t)ceil_div(d, kHK));
    return hipGetLastError();
}

hipError_t launch_bmu_half(const EvalArgs &a, hipStream_t s) {
    if (a.tiles_s != ceil_div(a.n, kHM) || a.tiles_u != ceil_div(a.N, kHN) || !a.xhalf ||
        !a.whalf || !a.bad || a.slabs != ceil_div(a.d, kHK))
        return hipErrorInvalidValue;
    if (a.splits <= 1) {
        if (a.ugroups < 1 || a.group_units % kHN != 0 ||
            (int64_t)a.ugroups * a.group_units < a.N || !a.cand)
            return hipErrorInvalidValue;
        half_candidates_kernel<<<dim3((unsigned)a.tiles_s, (unsigned)a.ugroups), dim3(kHThreads),
                                 kHalfLds, s>>>(a);
    } else {
        if (!a.part || a.split_len % kHK != 0 || (int64_t)a.splits * a.split_len < a.d ||
            (int64_t)(a.splits - 1) * a.split_len >= a.d)
            return hipErrorInvalidValue;
        half_partial_kernel<<<dim3((unsigned)a.tiles_s, (unsigned)a.tiles_u, (unsigned)a.splits),
                              dim3(kHThreads), kHalfLds, s>>>(a);
    }
    return hipGetLastError();
}

}  // namespace som
