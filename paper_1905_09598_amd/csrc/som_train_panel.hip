// Panel training: the online steps of Eq. (1) in panels of M steps, with the
// pass over the prototypes as two matrix products per panel and the steps
// themselves in the space of inner products.
//
// Within panel b (steps s0 .. s0 + M - 1, samples x_k, z one of them) every
// prototype is w = z + v, and a step with factor h moves v to
// (1 - h) v + h e_k, e_k = x_k - z.  With L_l = v . e_l and Q = |v|^2
//     D_k = |x_k - w|^2 = G_kk - 2 L_k + Q,        G_kl = e_k . e_l,
//     L_l <- (1 - h) L_l + h G_kl,
//     Q   <- (1 - h) Q + h (G_kk - (1 - h) D_k),
// so a step costs a unit O(M) operations whatever d is, and the prototypes
// are read and written once a panel.  Three roles work at a time:
//   * control: panel b's steps.  Up to 1024 units run on ONE workgroup, so a
//     step's arg-min never leaves the compute unit: its waves meet through
//     LDS.  Larger maps take one wave per workgroup and the grid exchange of
//     som_device.h;
//   * sweep: F_b <- beta F_(b-1) + sum_j gamma_j x_j (panel b - 1's updates, a
//     product over its steps), then V E^T and |V|^2 of F_b with panel b + 1's
//     samples (a product over d), both on fp32 matrix instructions in one pass
//     over the prototypes, held from then on as F_b;
//   * prepare: panel b + 2's samples gathered, centred and transposed, their
//     Gram matrix and their products with panel b + 1's samples; and the
//     distances that panel b + 4's centre is chosen by.
// The sweep sees F_b where panel b + 1 starts from F_(b+1), so its products
// are corrected once panel b's coefficients are known (correct): with a_j =
// x_j - z' the panel's samples in the next panel's centring,
//     (F_(b+1) - z') . e'_l = beta (F_b - z') . e'_l + sum_j gamma_j a_j . e'_l.
// Q is carried from panel to panel through the column of the next centre (in
// the place of the panel's own centre, whose column would be zero),
// Q' = Q - 2 v . (z' - z) + |z' - z|^2, and pulled to the sweep's |F_b - z'|^2
// with weight beta^2, so its rounding does not add up over panels.
//
// Distances are differences of terms at the scale of |x_k - z|^2 and |w - z|^2,
// so the centre has to lie among the samples: a panel's is, of eight of its
// samples, the one with the smallest median distance to the others (an outlier
// of 10,000 times the others' norm as the centre costs every distance of two
// panels its digits).  That keeps every term at the scale of sample-to-sample
// distances, as in the pipelined kernels; the blocked kernel's distances are
// direct differences, and its calls stay on it (persistent_train_first).
//
// The exchange between workgroups (1.0-1.2 us) bounds a step of the kernels
// that hold W across the grid, and the pass over W bounds the streamed ones;
// here the pass runs once per M steps beside the steps, and maps of up to 1024
// units need no exchange.  Measured, microseconds per step with those kernels
// and here: 10 x 10 units of 500 floats 1.26 and 0.66, 11 x 11 of 4545 1.54 and
// 0.91, 30 x 30 of 5000 2.18 and 1.60, 50 x 50 of 10000 6.35 and 3.25, 100 x 100
// of 2048 4.33 and 3.00.
#include "som_barrier.h"
#include "som_device.h"

#include <algorithm>

namespace som {
namespace {
using namespace dev;

constexpr int kSub = 16;         // steps whose L columns a lane holds at a time
constexpr int kSweepDims = 32;   // columns a sweep wave takes at a time (two tiles)
constexpr int kMaxKSplit = 4;    // column ranges of the pass over the prototypes
constexpr int kChain = 2;        // groups of 32 columns between two sums of a sweep wave
constexpr int kGatherDims = 64;  // columns of one gather task
constexpr int kPrepThreads = 256;
constexpr int kTPitch = kSub + 4;
constexpr int kCandidates = 8;   // samples of a panel its centre is chosen from
constexpr int kPairs = kCandidates * (kCandidates - 1) / 2;
constexpr int kPairStride = 32;

// Steps of panel `panel`.
template <int M>
__device__ inline int steps_of(const PanelArgs &p, int64_t panel) {
    const int64_t left = p.t.nsteps - panel * M;
    return (int)(left < M ? left : M);
}

__device__ inline f4 mfma4(const f4 &a, const f4 &b, f4 c) {
#pragma unroll
    for (int v = 0; v < 4; ++v) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v], b[v], c, 0, 0, 0);
    return c;
}

// Coefficients of panel `panel` for unit u, steps 16 t + 4 g .. : its
// sub-blocks' gamma times the later sub-blocks' beta; returns the product of
// all beta.  Every load is made first (a sub-block the panel does not have is
// read as the first one and replaced): one memory round trip.
template <int M>
__device__ inline float panel_coefs(const PanelArgs &p, int64_t panel, int u, int g,
                                    f4 (&gam)[M / 16]) {
    const int nsub = (steps_of<M>(p, panel) + kSub - 1) / kSub;
    const float *pg = p.gam[panel & 1], *pb = p.beta[panel & 1];
    float b[M / 16];
#pragma unroll
    for (int t = 0; t < M / 16; ++t) {
        const int64_t at = (int64_t)(t < nsub ? t : 0) * p.npad + u;
        gam[t] = reinterpret_cast<const f4 *>(pg)[at * 4 + g];
        b[t] = pb[at];
    }
    float bt = 1.f;
#pragma unroll
    for (int t = M / 16 - 1; t >= 0; --t) {
        const f4 zero = {0.f, 0.f, 0.f, 0.f};
        gam[t] = t < nsub ? gam[t] * bt : zero;
        bt *= t < nsub ? b[t] : 1.f;
    }
    return bt;
}

// ------------------------------------------------------------------- sweep

// Operands of one 16-column tile of the pass: lane (g, i) = (lane / 16,
// lane % 16).
template <int M, int TU, bool APPLY, bool PROD>
struct SweepTile {
    f4 w[TU];                       // unit i, columns 4 g .. 4 g + 3
    f4 ec[PROD ? M / 16 : 1];       // column set 16 t + i, columns 4 g ..
    f4 xt[APPLY ? M / 16 : 1];      // column i, steps 16 t + 4 g ..
    f4 z;                           // columns 4 g ..
};

// One task: units 16 TU ugrp .., column range kpart of p.ksplit; panel
// `panel` - 1's updates applied (APPLY) and the products with panel `panel` +
// 1's columns written (PROD).  Wave w of BW takes 32 columns at a time (a whole
// 128-byte line of each row).  Its products go to sums in LDS every 64 columns,
// and the waves' sums are added in fp64: in one chain of fp32 additions over all
// of a wave's columns the rounding of the last ones, at full magnitude, added up.
// Steps off the fp64 minimum on tight clusters (8 of spread 0.02 at unit
// distances), of 400, one chain, sums and the pipelined kernel: 100 x 100 units of
// 2048 floats 55, 25 and 27, 50 x 50 of 10000 87, 40 and 33; the sums cost nothing
// that shows.
//
// What bounds it: the 2 * 2 M N d flops of a panel on the fp32 matrix
// instructions (16x16x4: 32 cycles for 1024 multiply-adds), M / 2 of them per
// 16 x 16 tile of W; at M = 80 the tile's 2 KB of traffic take about 0.7 of
// that time.  The layouts make every operand a 16-byte load and the updated
// tile, the accumulator of the first product, the operand of the second
// without a move: D's row index is the column of W, so a lane ends with four
// consecutive columns of its unit.
template <int M, int TU, int BW, bool APPLY, bool PROD>
__device__ inline void sweep_task(const PanelArgs &p, int64_t panel, int ugrp, int kpart,
                                  unsigned char *smem) {
    constexpr int NT = M / 16;
    const TrainArgs &a = p.t;
    const bool stop = a.state->order_bad != 0;  // unusable input: no prototype is written
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int u0 = ugrp * 16 * TU;
    // the waves' sums of products, [BW][TU NT][64], and of squares, [BW][16 TU]
    f4 *sums = reinterpret_cast<f4 *>(smem);
    double *qred = reinterpret_cast<double *>(sums + BW * TU * NT * 64);
    f4 *own = sums + wave * TU * NT * 64 + lane;
    if constexpr (PROD) __syncthreads();  // (a workgroup's earlier task may still read them)
    f4 gam[TU][NT];
    float bt[TU];
    if constexpr (APPLY)
#pragma unroll
        for (int tu = 0; tu < TU; ++tu)
            bt[tu] = panel_coefs<M>(p, panel - 1, min(u0 + 16 * tu + i, a.N - 1), g, gam[tu]);
    f4 acc[TU][NT];
    double q[TU];
#pragma unroll
    for (int tu = 0; tu < TU; ++tu) {
        q[tu] = 0.0;
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[tu][t] = f4{0.f, 0.f, 0.f, 0.f};
    }
    const float *xt = p.xt[(panel + 3) & 3];  // panel - 1's samples
    const float *ec = p.ec[(panel + 1) & 1];  // panel + 1's columns
    const int groups = p.dpad / kSweepDims;
    const int k0 = (int)((int64_t)groups * kpart / p.ksplit);
    const int k1 = (int)((int64_t)groups * (kpart + 1) / p.ksplit);
    const int mine = k1 - k0 > wave ? (k1 - k0 - wave + BW - 1) / BW : 0;  // of this wave
    float *wrow[TU];
    bool real[TU];
#pragma unroll
    for (int tu = 0; tu < TU; ++tu) {
        const int u = u0 + 16 * tu + i;
        real[tu] = u < a.N && !stop;
        wrow[tu] = a.W + (int64_t)min(u, a.N - 1) * a.ld;
    }
    const auto first_col = [&](int n) {  // of tile n (two tiles per group)
        const int grp = min(n >> 1, mine - 1);
        return (k0 + wave + BW * grp) * kSweepDims + (n & 1) * 16;
    };
    typedef SweepTile<M, TU, APPLY, PROD> Tile;
    const auto load = [&](Tile &s, int n) {
        const int c = first_col(n);
#pragma unroll
        for (int tu = 0; tu < TU; ++tu)
            s.w[tu] = *reinterpret_cast<const f4 *>(wrow[tu] + c + 4 * g);
        if constexpr (PROD) {
            s.z = *reinterpret_cast<const f4 *>(ec + (int64_t)M * p.dpad + c + 4 * g);
#pragma unroll
            for (int t = 0; t < NT; ++t)
                s.ec[t] = *reinterpret_cast<const f4 *>(ec + (int64_t)(16 * t + i) * p.dpad + c +
                                                        4 * g);
        }
        if constexpr (APPLY) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
                s.xt[t] = *reinterpret_cast<const f4 *>(xt + (int64_t)(c + i) * M + 16 * t + 4 * g);
        }
    };
    const auto compute = [&](Tile &s, int n) {
        f4 w[TU];
#pragma unroll
        for (int tu = 0; tu < TU; ++tu) {
            w[tu] = s.w[tu];
            if constexpr (APPLY) w[tu] = w[tu] * bt[tu];
        }
        if constexpr (APPLY) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int tu = 0; tu < TU; ++tu)
                        w[tu] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.xt[t][v], gam[tu][t][v],
                                                                     w[tu], 0, 0, 0);
            const int c = first_col(n);
#pragma unroll
            for (int tu = 0; tu < TU; ++tu)
                if (real[tu]) *reinterpret_cast<f4 *>(wrow[tu] + c + 4 * g) = w[tu];
        }
        if constexpr (PROD) {
#pragma unroll
            for (int tu = 0; tu < TU; ++tu) {
                w[tu] = w[tu] - s.z;
                q[tu] += (double)fmaf(w[tu][0], w[tu][0], w[tu][1] * w[tu][1]) +
                         (double)fmaf(w[tu][2], w[tu][2], w[tu][3] * w[tu][3]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int tu = 0; tu < TU; ++tu)
                        acc[tu][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.ec[t][v], w[tu][v],
                                                                          acc[tu][t], 0, 0, 0);
        }
    };
    // The products so far to the wave's sums, which start at zero.
    const auto flush = [&](bool first) {
#pragma unroll
        for (int tu = 0; tu < TU; ++tu)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                f4 *to = own + (tu * NT + t) * 64;
                *to = first ? acc[tu][t] : *to + acc[tu][t];
                acc[tu][t] = f4{0.f, 0.f, 0.f, 0.f};
            }
    };
    if (mine > 0) {
        Tile t0, t1;
        load(t0, 0);
        for (int n = 0; n < 2 * mine; n += 2) {
            load(t1, n + 1);
            compute(t0, n);
            load(t0, n + 2);  // past the end: the last group again, unused
            compute(t1, n + 1);
            if constexpr (PROD)
                if ((n >> 1) % kChain == kChain - 1) flush(n >> 1 == kChain - 1);
        }
    }
    if constexpr (PROD) {
        flush(mine < kChain);
#pragma unroll
        for (int tu = 0; tu < TU; ++tu) {
            q[tu] += __shfl_xor(q[tu], 16, 64);
            q[tu] += __shfl_xor(q[tu], 32, 64);
            if (g == 0) qred[wave * 16 * TU + 16 * tu + i] = q[tu];
        }
        __syncthreads();
        // the waves' sums added in order, a share of them by each wave
        float *prod = p.prod[(panel + 1) & 1];
        double *qf = p.qf[(panel + 1) & 1];
        for (int e = wave; e < TU * NT; e += BW) {
            double v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = sums[e * 64 + lane][k];
#pragma unroll
            for (int w = 1; w < BW; ++w) {
                const f4 x = sums[(w * TU * NT + e) * 64 + lane];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] += (double)x[k];
            }
            const int tu = e / NT, t = e - tu * NT;
            const int64_t row = (int64_t)kpart * p.npad + u0 + 16 * tu + i;
            *reinterpret_cast<f4 *>(prod + row * M + 16 * t + 4 * g) =
                f4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
        }
        if (wave == BW - 1 && lane < 16 * TU) {
            double s = qred[lane];
#pragma unroll
            for (int w = 1; w < BW; ++w) s += qred[w * 16 * TU + lane];
            qf[(int64_t)kpart * p.npad + u0 + lane] = s;
        }
    }
}

template <int M, int TU, int BW>
constexpr size_t sweep_lds() {
    return (size_t)BW * TU * (M / 16) * 64 * 16 + (size_t)BW * 16 * TU * 8;
}

// Sweep task t of a panel: unit group t / ksplit, column range t % ksplit.
template <int M, int TU, int BW>
__device__ inline void sweep(const PanelArgs &p, int64_t panel, int t, bool apply, bool prod,
                             unsigned char *smem) {
    const int ugrp = t / p.ksplit, kpart = t - ugrp * p.ksplit;
    if (apply && prod)
        sweep_task<M, TU, BW, true, true>(p, panel, ugrp, kpart, smem);
    else if (apply)
        sweep_task<M, TU, BW, true, false>(p, panel, ugrp, kpart, smem);
    else
        sweep_task<M, TU, BW, false, true>(p, panel, ugrp, kpart, smem);
}

// ----------------------------------------------------------------- prepare

// Sample row of step s (the call's last step stands for the steps past it).
__device__ inline const float *step_row(const PanelArgs &p, int64_t s) {
    const TrainArgs &a = p.t;
    // (an index outside [0, n) stops the call before any update; here it only
    // must not be followed)
    const int idx = a.order[s < a.nsteps ? s : a.nsteps - 1];
    return a.X + (int64_t)(idx >= 0 && idx < a.n ? idx : 0) * a.d;
}

// Step, within its panel, of a panel's candidate c for its centre.
template <int M>
__device__ inline int candidate_step(const PanelArgs &p, int64_t panel, int c) {
    return steps_of<M>(p, panel) * c / kCandidates;
}
__device__ inline int pair_index(int i, int j) {  // i < j
    return i * (2 * kCandidates - 1 - i) / 2 + j - i - 1;
}

// Centre of a panel, as its step within the panel: of its candidates the one
// whose median squared distance to the other seven is smallest (the lowest
// such; 0 for a panel past the call's last).  Every wave finds it for itself,
// lane l for candidate l % 8.
template <int M>
__device__ inline int centre_step(const PanelArgs &p, int64_t panel) {
    if (panel * M >= p.t.nsteps) return 0;
    const int c = threadIdx.x & (kCandidates - 1);
    const float *near = p.near[panel & 3];
    float v[kCandidates - 1];
#pragma unroll
    for (int j = 0; j < kCandidates - 1; ++j) {
        const int o = j + (j >= c ? 1 : 0);  // the j-th other candidate
        const int at = pair_index(min(c, o), max(c, o));
        v[j] = 0.f;
        for (int k = 0; k < p.gsplit; ++k) v[j] += near[k * kPairStride + at];
    }
    float median = v[0];
#pragma unroll
    for (int j = 0; j < kCandidates - 1; ++j) {
        int place = 0;
#pragma unroll
        for (int k = 0; k < kCandidates - 1; ++k)
            place += v[k] < v[j] || (v[k] == v[j] && k < j) ? 1 : 0;
        median = place == (kCandidates - 1) / 2 ? v[j] : median;
    }
    unsigned long long key =
        ((unsigned long long)__float_as_uint(median) << 32) | (unsigned)c;
#pragma unroll
    for (int o = 1; o < kCandidates; o *= 2) key = u64_min(key, __shfl_xor(key, o, 64));
    return candidate_step<M>(p, panel, __builtin_amdgcn_readfirstlane((int)(unsigned)key));
}

// Step whose sample is column l of a panel with centre step z: its steps, but
// the next panel's centre (step `next` there) in the place of its own.
template <int M>
__device__ inline int64_t column_step(int64_t panel, int l, int z, int next) {
    return panel * M + (l == z ? M + next : l);
}

// Floats of one column range's part of a Gram matrix.
template <int M>
constexpr int gram_stride() {
    return M * M + 16;
}

// Columns c .. c + 3 of a sample row, zero past d.
__device__ inline f4 row_f4(const PanelArgs &p, const float *x, int c) {
    const int d = p.t.d;
    f4 v;
    if (p.x_vec4) {
        v = *reinterpret_cast<const f4 *>(x + (c < d ? c : d - 4));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = x[c + e < d ? c + e : d - 1];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = c + e < d ? v[e] : 0.f;
    return v;
}

// Gather task: columns 64 task .. of a panel: its column set less the centre
// into ec (row M: the centre), its steps' samples transposed into xt.
template <int M>
__device__ inline void gather_task(const PanelArgs &p, int64_t panel, int task, float *lds) {
    constexpr int P = kGatherDims + 1;
    const int t = threadIdx.x, c4 = t & 15, r0 = t >> 4;
    const int c = task * kGatherDims + 4 * c4;
    float *xt = p.xt[panel & 3], *ec = p.ec[panel & 1];
    const int zs = centre_step<M>(p, panel), next = centre_step<M>(p, panel + 1);
    const f4 z = row_f4(p, step_row(p, panel * M + zs), c);
    f4 x[M / 16];
#pragma unroll
    for (int k = 0; k < M / 16; ++k)
        x[k] = row_f4(p, step_row(p, column_step<M>(panel, r0 + 16 * k, zs, next)), c);
#pragma unroll
    for (int k = 0; k < M / 16; ++k) {
        const int r = r0 + 16 * k;
        *reinterpret_cast<f4 *>(ec + (int64_t)r * p.dpad + c) = x[k] - z;
#pragma unroll
        for (int e = 0; e < 4; ++e) lds[r * P + 4 * c4 + e] = r == zs ? z[e] : x[k][e];
    }
    if (r0 == 0) *reinterpret_cast<f4 *>(ec + (int64_t)M * p.dpad + c) = z;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < M / 16; ++k) {
        const int e = t + kPrepThreads * k, dim = e / (M / 4), j = 4 * (e % (M / 4));
        f4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = lds[(j + q) * P + dim];
        *reinterpret_cast<f4 *>(xt + (int64_t)(task * kGatherDims + dim) * M + j) = v;
    }
}

// Gram task: one 16 x 16 tile of products of a panel's column set over column
// range `part` of p.gsplit.  pair < M/16 (M/16 + 1) / 2: with its own steps
// e_j, into gm (both tiles of the pair); after that: with panel - 1's samples
// in this panel's centring, into gx.  Both are [column l][step j].
template <int M>
__device__ inline void gram_task(const PanelArgs &p, int64_t panel, int pair, int part, f4 *lds) {
    constexpr int NT = M / 16, kOwn = NT * (NT + 1) / 2;
    const bool own = pair < kOwn;
    int ti = 0, tj;  // tile of the steps, tile of the columns
    if (own) {
        int left = pair;
        while (left >= NT - ti) {
            left -= NT - ti;
            ++ti;
        }
        tj = ti + left;
    } else {
        if (panel == 0) return;  // (no panel before it)
        ti = (pair - kOwn) / NT;
        tj = (pair - kOwn) % NT;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
    const int64_t s0 = panel * M;
    const int z = centre_step<M>(p, panel), next = centre_step<M>(p, panel + 1);
    if (pair == 0 && part == 0 && threadIdx.x == 0) p.centre[panel & 3] = z;
    const float *xa = step_row(
        p, own ? column_step<M>(panel, 16 * ti + i, z, next) : s0 - M + 16 * ti + i);
    const float *xb = step_row(p, column_step<M>(panel, 16 * tj + i, z, next));
    const float *xz = step_row(p, s0 + z);
    const int tiles = p.dpad / 16;
    const int k0 = (int)((int64_t)tiles * part / p.gsplit);
    const int k1 = (int)((int64_t)tiles * (part + 1) / p.gsplit);
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    constexpr int kDepth = 4;
    for (int k = k0 + wave; k < k1; k += 4 * kDepth) {
        f4 va[kDepth], vb[kDepth], vz[kDepth];
#pragma unroll
        for (int n = 0; n < kDepth; ++n) {
            const int c = 16 * (k + 4 * n < k1 ? k + 4 * n : k) + 4 * g;
            va[n] = row_f4(p, xa, c);
            vb[n] = row_f4(p, xb, c);
            vz[n] = row_f4(p, xz, c);
        }
#pragma unroll
        for (int n = 0; n < kDepth; ++n)
            if (k + 4 * n < k1) acc = mfma4(va[n] - vz[n], vb[n] - vz[n], acc);
    }
    if (wave > 0) lds[(wave - 1) * 64 + lane] = acc;
    __syncthreads();
    if (wave > 0) return;
    acc = acc + lds[lane] + lds[64 + lane] + lds[128 + lane];
    // acc[v]: step 16 ti + 4 g + v, column 16 tj + i
    float *G = (own ? p.gm : p.gx)[panel % 3] + (int64_t)part * gram_stride<M>();
    // the centre's own step moves no column (its place among the columns holds
    // the next centre, whose norm goes behind the matrix)
    if (own && ti != tj)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            G[(16 * ti + 4 * g + v) * M + 16 * tj + i] = 16 * tj + i == z ? 0.f : acc[v];
    if (own)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (16 * ti + 4 * g + v == z) {
                if (16 * tj + i == z) G[M * M] = acc[v];
                acc[v] = 0.f;
            }
    *reinterpret_cast<f4 *>(G + (16 * tj + i) * M + 16 * ti + 4 * g) = acc;
}

template <int M>
constexpr int gram_pairs() {
    return (M / 16) * (M / 16 + 1) / 2 + (M / 16) * (M / 16);
}

// (the first kPrepThreads threads of a workgroup)
template <int M>
__device__ inline void prepare_task(const PanelArgs &p, int64_t panel, int task, float *lds) {
    // the Gram tasks first: they take longest
    const int ngram = gram_pairs<M>() * p.gsplit;
    if (task < ngram)
        gram_task<M>(p, panel, task % gram_pairs<M>(), task / gram_pairs<M>(),
                     reinterpret_cast<f4 *>(lds));
    else
        gather_task<M>(p, panel, task - ngram, lds);
}

constexpr size_t kPrepareLds = 80 * (kGatherDims + 1) * 4;

// Select task: the candidates' squared distances over column range `part`, from
// direct differences, for centre_step.
template <int M>
__device__ inline void select_task(const PanelArgs &p, int64_t panel, int part, float *lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float *x[kCandidates];
#pragma unroll
    for (int c = 0; c < kCandidates; ++c)
        x[c] = step_row(p, panel * M + candidate_step<M>(p, panel, c));
    const int quads = p.dpad / 4;
    const int q0 = (int)((int64_t)quads * part / p.gsplit);
    const int q1 = (int)((int64_t)quads * (part + 1) / p.gsplit);
    float acc[kPairs];
#pragma unroll
    for (int k = 0; k < kPairs; ++k) acc[k] = 0.f;
    for (int q = q0 + threadIdx.x; q < q1; q += kPrepThreads) {
        f4 v[kCandidates];
#pragma unroll
        for (int c = 0; c < kCandidates; ++c) v[c] = row_f4(p, x[c], 4 * q);
        int k = 0;
#pragma unroll
        for (int i = 0; i < kCandidates; ++i)
#pragma unroll
            for (int j = i + 1; j < kCandidates; ++j, ++k) {
                const f4 e = v[i] - v[j];
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[k] = fmaf(e[c], e[c], acc[k]);
            }
    }
    wave_sums<kPairs>(acc);
#pragma unroll
    for (int k = 0; k < kPairs; ++k)
        if (lane == k) lds[wave * kPairStride + k] = acc[k];
    __syncthreads();
    if (threadIdx.x < kPairs) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kPrepThreads / 64; ++w) s += lds[w * kPairStride + threadIdx.x];
        p.near[panel & 3][part * kPairStride + threadIdx.x] = s;
    }
}

// ----------------------------------------------------------------- correct

// A panel's centre, as its step within the panel.
__device__ inline int centre_of(const PanelArgs &p, int64_t panel) {
    return __builtin_amdgcn_readfirstlane(__hip_atomic_load(
        p.centre + (panel & 3), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// One wave: the products of units u0 .. u0 + 15 at panel `panel`'s start from
// the sweep's partial products and panel - 1's coefficients, into pc and qc.
// The coefficients' product runs from zero on the matrix instructions and is
// added in fp64, so units far from the BMUs, whose gamma vanish, keep the
// sweep's value exactly.  The next centre's column goes into pz; in its place
// stands the own centre's, zero.
template <int M>
__device__ inline void correct_tile(const PanelArgs &p, int64_t panel, int u0) {
    constexpr int NT = M / 16;
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int u = min(u0 + i, p.t.N - 1);
    const float *prod = p.prod[panel & 1], *gx = p.gx[panel % 3];
    const double *qf = p.qf[panel & 1];
    const int z = centre_of(p, panel);
    f4 gam[NT], part[kMaxKSplit][NT];
    double q = 0.0;
    const double qn = p.qn[u], qe = p.qe[u];
#pragma unroll
    for (int k = 0; k < kMaxKSplit; ++k) {
        const int64_t row = (int64_t)(k < p.ksplit ? k : 0) * p.npad + u;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            part[k][t] = *reinterpret_cast<const f4 *>(prod + row * M + 16 * t + 4 * g);
        const double v = qf[row];
        q += k < p.ksplit ? v : 0.0;
    }
    const float bt = panel > 0 ? panel_coefs<M>(p, panel - 1, u, g, gam) : 1.f;
    f4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
    if (panel > 0) {
        for (int k = 0; k < p.gsplit; ++k)
#pragma unroll
            for (int s = 0; s < NT; ++s) {
                f4 ga[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    ga[t] = *reinterpret_cast<const f4 *>(gx + (int64_t)k * gram_stride<M>() +
                                                          (16 * t + i) * M + 16 * s + 4 * g);
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ga[t][v], gam[s][v], acc[t],
                                                                      0, 0, 0);
            }
        q = fma((double)bt * bt, q - qe, qn);
    }
    if (u0 + i < p.t.N) {
        double next = 0.0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            typedef double d2 __attribute__((ext_vector_type(2)));
            double v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = part[0][t][e];
#pragma unroll
                for (int k = 1; k < kMaxKSplit; ++k)
                    v[e] += k < p.ksplit ? (double)part[k][t][e] : 0.0;
                v[e] = fma((double)bt, v[e], (double)acc[t][e]);
                const bool own = 16 * t + 4 * g + e == z;
                next = own ? v[e] : next;
                v[e] = own ? 0.0 : v[e];
            }
            d2 *to = reinterpret_cast<d2 *>(p.pc + (int64_t)u * M + 16 * t + 4 * g);
            to[0] = d2{v[0], v[1]};
            to[1] = d2{v[2], v[3]};
        }
        if (g == (z >> 2 & 3)) p.pz[u] = next;
        if (g == 0) p.qc[u] = q;
    }
}

// ----------------------------------------------------------------- control

// Smallest of the lanes' values over each row of 16 lanes, and over the wave.
template <int CTRL>
__device__ inline int dpp_min(int v) {
    return min(v, dpp_move<CTRL>(v));
}
__device__ inline int row_min_i32(int v) {
    v = dpp_min<0xB1>(v);     // quad_perm [1,0,3,2]
    v = dpp_min<0x4E>(v);     // quad_perm [2,3,0,1]
    v = dpp_min<0x141>(v);    // row_half_mirror
    return dpp_min<0x140>(v); // row_mirror
}
__device__ inline int rows01_min_i32(int v) {  // of rows 0 and 1, and of rows 2 and 3
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    return min((int)r[0], (int)r[1]);
}
__device__ inline int wave_min_i32(int v) {
    v = rows01_min_i32(row_min_i32(v));
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return min((int)h[0], (int)h[1]);
}

typedef double d2 __attribute__((ext_vector_type(2)));
__device__ inline void load_row(float (&r)[kSub], const float *src) {
#pragma unroll
    for (int v = 0; v < kSub / 4; ++v) {
        const f4 x = *reinterpret_cast<const f4 *>(src + 4 * v);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[4 * v + e] = x[e];
    }
}
__device__ inline void load_row(double (&r)[kSub], const double *src) {
#pragma unroll
    for (int v = 0; v < kSub / 2; ++v) {
        const d2 x = *reinterpret_cast<const d2 *>(src + 2 * v);
        r[2 * v] = x[0];
        r[2 * v + 1] = x[1];
    }
}
__device__ inline double lane_d(double v, int l) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// f(0), f(1), .. f(END - 1) with compile-time arguments until one is false
// (expanded by the front end, so that arrays indexed by the argument stay in
// registers whatever the body's size and exits).
template <int K, int END, typename F>
__device__ __forceinline__ void steps_from(F &&f) {
    if constexpr (K < END)
        if (f(std::integral_constant<int, K>{})) steps_from<K + 1, END>(f);
}

// Shape of a control workgroup: NW waves of U units per lane, unit
// (64 wave + lane) U + slot of its share, so that the lowest lane (and in it
// the lowest slot) of equal distances is the lowest unit.  LDS byte offsets;
// `rows` is the units whose coefficients are kept (a multiple of 16).
template <int M, int U, int NW>
struct ControlLds {
    static constexpr int kUnits = U * NW * 64;
    static constexpr int kGram = 0;
    static constexpr int kCentre = M * M * 4;                     // M + 16 floats
    static constexpr int kKeys = kCentre + (M + 16) * 4;          // [2][4 NW]
    static constexpr int kWhere = kKeys + 2 * 4 * NW * 8;         // [2][4 NW]
    static constexpr int kBlocks = kWhere + 2 * 4 * NW * 8;       // [M / 16][16][16] fp64
    static constexpr int kTrans = kBlocks + M * kSub * 8;         // 32 units a wave
    static constexpr int kCoef = kTrans + NW * 32 * kTPitch * 4;
    static constexpr size_t bytes(int rows) {
        return (size_t)kCoef + (size_t)(M / 16 - 1) * rows * (kSub + 1) * 4;
    }
};

// A bounded wait ran into its bound: the call ends with SOM_E_TIMEOUT, and what
// is still to run of it leaves.
__device__ inline void give_up(const TrainArgs &a) {
    __hip_atomic_store(&a.state->status, kStatusTimeout, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&a.state->order_bad, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The steps of one panel for a workgroup's units; false once an exchange, or a
// wait for the workgroup's other waves, was given up.  A lane holds, for each of
// its units, Q and the L columns of the current 16 steps; at the start of each 16
// they are formed from the panel's starting products and its earlier coefficients
// (matrix instructions, then through LDS from the accumulators' layout to one unit
// per lane).
//
// What bounds it: on one workgroup the chain of a step, distance - row
// minimum - LDS - minimum - factor, about 90 dependent instructions and one
// LDS round trip, and beyond 512 units the issue of U units a lane; on
// several the grid exchange.
template <int M, int U, int NW, bool GRID>
__device__ inline bool control_panel(const PanelArgs &p, int64_t panel, unsigned char *lds) {
    typedef ControlLds<M, U, NW> Lds;
    const TrainArgs &a = p.t;
    const int lane = threadIdx.x & 63;
    const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int rows = p.ctl_rows;
    const int base = GRID ? (int)blockIdx.x * Lds::kUnits : 0;
    const int mine = (wave * 64 + lane) * U;  // the lane's first unit of the workgroup's
    float *G = reinterpret_cast<float *>(lds + Lds::kGram);
    float *centre = reinterpret_cast<float *>(lds + Lds::kCentre);
    float *T = reinterpret_cast<float *>(lds + Lds::kTrans) + wave * 32 * kTPitch;
    double *blocks = reinterpret_cast<double *>(lds + Lds::kBlocks);
    unsigned long long *keys = reinterpret_cast<unsigned long long *>(lds + Lds::kKeys);
    unsigned long long *where = reinterpret_cast<unsigned long long *>(lds + Lds::kWhere);
    float *cg = reinterpret_cast<float *>(lds + Lds::kCoef);   // [q][rows][16]
    float *cb = cg + (M / 16 - 1) * rows * kSub;               // [q][rows]
    const int64_t s0 = panel * M;
    // the centre's step; its column is the next centre's
    const int z = centre_of(p, panel);
    const int nst = steps_of<M>(p, panel);
    const bool bad = a.state->order_bad != 0;

    // The 16 steps' starting products of the lane's units, loaded a sub-block
    // ahead so that their round trip runs under the steps.
    double ahead[U][kSub];
    const auto fetch = [&](int sub) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            load_row(ahead[u],
                     p.pc + (int64_t)min(base + mine + u, a.N - 1) * M + kSub * sub);
    };
    fetch(0);
    double Q[U], Lz[U], bsub[U];  // bsub: product of the panel's beta so far
    float row[U], col[U];
    const float rscale = a.topology == 1 ? 0.75f : 1.f;
    const float shift = a.topology == 1 ? 0.5f : 0.f;
    const float inv_cols = 1.f / (float)a.cols;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int unit = base + mine + u;
        const int at = min(unit, a.N - 1);
        const double q = p.qc[at];
        Q[u] = unit < a.N ? q : (double)INFINITY;  // a unit past N is never nearest
        Lz[u] = p.pz[at];
        bsub[u] = 1.0;
        int r, c;
        unit_rc(at, a.cols, inv_cols, r, c);
        // HEX: odd rows half a unit to the right, rows sqrt(3/4) apart
        row[u] = (float)r;
        col[u] = (float)c + shift * (float)(r & 1);
    }
    {
        // the Gram matrix; the next centre's row apart, zero in its place
        const float *src = p.gm[panel % 3];
        constexpr int kTotal = M * M / 4, kStep = NW * 64, kBatch = 5;
        for (int e0 = threadIdx.x; e0 < kTotal; e0 += kBatch * kStep) {
            f4 v[kBatch];
#pragma unroll
            for (int n = 0; n < kBatch; ++n)
                v[n] = reinterpret_cast<const f4 *>(src)[min(e0 + n * kStep, kTotal - 1)];
            for (int k = 1; k < p.gsplit; ++k)
#pragma unroll
                for (int n = 0; n < kBatch; ++n)
                    v[n] = v[n] + reinterpret_cast<const f4 *>(
                                      src + (int64_t)k * gram_stride<M>())[min(e0 + n * kStep,
                                                                               kTotal - 1)];
#pragma unroll
            for (int n = 0; n < kBatch; ++n) {
                const int e = e0 + n * kStep;
                const f4 zero = {0.f, 0.f, 0.f, 0.f};
                if (e < kTotal) {
                    const int l = 4 * e / M, c = 4 * e % M;
                    if (l == z) reinterpret_cast<f4 *>(centre)[c / 4] = v[n];
                    const f4 r = l == z ? zero : v[n];
                    reinterpret_cast<f4 *>(G)[e] = r;
                    if (l / kSub == c / kSub)
#pragma unroll
                        for (int x = 0; x < 4; ++x)
                            blocks[l * kSub + c % kSub + x] = (double)r[x];
                }
            }
        }
        if (threadIdx.x == 0) {
            float zz = src[M * M];
            for (int k = 1; k < p.gsplit; ++k) zz += src[(int64_t)k * gram_stride<M>() + M * M];
            centre[M] = zz;
        }
        if (NW > 1 && threadIdx.x < 2 * 4 * NW) keys[threadIdx.x] = 0ull;
    }
    if (NW > 1)
        __syncthreads();
    else
        __builtin_amdgcn_wave_barrier();
    if (!GRID && bad) return true;  // unusable input, or an earlier panel was given up
    const double zz = (double)centre[M];  // |z' - z|^2
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (base + mine + u < a.N) p.qe[base + mine + u] = fma(-2.0, Lz[u], Q[u]) + zz;
    PollRegs<4> polls;
#pragma unroll
    for (int q = 0; q < 4; ++q) polls.v[q] = 0;
    // rows of 16 lanes that hold units, of the 4 NW of the workgroup
    const int lanes = (min(a.N - base, Lds::kUnits) + U - 1) / U;
    const bool waits = (lane & (4 * NW - 1)) * 16 < lanes;
    // A wave without units leaves here: it would publish no keys, so nothing
    // would keep the other waves from overwriting, two steps on, those it
    // still waits for.
    if (!GRID && wave * 64 >= lanes) return true;
    // (failure-path tests: the last wave with units does not take part)
    if (!GRID && p.absent && (wave + 1) * 64 >= lanes) return true;
    const int wave_rows = min((lanes - wave * 64 + 15) / 16, 4);  // rows with units
    // Looks left at the keys this lane waits for in this panel: the bound of its
    // waits.  Beyond it the steps run on with what they have, until the end of
    // their 16.  (A counter of its own for every wait cost 1.2-2.5 % of a call.)
    int looks = waits ? p.max_looks : 0;

    for (int sub = 0; sub * kSub < nst; ++sub) {
        // ---- L columns of the 16 steps
        double L[U][kSub];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < kSub; ++k)
                L[u][k] = bsub[u] * ahead[u][k];
        fetch(sub + 1 < M / 16 ? sub + 1 : sub);
        if (sub > 0) {
            // the panel's earlier coefficients, from zero in fp32
#pragma unroll
            for (int u = 0; u < U; ++u) {
                f4 acc[4], ga, gb[4];
                int lr[4];
                float b[4];
#pragma unroll
                for (int tile = 0; tile < 4; ++tile) {
                    acc[tile] = f4{0.f, 0.f, 0.f, 0.f};
                    lr[tile] = min((wave * 64 + 16 * tile + i) * U + u, rows - 1);
                }
                const auto operands = [&](int q) {
                    ga = *reinterpret_cast<const f4 *>(G + (kSub * sub + i) * M + kSub * q +
                                                       4 * g);
#pragma unroll
                    for (int tile = 0; tile < 4; ++tile) {
                        gb[tile] = *reinterpret_cast<const f4 *>(
                            cg + (q * rows + lr[tile]) * kSub + 4 * g);
                        b[tile] = cb[q * rows + lr[tile]];
                    }
                };
                operands(0);
                for (int q = 0; q < sub; ++q) {
                    const f4 va = ga, vb[4] = {gb[0], gb[1], gb[2], gb[3]};
#pragma unroll
                    for (int tile = 0; tile < 4; ++tile) acc[tile] = acc[tile] * b[tile];
                    if (q + 1 < sub) operands(q + 1);
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int tile = 0; tile < 4; ++tile)
                            acc[tile] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[v], vb[tile][v],
                                                                             acc[tile], 0, 0, 0);
                }
                float own[kSub];
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    __builtin_amdgcn_wave_barrier();  // own wave's LDS, in program order
#pragma unroll
                    for (int tile = 0; tile < 2; ++tile)
                        *reinterpret_cast<f4 *>(T + (16 * tile + i) * kTPitch + 4 * g) =
                            acc[2 * half + tile];
                    __builtin_amdgcn_wave_barrier();
                    if ((lane >> 5) == half) load_row(own, T + (lane & 31) * kTPitch);
                }
#pragma unroll
                for (int k = 0; k < kSub; ++k) L[u][k] += (double)own[k];
            }
        }

        // ---- the steps
        float hs[U][kSub];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < kSub; ++k) hs[u][k] = 0.f;
        const double *Gs = blocks + sub * kSub * kSub;
        // lane k holds the k-th step's schedule entry, the Gram entries (k, k)
        // and (k, k + 1), which the chain of a step needs at once, and the
        // step's product with the next centre
        const int lk = lane & (kSub - 1);
        const float2 sched = fetch_entry(a, s0 + kSub * sub + lk, float2());
        const double diag = Gs[lk * (kSub + 1)];
        const float zcol = centre[kSub * sub + lk];
        const double above = Gs[lk * (kSub + 1) + (lk + 1 < kSub)];
        int trace = 0;
        double grow[kSub];  // the last step's row of the Gram matrix
        double hp[U];
        bool ok = true;
        // Step k - 1's factors reach column k at once and the later columns
        // here, while step k's keys are on their way.
        const auto later_columns = [&](auto kk) {
            constexpr int k = decltype(kk)::value;
            if constexpr (k > 0)
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int l = k + 1; l < kSub; ++l) {
                        L[u][l] = fma(hp[u], grow[l] - L[u][l], L[u][l]);
                        // (here, and not sunk to the column's first use)
                        asm volatile("" : "+v"(L[u][l]));
                    }
        };
        steps_from<0, kSub>([&](auto kk) {
            constexpr int k = decltype(kk)::value;
            if (kSub * sub + k >= nst) return false;
            const int64_t s = s0 + kSub * sub + k;
            const float lr = lane_f(sched.x, k), c2 = lane_f(sched.y, k);
            const double gkk = lane_d(diag, k), gk1 = lane_d(above, k);
            const double gkz = (double)lane_f(zcol, k);
            // The distances as integers: positive ones in order, negative ones
            // (the rounding of a distance near zero) below them, a NaN as inf.
            double D[U];
            int m = 0x7fffffff, unit = 0;
            float wr = 0.f, wc = 0.f;
#pragma unroll
            for (int u = U - 1; u >= 0; --u) {
                D[u] = fma(-2.0, L[u][k], gkk) + Q[u];
                const int ob = __float_as_int(fminf((float)D[u], INFINITY));
                const bool less = U == 1 || ob <= m;
                unit = less ? base + mine + u : unit;
                wr = less ? row[u] : wr;
                wc = less ? col[u] : wc;
                m = less ? ob : m;
            }
            float cr, cc;
            int c;
            if constexpr (GRID) {
                const int wm = wave_min_i32(m);
                const int at = __builtin_ctzll(__ballot(m == wm));
                const unsigned long long key =
                    ((unsigned long long)((unsigned)wm ^ 0x80000000u) << 32) |
                    (unsigned)__builtin_amdgcn_readlane(unit, at);
                exchange_publish(a, s, key);
                c = exchange_wait<4>(a, s, key, [&] { later_columns(kk); }, polls);
                if (c < 0) {
                    ok = false;
                    return false;
                }
                int r, q;
                unit_rc(c, a.cols, inv_cols, r, q);
                cr = (float)r;
                cc = (float)q + shift * (float)(r & 1);
            } else {
                // The lowest lane of each row of 16 lanes at the row's minimum
                // puts its key into LDS, tagged by step, after the position it
                // stands for (a wave's LDS operations keep their order, and the
                // fences keep the compiler's: position before key here, key
                // before position where they are read).  A wave overwrites
                // its keys of step s - 2 only after it has read all keys of
                // step s - 1, so after all have read those of step s - 2.
                const int rm = row_min_i32(m);
                bool win = m == rm && base + mine < a.N;
                const unsigned long long wins = __ballot(win);
                if (__builtin_popcountll(wins) > wave_rows)  // equal distances in a row
                    win = win && (((wins >> (lane & 48)) & ((1ull << i) - 1)) == 0);
                const unsigned tag = 0x80u | (unsigned)(k >> 1) | ((unsigned)sub << 3);
                unsigned long long *slots = keys + (k & 1) * 4 * NW,
                                   *pos = where + (k & 1) * 4 * NW;
                if (win) {
                    __hip_atomic_store(pos + wave * 4 + g,
                                       ((unsigned long long)__float_as_uint(wc) << 32) |
                                           __float_as_uint(wr),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __atomic_signal_fence(__ATOMIC_SEQ_CST);
                    __hip_atomic_store(slots + wave * 4 + g,
                                       ((unsigned long long)(unsigned)m << 32) |
                                           (tag << kUnitBits) | (unsigned)unit,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                later_columns(kk);
                unsigned long long v, w;
                do {
                    --looks;
                    v = __hip_atomic_load(slots + (lane & (4 * NW - 1)), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
                    __atomic_signal_fence(__ATOMIC_SEQ_CST);
                    w = __hip_atomic_load(pos + (lane & (4 * NW - 1)), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
                } while (__ballot(looks >= 0 && ((unsigned)(v >> kUnitBits) & 0xffu) != tag) != 0);
                const int hi = waits ? (int)(v >> 32) : 0x7fffffff;
                int mh = row_min_i32(hi);
                if constexpr (NW == 8) mh = rows01_min_i32(mh);
                const int win_lane = __builtin_ctzll(__ballot(hi == mh));
                cr = lane_f(__uint_as_float((unsigned)w), win_lane);
                cc = lane_f(__uint_as_float((unsigned)(w >> 32)), win_lane);
                c = __builtin_amdgcn_readlane((int)((unsigned)v & 0xffffffu), win_lane);
            }
            if (k + 2 < kSub) load_row(grow, Gs + k * kSub);
            trace = lane == k ? c : trace;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float dr = row[u] - cr, dx = col[u] - cc;
                const float h =
                    lr * __builtin_amdgcn_exp2f(-c2 * fmaf(dx, dx, (rscale * dr) * dr));
                const double hd = (double)h;
                hs[u][k] = h;
                // Q + h (G - Q - (1 - h) D)
                Q[u] = fma(hd, fma(hd, D[u], -D[u]) + (gkk - Q[u]), Q[u]);
                if constexpr (k + 1 < kSub)
                    L[u][k + 1] = fma(hd, gk1 - L[u][k + 1], L[u][k + 1]);
                Lz[u] = fma(hd, gkz - Lz[u], Lz[u]);
                hp[u] = hd;
            }
            return true;
        });
        if (GRID && !ok) return false;
        if (!GRID && __ballot(waits && looks < 0) != 0) {
            give_up(a);
            return false;
        }
        if (blockIdx.x == 0 && wave == 0 && a.bmu_trace && !bad && lane < kSub &&
            kSub * sub + lane < nst)
            a.bmu_trace[s0 + kSub * sub + lane] = trace;

        // ---- the 16 steps' coefficients: after them v = beta v + sum gamma e
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int lu = mine + u;
            double suffix = 1.0;
            float gm[kSub];
#pragma unroll
            for (int k = kSub - 1; k >= 0; --k) {
                const double hd = (double)hs[u][k];
                gm[k] = (float)(hd * suffix);
                suffix = fma(-hd, suffix, suffix);
            }
            const float beta = (float)suffix;
            bsub[u] *= (double)beta;
            if (sub + 1 < M / 16 && lu < rows) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    *reinterpret_cast<f4 *>(cg + (sub * rows + lu) * kSub + 4 * v) =
                        f4{gm[4 * v], gm[4 * v + 1], gm[4 * v + 2], gm[4 * v + 3]};
                cb[sub * rows + lu] = beta;
            }
            if (base + lu < a.N) {
                const int64_t to = (int64_t)sub * p.npad + base + lu;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    reinterpret_cast<f4 *>(p.gam[panel & 1])[to * 4 + v] =
                        f4{gm[4 * v], gm[4 * v + 1], gm[4 * v + 2], gm[4 * v + 3]};
                p.beta[panel & 1][to] = beta;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (base + mine + u < a.N) p.qn[base + mine + u] = fma(-2.0, Lz[u], Q[u]) + zz;
    return true;
}

// ----------------------------------------------------------------- kernels

// Work of a launch beside the control: the sweep of `panel`, then the
// preparation of `nprep` panels from `prep` on, then the distances for the
// centres of the panels from `sel` on.
struct SideWork {
    int64_t panel, prep, sel;
    int nsweep, nprep, nsel, apply, prod;
};
template <int M, int TU, int BW>
__device__ inline void side_task(const PanelArgs &p, const SideWork &w, int t,
                                 unsigned char *smem) {
    float *lds = reinterpret_cast<float *>(smem);
    if (t < w.nsweep) {
        sweep<M, TU, BW>(p, w.panel, t, w.apply, w.prod, smem);
    } else if (threadIdx.x < kPrepThreads) {
        t -= w.nsweep;
        if (t < w.nprep * p.prep)
            prepare_task<M>(p, w.prep + t / p.prep, t % p.prep, lds);
        else
            select_task<M>(p, w.sel + (t - w.nprep * p.prep) / p.gsplit,
                           (t - w.nprep * p.prep) % p.gsplit, lds);
    }
}
// Tasks of a launch.
int side_tasks(const PanelArgs &p, const SideWork &w) {
    return w.nsweep + w.nprep * p.prep + w.nsel * p.gsplit;
}

template <int M, int TU, int BW>
__global__ __launch_bounds__(64 * BW, 2) void panel_side_kernel(PanelArgs p, SideWork w) {
    extern __shared__ __align__(16) unsigned char smem[];
    side_task<M, TU, BW>(p, w, blockIdx.x, smem);
}

template <int M>
__global__ __launch_bounds__(64) void panel_correct_kernel(PanelArgs p, int64_t panel) {
    correct_tile<M>(p, panel, blockIdx.x * 16);
}

// One panel on one control workgroup (workgroup 0), the others beside it.
// With few units the control workgroup corrects their products itself.
template <int M, int U, int NW, int TU>
__global__ __launch_bounds__(64 * NW, 2) void panel_step_kernel(PanelArgs p, SideWork w) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t panel = w.panel;
    if (blockIdx.x > 0) {
        side_task<M, TU, NW>(p, w, (int)blockIdx.x - 1, smem);
        return;
    }
    if (!p.correct) {
        for (int t = threadIdx.x >> 6; t * 16 < p.t.N; t += NW) correct_tile<M>(p, panel, t * 16);
        __syncthreads();
    }
    control_panel<M, U, NW, false>(p, panel, smem);
}

// Barrier number n of the grid's workgroups; false once it, or an exchange,
// was given up.  The wait is bounded as an exchange's.
__device__ inline bool grid_barrier(const PanelArgs &p, unsigned n, unsigned char *lds) {
    int *gone = reinterpret_cast<int *>(lds);
    __syncthreads();
    if (threadIdx.x == 0) {
        const TrainArgs &a = p.t;
        __threadfence();
        __hip_atomic_fetch_add(p.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
        int out = 0;
        while (!arrivals_reached(__hip_atomic_load(p.arrived, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT),
                                 n * gridDim.x)) {
            if (__hip_atomic_load(&a.state->order_bad, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT) != 0)
                out = 1;
            else if (__builtin_amdgcn_s_memrealtime() - t0 > a.timeout_ticks)
                out = 2;
            if (out) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (out == 2) give_up(a);
        __threadfence();
        *gone = out;
    }
    __syncthreads();
    const int out = *gone;
    __syncthreads();
    return out == 0;
}

// The grid kernel's roles are functions of their own, so that each is given
// registers as if it were a kernel: inlined into one loop over the panels they
// spill (160 scalar and 160 vector registers).  They are handed the kernel's
// argument segment and the LDS offset as integers, which become uniform
// addresses the compiler can see to be constant memory and LDS.
typedef const __attribute__((address_space(4))) PanelArgs *ArgSegment;
__device__ inline const PanelArgs &segment_args(uint64_t at) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)at);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(at >> 32));
    return *(const PanelArgs *)(ArgSegment)(((uint64_t)hi << 32) | lo);
}
typedef __attribute__((address_space(3))) unsigned char *LdsBytes;
__device__ inline unsigned char *lds_at(uint32_t offset) {
    const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)offset);
    return (unsigned char *)(LdsBytes)(uintptr_t)at;
}
__device__ inline int64_t uniform64(int64_t v) {
    const int lo = __builtin_amdgcn_readfirstlane((int)(unsigned)v);
    const int hi = __builtin_amdgcn_readfirstlane((int)(unsigned)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)(unsigned)hi << 32) | (unsigned)lo);
}

template <int M, int TU, bool APPLY, bool PROD>
__device__ __attribute__((noinline)) void grid_sweep(uint64_t args, uint32_t lds,
                                                     int64_t panel, int t) {
    const PanelArgs &p = segment_args(args);
    t = __builtin_amdgcn_readfirstlane(t);
    const int ugrp = t / p.ksplit;
    sweep_task<M, TU, 4, APPLY, PROD>(p, uniform64(panel), ugrp, t - ugrp * p.ksplit,
                                      lds_at(lds));
}
template <int M>
__device__ __attribute__((noinline)) void grid_prepare(uint64_t args, uint32_t lds,
                                                     int64_t panel, int t) {
    const PanelArgs &p = segment_args(args);
    prepare_task<M>(p, uniform64(panel), __builtin_amdgcn_readfirstlane(t),
                    reinterpret_cast<float *>(lds_at(lds)));
}
template <int M>
__device__ __attribute__((noinline)) void grid_select(uint64_t args, uint32_t lds, int64_t panel,
                                                    int part) {
    const PanelArgs &p = segment_args(args);
    select_task<M>(p, uniform64(panel), __builtin_amdgcn_readfirstlane(part),
                   reinterpret_cast<float *>(lds_at(lds)));
}
template <int M, int U>
__device__ __attribute__((noinline)) void grid_correct(uint64_t args, int64_t panel) {
    const PanelArgs &p = segment_args(args);
    for (int t = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); t < 4 * U; t += 4) {
        const int u0 = (int)blockIdx.x * 64 * U + 16 * t;
        if (u0 < p.t.N) correct_tile<M>(p, uniform64(panel), u0);
    }
}
template <int M, int U>
__device__ __attribute__((noinline)) bool grid_control(uint64_t args, uint32_t lds,
                                                       int64_t panel) {
    return control_panel<M, U, 1, true>(segment_args(args), uniform64(panel), lds_at(lds));
}

// The whole call on a co-resident grid: workgroups 0 .. controllers - 1 run the
// panels' steps, the others everything beside them, and all meet after each
// panel.
template <int M, int U, int TU>
__global__ __launch_bounds__(256, 2) void panel_grid_kernel(PanelArgs p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LdsBytes)smem;
    const TrainArgs &a = p.t;
    if (a.state->order_bad) return;  // unusable input: the same for every workgroup
    const uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    const int C = p.controllers, b = blockIdx.x, others = (int)gridDim.x - C;
    if (b < C && b >= C - p.absent) return;
    const int64_t panels = (a.nsteps + M - 1) / M;
    const int nsweep = (a.N + 16 * TU - 1) / (16 * TU) * p.ksplit;
    unsigned n = 0;
    for (int t = b; t < (panels < 4 ? (int)panels : 4) * p.gsplit; t += gridDim.x) {
        grid_select<M>(args, lds, t / p.gsplit, t % p.gsplit);
        __syncthreads();
    }
    if (!grid_barrier(p, ++n, smem)) return;
    for (int t = b; t < 2 * p.prep; t += gridDim.x) {
        grid_prepare<M>(args, lds, t / p.prep, t % p.prep);
        __syncthreads();
    }
    if (!grid_barrier(p, ++n, smem)) return;
    for (int t = b; t < nsweep; t += gridDim.x) grid_sweep<M, TU, false, true>(args, lds, -1, t);
    if (!grid_barrier(p, ++n, smem)) return;
    for (int64_t k = 0; k < panels; ++k) {
        if (b < C) {
            grid_correct<M, U>(args, k);
            __syncthreads();
            if (threadIdx.x < 64 && !grid_control<M, U>(args, lds, k) && threadIdx.x == 0)
                __hip_atomic_store(&a.state->order_bad, 2, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        } else {
            const bool prod = k + 1 < panels;
            const int ns = k > 0 || prod ? nsweep : 0, np = k + 2 < panels ? p.prep : 0;
            const int nc = k + 4 < panels ? p.gsplit : 0;
            for (int t = b - C; t < ns + np + nc; t += others) {
                if (t >= ns + np)
                    grid_select<M>(args, lds, k + 4, t - ns - np);
                else if (t >= ns)
                    grid_prepare<M>(args, lds, k + 2, t - ns);
                else if (k == 0)
                    grid_sweep<M, TU, false, true>(args, lds, k, t);
                else if (prod)
                    grid_sweep<M, TU, true, true>(args, lds, k, t);
                else
                    grid_sweep<M, TU, true, false>(args, lds, k, t);
                __syncthreads();
            }
        }
        if (!grid_barrier(p, ++n, smem)) return;
    }
    for (int t = b; t < nsweep; t += gridDim.x) grid_sweep<M, TU, true, false>(args, lds, panels, t);
}

__global__ void panel_zero_kernel(unsigned *arrived) { *arrived = 0; }

// ------------------------------------------------------------------- host

struct PanelInstance {
    int m, u, nw, tu;
    bool grid;
    size_t (*lds)(int rows);
    void (*step)(PanelArgs, SideWork);
    void (*side)(PanelArgs, SideWork);
    void (*correct)(PanelArgs, int64_t);
    void (*whole)(PanelArgs);
};

template <int M, int U, int NW, int TU, bool GRID>
size_t panel_lds(int rows) {
    return std::max({ControlLds<M, U, NW>::bytes(rows), kPrepareLds,
                     sweep_lds<M, TU, GRID ? 4 : NW>()});
}
template <int M, int U, int NW, int TU>
constexpr PanelInstance one_workgroup() {
    return PanelInstance{M, U, NW, TU, false, panel_lds<M, U, NW, TU, false>,
                         panel_step_kernel<M, U, NW, TU>, panel_side_kernel<M, TU, NW>,
                         panel_correct_kernel<M>, nullptr};
}
template <int M, int U, int TU>
constexpr PanelInstance exchanging() {
    return PanelInstance{M, U, 1, TU, true, panel_lds<M, U, 1, TU, true>, nullptr, nullptr,
                         nullptr, panel_grid_kernel<M, U, TU>};
}

const PanelInstance kPanels[] = {
    one_workgroup<80, 1, 4, 1>(), one_workgroup<64, 1, 8, 1>(), one_workgroup<48, 2, 8, 2>(),
    one_workgroup<32, 2, 8, 2>(), exchanging<80, 1, 2>(),
};

// Up to this many units the control workgroup corrects the products itself;
// beyond, a launch of its own spreads them over the chip.
constexpr int kSelfCorrect = 256;

}  // namespace

bool plan_train_panel(int32_t N, int32_t d, int num_cus, int max_lds, PanelPlan *plan) {
    const int64_t dpad = ((int64_t)d + kGatherDims - 1) / kGatherDims * kGatherDims;
    for (int k = 0; k < (int)(sizeof(kPanels) / sizeof(kPanels[0])); ++k) {
        const PanelInstance &in = kPanels[k];
        const int per_wg = in.u * in.nw * 64;
        if (!in.grid && N > per_wg) continue;
        const int wgs = (N + per_wg - 1) / per_wg;
        if (in.grid && wgs > num_cus) continue;
        const int rows = ((in.grid ? per_wg : N) + 15) / 16 * 16;
        const size_t lds = in.lds(rows);
        if (lds > (size_t)max_lds) continue;
        const int nt = in.m / 16;
        const int gsplit = (int)std::min<int64_t>(std::max<int64_t>(dpad / 1024, 1), 8);
        plan->prep = (nt * (nt + 1) / 2 + nt * nt) * gsplit + (int)(dpad / kGatherDims);
        plan->gsplit = gsplit;
        // column ranges until two workgroups per CU sweep, each with at least
        // one group of 32 columns per wave
        const int64_t ug = (N + 16 * in.tu - 1) / (16 * in.tu);
        const int waves = in.grid ? 4 : in.nw;
        int64_t ks = 2 * num_cus * 4 / waves / ug;
        ks = std::min<int64_t>(ks, dpad / kSweepDims / waves);
        plan->ksplit = (int32_t)std::max<int64_t>(std::min<int64_t>(ks, kMaxKSplit), 1);
        if (in.grid) {
            // every workgroup co-resident
            int per_cu = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                    &per_cu, reinterpret_cast<const void *>(in.whole), 256, lds) != hipSuccess)
                return false;
            const int64_t most = (int64_t)std::min(per_cu, 2) * num_cus;
            if (wgs + 32 > most) continue;
            plan->grid = (int32_t)std::min<int64_t>(most, wgs + ug * plan->ksplit + plan->prep + plan->gsplit);
        }
        plan->instance = k;
        plan->m = in.m;
        plan->lane_units = in.u;
        plan->controllers = wgs;
        plan->ctl_rows = rows;
        plan->lds = (int32_t)lds;
        plan->dpad = (int32_t)dpad;
        plan->npad = (int32_t)(((int64_t)wgs * per_wg + 31) / 32 * 32);
        return true;
    }
    return false;
}

// The pipelined kernel with its rows in LDS pays the grid exchange a step and
// little else while a workgroup has few rows; one workgroup's panels cost more
// a step with every 256 units, and the panels of larger maps pay an exchange too.
// Measured, microseconds per step of that kernel and of panels: 625 units of
// 1024 floats 1.34 and 1.27, 676 of 64 1.27 and 1.27, 784 of 64 1.27 and 1.33,
// 1024 of 2048 1.41 and 1.59; 2500 of 1024 1.46 and 2.24; 2500 of 3072 (the
// longest rows of its instances for short samples) 2.07 and 2.58, 1024 of 4608
// 2.30 and 1.64; up to 512 floats 40 rows a workgroup (10000 of 512) 2.33 and
// 2.46, 46 rows (11664 of 512) 2.66 and 2.48; longer rows 25 a workgroup (6400
// of 1024) 2.29 and 2.55, 32 rows (8100 of 1024) 2.85 and 2.57.  The streamed
// pipelined kernel loses at every size measured: 4900 of 1536 3.04 and 2.56.
// Short calls pay for the panels' preparation, the first pass and the last.
// Microseconds per call: 10000 units of 2048, 80 steps 422 and 445, 160 steps
// 761 and 674; 2500 of 5000, 80 steps 383 and 384; 900 of 5000, 20 steps 90 and
// 97, 40 steps 132 and 119; 400 of 2000, 2 steps 49 and 51, 5 steps 54 and 50;
// 100 of 500, 1 step 45 and 38.
//
// The blocked kernel (maps of more than 64 units a workgroup, and beyond 2,560
// units rows of more than 3,072 floats) always stays: its distances are direct
// differences x - w, which keep more digits where many units lie close together.
// Relative root mean square error of the smallest distance over 20,000 uniform
// prototypes, that kernel and panels (emulated in fp32): d = 3 3e-8 and 2e-4, d = 8
// 5e-8 and 3e-6, d = 64 1e-7 and 4e-7.
bool persistent_train_first(int32_t N, int32_t d, int64_t nsteps, const TrainPlan &plan) {
    if (plan.variant < 2) return true;
    if (nsteps < (N > 1024 ? 96 : d > 2048 ? 40 : d > 1024 ? 4 : 1)) return true;
    constexpr int kOneWorkgroup = 700, kRowLength = 3072;
    const int rows = d <= 512 ? 40 : 28;
    return plan.variant == 3 && N > kOneWorkgroup && d <= kRowLength &&
           (N + plan.grid - 1) / plan.grid <= rows;
}

int64_t panel_floats(const PanelPlan &pl, PanelArgs *p, float *base) {
    PanelArgs none{};
    PanelArgs &a = p ? *p : none;
    int64_t off = 0;
    const auto take = [&](auto **at, int64_t count) {
        *at = p ? reinterpret_cast<std::remove_reference_t<decltype(**at)> *>(base + off) : nullptr;
        off += (count * (int64_t)(sizeof(**at) / sizeof(float)) + 63) & ~(int64_t)63;
    };
    const int64_t gram = (int64_t)pl.gsplit * (pl.m * pl.m + 16);
    for (int k = 0; k < 2; ++k) {
        take(&a.ec[k], (int64_t)(pl.m + 1) * pl.dpad);
        take(&a.prod[k], (int64_t)pl.ksplit * pl.npad * pl.m);
        take(&a.qf[k], (int64_t)pl.ksplit * pl.npad);
        take(&a.gam[k], (int64_t)pl.m * pl.npad);
        take(&a.beta[k], (int64_t)(pl.m / 16) * pl.npad);
    }
    for (int k = 0; k < 3; ++k) {
        take(&a.gm[k], gram);
        take(&a.gx[k], gram);
    }
    for (int k = 0; k < 4; ++k) {
        take(&a.xt[k], (int64_t)pl.dpad * pl.m);
        take(&a.near[k], (int64_t)pl.gsplit * kPairStride);
    }
    take(&a.pc, (int64_t)pl.npad * pl.m);
    take(&a.qc, (int64_t)pl.npad);
    take(&a.qn, (int64_t)pl.npad);
    take(&a.qe, (int64_t)pl.npad);
    take(&a.pz, (int64_t)pl.npad);
    take(&a.centre, (int64_t)64);
    take(&a.arrived, (int64_t)64);
    return off;
}

hipError_t launch_train_panel(const PanelArgs &args, const PanelPlan &pl, hipStream_t s) {
    const PanelInstance &in = kPanels[pl.instance];
    PanelArgs p = args;
    p.dpad = pl.dpad;
    p.npad = pl.npad;
    p.ksplit = pl.ksplit;
    p.gsplit = pl.gsplit;
    p.prep = pl.prep;
    p.controllers = pl.controllers;
    p.ctl_rows = pl.ctl_rows;
    p.t.grid = pl.controllers;
    if (p.dpad > p.t.ld || p.absent < 0 || p.absent > 1 ||
        (p.absent && pl.controllers < 2 && p.t.N <= 64 * in.u) || p.t.nsteps < 1)
        return hipErrorInvalidValue;
    // a look takes 60-100 ns, 6-10 ticks
    p.max_looks = (int32_t)std::min<uint64_t>(p.t.timeout_ticks / 6, INT32_MAX);
    hipError_t e;
    if (in.grid) {
        panel_zero_kernel<<<1, 1, 0, s>>>(p.arrived);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        void *params[] = {&p};
        return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(in.whole), dim3(pl.grid),
                                          dim3(256), params, (unsigned)pl.lds, s);
    }
    const int64_t panels = (p.t.nsteps + pl.m - 1) / pl.m;
    const int nsweep = (p.t.N + 16 * in.tu - 1) / (16 * in.tu) * pl.ksplit;
    const dim3 block(64 * in.nw);
    const size_t side_lds = in.lds(0);
    p.correct = p.t.N > kSelfCorrect;
    const auto side = [&](const SideWork &w) {
        in.side<<<dim3(side_tasks(p, w)), block, side_lds, s>>>(p, w);
    };
    SideWork w{};
    w.nsel = (int)std::min<int64_t>(panels, 4);
    side(w);
    w = SideWork{};
    w.nprep = 2;
    side(w);
    w = SideWork{};
    w.panel = -1;
    w.nsweep = nsweep;
    w.prod = 1;
    side(w);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int64_t b = 0; b < panels; ++b) {
        w.panel = b;
        w.prep = b + 2;
        w.sel = b + 4;
        w.apply = b > 0;
        w.prod = b + 1 < panels;
        w.nsweep = w.apply || w.prod ? nsweep : 0;
        w.nprep = b + 2 < panels;
        w.nsel = b + 4 < panels;
        if (p.correct) in.correct<<<dim3((p.t.N + 15) / 16), dim3(64), 0, s>>>(p, b);
        in.step<<<dim3(1 + side_tasks(p, w)), block, pl.lds, s>>>(p, w);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    w = SideWork{};
    w.panel = panels;
    w.nsweep = nsweep;
    w.apply = 1;
    side(w);
    return hipGetLastError();
}

}  // namespace som
