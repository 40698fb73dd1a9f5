// (dF/dC*)^T as an explicit k d x k d matrix, for codebooks small enough that one pass over W can form it.
//
// The codebook does not change during the backward solve, so the operator that the averaged iteration (Sec. 4.2) and the
// Krylov solve apply again and again is one fixed matrix.  With pi_i = a_ij a_il, beta_ij = h_j . (w_i - F_j) and
// delta_ij = d e_ij / d w_i,
//     ((dF/dC)^T g)_j = (1/tau) sum_i a_ij (beta_ij - sum_l a_il beta_il) delta_ij
//                     = (1/tau) sum_l sum_i pi_i (beta_ij - beta_il) delta_ij
// (the rows of A sum to one), so a pair of codewords contributes a few moments of its weight pi, taken about the midpoint of
// the pair, where pi lies: u = w - (c_j + c_l)/2,
//     squared energy  sum pi, sum pi u, sum pi u u^T     (1 + d + d(d+1)/2 sums, both directions of the pair)
//     plain norm      sum pi delta_j, sum pi delta_j u^T, the same with delta_l     (2 (d + d^2) sums)
// beta_j - beta_l = (h_j - h_l) . u + h_j . (mid - F_j) - h_l . (mid - F_l).  Nothing large cancels: a difference of the
// diagonal sum_i a_ij (..) and its square would lose what hard rows leave of it.
//
// The pass that forms them (PASS_BP) also forms v, so a solve of any length reads W twice (this pass and the last) and
// crosses the grid once.  What it costs against the (dF/dC)^T pass it replaces is said at pair_solve_pays().
#pragma once
#include "common.hpp"

namespace idkm {

constexpr int PAIR_WORDS_MAX = 128;  // sums of a pass that fit a workgroup's exchange line
__host__ __device__ constexpr int pair_moments(int D, int dist) { return dist == DIST_SQL2 ? 1 + D + D * (D + 1) / 2 : 2 * (D + D * D); }
// sums of PASS_BP: v, then the moments of the pairs (0,1), (0,2), ..., (1,2), ...
__host__ __device__ constexpr int pair_sums(int K, int D, int dist) { return K * D + K * (K - 1) / 2 * pair_moments(D, dist); }
__host__ __device__ constexpr bool pair_shape(int K, int D, int dist) { return pair_sums(K, D, dist) <= PAIR_WORDS_MAX; }
// Whether forming the operator beats applying it pass by pass.  Whole backward calls with 1 / 2 / 3 / 10 passes allowed, us, pass
// by pass and on the matrix: k = 4, d = 1 at 300,000 weights 29.8 / 32.7 / 36.2 / 56.9 and 29.0 from 2 on, at 2.4 M 43.1 /
// 49.0 / 54.3 / 96.4 and 40 to 41; k = 4, d = 4 at 300,000 vectors 33.2 / 37.0 / 41.4 / 68.7 and 36 to 38; k = 8, d = 1 at 300,000
// 30.9 / 34.3 / 37.8 / 62.1 and 33 to 36, k = 7 (padded to 8) 30.9 / 34.7 / 38.4 / 63.7 and 36 to 38.
// 2.4 M weights, k = 4, 83 steps: 797 -> 222 us for the forward solve and this backward.
__host__ __device__ constexpr bool pair_solve_pays(int K, int D, int max_iter) { return (K <= 4 && D == 1) || max_iter >= 3; }

__device__ __forceinline__ double lane_value_d(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Row of the matrix, in terms of g, that belongs to lane j d + r < k d: ((dF/dC)^T g)_jr = sum_c row[c] g_c.
// tot(i): total i of PASS_BP; c, F, rn: codebook, F(C*, W) and 1/(tau n).  Lanes from k d on return zeros.
template <int K, int D, int DIST, class T>
__device__ __forceinline__ void pair_row(T tot, const float* c, const double* F, const double* rn, float escale, double (&row)[K * D]) {
    constexpr int NM = pair_moments(D, DIST);
    const int lane = threadIdx.x & 63;
    const bool live = lane < K * D;
    const int j = live ? lane / D : 0, r = live ? lane % D : 0;
    // u is accumulated as the sum of the two differences (scalar weights: of the scaled ones, see estep_small)
    const double f = (D == 1) ? 0.5 / (double)escale : 0.5;
    double self[D];
#pragma unroll
    for (int s = 0; s < D; ++s) self[s] = 0.0;
#pragma unroll
    for (int l = 0; l < K; ++l) {
        const bool other = live && l != j;
        const int lo = l < j ? l : j, hi = l < j ? j : l;
        const int p = lo * K - lo * (lo + 1) / 2 + (hi - lo - 1);
        const int q = other ? K * D + p * NM : 0;
        double s0, s1[D];  // sum pi delta_jr and sum pi delta_jr u_s
        if constexpr (DIST == DIST_SQL2) {
            const double e = 0.5 * ((double)c[l * D + r] - (double)c[j * D + r]);  // mid - c_j
            s0 = 2.0 * (f * tot(q + 1 + r) + e * tot(q));
#pragma unroll
            for (int s = 0; s < D; ++s) {
                const int a = r < s ? r : s, b = r < s ? s : r;
                s1[s] = 2.0 * (f * f * tot(q + 1 + D + a * D - a * (a - 1) / 2 + (b - a)) + e * f * tot(q + 1 + s));
            }
        } else {
            const int side = q + (other && j > l ? D + D * D : 0);
            s0 = tot(side + r);
#pragma unroll
            for (int s = 0; s < D; ++s) s1[s] = f * tot(side + D + r * D + s);
        }
#pragma unroll
        for (int s = 0; s < D; ++s) {
            const double mid = 0.5 * ((double)c[l * D + s] + (double)c[j * D + s]);
            self[s] += other ? s1[s] + (mid - F[j * D + s]) * s0 : 0.0;
            row[l * D + s] = other ? -(s1[s] + (mid - F[l * D + s]) * s0) * rn[l] : 0.0;
        }
    }
#pragma unroll
    for (int l = 0; l < K; ++l)
#pragma unroll
        for (int s = 0; s < D; ++s)
            if (live && l == j) row[l * D + s] = self[s] * rn[j];
}

template <int N>
__device__ __forceinline__ double pair_apply(const double (&row)[N], double g) {
    double u[2] = {0.0, 0.0};
#pragma unroll
    for (int c = 0; c < N; ++c) u[c & 1] = fma(row[c], lane_value_d(g, c), u[c & 1]);
    return u[0] + u[1];
}

// The averaged iteration of Sec. 4.2 on that matrix, in one wavefront: g+ = alpha (v + (dF/dC)^T g) + (1 - alpha) g from g = v
// until ||g+ - g||^2 <= stop2, at most max_iter steps an attempt; a non-finite step or five growing ones in a row start over
// with half the step, at most six times -- the steps, counters and stop rule of the passes it replaces.  v, g: lane c < N owns
// component c (v is zero in the others).  F32: the squared step norm is rounded to float32, like the word that carries it
// between workgroups elsewhere.
struct AveragedResult {
    int iters, converged, bad, halvings;
    double alpha, step2;
};
template <int N, bool F32>
__device__ __forceinline__ AveragedResult averaged_iteration(const double (&row)[N], double v, double alpha, double stop2, int max_iter,
                                                             double& g) {
    AveragedResult o = {0, 0, 0, 0, alpha, 0.0};
    const int lane = threadIdx.x & 63;
    // up to four unknowns every lane keeps all of them: no value crosses lanes in the chain of a step (104 steps at k = 4)
    constexpr bool ALL = N <= 4;
    constexpr int NV = ALL ? N : 1, NR = ALL ? N : 1;
    double M[NR][N], b[NV], x[NV], v0[NV], J[NR][N];
    if constexpr (ALL) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            v0[i] = lane_value_d(v, i);
#pragma unroll
            for (int c = 0; c < N; ++c) J[i][c] = lane_value_d(row[c], i);
        }
    } else {
        v0[0] = v;
#pragma unroll
        for (int c = 0; c < N; ++c) J[0][c] = row[c];
    }
    int attempt = 0, grow = 0;
    double prev = __builtin_inf();
    bool start = true;
    for (;;) {
        if (start) {
            start = false;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                x[i] = v0[i];
                b[i] = o.alpha * v0[i];
#pragma unroll
                for (int c = 0; c < N; ++c) M[i][c] = o.alpha * J[i][c] + ((ALL ? i : lane) == c ? 1.0 - o.alpha : 0.0);
            }
        }
        double xn[NV], d2 = 0.0;
        if constexpr (ALL) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                xn[i] = b[i];
#pragma unroll
                for (int c = 0; c < N; ++c) xn[i] = fma(M[i][c], x[c], xn[i]);
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const double df = xn[i] - x[i];
                d2 = fma(df, df, d2);
            }
        } else {
            xn[0] = b[0] + pair_apply<N>(M[0], x[0]);
            const double df = lane < N ? xn[0] - x[0] : 0.0;
            d2 = first_lanes_sum_d_dpp<N>(df * df);
            d2 = lane_value_d(d2, 0);
        }
        if (F32) d2 = (double)(float)d2;
        o.iters += 1;
        attempt += 1;
        o.step2 = d2;
        bool diverged = !(d2 <= 1.7e308);
        if (!diverged) {
            if (d2 <= stop2) {
                o.converged = 1;
#pragma unroll
                for (int i = 0; i < NV; ++i) x[i] = xn[i];
                break;
            }
            grow = (d2 > prev) ? grow + 1 : 0;
            prev = d2;
            diverged = grow >= 5;
        }
        if (diverged && o.halvings < 6) {
            o.alpha *= 0.5;
            o.halvings += 1;
            attempt = 0;
            grow = 0;
            prev = __builtin_inf();
            start = true;
            continue;
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) x[i] = xn[i];
        if (diverged) {
            if (!(d2 <= 1.7e308)) o.bad = 1;  // every damping factor tried ended in a non-finite step
            break;
        }
        if (attempt >= max_iter) break;
    }
    if constexpr (ALL) {
        g = x[0];
#pragma unroll
        for (int i = 1; i < N; ++i) g = (lane == i) ? x[i] : g;
    } else {
        g = x[0];
    }
    return o;
}

}  // namespace idkm
