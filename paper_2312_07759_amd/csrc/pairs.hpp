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
// between workgroups elsewhere.  s_A: N x N doubles of LDS of this wavefront.
struct AveragedResult {
    int iters, converged, bad, halvings;
    double alpha, step2;
};

// Up to four unknowns: 64 steps at a time.  A step is delta_n = A^n delta_0 with A = alpha (dF/dC)^T + (1 - alpha) I, so lane j
// forms delta_{n+j} from delta_n by the powers A, A^2, A^4, ... its index asks for; the stop rule is evaluated for all of them at
// once, and g moves by the sum of the steps up to the one that ends the attempt.  One step after the other is a chain of
// about 350 cycles, 9.6 us for 64 of them; this way 64 take 2 us (2.4 M weights, k = 4, 104 steps: launch 47 -> 28 us).
template <int N, bool F32>
__device__ __forceinline__ AveragedResult averaged_iteration_wide(const double (&row)[N], double v, double alpha, double stop2,
                                                                  int max_iter, double* s_A, double& g) {
    static_assert(N <= 4, "every lane keeps a power of A");
    AveragedResult o = {0, 0, 0, 0, alpha, 0.0};
    const int lane = threadIdx.x & 63;
    double x[N];
    for (bool again = true; again;) {
        again = false;
        double dl[N];  // delta_n, the same in every lane
        const double d0 = o.alpha * pair_apply<N>(row, v);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            x[i] = lane_value_d(v, i);
            dl[i] = lane_value_d(d0, i);
        }
        if (lane < N) {
#pragma unroll
            for (int c = 0; c < N; ++c) s_A[lane * N + c] = o.alpha * row[c] + (lane == c ? 1.0 - o.alpha : 0.0);
        }
        double prev = __builtin_inf();
        int grow = 0, left = max_iter;
        for (;;) {
            double P[N][N], d[N];
            wave_lds_sync();  // (and A is read again, not held in registers across the loop)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                d[i] = dl[i];
#pragma unroll
                for (int c = 0; c < N; ++c) P[i][c] = s_A[i * N + c];
            }
#pragma nounroll
            for (int bit = 0; bit < 6; ++bit) {
                const bool on = (lane >> bit) & 1;
                double t[N], Q[N][N];
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    t[i] = P[i][0] * d[0];
#pragma unroll
                    for (int c = 1; c < N; ++c) t[i] = fma(P[i][c], d[c], t[i]);
#pragma unroll
                    for (int c = 0; c < N; ++c) {
                        Q[i][c] = P[i][0] * P[0][c];
#pragma unroll
                        for (int e = 1; e < N; ++e) Q[i][c] = fma(P[i][e], P[e][c], Q[i][c]);
                    }
                }
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    d[i] = on ? t[i] : d[i];
#pragma unroll
                    for (int c = 0; c < N; ++c) P[i][c] = Q[i][c];
                }
            }
            double d2 = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) d2 = fma(d[i], d[i], d2);
            if (F32) d2 = (double)(float)d2;
            const double before = __shfl_up(d2, 1, 64);
            const bool finite = d2 <= 1.7e308, conv = finite && d2 <= stop2;
            const bool up = finite && !conv && d2 > (lane == 0 ? prev : before);
            const unsigned long long mc = __builtin_amdgcn_ballot_w64(conv), mu = __builtin_amdgcn_ballot_w64(up);
            unsigned long long run = mu;  // steps that end five growing ones in a row; `grow` of them lie before lane 0
#pragma unroll
            for (int s = 1; s < 5; ++s) {
                const int old = grow < s ? grow : s;
                run &= (mu << s) | (((1ull << old) - 1ull) << (s - old));
            }
            const unsigned long long md = run | __builtin_amdgcn_ballot_w64(!finite);
            const unsigned long long ml = left <= 64 ? 1ull << (left - 1) : 0ull;
            const unsigned long long any = mc | md | ml;
            const int e = any ? (int)__builtin_ctzll(any) : 63;  // the last step taken
            o.iters += e + 1;
            o.step2 = lane_value_d(d2, e);
            const bool diverged = (md >> e) & 1ull & (any != 0);
            if (diverged && o.halvings < 6) {
                o.alpha *= 0.5;
                o.halvings += 1;
                again = true;
                break;
            }
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] += wave_sum_d_dpp(lane <= e ? d[i] : 0.0);
            if (any) {
                o.converged = (mc >> e) & 1ull ? 1 : 0;
                if (diverged && !(o.step2 <= 1.7e308)) o.bad = 1;  // every damping factor tried ended in a non-finite step
                break;
            }
            left -= 64;
            prev = o.step2;
            grow = (int)__builtin_clzll(~mu);
            wave_lds_sync();
#pragma unroll
            for (int i = 0; i < N; ++i) {
                double t = 0.0;
#pragma unroll
                for (int c = 0; c < N; ++c) t = fma(s_A[i * N + c], lane_value_d(d[c], 63), t);
                dl[i] = t;
            }
        }
    }
    g = x[0];
#pragma unroll
    for (int i = 1; i < N; ++i) g = (lane == i) ? x[i] : g;
    return o;
}

template <int N, bool F32>
__device__ __forceinline__ AveragedResult averaged_iteration(const double (&row)[N], double v, double alpha, double stop2, int max_iter,
                                                             double* s_A, double& g) {
    if constexpr (N <= 4) return averaged_iteration_wide<N, F32>(row, v, alpha, stop2, max_iter, s_A, g);
    AveragedResult o = {0, 0, 0, 0, alpha, 0.0};
    const int lane = threadIdx.x & 63;
    double M[N], b = 0.0, x = v, prev = __builtin_inf();
    int attempt = 0, grow = 0;
    bool start = true;
    for (;;) {
        if (start) {
            start = false;
            x = v;
            b = o.alpha * v;
#pragma unroll
            for (int c = 0; c < N; ++c) M[c] = o.alpha * row[c] + (lane == c ? 1.0 - o.alpha : 0.0);
        }
        const double xn = b + pair_apply<N>(M, x);
        const double df = lane < N ? xn - x : 0.0;
        double d2 = lane_value_d(first_lanes_sum_d_dpp<N>(df * df), 0);
        if (F32) d2 = (double)(float)d2;
        o.iters += 1;
        attempt += 1;
        o.step2 = d2;
        const bool finite = d2 <= 1.7e308;
        bool diverged = !finite;
        if (finite && d2 <= stop2) {
            o.converged = 1;
            x = xn;
            break;
        }
        if (finite) {
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
        x = xn;
        if (diverged) {
            if (!finite) o.bad = 1;  // every damping factor tried ended in a non-finite step
            break;
        }
        if (attempt >= max_iter) break;
    }
    g = x;
    return o;
}

}  // namespace idkm
