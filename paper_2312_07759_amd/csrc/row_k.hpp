// Row <-> vector kernels for codebooks of up to 256 codewords with d = 1, 2 and 8: a row of 16 lanes works on V vectors at
// a time, lane l of the row owning codewords l, l + 16, ...  (KB of them).  The softmax sums of a vector run over a lane's
// registers and then over the 16 lanes (four DPP additions for each of the V vectors, their chains side by side), and the
// M-step sums stay in the lane's registers until the end of the pass, where the four rows of a wavefront are added.
//
// Bound by issue on the vector ALU.  The lane <-> codeword form it replaces on these shapes (one vector per wavefront and
// step) pays a broadcast of the vector and a dependent six-step wavefront sum per vector whatever k is: at k = 64, d = 1
// about 20 issue slots per (vector, 64 codewords) against 7 slots per pair here plus about 112 / k for the row sums.
// 589,824 weights, k = 64, d = 1, 30 evaluations and a Jacobian-free backward: 1260 -> 671 us by this form alone, 550 with the
// exchange and the issue priority it has now (71 % of the issue slots of the launch taken; 10.1 slots per pair, row sums and
// exchange included); 4 vectors per row and step where they fit the registers.
// Vectors are read from the workgroup's LDS tile (all lanes of a row read the same address).
#pragma once
#include "common.hpp"
#include "lane_k.hpp"
#include "mfma_lane.hpp"

namespace idkm {

// Values per lane that a step may keep live (256 registers at two wavefronts per SIMD; at 160 the forward loop at k = 256,
// d = 2 spilled 46 registers).
constexpr int ROW_BUDGET = 150;
// d = 8: the sums alone are 144 at k = 256, and nothing else is kept.  The forward loop fits (226 registers).  The pass for v and
// the (dF/dC)^T pass do not at k = 256, with one vector a step either: the compiler brings operands forward from LDS and
// spills 50 to 137 registers inside the step loop (66 % of the issue slots taken in the pass for v, 179 us at 294,912 vectors).
constexpr int ROW_BUDGET_8 = 226;

template <int KB, int D, int DIST, int PASS>
struct RowWave {
    static constexpr bool STATS = (PASS == PASS_FWD || PASS == PASS_FIN);
    static constexpr bool BACK = (PASS == PASS_B1 || PASS == PASS_B2 || PASS == PASS_B3);
    static constexpr bool USE_G = (PASS == PASS_B1 || PASS == PASS_B3);
    static constexpr bool USE_H = (PASS == PASS_B2 || PASS == PASS_B3);
    static constexpr int ACCW = STATS ? (D + 1) : D;
    static constexpr int NA = (PASS == PASS_B3) ? 1 : KB * ACCW;
    // scaled coordinates t = s (w - c), as in the lane <-> codeword form: the forward loop, and the (dF/dC)^T pass of the
    // squared energy
    static constexpr bool SCALED = (PASS == PASS_FWD) || (PASS == PASS_B2 && DIST == DIST_SQL2);
    // d = 8: the codewords' operands (up to 384 values per lane) are read from LDS in every step instead of kept
    static constexpr bool REGS = D <= 2;
    static constexpr int NSTATE = BACK ? ((DIST == DIST_L2 && D > 1) ? 3 : 2) : 1;  // values per (vector, codeword) pair
    static constexpr int KEPT = NA + (REGS ? KB * D * (USE_H ? 3 : 1) : 2 * D);
    static constexpr int cost(int v) { return KEPT + v * (KB * NSTATE + D * (USE_G ? 3 : 2)); }
    static constexpr int BUDGET = D == 8 ? ROW_BUDGET_8 : ROW_BUDGET;
    static constexpr int V = (D <= 4 && cost(4) <= BUDGET) ? 4 : (cost(2) <= BUDGET ? 2 : 1);  // vectors of a row per step
    static constexpr int STEP = 4 * V;                                                      // vectors of a wavefront per step

    float rc[REGS ? KB : 1][D], rh[(REGS && USE_H) ? KB : 1][D], rf[(REGS && USE_H) ? KB : 1][D];
    const float *tc, *th_, *tf;  // d = 8: tables in LDS, [16 KB][D]
    float acc[NA];
    int k;

    // d = 8, scaled passes: the operands of the codewords in the coordinates of the pass, formed once per pass by the whole
    // workgroup (in every step they cost as much again as the energies): tab[j][.] = s c_j, 1e18 where no codeword is; the
    // (dF/dC)^T pass also h_j / s behind them, then h_j . F_j.  TAB floats of LDS; the caller's barrier follows.
    static constexpr int TAB = (!REGS && SCALED) ? 16 * KB * (USE_H ? 2 * D + 1 : D) : 1;
    template <int NT>
    static __device__ __forceinline__ void fill_table(float* tab, int k, const float* Cf, const float* Hs, const float* Ff, float escale) {
        if constexpr (!REGS && SCALED) {
            const float inv = 1.0f / escale;
            for (int i = threadIdx.x; i < 16 * KB * D; i += NT) {
                tab[i] = i < k * D ? Cf[i] * escale : 1e18f;
                if (USE_H) tab[16 * KB * D + i] = Hs[i] * inv;
            }
            if (USE_H)
                for (int j = threadIdx.x; j < 16 * KB; j += NT) {
                    float hf = 0.f;
#pragma unroll
                    for (int r = 0; r < D; ++r) hf = fmaf(Hs[j * D + r], Ff[j * D + r], hf);
                    tab[32 * KB * D + j] = hf;
                }
        }
    }

    // Cf, Hs, Ff: tables in LDS, [16 KB][D], zero from row k on (16-byte aligned for d = 8); scaled passes at d = 8: Cf is the
    // table above and the others are not read.
    __device__ __forceinline__ void init(int k_, const float* Cf, const float* Hs, const float* Ff, float escale) {
        const int j0 = threadIdx.x & 15;
        k = k_;
        tc = Cf;
        th_ = Hs;
        tf = Ff;
        if constexpr (REGS) {
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                const int j = j0 + 16 * b;
                const bool valid = j < k;
#pragma unroll
                for (int r = 0; r < D; ++r) {
                    // (scaled passes: a codeword that does not exist sits 1e18 away, its weight is exactly zero)
                    rc[b][r] = !SCALED ? Cf[j * D + r] : (valid ? Cf[j * D + r] * escale : 1e18f);
                    if (USE_H) {
                        rh[b][r] = Hs[j * D + r];
                        rf[b][r] = Ff[j * D + r];
                    }
                }
                if (PASS == PASS_B2 && DIST == DIST_SQL2) {
                    // h.(w - F) = (h/s).(s w) - h.F: rf[b][0] = h.F, rh = h/s
                    const float inv = 1.0f / escale;
                    float hf = 0.f;
#pragma unroll
                    for (int r = 0; r < D; ++r) {
                        hf = fmaf(rh[b][r], rf[b][r], hf);
                        rh[b][r] *= inv;
                    }
                    rf[b][0] = hf;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < NA; ++q) acc[q] = 0.f;
    }
    // d = 8: operands read in an earlier phase of a step are read again, not kept (they would spill).
    static __device__ __forceinline__ void next_phase() {
        if (!REGS) asm volatile("" ::: "memory");
    }
    // Operands of codeword j0 + 16 b (in the coordinates of the pass).
    __device__ __forceinline__ void table_row(const float* t, int b, float (&x)[D]) const {
        const int j = (threadIdx.x & 15) + 16 * b;
        const f32x4* p = reinterpret_cast<const f32x4*>(t + j * D);
#pragma unroll
        for (int h = 0; h < D / 4; ++h) {
            const f32x4 v = p[h];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * h + e] = v[e];
        }
    }
    __device__ __forceinline__ void codeword(int b, float escale, float (&c)[D]) const {
        if constexpr (REGS) {
#pragma unroll
            for (int r = 0; r < D; ++r) c[r] = rc[b][r];
        } else {
            table_row(tc, b, c);
        }
    }
    __device__ __forceinline__ void cotangent(int b, float (&h)[D]) const {
        if constexpr (REGS) {
#pragma unroll
            for (int r = 0; r < D; ++r) h[r] = rh[b][r];
        } else {
            table_row(th_, b, h);
        }
    }
    __device__ __forceinline__ void image(int b, float (&f)[D]) const {
        if constexpr (REGS) {
#pragma unroll
            for (int r = 0; r < D; ++r) f[r] = rf[b][r];
        } else {
            table_row(tf, b, f);
        }
    }

    // Vectors v0 .. v0 + STEP - 1 of the tile s_w (dL/dWq: s_g); those at or beyond vend contribute nothing and are not
    // read (FULL: there are none).  base: index of the tile's first vector in the layer.
    template <bool FULL>
    __device__ __forceinline__ void step(const Args& a, const float* s_w, const float* s_g, int64_t base, int v0, int vend) {
        const int j0 = threadIdx.x & 15, vb = v0 + V * ((threadIdx.x & 63) >> 4);
        const float inf = __builtin_inff();
        const float escale = a.escale;
        next_phase();
        float w[V][D], g[V][D], live[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const bool on = FULL || vb + i < vend;
            live[i] = on ? 1.f : 0.f;
            const int v = on ? vb + i : v0;  // (vector v0 exists)
#pragma unroll
            for (int r = 0; r < D; ++r) {
                w[i][r] = s_w[v * D + r];
                if (SCALED) w[i][r] *= escale;
                g[i][r] = USE_G ? s_g[v * D + r] : 0.f;
            }
        }
        if constexpr (SCALED) {
            step_scaled(a, w, live);
            return;
        }
        // general form: energies from differences, rows shifted by their largest exponent
        float p[KB][V], ri[(DIST == DIST_L2 && D > 1 && BACK) ? KB : 1][V], umax[V], S[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            umax[i] = -inf;
            S[i] = 0.f;
        }
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            float c[D];
            codeword(b, escale, c);
            const bool valid = j0 + 16 * b < k;
#pragma unroll
            for (int i = 0; i < V; ++i) {
                float e;
                const float d0 = w[i][0] - c[0];
                if (D == 1) {
                    e = (DIST == DIST_SQL2) ? d0 * d0 : fabsf(d0);
                } else {
                    float e2 = d0 * d0;
#pragma unroll
                    for (int r = 1; r < D; ++r) {
                        const float df = w[i][r] - c[r];
                        e2 = fmaf(df, df, e2);
                    }
                    if (DIST == DIST_SQL2) {
                        e = e2;
                    } else if constexpr (BACK) {
                        const float rs = (e2 > 0.f) ? fast_rsq(e2) : 0.f;
                        ri[b][i] = rs;
                        e = e2 * rs;
                    } else {
                        e = fast_sqrt(e2);
                    }
                }
                p[b][i] = valid ? e * a.nscale : -inf;
                umax[i] = fmaxf(umax[i], p[b][i]);
            }
        }
#pragma unroll
        for (int i = 0; i < V; ++i) umax[i] = row16_max(umax[i]);
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int i = 0; i < V; ++i) {
                p[b][i] = fast_exp2(p[b][i] - umax[i]);
                S[i] += p[b][i];
            }
#pragma unroll
        for (int i = 0; i < V; ++i) S[i] = fast_rcp(row16_sum(S[i])) * live[i];  // 1 / S_i from here on
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int i = 0; i < V; ++i) p[b][i] *= S[i];  // a_ij

        if constexpr (STATS) {
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    acc[b * ACCW] += p[b][i];
#pragma unroll
                    for (int r = 0; r < D; ++r) acc[b * ACCW + 1 + r] = fmaf(p[b][i], w[i][r], acc[b * ACCW + 1 + r]);
                }
        }
        if constexpr (PASS == PASS_FIN) {
            if (a.Wq_out) {
                next_phase();
                float s[V][D];
#pragma unroll
                for (int i = 0; i < V; ++i)
#pragma unroll
                    for (int r = 0; r < D; ++r) s[i][r] = 0.f;
#pragma unroll
                for (int b = 0; b < KB; ++b) {
                    float c[D];
                    codeword(b, escale, c);
#pragma unroll
                    for (int i = 0; i < V; ++i)
#pragma unroll
                        for (int r = 0; r < D; ++r) s[i][r] = fmaf(p[b][i], c[r], s[i][r]);
                }
                store_rows(s, a.Wq_out, base, vb, vend);
            }
            if (a.A_out) {
#pragma unroll
                for (int b = 0; b < KB; ++b)
#pragma unroll
                    for (int i = 0; i < V; ++i)
                        if (j0 + 16 * b < k && vb + i < vend) a.A_out[(base + vb + i) * (int64_t)k + j0 + 16 * b] = p[b][i];
            }
            if (a.assign_out) {
                // closest codeword on a float32 key with separately rounded operations; lowest index on ties
                next_phase();
                float best[V];
                int cand[V];
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    best[i] = inf;
                    cand[i] = 0x7fffffff;
                }
#pragma unroll
                for (int b = 0; b < KB; ++b) {
                    float c[D];
                    codeword(b, escale, c);
                    const bool valid = j0 + 16 * b < k;
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        float df[D];
#pragma unroll
                        for (int r = 0; r < D; ++r) df[r] = w[i][r] - c[r];
                        const float key = D == 1 ? fabsf(df[0]) : sum_sq_unfused<D>(df);
                        if (valid && (key < best[i] || cand[i] == 0x7fffffff)) {
                            best[i] = key;
                            cand[i] = j0 + 16 * b;
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const float kmin = row16_min(best[i]);
                    cand[i] = row16_min_i(best[i] == kmin ? cand[i] : 0x7fffffff);
                }
                int out = cand[0];
#pragma unroll
                for (int i = 1; i < V; ++i) out = (j0 == i) ? cand[i] : out;
                if (j0 < V && vb + j0 < vend) a.assign_out[base + vb + j0] = out;
            }
        }
        if constexpr (BACK) {
            next_phase();
            float q[KB][V], qb[V];
#pragma unroll
            for (int i = 0; i < V; ++i) qb[i] = 0.f;
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                float c[D], h[D], f[D];
                if (USE_G) codeword(b, escale, c);
                if (USE_H) {
                    cotangent(b, h);
                    image(b, f);
                }
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    float s = 0.f;
#pragma unroll
                    for (int r = 0; r < D; ++r) {
                        if (USE_G) s = fmaf(g[i][r] * a.inv_tau, c[r], s);
                        if (USE_H) s = fmaf(h[r], w[i][r] - f[r], s);
                    }
                    q[b][i] = s;
                    qb[i] = fmaf(p[b][i], q[b][i], qb[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < V; ++i) qb[i] = row16_sum(qb[i]);
            next_phase();
            float out[V][D];
#pragma unroll
            for (int i = 0; i < V; ++i)
#pragma unroll
                for (int r = 0; r < D; ++r) out[i][r] = 0.f;
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                float c[D], h[D];
                codeword(b, escale, c);
                if (PASS == PASS_B3) cotangent(b, h);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    // a_ij (q_ij - q_i) times the factor of w - c in d e / d w (2, or 1 / ||w - c||)
                    float th = p[b][i] * (q[b][i] - qb[i]);
                    if (DIST == DIST_SQL2) th *= 2.f;
                    if (DIST == DIST_L2 && D > 1) th *= ri[(DIST == DIST_L2 && D > 1) ? b : 0][i];
                    const float pt = PASS == PASS_B3 ? p[b][i] * a.tau : 0.f;
#pragma unroll
                    for (int r = 0; r < D; ++r) {
                        const float df = w[i][r] - c[r];
                        const float dl = (DIST == DIST_L2 && D == 1) ? ((df > 0.f) ? 1.f : ((df < 0.f) ? -1.f : 0.f)) : df;
                        if (PASS == PASS_B3) {
                            out[i][r] = fmaf(pt, h[r], out[i][r]);
                            out[i][r] = fmaf(-th, dl, out[i][r]);
                        } else {
                            float t = acc[b * ACCW + r];
                            if (PASS == PASS_B1) t = fmaf(p[b][i], g[i][r], t);
                            acc[b * ACCW + r] = fmaf(th, dl, t);
                        }
                    }
                }
            }
            if constexpr (PASS == PASS_B3) store_rows(out, a.dW_out, base, vb, vend);
        }
    }

    // The forward loop, and the (dF/dC)^T pass of the squared energy, in scaled coordinates (w is scaled): exp(-e/tau) =
    // exp2(-|t|^2) resp. exp2(-|t|).  Squared energy: the row is shifted only when the whole row underflows (decided per
    // vector from the unshifted sum; then all vectors of the wavefront's step are redone).
    __device__ __forceinline__ void step_scaled(const Args& a, const float (&w)[V][D], const float (&live)[V]) {
        const float escale = a.escale;
        float p[KB][V], S[V];
#pragma unroll
        for (int i = 0; i < V; ++i) S[i] = 0.f;
        auto energy = [&](const float (&c)[D], int i) {
            float t = w[i][0] - c[0];
            if (DIST == DIST_L2 && D == 1) return fabsf(t);
            float e2 = t * t;
#pragma unroll
            for (int r = 1; r < D; ++r) {
                t = w[i][r] - c[r];
                e2 = fmaf(t, t, e2);
            }
            return DIST == DIST_L2 ? fast_sqrt(e2) : e2;
        };
        // Two wavefronts of a SIMD issue additions and multiply-adds at twice the rate of one, but not next to an exponential: from
        // 16 pairs of a lane on the exponentials of a step stand together, apart from what goes before and after (per evaluation,
        // us, mixed / apart: 589,824 weights k = 64 15.58 / 15.28, 300,000 k = 256 28.2 / 27.2, 300,000 2-vectors k = 128 16.9 / 16.1,
        // 294,912 8-vectors k = 256 62.1 / 60.8; with 8 pairs, 20,000 weights k = 24, 4.96 / 5.07).  The same sums in the same order.
        // (Nothing gained where the row is shifted, as under the plain norm.)
        constexpr bool APART = KB * V >= 16;
        bool shift = DIST == DIST_L2;
        if constexpr (DIST == DIST_SQL2) {
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                float c[D];
                codeword(b, escale, c);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    p[b][i] = energy(c, i);
                    if (!APART) {
                        p[b][i] = fast_exp2(-p[b][i]);
                        S[i] += p[b][i];
                    }
                }
            }
            if constexpr (APART) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int b = 0; b < KB; ++b)
#pragma unroll
                    for (int i = 0; i < V; ++i) p[b][i] = fast_exp2(-p[b][i]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int b = 0; b < KB; ++b)
#pragma unroll
                    for (int i = 0; i < V; ++i) S[i] += p[b][i];
            }
            float smin = inf_();
#pragma unroll
            for (int i = 0; i < V; ++i) {
                S[i] = row16_sum(S[i]);
                smin = fminf(smin, S[i]);
            }
            shift = __builtin_amdgcn_ballot_w64(smin < 7.9e-31f) != 0ull;  // below 2^-100
        }
        if (shift) {
            next_phase();
            float emin[V];
#pragma unroll
            for (int i = 0; i < V; ++i) emin[i] = inf_();
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                float c[D];
                codeword(b, escale, c);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    p[b][i] = energy(c, i);
                    emin[i] = fminf(emin[i], p[b][i]);
                }
            }
#pragma unroll
            for (int i = 0; i < V; ++i) {
                emin[i] = row16_min(emin[i]);
                S[i] = 0.f;
            }
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    p[b][i] = fast_exp2(emin[i] - p[b][i]);
                    S[i] += p[b][i];
                }
#pragma unroll
            for (int i = 0; i < V; ++i) S[i] = row16_sum(S[i]);
        }
        float rS[V];
#pragma unroll
        for (int i = 0; i < V; ++i) rS[i] = fast_rcp(S[i]) * live[i];
        const float inv = 1.0f / escale;
        if constexpr (PASS == PASS_FWD) {
            float rw[V][D];
#pragma unroll
            for (int i = 0; i < V; ++i)
#pragma unroll
                for (int r = 0; r < D; ++r) rw[i][r] = w[i][r] * (rS[i] * inv);
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    acc[b * ACCW] = fmaf(p[b][i], rS[i], acc[b * ACCW]);
#pragma unroll
                    for (int r = 0; r < D; ++r) acc[b * ACCW + 1 + r] = fmaf(p[b][i], rw[i][r], acc[b * ACCW + 1 + r]);
                }
        } else {
            // delta = 2 (w - c) = (2/s) t: the factor 2/(s S) joins the row's scalar
            next_phase();
            float q[KB][V], qb[V];
#pragma unroll
            for (int i = 0; i < V; ++i) qb[i] = 0.f;
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                float h[D], hf;
                if constexpr (REGS) {
                    cotangent(b, h);
                    hf = rf[b][0];
                } else {
                    table_row(tc + 16 * KB * D, b, h);
                    hf = tc[32 * KB * D + (threadIdx.x & 15) + 16 * b];
                }
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    float s = fmaf(h[0], w[i][0], -hf);
#pragma unroll
                    for (int r = 1; r < D; ++r) s = fmaf(h[r], w[i][r], s);
                    q[b][i] = s;
                    qb[i] = fmaf(p[b][i], s, qb[i]);
                }
            }
            next_phase();
            float f[V];
#pragma unroll
            for (int i = 0; i < V; ++i) {
                f[i] = 2.f * rS[i] * inv;
                qb[i] = row16_sum(qb[i]) * rS[i];
            }
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                float c[D];
                codeword(b, escale, c);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const float th = (p[b][i] * f[i]) * (q[b][i] - qb[i]);
#pragma unroll
                    for (int r = 0; r < D; ++r) acc[b * ACCW + r] = fmaf(th, w[i][r] - c[r], acc[b * ACCW + r]);
                }
            }
        }
    }

    static __device__ __forceinline__ float inf_() { return __builtin_inff(); }
    static __device__ __forceinline__ int row16_min_i(int x) {
        const int big = 0x7fffffff;
        x = min(x, dpp_i<0xB1, 0xf>(big, x));
        x = min(x, dpp_i<0x4E, 0xf>(big, x));
        x = min(x, dpp_i<0x141, 0xf>(big, x));
        x = min(x, dpp_i<0x140, 0xf>(big, x));
        return x;
    }
    // Sums over the row's lanes of x[i][r], stored as vectors vb + i of the tile's share of out: the V D values of a row
    // lie together, lane V' D + r' stores one of them.
    __device__ __forceinline__ void store_rows(const float (&x)[V][D], float* out, int64_t base, int vb, int vend) const {
        static_assert(V * D <= 16, "one value per lane of a row");
        const int j0 = threadIdx.x & 15;
        float mine = 0.f;
#pragma unroll
        for (int i = 0; i < V; ++i)
#pragma unroll
            for (int r = 0; r < D; ++r) {
                const float s = row16_sum(x[i][r]);
                mine = (j0 == i * D + r) ? s : mine;
            }
        if (j0 < V * D && vb + j0 / D < vend) out[(base + vb) * D + j0] = mine;
    }

    // After the last step: the pass's sums over the wavefront into part[codeword][ACCW] (all 16 KB codewords).
    __device__ __forceinline__ void collect(float* part, int tid) const {
        const int lane = tid & 63, j0 = lane & 15, row = lane >> 4;
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            const float s = cross_row_sum(acc[q]);
            if (row == (q & 3)) part[(j0 + 16 * (q / ACCW)) * ACCW + q % ACCW] = s;
        }
    }
};

// The wavefronts of a workgroup of NT threads take the steps of a tile of cnt vectors in turn.
template <int KB, int D, int DIST, int PASS, int NT>
__device__ __forceinline__ void row_tile_pass(const Args& a, RowWave<KB, D, DIST, PASS>& st, const float* s_w,
                                              const float* s_g, int64_t base, int cnt) {
    constexpr int STEP = RowWave<KB, D, DIST, PASS>::STEP;
    int v0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * STEP;
    PassPriority prio((cnt - v0 + (NT / 64) * STEP - 1) / ((NT / 64) * STEP));
    for (; v0 + STEP <= cnt; v0 += (NT / 64) * STEP) {
        st.template step<true>(a, s_w, s_g, base, v0, cnt);
        prio.step_done();
    }
    if (v0 < cnt) st.template step<false>(a, s_w, s_g, base, v0, cnt);
}

// Stream path: one launch per pass.  A workgroup takes tiles b, b + grid, ... of vec_per_wg vectors, copies each into LDS
// (dL/dWq too) and adds the tile's sums to a.partials[workgroup][.] (float64) for reduce_rows and lane_tail.  Dynamic LDS: one
// tile, two for the passes that read dL/dWq.  SEVERAL = false (d = 8): the grid has a workgroup for every tile; as a loop the
// passes at k = 256 keep some 15 registers more, and spill them.  36 KB tiles: 294,912 8-vectors, k = 256, 62.2 us an
// evaluation against 66.4 with 18 KB and 72.5 with 12; 2.4 M 2-vectors, k = 64, 59.4 against 69.4 and 69.0.
constexpr int RST = 512;
// Vectors of the largest tile: 36 KB, and for scalars no more than 256 float32 additions to a sum before it is float64 (252
// vectors of a lane, the four rows of a wavefront).
constexpr int64_t row_tile_vectors(int d) { return d == 1 ? 252 * (RST / 64) * 4 : 9216 / d; }
template <int KB, int D, int DIST, int PASS, bool SEVERAL>
__global__ __launch_bounds__(RST) void row_pass(const Args a) {
    using RW = RowWave<KB, D, DIST, PASS>;
    if (PASS == PASS_FWD && a.ctrl->done) return;
    if (PASS == PASS_B2 && a.ctrl->b_done) return;
    constexpr int KDP = 16 * KB * D;
    extern __shared__ __align__(16) float s_tile[];
    __shared__ __align__(16) float s_Cf[KDP];
    __shared__ __align__(16) float s_Hs[RW::USE_H ? KDP : 1], s_Ff[RW::USE_H ? KDP : 1];
    __shared__ __align__(16) float s_rtab[RW::TAB];
    __shared__ float s_part[PASS == PASS_B3 ? 1 : RST / 64][PASS == PASS_B3 ? 1 : 16 * KB * RW::ACCW];
    const int tid = threadIdx.x, k = a.k, kd = k * D, per = (int)a.vec_per_wg;
    float* s_g = s_tile + (size_t)per * D;
    for (int i = tid; i < KDP; i += RST) {
        s_Cf[i] = i < kd ? a.Cf[i] : 0.f;
        if (RW::USE_H) {
            s_Hs[i] = i < kd ? a.Hs[i] : 0.f;
            s_Ff[i] = i < kd ? a.Ff[i] : 0.f;
        }
    }
    if (RW::TAB > 1) {
        __syncthreads();
        RW::template fill_table<RST>(s_rtab, k, s_Cf, s_Hs, s_Ff, a.escale);
    }
    auto tile = [&](int64_t t) {
        int tid = threadIdx.x;
        if (SEVERAL) asm volatile("" : "+v"(tid));  // (what every tile needs is formed again, not kept over the steps)
        const int64_t base = t * per;
        const int cnt = (a.m - base < per) ? (int)(a.m - base) : per;
        load_tile<RST>(s_tile, a.W + base * D, cnt * D);
        if (RW::USE_G) load_tile<RST>(s_g, a.G + base * D, cnt * D);
        __syncthreads();
        RW st;
        st.init(k, RW::TAB > 1 ? s_rtab : s_Cf, s_Hs, s_Ff, a.escale);
        row_tile_pass<KB, D, DIST, PASS, RST>(a, st, s_tile, s_g, base, cnt);
        if (SEVERAL) asm volatile("" : "+v"(tid));
        if constexpr (PASS != PASS_B3) {
            st.collect(s_part[tid >> 6], tid);
            __syncthreads();
            const int nacc = k * RW::ACCW;
            for (int idx = tid; idx < nacc; idx += RST) {
                double x = 0.0;
#pragma unroll
                for (int w = 0; w < RST / 64; ++w) x += (double)s_part[w][idx];
                double* p = &a.partials[(size_t)blockIdx.x * nacc + idx];
                *p = (!SEVERAL || t == (int64_t)blockIdx.x) ? x : *p + x;  // (a thread's own sums)
            }
        }
    };
    if constexpr (SEVERAL) {
        const int64_t tiles = (a.m + per - 1) / per;
        for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
            tile(t);
            if (PASS == PASS_B3) __syncthreads();  // (the other passes: the barrier behind collect)
        }
    } else {
        tile(blockIdx.x);
    }
}

}  // namespace idkm
