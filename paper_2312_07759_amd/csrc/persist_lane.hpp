// Persistent kernels for the lane<->codeword, row<->vector and matrix-core forms (k up to 512): one launch per solve, the
// workgroup's tile of W (and dL/dWq) resident in LDS, and per pass one exchange of the k (d+1) (backward: k d) sums:
//   hop 1  (inside a die) workgroup g stores its partial sums contiguously at buf1[parity][g][.]; the members of a die
//          (workgroups x, x + 8, ...) each own a slice of the words, read it from every member's line, add it in float64
//          in a fixed order and store the die's totals at buf3[parity][x][.];
//   hop 2  (across dies) every member adds the 8 dies' totals of its slice, in a fixed order, and stores the grid totals at
//          buf4[parity][x][.], where its die reads them; EVERY workgroup applies the O(k d) update itself, so that all
//          hold the same state and take the same stop decision.
// Workgroups' sums travel as float32 (d = 8: float64), the dies' and the grid's totals as float64 in two words (SumWords).
// As in persist_small.hpp a store of hop 1 only has to reach the die's L2 when all members of the die run there (checked at
// the start of a launch).  There one workgroup per die adds all of the at most 80 words.  The form this
// replaced had one reducer per codeword that read all 256 workgroups through memory, and a broadcast of the result.  Before
// and now: 589,824 weights under 64 codewords 671 -> 550 us (30 evaluations and a Jacobian-free backward; 598 -> 562 of it from
// the slices of hop 2), 589,824 4-vectors under 256 codewords (30 evaluations, 10 passes) 2484 -> 2461.  Totals in one word
// with 29 bits, for comparison: 553 and 2416; 64,000 8-vectors under 256 codewords (20 evaluations) 510 against 577.
// Waits are bounded exactly as in persist_small.hpp.
#pragma once
#include "common.hpp"
#include "lane_k.hpp"
#include "mfma_lane.hpp"
#include "persist_small.hpp"
#include "row_k.hpp"

namespace idkm {

constexpr int LT = 1024;          // threads per workgroup (16 wavefronts, 4 per SIMD)
constexpr int LWAVES = LT / 64;
constexpr int MT = 512;           // threads per workgroup of the matrix-core forward kernel (2 wavefronts per SIMD:
                                  // its accumulators and one 16 x 256 tile of weights need ~200 registers per lane)

// Threads per workgroup of the row <-> vector kernels.  With 1024, k = 64, d = 1 takes 610 us instead of 617 at 589,824
// weights, but 189 instead of 175 at 74,921 (k = 32) and 189 instead of 176 at 9,643 (k = 48): the shares of the wavefronts
// get too short.
constexpr int RT = 512;

struct LShared {
    double part[1024];    // hop 1: per-thread (or per-wavefront) sums of a slice
    double wsum[LWAVES];
    double scalar;        // result of block_sum
    int abort;
    int local;            // all members of this workgroup's die run on one die: hop 1 only has to reach its L2
};

__device__ __forceinline__ void raise_abort(const PArgs& pa, LShared& ls) {
    ls.abort = 1;
    raise_abort(pa);
}

// Sum of one float64 per thread over the workgroup, fixed order, returned to every thread.
template <int NT = LT>
__device__ __forceinline__ double block_sum_fixed(double x, LShared& ls) {
    x = wave_sum_d_dpp(x);
    if ((threadIdx.x & 63) == 0) ls.wsum[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) s += ls.wsum[w];
        ls.scalar = s;
    }
    __syncthreads();
    return ls.scalar;
}

// Hop-1 store: sum idx of this workgroup's line.  WIDE as in SumWords: the workgroups' sums of d = 8 travel as float64 (its
// solves on the stream path hand them on in that form), the others as float32; the totals are float64 from there on.
template <bool WIDE>
__device__ __forceinline__ void put_sum(const LShared& ls, unsigned long long* line, int nacc, unsigned int seq, int idx, double t) {
    st_sum<WIDE>(&line[idx], nacc, seq, t, ls.local != 0);
}
template <bool WIDE>
__device__ __forceinline__ unsigned long long* own_line(const PArgs& pa, unsigned int seq, int nacc) {
    return pa.buf1 + ((size_t)(seq & 1u) * pa.G + pa.wg) * nacc * SumWords<WIDE>::N;
}

// Workgroup partial of the lane accumulators (wavefronts add one after the other, float64) and hop-1 store.
template <int NA, int ACCW, int NT = LT>
__device__ __forceinline__ void publish_lane(const PArgs& pa, const LShared& ls, unsigned int seq, const float (&acc)[NA], int k,
                                             double (*s_acc)[NA]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int wv = 0; wv < NT / 64; ++wv) {
        if (wave == wv) {
#pragma unroll
            for (int q = 0; q < NA; ++q) {
                if (wv == 0)
                    s_acc[lane][q] = (double)acc[q];
                else
                    s_acc[lane][q] += (double)acc[q];
            }
        }
        __syncthreads();
    }
    const int nacc = k * ACCW;
    unsigned long long* dst = own_line<false>(pa, seq, nacc);
    for (int idx = tid; idx < nacc; idx += NT) {
        const int j = idx / ACCW, comp = idx - j * ACCW;
        put_sum<false>(ls, dst, nacc, seq, idx, s_acc[j & 63][(j >> 6) * ACCW + comp]);
    }
}

// Start of a launch: every workgroup says which die it runs on (before it loads its tile) and reads the words of its die's
// members: leaves ls.local.  Returns false if the wait was abandoned.  Called by all threads; ends with a barrier.
__device__ __forceinline__ void die_announce(const PArgs& pa) {
    if (threadIdx.x == 0) st_word(&pa.tab[pa.wg], pack_u(pa.seq_base + 1u, die_id()));
}
__device__ __forceinline__ bool die_handshake(const PArgs& pa, LShared& ls) {
    const int nmem = (pa.G - pa.wg % DIES + DIES - 1) / DIES;  // members of this die, at most PT / DIES = 32
    if (threadIdx.x < 64) {
        bool same = true, failed = false;
        if ((int)threadIdx.x < nmem) {
            unsigned long long w[1] = {0ull};
            failed = !poll_words<1>(pa, pa.tab + (pa.wg % DIES) + (size_t)threadIdx.x * DIES, 0, pa.seq_base + 1u, w);
            same = (unsigned int)w[0] == die_id();
        }
        const bool all_same = __builtin_amdgcn_ballot_w64(!same) == 0ull, any_failed = __builtin_amdgcn_ballot_w64(failed) != 0ull;
        if (threadIdx.x == 0) {
            ls.local = (all_same && pa.tree != 2) ? 1 : 0;  // 2: test support, every store at device scope
            if (any_failed) raise_abort(pa, ls);
        }
    }
    __syncthreads();
    return ls.abort == 0;
}

// Words of the dies' and the grid's totals: the halves of a sum lie next to each other, the lower one first.
__device__ __forceinline__ unsigned long long half_word(unsigned int seq, double t, int half) {
    return pack_u(seq, (unsigned int)(half ? __double2hiint(t) : __double2loint(t)));
}
// Hop 1, receiving side: this workgroup's slice of its die's totals.  S = ceil(nacc / members) words per member; SP, the
// power of two at or above it (at most NT), threads take one word each of NT / SP lines at a time; what several lines
// leave in the lanes of a wavefront is added across lanes, the wavefronts through LDS, all in a fixed order.  With one die
// (a team of one) the totals go straight to s_tot.  Returns false if the wait was abandoned.
template <int NT, bool WIDE = false>
__device__ __forceinline__ bool die_slice(const PArgs& pa, unsigned int seq, int nacc, LShared& ls, double* s_tot) {
    const int tid = threadIdx.x, lane = tid & 63, x = pa.wg % DIES, mi = pa.wg / DIES;
    const int nmem = (pa.G - x + DIES - 1) / DIES;
    const int S = (nacc + nmem - 1) / nmem, first = mi * S;
    const int n = nacc - first < S ? nacc - first : S;  // (the last members' slices may be short or empty)
    int lg = 0;
    while ((1 << lg) < S && (1 << lg) < NT) ++lg;
    const int SP = 1 << lg, LPR = NT >> lg;  // words and lines a round of loads covers
    constexpr int UNR = WIDE ? 8 : 4;        // lines in flight
    using Word = SumWords<WIDE>;
    const unsigned long long* src = pa.buf1 + (size_t)(seq & 1u) * pa.G * nacc * Word::N + first;
    unsigned long long* out = pa.buf3 + ((size_t)(seq & 1u) * DIES + x) * nacc * 2 + 2 * first;
    if (n <= 0) __syncthreads();  // (s_tot may share memory with what publish_lane reads; otherwise the barrier below)
    for (int w0 = 0; w0 < n; w0 += SP) {
        const int w = w0 + (tid & (SP - 1)), l0 = tid >> lg;
        double s = 0.0;
        bool aborted = false;
        for (int l = l0; l < nmem && w < n; l += UNR * LPR) {
            Word v[UNR];
            unsigned int spins = 0;
            for (;;) {
                bool ok = true;
#pragma unroll
                for (int u = 0; u < UNR; ++u) {
                    if (l + u * LPR < nmem)
                        v[u].load(src + (size_t)(x + (l + u * LPR) * DIES) * nacc * Word::N + w, nacc);
                    else
                        v[u].zero(seq);
                }
#pragma unroll
                for (int u = 0; u < UNR; ++u) ok = ok && v[u].arrived(seq);
                if (ok) break;
                ++spins;
                if (spins > pa.spin_limit ||
                    ((spins & 31u) == 0u && __hip_atomic_load(pa.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == pa.seq_base + 1u)) {
                    aborted = true;
                    break;
                }
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) s += v[u].value();
            if (aborted) break;
        }
        // lanes of a wavefront that hold the same word
        if (SP <= 32) {
            if (SP <= 1) s += dpp_d<0xB1, 0xf>(s);   // quad_perm [1,0,3,2]
            if (SP <= 2) s += dpp_d<0x4E, 0xf>(s);   // quad_perm [2,3,0,1]
            if (SP <= 4) s += dpp_d<0x124, 0xf>(s);  // row_ror:4 (lanes l and l + 4 hold the same pairs already)
            if (SP <= 8) s += dpp_d<0x128, 0xf>(s);  // row_ror:8
            if (SP <= 16) s = cross_row_sum_d(s);
            if (SP == 32) s = upper_lower_sum_d(s);
        }
        if (SP >= 64 || lane < SP) ls.part[SP >= 64 ? tid : (tid >> 6) * 64 + lane] = s;
        if (aborted) raise_abort(pa, ls);
        __syncthreads();
        if (ls.abort) return false;
        // (two lanes a sum, one for each word: a slice leaves in one run of stores)
        const int live = n - w0 < SP ? n - w0 : SP;
        for (int h = tid; h < 2 * live; h += NT) {
            const int q = h >> 1;
            const int groups = SP >= 64 ? LPR : NT / 64, stride = SP >= 64 ? SP : 64;
            double c2[2] = {0.0, 0.0};
            for (int g = 0; g + 1 < groups; g += 2) {
                c2[0] += ls.part[g * stride + q];
                c2[1] += ls.part[(g + 1) * stride + q];
            }
            if (groups & 1) c2[0] += ls.part[(groups - 1) * stride + q];
            const double t = c2[0] + c2[1];
            if (pa.G == 1)
                s_tot[first + w0 + q] = t;  // (both lanes the same value)
            else
                st_word(&out[2 * w0 + h], half_word(seq, t, h & 1));
        }
        if (w0 + SP < n) __syncthreads();
    }
    return true;
}

// Sum of nd dies' totals of one word pair, for a pair of lanes: each waits for its half from every die (src, src + line, ...)
// and gets the other from its neighbour.  Both return the sum, or false if the wait of either was abandoned.
__device__ __forceinline__ bool dies_sum(const PArgs& pa, const unsigned long long* src, int line, int nd, unsigned int seq, double& out) {
    unsigned long long v[DIES];
    unsigned int spins = 0;
    int failed = 0;
    for (;;) {
        bool ok = true;
#pragma unroll
        for (int x = 0; x < DIES; ++x) v[x] = x < nd ? ld_word(src + (size_t)x * line) : pack_u(seq, 0u);
#pragma unroll
        for (int x = 0; x < DIES; ++x) ok = ok && (unsigned int)(v[x] >> 32) == seq;
        if (ok) break;
        ++spins;
        if (spins > pa.spin_limit ||
            ((spins & 31u) == 0u && __hip_atomic_load(pa.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == pa.seq_base + 1u)) {
            failed = 1;
            break;
        }
    }
    failed |= dpp_i<0xB1, 0xf>(0, failed);  // quad_perm [1,0,3,2]
    double t[DIES];
#pragma unroll
    for (int x = 0; x < DIES; ++x) {
        const int own = (int)(unsigned int)v[x], other = dpp_i<0xB1, 0xf>(0, own);
        t[x] = (threadIdx.x & 1) ? __hiloint2double(own, other) : __hiloint2double(other, own);
    }
    out = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    return !failed;
}

// Hop 2 where dies have several members, in two steps: every workgroup adds the dies' totals of its own slice and stores the
// grid totals for its die, whose members read them from the L2.  (With one step every workgroup polls 8 nacc words through
// memory, and those polls hold up the stores they wait for: k = 64, d = 1 598 us against 562 with two steps.)  Leaves the
// totals in s_tot, in every workgroup; ends with a barrier.
template <int NT, int MAXACC, int MAXRND>
__device__ __forceinline__ bool grid_totals_by_slices(const PArgs& pa, unsigned int seq, int nacc, LShared& ls, double* s_tot) {
    const int x0 = pa.wg % DIES, mi = pa.wg / DIES;
    const int nmem = (pa.G - x0 + DIES - 1) / DIES;
    const int S = (nacc + nmem - 1) / nmem, first = mi * S;
    const int n = nacc - first < S ? nacc - first : S;
    const unsigned long long* src = pa.buf3 + (size_t)(seq & 1u) * DIES * nacc * 2 + 2 * first;
    unsigned long long* mine = pa.buf4 + ((size_t)(seq & 1u) * DIES + x0) * nacc * 2;
    bool aborted = false;
    auto give_up = [&](unsigned int& spins) {
        ++spins;
        return spins > pa.spin_limit ||
               ((spins & 31u) == 0u && __hip_atomic_load(pa.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == pa.seq_base + 1u);
    };
    auto pass_on = [&](int h, double t) {
        const unsigned long long word = half_word(seq, t, h & 1);
        if (ls.local)
            st_word_die(&mine[2 * first + h], word);
        else
            st_word(&mine[2 * first + h], word);
    };
    // A full device's slices: a row of 16 lanes takes a sum, lane 2 x + h waits for half h of die x's total, and the dies are
    // added across lanes; RND sums of a lane in flight.  Few members have long slices: two lanes a sum.  (232,121 weights,
    // k = 64, 20 evaluations and 10 passes: 394 us with rows, 405 with pairs; 95,909 8-vectors, k = 128, 20 evaluations: 481
    // and 494; the matrix-core kernel at k = 256, with two sums in flight, 2500 and 2473: MAXRND = 1 there.)
    constexpr int ROWS = NT / 16, RND = (MAXACC + (PT / DIES) * ROWS - 1) / ((PT / DIES) * ROWS);
    if (RND <= MAXRND && n <= ROWS * RND) {
        const int half = threadIdx.x & 1, x = (threadIdx.x >> 1) & (DIES - 1), w0 = threadIdx.x >> 4;
        unsigned long long v[RND];
        unsigned int spins = 0;
        if (w0 < n) {
            for (;;) {
                bool ok = true;
#pragma unroll
                for (int u = 0; u < RND; ++u)
                    v[u] = w0 + u * ROWS < n ? ld_word(src + (size_t)x * 2 * nacc + 2 * (w0 + u * ROWS) + half) : pack_u(seq, 0u);
#pragma unroll
                for (int u = 0; u < RND; ++u) ok = ok && (unsigned int)(v[u] >> 32) == seq;
                if (ok) break;
                if (give_up(spins)) {
                    aborted = true;
                    break;
                }
            }
            aborted = __builtin_amdgcn_ballot_w64(aborted) != 0ull;  // (nothing that is not whole is passed on)
        }
        if (w0 < n && !aborted) {
#pragma unroll
            for (int u = 0; u < RND; ++u) {
                if (w0 + u * ROWS >= n) break;
                const int own = (int)(unsigned int)v[u], other = dpp_i<0xB1, 0xf>(0, own);  // quad_perm [1,0,3,2]
                double t = half ? __hiloint2double(own, other) : __hiloint2double(other, own);
                t += dpp_d<0x4E, 0xf>(t);   // quad_perm [2,3,0,1]: dies x and x ^ 1
                t += dpp_d<0x141, 0xf>(t);  // row_half_mirror: the other quad
                t += dpp_d<0x140, 0xf>(t);  // row_mirror: the other half of the row
                if (x == 0) pass_on(2 * (w0 + u * ROWS) + half, t);
            }
        }
    } else {
        for (int h = threadIdx.x; h < 2 * n && !aborted; h += NT) {
            double t;
            aborted = !dies_sum(pa, src + h, 2 * nacc, DIES, seq, t);
            if (aborted) break;
            pass_on(h, t);
        }
    }
    // (the words lie as the halves of s_tot do)
    typedef unsigned int __attribute__((may_alias)) half_t;
    half_t* tot = reinterpret_cast<half_t*>(s_tot);
    constexpr int GW = (2 * MAXACC + NT - 1) / NT;  // words of a thread, all in flight
    if ((int)threadIdx.x < 2 * nacc && !aborted) {
        const int idx = threadIdx.x;
        unsigned long long v[GW];
        unsigned int spins = 0;
        for (;;) {
            bool ok = true;
#pragma unroll
            for (int u = 0; u < GW; ++u) v[u] = idx + u * NT < 2 * nacc ? ld_word(mine + idx + u * NT) : pack_u(seq, 0u);
#pragma unroll
            for (int u = 0; u < GW; ++u) ok = ok && (unsigned int)(v[u] >> 32) == seq;
            if (ok) break;
            if (give_up(spins)) {
                aborted = true;
                break;
            }
        }
#pragma unroll
        for (int u = 0; u < GW; ++u)
            if (idx + u * NT < 2 * nacc) tot[idx + u * NT] = (unsigned int)v[u];
    }
    if (aborted) raise_abort(pa, ls);
    __syncthreads();
    return ls.abort == 0;
}

// Hop 2, every workgroup: grid totals of the nacc <= MAXACC sums in s_tot.  Returns false if the wait was abandoned; ends with a
// barrier.
template <int NT, int MAXACC, int MAXRND>
__device__ __forceinline__ bool grid_totals(const PArgs& pa, unsigned int seq, int nacc, LShared& ls, double* s_tot) {
    if (pa.G > DIES) return grid_totals_by_slices<NT, MAXACC, MAXRND>(pa, seq, nacc, ls, s_tot);
    if (pa.G > 1) {  // one workgroup per die
        const unsigned long long* src = pa.buf3 + (size_t)(seq & 1u) * DIES * nacc * 2;
        bool aborted = false;
        for (int h = threadIdx.x; h < 2 * nacc && !aborted; h += NT) {
            double t;
            aborted = !dies_sum(pa, src + h, 2 * nacc, pa.G, seq, t);
            if (!(h & 1)) s_tot[h >> 1] = t;
        }
        if (aborted) raise_abort(pa, ls);
    }
    __syncthreads();
    return ls.abort == 0;
}

template <int KPL, int D, int DIST, int PASS, int NT = LT>
__device__ __forceinline__ void lane_tile_pass(const Args& a, LaneWave<KPL, D, DIST, PASS>& st, const float* s_w,
                                               const float* s_g, int64_t base, int cnt) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // every wavefront takes an equal contiguous share of the tile
    const int share = (cnt + NT / 64 - 1) / (NT / 64);
    const int w0 = wave * share;
    const int w1 = (w0 + share < cnt) ? w0 + share : cnt;
    for (int b = w0; b < w1; b += 64) {
        float wv[D], gv[D];
        const int i = b + lane;
#pragma unroll
        for (int r = 0; r < D; ++r) {
            wv[r] = (i < w1) ? s_w[i * D + r] : 0.f;
            gv[r] = (LaneWave<KPL, D, DIST, PASS>::USE_G && i < w1) ? s_g[i * D + r] : 0.f;
        }
        st.batch(a, base + b, (w1 - b < 64) ? (w1 - b) : 64, wv, gv);
    }
}

#ifdef IDKM_TRACE
#define IDKM_LSTAMP(slot)                                                                        \
    do {                                                                                         \
        if (pa.trace && threadIdx.x == 0 && iters == 20 && pa.wg < 256)                        \
            pa.trace[2 * 64 * 8 + pa.wg * 8 + (slot)] = (long long)wall_clock64();               \
    } while (0)
#else
#define IDKM_LSTAMP(slot)
#endif

// Hop-1 store of a pass whose wavefronts left their totals in part[wavefront][nacc]: they add up in wavefront order,
// float64, as in publish_lane.
template <int NW, bool WIDE = false>
__device__ __forceinline__ void publish_parts(const PArgs& pa, const LShared& ls, unsigned int seq, const float* part, int stride, int nacc) {
    unsigned long long* dst = own_line<WIDE>(pa, seq, nacc);
    for (int idx = threadIdx.x; idx < nacc; idx += NW * 64) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += (double)part[w * stride + idx];
        put_sum<WIDE>(ls, dst, nacc, seq, idx, t);
    }
}

// Forward solve (Alg. 1) and the evaluation at C*.  KB > 0: the passes run in the row <-> vector form (row_k.hpp) with
// NT threads, for up to 16 KB codewords.  MFMA: the loop's passes run on the matrix cores (mfma_lane.hpp;
// d = 4), with NT = MT threads; the dynamic LDS then holds the tile padded by 16 zero vectors and,
// behind it, -s^2 |w|^2 of every vector.
template <int KPL, int D, int DIST, int NT = LT, bool MFMA = false, int KB = 0>
__device__ __forceinline__ void persist_lane_fwd_body(const Args& a, const PArgs& pa) {
    static_assert(!MFMA || (D == 4 && KPL <= 4), "matrix-core loop: d = 4, k <= 256");
    constexpr int ACCW = D + 1;
    constexpr int NA = KPL * ACCW;
    constexpr int KMAX = KB > 0 ? 16 * KB : 64 * KPL;
    constexpr int KDP = KMAX * D;  // padded codebook size
    constexpr bool WIDE1 = D == 8;
    extern __shared__ float s_tile[];
    // workgroup sums of a vector-ALU pass; from the first hop on, the grid totals of the pass
    __shared__ double s_acc[KB > 0 ? KMAX : 64][KB > 0 ? ACCW : NA];
    double* s_tot = &s_acc[0][0];
    __shared__ LShared ls;
    __shared__ __align__(16) float s_Cf[KDP];
    __shared__ float s_rpart[KB > 0 ? NT / 64 : 1][KB > 0 ? KMAX * ACCW : 1];  // row form: totals of the wavefronts
    __shared__ __align__(16) float s_rtab[KB > 0 ? RowWave<(KB > 0 ? KB : 1), D, DIST, PASS_FWD>::TAB : 1];

    const int tid = threadIdx.x, wg = pa.wg;
    const int k = a.k, kd = k * D, nacc = k * ACCW;
    die_announce(pa);
    const int64_t base = (int64_t)wg * pa.per;
    int cnt = 0;
    if (base < a.m) cnt = (a.m - base < pa.per) ? (int)(a.m - base) : pa.per;
    load_tile<NT>(s_tile, a.W + base * D, cnt * D);
    for (int i = tid; i < kd; i += NT) {
        const float c0 = pa.C0[i];
        s_Cf[i] = c0;
    }
    if (KB > 0)
        for (int i = kd + tid; i < KDP; i += NT) s_Cf[i] = 0.f;
    if (tid == 0) ls.abort = 0;
    __syncthreads();
    if (!die_handshake(pa, ls)) return;
    const float* s_wn = s_tile + (size_t)(pa.per + 16) * D;
    __shared__ float s_mu[4];
    if constexpr (MFMA) {
        // reference point of the centred coordinates: the mean of the initial codewords
        if (tid < D) {
            float sm = 0.f;
            for (int j = 0; j < k; ++j) sm += s_Cf[j * D + tid];
            s_mu[tid] = sm / (float)k;
        }
        float* wn = s_tile + (size_t)(pa.per + 16) * D;
        for (int i = cnt * D + tid; i < (pa.per + 16) * D; i += NT) s_tile[i] = 0.f;
        __syncthreads();
        for (int i = tid; i < pa.per + 16; i += NT) {
            float n2 = 0.f;
#pragma unroll
            for (int r = 0; r < D; ++r) {
                const float t = (s_tile[i * D + r] - s_mu[r]) * a.escale;
                n2 = fmaf(t, t, n2);
            }
            wn[i] = -n2;
        }
        __syncthreads();
    }
    const double tol = pa.tol;
    const int max_iter = pa.max_iter;
    unsigned int seq = pa.seq_base;

    // matrix-core passes: per-wavefront partial sums, the codeword tables of the step, the table of the evaluation at C*
    constexpr int TS = MfmaFwd<(KPL <= 4 ? KPL : 4)>::TAB_STRIDE;
    __shared__ __align__(16) float s_part[MFMA ? NT / 64 : 1][MFMA ? 64 * KPL * ACCW : 1];
    __shared__ float2 s_tab[MFMA ? 4 * TS : 1];
    __shared__ float s_fac[MFMA ? TS : 1];
    __shared__ f32x4 s_ctab[MFMA ? TS : 1];
    // hop-1 store of a matrix-core pass: wavefront totals add up in wavefront order, float64, as in publish_lane
    auto publish_matrix = [&]() {
        if constexpr (MFMA) {
            publish_parts<NT / 64>(pa, ls, seq, &s_part[0][0], 64 * KPL * ACCW, nacc);
        }
    };

    // (every thread holds the state of the stop rule)
    int iters = 0;
    bool done = false, conv = false, bad = false;
    double res = 0.0;
    while (!done) {
        ++seq;
        IDKM_LSTAMP(0);
        if constexpr (MFMA) {
            const bool fold = MfmaFwd<KPL>::template fill_table<NT>(s_tab, s_fac, k, s_Cf, s_mu, a.escale) &&
                              DIST == DIST_SQL2;
            {
                MfmaFwd<KPL> st;
                st.init(s_tab, s_fac, s_mu);
                mfma_tile_pass<KPL, DIST, NT>(st, s_tile, s_wn, cnt, a.escale, fold);
                IDKM_LSTAMP(1);
                mfma_collect<KPL, NT>(st, &s_part[0][0], fold, s_fac);
            }
            __syncthreads();
            IDKM_LSTAMP(5);
            publish_matrix();
        } else if constexpr (KB > 0) {
            {
                using RW = RowWave<KB, D, DIST, PASS_FWD>;
                if (RW::TAB > 1) {
                    RW::template fill_table<NT>(s_rtab, k, s_Cf, nullptr, nullptr, a.escale);
                    __syncthreads();
                }
                RW st;
                st.init(k, RW::TAB > 1 ? s_rtab : s_Cf, nullptr, nullptr, a.escale);
                row_tile_pass<KB, D, DIST, PASS_FWD, NT>(a, st, s_tile, nullptr, base, cnt);
                IDKM_LSTAMP(1);
                st.collect(s_rpart[tid >> 6], tid);
            }
            __syncthreads();
            IDKM_LSTAMP(5);
            publish_parts<NT / 64, WIDE1>(pa, ls, seq, &s_rpart[0][0], KMAX * ACCW, nacc);
        } else {
            LaneWave<KPL, D, DIST, PASS_FWD> st;
            st.init(k, s_Cf, nullptr, nullptr, a.escale);
            lane_tile_pass<KPL, D, DIST, PASS_FWD, NT>(a, st, s_tile, nullptr, base, cnt);
            IDKM_LSTAMP(1);
            publish_lane<NA, ACCW, NT>(pa, ls, seq, st.acc, k, s_acc);
        }
        IDKM_LSTAMP(2);
        if (!die_slice<NT, WIDE1>(pa, seq, nacc, ls, s_tot)) return;
        IDKM_LSTAMP(3);
        if (!grid_totals<NT, KMAX * ACCW, KB ? 3 : 1>(pa, seq, nacc, ls, s_tot)) return;
        IDKM_LSTAMP(4);
        // centre update (Alg. 1) and stop test, the same in every workgroup; a non-finite sum gives NaN
        double r2 = 0.0;
        for (int i = tid; i < kd; i += NT) {
            const int j = i / D, rr = i - j * D;
            const double n = s_tot[j * ACCW], sv = s_tot[j * ACCW + 1 + rr];
            double cnew = (n > 0.0) ? fast_div_d(sv, n) : (double)s_Cf[i];
            if (!(n >= 0.0) || !(fabs(sv) <= 1.7e308) || !(fabs(cnew) <= 1.7e308)) cnew = __builtin_nan("");
            const float cn = (float)cnew;
            const double df = (double)cn - (double)s_Cf[i];
            r2 += df * df;
            s_Cf[i] = cn;
        }
        r2 = block_sum_fixed<NT>(r2, ls);
        IDKM_LSTAMP(6);
        iters += 1;
        res = r2;
        bad = !(r2 <= 1.7e308);
        conv = r2 < tol * tol;
        done = conv || bad || iters >= max_iter;
    }

    // evaluation at C*
    {
        ++seq;
        bool done_here = false;
        if constexpr (MFMA) {
            // n*, F* and Wq on the matrix cores; the assignment (its float32 key has a prescribed form) and the
            // matrix A are outputs of the vector-ALU pass
            if (!a.assign_out && !a.A_out) {
                const bool fold = MfmaFwd<KPL>::template fill_table<NT>(s_tab, s_fac, k, s_Cf, s_mu, a.escale) &&
                                  DIST == DIST_SQL2;
                MfmaFwd<KPL>::template fill_codeword_table<NT>(s_ctab, k, s_Cf, s_mu, s_fac, fold);
                __syncthreads();
                {
                    MfmaFwd<KPL> st;
                    st.init(s_tab, s_fac, s_mu);
                    if (a.Wq_out)
                        mfma_tile_pass<KPL, DIST, NT, true>(st, s_tile, s_wn, cnt, a.escale, fold, s_ctab, s_mu,
                                                            a.Wq_out + base * D);
                    else
                        mfma_tile_pass<KPL, DIST, NT>(st, s_tile, s_wn, cnt, a.escale, fold);
                    mfma_collect<KPL, NT>(st, &s_part[0][0], fold, s_fac);
                }
                __syncthreads();
                publish_matrix();
                done_here = true;
            }
        }
        if constexpr (KB > 0) {
            {
                RowWave<KB, D, DIST, PASS_FIN> st;
                st.init(k, s_Cf, nullptr, nullptr, a.escale);
                row_tile_pass<KB, D, DIST, PASS_FIN, NT>(a, st, s_tile, nullptr, base, cnt);
                st.collect(s_rpart[tid >> 6], tid);
            }
            __syncthreads();
            publish_parts<NT / 64, WIDE1>(pa, ls, seq, &s_rpart[0][0], KMAX * ACCW, nacc);
        } else if (!done_here) {
            LaneWave<KPL, D, DIST, PASS_FIN> st;
            st.init(k, s_Cf, nullptr, nullptr);
            lane_tile_pass<KPL, D, DIST, PASS_FIN, NT>(a, st, s_tile, nullptr, base, cnt);
            publish_lane<NA, ACCW, NT>(pa, ls, seq, st.acc, k, s_acc);
        }
        if (!die_slice<NT, WIDE1>(pa, seq, nacc, ls, s_tot)) return;
    }
    // only workgroup 0 needs these totals: it writes the state and, last, the word that says the launch ran to its end (the
    // others of its die pass their slices on)
    if (wg % DIES != 0) return;
    if (!grid_totals<NT, KMAX * ACCW, KB ? 3 : 1>(pa, seq, nacc, ls, s_tot)) return;
    if (wg != 0) return;
    double empty = 0.0, wrong = 0.0;
    for (int i = tid; i < kd; i += NT) {
        const int j = i / D, rr = i - j * D;
        const double n = s_tot[j * ACCW], sv = s_tot[j * ACCW + 1 + rr];
        const double cst = (double)s_Cf[i];
        const double f = (n > 0.0) ? fast_div_d(sv, n) : cst;
        a.Cd[i] = cst;
        a.Cf[i] = s_Cf[i];
        a.Fd[i] = f;
        a.Ff[i] = (float)f;
        if (a.C_out) a.C_out[i] = s_Cf[i];
        if (!(n >= 0.0) || !(fabs(sv) <= 1.7e308)) wrong = 1.0;
        if (rr == 0) {
            a.nd[j] = n;
            if (n == 0.0) empty += 1.0;
        }
    }
    empty = block_sum_fixed<NT>(empty, ls);
    wrong = block_sum_fixed<NT>(wrong, ls);
    if (tid == 0) {
        PResult* o = pa.out;
        o->iters = iters;
        o->residual = sqrt(res);
        o->converged = conv ? 1 : 0;
        o->nonfinite = (bad || wrong > 0.0) ? 1 : 0;
        o->empty[0] = (int)(empty + 0.5);
        o->done = pa.seq_base + 1u;
    }
}

// Backward: v, the averaged iteration of Sec. 4.2 (skipped for JFB), and dW.  MFMA: the (dF/dC)^T passes run on the
// matrix cores (MfmaB2; d = 4), with NT = MT threads; the dynamic LDS then holds the tile of W padded
// by 16 zero vectors and -s^2 |w - mu|^2 of every vector, and dL/dWq -- needed by the first and the last pass only --
// is read from memory.
template <int KPL, int D, int DIST, int NT = LT, bool MFMA = false, int KB = 0>
__device__ __forceinline__ void persist_lane_bwd_body(const Args& a, const PArgs& pa) {
    static_assert(!MFMA || (D == 4 && KPL <= 4), "matrix-core pass: d = 4, k <= 256");
    constexpr int NA = KPL * D;
    constexpr int KMAX = KB > 0 ? 16 * KB : 64 * KPL;
    constexpr int KDP = KMAX * D;
    extern __shared__ float s_tile[];
    // workgroup sums of a vector-ALU pass; from the first hop on, the grid totals of the pass
    __shared__ double s_acc[KB > 0 ? KMAX : 64][KB > 0 ? D : NA];
    double* s_tot = &s_acc[0][0];
    __shared__ LShared ls;
    __shared__ double s_v[KDP], s_g[KDP];
    __shared__ double s_rn[KMAX];          // 1/(tau n_j), zero for an empty cluster
    __shared__ float s_Cf[KDP], s_Hs[KDP], s_Hv[KDP], s_Ff[KDP];
    __shared__ float s_rpart[KB > 0 ? NT / 64 : 1][KB > 0 ? KDP : 1];  // row form: totals of the wavefronts

    const int tid = threadIdx.x, wg = pa.wg, G = pa.G;
    const int k = a.k, kd = k * D;
    die_announce(pa);
    const int64_t base = (int64_t)wg * pa.per;
    int cnt = 0;
    if (base < a.m) cnt = (a.m - base < pa.per) ? (int)(a.m - base) : pa.per;
    float* s_w = s_tile;
    const float* s_gt = MFMA ? a.G + base * D : s_tile + (size_t)pa.per * D;
    load_tile<NT>(s_w, a.W + base * D, cnt * D);
    if (!MFMA) load_tile<NT>(s_tile + (size_t)pa.per * D, a.G + base * D, cnt * D);
    for (int i = tid; i < kd; i += NT) {
        s_Cf[i] = a.Cf[i];
        s_Ff[i] = a.Ff[i];
        s_Hs[i] = 0.f;
        s_Hv[i] = 0.f;
    }
    if (KB > 0)
        for (int i = kd + tid; i < KDP; i += NT) s_Cf[i] = s_Ff[i] = s_Hs[i] = 0.f;
    for (int j = tid; j < k; j += NT) {
        const double n = a.nd[j];
        s_rn[j] = (n > 0.0) ? (double)a.inv_tau / n : 0.0;
    }
    const int mode = pa.mode;
    const double tol = pa.tol;
    const int max_iter = pa.max_iter;
    if (tid == 0) ls.abort = 0;
    __syncthreads();
    if (!die_handshake(pa, ls)) return;
    // (every thread holds the state of the stop and restart rules)
    bool done = mode == BWD_JFB, conv = mode == BWD_JFB, bad = false;
    int iters = 0, attempt = 0, grow = 0, halv = 0;
    double alpha = pa.alpha, prev = __builtin_inf(), vnorm2 = 0.0, res = 0.0;
    unsigned int seq = pa.seq_base;
    // matrix-core passes: reference point, vector norms and the codeword tables (C* does not change in the backward)
    constexpr int TS = MfmaFwd<(KPL <= 4 ? KPL : 4)>::TAB_STRIDE;
    __shared__ float2 s_tab0[MFMA ? 4 * TS : 1];
    __shared__ float s_fac0[MFMA ? TS : 1];
    __shared__ float s_hsb[MFMA ? 4 * TS : 1];
    __shared__ f32x4 s_hq[MFMA ? TS : 1];
    __shared__ __align__(16) float s_part[MFMA ? NT / 64 : 1][MFMA ? 64 * KPL * 5 : 1];
    const float* s_wn = s_tile + (size_t)(pa.per + 16) * D;
    __shared__ float s_mu[4];
    bool fold = false;
    if constexpr (MFMA) {
        if (tid < D) {
            float sm = 0.f;
            for (int j = 0; j < k; ++j) sm += s_Cf[j * D + tid];
            s_mu[tid] = sm / (float)k;
        }
        float* wn = s_tile + (size_t)(pa.per + 16) * D;
        for (int i = cnt * D + tid; i < (pa.per + 16) * D; i += NT) s_tile[i] = 0.f;
        __syncthreads();
        for (int i = tid; i < pa.per + 16; i += NT) {
            float n2 = 0.f;
#pragma unroll
            for (int r = 0; r < D; ++r) {
                const float t = (s_tile[i * D + r] - s_mu[r]) * a.escale;
                n2 = fmaf(t, t, n2);
            }
            wn[i] = -n2;
        }
    }

    if constexpr (MFMA)
        fold = MfmaFwd<KPL>::template fill_table<NT>(s_tab0, s_fac0, k, s_Cf, s_mu, a.escale) && DIST == DIST_SQL2;
    // Hop-1 store of a matrix-core pass: wavefront totals add up in wavefront order (float64), then the codeword
    // term and the fold factor (see MfmaB2).
    auto publish_matrix = [&]() {
        if constexpr (MFMA) {
            unsigned long long* dst = own_line<false>(pa, seq, kd);
            for (int idx = tid; idx < kd; idx += NT) {
                const int j = idx >> 2, r = idx & 3;
                double sw = 0.0, st1 = 0.0;
#pragma unroll
                for (int w = 0; w < NT / 64; ++w) {
                    sw += (double)s_part[w][j * 5 + 1 + r];
                    st1 += (double)s_part[w][j * 5];
                }
                const double o = sw - (double)(s_Cf[idx] - s_mu[r]) * st1;
                put_sum<false>(ls, dst, kd, seq, idx, fold ? o * (double)s_fac0[j] : o);
            }
        }
    };

    // B1
    {
        ++seq;
        if constexpr (MFMA) {
            {
                MfmaB2<KPL> st;
                st.init(s_tab0, s_fac0, s_hsb, s_hq, s_mu);
                mfma_b1_tile_pass<KPL, DIST, NT>(st, s_tile, s_wn, s_gt, cnt, a.escale, a.inv_tau, fold);
                mfma_b2_collect<KPL, NT>(st, &s_part[0][0]);
            }
            __syncthreads();
            publish_matrix();
        } else if constexpr (KB > 0) {
            {
                RowWave<KB, D, DIST, PASS_B1> st;
                st.init(k, s_Cf, s_Hs, s_Ff, a.escale);
                row_tile_pass<KB, D, DIST, PASS_B1, NT>(a, st, s_w, s_gt, base, cnt);
                st.collect(s_rpart[tid >> 6], tid);
            }
            __syncthreads();
            publish_parts<NT / 64>(pa, ls, seq, &s_rpart[0][0], KDP, kd);
        } else {
            LaneWave<KPL, D, DIST, PASS_B1> st;
            st.init(k, s_Cf, s_Hs, s_Ff, a.escale);
            lane_tile_pass<KPL, D, DIST, PASS_B1, NT>(a, st, s_w, s_gt, base, cnt);
            publish_lane<NA, D, NT>(pa, ls, seq, st.acc, k, s_acc);
        }
        if (!die_slice<NT>(pa, seq, kd, ls, s_tot) || !grid_totals<NT, KDP, KB ? 3 : 1>(pa, seq, kd, ls, s_tot)) return;
        // every workgroup holds the whole of v and starts the solve at g = v
        double v2 = 0.0;
        for (int i = tid; i < kd; i += NT) {
            const double v = s_tot[i];
            s_v[i] = v;
            s_g[i] = v;
            v2 += v * v;
            s_Hs[i] = s_Hv[i] = (float)(v * s_rn[i / D]);
        }
        vnorm2 = block_sum_fixed<NT>(v2, ls);  // squared norms throughout
        if (!(vnorm2 <= 1.7e308)) {
            bad = true;
            done = true;
        }
    }

    while (!done) {
        ++seq;
        if constexpr (MFMA) {
            MfmaB2<KPL>::template fill_cotangent<NT>(s_hsb, s_hq, k, s_Hs, s_Ff, s_mu, a.escale);
            __syncthreads();
            {
                MfmaB2<KPL> st;
                st.init(s_tab0, s_fac0, s_hsb, s_hq, s_mu);
                mfma_b2_tile_pass<KPL, DIST, NT>(st, s_tile, s_wn, cnt, a.escale, fold);
                mfma_b2_collect<KPL, NT>(st, &s_part[0][0]);
            }
            __syncthreads();
            publish_matrix();
        } else if constexpr (KB > 0) {
            {
                RowWave<KB, D, DIST, PASS_B2> st;
                st.init(k, s_Cf, s_Hs, s_Ff, a.escale);
                row_tile_pass<KB, D, DIST, PASS_B2, NT>(a, st, s_w, s_gt, base, cnt);
                st.collect(s_rpart[tid >> 6], tid);
            }
            __syncthreads();
            publish_parts<NT / 64>(pa, ls, seq, &s_rpart[0][0], KDP, kd);
        } else {
            LaneWave<KPL, D, DIST, PASS_B2> st;
            st.init(k, s_Cf, s_Hs, s_Ff, a.escale);
            lane_tile_pass<KPL, D, DIST, PASS_B2, NT>(a, st, s_w, s_gt, base, cnt);
            publish_lane<NA, D, NT>(pa, ls, seq, st.acc, k, s_acc);
        }
        if (!die_slice<NT>(pa, seq, kd, ls, s_tot) || !grid_totals<NT, KDP, KB ? 3 : 1>(pa, seq, kd, ls, s_tot)) return;
        double d2 = 0.0;
        for (int i = tid; i < kd; i += NT) {
            const double g = s_g[i];
            const double gn = alpha * (s_v[i] + s_tot[i]) + (1.0 - alpha) * g;
            const double df = gn - g;
            d2 += df * df;
            s_g[i] = gn;
        }
        d2 = block_sum_fixed<NT>(d2, ls);
        const double dn = d2;  // squared step norm: every comparison below is between squares
        bool restart = false, diverged = false;
        attempt += 1;
        if (!(dn <= 1.7e308)) {
            diverged = true;
        } else if (dn <= tol * tol * vnorm2) {
            conv = true;
            done = true;
        } else {
            grow = (dn > prev) ? grow + 1 : 0;
            if (grow >= 5) diverged = true;
            prev = dn;
        }
        if (!done && !diverged && attempt >= max_iter) done = true;
        if (diverged) {
            if (halv < 6) {
                restart = true;
            } else {
                done = true;
                if (!(dn <= 1.7e308)) bad = true;  // every damping factor tried ended in a non-finite step
            }
        }
        iters += 1;
        res = dn;
        if (restart) {
            alpha *= 0.5;
            halv += 1;
            attempt = 0;
            grow = 0;
            prev = __builtin_inf();
        }
        for (int i = tid; i < kd; i += NT) {  // (a thread's own elements)
            if (restart) s_g[i] = s_v[i];
            s_Hs[i] = restart ? s_Hv[i] : (float)(s_g[i] * s_rn[i / D]);
        }
        __syncthreads();
    }

    // B3
    if constexpr (MFMA) {
        // the output tables take the place of the per-wavefront partial sums, which no later pass needs
        f32x4* s_hc = reinterpret_cast<f32x4*>(&s_part[0][0]);
        static_assert(sizeof(s_part) >= 2 * TS * sizeof(f32x4), "output tables do not fit");
        MfmaB2<KPL>::template fill_cotangent<NT>(s_hsb, s_hq, k, s_Hs, s_Ff, s_mu, a.escale);
        MfmaB3<KPL>::template fill_output_tables<NT>(s_hc, k, s_Hs, s_Cf, s_mu, s_fac0, fold, a.tau,
                                                     DIST == DIST_SQL2 ? 2.f : a.escale);
        __syncthreads();
        MfmaB3<KPL> st;
        st.init(s_tab0, s_fac0, s_hsb, s_hq, s_hc, s_mu);
        mfma_b3_tile_pass<KPL, DIST, NT>(st, s_tile, s_wn, s_gt, a.dW_out + base * D, cnt, a.escale, a.inv_tau, fold);
    } else if constexpr (KB > 0) {
        RowWave<KB, D, DIST, PASS_B3> st;
        st.init(k, s_Cf, s_Hs, s_Ff, a.escale);
        row_tile_pass<KB, D, DIST, PASS_B3, NT>(a, st, s_w, s_gt, base, cnt);
    } else {
        LaneWave<KPL, D, DIST, PASS_B3> st;
        st.init(k, s_Cf, s_Hs, s_Ff, a.escale);
        lane_tile_pass<KPL, D, DIST, PASS_B3, NT>(a, st, s_w, s_gt, base, cnt);
    }
    if (wg == 0)
        for (int i = tid; i < kd; i += NT) {
            a.gd[i] = s_g[i];
            a.vd[i] = s_v[i];
            a.Hs[i] = s_Hs[i];
        }
    if (wg == G - 1 && tid == 0) {
        PResult* o = pa.out;
        o->iters = iters;
        o->converged = conv ? 1 : 0;
        o->residual = sqrt(res);
        o->alpha = alpha;
        o->vnorm = sqrt(vnorm2);
        o->halvings = halv;
        o->nonfinite = bad ? 1 : 0;
        o->done = pa.seq_base + 1u;
    }
}

// Launch forms: one team per grid, or one team per batched problem (see persist_small.hpp).
template <int KPL, int D, int DIST>
__global__ __launch_bounds__(LT) void persist_lane_fwd(const Args a, const PArgs pa_in) {
    PArgs pa = pa_in;
    pa.wg = blockIdx.x;
    pa.G = gridDim.x;
    persist_lane_fwd_body<KPL, D, DIST>(a, pa);
}
template <int KPL, int D, int DIST>
__global__ __launch_bounds__(LT) void persist_lane_fwd_batch(const BatchItem* items, const unsigned short* item_of_wg) {
    const BatchItem& it = items[item_of_wg[blockIdx.x]];
    const Args a = it.a;
    PArgs pa = it.p;
    pa.wg = (int)blockIdx.x - it.wg_begin;
    pa.G = it.wg_count;
    persist_lane_fwd_body<KPL, D, DIST>(a, pa);
}
// Forward solve with the loop on the matrix cores (d = 4): MT threads, see persist_lane_fwd_body.
template <int KPL, int DIST>
__global__ __launch_bounds__(MT) void persist_mfma_fwd(const Args a, const PArgs pa_in) {
    PArgs pa = pa_in;
    pa.wg = blockIdx.x;
    pa.G = gridDim.x;
    persist_lane_fwd_body<KPL, 4, DIST, MT, true>(a, pa);
}
template <int KPL, int DIST>
__global__ __launch_bounds__(MT) void persist_mfma_fwd_batch(const BatchItem* items, const unsigned short* item_of_wg) {
    const BatchItem& it = items[item_of_wg[blockIdx.x]];
    const Args a = it.a;
    PArgs pa = it.p;
    pa.wg = (int)blockIdx.x - it.wg_begin;
    pa.G = it.wg_count;
    persist_lane_fwd_body<KPL, 4, DIST, MT, true>(a, pa);
}
// Backward with the (dF/dC)^T passes on the matrix cores (d = 4), see persist_lane_bwd_body.  The plain norm's pass
// keeps more per lane than 256 registers hold at k = 256 (energies and u for 16 x 256 pairs, the accumulators, the
// row minima): that kernel runs one wavefront per SIMD, which may use the whole register file.
template <int KPL, int DIST>
constexpr int mfma_bwd_threads() {
    return (DIST == DIST_L2 && KPL == 4) ? 256 : MT;
}
template <int KPL, int DIST>
__global__ __launch_bounds__((mfma_bwd_threads<KPL, DIST>())) void persist_mfma_bwd(const Args a, const PArgs pa_in) {
    PArgs pa = pa_in;
    pa.wg = blockIdx.x;
    pa.G = gridDim.x;
    persist_lane_bwd_body<KPL, 4, DIST, mfma_bwd_threads<KPL, DIST>(), true>(a, pa);
}
template <int KPL, int DIST>
__global__ __launch_bounds__((mfma_bwd_threads<KPL, DIST>())) void persist_mfma_bwd_batch(const BatchItem* items, const unsigned short* item_of_wg) {
    const BatchItem& it = items[item_of_wg[blockIdx.x]];
    const Args a = it.a;
    PArgs pa = it.p;
    pa.wg = (int)blockIdx.x - it.wg_begin;
    pa.G = it.wg_count;
    persist_lane_bwd_body<KPL, 4, DIST, mfma_bwd_threads<KPL, DIST>(), true>(a, pa);
}
template <int KPL, int D, int DIST>
__global__ __launch_bounds__(LT) void persist_lane_bwd(const Args a, const PArgs pa_in) {
    PArgs pa = pa_in;
    pa.wg = blockIdx.x;
    pa.G = gridDim.x;
    persist_lane_bwd_body<KPL, D, DIST>(a, pa);
}
template <int KPL, int D, int DIST>
__global__ __launch_bounds__(LT) void persist_lane_bwd_batch(const BatchItem* items, const unsigned short* item_of_wg) {
    const BatchItem& it = items[item_of_wg[blockIdx.x]];
    const Args a = it.a;
    PArgs pa = it.p;
    pa.wg = (int)blockIdx.x - it.wg_begin;
    pa.G = it.wg_count;
    persist_lane_bwd_body<KPL, D, DIST>(a, pa);
}

// The row <-> vector form (d = 1 and 2, and the forward solve for d = 8; up to 16 KB codewords).
template <int KB, int D, int DIST>
__global__ __launch_bounds__(RT) void persist_row_fwd(const Args a, const PArgs pa_in) {
    PArgs pa = pa_in;
    pa.wg = blockIdx.x;
    pa.G = gridDim.x;
    persist_lane_fwd_body<1, D, DIST, RT, false, KB>(a, pa);
}
template <int KB, int D, int DIST>
__global__ __launch_bounds__(RT) void persist_row_fwd_batch(const BatchItem* items, const unsigned short* item_of_wg) {
    const BatchItem& it = items[item_of_wg[blockIdx.x]];
    const Args a = it.a;
    PArgs pa = it.p;
    pa.wg = (int)blockIdx.x - it.wg_begin;
    pa.G = it.wg_count;
    persist_lane_fwd_body<1, D, DIST, RT, false, KB>(a, pa);
}
template <int KB, int D, int DIST>
__global__ __launch_bounds__(RT) void persist_row_bwd(const Args a, const PArgs pa_in) {
    PArgs pa = pa_in;
    pa.wg = blockIdx.x;
    pa.G = gridDim.x;
    persist_lane_bwd_body<1, D, DIST, RT, false, KB>(a, pa);
}
template <int KB, int D, int DIST>
__global__ __launch_bounds__(RT) void persist_row_bwd_batch(const BatchItem* items, const unsigned short* item_of_wg) {
    const BatchItem& it = items[item_of_wg[blockIdx.x]];
    const Args a = it.a;
    PArgs pa = it.p;
    pa.wg = (int)blockIdx.x - it.wg_begin;
    pa.G = it.wg_count;
    persist_lane_bwd_body<1, D, DIST, RT, false, KB>(a, pa);
}

}  // namespace idkm
