// The stored form of a quantised layer (Sec. 3: every sub-vector is replaced by one of k = 2^b codewords):
// b-bit codes in one little-endian bit stream, and the reconstruction q(W, C) from codes and codebook.
#include "dispatch.h"

namespace idkm {

// Thread t packs codes [32 t, 32 t + 32) into exactly `bits` words [bits t, bits t + bits).
__global__ __launch_bounds__(256) void k_pack_codes(const int32_t* __restrict__ assign, int64_t m, int bits,
                                                     uint32_t* __restrict__ words, int64_t nwords) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t first = t * 32;
    if (first >= m) return;
    int32_t c[32];
    if (first + 32 <= m) {
        const int4* src = reinterpret_cast<const int4*>(assign + first);  // 128-byte aligned: first is a multiple of 32
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int4 v = src[q];
            c[4 * q] = v.x;
            c[4 * q + 1] = v.y;
            c[4 * q + 2] = v.z;
            c[4 * q + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 32; ++i) c[i] = (first + i < m) ? assign[first + i] : 0;
    }
    const uint32_t mask = (1u << bits) - 1u;
    unsigned long long buf = 0ull;
    int fill = 0;
    int64_t w = t * bits;
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        buf |= (unsigned long long)((uint32_t)c[i] & mask) << fill;
        fill += bits;
        if (fill >= 32) {
            if (w < nwords) words[w] = (uint32_t)buf;
            ++w;
            buf >>= 32;
            fill -= 32;
        }
    }
}

// Thread i reads code i and copies codeword row C[code] to out[i]; a code >= k (not a valid stream) gives NaN.
// Serves the row lengths and the alignments that k_unpack_quads does not.
__global__ __launch_bounds__(256) void k_unpack_quantize(const uint32_t* __restrict__ words, int64_t nwords, int64_t m,
                                                          int bits, const float* __restrict__ C, int k, int d,
                                                          float* __restrict__ out, int c_in_lds) {
    extern __shared__ float s_C[];
    if (c_in_lds) {
        for (int i = threadIdx.x; i < k * d; i += 256) s_C[i] = C[i];
        __syncthreads();
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    const int64_t off = i * bits;
    const int64_t w = off >> 5;
    const int sh = (int)(off & 31);
    unsigned long long win = words[w];
    if (sh + bits > 32 && w + 1 < nwords) win |= (unsigned long long)words[w + 1] << 32;
    const uint32_t code = (uint32_t)(win >> sh) & ((1u << bits) - 1u);
    const bool ok = code < (uint32_t)k;
    const float* row = (c_in_lds ? s_C : C) + (size_t)(ok ? code : 0u) * d;
    for (int r = 0; r < d; ++r) out[i * d + r] = ok ? row[r] : __builtin_nanf("");
}

// The same with one 16-byte store per thread and turn: four codes for d = 1, two for d = 2, a quarter of a row for d a
// multiple of four (DV = 4).  Bound by the stores: with one 4-byte store per thread and one copy of the codebook into LDS
// per 256 codes, a 16.8 M-code layer (k = 16, d = 1) took 36.8 us (2.0 TB/s); the workgroups now stay and take quads in turn, and it
// takes about 15 (5 TB/s, the rate of a plain copy).  `out` is 16-byte aligned.
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int DV>
__global__ __launch_bounds__(256) void k_unpack_quads(const uint32_t* __restrict__ words, int64_t nwords, int64_t m, int bits,
                                                       const float* __restrict__ C, int k, int d, float* __restrict__ out) {
    extern __shared__ __align__(16) float s_C[];
    for (int i = threadIdx.x; i < k * d; i += 256) s_C[i] = C[i];
    __syncthreads();
    constexpr int NC = 4 / DV;                // codes per quad
    const int qpr = DV == 4 ? d / 4 : 1;      // quads per row
    const int64_t nq = DV == 4 ? m * qpr : m / NC;
    const uint32_t mask = (1u << bits) - 1u;
    const float nan = __builtin_nanf("");
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < nq; q += step) {
        const int64_t i = DV == 4 ? (qpr == 1 ? q : (nq >> 31) == 0 ? (int64_t)((uint32_t)q / (uint32_t)qpr) : q / qpr) : q * NC;
        const int64_t off = i * bits, w = off >> 5;
        const int sh = (int)(off & 31);
        // the NC codes lie in at most 31 + 4 x 10 bits: up to three words, brought down to 64 bits (a word is read only
        // when one of these codes, which exist, has bits in it)
        unsigned long long win = words[w];
        if (sh + NC * bits > 32) win |= (unsigned long long)words[w + 1] << 32;
        win >>= sh;
        if (NC > 1 && sh + NC * bits > 64) win |= (unsigned long long)words[w + 2] << (64 - sh);
        f32x4 v;
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            const uint32_t code = (uint32_t)(win >> (e * bits)) & mask;
            const bool ok = code < (uint32_t)k;
            const uint32_t row = ok ? code : 0u;
            if constexpr (DV == 4) {
                const f32x4 x = reinterpret_cast<const f32x4*>(s_C)[(int)row * qpr + (qpr == 1 ? 0 : (int)(q - i * qpr))];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = ok ? x[r] : nan;
            } else {
#pragma unroll
                for (int r = 0; r < DV; ++r) v[e * DV + r] = ok ? s_C[row * DV + r] : nan;
            }
        }
        reinterpret_cast<f32x4*>(out)[q] = v;
    }
    // the up to NC - 1 codes behind the last whole quad
    const int64_t i = nq * NC + threadIdx.x;
    if (NC > 1 && blockIdx.x == 0 && i < m) {
        const int64_t off = i * bits, w = off >> 5;
        const int sh = (int)(off & 31);
        unsigned long long win = words[w];
        if (sh + bits > 32) win |= (unsigned long long)words[w + 1] << 32;
        const uint32_t code = (uint32_t)(win >> sh) & mask;
        for (int r = 0; r < d; ++r) out[i * d + r] = code < (uint32_t)k ? s_C[code * d + r] : nan;
    }
}

void launch_pack_codes(const int32_t* assign, int64_t m, int bits, uint32_t* words, int64_t nwords, hipStream_t s) {
    const int64_t threads = (m + 31) / 32;
    const unsigned grid = (unsigned)((threads + 255) / 256);
    hipLaunchKernelGGL(k_pack_codes, dim3(grid), dim3(256), 0, s, assign, m, bits, words, nwords);
}

void launch_unpack_quantize(const uint32_t* words, int64_t nwords, int64_t m, int bits, const float* C, int k, int d,
                            float* out, hipStream_t s) {
    const size_t cbytes = (size_t)k * d * sizeof(float);
    const int in_lds = cbytes <= 32 * 1024 ? 1 : 0;
    if (in_lds && (d == 1 || d == 2 || d % 4 == 0) && (reinterpret_cast<uintptr_t>(out) & 15u) == 0) {
        const int64_t nq = d % 4 == 0 ? m * (d / 4) : m / (4 / d);
        int64_t grid = (nq + 255) / 256;
        if (grid < 1) grid = 1;
        if (grid > 2048) grid = 2048;  // eight workgroups per compute unit
        auto fn = d == 1 ? k_unpack_quads<1> : (d == 2 ? k_unpack_quads<2> : k_unpack_quads<4>);
        hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(256), cbytes, s, words, nwords, m, bits, C, k, d, out);
        return;
    }
    const unsigned grid = (unsigned)((m + 255) / 256);
    hipLaunchKernelGGL(k_unpack_quantize, dim3(grid), dim3(256), in_lds ? cbytes : 0, s, words, nwords, m, bits, C, k, d,
                       out, in_lds);
}

}  // namespace idkm
