// sj_front.hip -- Section 4's ip-distance front ends on gfx950: the rows the
// join's matrix-core kernels read for cosine similarity (f = g = x / ||x||)
// and for the Hamming distance (+-1 codes of {0, 1}^d).  Both are O(n d) passes
// over the rows, bound by HBM.
#include "sj_internal.h"

namespace sjk {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------------ cosine
// Exact value of element k of a row of dtype DT.
template <int DT>
__device__ __forceinline__ double elem_value(const uint8_t *row, uint32_t k)
{
    if constexpr (DT == DT_I8) {
        return (double)(int8_t)row[k];
    } else if constexpr (DT == DT_F16) {
        return (double)(float)((const _Float16 *)row)[k];
    } else {
        const uint32_t b = (uint32_t)((const uint16_t *)row)[k] << 16;
        return (double)__uint_as_float(b);
    }
}

// The nearest value with P significand bits (binary16: P = 11, smallest
// normal exponent -14; bfloat16: P = 8, -126) of a double, ties to even, as a
// 16-bit pattern.  From the double's bit pattern: the value is sig * 2^e2
// with an integer significand; the result's quantum is 2^q with q = max(lg -
// (P - 1), EMIN - (P - 1)) where lg = floor(log2 |v|); the bits of sig below
// the quantum are dropped and decide the rounding (above half: up; exactly
// half: up when the kept part is odd).  The pattern is then
// ((q - EMIN + P) << (P - 1)) + kept - 2^(P - 1) for normal and subnormal
// results alike, a kept significand of 2^P carrying into the exponent field;
// |v| at or above 2^(EMAX + 1) is infinity.
template <int P, int EMIN, int EMAX>
__device__ __forceinline__ uint16_t round_double_rne(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint16_t sign = (uint16_t)((b >> 48) & 0x8000u);
    const uint32_t E = (uint32_t)(b >> 52) & 0x7ffu;
    const uint64_t frac = b & ((1ull << 52) - 1);
    if (E == 0 && frac == 0)
        return sign;
    const uint64_t sig = E == 0 ? frac : (frac | (1ull << 52));
    const int e2 = (E == 0 ? 1 : (int)E) - 1075;
    const int lg = 63 - __clzll((long long)sig) + e2;
    if (lg > EMAX)
        return sign | (uint16_t)(((EMAX - EMIN + 2) << (P - 1)));   // infinity
    const int q = lg - (P - 1) > EMIN - (P - 1) ? lg - (P - 1) : EMIN - (P - 1);
    const int shift = q - e2;   // > 0: a double has more significand bits
    if (shift >= 64)
        return sign;            // far below half the smallest subnormal
    const uint64_t kept0 = sig >> shift;
    const uint64_t rem = sig & ((1ull << shift) - 1);
    const uint64_t half = 1ull << (shift - 1);
    const uint64_t kept = kept0 + ((rem > half || (rem == half && (kept0 & 1))) ? 1 : 0);
    const uint32_t bits =
        ((uint32_t)(q - EMIN + P) << (P - 1)) + (uint32_t)kept - (1u << (P - 1));
    return sign | (uint16_t)bits;
}

// Norm of every row: sqrt of the sum of the squares in double, ascending k
// (one thread per row; every square of a decoded element is exact).
template <int DT>
__global__ void __launch_bounds__(256) row_norms_f64(const uint8_t *X, uint32_t n, uint32_t d,
                                                     uint32_t row_bytes, double *norm)
{
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n)
        return;
    const uint8_t *row = X + (size_t)i * row_bytes;
    double s = 0.0;
    for (uint32_t k = 0; k < d; ++k) {
        const double x = elem_value<DT>(row, k);
        s += x * x;
    }
    norm[i] = __builtin_sqrt(s);
}

// y = x / ||x|| rounded to the output type (binary16 for fp16 and int8 rows,
// bfloat16 for bfloat16 rows); a row of norm 0 is written as +0.
template <int DT>
__global__ void __launch_bounds__(256) normalize_rows(const uint8_t *X, uint32_t n, uint32_t d,
                                                      uint32_t row_bytes, const double *norm,
                                                      uint16_t *Y)
{
    const uint64_t total = (uint64_t)n * d;
    for (uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x; t < total;
         t += (uint64_t)gridDim.x * 256) {
        const uint32_t i = (uint32_t)(t / d), k = (uint32_t)(t - (uint64_t)i * d);
        const double nr = norm[i];
        uint16_t y = 0;
        if (nr != 0.0) {
            const double q = elem_value<DT>(X + (size_t)i * row_bytes, k) / nr;
            y = DT == DT_BF16 ? round_double_rne<8, -126, 127>(q) : round_double_rne<11, -14, 15>(q);
        }
        Y[t] = y;
    }
}

template <int DT>
static hipError_t normalize_dt(const uint8_t *X, uint32_t n, uint32_t d, double *norm, uint16_t *Y,
                               hipStream_t st)
{
    const uint32_t row_bytes = d * (DT == DT_I8 ? 1u : 2u);
    hipLaunchKernelGGL((row_norms_f64<DT>), dim3((n + 255) / 256), dim3(256), 0, st, X, n, d,
                       row_bytes, norm);
    const uint64_t total = (uint64_t)n * d;
    const uint64_t blocks = (total + 255) / 256;
    hipLaunchKernelGGL((normalize_rows<DT>), dim3((uint32_t)(blocks < 65536 ? blocks : 65536)),
                       dim3(256), 0, st, X, n, d, row_bytes, norm, Y);
    return hipGetLastError();
}

hipError_t launch_normalize(int dtype, const void *X, uint32_t n, uint32_t d, double *norm,
                            void *Y, hipStream_t stream)
{
    if (n == 0 || d == 0)
        return hipSuccess;
    const uint8_t *x = (const uint8_t *)X;
    uint16_t *y = (uint16_t *)Y;
    switch (dtype) {
    case DT_F16: return normalize_dt<DT_F16>(x, n, d, norm, y, stream);
    case DT_BF16: return normalize_dt<DT_BF16>(x, n, d, norm, y, stream);
    case DT_I8: return normalize_dt<DT_I8>(x, n, d, norm, y, stream);
    }
    return hipErrorInvalidValue;
}

// ----------------------------------------------------------------- Hamming
// Bit rows unpacked to +-1 as 4-bit floats (E2M1: +1 = 0x2, -1 = 0xa, 0 = 0x0):
// x_m = 0 gives +1, 1 gives -1, so <f(x), f(y)> = d - 2 Hamming(x, y), one
// matrix-core multiply-add per coordinate where Section 4's f(x) = (x, 1 - x),
// g(y) = (1 - y, y) takes two, and half a byte per coordinate where int8 rows
// of (x, 1 - x) take two bytes.  A thread writes 16 bytes: 32 coordinates from
// four bytes of bits.  2^team_lg threads share a row (no division per thread).
// Bound by HBM (d / 8 bytes read, d / 2 written per row); 65536 rows of 256
// bits: 3 us, where the int8 form took 31 us.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256) unpack_hamming(const uint8_t *bits, uint32_t n, uint32_t d,
                                                      uint32_t out_bytes, uint32_t team_lg,
                                                      uint8_t *out)
{
    const uint32_t row = blockIdx.x * (256u >> team_lg) + (threadIdx.x >> team_lg);
    if (row >= n)
        return;
    const uint32_t in_stride = (d + 7) / 8, team = 1u << team_lg;
    const uint8_t *rb = bits + (size_t)row * in_stride;
    uint8_t *o = out + (size_t)row * out_bytes;
    for (uint32_t c = threadIdx.x & (team - 1); c < out_bytes / 16; c += team) {
        u32x4 v;
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
            const uint32_t byte = 4 * c + w;
            // bit k of the byte to bit 4 k, then to the nibble's sign
            uint32_t x = byte < in_stride ? rb[byte] : 0u;
            x = (x | (x << 12)) & 0x000f000fu;
            x = (x | (x << 6)) & 0x03030303u;
            x = (x | (x << 3)) & 0x11111111u;
            const uint32_t m0 = 8 * byte;   // the word's first coordinate
            const uint32_t valid = m0 + 8 <= d ? 0xffffffffu
                                   : m0 >= d   ? 0u
                                               : (1u << (4 * (d - m0))) - 1u;
            v[w] = (0x22222222u | (x << 3)) & valid;
        }
        *(u32x4 *)(o + 16 * c) = v;
    }
}

hipError_t launch_unpack_hamming(const uint8_t *bits, uint32_t n, uint32_t d, uint32_t out_bytes,
                                 uint8_t *out, hipStream_t stream)
{
    if (n == 0)
        return hipSuccess;
    uint32_t team_lg = 0;
    while (team_lg < 8 && (16u << team_lg) < out_bytes)
        ++team_lg;
    const uint64_t rows = 256u >> team_lg;
    hipLaunchKernelGGL(unpack_hamming, dim3((uint32_t)((n + rows - 1) / rows)), dim3(256), 0,
                       stream, bits, n, d, out_bytes, team_lg, out);
    return hipGetLastError();
}

}  // namespace sjk
