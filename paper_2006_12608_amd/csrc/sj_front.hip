// sj_front.hip -- Section 4's ip-distance front ends on gfx950: the rows the
// join's matrix-core kernels read for cosine similarity (f = g = x / ||x||)
// and for the Hamming distance (+-1 codes of {0, 1}^d).  Both are O(n d) passes
// over the rows, bound by HBM.
#include "sj_internal.h"

#include <type_traits>

namespace sjk {

// ------------------------------------------------------------------ cosine
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

// One 16-byte chunk of a row: E elements, chunk c holds elements [E c, E c + E),
// zeros past d.  VEC: rows are 16-byte aligned and d is a multiple of E;
// otherwise whole chunks are one load of 16 bytes at the elements' alignment and
// only the row's last, partial chunk is loaded element by element.
template <int DT>
struct FrontChunk {
    static constexpr int E = DT == DT_I8 ? 16 : 8;
    template <bool VEC>
    static __device__ __forceinline__ i32x4 load(const uint8_t *row, uint32_t d, uint32_t c)
    {
        if constexpr (VEC) {
            return E * c < d ? *(const i32x4 *)(row + 16 * (size_t)c) : i32x4{0, 0, 0, 0};
        } else {
            if (E * c + E <= d) {
                i32x4 v;
                __builtin_memcpy(&v, row + 16 * (size_t)c, 16);
                return v;
            }
            uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t k = E * c + e;
                if constexpr (DT == DT_I8)
                    w[e >> 2] |= k < d ? (uint32_t)row[k] << (8 * (e & 3)) : 0u;
                else
                    w[e >> 1] |= k < d ? (uint32_t)((const uint16_t *)row)[k] << (16 * (e & 1)) : 0u;
            }
            return i32x4{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
        }
    }
    // exact value of element e
    static __device__ __forceinline__ double at(const i32x4 &v, int e)
    {
        if constexpr (DT == DT_I8)
            return (double)(int8_t)((uint32_t)v[e >> 2] >> (8 * (e & 3)));
        const uint32_t h = ((uint32_t)v[e >> 1] >> (16 * (e & 1))) & 0xffffu;
        if constexpr (DT == DT_F16)
            return (double)(float)__builtin_bit_cast(_Float16, (uint16_t)h);
        else
            return (double)__uint_as_float(h << 16);
    }
};

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

// x / ||x|| as the output type's 16 bits: the double quotient x / nr rounded to
// nearest even, without a division for nearly every element.  p = x * (1 / nr)
// is within 2^-52 of the quotient; rounded to fp32 and then to P bits it gives
// the quotient's P bits unless the fp32 value is a midpoint of two P-bit values
// (any other fp32 value lies on the side of the midpoint that both p and the
// quotient lie on).  Midpoints, results below the output type's normal range
// and anything not finite take the division.
template <int DT>
__device__ __forceinline__ uint16_t unit_value(double x, double nr, double inv)
{
    const float f = (float)(x * inv);
    const uint32_t b = __float_as_uint(f), mag = b & 0x7fffffffu;
    if constexpr (DT == DT_BF16) {
        const bool sure = mag == 0 ||
                          (mag >= 0x00800000u && mag <= 0x40000000u && (b & 0xffffu) != 0x8000u);
        if (__builtin_expect(sure, 1))
            return (uint16_t)((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
        return round_double_rne<8, -126, 127>(x / nr);
    } else {
        const bool sure = mag == 0 ||
                          (mag >= 0x38800000u && mag <= 0x40000000u && (b & 0x1fffu) != 0x1000u);
        if (__builtin_expect(sure, 1))
            return __builtin_bit_cast(uint16_t, (_Float16)f);
        return round_double_rne<11, -14, 15>(x / nr);
    }
}

// The double held by lane Q of this lane's group of four.
template <int Q>
__device__ __forceinline__ double quad_value(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x55 * Q, 0xf, 0xf, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x55 * Q, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Y = the rows of X divided by their norms.  Four lanes share a row (16 rows per
// wave): lane q of the group loads chunks q, q + 4, ... (64 contiguous bytes of
// each row per step).  The norm's double sum runs through the elements in
// ascending order: in turn q = 0 .. 3 every lane adds its own chunk to the sum
// so far and the group keeps lane q's.  Then each lane scales its chunks and
// writes them.  A row of norm 0 is written as +0.  Bound by HBM: one pass over X
// (the second reading comes from cache) and one over Y.  A sj_normalize call on
// 262144 x 256 fp16 rows takes 94 us; with a thread per row for the norms (its
// lanes 512 bytes apart) and a thread per element with a double division and a
// 64-bit index division each it took 437 us.  100000 rows of 250: 196 -> 66 us.
template <int DT, bool VEC>
__global__ void __launch_bounds__(256) normalize_rows(const uint8_t *X, uint32_t n, uint32_t d,
                                                      uint16_t *Y)
{
    typedef FrontChunk<DT> C;
    constexpr int E = C::E;
    const uint32_t i = blockIdx.x * 64 + (threadIdx.x >> 2), q = threadIdx.x & 3;
    const bool mine = i < n;
    const uint32_t r = mine ? i : n - 1;   // lanes past the rows follow the last one
    const uint8_t *row = X + (size_t)r * d * (DT == DT_I8 ? 1 : 2);
    const uint32_t nch = (d + E - 1) / E;
    double s = 0.0;
    i32x4 v = C::template load<VEC>(row, d, q);
    for (uint32_t c0 = 0; c0 < nch; c0 += 4) {
        const i32x4 nx = C::template load<VEC>(row, d, c0 + 4 + q);
        double x[E];
#pragma unroll
        for (int e = 0; e < E; ++e)
            x[e] = C::at(v, e);
        auto turn = [&](auto Q) {
            double t = s;
#pragma unroll
            for (int e = 0; e < E; ++e)
                t += x[e] * x[e];   // exact squares
            s = quad_value<decltype(Q)::value>(t);
        };
        turn(std::integral_constant<int, 0>{});
        turn(std::integral_constant<int, 1>{});
        turn(std::integral_constant<int, 2>{});
        turn(std::integral_constant<int, 3>{});
        v = nx;
    }
    if (!mine)
        return;
    const double nr = __builtin_sqrt(s), inv = 1.0 / nr;
    const bool zero = nr == 0.0;
    uint16_t *yr = Y + (size_t)i * d;
    for (uint32_t c = q; c < nch; c += 4) {
        const i32x4 xv = C::template load<VEC>(row, d, c);
        uint16_t y[E];
#pragma unroll
        for (int e = 0; e < E; ++e)
            y[e] = zero ? (uint16_t)0 : unit_value<DT>(C::at(xv, e), nr, inv);
        if constexpr (VEC) {
#pragma unroll
            for (int k = 0; k < E / 8; ++k) {
                u16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    o[e] = y[8 * k + e];
                *(u16x8 *)(yr + E * c + 8 * k) = o;
            }
        } else if (E * c + E <= d) {
            __builtin_memcpy(yr + E * c, y, sizeof y);
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (E * c + e < d)
                    yr[E * c + e] = y[e];
        }
    }
}

static const uint64_t kRowsPerLaunch = 1ull << 29;

template <int DT>
static hipError_t normalize_dt(const uint8_t *X, uint32_t n, uint32_t d, uint16_t *Y,
                               hipStream_t st)
{
    // whole 16-byte chunks, both sides aligned
    const bool vec = d % FrontChunk<DT>::E == 0 && (((uintptr_t)X | (uintptr_t)Y) & 15) == 0;
    // (a launch holds fewer than 2^32 threads; 2^29 rows are a multiple of 16 bytes)
    for (uint64_t r = 0; r < n; r += kRowsPerLaunch) {
        const uint32_t m = (uint32_t)(n - r < kRowsPerLaunch ? n - r : kRowsPerLaunch);
        const dim3 grid((m + 63) / 64);
        const uint8_t *x = X + (size_t)r * d * (DT == DT_I8 ? 1 : 2);
        uint16_t *y = Y + (size_t)r * d;
        if (vec)
            hipLaunchKernelGGL((normalize_rows<DT, true>), grid, dim3(256), 0, st, x, m, d, y);
        else
            hipLaunchKernelGGL((normalize_rows<DT, false>), grid, dim3(256), 0, st, x, m, d, y);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_normalize(int dtype, const void *X, uint32_t n, uint32_t d, void *Y,
                            hipStream_t stream)
{
    if (n == 0 || d == 0)
        return hipSuccess;
    const uint8_t *x = (const uint8_t *)X;
    uint16_t *y = (uint16_t *)Y;
    switch (dtype) {
    case DT_F16: return normalize_dt<DT_F16>(x, n, d, y, stream);
    case DT_BF16: return normalize_dt<DT_BF16>(x, n, d, y, stream);
    case DT_I8: return normalize_dt<DT_I8>(x, n, d, y, stream);
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
    const uint32_t in_stride = (d + 7) / 8, team = 1u << team_lg, rows = 256u >> team_lg;
    for (uint64_t row = (uint64_t)blockIdx.x * rows + (threadIdx.x >> team_lg); row < n;
         row += (uint64_t)gridDim.x * rows) {
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
    // (a launch holds fewer than 2^32 threads)
    const uint64_t blocks = (n + rows - 1) / rows;
    const dim3 grid((uint32_t)(blocks < (1u << 20) ? blocks : 1u << 20));
    hipLaunchKernelGGL(unpack_hamming, grid, dim3(256), 0, stream, bits, n, d, out_bytes, team_lg,
                       out);
    return hipGetLastError();
}

}  // namespace sjk
