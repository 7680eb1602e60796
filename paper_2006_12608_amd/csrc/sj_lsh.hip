// sj_lsh.hip -- gfx950 kernels of the LSH-bucketed join (Ahle & Silvestri,
// "Similarity Search with Tensor Core Units", Section 4, the LSH method of
// Theorem 3): hash every point into L tables, bring each table's equal keys
// together with a radix sort, list the buckets that P and Q share, and run the
// exact join inside every shared bucket on the matrix cores.
//
// The bucket join is the brute-force join of Section 4 restricted to a pair of
// buckets: Theorem 3's cost is the sum over tables and shared buckets of
// |P bucket| x |Q bucket| inner products, each bucket pair handled as a
// blocked product on 256 x 256 workgroup tiles (32 x 32 MFMA blocks), with the
// same fused threshold test and wave-ballot compaction as the all-pairs join.
#include "sj_lsh.h"

#include "sj_internal.h"
#include "sj_join_kernels.h"
#include "sj_search.h"

namespace sjl {
namespace {

using sjk::DT_BF16;
using sjk::DT_F16;
using sjk::DT_I8;
using sjk::i32x4;
using sjk::MET_IP;
using sjk::MET_L2;

// ----------------------------------------------------------------- keys

// The E stored elements of one 16-byte chunk as exact values; `acc_t` is the
// projection's accumulator and `a_t` the type the projection entries are
// converted to once, before the hash (so that the inner loop is one fused
// multiply-add per element and function, its entry read through the scalar
// path: the entries are the same for every row of a workgroup).
template <int DT>
struct Chunk;

template <>
struct Chunk<DT_F16> {
    static constexpr int E = 8;
    typedef double acc_t;
    typedef double a_t;
    static __device__ __forceinline__ double at(const i32x4 &v, int e)
    {
        const uint16_t h = (uint16_t)((uint32_t)v[e >> 1] >> (16 * (e & 1)));
        return (double)(float)__builtin_bit_cast(_Float16, h);
    }
};

template <>
struct Chunk<DT_BF16> {
    static constexpr int E = 8;
    typedef double acc_t;
    typedef double a_t;
    static __device__ __forceinline__ double at(const i32x4 &v, int e)
    {
        const uint32_t h = ((uint32_t)v[e >> 1] >> (16 * (e & 1))) & 0xffffu;
        return (double)__builtin_bit_cast(float, h << 16);
    }
};

template <>
struct Chunk<DT_I8> {
    static constexpr int E = 16;
    typedef int32_t acc_t;   // |z| <= 32768 * 128 * 128 = 2^29: exact
    typedef int32_t a_t;
    static __device__ __forceinline__ int32_t at(const i32x4 &v, int e)
    {
        return (int32_t)(int8_t)((uint32_t)v[e >> 2] >> (8 * (e & 3)));
    }
};

// Projection rows are widened with their length padded to a multiple of the
// chunk's E elements (zeros past d): together with the zero padding of the
// rows this adds only exact zeros to each sum, and the inner loop needs no
// bounds test.
template <int DT>
constexpr uint32_t padded_d(uint32_t d)
{
    return (d + Chunk<DT>::E - 1) / Chunk<DT>::E * Chunk<DT>::E;
}

template <typename T>
__global__ void widen_kernel(const int8_t *A, T *out, uint32_t d, uint32_t dp, uint64_t n_out)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_out) {
        const uint64_t f = i / dp, m = i - f * dp;
        out[i] = m < d ? T(A[f * d + m]) : T(0);
    }
}

// Rows a workgroup of the key kernel stages in LDS at once (one per lane of a
// wave), and the bytes of a row it stages per pass.
constexpr int KROWS = 64;
constexpr int KSEG = 512;

// G consecutive functions of one row segment: z[g] += sum_m A[f0 + g][m0 + m] x_m
// over the segment's nch chunks (x: this lane's row in LDS) in ascending m.
// The entries' addresses are the same for every lane (the compiler reads them
// with scalar loads).
template <int DT, int G>
__device__ __forceinline__ void project(const uint8_t *x, uint32_t nch, uint32_t dp,
                                        const typename Chunk<DT>::a_t *a,
                                        typename Chunk<DT>::acc_t (&z)[G])
{
    typedef Chunk<DT> C;
    typedef typename C::acc_t acc_t;
    for (uint32_t c = 0; c < nch; ++c) {
        const i32x4 v = *(const i32x4 *)(x + 16 * c);
        acc_t xe[C::E];
#pragma unroll
        for (int e = 0; e < C::E; ++e)
            xe[e] = C::at(v, e);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const typename C::a_t *ag = a + (size_t)g * dp + c * C::E;
#pragma unroll
            for (int e = 0; e < C::E; ++e)
                z[g] += acc_t(ag[e]) * xe[e];
        }
    }
}

// Function u's value folded into the key (see launch_keys).
template <typename T>
__device__ __forceinline__ void fold_value(uint64_t &key, T z, uint32_t u, uint32_t beta,
                                           uint64_t low, const int32_t *B, uint32_t f,
                                           int32_t w)
{
    if (w == 0) {
        key |= (uint64_t)(z >= T(0)) << u;
    } else {
        const double q = ((double)z + (double)B[f]) / (double)w;
        const int64_t v = (int64_t)floor(q);
        key |= ((uint64_t)v & low) << (beta * u);
    }
}

// A workgroup of 4 waves takes KROWS rows: it stages them in LDS in segments
// of KSEG bytes per row (coalesced loads; rows padded by 16 bytes so that the
// lanes' 16-byte reads of their own rows hit distinct banks) and each lane
// computes the keys of its row; wave v takes the tables v, v + 4, ...  Per
// table: z_f = sum_m A[f][m] x_m in ascending m (exact products; for
// fp16/bf16 a double sum in that order, for int8 an exact int32 sum), then the
// function values and the key (see launch_keys).  Rows of at
// most KSEG bytes are staged once for every table; longer rows once per table
// and segment, with the partial sums kept for at most 16 functions per pass.
template <int DT, bool LONG>
__global__ void __launch_bounds__(256) keys_kernel(Rows r, uint32_t d, uint32_t L, uint32_t k,
                                                   const typename Chunk<DT>::a_t *A,
                                                   const int32_t *B, int32_t w,
                                                   uint64_t *keys)
{
    typedef Chunk<DT> C;
    typedef typename C::acc_t acc_t;
    constexpr int RS = KSEG + 16;   // LDS row stride
    __shared__ __attribute__((aligned(16))) uint8_t xs[KROWS * RS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t row0 = blockIdx.x * KROWS;
    const uint32_t rows = min(r.n - row0, (uint32_t)KROWS);
    const uint32_t dp = padded_d<DT>(d);
    const uint32_t rb = dp * (DT == DT_I8 ? 1 : 2);   // bytes hashed per row (<= row_bytes)
    const uint32_t beta = k ? 64 / k : 64;
    const uint64_t low = beta >= 64 ? ~0ull : (1ull << beta) - 1;

    auto stage = [&](uint32_t seg0, uint32_t segb) {
        // segb bytes of every row from byte seg0; 16 bytes per lane per step
        const uint32_t cpr = segb / 16;
        for (uint32_t q = tid; q < KROWS * cpr; q += 256) {
            const uint32_t rr = q / cpr, cc = q - rr * cpr;
            i32x4 v = {0, 0, 0, 0};
            if (rr < rows)
                v = *(const i32x4 *)(r.X + (size_t)(row0 + rr) * r.row_bytes + seg0 + 16 * cc);
            *(i32x4 *)(xs + rr * RS + 16 * cc) = v;
        }
    };
    const uint8_t *mine = xs + lane * RS;
    if constexpr (!LONG) {
        if (rb)
            stage(0, rb);
        __syncthreads();
        const uint32_t nch = rb / 16;
        for (uint32_t t = wave; t < L; t += 4) {
            uint64_t key = 0ull;
            uint32_t u = 0;
            for (; u + 4 <= k; u += 4) {
                acc_t z[4] = {};
                project<DT, 4>(mine, nch, dp, A + (size_t)(t * k + u) * dp, z);
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    fold_value(key, z[g], u + g, beta, low, B, t * k + u + g, w);
            }
            if (u + 2 <= k) {
                acc_t z[2] = {};
                project<DT, 2>(mine, nch, dp, A + (size_t)(t * k + u) * dp, z);
#pragma unroll
                for (int g = 0; g < 2; ++g)
                    fold_value(key, z[g], u + g, beta, low, B, t * k + u + g, w);
                u += 2;
            }
            if (u < k) {
                acc_t z[1] = {};
                project<DT, 1>(mine, nch, dp, A + (size_t)(t * k + u) * dp, z);
                fold_value(key, z[0], u, beta, low, B, t * k + u, w);
            }
            if ((uint32_t)lane < rows)
                keys[(size_t)t * r.n + row0 + lane] = key;
        }
        return;
    } else {
    // long rows: segments of KSEG bytes, every wave takes table t = wave + 4 j
    // in turn (all waves pass every barrier: the table loop is uniform)
    const uint32_t tl = (L + 3) / 4 * 4;
    for (uint32_t t0 = 0; t0 < tl; t0 += 4) {
        const uint32_t t = t0 + wave;
        uint64_t key = 0ull;
        for (uint32_t u = 0; u < k; u += 16) {
            acc_t z[16] = {};
            for (uint32_t seg0 = 0; seg0 < rb; seg0 += KSEG) {
                const uint32_t segb = min(rb - seg0, (uint32_t)KSEG);
                __syncthreads();   // the previous segment is consumed
                stage(seg0, segb);
                __syncthreads();
                if (t < L) {
                    const typename C::a_t *a = A + (size_t)(t * k + u) * dp +
                                               seg0 / 16 * C::E;
                    if (u + 16 <= k)
                        project<DT, 16>(mine, segb / 16, dp, a, z);
                    else
#pragma unroll
                        for (int g = 0; g < 16; ++g)
                            if (u + g < k) {
                                acc_t zg[1] = {z[g]};
                                project<DT, 1>(mine, segb / 16, dp, a + (size_t)g * dp, zg);
                                z[g] = zg[0];
                            }
                }
            }
#pragma unroll
            for (int g = 0; g < 16; ++g)
                if (t < L && u + g < k)
                    fold_value(key, z[g], u + g, beta, low, B, t * k + u + g, w);
        }
        if (t < L && (uint32_t)lane < rows)
            keys[(size_t)t * r.n + row0 + lane] = key;
    }
    }
}

// ------------------------------------------------ keys on the matrix cores
//
// For rows of at most 512 bytes and at most HF_MAX functions in all: the
// projections z_f(x) of 32 rows by 32 functions come from one MFMA block
// (int8: exact int32 sums, so every decision is taken here; fp16 / bf16:
// products exact in fp32, sums rounded).  A
// decision (sign, or floor((z + B) / w)) is taken from the fp32 value only when
// it is certain: the fp32 sum and the double sum in ascending m both differ
// from the exact sum by at most gamma(d) sum_m |A_m x_m| <= gamma(d) ||A|| ||x||
// (any summation order; gamma(d) = d u / (1 - d u)), so when |z| exceeds twice
// the sum of both bounds the sign is the double sum's, and when the interval
// z +- that margin maps to one bucket the quantised value is.  A (row, table)
// with uncertain functions is queued with their mask, and fix_kernel computes
// those with the exact double evaluation, so the keys equal keys_kernel's.
constexpr int HF_MAX = 512;

template <int DT>
__global__ void widen_h_kernel(const int8_t *A, uint16_t *Ah, uint32_t d, uint32_t rl,
                               uint64_t n_out)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_out) {
        const uint64_t f = i / rl, m = i - f * rl;
        const float a = m < d ? (float)A[f * d + m] : 0.0f;   // |a| <= 128: exact in both
        if constexpr (DT == DT_F16)
            Ah[i] = __builtin_bit_cast(uint16_t, (_Float16)a);
        else
            Ah[i] = (uint16_t)(__builtin_bit_cast(uint32_t, a) >> 16);
    }
}

// int8 projection rows copied into rows of rb bytes (zero padded): the int8
// matrix cores' operand layout.
__global__ void pad_b_kernel(const int8_t *A, int8_t *Ab, uint32_t d, uint32_t rb,
                             uint64_t n_out)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_out) {
        const uint64_t f = i / rb, m = i - f * rb;
        Ab[i] = m < d ? A[f * d + m] : (int8_t)0;
    }
}

// Upper bounds of the projection rows' Euclidean norms, a wave per row: the
// double sum rounded up by a relative 2^-20.
__global__ void __launch_bounds__(64) anorm_kernel(const int8_t *A, uint32_t d, float *out)
{
    const uint32_t f = blockIdx.x;
    double s = 0.0;
    for (uint32_t m = threadIdx.x; m < d; m += 64)
        s += (double)A[(uint64_t)f * d + m] * A[(uint64_t)f * d + m];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        s += __shfl_xor(s, o, 64);
    if (threadIdx.x == 0)
        out[f] = (float)(sqrt(s) * (1.0 + 0x1p-20));
}

// floor(n / w) mod 2^32 for integers |n| < 2^53, 0 < w < 2^31, given inv = 1 / w:
// the quotient from the reciprocal is within one of the floor, which the
// remainder (exact) settles.
__device__ __forceinline__ uint32_t floor_div_low(double n, double w, double inv)
{
    double t = __builtin_floor(n * inv);
    const double r = __builtin_fma(-t, w, n);
    t += r < 0.0 ? -1.0 : r >= w ? 1.0 : 0.0;
    return (uint32_t)__builtin_fma(-__builtin_floor(t * 0x1p-32), 0x1p32, t);
}

// Functions come in MFMA blocks of at most 32: whole tables (32 / k of them) or,
// for k > 32, one half of a table (its first 32 functions, then the rest).  A
// workgroup of 4 waves stages each block's projection rows in LDS (the next
// block's while the current one is multiplied); each wave holds 32 rows as
// A-fragments of KS k-steps in registers.  In a result register the lanes of a
// half hold one row's 32 functions, so a sign ballot is that row's bits of the
// block, and a row's keys are bit ranges of one word; quantised values pass
// through LDS to be put together.  Uncertain decisions are ballots too: each
// (row, table) with some goes to the wave's list and from there to the queue,
// one reservation per 64.  262144 x 256 fp16, 160 signs: 121 us (196 us with
// 64-bit LDS atomics per decision, every wave reading all projection rows
// itself, and 53 us for the row norms in a kernel of their own); 1048576 x 64
// int8, 96 quantised values: 98 us (179 us with a double division per value).
template <int DT, int KS, bool QUANT>
__global__ void __launch_bounds__(256) keys_mfma_kernel(
    Rows r, uint32_t L, uint32_t k, const uint8_t *Ah, const float *anorm, const int32_t *B,
    int32_t w, float gam, uint64_t *keys, uint4 *fix, unsigned long long *nfix)
{
    typedef sjk::Mma<DT> M;
    typedef typename M::acc_t acc_t;
    constexpr int CPR = 2 * KS;                       // chunks per staged row
    constexpr int SWS = KS == 2 ? 2 : KS == 4 ? 1 : 0;   // chunk c of row i at c ^ (i >> SWS) % 16:
    constexpr int SWM = CPR < 16 ? CPR - 1 : 15;         // 16 rows' reads of a chunk hit all banks
    constexpr bool EXACT = DT == DT_I8;               // sums exact: nothing uncertain
    __shared__ __attribute__((aligned(16))) uint8_t s_b0[32 * CPR * 16], s_b1[32 * CPR * 16];
    __shared__ uint32_t s_val[QUANT ? 4 : 1][QUANT ? 32 : 1][33];
    __shared__ uint4 s_fix[EXACT ? 1 : 4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int h = lane >> 5, c32 = lane & 31;
    const uint32_t row0 = (blockIdx.x * 4 + wv) * 32, row = row0 + c32;
    const uint32_t nf = L * k, beta = 64 / k;
    const uint32_t low = beta >= 32 ? 0xffffffffu : (1u << beta) - 1u;
    const uint32_t tpb = k <= 32 ? 32 / k : 1;        // tables per block
    const uint32_t n_blk = k <= 32 ? (L + tpb - 1) / tpb : 2 * L;
    auto first_fn = [&](uint32_t b) { return k <= 32 ? b * tpb * k : (b >> 1) * k + 32 * (b & 1); };
    auto n_fn = [&](uint32_t b) {
        return k <= 32 ? min(tpb * k, nf - b * tpb * k) : b & 1 ? k - 32 : 32u;
    };

    i32x4 af[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const uint32_t off = 32 * ks + 16 * h;
        af[ks] = row < r.n && off < r.row_bytes
                     ? *(const i32x4 *)(r.X + (size_t)row * r.row_bytes + off)
                     : i32x4{0, 0, 0, 0};
    }
    // upper bounds of the rows' norms (as anorm_kernel's): this lane's half of
    // row c32, then both halves, then the rows of its result registers
    float xn[EXACT ? 1 : 16];
    if constexpr (!EXACT) {
        double s = 0.0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int e = 0; e < Chunk<DT>::E; ++e) {
                const double x = Chunk<DT>::at(af[ks], e);
                s += x * x;
            }
        s += __shfl_xor(s, 32, 64);
        const float nx = (float)(sqrt(s) * (1.0 + 0x1p-20));
#pragma unroll
        for (int q = 0; q < 16; ++q)
            xn[q] = __shfl(nx, 8 * (q >> 2) + 4 * h + (q & 3), 64);
    }
    auto stage = [&](uint32_t b, uint8_t *dst) {
        const uint32_t f0 = first_fn(b), n = n_fn(b), bytes = nf * r.row_bytes;
#pragma unroll
        for (int i = 0; i < (KS + 3) / 4; ++i) {
            const int kk = 4 * i + wv;
            if (kk < KS) {
                const uint32_t p = 64 * kk + lane, fr = p / CPR, pos = p % CPR;
                const uint32_t off = 16 * (pos ^ ((fr >> SWS) & SWM));
                const bool in = fr < n && off < r.row_bytes;
                sjk::buffer_load_lds16(Ah, bytes, in ? (f0 + fr) * r.row_bytes + off : bytes,
                                       dst + 1024 * kk);
            }
        }
    };
    uint32_t n_list = 0;   // wave-uniform: entries of s_fix[wave]
    auto flush = [&]() {
        unsigned long long base = 0;
        if (lane == 0)
            base = atomicAdd(nfix, (unsigned long long)n_list);
        base = sjk::first_lane_u64(base);
        if ((uint32_t)lane < n_list)
            fix[base + lane] = s_fix[EXACT ? 0 : wave][lane];
        n_list = 0;
    };
    auto queue = [&](bool some, uint32_t t, uint64_t m) {
        const uint64_t bits = __ballot(some);
        const uint32_t n = (uint32_t)__popcll(bits);
        if (n == 0)
            return;
        if (n_list + n > 64) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            flush();
        }
        if (some)
            s_fix[EXACT ? 0 : wave][n_list + sjk::lanes_below(bits)] =
                make_uint4(row, t, (uint32_t)m, (uint32_t)(m >> 32));
        n_list += n;
    };

    uint64_t key0 = 0, unc0 = 0;   // k > 32: the table's first half
    auto block = [&](uint32_t b, const uint8_t *cur, uint8_t *nxt) __attribute__((always_inline)) {
        if (b + 1 < n_blk)
            stage(b + 1, nxt);
        acc_t acc = acc_t{};
        const uint32_t sw = (c32 >> SWS) & SWM;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const i32x4 fb = *(const i32x4 *)(cur + c32 * CPR * 16 + 16 * ((2 * ks + h) ^ sw));
            acc = M::mma(af[ks], fb, acc);
        }
        const uint32_t f0 = first_fn(b), n = n_fn(b), f = f0 + c32;
        const bool fok = (uint32_t)c32 < n;
        const float na = EXACT || !fok ? 0.0f : anorm[f];
        const double bf = QUANT && fok ? (double)B[f] : 0.0;
        const double wd = (double)w, inv = 1.0 / wd;
        uint32_t word = 0, unc = 0;   // row c32's sign bits / uncertain functions
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int ra = 8 * (q >> 2) + (q & 3);   // the lower half's row; ra + 4 the upper's
            bool sure = true;
            uint32_t v = 0;
            bool pos = false;
            if constexpr (EXACT) {
                if constexpr (QUANT)
                    v = floor_div_low((double)acc[q] + bf, wd, inv) & low;
                else
                    pos = acc[q] >= 0;
            } else {
                const float z = acc[q], e = gam * na * xn[q];
                if constexpr (QUANT) {
                    const double lo = floor(((double)z - (double)e + bf) / wd);
                    const double hi = floor(((double)z + (double)e + bf) / wd);
                    sure = lo == hi;
                    v = sure ? (uint32_t)((uint64_t)(int64_t)lo) & low : 0u;
                } else {
                    sure = __builtin_fabsf(z) > e;
                    pos = z >= 0.0f && sure;
                }
                const uint64_t nb = __ballot(fok && !sure);
                if (nb != 0) {   // uniform, rare
                    unc = c32 == ra ? (uint32_t)nb : unc;
                    unc = c32 == ra + 4 ? (uint32_t)(nb >> 32) : unc;
                }
            }
            if constexpr (QUANT) {
                s_val[wave][ra + 4 * h][c32] = v;
            } else {
                const uint64_t bits = __ballot(pos);
                word = c32 == ra ? (uint32_t)bits : word;
                word = c32 == ra + 4 ? (uint32_t)(bits >> 32) : word;
            }
        }
        if constexpr (QUANT) {
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        // the block's tables: lanes of half h take tables h, h + 2, ...
        const uint32_t kb = k <= 32 ? k : n;             // functions per table here
        const uint32_t t0 = k <= 32 ? b * tpb : b >> 1, nt = k <= 32 ? n / k : 1;
        for (uint32_t tl2 = 0; tl2 < nt; tl2 += 2) {
            const uint32_t tl = tl2 + h;
            const bool on = tl < nt && row < r.n;
            const uint32_t sh = on ? tl * kb : 0u, mask = kb >= 32 ? 0xffffffffu : (1u << kb) - 1u;
            uint64_t key = 0, um = (unc >> sh) & mask;
            if constexpr (QUANT) {
                if (on)
                    for (uint32_t u = 0; u < kb; ++u)
                        key |= (uint64_t)s_val[wave][c32][sh + u]
                               << (beta * (u + (k > 32 ? 32 * (b & 1) : 0)));
            } else {
                key = (word >> sh) & mask;
                if (k > 32)
                    key <<= 32 * (b & 1);
            }
            if (k > 32) {
                um <<= 32 * (b & 1);
                if (!(b & 1)) {   // the first half: kept for the second
                    key0 = key;
                    unc0 = um;
                    continue;
                }
                key |= key0;
                um |= unc0;
            }
            if (on)
                keys[(size_t)(t0 + tl) * r.n + row] = key;
            if constexpr (!EXACT)
                queue(on && um != 0, t0 + tl, um);
        }
        __builtin_amdgcn_s_waitcnt(0);   // the next block's rows landed
        __syncthreads();
    };
    stage(0, s_b0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (uint32_t b = 0; b < n_blk; b += 2) {
        block(b, s_b0, s_b1);
        if (b + 1 < n_blk)
            block(b + 1, s_b1, s_b0);
    }
    if constexpr (!EXACT) {
        if (n_list) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            flush();
        }
    }
}

// The queued (row, table) keys: the functions the matrix-core pass could not
// decide, recomputed exactly as keys_kernel does (the row read from global
// memory), OR-ed into the key (whose bits for them are still zero); one
// thread per entry, grid-stride over the queue's length read from device
// memory.
template <int DT>
__global__ void __launch_bounds__(256) fix_kernel(Rows r, uint32_t d, uint32_t k,
                                                  const typename Chunk<DT>::a_t *A,
                                                  const int32_t *B, int32_t w,
                                                  const uint4 *fix,
                                                  const unsigned long long *nfix, uint64_t *keys)
{
    typedef Chunk<DT> C;
    typedef typename C::acc_t acc_t;
    const uint64_t n_fix = *nfix;
    const uint32_t dp = padded_d<DT>(d), nch = dp / C::E;
    const uint32_t beta = k ? 64 / k : 64;
    const uint64_t low = beta >= 64 ? ~0ull : (1ull << beta) - 1;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n_fix;
         i += (uint64_t)gridDim.x * 256) {
        const uint4 e = fix[i];
        const uint32_t row = e.x, t = e.y;
        uint64_t m = (uint64_t)e.z | ((uint64_t)e.w << 32);
        const uint8_t *x = r.X + (size_t)row * r.row_bytes;
        uint64_t key = 0;
        while (m) {
            const uint32_t u = (uint32_t)__builtin_ctzll(m);
            m &= m - 1;
            const typename C::a_t *a = A + (size_t)(t * k + u) * dp;
            acc_t z = acc_t(0);
            for (uint32_t c = 0; c < nch; ++c) {
                const i32x4 v = *(const i32x4 *)(x + 16 * c);
#pragma unroll
                for (int q = 0; q < C::E; ++q)
                    z += acc_t(a[c * C::E + q]) * C::at(v, q);
            }
            fold_value(key, z, u, beta, low, B, t * k + u, w);
        }
        keys[(size_t)t * r.n + row] |= key;
    }
}

// ------------------------------------------------------------ bucket pairs

// First sorted position in [lo, hi) whose key is > key (keys ascending).
__device__ __forceinline__ uint32_t upper_bound(const uint64_t *s, uint32_t lo, uint32_t hi,
                                                uint64_t key)
{
    return first_above([s](uint32_t i) { return s[i]; }, lo, hi, key);
}

__device__ __forceinline__ uint32_t lower_bound(const uint64_t *s, uint32_t lo, uint32_t hi,
                                                uint64_t key)
{
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (s[mid] < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Per table and block of 256 sorted positions of P, the range of Q's sorted
// positions whose keys lie between the block's first and last keys: qr[t nb +
// b] = {first position with key >= the block's first, first with key > its
// last} (one thread each, so the searches of every block run at once).
__global__ void __launch_bounds__(256) qrange_kernel(const uint64_t *sorted_p, uint32_t n_p,
                                                     const uint64_t *sorted_q, uint32_t n_q,
                                                     uint32_t L, uint2 *qr)
{
    const uint32_t nb = (n_p + 255) / 256;
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (uint64_t)nb * L)
        return;
    const uint32_t t = (uint32_t)(i / nb), b = (uint32_t)(i - (uint64_t)t * nb);
    const uint64_t *sp = sorted_p + (size_t)t * n_p;
    const uint64_t *sq = sorted_q + (size_t)t * n_q;
    const uint32_t pf = 256 * b;
    qr[i] = make_uint2(lower_bound(sq, 0, n_q, sp[pf]),
                       upper_bound(sq, 0, n_q, sp[min(pf + 255, n_p - 1)]));
}

// One thread per (sorted position of P, table): a position that starts a P
// bucket looks its key up in Q's sorted keys within the block's range
// (qrange_kernel), staged in LDS when it holds at most QCAP keys, and, when Q
// has the key, is a record.  A bucket ends at the block's next start (a bit
// mask of the starts), only the block's last one is followed in memory.  The
// block's records are written one after the other at tmp[256 block] with their
// number in n_rec, so that the scan and the copy that follow work on blocks and
// records instead of positions.  16 tables of 1048576 positions: 233 us (291
// with a search for every end and three words written per position), the scan
// and the copy that follow 30 us (190).
constexpr uint32_t QCAP = 2048;

__global__ void __launch_bounds__(256) bucket_find_kernel(const uint64_t *sorted_p, uint32_t n_p,
                                                          const uint64_t *sorted_q, uint32_t n_q,
                                                          const uint2 *qr, uint4 *tmp,
                                                          uint32_t *n_rec, ulonglong2 *part)
{
    __shared__ uint64_t s_q[QCAP];
    __shared__ unsigned long long s_cand[4], s_rows[4];
    __shared__ uint64_t s_start[4];
    __shared__ uint32_t s_n[4];
    const uint32_t t = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t pf = blockIdx.x * 256, p = pf + tid;
    const size_t blk = (size_t)t * gridDim.x + blockIdx.x;
    const uint64_t *sp = sorted_p + (size_t)t * n_p;
    const uint64_t *sq = sorted_q + (size_t)t * n_q;
    const uint2 range = qr[blk];
    const uint32_t qa = range.x, qb = range.y, qn = qb - qa;
    const bool staged = qn <= QCAP;   // uniform
    const uint64_t key = p < n_p ? sp[p] : 0;
    const bool start = p < n_p && (p == 0 || sp[p - 1] != key);
    const uint64_t starts = __ballot(start);
    if (lane == 0)
        s_start[wave] = starts;
    if (staged)
        for (uint32_t i = tid; i < qn; i += 256)
            s_q[i] = sq[qa + i];
    __syncthreads();
    uint64_t cand = 0, rows = 0;
    uint4 rec = make_uint4(0, 0, 0, 0);
    bool found = false;
    if (start) {
        uint32_t q0, qe;
        if (staged) {
            // first position with key >= key, then doubling steps to the end of
            // its run
            uint32_t lo = 0, hi = qn;
            while (lo < hi) {
                const uint32_t mid = lo + (hi - lo) / 2;
                if (s_q[mid] < key)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            uint32_t e = lo, step = 1;
            while (e + step <= qn && s_q[e + step - 1] == key) {
                e += step;
                step *= 2;
            }
            hi = min(e + step, qn);
            while (e < hi) {
                const uint32_t mid = e + (hi - e) / 2;
                if (s_q[mid] == key)
                    e = mid + 1;
                else
                    hi = mid;
            }
            q0 = qa + lo;
            qe = qa + e;
        } else {
            q0 = lower_bound(sq, qa, qb, key);
            qe = upper_bound(sq, q0, qb, key);
        }
        found = q0 < qe;
        if (found) {
            uint32_t np = 0;
            uint64_t m = lane < 63 ? s_start[wave] >> (lane + 1) << (lane + 1) : 0;
            uint32_t w = wave;
            while (m == 0 && ++w < 4)
                m = s_start[w];
            if (m != 0)
                np = 64 * w + (uint32_t)__builtin_ctzll(m) - tid;
            else   // the block's last bucket: up to the block's end and beyond
                np = run_end([sp](uint32_t i) { return sp[i]; }, min(pf + 256, n_p), n_p, key) - p;
            rec = make_uint4(p, np, q0, qe - q0);
            cand = (uint64_t)np * (qe - q0);
            rows = (uint64_t)np + (qe - q0);
        }
    }
    const uint64_t bits = __ballot(found);
    if (lane == 0)
        s_n[wave] = (uint32_t)__popcll(bits);
    // the block's pair evaluations and rows, summed by sum_parts_kernel (one
    // counter updated by every block serialises the blocks on its address)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        cand += __shfl_xor(cand, o, 64);
        rows += __shfl_xor(rows, o, 64);
    }
    if (lane == 0) {
        s_cand[wave] = cand;
        s_rows[wave] = rows;
    }
    __syncthreads();
    if (found) {
        uint32_t at = sjk::lanes_below(bits);
        for (uint32_t w = 0; w < wave; ++w)
            at += s_n[w];
        tmp[blk * 256 + at] = rec;
    }
    if (tid == 0) {
        n_rec[blk] = s_n[0] + s_n[1] + s_n[2] + s_n[3];
        part[blk] = make_ulonglong2(s_cand[0] + s_cand[1] + s_cand[2] + s_cand[3],
                                    s_rows[0] + s_rows[1] + s_rows[2] + s_rows[3]);
    }
}

// One block of 1024 threads: out[0] = sum of the parts' pair evaluations,
// out[7] = sum of their rows (the counters' slots; written, not added to).
__global__ void __launch_bounds__(1024) sum_parts_kernel(const ulonglong2 *part, uint64_t n,
                                                         unsigned long long *out)
{
    __shared__ unsigned long long s_c[16], s_r[16];
    const uint32_t tid = threadIdx.x;
    unsigned long long c = 0, r = 0;
    for (uint64_t i = tid; i < n; i += 1024) {
        const ulonglong2 v = part[i];
        c += v.x;
        r += v.y;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        c += __shfl_xor(c, o, 64);
        r += __shfl_xor(r, o, 64);
    }
    if ((tid & 63) == 0) {
        s_c[tid >> 6] = c;
        s_r[tid >> 6] = r;
    }
    __syncthreads();
    if (tid == 0) {
        unsigned long long tc = 0, tr = 0;
        for (int w = 0; w < 16; ++w) {
            tc += s_c[w];
            tr += s_r[w];
        }
        out[0] = tc;
        out[7] = tr;
    }
}

// The blocks' records (bucket_find_kernel) one after the other; a wave per
// block, rec_off the scan of n_rec, nb blocks per table.
__global__ void __launch_bounds__(256) bucket_write_kernel(uint32_t nb, uint64_t n_blk,
                                                           const uint4 *tmp, const uint32_t *n_rec,
                                                           const unsigned long long *rec_off,
                                                           Records rec)
{
    const uint64_t blk = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (blk >= n_blk)
        return;
    const uint32_t n = n_rec[blk], t = (uint32_t)(blk / nb);
    const unsigned long long off = rec_off[blk];
    for (uint32_t i = threadIdx.x & 63; i < n; i += 64) {
        rec.t[off + i] = t;
        rec.pq[off + i] = tmp[blk * 256 + i];
    }
}

// One block per chunk of PACK_CHUNK records (see sj_lsh.h).  The sizes of the
// records that fit a tile are prefix-summed; then the first wave forms the
// groups, each in one step: lane k tests whether records i .. i + k still fit.
// In the write pass the block copies the groups' rows to their lists, a thread
// per row.  (One thread walking the records took 70 us for 660 000 of them.)
__global__ void __launch_bounds__(256) pack_kernel(Records rec, uint32_t n_rec, int write,
                                                   uint32_t *chunk_desc, uint32_t *chunk_tiles,
                                                   const unsigned long long *desc_off,
                                                   const unsigned long long *tile_off, Descs desc,
                                                   Lists ls, unsigned long long *overflow)
{
    static_assert(PACK_CHUNK <= 256, "one record per thread");
    __shared__ uint4 spq[PACK_CHUNK];
    __shared__ uint32_t st[PACK_CHUNK], sfirst[PACK_CHUNK];
    __shared__ uint32_t PS[PACK_CHUNK + 1], QS[PACK_CHUNK + 1], sw[8];
    const uint32_t c = blockIdx.x, r0 = c * PACK_CHUNK, tid = threadIdx.x, lane = tid & 63;
    const uint32_t rn = min((uint32_t)PACK_CHUNK, n_rec - r0);
    uint4 pq = make_uint4(0, 0, 0, 0);
    if (tid < rn) {
        pq = rec.pq[r0 + tid];
        spq[tid] = pq;
        st[tid] = rec.t[r0 + tid];
    }
    const bool big = pq.y > TILE || pq.w > TILE;
    uint32_t ip = big ? 0u : pq.y, iq = big ? 0u : pq.w;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(ip, o, 64), uq = __shfl_up(iq, o, 64);
        if ((int)lane >= o) {
            ip += up;
            iq += uq;
        }
    }
    if (lane == 63) {
        sw[tid >> 6] = ip;
        sw[4 + (tid >> 6)] = iq;
    }
    __syncthreads();
    for (uint32_t w = 0; w < tid >> 6; ++w) {
        ip += sw[w];
        iq += sw[4 + w];
    }
    if (tid < PACK_CHUNK) {   // inclusive sums (a chunk's rows fit 32 bits)
        PS[tid + 1] = ip;
        QS[tid + 1] = iq;
    }
    if (tid == 0)
        PS[0] = QS[0] = 0;
    __syncthreads();
    if (tid < 64) {
        const uint64_t dbase = write ? desc_off[c] : 0, tbase = write ? tile_off[c] : 0;
        uint32_t nd = 0;
        uint64_t nt = 0;
        auto emit = [&](uint4 rows, uint32_t table, uint32_t packed, uint64_t tiles) {
            if (write && lane == 0) {
                const uint64_t tl = tbase + nt;
                desc.pq[dbase + nd] = rows;
                desc.info[dbase + nd] = make_uint4(table, packed, (uint32_t)tl, (uint32_t)(tl >> 32));
            }
            ++nd;
            nt += tiles;
        };
        for (uint32_t i = 0; i < rn;) {
            const uint4 ri = spq[i];
            const uint32_t ti = st[i];
            if (ri.y > TILE || ri.w > TILE) {
                emit(ri, ti, 0, (uint64_t)((ri.y + TILE - 1) / TILE) * ((ri.w + TILE - 1) / TILE));
                if (lane == 0)
                    sfirst[i] = 0xffffffffu;
                ++i;
                continue;
            }
            uint32_t e = i;   // the group is [i, e)
            for (;;) {
                const uint32_t k = e + lane;
                bool ok = k < rn;
                if (ok)
                    ok = spq[k].y <= TILE && spq[k].w <= TILE && st[k] == ti &&
                         PS[k + 1] - PS[i] <= TILE && QS[k + 1] - QS[i] <= TILE;
                const uint64_t m = __ballot(ok);
                const uint32_t run = m == ~0ull ? 64u : (uint32_t)__builtin_ctzll(~m);
                if (lane < run)
                    sfirst[k] = i;
                e += run;
                if (run < 64)
                    break;
            }
            if (e == i + 1) {   // alone in its tile: no list
                if (lane == 0)
                    sfirst[i] = 0xffffffffu;
                emit(ri, ti, 0, 1);
            } else {
                emit(make_uint4(ri.x, PS[e] - PS[i], ri.z, QS[e] - QS[i]), ti, 1, 1);
            }
            i = e;
        }
        if (!write && lane == 0) {
            chunk_desc[c] = nd;
            chunk_tiles[c] = (uint32_t)min(nt, (uint64_t)0xffffffffu);
            if (nt > 0xffffffffull)
                atomicMax(overflow, 1ull);
        }
    }
    if (!write)
        return;
    __syncthreads();
    // the groups' rows alone, prefix-summed again (a chunk of large buckets has
    // few); then x is a row's place among them
    const bool mine = tid < rn && sfirst[tid] != 0xffffffffu;
    ip = mine ? pq.y : 0u;
    iq = mine ? pq.w : 0u;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(ip, o, 64), uq = __shfl_up(iq, o, 64);
        if ((int)lane >= o) {
            ip += up;
            iq += uq;
        }
    }
    if (lane == 63) {
        sw[tid >> 6] = ip;
        sw[4 + (tid >> 6)] = iq;
    }
    __syncthreads();
    for (uint32_t w = 0; w < tid >> 6; ++w) {
        ip += sw[w];
        iq += sw[4 + w];
    }
    if (tid < PACK_CHUNK) {
        PS[tid + 1] = ip;
        QS[tid + 1] = iq;
    }
    __syncthreads();
    auto copy = [&](const uint32_t *S, bool q) {
        const uint32_t total = S[rn];
        constexpr int U = 4;   // rows per thread and round: their loads overlap
        for (uint32_t x0 = tid; x0 < total; x0 += 256 * U) {
            uint32_t row[U];
            size_t dst[U];
            uint8_t tag[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t x = min(x0 + 256 * u, total - 1);
                uint32_t lo = 0, hi = rn;   // the last record with S[lo] <= x
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (S[mid] <= x)
                        lo = mid;
                    else
                        hi = mid;
                }
                const uint32_t first = sfirst[lo];
                const size_t tb = (size_t)st[lo] * (q ? ls.n_q : ls.n_p);
                const uint32_t p0 = q ? spq[lo].z : spq[lo].x, d0 = q ? spq[first].z : spq[first].x;
                dst[u] = tb + d0 + (x - S[first]);
                tag[u] = (uint8_t)(lo - first);
                row[u] = (q ? ls.perm_q : ls.perm_p)[tb + p0 + (x - S[lo])];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (x0 + 256 * u < total) {
                    (q ? ls.list_q : ls.list_p)[dst[u]] = row[u];
                    (q ? ls.tag_q : ls.tag_p)[dst[u]] = tag[u];
                }
        }
    };
    copy(PS, false);
    copy(QS, true);
}

// ------------------------------------------------------------ bucket join

template <int DT, int MET>
__device__ __forceinline__ bool matches(typename sjk::Mma<DT>::val_t acc,
                                        typename sjk::Mma<DT>::val_t nx,
                                        typename sjk::Mma<DT>::val_t ny, const JoinArgs &g)
{
    if constexpr (MET == MET_IP) {
        if constexpr (DT == DT_I8)
            return acc >= g.thr_i;
        else
            return acc >= g.thr_f;
    } else {
        if constexpr (DT == DT_I8)
            return 2 * acc >= nx + ny - g.thr_i;
        else
            return 2.0f * acc >= (nx + ny) - g.thr_f;
    }
}

// Bit u: byte u of two rows' 16 fingerprint bytes is equal, of the first `tables`
// bytes (equal keys give equal bytes).
__device__ __forceinline__ uint32_t equal_bytes(const uint4 &fi, const uint4 &fj, uint32_t tables)
{
    const uint32_t xw[4] = {fi.x ^ fj.x, fi.y ^ fj.y, fi.z ^ fj.z, fi.w ^ fj.w};
    uint32_t eq = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t x = xw[q];
        const uint32_t y = ~(((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x | 0x7f7f7f7fu);
        eq |= (((y >> 7) & 1u) | ((y >> 14) & 2u) | ((y >> 21) & 4u) | ((y >> 28) & 8u))
              << (4 * q);
    }
    return eq & (tables >= 16 ? 0xffffu : (1u << tables) - 1u);
}

// Whether the keys of rows i of P and j of Q are equal in one of the tables t0 + u,
// bit u of eq.
__device__ __forceinline__ bool equal_key(const JoinArgs &g, uint32_t i, uint32_t j, uint32_t t0,
                                          uint32_t eq)
{
    while (eq) {
        const uint32_t t2 = t0 + __builtin_ctz(eq);
        eq &= eq - 1;
        if (g.keys_p[(size_t)t2 * g.P.n + i] == g.keys_q[(size_t)t2 * g.Q.n + j])
            return true;
    }
    return false;
}

// The same for the tables without a fingerprint byte before t, 8 per round of
// independent loads.
__device__ __forceinline__ bool equal_later_key(const JoinArgs &g, uint32_t i, uint32_t j,
                                                uint32_t t)
{
    for (uint32_t t2 = FP_MAX; t2 < t; t2 += 8) {
        bool same = false;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const uint32_t tt = t2 + u < t ? t2 + u : t - 1;
            same |= g.keys_p[(size_t)tt * g.P.n + i] == g.keys_q[(size_t)tt * g.Q.n + j];
        }
        if (same)
            return true;
    }
    return false;
}

// Whether rows i of P and j of Q agree in a table before t (the first-table
// rule: such a pair is reported there).
__device__ __forceinline__ bool in_earlier_table(const JoinArgs &g, uint32_t i, uint32_t j,
                                                 uint32_t t)
{
    if (t == 0)
        return false;
    const uint32_t fc = fp_chunks(g.L), tf = t < FP_MAX ? t : FP_MAX;
    for (uint32_t c = 0; 16 * c < tf; ++c) {
        const uint32_t eq = equal_bytes(g.fp_p[(size_t)i * fc + c], g.fp_q[(size_t)j * fc + c],
                                        tf - 16 * c);
        if (equal_key(g, i, j, 16 * c, eq))
            return true;
    }
    return equal_later_key(g, i, j, t);
}

// The bits set in a wave's w[4] and this lane's exclusive prefix of them.
__device__ __forceinline__ void wave_totals(const uint32_t (&w)[4], uint32_t &tot, uint32_t &pre)
{
    const uint32_t cnt = (uint32_t)(__builtin_popcount(w[0]) + __builtin_popcount(w[1]) +
                                    __builtin_popcount(w[2]) + __builtin_popcount(w[3]));
    tot = pre = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) {   // at most 128 a lane
        const uint64_t bits = __ballot((cnt >> b) & 1);
        tot += (uint32_t)__popcll(bits) << b;
        pre += sjk::lanes_below(bits) << b;
    }
}

// The bucket join.  A persistent workgroup of 8 waves takes a contiguous range
// of the tiles (TILE x TILE results at most; descriptors in sj_lsh.h) and walks
// it as one stream of stages, a stage being 128 bytes of each row of a tile.
// Bound by the gathers: every stage needs loads that depend on loads (the
// descriptor, the rows' indices, the rows), so they run ahead by whole stages
// and a stage waits for all of its loads once, at its end:
//   rows of the next stage (the tile's next 128 bytes, or the next tile's first)
//   straight into the other LDS buffer; with a tile's first stage the row
//   indices (and tags) of the tile after the next; with its last stage the
//   next tile's norms; descriptors one ahead, through the scalar path.
// Rows of 128-byte stages are 8 chunks of 16 bytes, chunk c of row r at position
// c ^ (r / 2 % 8) of the row: 16 consecutive rows' reads of one chunk hit all
// banks.  Wave (wr, wc) of 4 x 2 multiplies rows 64 wr .. by columns 128 wc ..
// (2 x 4 blocks of 32 x 32).  Tiles of 256 x 256 instead of 128 x 128 read a
// bucket's rows once or twice instead of two or three times.  128 x 128 tiles with
// four workgroups per CU that each ran the chain of loads tile by tile, after a copy
// of the rows into records, took 2200 us for 262144 x 256 fp16, 16 tables x 10 signs
// and 4590 us for 1048576 x 64 int8, 16 tables x 6 values; in kernel traces this
// takes 1622 us (6.8 GB read a call, 4.2 TB/s) and 3104 us.
// Matches go to an LDS list (JCAP pairs with their table); the first-table rule,
// a chain of loads per match, then runs for the list at once, a thread per
// match, and reserves output slots once.  A wave whose matches of a tile do not
// fit the list's end holds them: their bits and the rows' indices go to its
// workgroup's held records (resolved by held_kernel, which has the waves to hide
// the rule's chains of loads), and a workgroup whose records may not hold another
// tile's stops and is launched again after they are resolved.
// FAR: operands of 4 GiB or more, rows through registers (64-bit addresses).
constexpr int JT = 512;            // threads
constexpr uint32_t JCAP = 1024;    // list entries: a whole 32 x 32 block fits an empty list

template <int DT, int MET, bool FAR>
__global__ void __launch_bounds__(JT) join_kernel(JoinArgs g)
{
    typedef sjk::Mma<DT> M;
    typedef typename M::acc_t acc_t;
    typedef typename M::val_t V;
    constexpr bool L2N = MET == MET_L2;
    constexpr int SA = 2, SB = 4;
    constexpr int ROWS = 2 * TILE;              // P rows, then Q rows
    constexpr int NLD = ROWS * 8 / JT;          // 16-byte loads per thread and stage
    __shared__ __attribute__((aligned(16))) uint8_t s_r0[ROWS * 128], s_r1[ROWS * 128];
    __shared__ uint32_t s_idx[3][ROWS];         // row indices of tiles k % 3
    __shared__ uint8_t s_tag[3][ROWS];          // packed tiles: the rows' records
    __shared__ V s_norm[2][L2N ? ROWS : 1];     // norms of tiles k % 2
    __shared__ uint2 s_pair[JCAP];
    __shared__ uint8_t s_pt[JCAP];
    __shared__ uint32_t s_cnt, s_lim;           // list entries reserved; first that did not fit
    __shared__ uint32_t s_held;                 // held records
    __shared__ uint32_t s_sum[JT / 64];         // list: pairs of each wave
    __shared__ unsigned long long s_base;       // list: their first output slot
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int wr = wv >> 1, wc = wv & 1, half = lane >> 5, c32 = lane & 31;
    const uint32_t rb = g.P.row_bytes;   // == g.Q.row_bytes
    const uint32_t n_st = (rb + 127) / 128;
    const uint64_t T0 = g.resume ? g.next[blockIdx.x] : (uint64_t)blockIdx.x * g.n_tiles / gridDim.x;
    const uint64_t T1 = (uint64_t)(blockIdx.x + 1) * g.n_tiles / gridDim.x;
    if (T0 >= T1) {   // the whole workgroup
        if (tid == 0) {
            g.n_held[blockIdx.x] = 0;
            g.next[blockIdx.x] = T1;
        }
        return;
    }

    // ---- the tiles in order (all uniform)
    // what stays with a tile, in one register: its rows of P and Q (9 bits
    // each), its table, whether it is packed
    struct Tile {
        uint32_t w;
        __device__ __forceinline__ uint32_t np() const { return w & 511u; }
        __device__ __forceinline__ uint32_t nq() const { return (w >> 9) & 511u; }
        __device__ __forceinline__ uint32_t t() const { return (w >> 18) & 255u; }
        __device__ __forceinline__ bool packed() const { return (w >> 26) != 0; }
    };
    static_assert(TILE < 512, "9 bits");
    uint32_t dsc = 0;
    {
        uint32_t hi = g.n_desc;
        while (hi - dsc > 1) {
            const uint32_t mid = (dsc + hi) >> 1;
            const uint4 f = g.desc.info[mid];
            if ((((uint64_t)f.w << 32) | f.z) <= T0)
                dsc = mid;
            else
                hi = mid;
        }
    }
    uint4 dpq = g.desc.pq[dsc], npq = g.desc.pq[min(dsc + 1, g.n_desc - 1)];
    uint2 dinf, ninf = *(const uint2 *)&g.desc.info[min(dsc + 1, g.n_desc - 1)];   // table, packed
    uint32_t tp, tq;
    {
        const uint4 f = g.desc.info[dsc];
        dinf = make_uint2(f.x, f.y);
        const uint32_t ntq = (dpq.w + TILE - 1) / TILE;
        const uint64_t local = T0 - (((uint64_t)f.w << 32) | f.z);
        tp = (uint32_t)(local / ntq);
        tq = (uint32_t)(local % ntq);
    }
    // thread tid < TILE: P row tid of a tile, else Q row tid - TILE
    const bool is_q = wv >= (int)TILE / 64;   // uniform
    const uint32_t li = tid & (TILE - 1);
    // (this wave's norms: read from the arguments once, not at every tile before the
    // load that waits for it)
    const V *norms = (const V *)(is_q ? g.norm_q : g.norm_p);
    asm volatile("" : "+s"(norms));
    // the next tile: this thread's row of it is loaded (0xffffffff: none)
    auto take = [&](uint32_t &idx, uint32_t &tag) -> Tile {
        const uint32_t np = min(dpq.y - tp * TILE, TILE), nq = min(dpq.w - tq * TILE, TILE);
        const uint32_t t = dinf.x;
        const bool packed = dinf.y != 0;
        const size_t at = is_q ? (size_t)t * g.Q.n + dpq.z + tq * TILE + li
                               : (size_t)t * g.P.n + dpq.x + tp * TILE + li;
        idx = 0xffffffffu;
        tag = 0;
        if (li < (is_q ? nq : np)) {
            const uint32_t *src = packed ? (is_q ? g.ls.list_q : g.ls.list_p)
                                         : (is_q ? g.ls.perm_q : g.ls.perm_p);
            idx = src[at];
            if (packed)
                tag = (is_q ? g.ls.tag_q : g.ls.tag_p)[at];
        }
        if (++tq * TILE >= dpq.w) {
            tq = 0;
            if (++tp * TILE >= dpq.y) {
                tp = 0;
                ++dsc;
                dpq = npq;
                dinf = ninf;
                const uint32_t nx = min(dsc + 1, g.n_desc - 1);
                npq = g.desc.pq[nx];
                const uint2 f = *(const uint2 *)&g.desc.info[nx];
                ninf = f;
            }
        }
        return Tile{np | (nq << 9) | (t << 18) | (packed ? 1u << 26 : 0u)};
    };
    auto norm_load = [&](uint32_t idx) -> V {
        V v = V(0);
        if constexpr (L2N) {
            if (idx != 0xffffffffu)
                v = norms[idx];
        }
        return v;
    };
    // One stage of a tile's rows into `dst`: wave instruction k fills rows
    // 8 k .. 8 k + 7; lane l its row l / 8 and position l % 8.  Rows past the
    // tile's and chunks past a row read zeros (an offset past the buffer).
    static_assert(JT / 64 * 8 * (NLD / 2) == (int)TILE, "a thread's first half of loads is P's");
    const uint32_t bytes_p = FAR ? 0u : g.P.n * rb, bytes_q = FAR ? 0u : g.Q.n * rb;
    auto rows_issue = [&](const uint32_t *idx, uint32_t st, uint8_t *dst) {
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int k = wv + (JT / 64) * i;
            const uint32_t row = 8 * k + (lane >> 3);
            const uint32_t c = 128 * st + 16 * ((lane & 7) ^ ((row >> 1) & 7));
            const uint32_t r = idx[row];
            const bool in = r != 0xffffffffu && c < rb;
            const bool q = i >= NLD / 2;         // 8 k >= TILE
            if constexpr (FAR) {
                i32x4 v = {0, 0, 0, 0};
                if (in)
                    v = *(const i32x4 *)((q ? g.Q.X : g.P.X) + (size_t)r * rb + c);
                *(i32x4 *)(dst + 1024 * k + 16 * lane) = v;
            } else {
                sjk::buffer_load_lds16(q ? g.Q.X : g.P.X, q ? bytes_q : bytes_p,
                                       in ? r * rb + c : q ? bytes_q : bytes_p, dst + 1024 * k);
            }
        }
    };

    // ---- matches
    // block s of a wave's results: row block a = s % SA, column block b = s / SA; its
    // match bits (bit r: register r) are w[b] >> 16 a.  Places come from the lane
    // given: one that the compiler does not know as such, so that it computes them
    // where they are needed and keeps no register for them.
    auto bits_of = [](const uint32_t (&w)[SB], int s) {
        const int b = s >> 1;
        const uint32_t wb = b == 0 ? w[0] : b == 1 ? w[1] : b == 2 ? w[2] : w[3];
        return (wb >> (16 * (s & 1))) & 0xffffu;
    };
    auto row_of = [&](int s, int l, int r) {
        return 64 * wr + 32 * (s & 1) + 4 * (l >> 5) + 8 * (r >> 2) + (r & 3);
    };
    auto col_of = [&](int s, int l) { return 128 * wc + 32 * (s >> 1) + (l & 31); };
    // The list's pairs to the output, and the list empty.  Every wave calls it after a
    // barrier (and passes two more in it).
    auto resolve_list = [&]() __attribute__((always_inline)) {
        constexpr int U = JCAP / JT;
        const uint32_t n = min(min(s_cnt, s_lim), JCAP);
        uint2 pr[U];
        uint64_t kept[U];
        uint32_t tot = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t e = u * JT + tid;
            bool keep = e < n;
            pr[u] = make_uint2(0, 0);
            if (keep) {
                pr[u] = s_pair[e];
                keep = !in_earlier_table(g, pr[u].x, pr[u].y, s_pt[e]);
            }
            kept[u] = __ballot(keep);
            tot += (uint32_t)__popcll(kept[u]);
        }
        if (lane == 0)
            s_sum[wv] = tot;
        __syncthreads();   // (every wave has read the list)
        if (tid == 0) {
            uint32_t sum = 0;
            for (int k = 0; k < JT / 64; ++k)
                sum += s_sum[k];
            s_base = sum ? atomicAdd(g.counter, (unsigned long long)sum) : 0ull;
            s_cnt = 0;
            s_lim = 0xffffffffu;
        }
        __syncthreads();
        uint64_t slot = s_base;
        for (int k = 0; k < wv; ++k)
            slot += s_sum[k];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t at = slot + sjk::lanes_below(kept[u]);
            if (((kept[u] >> lane) & 1) && at < g.cap)
                ((sjk::global_pair *)g.pairs)[at] = sjk::pack_pair(pr[u].x, pr[u].y);
            slot += (uint64_t)__popcll(kept[u]);
        }
    };

    acc_t acc[SA][SB];
    // Tile x's matches to the list, or the wave's to a held record.
    auto epilogue = [&](const Tile &x, const uint32_t *idx, const uint8_t *tag, const V *nm) {
        int l = tid;
        asm volatile("" : "+v"(l));
        l &= 63;
        const uint32_t i0 = 64 * wr + 4 * (l >> 5);
        uint32_t w[SB] = {};   // match bits: row block a of column block b at 16 a
#pragma unroll
        for (int a = 0; a < SA; ++a) {
            if (64 * wr + 32 * a >= (int)x.np())
                continue;   // uniform
            const uint32_t il0 = i0 + 32 * a;
            V nx[L2N ? 16 : 1];
            V nmin = V(0);
            if constexpr (L2N) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    nx[r] = nm[il0 + 8 * (r >> 2) + (r & 3)];
                    nmin = r == 0 ? nx[0] : sjk::vmin(nmin, nx[r]);
                }
            }
#pragma unroll
            for (int b = 0; b < SB; ++b) {
                if (128 * wc + 32 * b >= (int)x.nq())
                    continue;   // uniform
                const uint32_t jl = 128 * wc + 32 * b + (l & 31);
                const V ny = L2N ? nm[TILE + jl] : V(0);
                // a necessary condition from the block's largest product (rows
                // and columns past the tile's have norm 0 and products 0 and
                // are excluded below)
                V mx = acc[a][b][0];
#pragma unroll
                for (int r = 1; r < 16; ++r)
                    mx = sjk::vmax(mx, acc[a][b][r]);
                if (__ballot(matches<DT, MET>(mx, nmin, ny, g)) == 0)
                    continue;
                uint32_t m = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const uint32_t il = il0 + 8 * (r >> 2) + (r & 3);
                    const bool ok = il < x.np() && matches<DT, MET>(acc[a][b][r], L2N ? nx[L2N ? r : 0] : V(0), ny, g);
                    m |= ok ? (1u << r) : 0u;
                }
                w[b] |= (jl < x.nq() ? m : 0u) << (16 * a);
            }
        }
        static_assert(SB == 4 && SA == 2, "one word per column block");
        if (__ballot((w[0] | w[1] | w[2] | w[3]) != 0) == 0)
            return;
        if (x.packed()) {
            // rows of the same bucket only
#pragma nounroll
            for (int s = 0; s < SA * SB; ++s) {
                uint32_t m = bits_of(w, s), drop = 0;
                const uint32_t tj = tag[TILE + col_of(s, l)];
                while (m) {
                    const int r = __builtin_ctz(m);
                    m &= m - 1;
                    if (tag[row_of(s, l, r)] != tj)
                        drop |= 1u << r;
                }
                drop <<= 16 * (s & 1);
#pragma unroll
                for (int b = 0; b < SB; ++b)
                    w[b] &= b == s >> 1 ? ~drop : ~0u;
            }
        }
        uint32_t tot, pre, base = 0;
        wave_totals(w, tot, pre);
        if (tot == 0)
            return;
        if (l == 0)
            base = atomicAdd(&s_cnt, tot);
        base = __builtin_amdgcn_readfirstlane(base);
        if (base + tot > JCAP) {
            // no room: nor for any later reservation of the tile (entries from the
            // first refused one on are not read)
            uint32_t k = 0;
            if (l == 0) {
                atomicMin(&s_lim, base);
                k = atomicAdd(&s_held, 1u);
            }
            k = __builtin_amdgcn_readfirstlane(k);
            if (k < g.held_cap) {   // always: a workgroup stops before its records are full
                Held *hd = g.held + (uint64_t)blockIdx.x * g.held_cap + k;
#pragma unroll
                for (int b = 0; b < SB; ++b)
                    hd->w[b][l] = w[b];
                hd->p[l] = idx[64 * wr + l];
                hd->q[l] = idx[TILE + 128 * wc + l];
                hd->q[64 + l] = idx[TILE + 128 * wc + 64 + l];
                if (l == 0)
                    hd->t = x.t();
            }
            return;
        }
        uint32_t at = base + pre;
#pragma nounroll
        for (int s = 0; s < SA * SB; ++s) {
            uint32_t m = bits_of(w, s);
            const uint32_t j = idx[TILE + col_of(s, l)];
            while (m) {
                const int r = __builtin_ctz(m);
                m &= m - 1;
                s_pair[at] = make_uint2(idx[row_of(s, l, r)], j);
                s_pt[at++] = (uint8_t)x.t();
            }
        }
    };

    // ---- prologue: indices of the first two tiles, the first tile's norms and
    // first stage
    uint64_t left = T1 - T0;   // tiles from the current one on
    uint32_t idx0, tag0;
    Tile cur = take(idx0, tag0);
    s_idx[0][tid] = idx0;
    s_tag[0][tid] = (uint8_t)tag0;
    if constexpr (L2N)
        s_norm[0][tid] = norm_load(idx0);
    Tile nxt = cur;
    if (left > 1) {
        nxt = take(idx0, tag0);
        s_idx[1][tid] = idx0;
        s_tag[1][tid] = (uint8_t)tag0;
    }
    Tile pend = nxt;   // the one after the next
    if (tid == 0) {
        s_cnt = s_held = 0;
        s_lim = 0xffffffffu;
    }
    __syncthreads();
    rows_issue(s_idx[0], 0, s_r0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    uint32_t k3 = 0, par = 0, st = 0;   // current tile mod 3 and mod 2, its stage
    auto stage = [&](const uint8_t *buf, uint8_t *oth) __attribute__((always_inline)) -> bool {
        const uint32_t n3 = k3 == 2 ? 0 : k3 + 1, f3 = n3 == 2 ? 0 : n3 + 1;
        const bool first = st == 0, last = st + 1 == n_st;
        // loads ahead
        uint32_t idx = 0xffffffffu, tag = 0;
        V nrm = V(0);
        if (first && left > 2)
            pend = take(idx, tag);
        if (last && left > 1) {
            if constexpr (L2N)
                nrm = norm_load(s_idx[n3][tid]);
            rows_issue(s_idx[n3], 0, oth);
        } else if (!last) {
            rows_issue(s_idx[k3], st + 1, oth);
        }
        // products
        if (64 * wr < (int)cur.np() && 128 * wc < (int)cur.nq()) {   // uniform
            if (first) {
#pragma unroll
                for (int a = 0; a < SA; ++a)
#pragma unroll
                    for (int b = 0; b < SB; ++b)
                        acc[a][b] = acc_t{};
            }
            const uint32_t nks = min(4u, (rb - 128 * st + 31) / 32);
            const uint32_t sw = (c32 >> 1) & 7;   // (row / 2) % 8 of every row this lane reads
            const uint8_t *pa = buf + (64 * wr + c32) * 128;
            const uint8_t *pb = buf + (TILE + 128 * wc + c32) * 128;
#pragma unroll
            for (uint32_t ks = 0; ks < 4; ++ks)
                if (ks < nks) {
                    const uint32_t o = 16 * ((2 * ks + half) ^ sw);
                    i32x4 fa[SA], fb[SB];
#pragma unroll
                    for (int a = 0; a < SA; ++a)
                        fa[a] = *(const i32x4 *)(pa + 32 * 128 * a + o);
#pragma unroll
                    for (int b = 0; b < SB; ++b)
                        fb[b] = *(const i32x4 *)(pb + 32 * 128 * b + o);
#pragma unroll
                    for (int a = 0; a < SA; ++a)
#pragma unroll
                        for (int b = 0; b < SB; ++b)
                            acc[a][b] = M::mma(fa[a], fb[b], acc[a][b]);
                }
            if (last)
                epilogue(cur, s_idx[k3], s_tag[k3], s_norm[par]);
        }
        __builtin_amdgcn_s_waitcnt(0);   // this stage's loads landed
        if (first && left > 2) {
            s_idx[f3][tid] = idx;
            s_tag[f3][tid] = (uint8_t)tag;
        }
        if constexpr (L2N) {
            if (last && left > 1)
                s_norm[par ^ 1][tid] = nrm;
        }
        __syncthreads();
        if (last) {
            // (both read by every wave before the next tile's matches change them)
            const uint32_t n_list = s_cnt, n_held = s_held;
            // a tile's waves may hold one record each
            const bool stop = left == 1 || n_held + JT / 64 > g.held_cap;   // uniform
            if (n_list >= JCAP / 2 || stop)
                resolve_list();
            else
                __syncthreads();
            --left;
            if (stop) {
                if (tid == 0) {
                    g.n_held[blockIdx.x] = n_held;
                    g.next[blockIdx.x] = T1 - left;
                }
                return false;
            }
            cur = nxt;
            nxt = pend;
            k3 = n3;
            par ^= 1;
            st = 0;
        } else {
            ++st;
        }
        return true;
    };
    for (;;) {
        if (!stage(s_r0, s_r1) || !stage(s_r1, s_r0))
            break;
    }
}

// The held records of every workgroup of join_kernel: the first-table rule on their
// bits, then the pairs.  Four waves per record, one for each column block; workgroups
// (b, *) take b's records, two at a time.  The rows' fingerprints wait in LDS; a lane
// tests its bits there (its column's bytes against its rows') and looks keys up only
// for the ones with an equal byte, four pairs' first at once.  The pairs are written
// by ballots, contiguous over the lanes, with one reservation for the two records.
// Where join_kernel's waves resolved such matches one after the other from
// memory, with a reservation per 32 x 32 block: 50000 x 100 int8, 16 tables x 10 signs, 14.7 M
// pairs, a call 1975 us, now 826; 262144 x 64 int8, one table of 10, 23.9 M pairs 1758
// and 679.
constexpr int HT = 512, HR = HT / 256;   // threads, records

__global__ void __launch_bounds__(HT) held_kernel(JoinArgs g)
{
    constexpr int RN = 192;           // rows of a record: 64 of P, 128 of Q
    extern __shared__ uint4 s_fp[];   // [record][chunk][row]
    __shared__ uint32_t s_row[HR][RN];
    __shared__ uint32_t s_sum[HT / 64];
    __shared__ unsigned long long s_base;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, c32 = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = wv >> 2, b = wv & 3;
    const uint32_t n = g.n_held[blockIdx.x], fc = fp_chunks(g.L);
    uint4 *fp = s_fp + (size_t)h * fc * RN;
    const uint32_t *rows = s_row[h];
    const int jl = 64 + 32 * b + c32;   // this lane's column
    // bit x of a word: row block x / 16, register x % 16
    auto row_of = [&](int x) { return 2 * (x & 28) + 4 * half + (x & 3); };
    for (uint32_t k0 = HR * blockIdx.y; k0 < n; k0 += HR * gridDim.y) {   // uniform
        const bool on = k0 + h < n;   // uniform for a record's waves
        const Held *hd = g.held + ((uint64_t)blockIdx.x * g.held_cap + k0 + h);
        uint32_t w = 0, t = 0, tf = 0;
        if (on) {
            w = hd->w[b][lane];
            t = __builtin_amdgcn_readfirstlane(hd->t);
            tf = min(t, FP_MAX);
            const int r = tid & 255;
            if (r < RN) {
                const uint32_t i = r < 64 ? hd->p[r] : hd->q[r - 64];
                s_row[h][r] = i;
                if (i != 0xffffffffu)
                    for (uint32_t c = 0; 16 * c < tf; ++c)
                        fp[c * RN + r] = (r < 64 ? g.fp_p : g.fp_q)[(size_t)i * fc + c];
            }
        }
        __syncthreads();
        if (t != 0) {
            uint32_t maybe = t > FP_MAX ? w : 0u;
            for (uint32_t c = 0; 16 * c < tf; ++c) {
                const uint4 fj = fp[c * RN + jl];
                uint32_t mm = w & ~maybe;
                while (mm) {
                    const int x = __builtin_ctz(mm);
                    mm &= mm - 1;
                    if (equal_bytes(fp[c * RN + row_of(x)], fj, tf - 16 * c))
                        maybe |= 1u << x;
                }
            }
            const uint32_t j = rows[jl];
            while (maybe) {
                constexpr int K = 4;
                uint32_t bit[K];
                uint64_t kp[K], kq[K];
#pragma unroll
                for (int u = 0; u < K; ++u) {
                    bit[u] = maybe & (0u - maybe);
                    maybe &= maybe - 1u;
                    const int il = bit[u] ? row_of(__builtin_ctz(bit[u])) : 0;
                    uint32_t eq = 0, c = 0;
                    if (bit[u])
                        for (; 16 * c < tf; ++c)
                            if ((eq = equal_bytes(fp[c * RN + il], fp[c * RN + jl], tf - 16 * c)))
                                break;
                    kp[u] = 0;
                    kq[u] = 1;
                    if (eq) {   // (none: the pair goes through the other tables)
                        const size_t t2 = 16 * c + __builtin_ctz(eq);
                        kp[u] = g.keys_p[t2 * g.P.n + rows[il]];
                        kq[u] = g.keys_q[t2 * g.Q.n + j];
                    }
                }
#pragma unroll
                for (int u = 0; u < K; ++u)
                    if (kp[u] == kq[u] ||
                        (bit[u] && in_earlier_table(g, rows[row_of(__builtin_ctz(bit[u]))], j, t)))
                        w &= ~bit[u];
            }
        }
        const uint32_t cnt = (uint32_t)__builtin_popcount(w);
        uint32_t tot = 0;
#pragma unroll
        for (int u = 0; u < 6; ++u)
            tot += (uint32_t)__popcll(__ballot((cnt >> u) & 1)) << u;
        if (lane == 0)
            s_sum[wv] = tot;
        __syncthreads();
        if (tid == 0) {
            uint32_t sum = 0;
            for (int u = 0; u < HT / 64; ++u)
                sum += s_sum[u];
            s_base = sum ? atomicAdd(g.counter, (unsigned long long)sum) : 0ull;
        }
        __syncthreads();
        if (tot) {
            uint64_t slot = s_base;
            for (int u = 0; u < wv; ++u)
                slot += s_sum[u];
            const uint32_t j = rows[jl];
#pragma nounroll
            for (int x = 0; x < 32; ++x) {
                const bool set = (w >> x) & 1u;
                const uint64_t bits = __ballot(set);
                if (bits == 0)
                    continue;
                const uint64_t at = slot + sjk::lanes_below(bits);
                if (set && at < g.cap)
                    ((sjk::global_pair *)g.pairs)[at] = sjk::pack_pair(rows[row_of(x)], j);
                slot += (uint64_t)__popcll(bits);
            }
        }
        __syncthreads();   // the rows and sums are read
    }
}

// After join_kernel: host[0] = pairs so far, host[1] = held records, host[2] =
// workgroups with tiles left; the counter is cleared when that is all.
__global__ void __launch_bounds__(256) join_state_kernel(unsigned long long *counter,
                                                         const uint32_t *n_held,
                                                         const uint64_t *next, uint64_t n_tiles,
                                                         uint32_t grid, unsigned long long *host)
{
    __shared__ uint32_t s_h, s_l;
    if (threadIdx.x == 0)
        s_h = s_l = 0;
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < grid; b += 256) {
        if (n_held[b])
            atomicAdd(&s_h, n_held[b]);
        if (next[b] < (uint64_t)(b + 1) * n_tiles / grid)
            atomicAdd(&s_l, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        host[0] = *counter;
        host[1] = s_h;
        host[2] = s_l;
        if (s_h == 0 && s_l == 0)
            *counter = 0ull;
    }
}

// Fingerprints (sj_lsh.h), a thread per row and 16 tables: byte t is the top
// byte of keys[t n + row] times an odd constant, so rows with equal keys in
// table t have equal bytes t (and rows with different keys rarely do).
__global__ void __launch_bounds__(256) fingerprint_kernel(const uint64_t *keys, uint32_t n,
                                                          uint32_t L, uint32_t fc, uint4 *fp)
{
    const uint32_t row = blockIdx.x * 256 + threadIdx.x, c = blockIdx.y;
    if (row >= n)
        return;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    const uint32_t t0 = 16 * c, tl = min(L - t0, 16u);
    for (uint32_t t = 0; t < tl; ++t) {
        const uint32_t byte =
            (uint32_t)((keys[(size_t)(t0 + t) * n + row] * 0x9E3779B97F4A7C15ull) >> 56);
        w[t >> 2] |= byte << (8 * (t & 3));
    }
    fp[(size_t)row * fc + c] = make_uint4(w[0], w[1], w[2], w[3]);
}

template <int DT>
hipError_t launch_keys_t(const Rows &r, uint32_t d, uint32_t L, uint32_t k, const void *Aw,
                         const int32_t *B, int32_t w, uint64_t *keys,
                         hipStream_t s)
{
    const dim3 grid((r.n + KROWS - 1) / KROWS);
    const uint32_t rb = padded_d<DT>(d) * (DT == DT_I8 ? 1 : 2);
    if (rb <= KSEG)
        hipLaunchKernelGGL((keys_kernel<DT, false>), grid, dim3(256), 0, s, r, d, L, k,
                           (const typename Chunk<DT>::a_t *)Aw, B, w, keys);
    else
        hipLaunchKernelGGL((keys_kernel<DT, true>), grid, dim3(256), 0, s, r, d, L, k,
                           (const typename Chunk<DT>::a_t *)Aw, B, w, keys);
    return hipGetLastError();
}

template <int DT, int MET>
hipError_t launch_join_t(const JoinArgs &g, uint32_t grid, hipStream_t s)
{
    // the row gathers' 32-bit offsets reach 4 GiB
    const uint64_t far = (uint64_t)max(g.P.n, g.Q.n) * g.P.row_bytes;
    if (far < 0xffffffffull)
        hipLaunchKernelGGL((join_kernel<DT, MET, false>), dim3(grid), dim3(JT), 0, s, g);
    else
        hipLaunchKernelGGL((join_kernel<DT, MET, true>), dim3(grid), dim3(JT), 0, s, g);
    return hipGetLastError();
}

}  // namespace

uint32_t key_bits(uint32_t k, int32_t w)
{
    if (k == 0)
        return 1;
    if (w == 0)
        return k;
    const uint32_t b = (64 / k) * k;
    return b > 64 ? 64 : b;
}

size_t widened_bytes(int dtype, uint32_t L, uint32_t k, uint32_t d)
{
    return dtype == DT_I8 ? (size_t)L * k * padded_d<DT_I8>(d) * 4
                          : (size_t)L * k * padded_d<DT_F16>(d) * 8;
}

hipError_t launch_keys(int dtype, const Rows &r, uint32_t d, uint32_t L, uint32_t k,
                       const void *Aw, const int32_t *B, int32_t w,
                       uint64_t *keys, hipStream_t s)
{
    if (r.n == 0 || L == 0)
        return hipSuccess;
    switch (dtype) {
    case DT_F16:
        return launch_keys_t<DT_F16>(r, d, L, k, Aw, B, w, keys, s);
    case DT_BF16:
        return launch_keys_t<DT_BF16>(r, d, L, k, Aw, B, w, keys, s);
    default:
        return launch_keys_t<DT_I8>(r, d, L, k, Aw, B, w, keys, s);
    }
}

bool keys_fast_applies(int dtype, uint32_t row_bytes, uint32_t L, uint32_t k, int32_t w)
{
    return row_bytes <= 512 && k >= 1 &&
           (uint64_t)L * k <= HF_MAX && L <= 64 && (w == 0 || k >= 2);
}

size_t keys_fast_bytes(uint32_t n_max, uint32_t L, uint32_t k, uint32_t row_bytes)
{
    // fp16 / bf16 projection rows, their norms, the fix queue
    return (size_t)L * k * row_bytes + 256 + (size_t)L * k * 4 + 256 + (size_t)L * n_max * 16;
}

template <int DT, int KS>
static void launch_mfma_t(const Rows &r, uint32_t L, uint32_t k, const uint8_t *Ah,
                          const float *an, const int32_t *B, int32_t w, float gam, uint64_t *keys,
                          uint4 *fix, unsigned long long *nfix, hipStream_t s)
{
    const dim3 grid((r.n + 127) / 128);
    if (w > 0)
        hipLaunchKernelGGL((keys_mfma_kernel<DT, KS, true>), grid, dim3(256), 0, s, r, L, k, Ah,
                           an, B, w, gam, keys, fix, nfix);
    else
        hipLaunchKernelGGL((keys_mfma_kernel<DT, KS, false>), grid, dim3(256), 0, s, r, L, k, Ah,
                           an, B, w, gam, keys, fix, nfix);
}

template <int DT>
static hipError_t keys_fast_t(const Rows &r, uint32_t d, uint32_t L, uint32_t k,
                              const int8_t *A, const void *Aw, const int32_t *B, int32_t w, uint64_t *keys, uint8_t *ws, bool widen,
                              unsigned long long *nfix, hipStream_t s)
{
    const uint32_t nf = L * k;
    uint8_t *Ah = ws;
    float *an = (float *)(ws + (((size_t)nf * r.row_bytes + 255) & ~(size_t)255));
    uint4 *fix = (uint4 *)((uint8_t *)an + (((size_t)nf * 4 + 255) & ~(size_t)255));
    if constexpr (DT == DT_I8) {
        // the projection rows as int8 operand rows; sums exact: no norms, no queue
        if (widen) {
            const uint64_t n_out = (uint64_t)nf * r.row_bytes;
            hipLaunchKernelGGL(pad_b_kernel, dim3((unsigned)((n_out + 255) / 256)), dim3(256), 0,
                               s, A, (int8_t *)Ah, d, r.row_bytes, n_out);
        }
    } else {
        if (widen) {
            const uint32_t rl = r.row_bytes / 2;
            const uint64_t n_out = (uint64_t)nf * rl;
            hipLaunchKernelGGL(widen_h_kernel<DT>, dim3((unsigned)((n_out + 255) / 256)),
                               dim3(256), 0, s, A, (uint16_t *)Ah, d, rl, n_out);
            hipLaunchKernelGGL(anorm_kernel, dim3(nf), dim3(64), 0, s, A, d, an);
        }
    }
    // twice the fp32 and double summation bounds for d terms
    const double dd = d ? (double)d : 1.0;
    const double g24 = dd * 0x1p-24 / (1.0 - dd * 0x1p-24);
    const double g53 = dd * 0x1p-53 / (1.0 - dd * 0x1p-53);
    const float gam = (float)(2.0 * (g24 + g53) * (1.0 + 0x1p-10));
    const uint32_t ks = (r.row_bytes + 31) / 32;
    if (ks <= 2)
        launch_mfma_t<DT, 2>(r, L, k, Ah, an, B, w, gam, keys, fix, nfix, s);
    else if (ks <= 4)
        launch_mfma_t<DT, 4>(r, L, k, Ah, an, B, w, gam, keys, fix, nfix, s);
    else if (ks <= 8)
        launch_mfma_t<DT, 8>(r, L, k, Ah, an, B, w, gam, keys, fix, nfix, s);
    else
        launch_mfma_t<DT, 16>(r, L, k, Ah, an, B, w, gam, keys, fix, nfix, s);
    if constexpr (DT != DT_I8)
        hipLaunchKernelGGL(fix_kernel<DT>, dim3(512), dim3(256), 0, s, r, d, k,
                           (const typename Chunk<DT>::a_t *)Aw, B, w, fix,
                           (const unsigned long long *)nfix, keys);
    return hipGetLastError();
}

hipError_t launch_keys_fast(int dtype, const Rows &r, uint32_t d, uint32_t L, uint32_t k,
                            const int8_t *A, const void *Aw, const int32_t *B, int32_t w, uint64_t *keys, void *ws, bool widen,
                            unsigned long long *nfix, hipStream_t s)
{
    if (r.n == 0)
        return hipSuccess;
    if (dtype == DT_F16)
        return keys_fast_t<DT_F16>(r, d, L, k, A, Aw, B, w, keys, (uint8_t *)ws, widen,
                                   nfix, s);
    if (dtype == DT_I8)
        return keys_fast_t<DT_I8>(r, d, L, k, A, Aw, B, w, keys, (uint8_t *)ws, widen,
                                  nfix, s);
    return keys_fast_t<DT_BF16>(r, d, L, k, A, Aw, B, w, keys, (uint8_t *)ws, widen,
                                nfix, s);
}

hipError_t launch_widen(int dtype, const int8_t *A, uint32_t n_fn, uint32_t d, void *out,
                        hipStream_t s)
{
    const uint32_t dp = dtype == DT_I8 ? padded_d<DT_I8>(d) : padded_d<DT_F16>(d);
    const uint64_t n = (uint64_t)n_fn * dp;
    if (n == 0)
        return hipSuccess;
    const dim3 grid((unsigned)((n + 255) / 256));
    if (dtype == DT_I8)
        hipLaunchKernelGGL(widen_kernel<int32_t>, grid, dim3(256), 0, s, A, (int32_t *)out, d,
                           dp, n);
    else
        hipLaunchKernelGGL(widen_kernel<double>, grid, dim3(256), 0, s, A, (double *)out, d, dp,
                           n);
    return hipGetLastError();
}

hipError_t launch_fingerprints(const uint64_t *keys, uint32_t n, uint32_t L, uint4 *fp,
                               hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    const uint32_t fc = fp_chunks(L);
    hipLaunchKernelGGL(fingerprint_kernel, dim3((n + 255) / 256, fc), dim3(256), 0, s, keys, n, L,
                       fc, fp);
    return hipGetLastError();
}

hipError_t launch_bucket_find(const uint64_t *sorted_p, uint32_t n_p, const uint64_t *sorted_q,
                              uint32_t n_q, uint32_t L, void *ws, uint4 *tmp, uint32_t *n_rec,
                              unsigned long long *n_cand, hipStream_t s)
{
    if (n_p == 0 || n_q == 0 || L == 0)
        return hipSuccess;
    const uint32_t nb = find_blocks(n_p);
    const uint64_t nr = (uint64_t)nb * L;
    // workspace: the block sums, then the block ranges of Q
    ulonglong2 *part = (ulonglong2 *)ws;
    uint2 *qr = (uint2 *)(part + nr);
    hipLaunchKernelGGL(qrange_kernel, dim3((uint32_t)((nr + 255) / 256)), dim3(256), 0, s,
                       sorted_p, n_p, sorted_q, n_q, L, qr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(bucket_find_kernel, dim3(nb, L), dim3(256), 0, s, sorted_p, n_p, sorted_q,
                       n_q, (const uint2 *)qr, tmp, n_rec, part);
    e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(sum_parts_kernel, dim3(1), dim3(1024), 0, s, (const ulonglong2 *)ws,
                       (uint64_t)nb * L, n_cand);
    return hipGetLastError();
}

hipError_t launch_bucket_write(uint32_t n_p, uint32_t L, const uint4 *tmp, const uint32_t *n_rec,
                               const unsigned long long *rec_off, const Records &rec,
                               hipStream_t s)
{
    const uint32_t nb = find_blocks(n_p);
    const uint64_t n_blk = (uint64_t)nb * L;
    if (n_blk == 0)
        return hipSuccess;
    hipLaunchKernelGGL(bucket_write_kernel, dim3((uint32_t)((n_blk + 3) / 4)), dim3(256), 0, s, nb,
                       n_blk, tmp, n_rec, rec_off, rec);
    return hipGetLastError();
}

hipError_t launch_pack(const Records &rec, uint32_t n_rec, bool write, uint32_t *chunk_desc,
                       uint32_t *chunk_tiles, const unsigned long long *desc_off,
                       const unsigned long long *tile_off, const Descs &desc, const Lists &ls,
                       unsigned long long *overflow, hipStream_t s)
{
    if (n_rec == 0)
        return hipSuccess;
    hipLaunchKernelGGL(pack_kernel, dim3((n_rec + PACK_CHUNK - 1) / PACK_CHUNK), dim3(256), 0, s,
                       rec, n_rec, write ? 1 : 0, chunk_desc, chunk_tiles, desc_off, tile_off,
                       desc, ls, overflow);
    return hipGetLastError();
}

uint32_t join_grid(uint64_t n_tiles, uint64_t held, int num_cus)
{
    // one workgroup per CU (their LDS fills it), and room for a tile's records each
    uint64_t n = (uint64_t)num_cus;
    n = n < n_tiles ? n : n_tiles;
    n = n < held / HELD_MIN ? n : held / HELD_MIN;
    return (uint32_t)n;
}

hipError_t launch_join(int dtype, int metric, const JoinArgs &g, uint32_t grid, hipStream_t s)
{
    static_assert(HELD_MIN == JT / 64, "a record per wave");
    if (grid == 0)
        return hipSuccess;
    const bool l2 = metric == MET_L2;
    switch (dtype) {
    case DT_F16:
        return l2 ? launch_join_t<DT_F16, MET_L2>(g, grid, s)
                  : launch_join_t<DT_F16, MET_IP>(g, grid, s);
    case DT_BF16:
        return l2 ? launch_join_t<DT_BF16, MET_L2>(g, grid, s)
                  : launch_join_t<DT_BF16, MET_IP>(g, grid, s);
    default:
        return l2 ? launch_join_t<DT_I8, MET_L2>(g, grid, s)
                  : launch_join_t<DT_I8, MET_IP>(g, grid, s);
    }
}

hipError_t launch_join_state(const JoinArgs &g, uint32_t grid, unsigned long long *host,
                             hipStream_t s)
{
    hipLaunchKernelGGL(join_state_kernel, dim3(1), dim3(256), 0, s, g.counter, g.n_held, g.next,
                       g.n_tiles, grid, host);
    return hipGetLastError();
}

hipError_t launch_held(const JoinArgs &g, uint32_t grid, uint64_t records, hipStream_t s)
{
    if (grid == 0)
        return hipSuccess;
    // workgroups enough for every record were they evenly spread, twice over
    const uint64_t ny = (records + HR * grid - 1) / (HR * (uint64_t)grid) * 2;
    const uint32_t lds = HR * 192 * 16 * fp_chunks(g.L);
    hipLaunchKernelGGL(held_kernel, dim3(grid, (uint32_t)(ny < 256 ? ny : 256)), dim3(HT), lds, s, g);
    return hipGetLastError();
}

}  // namespace sjl
