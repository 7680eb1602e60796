// sj_jl.hip -- the TCU Johnson-Lindenstrauss transform of Ahle & Silvestri,
// "Similarity Search with Tensor Core Units", Lemma 3 / Theorem 2, on gfx950.
//
// M = (I_{r_l} (x) A_l) ... (I_{r_1} (x) A_1): since I_r (x) A is A copied
// r times along the diagonal, a batch of n row vectors of length r_i c_i,
// read as n r_i rows of c_i entries, is multiplied by A_i^T as one dense
// product, and the result (n r_i rows of k_i entries) read back as n rows of
// r_i k_i entries is the next level's input -- no data moves between levels.
// Each level is an fp32 product Y = X A_i^T on the matrix cores
// (v_mfma_f32_32x32x2_f32); the first level decodes fp16 / bf16 / int8 rows
// exactly to fp32.  Chains of two or three levels whose factors fit LDS run in
// one kernel (jl_chain); others one kernel per level (jl_level).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sj_internal.h"

namespace sjj {

using sjk::DT_BF16;
using sjk::DT_F16;
using sjk::DT_I8;

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int SRC_F32 = 0;

// Rows per workgroup tile and entries of K per LDS chunk (the column blocks
// of 32 a wave keeps accumulators for at once, NCB, are a template argument:
// as many as the level's N needs, up to 4).
constexpr int NCBMAX = 4;
constexpr int TR = 128;
constexpr int KC = 32;
constexpr int XS = KC + 1;   // LDS row stride (floats): lanes of a fragment read distinct banks

// Raw source bits of one entry / four consecutive entries (idx a multiple
// of 4, the row 4-entry aligned), decoded by dec1 / dec4 once they are used:
// loads in flight hold only the raw words.
template <int SRC>
__device__ __forceinline__ uint32_t raw1(const void *X, uint64_t idx)
{
    if constexpr (SRC == SRC_F32)
        return __builtin_bit_cast(uint32_t, ((const float *)X)[idx]);
    else if constexpr (SRC == DT_I8)
        return (uint32_t)(uint8_t)((const int8_t *)X)[idx];
    else
        return ((const uint16_t *)X)[idx];
}

template <int SRC>
__device__ __forceinline__ float dec1(uint32_t w)
{
    if constexpr (SRC == SRC_F32)
        return __builtin_bit_cast(float, w);
    else if constexpr (SRC == DT_I8)
        return (float)(int8_t)w;
    else if constexpr (SRC == DT_F16)
        return (float)__builtin_bit_cast(_Float16, (uint16_t)w);
    else
        return __builtin_bit_cast(float, w << 16);
}

template <int SRC>
__device__ __forceinline__ uint4 raw4(const void *X, uint64_t idx)
{
    if constexpr (SRC == SRC_F32) {
        return *(const uint4 *)((const float *)X + idx);
    } else if constexpr (SRC == DT_I8) {
        return make_uint4(*(const uint32_t *)((const int8_t *)X + idx), 0u, 0u, 0u);
    } else {
        const uint2 w = *(const uint2 *)((const uint16_t *)X + idx);
        return make_uint4(w.x, w.y, 0u, 0u);
    }
}

template <int SRC>
__device__ __forceinline__ void dec4(uint4 w, float (&v)[4])
{
    if constexpr (SRC == SRC_F32) {
        v[0] = __builtin_bit_cast(float, w.x), v[1] = __builtin_bit_cast(float, w.y);
        v[2] = __builtin_bit_cast(float, w.z), v[3] = __builtin_bit_cast(float, w.w);
    } else if constexpr (SRC == DT_I8) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            v[j] = (float)(int8_t)(w.x >> (8 * j));
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            v[j] = dec1<SRC>(((j < 2 ? w.x : w.y) >> (16 * (j & 1))) & 0xffffu);
    }
}

// Y (rows x N, fp32) = X (rows x K) A^T, A N x K fp32 row-major.  A workgroup
// of 4 waves owns TR rows; for each group of NCB column blocks it walks K in
// chunks of KC entries, staging the chunk of its TR rows and of the group's
// rows of A in LDS as fp32 (consecutive threads load consecutive entries of
// a row: coalesced), and wave w multiplies rows 32 w .. 32 w + 31 on the
// matrix cores (per k-step, lane l supplies X[row l % 32][k + l / 32] and
// A[column l % 32][k + l / 32]).  The next chunk's entries are loaded into
// registers (raw) while the current chunk's MFMAs run.  Entries past the
// matrices read as zero; results outside rows x N are not stored.
template <int SRC, bool VEC, int NCB>
__global__ void __launch_bounds__(256, NCB >= 4 ? 2 : 4) jl_level(const void *X, uint64_t rows, uint32_t K,
                                                   const float *A, uint32_t N, float *Y)
{
    __shared__ float sx[TR * XS];
    __shared__ float sa[32 * NCB * XS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, c32 = lane & 31;
    const uint64_t tile0 = (uint64_t)blockIdx.x * TR;
    const uint64_t row0 = tile0 + 32 * wave;
    // per thread: XQ quads (VEC) or XE entries of X, AE entries of A per chunk
    constexpr int XQ = TR * KC / 4 / 256, XE = TR * KC / 256, AE = 32 * NCB * KC / 256;
    for (uint32_t cb0 = 0; cb0 < N; cb0 += 32 * NCB) {
        // only the column blocks this group uses (whole blocks of 32 rows)
        const uint32_t arows = min((N - cb0 + 31) / 32 * 32, 32u * NCB);
        uint4 rq[VEC ? XQ : 1];
        uint32_t re[VEC ? 1 : XE];
        float ra[AE];
        // this thread's entries: X rows xr + XRS u at column xc (quads: 4
        // entries from xc), A rows ar + 8 u at column ac; element indices from
        // one base per chunk (opaque to the optimiser, so the per-load
        // addresses are not all computed up front and kept)
        constexpr uint32_t XRS = VEC ? 256 / (KC / 4) : 256 / KC;
        const uint32_t xr = VEC ? tid / (KC / 4) : tid / KC;
        const uint32_t xc = VEC ? 4 * (tid % (KC / 4)) : tid % KC;
        const uint32_t ar = tid / KC, ac = tid % KC;
        auto fetch = [&](uint32_t k0) {
            uint64_t xb = (tile0 + xr) * K + k0 + xc;
            asm volatile("" : "+v"(xb));
            const uint64_t xs = (uint64_t)XRS * K;
            const bool kx = k0 + xc < K;
            if constexpr (VEC) {
#pragma unroll
                for (int u = 0; u < XQ; ++u)
                    rq[u] = kx && tile0 + xr + XRS * u < rows ? raw4<SRC>(X, xb + xs * u)
                                                               : make_uint4(0u, 0u, 0u, 0u);
            } else {
#pragma unroll
                for (int u = 0; u < XE; ++u)
                    re[u] = kx && tile0 + xr + XRS * u < rows ? raw1<SRC>(X, xb + xs * u) : 0u;
            }
            uint64_t ab = (uint64_t)(cb0 + ar) * K + k0 + ac;
            asm volatile("" : "+v"(ab));
            const bool ka = k0 + ac < K;
#pragma unroll
            for (int u = 0; u < AE; ++u) {
                const uint32_t r = ar + 8 * u;
                ra[u] = ka && r < arows && cb0 + r < N ? A[ab + (uint64_t)8 * u * K] : 0.0f;
            }
        };
        auto put = [&]() {
            if constexpr (VEC) {
#pragma unroll
                for (int u = 0; u < XQ; ++u) {
                    const int q = tid + 256 * u, r = q / (KC / 4), e = 4 * (q % (KC / 4));
                    float v[4];
                    dec4<SRC>(rq[u], v);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        sx[r * XS + e + j] = v[j];
                }
            } else {
#pragma unroll
                for (int u = 0; u < XE; ++u) {
                    const int q = tid + 256 * u;
                    sx[(q / KC) * XS + q % KC] = dec1<SRC>(re[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < AE; ++u) {
                const int q = tid + 256 * u;
                sa[(q / KC) * XS + q % KC] = ra[u];
            }
        };
        f32x16 acc[NCB];
#pragma unroll
        for (int b = 0; b < NCB; ++b)
            acc[b] = f32x16{};
        fetch(0);
        for (uint32_t k0 = 0; k0 < K; k0 += KC) {
            __syncthreads();   // the previous chunk is consumed
            put();
            if (k0 + KC < K)
                fetch(k0 + KC);   // lands while this chunk's MFMAs run
            __syncthreads();
#pragma unroll
            for (int ks = 0; ks < KC / 2; ++ks) {
                const float a = sx[(32 * wave + c32) * XS + 2 * ks + h];
#pragma unroll
                for (int b = 0; b < NCB; ++b)
                    if (cb0 + 32 * b < N) {   // uniform
                        const float bv = sa[(32 * b + c32) * XS + 2 * ks + h];
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, bv, acc[b], 0, 0, 0);
                    }
            }
        }
        // register r of lane l: (row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32)
#pragma unroll
        for (int b = 0; b < NCB; ++b) {
            const uint32_t col = cb0 + 32 * b + c32;
            if (cb0 + 32 * b >= N || col >= N)
                continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint64_t orow = row0 + 8 * (r >> 2) + 4 * h + (r & 3);
                if (orow < rows)
                    Y[orow * N + col] = acc[b][r];
            }
        }
    }
}

template <int SRC, int NCB>
void launch_level_n(bool vec, uint64_t blocks, const void *X, uint64_t rows, uint32_t K,
                    const float *A, uint32_t N, float *Y, hipStream_t s)
{
    if (vec)
        hipLaunchKernelGGL((jl_level<SRC, true, NCB>), dim3((uint32_t)blocks), dim3(256), 0, s, X,
                           rows, K, A, N, Y);
    else
        hipLaunchKernelGGL((jl_level<SRC, false, NCB>), dim3((uint32_t)blocks), dim3(256), 0, s,
                           X, rows, K, A, N, Y);
}

template <int SRC>
hipError_t launch_level_t(const void *X, uint64_t rows, uint32_t K, const float *A, uint32_t N,
                          float *Y, hipStream_t s)
{
    const uint64_t blocks = (rows + TR - 1) / TR;
    const size_t esz = SRC == SRC_F32 ? 4 : SRC == DT_I8 ? 1 : 2;
    const bool vec = K % 4 == 0 && (uintptr_t)X % (4 * esz) == 0;
    if (N <= 32)
        launch_level_n<SRC, 1>(vec, blocks, X, rows, K, A, N, Y, s);
    else if (N <= 64)
        launch_level_n<SRC, 2>(vec, blocks, X, rows, K, A, N, Y, s);
    else
        launch_level_n<SRC, NCBMAX>(vec, blocks, X, rows, K, A, N, Y, s);
    return hipGetLastError();
}

// One level: Y (rows x N) = X (rows x K) A^T; src = 0 for fp32 rows, else the
// dtype code of the caller's rows.
hipError_t launch_level(int src, const void *X, uint64_t rows, uint32_t K, const float *A,
                        uint32_t N, float *Y, hipStream_t s)
{
    if (rows == 0 || N == 0)
        return hipSuccess;
    switch (src) {
    case SRC_F32: return launch_level_t<SRC_F32>(X, rows, K, A, N, Y, s);
    case DT_F16: return launch_level_t<DT_F16>(X, rows, K, A, N, Y, s);
    case DT_BF16: return launch_level_t<DT_BF16>(X, rows, K, A, N, Y, s);
    case DT_I8: return launch_level_t<DT_I8>(X, rows, K, A, N, Y, s);
    }
    return hipErrorInvalidValue;
}

// ------------------------------------------------- all levels in one kernel
//
// A wave takes 32 of the batch's rows through every level, the intermediate
// values in its registers.  Each product is taken transposed, D = A_i X^T: lane
// l of the result holds features 8 (r / 4) + 4 (l / 32) + r % 4 (register r) of
// row l % 32, and as the other operand of the next level's product register r of
// the two halves is one step's pair of features of that row, so a result is the
// next level's operand as it stands when the next factor's columns are taken in
// that order.  The order of a sum is free, so LDS holds every factor as the lanes
// read it: four consecutive columns of a row (float4) per half and four steps,
// at [(4 steps) * 2 + half][row].  The levels are walked depth first (a level-1
// product row is added to its level-2 row as soon as it is complete, and so on),
// which keeps B1 + B2 + B3 blocks of 32 x 32 per wave whatever r_1 is.
// Bound by the fp32 matrix cores: 262144 x 256 fp16 to 32 (zeta = 2) are 10.7
// GFLOP, 68 us at their peak; HBM moves X and Y only (168 MB, 21 us at 8 TB/s)
// where a kernel per level moves every level's values out and in (705 MB): that
// call 180 -> 111 us (the kernel alone 96 us, traced from a cold clock), 32768 rows
// of 1024 to 16 (zeta = 4) 51 -> 34 us.
struct ChainArgs {
    const uint8_t *X;
    const float *A;
    float *Y;
    uint32_t n, row_bytes;
    uint32_t k1, c1, k2, c2, k3, c3;   // level sizes (k3 = c3 = 0: two levels)
    uint32_t z1, z2;                   // level-1 rows per level-2 row, level-2 rows per level-3 row
};

typedef int jl_i32x4 __attribute__((ext_vector_type(4)));
typedef float jl_f32x4 __attribute__((ext_vector_type(4)));

// Element e of a 16-byte chunk.
template <int SRC>
__device__ __forceinline__ float chunk_at(const jl_i32x4 &v, int e)
{
    if constexpr (SRC == DT_I8)
        return (float)(int8_t)((uint32_t)v[e >> 2] >> (8 * (e & 3)));
    else
        return dec1<SRC>(((uint32_t)v[e >> 1] >> (16 * (e & 1))) & 0xffffu);
}

// A factor (N x K, N padded with zero rows to 32 B) as the lanes read it; col(kq, h):
// the first of the four columns of steps 4 kq .. 4 kq + 3 in half h.
template <int B, typename F>
__device__ __forceinline__ void stage_factor(jl_f32x4 *dst, const float *A, uint32_t N, uint32_t K,
                                             F col)
{
    for (uint32_t i = threadIdx.x; i < K / 4 * 32 * B; i += blockDim.x) {
        const uint32_t o = i % (32 * B), hq = i / (32 * B);
        jl_f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (o < N)
            __builtin_memcpy(&v, A + (size_t)o * K + col(hq >> 1, hq & 1), 16);
        dst[i] = v;
    }
}

// acc += A_{i+1}[:, one level-i row's features] * those features (k of them in x,
// first float4 step kq0); w: the factor at this lane's half and row.
template <int BI, int BO>
__device__ __forceinline__ void chain_step(const f32x16 (&x)[BI], uint32_t k, uint32_t kq0,
                                           const jl_f32x4 *w, f32x16 (&acc)[BO])
{
#pragma unroll
    for (int ib = 0; ib < BI; ++ib)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (32u * ib + 8u * q < k) {   // uniform
                const jl_f32x4 *wq = w + (size_t)(kq0 + 4 * ib + q) * 64 * BO;
                jl_f32x4 f[BO];
#pragma unroll
                for (int b = 0; b < BO; ++b)
                    f[b] = wq[32 * b];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int b = 0; b < BO; ++b)
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(f[b][e], x[ib][4 * q + e],
                                                                      acc[b], 0, 0, 0);
            }
}

constexpr int CHAIN_T = 512;   // threads

// B1, B2, B3: 32-feature blocks of the levels (B3 = 0: two levels); SC: 32-byte
// pieces of a row loaded at once (a whole number of times in a level-1 row);
// CAP: float4 of factors LDS holds (two workgroups per CU up to 80 KB).
template <int SRC, int B1, int B2, int B3, int SC, int CAP>
__global__ void __launch_bounds__(CHAIN_T, CAP <= 5120 ? 4 : 2) jl_chain(ChainArgs g)
{
    constexpr int E = SRC == DT_I8 ? 16 : 8;   // elements per 16-byte chunk
    constexpr int BL = B3 ? B3 : B2;
    __shared__ jl_f32x4 s_w[CAP];
    const int lane = threadIdx.x & 63, h = lane >> 5, c32 = lane & 31;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    jl_f32x4 *w1 = s_w, *w2 = w1 + g.c1 * 8 * B1, *w3 = w2 + g.c2 * 8 * B2;
    // level 1: half h holds chunk h of each 32-byte piece of a row
    stage_factor<B1>(w1, g.A, g.k1, g.c1, [](uint32_t kq, uint32_t hh) {
        return kq / (E / 4) * 2 * E + hh * E + kq % (E / 4) * 4;
    });
    auto packed = [](uint32_t kq, uint32_t hh) { return 8 * kq + 4 * hh; };
    const float *A2 = g.A + (size_t)g.k1 * g.c1;
    stage_factor<B2>(w2, A2, g.k2, g.c2, packed);
    if constexpr (B3 != 0)
        stage_factor<B3>(w3, A2 + (size_t)g.k2 * g.c2, g.k3, g.c3, packed);
    __syncthreads();
    w1 += 32 * B1 * h + c32;
    w2 += 32 * B2 * h + c32;
    w3 += 32 * B3 * h + c32;

    // blocks of 32 rows, dealt over the workgroups first
    const uint32_t n_blk = (uint32_t)(((uint64_t)g.n + 31) / 32), step = gridDim.x * (CHAIN_T / 64);
    const uint32_t spc = g.c1 * (SRC == DT_I8 ? 1 : 2) / (32 * SC);   // loads per level-1 row
    auto row_at = [&](uint64_t blk) {   // rows past the batch read its last one
        const uint64_t r = 32 * blk + c32;
        return g.X + (size_t)(r < g.n ? r : g.n - 1) * g.row_bytes + 16 * h;
    };
    uint32_t blk = wave * gridDim.x + blockIdx.x;
    if (blk >= n_blk)
        return;
    jl_i32x4 xv[SC];
    const uint8_t *at = row_at(blk);
#pragma unroll
    for (int c = 0; c < SC; ++c)
        xv[c] = *(const jl_i32x4 *)(at + 32 * c);
    for (;;) {
        const uint8_t *end = at + g.row_bytes, *after = row_at((uint64_t)blk + step);
        f32x16 last[BL];
#pragma unroll
        for (int b = 0; b < BL; ++b)
            last[b] = f32x16{};
        for (uint32_t j2 = 0; j2 < g.z2; ++j2) {
            f32x16 acc2[B2];
#pragma unroll
            for (int b = 0; b < B2; ++b)
                acc2[b] = f32x16{};
            for (uint32_t j1 = 0; j1 < g.z1; ++j1) {
                f32x16 acc1[B1];
#pragma unroll
                for (int b = 0; b < B1; ++b)
                    acc1[b] = f32x16{};
                for (uint32_t s = 0; s < spc; ++s) {
                    // the row's next piece, or the next row's first
                    at += 32 * SC;
                    if (at == end)
                        at = after;
                    jl_i32x4 xn[SC];
#pragma unroll
                    for (int c = 0; c < SC; ++c)
                        xn[c] = *(const jl_i32x4 *)(at + 32 * c);
                    const jl_f32x4 *ws = w1 + (size_t)s * (SC * (E / 4)) * 64 * B1;
#pragma unroll
                    for (int c = 0; c < SC; ++c)
#pragma unroll
                        for (int q = 0; q < E / 4; ++q) {
                            jl_f32x4 f[B1];
#pragma unroll
                            for (int b = 0; b < B1; ++b)
                                f[b] = ws[(c * (E / 4) + q) * 64 * B1 + 32 * b];
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float x = chunk_at<SRC>(xv[c], 4 * q + e);
#pragma unroll
                                for (int b = 0; b < B1; ++b)
                                    acc1[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                                        f[b][e], x, acc1[b], 0, 0, 0);
                            }
                        }
#pragma unroll
                    for (int c = 0; c < SC; ++c)
                        xv[c] = xn[c];
                }
                if constexpr (B3 != 0)
                    chain_step<B1, B2>(acc1, g.k1, j1 * (g.k1 / 8), w2, acc2);
                else
                    chain_step<B1, B2>(acc1, g.k1, j1 * (g.k1 / 8), w2, last);
            }
            if constexpr (B3 != 0)
                chain_step<B2, B3>(acc2, g.k2, j2 * (g.k2 / 8), w3, last);
        }
        const uint64_t row = 32 * (uint64_t)blk + c32;
        if (row < g.n) {
            const uint32_t kl = B3 ? g.k3 : g.k2;
            float *y = g.Y + row * kl + 4 * h;
#pragma unroll
            for (int b = 0; b < BL; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (32u * b + 8u * q < kl)
                        *(jl_f32x4 *)(y + 32 * b + 8 * q) =
                            jl_f32x4{last[b][4 * q], last[b][4 * q + 1], last[b][4 * q + 2],
                                     last[b][4 * q + 3]};
        }
        if (n_blk - blk <= step)
            break;
        blk += step;
    }
}

template <int SRC, int B1, int B2, int B3, int CAP>
hipError_t launch_chain_b(const ChainArgs &g, int num_cus, hipStream_t s)
{
    // one workgroup per CU while it has a wave for every block (its waves spread
    // over the SIMDs: 32768 x 256 fp16 28 us with two, 19 with one), else as many as
    // LDS holds
    const uint64_t n_blk = ((uint64_t)g.n + 31) / 32;
    const uint64_t wgs = (uint64_t)num_cus *
                         (CAP <= 5120 && n_blk > (uint64_t)num_cus * (CHAIN_T / 64) ? 2 : 1);
    const dim3 grid((uint32_t)(n_blk < wgs ? n_blk : wgs));
    const uint32_t piece = g.c1 * (SRC == DT_I8 ? 1 : 2);
    if (piece % 128 == 0)
        hipLaunchKernelGGL((jl_chain<SRC, B1, B2, B3, 4, CAP>), grid, dim3(CHAIN_T), 0, s, g);
    else if (piece % 64 == 0)
        hipLaunchKernelGGL((jl_chain<SRC, B1, B2, B3, 2, CAP>), grid, dim3(CHAIN_T), 0, s, g);
    else
        hipLaunchKernelGGL((jl_chain<SRC, B1, B2, B3, 1, CAP>), grid, dim3(CHAIN_T), 0, s, g);
    return hipGetLastError();
}

// The variants: blocks of each level, float4 of LDS (launch_chain_t).
static const uint32_t kChainB[5][4] = {{1, 1, 0, 5120}, {1, 1, 1, 5120}, {1, 2, 1, 5120},
                                       {2, 2, 0, 10240}, {2, 4, 2, 10240}};

// The variant whose blocks cover the levels' sizes: its number, or -1.
static int chain_variant(const ChainArgs &g)
{
    for (int v = 0; v < 5; ++v) {
        const uint32_t b1 = kChainB[v][0], b2 = kChainB[v][1], b3 = kChainB[v][2];
        if ((b3 != 0) == (g.k3 != 0) && g.k1 <= 32 * b1 && g.k2 <= 32 * b2 && g.k3 <= 32 * b3)
            return (uint64_t)g.c1 * 8 * b1 + (uint64_t)g.c2 * 8 * b2 + (uint64_t)g.c3 * 8 * b3 <=
                           kChainB[v][3]
                       ? v
                       : -1;
    }
    return -1;
}

template <int SRC>
hipError_t launch_chain_t(int v, const ChainArgs &g, int num_cus, hipStream_t s)
{
    switch (v) {
    case 0: return launch_chain_b<SRC, 1, 1, 0, 5120>(g, num_cus, s);
    case 1: return launch_chain_b<SRC, 1, 1, 1, 5120>(g, num_cus, s);
    case 2: return launch_chain_b<SRC, 1, 2, 1, 5120>(g, num_cus, s);
    case 3: return launch_chain_b<SRC, 2, 2, 0, 10240>(g, num_cus, s);
    default: return launch_chain_b<SRC, 2, 4, 2, 10240>(g, num_cus, s);
    }
}

// Whether [a, a + na) and [b, b + nb) have no byte in common.
static bool apart(const void *a, uint64_t na, const void *b, uint64_t nb)
{
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x + na <= y || y + nb <= x;
}

// Whether jl_chain takes the transform: two or three levels, the last of one row;
// sizes k_i in whole quads of both halves (multiples of 8), level-1 rows of whole
// 32-byte pieces, rows and results 16-byte aligned, factors that fit LDS, and
// enough rows: one wave works through 32 rows alone, so few rows leave matrix
// cores idle where a kernel per level spreads their level-1 rows.  Measured (256
// CUs, us, this against a kernel per level): 320 MFMAs per 32 rows, 512 to 32
// (zeta = 4): 8192 rows 17.7 / 15.6, 12288 rows 18.1 / 19.0, 262144 rows 97 / 159;
// 1280, 1024 to 64 (zeta = 4): 16384 rows 55 / 47, 24576 rows 56 / 57, 262144 rows
// 341 / 456; 1664, 2048 to 32 (zeta = 4): 16384 rows 70 / 60, 24576 rows 72 / 78,
// 262144 rows 447 / 700.
// A variant with more blocks of 32 features than the sizes fill multiplies zeros: it pays
// while that is less than what the values between the levels cost in memory, about
// 1.4 MFMAs per 32 rows for each with two levels and 0.75 with three.  200000 fp16 rows, us,
// MFMAs here / by levels and values between: 1088 / 576, 64: 269 / 189; 640 / 384, 128: 171
// / 154; 176 / 112, 48: 73 / 81; 832 / 672, 320: 210 / 241; three levels 1152 / 512, 384: 274 /
// 218; 960 / 544, 320: 235 / 218; 1104 / 808, 336: 261 / 267; 1024 / 1024, 512: 250 / 353.
static bool chain_args(int src, const void *X, uint32_t n, uint32_t d, uint32_t levels,
                       const uint32_t *shape, const float *A, float *Y, int num_cus, ChainArgs *g)
{
    if (levels < 2 || levels > 3)
        return false;
    const uint32_t *l1 = shape, *l2 = shape + 3, *l3 = shape + 6;
    const uint32_t *last = levels == 3 ? l3 : l2;
    const uint64_t es = src == DT_I8 ? 1 : 2;
    if (last[2] != 1 || (l1[0] | l2[0] | last[0]) % 8 != 0 || l1[1] * es % 32 != 0 ||
        l1[2] % l2[2] != 0 || (((uintptr_t)X | (uintptr_t)Y) & 15) != 0)
        return false;
    *g = ChainArgs{(const uint8_t *)X, A, Y, n, (uint32_t)(d * es), l1[0], l1[1], l2[0], l2[1],
                   levels == 3 ? l3[0] : 0, levels == 3 ? l3[1] : 0, l1[2] / l2[2], l2[2]};
    const int v = d * es < ((uint64_t)1 << 32) ? chain_variant(*g) : -1;
    if (v < 0)
        return false;
    // a kernel per level reads the rows before the results are written; here they
    // are written while other rows and the factors are still read
    const uint64_t kl = last[0], factors = (uint64_t)l1[0] * l1[1] + (uint64_t)l2[0] * l2[1] +
                                           (uint64_t)g->k3 * g->c3;
    if (!apart(Y, n * kl * 4, X, n * d * es) || !apart(Y, n * kl * 4, A, factors * 4))
        return false;
    // MFMAs per 32 rows here and by levels, and values between the levels of one row
    const uint32_t kk[3] = {l1[0], l2[0], g->k3}, cc[3] = {l1[1], l2[1], g->c3};
    const uint32_t rr[3] = {l1[2], l2[2], 1};
    uint64_t steps = 0, by_levels = 0, between = 0;
    for (uint32_t i = 0; i < levels; ++i) {
        const uint64_t per_block = (uint64_t)rr[i] * cc[i] / 2;
        steps += per_block * kChainB[v][i];
        by_levels += per_block * ((kk[i] + 31) / 32);
        between += i + 1 < levels ? (uint64_t)rr[i] * kk[i] : 0;
    }
    if ((levels == 2 ? 5 : 4) * (steps - by_levels) > (levels == 2 ? 7 : 3) * between)
        return false;
    return (uint64_t)n >= (steps <= 400 ? 48ull : 96ull) * (uint64_t)num_cus;
}

bool chain_applies(int src, const void *X, uint32_t n, uint32_t d, uint32_t levels,
                   const uint32_t *shape, const float *A, float *Y, int num_cus)
{
    ChainArgs g;
    return chain_args(src, X, n, d, levels, shape, A, Y, num_cus, &g);
}

// The whole transform, where chain_applies.
hipError_t launch_chain(int src, const void *X, uint32_t n, uint32_t d, uint32_t levels,
                        const uint32_t *shape, const float *A, float *Y, int num_cus,
                        hipStream_t s)
{
    ChainArgs g;
    if (!chain_args(src, X, n, d, levels, shape, A, Y, num_cus, &g))
        return hipErrorInvalidValue;
    const int v = chain_variant(g);
    switch (src) {
    case DT_F16: return launch_chain_t<DT_F16>(v, g, num_cus, s);
    case DT_BF16: return launch_chain_t<DT_BF16>(v, g, num_cus, s);
    default: return launch_chain_t<DT_I8>(v, g, num_cus, s);
    }
}

}  // namespace sjj
