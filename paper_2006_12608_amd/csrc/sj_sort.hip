// sj_sort.hip -- the sort of the LSH-bucketed join (Section 4: the points of a
// table are grouped by bucket): every table's n keys sorted with their rows,
// on gfx950.
//
// Only the grouping of equal keys matters, so a table's keys are sorted in
// the order of a bijective mix of them, m(key), when they use more than 32
// bits: 32-bit sort keys (the key itself, or the top half of m(key)) are
// sorted with their rows, the low half of m(key) of every sorted position is
// then gathered through the permutation, and the rare runs whose top halves are
// equal but whose m differ are put in the order of m by a local sort.  The
// outputs are the sorted m(key) (or keys) and their rows; equal outputs are
// exactly equal keys, and P and Q are sorted in one order.
//
// The 32-bit sort is a stable least-significant-digit radix sort over 8-bit
// digits, run on all L tables at once: each table is a segment of n entries,
// each segment is cut into blocks of SORT_TILE entries, and every pass is
//   sort_hist:    per (segment, block, digit) counts of the pass's digit;
//   column_sums:  per (segment, digit) the running sums of the counts over the
//                 blocks, in their place, and the total (sort_columns or
//                 sort_runs, by the number of blocks);
//   sort_scatter: each block ranks its entries stably by digit (wave ballots
//                 find the lanes that share a digit; a per-wave running count
//                 per digit continues the rank across the wave's rounds), puts
//                 them in digit order in LDS and writes each digit's run to its
//                 position (s n, since every segment holds n entries, + the
//                 segment's smaller digits + the digit's earlier blocks), so a
//                 block's stores are contiguous runs.
// A block's counts lie together: laid out [segment][digit][block] for one scan
// over all of them, every count was a store and a load of 4 and 8 bytes in a line
// of its own (16 tables of 1048576 entries: counts 44 -> 36 us, sums 30 -> 7 us a
// pass; the LSH call on 1048576 x 64 int8 5719 -> 5527 us, 262144 x 256 fp16 2633 ->
// 2568 us).
// Bound by HBM: each pass reads the sort keys twice and the rows once and
// writes both (20 bytes per entry).
#include "sj_internal.h"
#include "sj_lsh.h"
#include "sj_search.h"

namespace sjl {

constexpr int SORT_T = 256;                    // threads per block (4 waves)
constexpr int SORT_IPT = 8;                    // entries per thread
constexpr int SORT_TILE = SORT_T * SORT_IPT;   // entries per block
constexpr int SORT_BITS = 8;                   // digit width
constexpr int SORT_BINS = 1 << SORT_BITS;
static_assert(SORT_BINS == SORT_T, "one thread per digit in the block-wide steps");

// Counts of the digit (key >> shift) & mask in block `blk` of segment `seg`.
__global__ void __launch_bounds__(SORT_T) sort_hist(const uint32_t *keys, uint32_t n, uint32_t bps,
                                                    uint32_t shift, uint32_t mask, uint32_t *hist)
{
    __shared__ uint32_t cnt[SORT_T / 64][SORT_BINS];
    const uint32_t b = blockIdx.x, seg = b / bps, blk = b - seg * bps;
    const int tid = threadIdx.x, wave = tid >> 6;
    for (int i = tid; i < (SORT_T / 64) * SORT_BINS; i += SORT_T)
        (&cnt[0][0])[i] = 0u;
    __syncthreads();
    const uint64_t base = (uint64_t)seg * n;
    const uint32_t lo = blk * SORT_TILE, entries = block_entries(blk, SORT_TILE, n);
    // all of this thread's keys are loaded before the first count
    uint32_t dg[SORT_IPT];
#pragma unroll
    for (int r = 0; r < SORT_IPT; ++r) {
        const uint32_t i = r * SORT_T + tid;
        dg[r] = i < entries ? (keys[base + lo + i] >> shift) & mask : 0xffffffffu;
    }
#pragma unroll
    for (int r = 0; r < SORT_IPT; ++r)
        if (dg[r] != 0xffffffffu)
            atomicAdd(&cnt[wave][dg[r]], 1u);
    __syncthreads();
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < SORT_T / 64; ++w)
        c += cnt[w][tid];
    hist[(uint64_t)b * SORT_BINS + tid] = c;
}

// Runs of at most RUN_B blocks of a segment, a workgroup each, a thread per digit
// (every block's counts are one coalesced load).  SUMS: the run's sums to part[run].
// Otherwise the counts become their exclusive sums in place, from part[run] on
// (part null: the segment is one run, whose totals are written).
constexpr uint32_t RUN_B = 64;

template <bool SUMS>
__global__ void __launch_bounds__(SORT_BINS) sort_runs(uint32_t *hist, uint32_t bps, uint32_t runs,
                                                       uint32_t *part, uint32_t *total)
{
    const uint32_t b = blockIdx.x, seg = b / runs, dg = threadIdx.x;
    const uint32_t b0 = (b - seg * runs) * RUN_B, b1 = min(b0 + RUN_B, bps);
    uint32_t *h = hist + (uint64_t)seg * bps * SORT_BINS + dg;
    const uint64_t at = (uint64_t)b * SORT_BINS + dg;
    uint32_t run = SUMS || !part ? 0u : part[at];
#pragma unroll 16
    for (uint32_t k = b0; k < b1; ++k) {
        const uint32_t v = h[(uint64_t)k * SORT_BINS];
        if constexpr (!SUMS)
            h[(uint64_t)k * SORT_BINS] = run;
        run += v;
    }
    if constexpr (SUMS)
        part[at] = run;
    else if (!part)
        total[at] = run;
}

// The counts of COL_D digits of one segment: their exclusive sums over the
// segment's blocks, in place, and the digits' totals.  COL_C threads share a digit,
// a run of blocks each (loaded twice; the second time from cache).
constexpr int COL_D = 8, COL_C = 128;
constexpr uint32_t kColSegs = 1u << 20;   // segments of one launch

__global__ void __launch_bounds__(COL_D * COL_C) sort_columns(uint32_t *hist, uint32_t bps,
                                                              uint32_t *total)
{
    __shared__ uint32_t s_sum[COL_C][COL_D];
    const uint32_t d = threadIdx.x % COL_D, c = threadIdx.x / COL_D, seg = blockIdx.x;
    const uint32_t dg = blockIdx.y * COL_D + d;
    const uint32_t per = (bps + COL_C - 1) / COL_C;
    const uint32_t b0 = min(c * per, bps), b1 = min(b0 + per, bps);
    uint32_t *h = hist + (uint64_t)seg * bps * SORT_BINS + dg;
    uint32_t sum = 0;
#pragma unroll 8
    for (uint32_t b = b0; b < b1; ++b)
        sum += h[(uint64_t)b * SORT_BINS];
    s_sum[c][d] = sum;
    __syncthreads();
    // inclusive sums over the digit's threads, by doubling steps
    for (uint32_t o = 1; o < COL_C; o <<= 1) {
        const uint32_t up = c >= o ? s_sum[c - o][d] : 0u;
        __syncthreads();
        s_sum[c][d] += up;
        __syncthreads();
    }
    uint32_t run = s_sum[c][d] - sum;
    if (c == COL_C - 1)
        total[seg * SORT_BINS + dg] = s_sum[c][d];
#pragma unroll 8
    for (uint32_t b = b0; b < b1; ++b) {
        const uint32_t v = h[(uint64_t)b * SORT_BINS];
        h[(uint64_t)b * SORT_BINS] = run;
        run += v;
    }
}

__device__ __forceinline__ uint32_t lanes_below_mask(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Exclusive prefix over the block's SORT_T threads of v (one value each).
__device__ __forceinline__ uint32_t block_excl_prefix(uint32_t v, uint32_t *s_w)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(inc, o, 64);
        if (lane >= o)
            inc += u;
    }
    if (lane == 63)
        s_w[wave] = inc;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int w = 0; w < SORT_T / 64; ++w)
        before += w < wave ? s_w[w] : 0u;
    return before + inc - v;
}

// One pass: entries of kin / vin (vin null: the row index, i.e. the entry's
// position in its segment) to kout / vout in stable order of their digit.
// Wave w of a block owns the block's entries [PER_WAVE w, PER_WAVE (w + 1)) and takes
// them 64 at a time in order, so a digit's rank within the block is (its
// count in earlier waves) + (its count in this wave's earlier rounds) + (the
// lanes below with the same digit).
__global__ void __launch_bounds__(SORT_T) sort_scatter(const uint32_t *kin, const uint32_t *vin,
                                                       uint32_t *kout, uint32_t *vout, uint32_t n,
                                                       uint32_t bps, uint32_t shift,
                                                       uint32_t nbits, const uint32_t *offs,
                                                       const uint32_t *total)
{
    __shared__ uint32_t s_k[SORT_TILE];
    __shared__ uint32_t s_v[SORT_TILE];
    __shared__ uint32_t s_run[SORT_T / 64][SORT_BINS];
    __shared__ uint32_t s_start[SORT_BINS];
    __shared__ unsigned long long s_off[SORT_BINS];
    __shared__ uint32_t s_w[2][SORT_T / 64];
    const uint32_t b = blockIdx.x, seg = b / bps, blk = b - seg * bps;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t mask = (1u << nbits) - 1u;
    const uint32_t lo = blk * SORT_TILE;
    const uint32_t cnt = block_entries(blk, SORT_TILE, n);
    const uint64_t base = (uint64_t)seg * n + lo;
    for (int i = tid; i < (SORT_T / 64) * SORT_BINS; i += SORT_T)
        (&s_run[0][0])[i] = 0u;
    __syncthreads();

    constexpr int PER_WAVE = SORT_TILE / (SORT_T / 64);
    uint32_t key[SORT_IPT];
    uint32_t val[SORT_IPT], rank[SORT_IPT];
#pragma unroll
    for (int r = 0; r < SORT_IPT; ++r) {
        const uint32_t li = wave * PER_WAVE + r * 64 + lane;
        const bool valid = li < cnt;
        key[r] = valid ? kin[base + li] : 0u;
        val[r] = valid ? (vin ? vin[base + li] : lo + li) : 0u;
    }
#pragma unroll
    for (int r = 0; r < SORT_IPT; ++r) {
        const uint32_t li = wave * PER_WAVE + r * 64 + lane;
        const bool valid = li < cnt;
        const uint32_t dg = (key[r] >> shift) & mask;
        uint64_t peers = __ballot(valid);
        for (uint32_t bit = 0; bit < nbits; ++bit) {
            const bool set = (dg >> bit) & 1u;
            const uint64_t bal = __ballot(set);
            peers &= set ? bal : ~bal;
        }
        const uint32_t below = lanes_below_mask(peers);
        const uint32_t before = s_run[wave][dg];
        rank[r] = before + below;
        // the group's first lane moves the wave's running count past it
        if (valid && below == 0)
            s_run[wave][dg] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    }
    __syncthreads();
    // digit `tid`: each wave's base (count in earlier waves), the digit's first
    // local position and its first output position
    {
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < SORT_T / 64; ++w) {
            const uint32_t c = s_run[w][tid];
            s_run[w][tid] = run;
            run += c;
        }
        s_start[tid] = block_excl_prefix(run, s_w[0]);
        s_off[tid] = (uint64_t)seg * n + block_excl_prefix(total[seg * SORT_BINS + tid], s_w[1]) +
                     (offs ? offs[(uint64_t)b * SORT_BINS + tid] : 0u);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SORT_IPT; ++r) {
        const uint32_t li = wave * PER_WAVE + r * 64 + lane;
        if (li < cnt) {
            const uint32_t dg = (key[r] >> shift) & mask;
            const uint32_t pos = s_start[dg] + s_run[wave][dg] + rank[r];
            if (pos < (uint32_t)SORT_TILE) {   // always: the ranks are a permutation
                s_k[pos] = key[r];
                s_v[pos] = val[r];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < SORT_IPT; ++j) {
        const uint32_t p = j * SORT_T + tid;
        if (p < cnt) {
            const uint32_t k = s_k[p];
            const uint32_t dg = (k >> shift) & mask;
            const unsigned long long at = s_off[dg] + (p - s_start[dg]);
            if (at < (unsigned long long)n * gridDim.x / bps) {   // within L n
                kout[at] = k;
                vout[at] = s_v[p];
            }
        }
    }
}

// A bijection of 64-bit keys (a multiplication by an odd constant, then an
// xor of the high half into the low half, both invertible).
__device__ __forceinline__ uint64_t mix_key(uint64_t k)
{
    k *= 0x9E3779B97F4A7C15ull;
    return k ^ (k >> 32);
}

// The 32-bit sort keys: the key itself (keys of at most 32 bits) or the top
// half of its mix, whose low half is kept for the gather.
__global__ void __launch_bounds__(256) sort_key_kernel(const uint64_t *keys, uint64_t total,
                                                       int wide, uint32_t *sk, uint32_t *low)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total)
        return;
    if (wide) {
        const uint64_t m = mix_key(keys[i]);
        sk[i] = (uint32_t)(m >> 32);
        low[i] = (uint32_t)m;
    } else {
        sk[i] = (uint32_t)keys[i];
    }
}

// The sorted outputs of keys of at most 32 bits: the sort keys as they stand.
__global__ void __launch_bounds__(256) expand_key_kernel(const uint32_t *sk, uint64_t total,
                                                         uint64_t *sorted)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < total)
        sorted[i] = sk[i];
}

// The sorted outputs of wide keys: the sort key is the mix's top half, the low
// half comes through the permutation (4 bytes of a table's n, not the 8-byte
// key: 16 tables of 1048576 rows 164 us instead of 204, the same with each XCD's
// blocks on tables of their own).  A break is a position
// whose mix differs from its predecessor's within a run of equal top halves;
// the run's first break walks back to the run's first position and lists it, in
// its block's 256 entries of the list (the block's number in n_list; one counter
// for all blocks serialised them: 524000 runs among 67108864 keys, 8.0 ms a call,
// 4.2 by blocks).
__global__ void __launch_bounds__(256) gather_low_kernel(const uint32_t *sk, const uint32_t *low,
                                                         uint32_t n, uint64_t total,
                                                         const uint32_t *perm, uint64_t *sorted,
                                                         uint32_t *list, uint32_t *n_list)
{
    __shared__ uint32_t s_n;
    if (threadIdx.x == 0)
        s_n = 0;
    __syncthreads();
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const bool in = i < total;
    const uint64_t s0 = in ? i / n * n : 0;
    uint32_t k = 0, l = 0;
    if (in) {
        k = sk[i];
        l = low[s0 + perm[i]];
        sorted[i] = ((uint64_t)k << 32) | l;
    }
    // the predecessor, from the lane below (lane 0 reads it)
    uint32_t kp = __shfl_up(k, 1, 64), lp = __shfl_up(l, 1, 64);
    if (in && i != s0) {
        if ((threadIdx.x & 63) == 0) {
            kp = sk[i - 1];
            if (kp == k)
                lp = low[s0 + perm[i - 1]];
        }
        if (kp == k && lp != l) {
            uint64_t a = i - 1;
            bool first = true;   // else an earlier break lists the run
            while (first && a > s0 && sk[a - 1] == k) {
                first = low[s0 + perm[a - 1]] == lp;
                --a;
            }
            if (first)
                list[(uint64_t)blockIdx.x * 256 + atomicAdd(&s_n, 1u)] = (uint32_t)a;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0)
        n_list[blockIdx.x] = s_n;
}

// Sorts every listed run by the mixed key, stably (insertion sort).  Two
// distinct keys share a top half with probability 2^-32, so D distinct keys in
// a table give about D^2 / 2^33 listed runs (about 100 at D = 10^6), each
// joining the rows of two buckets; the cost of a run is its number of
// inversions, at most the product of the two buckets' sizes.  Runs are
// disjoint and each has one first position, so no two threads write the same
// entries.  A thread per block of the list (gather_low_kernel).
__global__ void __launch_bounds__(256) fixup_kernel(const uint32_t *sk, const uint32_t *list,
                                                    const uint32_t *n_list, uint32_t blocks,
                                                    uint32_t n, uint64_t *sorted, uint32_t *perm)
{
    const uint64_t blk = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint32_t n_run = blk < blocks ? n_list[blk] : 0u;
    for (uint32_t x = 0; x < n_run; ++x) {
        const uint64_t i = list[256 * blk + x];
        const uint64_t end = (i / n + 1) * n;
        uint64_t e = i + 1;
        while (e < end && sk[e] == sk[i])
            ++e;
        for (uint64_t a = i + 1; a < e; ++a) {
            const uint64_t k = sorted[a];
            const uint32_t v = perm[a];
            uint64_t b = a;
            while (b > i && sorted[b - 1] > k) {
                sorted[b] = sorted[b - 1];
                perm[b] = perm[b - 1];
                --b;
            }
            sorted[b] = k;
            perm[b] = v;
        }
    }
}

// Blocks per segment, and their runs of RUN_B.
static uint32_t blocks_per_segment(uint32_t n)
{
    return (uint32_t)(((uint64_t)n + SORT_TILE - 1) / SORT_TILE);
}
static uint32_t runs_per_segment(uint32_t bps) { return (bps + RUN_B - 1) / RUN_B; }

size_t sort_temp_bytes(uint32_t n, uint32_t L)
{
    const uint64_t total = (uint64_t)n * L;
    const uint64_t counts = (uint64_t)L * SORT_BINS * blocks_per_segment(n);
    auto up = [](uint64_t x) { return (x + 255) & ~(uint64_t)255; };
    const uint64_t parts = (uint64_t)L * SORT_BINS * runs_per_segment(blocks_per_segment(n));
    return 4 * up(total * 4) + up(counts * 4) + up(parts * 4) + up((uint64_t)L * SORT_BINS * 4);
}

// sort_columns over the counts (or the runs' sums) of L segments.
static hipError_t launch_columns(uint32_t *hist, uint32_t bps, uint32_t L, uint32_t *total,
                                 hipStream_t s)
{
    for (uint64_t l = 0; l < L; l += kColSegs) {   // (fewer than 2^32 threads a launch)
        hipLaunchKernelGGL(sort_columns, dim3((uint32_t)min((uint64_t)L - l, (uint64_t)kColSegs),
                                              SORT_BINS / COL_D),
                           dim3(COL_D * COL_C), 0, s, hist + l * bps * SORT_BINS, bps,
                           total + l * SORT_BINS);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// The counts' exclusive sums over each segment's blocks, in place, and the totals.
// sort_columns has 32 workgroups of 1024 threads per segment: too many for segments
// of a few blocks (1000 tables of 1000 entries, 24 bits: a call 384 us, 71 with
// none; 100000 of 50: 34 ms and 1.5 ms), too few for one segment of many (67108864
// entries: 2764 us, 2247 by runs).  A single run takes 2.2 us and 0.12 for each
// block (25 blocks 5.3), sort_columns 3.8 of 16 segments and 104 of 1000.  By runs and their
// sums, three launches, from 4096 blocks on (1 and 4 tables of 4096 blocks: 313 and
// 1128 us by columns, 288 and 1092 by runs; of 512 blocks 97 and 167 against 113 and
// 179).
static hipError_t column_sums(uint32_t *hist, uint32_t bps, uint32_t runs, uint32_t L,
                              uint32_t *part, uint32_t *total, hipStream_t s)
{
    if (bps <= 1)
        return hipSuccess;   // a block's counts are its segment's totals
    if (runs > 1 ? bps < 4096 : bps > 4 + L / 2)
        return launch_columns(hist, bps, L, total, s);
    if (runs > 1) {
        hipLaunchKernelGGL(sort_runs<true>, dim3(L * runs), dim3(SORT_BINS), 0, s, hist, bps, runs,
                           part, nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || (e = launch_columns(part, runs, L, total, s)) != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL(sort_runs<false>, dim3(L * runs), dim3(SORT_BINS), 0, s, hist, bps, runs,
                       runs > 1 ? part : nullptr, total);
    return hipGetLastError();
}

hipError_t sort_tables(const uint64_t *keys, uint64_t *sorted, uint32_t *perm, uint32_t n,
                       uint32_t L, uint32_t bits, void *temp, hipStream_t s)
{
    if (n == 0 || L == 0)
        return hipSuccess;
    const uint64_t total = (uint64_t)n * L;
    const uint32_t bps = blocks_per_segment(n);
    const uint64_t counts = (uint64_t)L * SORT_BINS * bps;
    auto up = [](uint64_t x) { return (x + 255) & ~(uint64_t)255; };
    uint8_t *t = (uint8_t *)temp;
    uint32_t *ska = (uint32_t *)t;                             // sort keys, two buffers
    uint32_t *skb = (uint32_t *)(t + up(total * 4));
    uint32_t *tv = (uint32_t *)(t + 2 * up(total * 4));        // rows, second buffer
    uint32_t *low = (uint32_t *)(t + 3 * up(total * 4));       // wide keys: low halves
    uint32_t *hist = (uint32_t *)(t + 4 * up(total * 4));
    const uint32_t runs = runs_per_segment(bps);
    const uint64_t parts = (uint64_t)L * SORT_BINS * runs;
    uint32_t *part = (uint32_t *)((uint8_t *)hist + up(counts * 4));
    uint32_t *total_d = (uint32_t *)((uint8_t *)part + up(parts * 4));
    const bool wide = bits > 32;
    const uint32_t sbits = wide ? 32u : bits;
    const dim3 g1((uint32_t)((total + 255) / 256));
    hipLaunchKernelGGL(sort_key_kernel, g1, dim3(256), 0, s, keys, total, wide ? 1 : 0, ska,
                       low);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    // at least one pass (with no key bits it is a stable copy that also
    // writes the rows); the last pass leaves the rows in `perm`
    const uint32_t passes = sbits == 0 ? 1u : (sbits + SORT_BITS - 1) / SORT_BITS;
    const uint32_t grid = L * bps;
    const uint32_t *kin = ska;
    const uint32_t *vin = nullptr;
    for (uint32_t pass = 0; pass < passes; ++pass) {
        const uint32_t shift = pass * SORT_BITS;
        const uint32_t nbits = sbits == 0 ? 0u : min((uint32_t)SORT_BITS, sbits - shift);
        const bool to_out = ((passes - 1 - pass) & 1u) == 0;
        uint32_t *kout = kin == ska ? skb : ska;
        uint32_t *vout = to_out ? perm : tv;
        hipLaunchKernelGGL(sort_hist, dim3(grid), dim3(SORT_T), 0, s, kin, n, bps, shift,
                           (1u << nbits) - 1u, hist);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        if ((e = column_sums(hist, bps, runs, L, part, total_d, s)) != hipSuccess)
            return e;
        hipLaunchKernelGGL(sort_scatter, dim3(grid), dim3(SORT_T), 0, s, kin, vin, kout, vout, n,
                           bps, shift, nbits, bps > 1 ? hist : nullptr, bps > 1 ? total_d : hist);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        kin = kout;
        vin = vout;
    }
    if (!wide) {
        hipLaunchKernelGGL(expand_key_kernel, g1, dim3(256), 0, s, kin, total, sorted);
        return hipGetLastError();
    }
    // the rows' second buffer is free after the last pass, and so are the counts:
    // the list of runs, and each block's number of them
    hipLaunchKernelGGL(gather_low_kernel, g1, dim3(256), 0, s, kin, low, n, total, perm, sorted,
                       tv, hist);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    hipLaunchKernelGGL(fixup_kernel, dim3((g1.x + 255) / 256), dim3(256), 0, s, kin, tv, hist,
                       g1.x, n, sorted, perm);
    return hipGetLastError();
}

}  // namespace sjl
