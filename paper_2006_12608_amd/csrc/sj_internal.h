// sj_internal.h -- interface between the host API (sj_api.cpp) and the gfx950
// kernels (sj_kernels_*.hip).  Not part of the public C-ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sjk {

// DT_FP4: rows of 4-bit floats (two per byte), made by the Hamming front end
// only; the kernels count its rows in bytes like every other type's.
enum { DT_F16 = 1, DT_BF16 = 2, DT_I8 = 3, DT_FP4 = 4 };
enum { MET_IP = 0, MET_L2 = 1 };

// What the fused epilogue does with the matches it finds.
enum Mode {
    MODE_SINGLE = 0,  // append through one atomic counter per wave (single pass)
    MODE_COUNT = 1,   // count the matches of every output block, write no pairs
    MODE_EMIT = 2,    // write each block's matches at its precomputed offset
    MODE_MASK = 3,    // count as MODE_COUNT and keep every result's match bit
                      // (K-streamed kernel only), for an emit pass that reads
                      // the bits instead of recomputing the product
    MODE_RECORD = 4,  // count as MODE_COUNT and append one MatchRecord per
                      // 32x32 block with matches to the workgroup's own list
                      // (resident kernel only), for an emit pass that reads
                      // the records instead of recomputing
    MODE_TRI = 5      // single pass of a self-join (Q is P) over the upper
                      // triangle only: tiles below the diagonal are skipped,
                      // each match (i, j) with i < j is written as (i, j) and
                      // (j, i), and (i, i) once
};

// The matches of one 32x32 block of results, as found by the first pass of
// count-then-emit (MODE_RECORD): the block's output block, the number of that
// output block's matches that precede this block's, the block's first row and
// column, and 64 lane masks in the MFMA accumulator layout (bit r of lane l's
// mask is row i0 + 8 (r / 4) + 4 (l / 32) + r % 4, column j0 + l % 32).
struct MatchRecord {
    uint64_t blk;
    uint32_t pos, i0, j0, pad[3];
    uint16_t mask[64];
};
static_assert(sizeof(MatchRecord) == 160, "record layout");

// Kernel families.
enum Family {
    FAM_RESIDENT = 1,  // P rows held in VGPRs for the whole of d; Q tiles streamed via LDS
    FAM_STREAMED = 2   // both operands streamed through LDS in K chunks (large d)
};

// Tile geometry of the K-streamed kernel, shared by its planner and by the
// pass that emits pairs from its match bits: workgroup tiles of ST_BM rows of
// P by ST_BN rows of Q, ST_NW waves, each owning ST_SA x ST_SB blocks of 32x32
// results (rows 32 ST_SA wave_row + ..., columns 32 ST_SB wave_col + ...; the
// waves of a workgroup form a (ST_NW / 2) x 2 grid).  One output block per
// wave and tile.
constexpr int ST_BM = 256, ST_BN = 256, ST_NW = 8, ST_SA = 2, ST_SB = 4;
static_assert(ST_BM == 32 * ST_SA * (ST_NW / 2) && ST_BN == 32 * ST_SB * 2, "wave grid");
// Match bits of one output block: ST_SA * ST_SB blocks of 32x32 results as
// 16-bit lane masks in the MFMA accumulator layout (bit r of lane l's mask is
// row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of the block), stored
// lane-major: lane l's masks of blocks s = column block * ST_SA + row block
// are the 16 contiguous bytes [16 l, 16 l + 16) (mask s in bytes 2 s, 2 s + 1).
constexpr uint32_t ST_MASK_WORDS = ST_SA * ST_SB * 64;
static_assert(ST_SA * ST_SB == 8, "one 16-byte access per lane");

struct JoinArgs {
    const uint8_t *P;            // n_p rows of row_bytes bytes
    const uint8_t *Q;            // n_q rows of row_bytes bytes
    uint32_t n_p, n_q;
    uint32_t row_bytes;          // bytes per row: a multiple of 16, rows 16-byte aligned
    float thr_f;                 // fp16/bf16: IP s32 (acc >= thr_f); L2 r2_32
    int32_t thr_i;               // int8: IP ceil(s) (acc >= thr_i); L2 floor(r2)
    const void *norm_p;          // L2: squared norms of P rows (int32 for int8, float otherwise)
    const void *norm_q;          // L2: squared norms of Q rows
    uint32_t *pairs;             // cap x {i, j}
    uint64_t cap;
    unsigned long long *counter; // MODE_SINGLE: running match count
    uint32_t *block_counts;      // MODE_COUNT: one count per output block
    const unsigned long long *block_offsets;  // MODE_EMIT: exclusive prefix of block_counts
    uint16_t *masks;             // MODE_MASK: ST_MASK_WORDS per output block
    MatchRecord *records;        // MODE_RECORD: rec_cap records per workgroup, by workgroup
    uint32_t rec_cap;
    uint32_t *rec_counts;        // MODE_RECORD: records found per workgroup (may pass rec_cap)
    uint32_t qsplit;             // FAM_RESIDENT: Q ranges per P block
};

// A launch decided by plan_join; the count and emit passes of one call use the
// same plan so that their output blocks coincide.
struct Plan {
    int family;
    int variant;                 // index into the family's instantiation table
    uint32_t grid, block;        // FAM_STREAMED: tile numbers (a workgroup takes several)
    uint32_t cus;                // FAM_STREAMED: workgroups at most
    uint32_t qsplit;
    bool small;                  // FAM_RESIDENT: the small geometry (sj_join_kernels.h)
    uint64_t n_blocks;           // number of output blocks (entries of block_counts)
    uint64_t wg_blocks32;        // FAM_RESIDENT: most 32x32 result blocks of one workgroup
};

// Chooses the kernel for (dtype, metric, shape) on a GPU with `num_cus` CUs
// (small_ok: the small geometry may be taken; MODE_TRI has none, and its
// smaller output blocks need a little more room in count-then-emit's arrays).
// Returns false when the shape is unsupported.
bool plan_join(int dtype, int metric, uint32_t n_p, uint32_t n_q, uint32_t row_bytes,
               bool small_ok, int num_cus, Plan *plan);

hipError_t launch_join(const Plan &plan, int dtype, int metric, int mode, const JoinArgs &args,
                       hipStream_t stream);

// Second pass of count-then-emit for the K-streamed kernel after a MODE_MASK
// first pass: every output block's pairs from its match bits, written at its
// offset in the same order as a MODE_EMIT pass (reads g.masks, g.block_counts,
// g.block_offsets; writes g.pairs below g.cap).
hipError_t launch_emit_masks(const Plan &plan, const JoinArgs &g, hipStream_t stream);

// Second pass of count-then-emit after a MODE_RECORD first pass of the
// resident kernel (n_wg workgroups, none with more than rec_cap records): the
// pairs of every record, each written at its output block's offset plus its
// position, in the order of a MODE_EMIT pass.
hipError_t launch_emit_records(const JoinArgs &g, uint32_t n_wg, hipStream_t stream);

// The rows of both operands as the kernels read them, in one launch: copies of
// rows of src_bytes bytes (any alignment) in rows of row_bytes bytes (a multiple
// of 16, zero-filled tail) when copy_p / copy_q are not null, and squared row
// norms (int32 for int8, fp32 otherwise) when norm_p / norm_q are not null (both
// or neither operand; without copies src_bytes == row_bytes, rows 16-byte
// aligned).  n_q = 0 when Q is P.
hipError_t launch_prep(int dtype, const void *P, uint32_t n_p, const void *Q, uint32_t n_q,
                       uint32_t src_bytes, uint32_t row_bytes, uint8_t *copy_p, uint8_t *copy_q,
                       void *norm_p, void *norm_q, hipStream_t stream);

// Section 4's cosine front end: Y (n x d, 16-bit) = every row of X (n x d of
// dtype, row-major) divided by its Euclidean norm (double, ascending k) and
// rounded to the nearest binary16 (fp16 and int8 inputs) or bfloat16 (bf16
// inputs), ties to even; zero rows give zeros.
hipError_t launch_normalize(int dtype, const void *X, uint32_t n, uint32_t d, void *Y,
                            hipStream_t stream);

// Hamming front end: bit rows (ceil(d / 8) bytes, coordinate m in bit m % 8 of
// byte m / 8) to rows of 4-bit floats of out_bytes bytes (a multiple of 16, at
// least d / 2): coordinate m is +1 or -1 (bit 0 or 1) in nibble m, nibbles past
// d are 0, so that the inner product of two rows is d - 2 Hamming(x, y).
hipError_t launch_unpack_hamming(const uint8_t *bits, uint32_t n, uint32_t d, uint32_t out_bytes,
                                 uint8_t *out, hipStream_t stream);

// Zeroes n 64-bit words on `stream` (one small kernel, no memset node).
hipError_t launch_zero_u64(unsigned long long *p, uint32_t n, hipStream_t stream);

// Writes *counter to host[0] (pinned host memory) and clears it.
hipError_t launch_publish(unsigned long long *counter, unsigned long long *host,
                          hipStream_t stream);

// Exclusive scan of n uint32 counts into n uint64 offsets; *total receives the
// sum.  `partials` needs scan_partials_size(n) elements of scratch.  With `host`
// (pinned host memory) the sum also goes to host[0] and the largest of the
// n_max values at `max_of` (may be none) to host[1].
uint64_t scan_partials_size(uint64_t n);
hipError_t launch_scan(const uint32_t *counts, uint64_t n, unsigned long long *offsets,
                       unsigned long long *partials, unsigned long long *total,
                       hipStream_t stream, unsigned long long *host = nullptr,
                       const uint32_t *max_of = nullptr, uint32_t n_max = 0);

// Launchers and occupancy (workgroups of a resident-kernel variant that one CU
// holds at once) per element type and metric, one translation unit each.
#define SJ_JOIN_DECL(NAME)                                                            \
    hipError_t launch_join_##NAME(const Plan &, int mode, const JoinArgs &, hipStream_t); \
    int resident_occupancy_##NAME(int variant);
SJ_JOIN_DECL(f16_ip)
SJ_JOIN_DECL(f16_l2)
SJ_JOIN_DECL(bf16_ip)
SJ_JOIN_DECL(bf16_l2)
SJ_JOIN_DECL(i8_ip)
SJ_JOIN_DECL(i8_l2)
SJ_JOIN_DECL(fp4_ip)
#undef SJ_JOIN_DECL

}  // namespace sjk
