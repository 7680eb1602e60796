// sj_lsh.h -- interface between the LSH-bucketed join's host code (sj_lsh_api.cpp)
// and its gfx950 kernels (sj_lsh.hip).  Not part of the public C-ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sjl {

// Rows of one operand as the kernels read them: n rows of row_bytes bytes
// (a multiple of 16, 16-byte aligned, zero beyond the d stored elements).
struct Rows {
    const uint8_t *X;
    uint32_t n, row_bytes;
};

// Bucket keys of every row in every table, table-major: keys[t * n + i].
// Sign hashes (w == 0) are stored compressed, bit u = v_{t k + u}; quantised
// hashes (w > 0) as the concatenation of their values' low floor(64 / k) bits.
// Either way two rows share a bucket of table t exactly when their keys are
// equal.  key_bits(k, w) is the number of low bits a key can occupy.
// The projection entries come widened by launch_widen (widened_bytes(...)
// bytes: int32 for int8 rows, double otherwise; each row padded with zeros
// to a whole number of 16-byte chunks of the input rows).
uint32_t key_bits(uint32_t k, int32_t w);
size_t widened_bytes(int dtype, uint32_t L, uint32_t k, uint32_t d);
hipError_t launch_widen(int dtype, const int8_t *A, uint32_t n_fn, uint32_t d, void *out,
                        hipStream_t s);
hipError_t launch_keys(int dtype, const Rows &r, uint32_t d, uint32_t L, uint32_t k,
                       const void *Aw, const int32_t *B, int32_t w,
                       uint64_t *keys, hipStream_t s);

// The same keys with the projections on the matrix cores (rows of at most
// 512 bytes, L k <= 512, k >= 2 for quantised hashes:
// keys_fast_applies): decisions the fp32 sums make certain are kept, the
// other (row, table) keys are recomputed exactly.  `ws` is workspace of
// keys_fast_bytes(n_max, L, k, row_bytes) bytes whose first part (the fp16 /
// bf16 projection rows and their norms) is filled when `widen` is set and
// reused otherwise; `nfix` a zeroed device counter per call; Aw as launch_keys.
bool keys_fast_applies(int dtype, uint32_t row_bytes, uint32_t L, uint32_t k, int32_t w);
size_t keys_fast_bytes(uint32_t n_max, uint32_t L, uint32_t k, uint32_t row_bytes);
hipError_t launch_keys_fast(int dtype, const Rows &r, uint32_t d, uint32_t L, uint32_t k,
                            const int8_t *A, const void *Aw, const int32_t *B, int32_t w, uint64_t *keys, void *ws, bool widen,
                            unsigned long long *nfix, hipStream_t s);

// Sorts each table's keys with the row indices as values (n rows per table):
// sorted[t * n + p], perm[t * n + p] = the p-th smallest sort key of table t
// and its row, rows of equal keys in increasing order, where the sort key is
// the key itself when `bits` <= 32 and a fixed bijective mix of it otherwise
// (sj_sort.hip): equal sort keys are exactly equal keys, and every operand is
// sorted in the same order.  `temp` must hold sort_temp_bytes(n, L) bytes;
// `keys` is not modified.
size_t sort_temp_bytes(uint32_t n, uint32_t L);
hipError_t sort_tables(const uint64_t *keys, uint64_t *sorted, uint32_t *perm, uint32_t n,
                       uint32_t L, uint32_t bits, void *temp, hipStream_t s);

// Tile edge of the bucket join (rows of P and of Q per workgroup tile).
constexpr uint32_t TILE = 256;

// The buckets P and Q share, as records in key order within each table,
// tables in order: record r is table t[r] and pq[r] = {p0, np, q0, nq}: P's
// sorted positions [p0, p0 + np) and Q's [q0, q0 + nq) of that table
// (positions within the table's segment).
struct Records {
    uint32_t *t;
    uint4 *pq;
};

// Per row a fingerprint of its keys in the first min(L, 64) tables, in
// fp_chunks(L) chunks of 16 bytes (byte t: 8 bits of a multiplicative hash of
// keys[t n + row]), for the bucket join's first-table rule.
constexpr uint32_t FP_MAX = 64;
constexpr uint32_t fp_chunks(uint32_t L) { return ((L < FP_MAX ? L : FP_MAX) + 15) / 16; }
hipError_t launch_fingerprints(const uint64_t *keys, uint32_t n, uint32_t L, uint4 *fp,
                               hipStream_t s);

// The records, in blocks of 256 sorted positions of P (find_blocks(n_p) per
// table, tables in order): n_rec[block] records at tmp[256 block ..]; writes the
// bucket pairs' pair evaluations (sum of np nq) to n_cand[0] and their rows (sum
// of np + nq) to n_cand[7].  ws: bucket_find_ws_bytes(n_p, L) bytes.
inline uint32_t find_blocks(uint32_t n_p) { return (uint32_t)(((uint64_t)n_p + 255) / 256); }
inline size_t bucket_find_ws_bytes(uint32_t n_p, uint32_t L)
{
    return (size_t)find_blocks(n_p) * L * 24;
}
hipError_t launch_bucket_find(const uint64_t *sorted_p, uint32_t n_p, const uint64_t *sorted_q,
                              uint32_t n_q, uint32_t L, void *ws, uint4 *tmp, uint32_t *n_rec,
                              unsigned long long *n_cand, hipStream_t s);
// Writes them one after the other (rec_off: exclusive scan of n_rec).
hipError_t launch_bucket_write(uint32_t n_p, uint32_t L, const uint4 *tmp, const uint32_t *n_rec,
                               const unsigned long long *rec_off, const Records &rec,
                               hipStream_t s);

// Tiles.  The records are cut into chunks of PACK_CHUNK; within a chunk,
// consecutive records of one table that each fit one tile (np, nq <= TILE) are
// packed greedily into groups of at most TILE P rows and TILE Q rows, one tile
// per group, and every other record is tiled alone by ceil(np / TILE) x
// ceil(nq / TILE) tiles.  A descriptor is pq = {p0, np, q0, nq} and info =
// {table, packed, first tile (64 bits)}: P's rows of the tiles are the entries
// [t n_p + p0, + np) of the sorted permutation, or, for a group, of list_p, where
// the group's rows (a subset of the sorted positions from its first record's
// on) are written one after the other with their record's place in the group
// in tag_p; Q's alike.
// count pass (write = false): per chunk the number of descriptors and of
// tiles (chunk_desc, chunk_tiles; *overflow set when a chunk's tiles do not
// fit 32 bits); write pass: the descriptors at desc_off[chunk] with tiles
// numbered from tile_off[chunk], and the lists.
constexpr uint32_t PACK_CHUNK = 128;
struct Descs {
    uint4 *pq, *info;
};
struct Lists {
    uint32_t n_p, n_q;
    const uint32_t *perm_p, *perm_q;      // L x n sorted position -> row
    uint32_t *list_p, *list_q;            // L x n
    uint8_t *tag_p, *tag_q;               // L x n
};
hipError_t launch_pack(const Records &rec, uint32_t n_rec, bool write, uint32_t *chunk_desc,
                       uint32_t *chunk_tiles, const unsigned long long *desc_off,
                       const unsigned long long *tile_off, const Descs &desc, const Lists &ls,
                       unsigned long long *overflow, hipStream_t s);

// A wave's matches of one tile that found no room in the join's list: match bits of
// its 64 x 128 results (four column blocks of 32; lane l's word b: bit x is row 32 (x /
// 16) + 8 (x % 16 / 4) + 4 (l / 32) + x % 4, column 32 b + l % 32), the rows they
// stand for (0xffffffff: none) and the tile's table.
struct Held {
    uint32_t w[4][64], p[64], q[128], t, pad[3];
};
constexpr uint32_t HELD_MIN = 8;   // records a tile may need

struct JoinArgs {
    Rows P, Q;
    uint32_t L;
    Lists ls;
    const uint64_t *keys_p, *keys_q;      // L x n row -> key (first-table rule)
    const uint4 *fp_p, *fp_q;             // per row: launch_fingerprints
    Descs desc;
    uint32_t n_desc;
    uint64_t n_tiles;
    float thr_f;                          // as sjk::JoinArgs
    int32_t thr_i;
    const void *norm_p, *norm_q;
    uint32_t *pairs;
    uint64_t cap;
    unsigned long long *counter;
    Held *held;                           // held_cap records per workgroup (at least HELD_MIN)
    uint32_t held_cap;
    uint32_t *n_held;                     // per workgroup: records held
    uint64_t *next;                       // per workgroup: the tile it goes on with
    bool resume;
};

// The join takes launches of join_grid(..) workgroups (`held`: records in all): a
// workgroup stops when its records may not hold another tile's.  launch_join_state
// tells (host: pinned memory, read after synchronising) the pairs so far, the records
// held and the workgroups with tiles left, and clears the pair counter when both are
// 0; launch_held resolves the records; then, with tiles left, launch_join again with
// `resume`.
uint32_t join_grid(uint64_t n_tiles, uint64_t held, int num_cus);
hipError_t launch_join(int dtype, int metric, const JoinArgs &g, uint32_t grid, hipStream_t s);
hipError_t launch_join_state(const JoinArgs &g, uint32_t grid, unsigned long long *host,
                             hipStream_t s);
hipError_t launch_held(const JoinArgs &g, uint32_t grid, uint64_t records, hipStream_t s);

}  // namespace sjl
