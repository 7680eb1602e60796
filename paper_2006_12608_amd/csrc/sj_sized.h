// sj_sized.h -- joins whose output the library sizes and the caller allocates
// half-way: the entry points the Python binding's calls without a capacity use.
// Not part of the public C-ABI.
//
// A caller of the public entry points that does not know the number of pairs
// counts first and joins again, which computes the product twice (or hashes and
// sorts twice).  These run the counting pass once, call `alloc` with the number
// of pairs (not when it is 0) on the calling thread, and write the pairs to the
// device memory it returns, with the checks, order, flags and errors of the
// public call with that buffer.  A NULL from `alloc` ends the call with
// SJ_E_NOMEM.  Nothing is kept from one call for the next.
#pragma once

#include "sj.h"

extern "C" {

typedef void *(*sj_alloc_fn)(void *user, uint64_t n_pairs);

// kind 0: sj_join_ip, 1: sj_join_l2, 2: sj_join_hamming (dtype ignored), each
// with SJ_FLAG_TWO_PASS implied.
int sji_join_sized(sj_ctx *ctx, int kind, int dtype, const void *P, uint32_t n_p, const void *Q,
                   uint32_t n_q, uint32_t d, double thr, sj_alloc_fn alloc, void *user,
                   uint64_t *n_out, unsigned flags);

// sj_join_lsh.
int sji_lsh_sized(sj_ctx *ctx, int metric, int dtype, const void *P, uint32_t n_p, const void *Q,
                  uint32_t n_q, uint32_t d, double thr, uint32_t L, uint32_t k, const int8_t *A,
                  const int32_t *B, int32_t w, sj_alloc_fn alloc, void *user, uint64_t *n_out,
                  uint64_t *n_cand);

}  // extern "C"

namespace sjh {

// The allocation half-way: set in a request, null in the public calls.
struct Sized {
    sj_alloc_fn alloc;
    void *user;
};

}  // namespace sjh
