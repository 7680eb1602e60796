// sj_lsh_layout.h -- the scratch of one LSH-bucketed join (host arithmetic only).
//
// Arrays that are never needed together share their place, so that the largest
// calls a card holds stay as large as their keys and sort need.  In stream order a
// call writes and reads
//   the rows' copies and norms, keys, sorted rows (perm), counters: throughout;
//   early: the hash's workspaces, then the sorted keys and the sort's workspace,
//          then the shared buckets as found per block;
//   mid:   the buckets' records and the packing's counts, from the found ones;
//   late:  the packed tiles' row lists and the tiles' descriptors, from the records,
//          then the fingerprints and the output a call that sizes its own keeps;
//   last:  the join's held records.
// Late starts where early does; mid follows both; the held records have all that
// late leaves.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace sjl {

// What a call's sizes come to (bytes where not said otherwise).
struct ScratchNeeds {
    uint64_t n_p, n_q, L;
    bool self;                    // Q is P: its arrays are P's
    size_t copy_row, norm;        // bytes per row of the copies and norms (0: none)
    size_t fingerprint;           // bytes per row
    size_t hash_ws, widened, sort_ws;
    uint64_t find_blocks;         // over all tables, 256 entries of 16 bytes each
    uint64_t records, chunks;     // at most
    size_t scan_partials;
    uint64_t own_pairs;           // 8 bytes each
    uint64_t held_bytes;          // at least, for the join's held records
    uint64_t workgroups;          // of the join
};

struct ScratchLayout {
    size_t row_p, row_q, norm_p, norm_q, key_p, key_q, perm_p, perm_q, counters, n_held, next, partials;
    size_t hash_ws, widened, sorted_p, sorted_q, sort_ws, found, n_found, found_off;   // early
    size_t rec_t, rec_pq, n_desc, n_tile, desc_off, tile_off;                          // mid
    size_t list_p, list_q, tag_p, tag_q, desc_info, desc_pq, fp_p, fp_q, own;          // late
    size_t held, held_bytes;
    size_t early, early_end, late_end, mid, total;
};

inline ScratchLayout scratch_layout(const ScratchNeeds &c)
{
    ScratchLayout y = {};
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t here = at;
        at = (at + bytes + 255) & ~(size_t)255;
        return here;
    };
    const size_t pos_p = c.L * c.n_p, pos_q = c.L * c.n_q;
    // an array of P's and one of Q's, of b bytes per entry
    auto both = [&](size_t &p, size_t &q, size_t entries_p, size_t entries_q, size_t b) {
        p = take(entries_p * b);
        q = c.self ? p : take(entries_q * b);
    };
    both(y.row_p, y.row_q, c.n_p, c.n_q, c.copy_row);
    both(y.norm_p, y.norm_q, c.n_p, c.n_q, c.norm);
    both(y.key_p, y.key_q, pos_p, pos_q, 8);
    both(y.perm_p, y.perm_q, pos_p, pos_q, 4);
    y.counters = take(8 * 8);
    y.n_held = take(c.workgroups * 4);
    y.next = take(c.workgroups * 8);
    y.partials = take(c.scan_partials);

    y.early = at;
    both(y.sorted_p, y.sorted_q, pos_p, pos_q, 8);
    y.sort_ws = take(c.sort_ws);
    y.found = take(c.find_blocks * 256 * 16);
    y.n_found = take(c.find_blocks * 4);
    y.found_off = take(c.find_blocks * 8);
    y.early_end = at;
    at = y.early;   // the hash is done before the sorts
    y.widened = take(c.widened);
    y.hash_ws = take(c.hash_ws);
    y.early_end = at > y.early_end ? at : y.early_end;

    at = y.early;
    both(y.list_p, y.list_q, pos_p, pos_q, 4);
    both(y.tag_p, y.tag_q, pos_p, pos_q, 1);
    y.desc_info = take(c.records * 16);
    y.desc_pq = take(c.records * 16);
    both(y.fp_p, y.fp_q, c.n_p, c.n_q, c.fingerprint);
    y.own = take(c.own_pairs * 8);
    y.late_end = at;

    y.mid = at = y.late_end > y.early_end ? y.late_end : y.early_end;
    y.rec_t = take(c.records * 4);
    y.rec_pq = take(c.records * 16);
    y.n_desc = take(c.chunks * 4);
    y.n_tile = take(c.chunks * 4);
    y.desc_off = take(c.chunks * 8);
    y.tile_off = take(c.chunks * 8);
    // the held records: all that is left after late, mid's place included
    y.held = y.late_end;
    y.total = at > y.held + c.held_bytes ? at : y.held + c.held_bytes;
    y.held_bytes = y.total - y.held;
    return y;
}

}  // namespace sjl
