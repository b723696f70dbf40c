// pasur_sort.hpp -- the radix sort of pasur_sort.hip (not part of the ABI).
#pragma once

#include "pasur_scan.hpp"

namespace pasur {

// Scratch of a sort of n pairs: int32 and int64 words.
int64_t sort_scratch_ints(int64_t n);
int64_t sort_scratch_words(int64_t n);

// Stable sort of n pairs by key.  The pairs are in keys[0]/vals[0]; the sorted
// ones end in keys[*result]/vals[*result], the other pair of arrays holds an
// earlier order.  host: two device-visible words.  Waits once for the stream
// (for the key bits that vary), enqueues the passes and returns.
int sort_pairs(uint64_t *const keys[2], int32_t *const vals[2], int64_t n, int32_t *ints,
               int64_t *words, int64_t *host, int *result, hipStream_t s);

}  // namespace pasur
