// The range check of a request's rows in the packed batch, shared by every kernel that reads
// qo_indptr (or a plan's copy of it) before it addresses rows with it.
#pragma once
#include <hip/hip_runtime.h>

namespace sv {

// k rows from q0 lie inside a batch of `total` >= 0 rows, 1 <= k <= block. q0 and k may be any
// words: a signed sum of them wraps for packings that are garbage, and a wrapped sum would pass.
// (The unsigned sum of two values below 2^31 does not wrap. Bitwise and: no branches, where the
// attention over ranges took 2% longer with 27 requests of 1000..8191 tokens.)
__device__ inline bool rows_in_batch(int q0, int k, int block, int total) {
    return ((unsigned)k - 1u < (unsigned)block) & (q0 >= 0) & ((unsigned)q0 + (unsigned)k <= (unsigned)total);
}

}  // namespace sv
