// The range check of a request's rows in the packed batch, shared by every kernel that reads
// qo_indptr (or a plan's copy of it) before it addresses rows with it.
#pragma once
#include <hip/hip_runtime.h>

namespace sv {

// k rows from q0 lie inside a batch of `total` rows, 1 <= k <= block. No value of any argument
// overflows: sums of q0 and k wrap for packings that are garbage, and a wrapped sum would pass.
__device__ inline bool rows_in_batch(int q0, int k, int block, int total) {
    return k >= 1 && k <= block && q0 >= 0 && k <= total && q0 <= total - k;
}

}  // namespace sv
