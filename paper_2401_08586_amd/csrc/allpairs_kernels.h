// All-list neighbour search for small sets (launchers; the C ABI is in capi.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace nnps {

struct ApBox {
    double lo[3], hi[3];
};

// Largest set the all-list path takes (its work grows as n^2).
constexpr int kAllPairsMaxN = 65536;

// Count: row_ptr [n + 1] of the set; host[0] = nnz, host[1] = 1 if a position lies outside
// [lo, hi] or is not finite, else 0 (host: memory that the host reads after the stream).
// flag: a device int, zero before and after.
hipError_t launch_allpairs_count(int dim, int n, const double* pos, double R2, const ApBox& box, int64_t* row_ptr,
                                 int* flag, int64_t* host, hipStream_t st);
// Fill: row i's pairs in ascending j from row_ptr[i] on, never at or past min(row_ptr[i + 1],
// cap); a row whose pairs do not match its count sets kApErrFill in *err.
constexpr int kApErrFill = 1;
hipError_t launch_allpairs_fill(int dim, int n, const double* pos, double R2, const int64_t* row_ptr, int32_t* col,
                                float* dist, int64_t cap, int* err, hipStream_t st);

}  // namespace nnps
