// SpMM of any width in one launch.  Internal.
#pragma once

#include <hip/hip_runtime_api.h>

#include "kernels.h"

namespace rg {

constexpr int kSpmmMax = 32;  // right-hand sides of one launch
// Wavefronts of row groups (eight per CU) from which a launch is bound by its
// loads rather than by their latency.
constexpr int64_t kSpmmBusyWaves = 2048;

struct SpmmFill {
    int64_t rows, slots, nnz;  // of the grouped part
};

// Y = A X for k (2 .. kSpmmMax) right-hand sides, any alignment and leading
// dimension: F32 or F64 stored values, one lane per row.  P as for launch_spmv
// with one row per lane (P.compact = kCompactPattern: columns from the row
// patterns); nwg workgroups stride over P.total_units units.
hipError_t launch_spmm(const SpmvParams &P, const SpmmFill &F, int vdt, int vec_f64, int k, int nwg, hipStream_t st);
// Adds the chunk partial sums of rows over kBlockChunk nonzeros, in order.
hipError_t launch_spmm_combine(const LongItem *items, int32_t n, const int32_t *long_row, const void *partial, void *Y,
                               int64_t ldy, int vec_f64, int k, hipStream_t st);

}  // namespace rg
