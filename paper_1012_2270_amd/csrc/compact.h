// Compact column storage of the grouped rows.  Internal.
//
// The SpMV reads a value and a 32-bit column per nonzero and gathers x at the
// columns once they have arrived, so on matrices whose columns follow a rule
// the column stream is up to two thirds of the bytes, and the gathers a second
// memory latency.  A handle built with the automatic kernel schedule (one lane
// per row, groups that fill whole wavefronts, no long rows) therefore keeps,
// beside the layout's own 32-bit columns, one of two shorter forms of them:
//   row patterns  every row's offsets (column - row) are one of at most 256
//                 lists: one byte per row names the list, the lists sit in a
//                 small table that each workgroup copies to LDS (structured
//                 grids: the row lists of the interior, the faces, the edges
//                 and the corners);
//   x windows     the columns of each workgroup's rows span at most kWinCols:
//                 16-bit offsets from the window's first column, and the
//                 workgroup copies that window of x to LDS and gathers there
//                 (banded matrices).
// Launches over the handle read the compact form instead of the columns; the
// values, the step order within a row and so the results are the same.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <vector>

#include "internal.h"
#include "kernels.h"

namespace rg {

enum { kCompactNone = 0, kCompactPattern = 1, kCompactWindow = 2 };

constexpr int kPatMax = 256;    // row patterns (one byte names one)
constexpr int kPatTab = 2048;   // table entries: an 8 KB copy in LDS per workgroup
constexpr int kPatLen = 255;    // longest row of a pattern
constexpr int kPatHash = 1024;  // hash slots of the search on the device
constexpr int kWinCols = 4096;  // x entries of a window: 16 KB of LDS in FP32, 32 KB in FP64
// Fewer grouped slots than this: no windows.  Such a launch is over in the few
// microseconds that its first loads take, whatever it reads (4.5 to 5.2 us
// either way up to 120,000 slots; 166,000: 4.6 against 5.2 us).
constexpr int64_t kWinMinSlots = int64_t(1) << 17;
// Windows need a layout whose padding is at most its nonzeros (padding is
// stored again and read) and windows that hold no more entries than the slots
// that read them (4 nonzeros a row, half band 1,000: 6.0 against 6.2 us at
// 0.95 entries per slot; 8 and 1,700: 6.7 against 9.3 us).
constexpr bool win_pays(int64_t entries, int64_t slots, int64_t nnz) {
    return entries <= slots && slots - nnz <= nnz;
}

// Row stride of the pattern table: the length, then the offsets (at least
// one, which a masked step may read).
constexpr int32_t pat_stride(int32_t longest) { return longest + 1 > 2 ? longest + 1 : 2; }
// A table pays while it is small against the columns it replaces (each
// workgroup reads it).
constexpr bool pat_pays(int64_t n_pat, int64_t stride, int64_t slots) {
    return n_pat * stride <= kPatTab && n_pat * stride * 8 <= slots;
}

// Rows each lane multiplies per pass: two when they fit 16 steps together and
// the values take 4 bytes or less.
constexpr int compact_rows(int64_t width, int esz) { return width <= 8 && esz < 8 ? 2 : 1; }

// The x entries that a workgroup's rows (kBlockThreads consecutive ones, one
// lane per row) need under the row patterns: for each of n runs of nearby
// offsets, x at its first row + lo and the kBlockThreads + span - 1 entries
// behind it.  The workgroup copies them to LDS, the run's first at `base`, so
// a row's step reads LDS where it would gather.
constexpr int kPatSegs = 9;
struct PatSegs {
    int32_t n = 0;      // 0: not used; entries behind n repeat the last
    int32_t extra = 0;  // sum of the spans
    int32_t total = 0;  // entries in LDS
    int32_t lo[kPatSegs] = {}, span[kPatSegs] = {}, base[kPatSegs] = {};
};
PatSegs pattern_segments(const int32_t *tab, int32_t n_pat, int32_t stride);

struct HostCompact {
    int mode = kCompactNone;
    int32_t rows = 1;              // rows per lane
    int32_t width = 0;             // widest group (patterns)
    int32_t n_pat = 0, stride = 0;
    std::vector<uint8_t> pat_id;   // [ns] pattern of each grouped row
    std::vector<int32_t> pat_tab;  // [n_pat * stride] length, offsets
    PatSegs segs;
    std::vector<int32_t> win;      // [2 * units] first column and column count of each unit's window
    std::vector<uint16_t> col16;   // [slots] column - first column of the unit (0 in padding of empty rows)
};

// Chooses and builds the compact form of layout L (T = 1, G a multiple of 64,
// no long rows; otherwise none).
void build_compact(const HostLayout &L, HostCompact &C);

// The same search on device CSR arrays (convert.hip): ids of the n rows in
// CSR row order, the table, and whether the patterns suffice.  All device
// memory comes from the caller: key [kPatHash] uint64, rep [2 * kPatHash]
// int32, state [4] int32 (key and state zeroed), slot [n] uint16,
// id [n] uint8, tab [kPatTab] int32.  After the stream has run, state[0] is
// the pattern count, state[1] != 0 means no patterns, state[2] is the table's
// row stride.
hipError_t launch_find_patterns(const int64_t *rp, const int32_t *col, int64_t n, uint64_t *key, int32_t *rep,
                                int32_t *state, uint16_t *slot, uint8_t *id, int32_t *tab, hipStream_t st);
// Window of each unit of unit_rows grouped rows (win, as HostCompact), and in
// count[0] the sum of the window sizes and count[1] the widest (both zeroed
// by the caller).
hipError_t launch_windows(const int32_t *sv, const int64_t *rp, const int32_t *col, int64_t ns, int32_t unit_rows,
                          int64_t units, int32_t *win, unsigned long long *count, hipStream_t st);
// id_s[i] = id[sv[i]]
hipError_t launch_gather_id(const int32_t *sv, const uint8_t *id, int64_t ns, uint8_t *id_s, hipStream_t st);
// col16 of the slots of every unit (unit_groups groups each)
hipError_t launch_col16(const int64_t *gp, int64_t ng, int32_t unit_groups, int64_t units, const int32_t *win,
                        const int32_t *slot_col, uint16_t *col16, hipStream_t st);

// SpMV of one right-hand side over the compact form (P.compact):
// P.n_wave_items wavefronts of `rows` groups each, four to a workgroup.
// width: the widest group (patterns).  segs: of the patterns, when every
// workgroup's rows are consecutive; null otherwise.
hipError_t launch_spmv_compact(const SpmvParams &P, int vdt, int vec_f64, int32_t rows, int32_t width,
                               const PatSegs *segs, hipStream_t st);

}  // namespace rg
