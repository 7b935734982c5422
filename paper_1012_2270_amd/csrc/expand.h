// Two-step SpMV of matrices with long rows and columns all over x.  Internal.
//
// Such a matrix gathers x at random: one request and one cache line per
// nonzero, whatever the format, and the requests bound the SpMV (6.5M nonzeros
// over 10^6 columns, FP32: 51 us for 64 MB, 43 us with the longest rows in
// column tiles).  The two steps move the gathers into LDS instead (31 to 35 us,
// 13.5 + 19.2, for about 135 MB of which half is x on its way):
//   expand   each workgroup holds a tile of x in LDS and writes x at the
//            columns of the entries of that tile, in runs of 16 entries: 2
//            bytes read and one vector element written per entry;
//   multiply each workgroup reads the x entries of one unit (some rows, about
//            4,096 entries) from the runs, puts each at its place in
//            LDS, and multiplies the layout's values against them.
// The entries of a (tile, unit) pair are contiguous in both orders, padded to
// whole runs.  Only the pattern is stored a second time: values are the
// layout's, so a value update has nothing to follow.  The runs of x entries are
// one buffer of the handle, which every product writes, as the tiles' partial
// sums are: products of one handle have to be ordered with each other.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <vector>

#include "internal.h"
#include "kernels.h"

namespace rg {

constexpr int kRunLen = 16;              // entries of a run: 64 bytes of FP32
constexpr int kExpandBytes = 64 << 10;   // a tile of x in LDS
constexpr int kExpandThreads = 1024;     // expand workgroup
constexpr int kExpandMaxTiles = 1024;    // tiles per matrix (counters of a unit, in LDS)
constexpr int kExpandUnit = 4096;        // entries of a unit (more only where one row group is wider)
constexpr int kExpandUnitBytes = 60 << 10;  // LDS of a unit (a launch may take 64 KB)
constexpr int kExpandMinRun = 12;        // mean entries of a (tile, unit) pair; below it the padding to
                                         // whole runs costs as much as the entries (FP64, 6.5M nonzeros
                                         // at 22 a pair: 60.1 against 64.2 us with column tiles)
// FP64 storage: fewer nonzeros stay with the column tiles, whose x a handle
// multiplied again and again finds in the L2 (Zipf rows, two steps against tiles,
// one handle repeated and three in turn: 1.35M nonzeros 20.3 and 18.1 against 16.2
// and 18.9 us, 2.0M 23.5 and 20.6 against 20.2 and 22.3, 2.3M 24.3 and 21.9
// against 24.4 and 26.0).
constexpr int64_t kExpandMinNnz64 = 2200000;
constexpr int expand_cols(int f64) { return kExpandBytes / (f64 ? 8 : 4); }

// Unit of the multiply step: slots [begin, begin + n) of the grouped part (row
// groups [g0, g1)) or of the long-row segment.  A block item of up to
// kBlockChunk entries is several units, run one after the other by its
// workgroup.
struct ExpandUnit {
    int64_t begin;
    int32_t n, is_long, g0, g1;
};

// Workgroups of the multiply step, in this order: block items, wavefront
// items of long rows (four each), runs of row groups (four wavefronts each).
// Unit w is the first of workgroup w; the further units of block items follow
// behind all of those.
struct HostExpand {
    std::vector<ExpandUnit> units;
    std::vector<int32_t> more;   // [2 * n_block] further units of each block item: first, count
    std::vector<int32_t> runs;   // runs of row groups, one per wavefront: first group << 2 | log2 of the count
    int32_t n_block = 0, n_long = 0, n_short = 0;  // workgroups of each kind
    int32_t max_n = 0;           // widest unit
    int64_t n_tiles = 0;
};

// What a workgroup needs before its first load, in one scalar load each (a
// chain of dependent ones costs a microsecond a link): expand workgroup
// (entries [e0, e0 + n) of tile t; t < 0: none) ...
struct ExpandPart {
    int64_t e0;
    int32_t n, t;
};
// ... unit of the multiply step (n entries at `begin` of the layout, n_pad
// entries with padding at e0 of the runs; block items: `count` further units
// from `next`) ...
struct ExpandRec {
    int64_t begin, e0;
    int32_t n, n_pad, next, count;
};
// ... wavefront item of long rows (n entries at `off` of the unit; rows
// row .. row + rows - 1 of the long list, lanes per row).
struct ExpandWave {
    int32_t off, n, row;
    int16_t rows, lanes;
};

// Everything the two kernels read.  Device pointers.
struct ExpandParams {
    SpmvParams P;             // layout, x (unit stride), y (any)
    const ExpandPart *parts;  // [n_parts]
    const uint16_t *lcol;     // [entries] column within the tile, tile order
    const int32_t *dst;       // [runs] the run's place in unit order
    const uint16_t *pos;      // [entries] place in the unit's LDS buffer, unit order (n of the unit: padding)
    const ExpandRec *recs;    // [units]
    const ExpandWave *waves;  // [n_waves]
    const int32_t *runs;      // [n_runs]
    void *xg;                 // [entries] x entries in unit order
    int32_t n_parts, n_waves, n_runs;
    int32_t n_block, n_long, n_short, max_n;
    int32_t x_aligned;
};
hipError_t launch_expand(const ExpandParams &E, int vdt, hipStream_t st);
hipError_t launch_expand_spmv(const ExpandParams &E, int vdt, hipStream_t st);

// Builds the runs of a layout that is on the device.  Counts first (cnt:
// [units * n_tiles] runs of each pair, unit-major), then the arrays from the
// exclusive scans of the counts in unit order (by_unit) and in tile order
// (by_tile, tile-major).
hipError_t launch_expand_count(const SpmvParams &P, const ExpandUnit *units, int32_t n_units, int f64, int32_t n_tiles,
                               int32_t *cnt, int32_t *cnt_tile, hipStream_t st);
hipError_t launch_expand_fill(const SpmvParams &P, const ExpandUnit *units, int32_t n_units, int f64, int32_t n_tiles,
                              const int32_t *by_unit, const int32_t *by_tile, uint16_t *lcol, int32_t *dst,
                              uint16_t *pos, hipStream_t st);
// Exclusive scans of both counts (scratch from the caller's DevScratch-like
// allocator), the run totals of the units and tiles, and the run count.
hipError_t expand_scan_bytes(int64_t n, size_t *bytes);
hipError_t launch_expand_scan(const int32_t *cnt, int32_t *out, int64_t n, void *temp, size_t bytes, hipStream_t st);
hipError_t launch_expand_ptrs(const int32_t *scan, int64_t stride, int32_t n, const int32_t *last_scan,
                              const int32_t *last_cnt, int32_t *ptr, hipStream_t st);

}  // namespace rg
