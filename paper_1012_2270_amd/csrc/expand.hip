// Two-step SpMV (expand.h): the expand and multiply kernels, and the device
// build of the runs.
#include <hip/hip_runtime.h>

#include <rocprim/device/device_scan.hpp>

#include "device.h"
#include "expand.h"

namespace rg {

// ---------------------------------------------------------------------------
// Expand: xg[place of entry] = x[column of entry], tile by tile
//
// Streams 2.25 bytes per entry and writes one element, four entries per
// thread and pass; kExpandAhead passes are loaded with the tile, before
// anything waits.  A tile is dealt to the workgroups b with b % 8 equal, one
// XCD's, so each L2 reads its own tiles of x.  The loads are cached: a matrix
// multiplied again finds them in the Infinity Cache (10.9 us; nontemporal
// 16.2; several matrices in turn 14.5 and 15.5).
// ---------------------------------------------------------------------------
constexpr int kExpandAhead = 4;

template <class A>
__global__ __launch_bounds__(kExpandThreads) void expand_k(const ExpandPart *parts, const uint16_t *lcols,
                                                           const int32_t *dsts, const A *X, A *out, int64_t n_cols,
                                                           int32_t x_aligned) {
    constexpr int C = kExpandBytes / (int)sizeof(A);
    constexpr int X4 = kExpandBytes / 16 / kExpandThreads;
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    __shared__ __align__(16) A xs[C];
    const ExpandPart part = ldc(parts, blockIdx.x);
    if (part.t < 0) return;
    const int64_t c0 = (int64_t)part.t * C;
    const int nc = (int)min((int64_t)C, n_cols - c0);
    const A *x = X + c0;
    const int32_t n = part.n;
    const uint16_t *lcol = lcols + part.e0;
    const int32_t *dst = dsts + part.e0 / kRunLen;
    const bool vec = x_aligned && nc == C;
    // assigned on every path, so the array stays in registers
    float4 xr[X4];
#pragma unroll
    for (int i = 0; i < X4; i++)
        xr[i] = vec ? reinterpret_cast<const float4 *>(x)[threadIdx.x + i * kExpandThreads]
                    : make_float4(0.f, 0.f, 0.f, 0.f);
    u32x2 lc[kExpandAhead];
    int32_t d[kExpandAhead];
    // (passes past the end re-read the first entries, which exist: every
    // array ends with a spare run)
    auto load = [&](int32_t first) {
#pragma unroll
        for (int i = 0; i < kExpandAhead; i++) {
            const int32_t q = first + ((int)threadIdx.x + i * kExpandThreads) * 4;
            const int32_t at = q < n ? q : 0;
            lc[i] = *reinterpret_cast<const u32x2 *>(lcol + at);
            d[i] = dst[at / kRunLen];
        }
    };
    load(0);
    if (vec) {
#pragma unroll
        for (int i = 0; i < X4; i++) reinterpret_cast<float4 *>(xs)[threadIdx.x + i * kExpandThreads] = xr[i];
    } else {
        for (int i = threadIdx.x; i < nc; i += kExpandThreads) xs[i] = x[i];
    }
    __syncthreads();
    for (int32_t first = 0; first < n; first += kExpandAhead * kExpandThreads * 4) {
        if (first) load(first);
#pragma unroll
        for (int i = 0; i < kExpandAhead; i++) {
            const int32_t q = first + ((int)threadIdx.x + i * kExpandThreads) * 4;
            const A v[4] = {xs[lc[i].x & 0xffff], xs[lc[i].x >> 16], xs[lc[i].y & 0xffff], xs[lc[i].y >> 16]};
            if (q < n) store_row<A, 4>(out + (int64_t)d[i] * kRunLen + (q & (kRunLen - 1)), v);
        }
    }
}

// ---------------------------------------------------------------------------
// Multiply
// ---------------------------------------------------------------------------
constexpr int kMulPer = 4096 / kBlockThreads;  // elements per thread of a unit of 4,096

// The unit's x entries into its LDS buffer, each at its place; padding goes
// to the slot behind the unit.  kFillRegs passes of four entries per thread
// are loaded before the caller's other loads are waited for.
constexpr int kFillRegs = 4;
template <class A> struct UnitFill {
    int64_t e0;
    int32_t n;
    A g[kFillRegs][4];
    uint2 p[kFillRegs];

    __device__ __forceinline__ void put(A *xs, const A (&v)[4], uint2 q) const {
        xs[q.x & 0xffff] = v[0];
        xs[q.x >> 16] = v[1];
        xs[q.y & 0xffff] = v[2];
        xs[q.y >> 16] = v[3];
    }
    __device__ __forceinline__ void load(const ExpandParams &E, const ExpandRec &rec) {
        e0 = rec.e0;
        n = rec.n_pad;
#pragma unroll
        for (int i = 0; i < kFillRegs; i++) {
            // passes past the end re-read the unit's first entries (every
            // array ends with a spare run)
            const int32_t q = ((int)threadIdx.x + i * kBlockThreads) * 4;
            const int64_t at = e0 + (q < n ? q : 0);
            load_row<A, 4>((const A *)E.xg + at, g[i]);
            p[i] = *reinterpret_cast<const uint2 *>(E.pos + at);
        }
    }
    __device__ __forceinline__ void store(const ExpandParams &E, A *xs) {
#pragma unroll
        for (int i = 0; i < kFillRegs; i++)
            if (((int)threadIdx.x + i * kBlockThreads) * 4 < n) put(xs, g[i], p[i]);
        for (int32_t q = ((int)threadIdx.x + kFillRegs * kBlockThreads) * 4; q < n; q += kBlockThreads * 4) {
            A v[4];
            load_row<A, 4>((const A *)E.xg + e0 + q, v);
            put(xs, v, *reinterpret_cast<const uint2 *>(E.pos + e0 + q));
        }
    }
};

// A run of R row groups of one wavefront: its values (16 steps over R rows
// per lane), lengths and output rows.
struct ShortRun {
    int32_t len[8], row[8];
};
template <int VD, int R>
__device__ __forceinline__ void run_load(const SpmvParams &P, int32_t first, int lane,
                                         typename Val<VD>::S (&v)[kLaneSteps], ShortRun &h) {
    using S = typename Val<VD>::S;
    constexpr int U = kLaneSteps / R;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const GroupMeta m = group_meta_uniform(P, first + r);
        const bool ok = lane < m.sg;
        const int32_t i = ok ? (int32_t)m.row0 + lane : 0;
        h.len[r] = ok ? P.short_len[i] : -1;
        h.row[r] = P.perm ? P.short_row[i] : i;
        const int32_t wc = m.g1 > m.g0 ? (int32_t)((uint32_t)(m.g1 - m.g0) / (uint32_t)m.sg) : 0;
        const S *vb = (const S *)P.slot_val + (wc ? m.g0 : 0);
#pragma unroll
        for (int u = 0; u < U; u++) v[r * U + u] = ldnt(vb + (ok && u < wc ? lane + u * m.sg : 0));
    }
}
template <int VD, class A, int R>
__device__ __forceinline__ void run_multiply(const SpmvParams &P, int32_t first, int lane, int64_t begin,
                                             typename Val<VD>::S (&v)[kLaneSteps], const ShortRun &h, const A *xs) {
    using V = Val<VD>;
    using S = typename V::S;
    constexpr int U = kLaneSteps / R;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const GroupMeta m = group_meta_uniform(P, first + r);
        const int32_t wc = m.g1 > m.g0 ? (int32_t)((uint32_t)(m.g1 - m.g0) / (uint32_t)m.sg) : 0;
        const A *xb = xs + (wc && h.len[r] >= 0 ? (int32_t)(m.g0 - begin) + lane : 0);
        A acc = A(0);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const A f = fmaA(V::template cvt<A>(v[r * U + u]), xb[u < h.len[r] ? u * m.sg : 0], acc);
            acc = u < h.len[r] ? f : acc;
        }
        // groups wider than the run's steps
        const S *vb = (const S *)P.slot_val + m.g0 + lane;
        for (int c0 = U; c0 < wc; c0 += 8) {
            S w[8];
#pragma unroll
            for (int u = 0; u < 8; u++) w[u] = ldnt(c0 + u < h.len[r] ? vb + (c0 + u) * m.sg : (const S *)P.slot_val);
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const A f = fmaA(V::template cvt<A>(w[u]), xb[c0 + u < h.len[r] ? (c0 + u) * m.sg : 0], acc);
                acc = c0 + u < h.len[r] ? f : acc;
            }
        }
        if (h.len[r] >= 0) ((A *)P.y)[(int64_t)h.row[r] * P.ldy] = acc;
    }
}

__device__ __forceinline__ ExpandRec rec_at(const ExpandRec *recs, int64_t i) {
    // two 16-byte scalar loads
    ExpandRec r;
    const i32x4 lo = ldc((const i32x4 *)(recs + i), 0), hi = ldc((const i32x4 *)(recs + i), 1);
    __builtin_memcpy(&r, &lo, 16);
    __builtin_memcpy((char *)&r + 16, &hi, 16);
    return r;
}

// One workgroup per block item, four wavefront items of long rows, or four
// runs of row groups.  The unit's x entries go to LDS before the values are
// loaded: their registers are then free (94 instead of 106; 19.9 against
// 21.0 us).  Element-parallel products of the row groups, summed from LDS in
// units of up to 4,096 slots, were no faster, and fewer registers by force
// spilled.
template <int VD, class A>
__global__ __launch_bounds__(kBlockThreads) void expand_spmv_k(ExpandParams E) {
    using V = Val<VD>;
    using S = typename V::S;
    extern __shared__ __align__(16) unsigned char dyn[];
    A *xs = (A *)dyn;  // max_n + 1 entries
    __shared__ A red[kBlockWaves];
    const SpmvParams &P = E.P;
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int32_t n_wg = E.n_block + E.n_long + E.n_short;
    const int32_t nl = E.n_block + E.n_long;
    // long-row work keeps the dispatch order (heaviest first, dealt over the
    // XCDs), row groups go in contiguous ranges to each XCD
    const int32_t h = min((nl + 7) & ~7, n_wg);
    const int32_t wg = (int32_t)blockIdx.x < h ? (int32_t)blockIdx.x : h + xcd_remap(blockIdx.x - h, n_wg - h);
    const ExpandRec rec = rec_at(E.recs, wg);
    UnitFill<A> F;
    F.load(E, rec);
    if (wg >= nl) {
        const int32_t w = __builtin_amdgcn_readfirstlane((wg - nl) * kBlockWaves + wv);
        const int64_t begin = rec.begin;
        const int32_t it = w < E.n_runs ? ldc(E.runs, w) : 0;
        const int32_t first = w < E.n_runs ? it >> 2 : (int32_t)P.ng;
        S v[kLaneSteps];
        ShortRun sr;
        F.store(E, xs);
        switch (it & 3) {
            case 0: run_load<VD, 1>(P, first, lane, v, sr); break;
            case 1: run_load<VD, 2>(P, first, lane, v, sr); break;
            case 2: run_load<VD, 4>(P, first, lane, v, sr); break;
            default: run_load<VD, 8>(P, first, lane, v, sr); break;
        }
        __syncthreads();
        switch (it & 3) {
            case 0: run_multiply<VD, A, 1>(P, first, lane, begin, v, sr, xs); break;
            case 1: run_multiply<VD, A, 2>(P, first, lane, begin, v, sr, xs); break;
            case 2: run_multiply<VD, A, 4>(P, first, lane, begin, v, sr, xs); break;
            default: run_multiply<VD, A, 8>(P, first, lane, begin, v, sr, xs); break;
        }
        return;
    }
    if (wg >= E.n_block) {
        // wavefront items of long rows: products element-parallel in place,
        // then the item's lanes per row add them (the order of
        // spmv_wave_long_lds)
        const int32_t w = __builtin_amdgcn_readfirstlane((wg - E.n_block) * kBlockWaves + wv);
        const ExpandWave it = ldc(E.waves, w < E.n_waves ? w : 0);
        const int32_t n = w < E.n_waves ? it.n : 0;
        const int64_t item0 = rec.begin + it.off;
        constexpr int U = kWaveRowMax / 64;
        const S *vb = (const S *)P.long_val + (n > 0 ? item0 : 0);
        S v[U];
        F.store(E, xs);
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = ldnt(vb + (lane + 64 * u < n ? lane + 64 * u : 0));
        const int TL = it.lanes;
        const int sh = 31 - __builtin_clz(TL);
        const int r = lane >> sh, q = lane & (TL - 1);
        const bool ok = n > 0 && r < it.rows;
        const int64_t li = (int64_t)it.row + (ok ? r : 0);
        const int32_t b = (int32_t)(P.long_ptr[li] - item0), e = (int32_t)(P.long_ptr[li + 1] - item0);
        const int32_t orow = P.long_row[li];
        __syncthreads();
        A *buf = xs + (n > 0 ? it.off : 0);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int32_t k = lane + 64 * u;
            if (k < n) buf[k] *= V::template cvt<A>(v[u]);
        }
        // the item's part of the buffer is this wavefront's own
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int32_t nj = ok && e - b > q ? (e - b - q + TL - 1) >> sh : 0;
        A acc = A(0);
#pragma nounroll
        for (int j0 = 0; j0 < kWaveUnroll; j0 += 4)
#pragma unroll
            for (int j = j0; j < j0 + 4; j++) {
                const A t = buf[j < nj ? b + q + j * TL : 0];
                acc = j < nj ? acc + t : acc;
            }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
            if (off < TL) acc += __shfl_xor(acc, off);
        if (ok && q == 0) ((A *)P.y)[(int64_t)orow * P.ldy] = acc;
        return;
    }
    // block item: a chunk of one row, unit after unit; sums of one unit, then
    // of the units (short chains)
    const LongItem it = ldc(P.block_work, wg);
    A tot = A(0);
    for (int32_t u = 0; u <= rec.count; u++) {
        const ExpandRec cur = u ? rec_at(E.recs, rec.next + u - 1) : rec;
        if (u) F.load(E, cur);
        const int32_t n = cur.n;
        const S *vb = (const S *)P.long_val + cur.begin;
        S v[kMulPer];
        F.store(E, xs);
#pragma unroll
        for (int k = 0; k < kMulPer; k++) {
            const int32_t q = (int)threadIdx.x + k * kBlockThreads;
            v[k] = ldnt(vb + (q < n ? q : 0));
        }
        __syncthreads();
        A acc = A(0);
#pragma unroll
        for (int k = 0; k < kMulPer; k++) {
            const int32_t q = (int)threadIdx.x + k * kBlockThreads;
            const A f = fmaA(V::template cvt<A>(v[k]), xs[q < n ? q : 0], acc);
            acc = q < n ? f : acc;
        }
        tot += acc;
        __syncthreads();
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off);
    if (lane == 0) red[wv] = tot;
    __syncthreads();
    if (threadIdx.x == 0) {
        tot = A(0);
        for (int i = 0; i < kBlockWaves; i++) tot += red[i];
        if (it.c == 1) ((A *)P.y)[(int64_t)ldc(P.long_row, (int64_t)it.a) * P.ldy] = tot;
        else ((A *)P.partial)[(int64_t)it.d + it.b] = tot;
    }
}

template <class A> static hipError_t launch_expand_a(const ExpandParams &E, hipStream_t st) {
    hipLaunchKernelGGL(expand_k<A>, dim3(E.n_parts), dim3(kExpandThreads), 0, st, E.parts, E.lcol, E.dst,
                       (const A *)E.P.x, (A *)E.xg, (int64_t)E.P.last_col + 1, E.x_aligned);
    return hipGetLastError();
}

hipError_t launch_expand(const ExpandParams &E, int vdt, hipStream_t st) {
    return vdt == RGCSR_F64 ? launch_expand_a<double>(E, st) : launch_expand_a<float>(E, st);
}

template <int VD, class A> static hipError_t launch_expand_spmv_v(const ExpandParams &E, hipStream_t st) {
    const size_t lds = ((size_t)E.max_n + 4) * sizeof(A);
    hipLaunchKernelGGL((expand_spmv_k<VD, A>), dim3(E.n_block + E.n_long + E.n_short), dim3(kBlockThreads), lds, st, E);
    return hipGetLastError();
}

hipError_t launch_expand_spmv(const ExpandParams &E, int vdt, hipStream_t st) {
    switch (vdt) {
    case RGCSR_F64: return launch_expand_spmv_v<RGCSR_F64, double>(E, st);
    case RGCSR_F32: return launch_expand_spmv_v<RGCSR_F32, float>(E, st);
    case RGCSR_F16: return launch_expand_spmv_v<RGCSR_F16, float>(E, st);
    case RGCSR_BF16: return launch_expand_spmv_v<RGCSR_BF16, float>(E, st);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Build
// ---------------------------------------------------------------------------

// f(column, place in the unit) for every entry of the unit (padding skipped).
template <class F> __device__ __forceinline__ void unit_entries(const SpmvParams &P, const ExpandUnit &u, F f) {
    if (u.is_long) {
        for (int32_t i = threadIdx.x; i < u.n; i += 256) f(P.long_col[u.begin + i], i);
        return;
    }
    const int lane = threadIdx.x & 63;
    for (int32_t g = u.g0 + (int)(threadIdx.x >> 6); g < u.g1; g += 4) {
        const GroupMeta m = group_meta_uniform(P, __builtin_amdgcn_readfirstlane(g));
        const int32_t len = lane < m.sg ? P.short_len[m.row0 + lane] : 0;
        for (int32_t j = 0; j < len; j++) {
            const int64_t s = m.g0 + (int64_t)j * m.sg + lane;
            f(P.slot_col[s], (int32_t)(s - u.begin));
        }
    }
}

__global__ __launch_bounds__(256) void expand_count_k(SpmvParams P, const ExpandUnit *units, int32_t n_units,
                                                      int32_t cols, int32_t n_tiles, int32_t *cnt, int32_t *cnt_tile) {
    __shared__ int32_t c[kExpandMaxTiles];
    const ExpandUnit u = units[blockIdx.x];
    for (int t = threadIdx.x; t < n_tiles; t += 256) c[t] = 0;
    __syncthreads();
    unit_entries(P, u, [&](int32_t col, int32_t) { atomicAdd(&c[col / cols], 1); });
    __syncthreads();
    for (int t = threadIdx.x; t < n_tiles; t += 256) {
        const int32_t runs = (c[t] + kRunLen - 1) / kRunLen;
        cnt[(int64_t)blockIdx.x * n_tiles + t] = runs;
        cnt_tile[(int64_t)t * n_units + blockIdx.x] = runs;
    }
}

__global__ __launch_bounds__(256) void expand_fill_k(SpmvParams P, const ExpandUnit *units, int32_t n_units,
                                                     int32_t cols, int32_t n_tiles, const int32_t *by_unit,
                                                     const int32_t *by_tile, uint16_t *lcol, int32_t *dst,
                                                     uint16_t *pos) {
    __shared__ int32_t c[kExpandMaxTiles], du[kExpandMaxTiles], su[kExpandMaxTiles];
    const ExpandUnit u = units[blockIdx.x];
    for (int t = threadIdx.x; t < n_tiles; t += 256) {
        c[t] = 0;
        du[t] = by_unit[(int64_t)blockIdx.x * n_tiles + t];
        su[t] = by_tile[(int64_t)t * n_units + blockIdx.x];
    }
    __syncthreads();
    unit_entries(P, u, [&](int32_t col, int32_t place) {
        const int32_t t = col / cols;
        const int32_t i = atomicAdd(&c[t], 1);
        lcol[(int64_t)su[t] * kRunLen + i] = (uint16_t)(col - t * cols);
        pos[(int64_t)du[t] * kRunLen + i] = (uint16_t)place;
    });
    __syncthreads();
    for (int t = threadIdx.x; t < n_tiles; t += 256) {
        const int32_t n = c[t], runs = (n + kRunLen - 1) / kRunLen;
        for (int32_t k = 0; k < runs; k++) dst[su[t] + k] = du[t] + k;
        // padding: the tile's first column, put behind the unit
        for (int32_t i = n; i < runs * kRunLen; i++) {
            lcol[(int64_t)su[t] * kRunLen + i] = 0;
            pos[(int64_t)du[t] * kRunLen + i] = (uint16_t)u.n;
        }
    }
}

hipError_t launch_expand_count(const SpmvParams &P, const ExpandUnit *units, int32_t n_units, int f64, int32_t n_tiles,
                               int32_t *cnt, int32_t *cnt_tile, hipStream_t st) {
    hipLaunchKernelGGL(expand_count_k, dim3(n_units), dim3(256), 0, st, P, units, n_units, expand_cols(f64), n_tiles,
                       cnt, cnt_tile);
    return hipGetLastError();
}

hipError_t launch_expand_fill(const SpmvParams &P, const ExpandUnit *units, int32_t n_units, int f64, int32_t n_tiles,
                              const int32_t *by_unit, const int32_t *by_tile, uint16_t *lcol, int32_t *dst,
                              uint16_t *pos, hipStream_t st) {
    hipLaunchKernelGGL(expand_fill_k, dim3(n_units), dim3(256), 0, st, P, units, n_units, expand_cols(f64), n_tiles,
                       by_unit, by_tile, lcol, dst, pos);
    return hipGetLastError();
}

hipError_t expand_scan_bytes(int64_t n, size_t *bytes) {
    *bytes = 0;
    return rocprim::exclusive_scan(nullptr, *bytes, (const int32_t *)nullptr, (int32_t *)nullptr, 0, (size_t)n,
                                   rocprim::plus<int32_t>(), (hipStream_t) nullptr);
}

hipError_t launch_expand_scan(const int32_t *cnt, int32_t *out, int64_t n, void *temp, size_t bytes, hipStream_t st) {
    return rocprim::exclusive_scan(temp, bytes, cnt, out, 0, (size_t)n, rocprim::plus<int32_t>(), st);
}

// ptr[i] = scan[i * stride] for i < n, ptr[n] = the total
__global__ __launch_bounds__(256) void expand_ptrs_k(const int32_t *scan, int64_t stride, int32_t n,
                                                     const int32_t *last_scan, const int32_t *last_cnt, int32_t *ptr) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) ptr[i] = scan[(int64_t)i * stride];
    else if (i == n) ptr[n] = *last_scan + *last_cnt;
}

hipError_t launch_expand_ptrs(const int32_t *scan, int64_t stride, int32_t n, const int32_t *last_scan,
                              const int32_t *last_cnt, int32_t *ptr, hipStream_t st) {
    hipLaunchKernelGGL(expand_ptrs_k, dim3(n / 256 + 1), dim3(256), 0, st, scan, stride, n, last_scan, last_cnt, ptr);
    return hipGetLastError();
}

}  // namespace rg
