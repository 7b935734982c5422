// SpMV over the compact column storage (compact.h) and the search for it on
// device CSR arrays.
#include <hip/hip_runtime.h>

#include <initializer_list>

#include "compact.h"
#include "device.h"

namespace rg {

// ---------------------------------------------------------------------------
// SpMV of the row groups (one lane per row, G a multiple of 64)
//
// As spmv_groups_uniform (kernels.hip): value loads, x gathers and
// multiply-adds in branch-free phases, each lane in its row's serial order,
// so the results are the same bits.  What a workgroup needs first -- the table
// or the x window, its rows' metadata, the values (and 16-bit columns) of the
// first pass -- is loaded before anything waits: one memory latency, then one
// for the gathers of a pattern (an x window has none, it gathers from LDS).
//
// Bound by the value stream (patterns: 7-point 128^3 FP32 77 MB instead of
// 134, 23.5 -> 14.4 us, 5.4 TB/s; 27-point 101^3 FP64 238 MB instead of 344,
// 64.5 -> 40.7 us) and, where the columns are random in a band, by the x
// gathers: one touches about 28 cache lines, so gathering from LDS counts for
// more than the two bytes saved (400,009 rows of 24 nonzeros, half band 500,
// BF16: 20.0 -> 11.4 us; with the 16-bit columns alone 18.9).
// Tried and slower: a resident grid that walks the units and prefetches the
// next pass's values (7-point 16.6-23 us, 27-point FP64 53-60), prefetching
// the next pass within a unit (windows 13.6 us), the table behind a barrier
// before the first loads (7-point 15.6 us).
// ---------------------------------------------------------------------------

// The R groups of one wavefront: metadata of each lane's rows, and the first
// U steps of their values (and columns).
template <int VD, int R, int U, bool WIN, bool LEN> struct CompactRows {
    using S = typename Val<VD>::S;
    const S *vb[R];
    const uint16_t *cb[R];
    int32_t t[R], stride[R], nl[R], rowi[R], orow[R], len[R];
    bool ok[R];
    int cmax;  // widest of the groups (uniform)
    S v[R][U];
    int32_t c[R][U];

    __device__ __forceinline__ void meta(const SpmvParams &P, int32_t first, int lane) {
        cmax = 0;
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int32_t wr = first + r;
            const int32_t g = WIN ? wr : __builtin_amdgcn_readfirstlane(wr / P.wpg);
            t[r] = WIN ? lane : (wr - g * P.wpg) * 64 + lane;
            // loads at a clamped group, no branch around them: a count of
            // outstanding loads that differs by path would make the first
            // wait wait for all of them
            const int64_t gc = min((int64_t)g, P.ng - 1);
            const int64_t g0 = ldc(P.gp, gc), g1 = ldc(P.gend ? P.gend : P.gp + 1, gc);
            int64_t row0 = gc * P.G;
            int32_t sg = (int32_t)min((int64_t)P.G, P.ns - row0);
            if (P.ragged) {
                row0 = ldc(P.grp_row0, gc);
                sg = ldc(P.grp_row0, gc + 1) - (int32_t)row0;
            }
            ok[r] = t[r] < sg && g < P.ng;
            rowi[r] = ok[r] ? (int32_t)row0 + t[r] : 0;
            orow[r] = P.perm ? P.short_row[rowi[r]] : rowi[r];
            if constexpr (WIN && LEN) len[r] = P.short_len[rowi[r]];
            stride[r] = sg;
            const bool has = g1 > g0;
            const int64_t gb = has ? g0 : 0;
            vb[r] = (const S *)P.slot_val + gb;
            if constexpr (WIN) cb[r] = P.col16 + gb;
            const int32_t wc = has ? (int32_t)((uint32_t)(g1 - g0) / (uint32_t)sg) : 0;
            nl[r] = ok[r] ? wc : 0;
            cmax = max(cmax, g < P.ng ? wc : 0);
        }
    }
    // steps past a row's slots re-read the group's first slot
    __device__ __forceinline__ void load(int c0) {
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint32_t o = c0 + u < nl[r] ? (uint32_t)(t[r] + (c0 + u) * stride[r]) : 0u;
                v[r][u] = ldnt((const S *)((const char *)vb[r] + o * (uint32_t)sizeof(S)));
                if constexpr (WIN) c[r][u] = ldnt((const uint16_t *)((const char *)cb[r] + o * 2u));
            }
    }
};

// The workgroup's part of x.y
__device__ __forceinline__ void put_dot(const SpmvParams &P, double d) {
    __shared__ double part[kBlockWaves];
    for (int off = 32; off > 0; off >>= 1) d += __shfl_xor(d, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = part[0];
        for (int i = 1; i < kBlockWaves; i++) t += part[i];
        P.dot_part[blockIdx.x] = t;
    }
}

// Row patterns.  Steps past a row's length read on in the table (the entries
// behind it are another row's, or none) and gather at the clamped column they
// give; the multiply masks them.  Nothing is read under a condition: the
// compiler would wait for each LDS read inside its branch.
//
// DOT: the workgroup's part of x.y as well, which a conjugate-gradient
// iteration asks for (27-point 96^3, BF16: 0.9 us more here than without and 1.1
// more to add 3,456 parts in the next kernel, for a launch of 4.1 and the gap
// before it; the solve 4.88 -> 4.64 ms).
template <int VD, class A, int R, int U, bool DOT>
__global__ __launch_bounds__(kBlockThreads) void spmv_pattern_k(SpmvParams P) {
    using V = Val<VD>;
    __shared__ int32_t tab[kPatTab + 32];
    const int lane = threadIdx.x & 63;
    int32_t tv[kPatTab / kBlockThreads];
#pragma unroll
    for (int i = 0; i < kPatTab / kBlockThreads; i++) {
        const int32_t e = (int)threadIdx.x + i * kBlockThreads;
        if (i * kBlockThreads < P.pat_ints) tv[i] = P.pat_tab[e < P.pat_ints ? e : 0];
    }
    const int32_t unit = xcd_remap(blockIdx.x, gridDim.x);
    const int32_t w = __builtin_amdgcn_readfirstlane(unit * kBlockWaves + (int)(threadIdx.x >> 6));
    CompactRows<VD, R, U, false, false> G;
    G.meta(P, w * R, lane);
    int32_t pt[R];
#pragma unroll
    for (int r = 0; r < R; r++) pt[r] = P.pat_id[G.rowi[r]];
    A xd[R];
    if constexpr (DOT) {
#pragma unroll
        for (int r = 0; r < R; r++) xd[r] = ((const A *)P.x)[(int64_t)G.orow[r] * P.ldx];
    }
    G.load(0);
#pragma unroll
    for (int i = 0; i < kPatTab / kBlockThreads; i++) {
        const int32_t e = (int)threadIdx.x + i * kBlockThreads;
        if (e < P.pat_ints) tab[e] = tv[i];
    }
    __syncthreads();
    const A *X = (const A *)P.x;
    const uint32_t xrow = (uint32_t)(P.ldx * (int64_t)sizeof(A));
    int32_t len[R];
    A acc[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        pt[r] *= P.pat_stride;
        len[r] = G.ok[r] ? tab[pt[r]] : 0;
        acc[r] = A(0);
    }
    for (int c0 = 0; c0 < G.cmax; c0 += U) {
        if (c0) G.load(c0);
        A xv[R][U];
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int32_t c = (int32_t)min((uint32_t)(G.orow[r] + tab[pt[r] + 1 + c0 + u]), (uint32_t)P.last_col);
                xv[r][u] = ldx32<0>(X, c, xrow);
            }
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const A f = fmaA(V::template cvt<A>(G.v[r][u]), xv[r][u], acc[r]);
                acc[r] = c0 + u < len[r] ? f : acc[r];
            }
    }
#pragma unroll
    for (int r = 0; r < R; r++)
        if (G.ok[r]) ((A *)P.y)[(int64_t)G.orow[r] * P.ldy] = acc[r];
    if constexpr (DOT) {
        double d = 0.0;
#pragma unroll
        for (int r = 0; r < R; r++) d += G.ok[r] ? (double)xd[r] * (double)acc[r] : 0.0;
        put_dot(P, d);
    }
}

// Row patterns whose x comes from LDS (PatSegs): 27 steps issue 27 value loads
// and 10 of x instead of 27 gathers, all before anything waits (27-point 101^3,
// FP64: 48.0 -> 40.7 us, 5.8 TB/s).  Where they pay: runs_width below.  NS: the runs, a constant, as a count read from
// memory made each run's load wait for a scalar load of its own (FP32 96^3:
// 24.8 us); further ones repeat the last.
template <int VD, class A, int U, int NS, bool DOT>
__global__ __launch_bounds__(kBlockThreads) void spmv_segment_k(SpmvParams P, PatSegs Q) {
    using V = Val<VD>;
    __shared__ int32_t tab[kPatTab + 32];
    extern __shared__ __align__(16) char seg_lds[];
    A *xs = (A *)seg_lds;  // [Q.total]
    const int tid = threadIdx.x, lane = tid & 63;
    int32_t tv[kPatTab / kBlockThreads];
#pragma unroll
    for (int i = 0; i < kPatTab / kBlockThreads; i++) {
        const int32_t e = tid + i * kBlockThreads;
        if (i * kBlockThreads < P.pat_ints) tv[i] = P.pat_tab[e < P.pat_ints ? e : 0];
    }
    const int32_t unit = xcd_remap(blockIdx.x, gridDim.x);
    const int32_t row0 = unit * kBlockThreads;
    const A *X = (const A *)P.x;
    auto at = [&](int64_t c) { return X[min(max(c, (int64_t)0), (int64_t)P.last_col) * P.ldx]; };
    A xr[NS];
#pragma unroll
    for (int s = 0; s < NS; s++) xr[s] = at((int64_t)row0 + Q.lo[s] + tid);
    // the entries behind each run's first kBlockThreads, one lane each
    int32_t eo = 0, ed = 0;
    {
        int32_t before = 0;
#pragma unroll
        for (int s = 0; s < NS; s++) {
                if (tid >= before) {
                    eo = Q.lo[s] + kBlockThreads + tid - before;
                    ed = Q.base[s] + kBlockThreads + tid - before;
                }
                before += Q.span[s];
            }
    }
    const A xe = at((int64_t)row0 + eo);
    const int32_t w = __builtin_amdgcn_readfirstlane(unit * kBlockWaves + (tid >> 6));
    CompactRows<VD, 1, U, false, false> G;
    G.meta(P, w, lane);
    int32_t pt = P.pat_id[G.rowi[0]];
    A xd = A(0);
    if constexpr (DOT) xd = X[(int64_t)G.orow[0] * P.ldx];
    G.load(0);
#pragma unroll
    for (int s = 0; s < NS; s++) xs[Q.base[s] + tid] = xr[s];
    if (tid < Q.extra) xs[ed] = xe;
    // offsets become places in xs (of the workgroup's first row); the lengths
    // before each list stay
#pragma unroll
    for (int i = 0; i < kPatTab / kBlockThreads; i++) {
        const int32_t e = tid + i * kBlockThreads;
        if (i * kBlockThreads < P.pat_ints) {
            int32_t place = 0;
#pragma unroll
            for (int s = 0; s < NS; s++)
                if (tv[i] >= Q.lo[s]) place = tv[i] - Q.lo[s] + Q.base[s];
            if (e < P.pat_ints) tab[e] = e % P.pat_stride ? place : tv[i];
        }
    }
    __syncthreads();
    pt *= P.pat_stride;
    const int32_t len = G.ok[0] ? tab[pt] : 0;
    A acc = A(0);
    for (int c0 = 0; c0 < G.cmax; c0 += U) {
        if (c0) G.load(c0);
        A xv[U];
#pragma unroll
        for (int u = 0; u < U; u++)
            xv[u] = xs[min((uint32_t)(tid + tab[pt + 1 + c0 + u]), (uint32_t)(Q.total - 1))];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const A f = fmaA(V::template cvt<A>(G.v[0][u]), xv[u], acc);
            acc = c0 + u < len ? f : acc;
        }
    }
    if (G.ok[0]) ((A *)P.y)[(int64_t)G.orow[0] * P.ldy] = acc;
    if constexpr (DOT) put_dot(P, G.ok[0] ? (double)xd * (double)acc : 0.0);
}

// x windows, one right-hand side of unit stride or not.  LEN: row lengths are
// read; otherwise (no empty rows) a step is multiplied when its column
// exceeds the previous one, as pad_loads = 3 does.
template <int VD, class A, int R, int U, bool LEN>
__global__ __launch_bounds__(kBlockThreads) void spmv_window_k(SpmvParams P) {
    using V = Val<VD>;
    __shared__ A xs[kWinCols];
    const int lane = threadIdx.x & 63;
    const int32_t unit = xcd_remap(blockIdx.x, gridDim.x);
    const int32_t base = ldc(P.win, 2 * (int64_t)unit), n = ldc(P.win, 2 * (int64_t)unit + 1);
    const A *X = (const A *)P.x + (int64_t)base * P.ldx;
    A xr[kWinCols / kBlockThreads];
#pragma unroll
    for (int i = 0; i < kWinCols / kBlockThreads; i++)
        if (i * kBlockThreads < n) {
            const int32_t e = (int)threadIdx.x + i * kBlockThreads;
            xr[i] = X[(e < n ? e : 0) * P.ldx];
        }
    const int32_t w = __builtin_amdgcn_readfirstlane(unit * kBlockWaves + (int)(threadIdx.x >> 6));
    CompactRows<VD, R, U, true, LEN> G;
    G.meta(P, w * R, lane);
    G.load(0);
#pragma unroll
    for (int i = 0; i < kWinCols / kBlockThreads; i++)
        if (i * kBlockThreads < n) {
            const int32_t e = (int)threadIdx.x + i * kBlockThreads;
            if (e < n) xs[e] = xr[i];
        }
    __syncthreads();
    A acc[R];
    int32_t prevc[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        acc[r] = A(0);
        prevc[r] = -1;
    }
    for (int c0 = 0; c0 < G.cmax; c0 += U) {
        if (c0) G.load(c0);
        A xv[R][U];
        bool on[R][U];
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                if constexpr (LEN) {
                    on[r][u] = G.ok[r] && c0 + u < G.len[r];
                } else {
                    on[r][u] = c0 + u < G.nl[r] && G.c[r][u] > prevc[r];
                    prevc[r] = G.c[r][u];
                }
                xv[r][u] = xs[G.c[r][u]];  // every slot's offset lies in the window buffer
            }
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const A f = fmaA(V::template cvt<A>(G.v[r][u]), xv[r][u], acc[r]);
                acc[r] = on[r][u] ? f : acc[r];
            }
    }
#pragma unroll
    for (int r = 0; r < R; r++)
        if (G.ok[r]) ((A *)P.y)[(int64_t)G.orow[r] * P.ldy] = acc[r];
}

#define RG_GO(...)                                                                                          \
    do {                                                                                                    \
        hipLaunchKernelGGL((__VA_ARGS__), dim3(nwg), dim3(kBlockThreads), 0, st, P);                        \
        return hipGetLastError();                                                                           \
    } while (0)

// Steps per pass of one right-hand side: of the compiled counts the one that
// pads the width least, the larger of equals.
static int pattern_steps(int32_t width, std::initializer_list<int> counts) {
    int best = 0;
    int64_t cost = 0;
    for (int u : counts) {
        const int64_t c = (int64_t)(width + u - 1) / u * u;
        if (best == 0 || c <= cost) {
            best = u;
            cost = c;
        }
    }
    return best;
}

template <int VD, class A, int NS, bool DOT>
static hipError_t launch_segment_v(const SpmvParams &P, int32_t width, int nwg, const PatSegs &segs, hipStream_t st) {
    const dim3 g(nwg), b(kBlockThreads);
    const size_t lds = segs.total * sizeof(A);
    if (pattern_steps(width, {9, 27}) == 9)
        hipLaunchKernelGGL((spmv_segment_k<VD, A, 9, NS, DOT>), g, b, lds, st, P, segs);
    else
        hipLaunchKernelGGL((spmv_segment_k<VD, A, 27, NS, DOT>), g, b, lds, st, P, segs);
    return hipGetLastError();
}

// x from LDS runs pays for rows wide enough against the loads of the kernel
// that is compiled (3 or 9 runs, and their ends).  400,000 rows on diagonals in
// k runs of w, one handle repeated, gathered against runs, us.  FP64:
//   1 x 6   6.0, 6.6       3 x 3   7.4, 6.9     1 x 17  13.7, 11.2    3 x 9  19.9, 15.6
//   4 x 4  12.1, 12.8      5 x 3  12.2, 12.2    6 x 3   13.7, 13.1    9 x 3  20.1, 17.2
// FP32 values with FP64 vectors:
//   3 x 5   7.9, 8.5       1 x 17  9.3, 8.7     3 x 9   13.1, 10.6    9 x 3  13.1, 13.2
// FP32: 3 x 3 4.8, 5.8; 4 x 3 5.0, 9.1; 5 x 5 8.8, 11.2; 1 x 17 6.6, 7.7; but 27 points
// on a grid of 30 x 200 x 200 (3 runs) 28.4, 22.5, and of 160^3 (9 runs) 84.0, 83.3, with
// p.q 1.5% of a solve.  16-bit values gather: what the runs save on requests the
// longer way to the first step costs (27-point 96^3 in BF16 16.1, 18.6).
template <int VD, class A> constexpr int32_t runs_width(bool three) {
    if (VD == RGCSR_F64) return three ? 8 : 18;
    return three ? (sizeof(A) == 8 ? 16 : 18) : 27;
}

template <int VD, class A, bool DOT>
static hipError_t launch_pattern_v(const SpmvParams &P, int32_t rows, int32_t width, int nwg, const PatSegs *segs,
                                   hipStream_t st) {
    if constexpr (VD == RGCSR_F64 || VD == RGCSR_F32)
        if (segs && width >= runs_width<VD, A>(segs->n <= 3)) {
            if (segs->n <= 3) return launch_segment_v<VD, A, 3, DOT>(P, width, nwg, *segs, st);
            return launch_segment_v<VD, A, kPatSegs, DOT>(P, width, nwg, *segs, st);
        }
    if (rows == 2) {
        switch (pattern_steps(width, {4, 5, 7, 8})) {
        case 4: RG_GO(spmv_pattern_k<VD, A, 2, 4, DOT>);
        case 5: RG_GO(spmv_pattern_k<VD, A, 2, 5, DOT>);
        case 7: RG_GO(spmv_pattern_k<VD, A, 2, 7, DOT>);
        default: RG_GO(spmv_pattern_k<VD, A, 2, 8, DOT>);
        }
    }
    switch (pattern_steps(width, {5, 7, 9, 14, 16})) {
    case 5: RG_GO(spmv_pattern_k<VD, A, 1, 5, DOT>);
    case 7: RG_GO(spmv_pattern_k<VD, A, 1, 7, DOT>);
    case 9: RG_GO(spmv_pattern_k<VD, A, 1, 9, DOT>);
    case 14: RG_GO(spmv_pattern_k<VD, A, 1, 14, DOT>);
    default: RG_GO(spmv_pattern_k<VD, A, 1, 16, DOT>);
    }
}

template <int VD, class A>
static hipError_t launch_compact_v(const SpmvParams &P, int32_t rows, int32_t width, const PatSegs *segs,
                                   hipStream_t st) {
    const int nwg = (P.n_wave_items + kBlockWaves - 1) / kBlockWaves;
    if (P.compact == kCompactWindow) {
        // 8-byte values: half the steps (22.1 against 23.0 us on 9.6M nonzeros)
        constexpr int U = VD == RGCSR_F64 ? 8 : kLaneSteps;
        const bool len = P.pad != 3;
        if (rows == 2) {
            if (len) RG_GO(spmv_window_k<VD, A, 2, U / 2, true>);
            RG_GO(spmv_window_k<VD, A, 2, U / 2, false>);
        }
        if (len) RG_GO(spmv_window_k<VD, A, 1, U, true>);
        RG_GO(spmv_window_k<VD, A, 1, U, false>);
    }
    if (P.dot_part) return launch_pattern_v<VD, A, true>(P, rows, width, nwg, segs, st);
    return launch_pattern_v<VD, A, false>(P, rows, width, nwg, segs, st);
}

hipError_t launch_spmv_compact(const SpmvParams &P, int vdt, int vec_f64, int32_t rows, int32_t width,
                               const PatSegs *segs, hipStream_t st) {
    if (vec_f64) {
        if (vdt == RGCSR_F64) return launch_compact_v<RGCSR_F64, double>(P, rows, width, segs, st);
        if (vdt == RGCSR_F32) return launch_compact_v<RGCSR_F32, double>(P, rows, width, segs, st);
        return hipErrorInvalidValue;
    }
    switch (vdt) {
    case RGCSR_F32: return launch_compact_v<RGCSR_F32, float>(P, rows, width, segs, st);
    case RGCSR_F16: return launch_compact_v<RGCSR_F16, float>(P, rows, width, segs, st);
    case RGCSR_BF16: return launch_compact_v<RGCSR_BF16, float>(P, rows, width, segs, st);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Pattern search on device CSR arrays
// ---------------------------------------------------------------------------
// (the same combination as on the host)
__device__ __forceinline__ uint64_t pat_mix(uint64_t h, uint64_t v) {
    h ^= v + 0x9e3779b97f4a7c15ull + (h << 6) + (h >> 2);
    h *= 0xff51afd7ed558ccdull;
    return h ^ (h >> 32);
}

// Slot of hash h in the open-addressing table of kPatHash slots, row i put
// down as its representative if it is new; -1 when there are too many lists.
__device__ __forceinline__ int pat_slot(uint64_t h, int64_t i, uint64_t *key, int32_t *rep, int32_t *state) {
    int s = (int)(h % kPatHash);
    for (int probe = 0; probe < kPatHash; probe++, s = (s + 1) % kPatHash) {
        unsigned long long *at = (unsigned long long *)key + s;
        unsigned long long k = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (k == 0) {
            k = atomicCAS(at, 0ull, (unsigned long long)h);
            if (k == 0) {
                rep[s] = (int32_t)i;
                if (atomicAdd(state, 1) >= kPatMax) state[1] = 1;
                return s;
            }
        }
        if (k == h) return s;
        if (__hip_atomic_load(state + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return -1;
    }
    state[1] = 1;
    return -1;
}

// One lane per row: the row's list hashed; the distinct hashes of a wavefront
// (a few on a structured grid) are looked up one after the other, by one lane
// each, so that the table's cache lines are not asked once per row.  Gives up
// (state[1]) at more than kPatMax lists or a row longer than kPatLen.
__global__ __launch_bounds__(256) void pat_hash_k(const int64_t *rp, const int32_t *col, int64_t n, uint64_t *key,
                                                  int32_t *rep, int32_t *state, uint16_t *slot) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n || __hip_atomic_load(state + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int64_t b = rp[i];
    const int32_t len = (int32_t)min(rp[i + 1] - b, (int64_t)kPatLen + 1);
    if (len > kPatLen) {
        state[1] = 1;
        return;
    }
    uint64_t h = pat_mix(0, (uint64_t)len);
    constexpr int U = 8;
    for (int32_t j0 = 0; j0 < len; j0 += U) {
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; u++) c[u] = col[b + min(j0 + u, len - 1)];
#pragma unroll
        for (int u = 0; u < U; u++)
            if (j0 + u < len) h = pat_mix(h, (uint64_t)((int64_t)c[u] - i));
    }
    if (h == 0) h = 1;  // 0 marks a free slot
    // each round settles the first open lane's hash and every lane that shares it
    bool open = true;
    while (open) {
        const uint64_t h0 = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(h >> 32)) << 32) |
                            (uint32_t)__builtin_amdgcn_readfirstlane((int)h);
        const int32_t i0 = __builtin_amdgcn_readfirstlane((int32_t)i);
        int s = 0;
        if ((int32_t)i == i0) s = pat_slot(h0, i, key, rep, state);
        s = __builtin_amdgcn_readfirstlane(s);
        if (s < 0) return;
        if (h == h0) {
            slot[i] = (uint16_t)s;
            open = false;
        }
    }
}

// One workgroup: the used hash slots numbered in slot order (dense) and the
// lists of their rows written to the table.
__global__ __launch_bounds__(kPatHash) void pat_table_k(const int64_t *rp, const int32_t *col, const uint64_t *key,
                                                        const int32_t *rep, int32_t *state, int32_t *dense,
                                                        int32_t *tab) {
    __shared__ int32_t cnt[kPatHash];
    __shared__ int32_t longest;
    const int t = threadIdx.x;
    if (t == 0) longest = 0;
    const bool used = !state[1] && key[t] != 0;
    cnt[t] = used;
    __syncthreads();
    const int64_t r = used ? rep[t] : 0;
    const int32_t len = used ? (int32_t)(rp[r + 1] - rp[r]) : 0;
    if (used) atomicMax(&longest, len);
    for (int off = 1; off < kPatHash; off <<= 1) {
        const int32_t v = t >= off ? cnt[t - off] : 0;
        __syncthreads();
        cnt[t] += v;
        __syncthreads();
    }
    const int32_t n_pat = cnt[kPatHash - 1], str = pat_stride(longest);
    if (n_pat == 0 || n_pat > kPatMax || n_pat * str > kPatTab) {
        if (t == 0) state[1] = 1;
        return;
    }
    if (t == 0) {
        state[0] = n_pat;
        state[2] = str;
    }
    if (!used) return;
    const int32_t p = cnt[t] - 1;
    dense[t] = p;
    int32_t *d = tab + p * str;
    d[0] = len;
    for (int32_t j = 1; j < str; j++) d[j] = j <= len ? (int32_t)((int64_t)col[rp[r] + j - 1] - r) : 0;
}

// Pattern of each row, its list compared with the table entry by entry (two
// lists of one hash: no patterns).
__global__ __launch_bounds__(256) void pat_id_k(const int64_t *rp, const int32_t *col, int64_t n, const uint16_t *slot,
                                                const int32_t *dense, const int32_t *tab, int32_t *state,
                                                uint8_t *id) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n || __hip_atomic_load(state + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int32_t p = dense[slot[i]];
    const int32_t *d = tab + p * state[2];
    const int64_t b = rp[i], len = rp[i + 1] - b;
    bool same = len == d[0];
    for (int64_t j = 0; same && j < len; j++) same = (int64_t)col[b + j] - i == d[1 + j];
    if (!same) state[1] = 1;
    id[i] = (uint8_t)p;
}

hipError_t launch_find_patterns(const int64_t *rp, const int32_t *col, int64_t n, uint64_t *key, int32_t *rep,
                                int32_t *state, uint16_t *slot, uint8_t *id, int32_t *tab, hipStream_t st) {
    const unsigned nb = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(pat_hash_k, dim3(nb), dim3(256), 0, st, rp, col, n, key, rep, state, slot);
    hipLaunchKernelGGL(pat_table_k, dim3(1), dim3(kPatHash), 0, st, rp, col, key, rep, state, rep + kPatHash, tab);
    hipLaunchKernelGGL(pat_id_k, dim3(nb), dim3(256), 0, st, rp, col, n, slot, rep + kPatHash, tab, state, id);
    return hipGetLastError();
}

// One workgroup per unit: smallest and largest column of its grouped rows
// (ascending within a row).
__global__ __launch_bounds__(256) void windows_k(const int32_t *sv, const int64_t *rp, const int32_t *col, int64_t ns,
                                                 int32_t unit_rows, int32_t *win, unsigned long long *count) {
    __shared__ int32_t slo[4], shi[4];
    int32_t lo = INT32_MAX, hi = -1;
    const int64_t s1 = min(((int64_t)blockIdx.x + 1) * unit_rows, ns);
    for (int64_t s = (int64_t)blockIdx.x * unit_rows + threadIdx.x; s < s1; s += 256) {
        const int64_t b = rp[sv[s]], e = rp[sv[s] + 1];
        if (e > b) {
            lo = min(lo, col[b]);
            hi = max(hi, col[e - 1]);
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, __shfl_xor(lo, off));
        hi = max(hi, __shfl_xor(hi, off));
    }
    if ((threadIdx.x & 63) == 0) {
        slo[threadIdx.x >> 6] = lo;
        shi[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x) return;
    for (int i = 1; i < 4; i++) {
        lo = min(lo, slo[i]);
        hi = max(hi, shi[i]);
    }
    const int32_t n = hi >= 0 ? hi - lo + 1 : 0;
    win[2 * (int64_t)blockIdx.x] = n ? lo : 0;
    win[2 * (int64_t)blockIdx.x + 1] = n;
    atomicAdd(count, (unsigned long long)n);
    atomicMax(count + 1, (unsigned long long)n);
}

hipError_t launch_windows(const int32_t *sv, const int64_t *rp, const int32_t *col, int64_t ns, int32_t unit_rows,
                          int64_t units, int32_t *win, unsigned long long *count, hipStream_t st) {
    hipLaunchKernelGGL(windows_k, dim3((unsigned)units), dim3(256), 0, st, sv, rp, col, ns, unit_rows, win, count);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void gather_id_k(const int32_t *sv, const uint8_t *id, int64_t ns, uint8_t *id_s) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < ns) id_s[i] = id[sv[i]];
}

hipError_t launch_gather_id(const int32_t *sv, const uint8_t *id, int64_t ns, uint8_t *id_s, hipStream_t st) {
    hipLaunchKernelGGL(gather_id_k, dim3((unsigned)((ns + 255) / 256)), dim3(256), 0, st, sv, id, ns, id_s);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void col16_k(const int64_t *gp, int64_t ng, int32_t unit_groups, const int32_t *win,
                                               const int32_t *slot_col, uint16_t *col16) {
    const int64_t g = (int64_t)blockIdx.x * unit_groups;
    const int64_t e = gp[min(g + unit_groups, ng)];
    const int32_t b = win[2 * (int64_t)blockIdx.x];
    for (int64_t s = gp[g] + threadIdx.x; s < e; s += 256) col16[s] = (uint16_t)max(slot_col[s] - b, 0);
}

hipError_t launch_col16(const int64_t *gp, int64_t ng, int32_t unit_groups, int64_t units, const int32_t *win,
                        const int32_t *slot_col, uint16_t *col16, hipStream_t st) {
    hipLaunchKernelGGL(col16_k, dim3((unsigned)units), dim3(256), 0, st, gp, ng, unit_groups, win, slot_col, col16);
    return hipGetLastError();
}

}  // namespace rg
