// SpMM of any width in one launch (spmm.h).
//
// KL lanes share a row of the product, each with VW neighbouring columns (16
// bytes; the last lane's start moves back to end at column k, so rows of any
// width and alignment are read whole and no lane reads past them).  A load
// instruction then covers 64 / KL rows of X, each as one run of bytes: with a
// lane per row every one of the k / 4 loads of a nonzero touched 64 cache
// lines, 64 k / 4 requests where the X rows take 64 to 128.  The row groups'
// values and columns are loaded one row per lane, as they lie, and handed to
// the lanes of each row by cross-lane reads.
//
// Bound by the X requests.  With blocks of 16, 8, 4, 2 and 1 columns and one
// lane per row before: 27-point 80^3 FP32, k = 7 (rows of 28 bytes, four
// launches) 134.3 -> 32.0 us, k = 16 91.6 -> 61.6, k = 32 224 -> 115; Zipf
// 10^6, k = 7 501 -> 148, k = 31 2383 -> 275, k = 32 198 -> 173; FP64 27-point
// 60^3, k = 17 775 -> 89.
#include <hip/hip_runtime.h>

#include "compact.h"
#include "device.h"
#include "spmm.h"

namespace rg {

template <class A, int VW> struct VecOf {
    typedef A type __attribute__((ext_vector_type(VW)));
    // rows of X and Y start at any element
    typedef type at __attribute__((aligned(sizeof(A))));
};

// Steps in flight: about 32 registers of X (16 for two and three columns), 64
// in FP64, and at most 8 steps, since narrow rows waste the rest (27-point
// 80^3 FP32, k = 7: 31.6 us with 32 registers, 34.6 with 64, 35.6 with 16;
// 7-point 80^3, k = 2: 7.3 us with 8 steps, 10.6 with 16; 27-point 60^3 FP64,
// k = 12: 70 with 64 registers, 101 with 32).
template <class A, int VW, int NB> constexpr int spmm_steps() {
    constexpr int regs = sizeof(A) == 8 ? 64 : (VW == 2 ? 16 : 32);
    constexpr int u = regs * 4 / (int)sizeof(A) / (NB * VW);
    return u > 8 ? 8 : (u > 0 ? u : 1);
}

template <class A, int VW> struct SpmmCols {
    const A *x;   // X + this lane's first column
    A *y;
    int64_t ldx, ldy;
};

// acc += a * xv where on (a row's steps end at its length: what lies behind
// is never multiplied)
template <class A, int VW>
__device__ __forceinline__ void spmm_fma(A a, const typename VecOf<A, VW>::type &xv, bool on,
                                         typename VecOf<A, VW>::type &acc) {
#pragma unroll
    for (int i = 0; i < VW; i++) {
        const A f = fmaA(a, xv[i], acc[i]);
        acc[i] = on ? f : acc[i];
    }
}

// 64 rows of the grouped part (a wave item).  MASK: X rows are loaded up to a
// row's own length only (spmm_masked); otherwise steps past it load again, with
// no branch around a load.
template <int VD, class A, int VW, int KL, bool PAT, bool MASK>
__device__ __forceinline__ void spmm_groups(const SpmvParams &P, const SpmmCols<A, VW> &C, int32_t w, int lane,
                                            const int32_t *tab) {
    using V = Val<VD>;
    using S = typename V::S;
    using X = typename VecOf<A, VW>::type;
    using XA = typename VecOf<A, VW>::at;
    constexpr int NB = KL, RW = 64 / KL, U = spmm_steps<A, VW, NB>();
    const LaneRow L = lane_row<1>(P, w, lane);
    const int32_t orow = L.ok ? (P.perm ? P.short_row[L.i] : (int32_t)L.i) : -1;
    // sliced ELLPACK multiplies its padding
    const int32_t len = L.ok && P.pad == 2 ? L.wc : L.len;
    int32_t cmax = len;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cmax = max(cmax, __shfl_xor(cmax, off));
    cmax = __builtin_amdgcn_readfirstlane(cmax);
    const int32_t pt = PAT && L.ok ? (int32_t)P.pat_id[L.i] * P.pat_stride + 1 : 0;
    int32_t lenb[NB], rowb[NB], ptb[NB];
    X acc[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const int src = b * RW + lane / KL;
        lenb[b] = KL == 1 ? len : __shfl(len, src);
        rowb[b] = KL == 1 ? orow : __shfl(orow, src);
        ptb[b] = PAT ? (KL == 1 ? pt : __shfl(pt, src)) : 0;
        acc[b] = X(A(0));
    }
    const S *vals = (const S *)P.slot_val;
    // steps past a row's length re-read its first slot (slot 0 in a group
    // without slots)
    const int64_t base0 = L.wc > 0 ? L.base : 0;
    for (int32_t c0 = 0; c0 < cmax; c0 += U) {
        S v[U];
        int32_t ci[U];
        X xv[U][NB];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t s = c0 + u < len ? L.base + (int64_t)(c0 + u) * L.stride : base0;
            v[u] = ldnt(vals + s);
            if constexpr (!PAT) ci[u] = ldnt(P.slot_col + s);
        }
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const int src = b * RW + lane / KL;
                int32_t c;
                if constexpr (PAT) c = (int32_t)min((uint32_t)(rowb[b] + tab[ptb[b] + c0 + u]), (uint32_t)P.last_col);
                else c = KL == 1 ? ci[u] : __shfl(ci[u], src);
                if constexpr (MASK) xv[u][b] = X(A(0));
                if (!MASK || c0 + u < lenb[b]) xv[u][b] = *reinterpret_cast<const XA *>(C.x + (int64_t)c * C.ldx);
            }
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const S t = KL == 1 ? v[u] : __shfl(v[u], b * RW + lane / KL);
                spmm_fma<A, VW>(V::template cvt<A>(t), xv[u][b], c0 + u < lenb[b], acc[b]);
            }
    }
#pragma unroll
    for (int b = 0; b < NB; b++)
        if (rowb[b] >= 0) *reinterpret_cast<XA *>(C.y + (int64_t)rowb[b] * C.ldy) = acc[b];
}

// acc += elements o, o + stride, ... < e of the long-row segment
template <int VD, class A, int VW>
__device__ __forceinline__ void spmm_strided(const SpmvParams &P, const SpmmCols<A, VW> &C, int64_t base, int32_t o,
                                             int32_t e, int32_t stride, typename VecOf<A, VW>::type &acc) {
    using V = Val<VD>;
    using S = typename V::S;
    using X = typename VecOf<A, VW>::type;
    using XA = typename VecOf<A, VW>::at;
    constexpr int U = 8;
    const S *vb = (const S *)P.long_val + base;
    const int32_t *cb = P.long_col + base;
    for (int32_t o0 = o; o0 < e; o0 += stride * U) {
        S v[U];
        int32_t ci[U];
        X xv[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int32_t oo = o0 + u * stride < e ? o0 + u * stride : o;
            v[u] = ldnt(vb + oo);
            ci[u] = ldnt(cb + oo);
        }
#pragma unroll
        for (int u = 0; u < U; u++) xv[u] = *reinterpret_cast<const XA *>(C.x + (int64_t)ci[u] * C.ldx);
#pragma unroll
        for (int u = 0; u < U; u++)
            spmm_fma<A, VW>(V::template cvt<A>(v[u]), xv[u], o0 + u * stride < e, acc);
    }
}

// A wavefront item of long rows: each row takes its item's lanes, KL of them
// at least, so that every column part has a lane; KL of them share an element.
template <int VD, class A, int VW, int KL>
__device__ __forceinline__ void spmm_wave_long(const SpmvParams &P, const SpmmCols<A, VW> &C, int32_t w, int lane) {
    using X = typename VecOf<A, VW>::type;
    using XA = typename VecOf<A, VW>::at;
    const LongItem it = ldc(P.wave_work, w);
    const int64_t item0 = ldc(P.long_ptr, (int64_t)it.a);
    const int LPR = max(it.c, KL), sh = 31 - __builtin_clz(LPR);
    const int rpp = 64 >> sh, slot = (lane & (LPR - 1)) / KL;
    for (int r0 = 0; r0 < it.b; r0 += rpp) {
        const int r = r0 + (lane >> sh);
        const bool ok = r < it.b;
        const int64_t li = (int64_t)it.a + (ok ? r : 0);
        const int32_t b = (int32_t)(P.long_ptr[li] - item0), e = ok ? (int32_t)(P.long_ptr[li + 1] - item0) : 0;
        const int32_t orow = P.long_row[li];
        X acc = X(A(0));
        spmm_strided<VD, A, VW>(P, C, item0, b + slot, e, LPR / KL, acc);
#pragma unroll
        for (int off = 32; off >= KL; off >>= 1)
            if (off < LPR)
#pragma unroll
                for (int i = 0; i < VW; i++) acc[i] += __shfl_xor(acc[i], off);
        if (ok && slot == 0) *reinterpret_cast<XA *>(C.y + (int64_t)orow * C.ldy) = acc;
    }
}

// One chunk of a very long row, reduced by the workgroup in LDS.
template <int VD, class A, int VW, int KL>
__device__ __forceinline__ void spmm_block_item(const SpmvParams &P, const SpmmCols<A, VW> &C, int32_t u, int k,
                                                int32_t cs, typename VecOf<A, VW>::type (*red)[KL]) {
    using X = typename VecOf<A, VW>::type;
    using XA = typename VecOf<A, VW>::at;
    const LongItem it = ldc(P.block_work, u);
    const int64_t li = it.a;
    const int64_t beg = ldc(P.long_ptr, li) + (int64_t)it.b * kBlockChunk;
    const int32_t n = (int32_t)min(ldc(P.long_ptr, li + 1) - beg, kBlockChunk);
    X acc = X(A(0));
    spmm_strided<VD, A, VW>(P, C, beg, (int32_t)threadIdx.x / KL, n, kBlockThreads / KL, acc);
#pragma unroll
    for (int off = 32; off >= KL; off >>= 1)
#pragma unroll
        for (int i = 0; i < VW; i++) acc[i] += __shfl_xor(acc[i], off);
    const int wv = threadIdx.x >> 6, p = threadIdx.x % KL;
    if ((threadIdx.x & 63) < KL) red[wv][p] = acc;
    __syncthreads();
    if (threadIdx.x < KL) {
        X tot = red[0][p];
#pragma unroll
        for (int i = 1; i < kBlockWaves; i++) tot += red[i][p];
        if (it.c == 1) *reinterpret_cast<XA *>(C.y + (int64_t)ldc(P.long_row, li) * C.ldy) = tot;
        else *reinterpret_cast<XA *>((A *)P.partial + ((int64_t)it.d + it.b) * k + cs) = tot;
    }
    __syncthreads();
}

template <int VD, class A, int VW, int KL, bool LONG, bool PAT, bool MASK>
__global__ __launch_bounds__(kBlockThreads) void spmm_k(SpmvParams P, int32_t k) {
    using X = typename VecOf<A, VW>::type;
    __shared__ X red[LONG ? kBlockWaves : 1][KL];
    __shared__ int32_t tab[PAT ? kPatTab + 32 : 1];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int32_t cs = min((lane % KL) * VW, k - VW);
    const SpmmCols<A, VW> C{(const A *)P.x + cs, (A *)P.y + cs, P.ldx, P.ldy};
    if constexpr (PAT) {
        for (int i = threadIdx.x; i < P.pat_ints; i += kBlockThreads) tab[i] = P.pat_tab[i];
        __syncthreads();
    }
    const int nwg = gridDim.x;
    for (int32_t u = first_unit(blockIdx.x, nwg, P.n_long_units); u < P.total_units; u += nwg) {
        if (LONG && u < P.n_block_items) {
            spmm_block_item<VD, A, VW, KL>(P, C, u, k, cs, red);
            continue;
        }
        const int32_t w = __builtin_amdgcn_readfirstlane((u - (LONG ? P.n_block_items : 0)) * kBlockWaves + wv);
        if (w >= P.n_wave_items) continue;
        if (LONG && w < P.n_wave_long) spmm_wave_long<VD, A, VW, KL>(P, C, w, lane);
        else spmm_groups<VD, A, VW, KL, PAT, MASK>(P, C, w - (LONG ? P.n_wave_long : 0), lane, tab);
    }
}

// Whether X rows past a row's length are left out.  It pays where the loads are
// what bounds the launch, from about eight wavefronts of row groups per CU, four
// with long rows beside them, and while the steps walked are 3/2 of the nonzeros
// or more (twice with one step in flight).  Loaded again against left out:
// 300,000 rows of 4 nonzeros in a band, rows as they come (2.8 and 2.5 steps a
// nonzero), FP32 k = 8 20.7 against 15.8 us, FP64 k = 16 45.4 against 37.2; of 20
// (1.66), FP32 k = 8 50.7 against 46.4; 200,000 Zipf rows (8 steps), FP64 k = 32
// 206 against 130; but rows of 24, sorted (1.2), FP32 k = 32 92 against 101, and
// 30,000 rows of 4 (470 wavefronts), FP32 k = 16 6.6 against 8.9, 100,000 8.5
// against 9.6.  Beside long rows one step in flight needs 3/2 as well (Zipf 10^6,
// tau = 6, 1.7 steps: FP64 k = 32 390 against 331), and in FP64 no number of rows
// (30,000 Zipf rows: 77 against 58).
static bool spmm_masked(const SpmmFill &F, int steps, bool long_rows, bool f64) {
    const bool busy = F.rows >= kSpmmBusyWaves * 64 / (long_rows ? 2 : 1) || (long_rows && f64 && steps == 1);
    const int64_t walked = F.slots + F.rows * steps / 2;
    return busy && (steps > 1 || long_rows ? 2 * walked >= 3 * F.nnz : walked >= 2 * F.nnz);
}

template <int VD, class A, int VW, int KL>
static hipError_t launch_spmm_t(const SpmvParams &P, const SpmmFill &F, int k, int nwg, hipStream_t st) {
    const dim3 g(nwg), b(kBlockThreads);
    const bool long_rows = P.n_block_items + P.n_wave_long > 0;
    const bool mask = spmm_masked(F, spmm_steps<A, VW, KL>(), long_rows, sizeof(A) == 8);
    if (long_rows) {
        if (mask) hipLaunchKernelGGL((spmm_k<VD, A, VW, KL, true, false, true>), g, b, 0, st, P, k);
        else hipLaunchKernelGGL((spmm_k<VD, A, VW, KL, true, false, false>), g, b, 0, st, P, k);
    } else if (P.compact == kCompactPattern) {
        hipLaunchKernelGGL((spmm_k<VD, A, VW, KL, false, true, false>), g, b, 0, st, P, k);
    } else {
        if (mask) hipLaunchKernelGGL((spmm_k<VD, A, VW, KL, false, false, true>), g, b, 0, st, P, k);
        else hipLaunchKernelGGL((spmm_k<VD, A, VW, KL, false, false, false>), g, b, 0, st, P, k);
    }
    return hipGetLastError();
}

// lanes per row: the power of two that covers k columns
template <int VD, class A> static hipError_t launch_spmm_v(const SpmvParams &P, const SpmmFill &F, int k, int nwg, hipStream_t st) {
    constexpr int VW = 16 / (int)sizeof(A);
    if constexpr (sizeof(A) == 4) {
        if (k == 2) return launch_spmm_t<VD, A, 2, 1>(P, F, k, nwg, st);
        if (k == 3) return launch_spmm_t<VD, A, 2, 2>(P, F, k, nwg, st);
    }
    if (k <= VW) return launch_spmm_t<VD, A, VW, 1>(P, F, k, nwg, st);
    if (k <= 2 * VW) return launch_spmm_t<VD, A, VW, 2>(P, F, k, nwg, st);
    if (k <= 4 * VW) return launch_spmm_t<VD, A, VW, 4>(P, F, k, nwg, st);
    if (k <= 8 * VW) return launch_spmm_t<VD, A, VW, 8>(P, F, k, nwg, st);
    if constexpr (sizeof(A) == 8) return launch_spmm_t<VD, A, VW, 16>(P, F, k, nwg, st);
    return hipErrorInvalidValue;
}

hipError_t launch_spmm(const SpmvParams &P, const SpmmFill &F, int vdt, int vec_f64, int k, int nwg, hipStream_t st) {
    if (k < 2 || k > kSpmmMax) return hipErrorInvalidValue;
    if (vec_f64) {
        if (vdt == RGCSR_F64) return launch_spmm_v<RGCSR_F64, double>(P, F, k, nwg, st);
        if (vdt == RGCSR_F32) return launch_spmm_v<RGCSR_F32, double>(P, F, k, nwg, st);
        return hipErrorInvalidValue;
    }
    if (vdt == RGCSR_F32) return launch_spmm_v<RGCSR_F32, float>(P, F, k, nwg, st);
    return hipErrorInvalidValue;
}

template <class A>
__global__ __launch_bounds__(256) void spmm_combine_k(const LongItem *items, int32_t n, const int32_t *long_row,
                                                      const A *partial, A *Y, int64_t ldy, int32_t k) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)n * k) return;
    const LongItem it = items[t / k];
    const int32_t j = (int32_t)(t % k);
    A tot = A(0);
    for (int c = 0; c < it.c; c++) tot += partial[((int64_t)it.d + c) * k + j];
    Y[(int64_t)long_row[it.a] * ldy + j] = tot;
}

hipError_t launch_spmm_combine(const LongItem *items, int32_t n, const int32_t *long_row, const void *partial, void *Y,
                               int64_t ldy, int vec_f64, int k, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const dim3 g((unsigned)(((int64_t)n * k + 255) / 256)), b(256);
    if (vec_f64)
        hipLaunchKernelGGL(spmm_combine_k<double>, g, b, 0, st, items, n, long_row, (const double *)partial,
                           (double *)Y, ldy, k);
    else
        hipLaunchKernelGGL(spmm_combine_k<float>, g, b, 0, st, items, n, long_row, (const float *)partial, (float *)Y,
                           ldy, k);
    return hipGetLastError();
}

}  // namespace rg
