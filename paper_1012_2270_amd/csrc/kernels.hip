// HIP kernels of librgcsr for gfx950 (MI355X: 256 CUs in 8 XCDs, wave64).
//
// SpMV is memory bound (Section 1: one multiply and one add per nonzero,
// arithmetic intensity below one flop per byte), so nothing here uses MFMA:
// the kernels are about coalesced value/column streams, keeping x in cache
// and enough independent loads in flight per wavefront.
//
//   rgcsr_spmv_k   RgCSR SpMV/SpMM (Section 3.4).  Wavefronts [0, n_long)
//                  run long-row work items, the rest run row groups.  In a
//                  group the lanes walk rows with the group's row count as
//                  stride and stop after rowLength steps, so padding is never
//                  multiplied; loads of up to 8 steps are issued before the
//                  dependent x gathers.  Value and column streams use
//                  nontemporal loads so x keeps the caches.
//   hyb_ell_k /    Hybrid ELL + COO (Section 3.3): ELL writes every row, COO
//   hyb_coo_k      adds the remaining entries per row run.
//   setval_k,      value update and backward pass over the same walk.
//   grad_k
//   dot/refine     conjugate-gradient vector kernels (FP64 dot accumulation).
#include <hip/hip_runtime.h>

#include <mutex>

#include "device.h"
#include "internal.h"
#include "kernels.h"

namespace rg {

// ---------------------------------------------------------------------------
// RgCSR SpMV / SpMM
//
// Every loop body is split into three phases so that all loads of a phase are
// in flight together: (1) value and column loads of U steps, (2) the x
// gathers those columns select, (3) the multiply-adds.  Steps past a row's
// length are neither loaded nor multiplied (the row-length bound of the RgCSR
// kernel), and each lane keeps the paper's serial order within its row.
// ---------------------------------------------------------------------------
// Row groups when every lane of a wavefront belongs to the same group
// (G*T a multiple of 64): the group pointers are scalar, value/column loads
// use 32-bit offsets from the group's first slot.  PAD: 0 = loads and
// multiplies stop at the row length (the RgCSR kernel of Section 3.4); 1 =
// loads run over the group width, multiplies stop at the row length; 2 =
// sliced ELLPACK (Section 3.3): no row lengths, every slot of the group width
// is multiplied, padding included; 3 = loads over the group width and the row
// length read off the columns: they ascend strictly within a row and padding
// repeats the row's last column, so a step is multiplied exactly when its
// column exceeds the previous step's (one lane per row, no empty rows; the
// host checks both).
template <int VD, class A, int K, int T, int R, int PAD, int LP, int SB>
__device__ __forceinline__ void spmv_groups_uniform(const SpmvParams &P, int32_t first, int lane) {
    using V = Val<VD>;
    using S = typename V::S;
    const A *X = (const A *)P.x;
    A *Y = (A *)P.y;
    const uint32_t xrow = (uint32_t)(P.ldx * (int64_t)sizeof(A));
    const S *vb[R];
    const int32_t *cb[R];
    int32_t off0[R], stride[R], nl[R], len[R], rowi[R], orow[R];
    bool ok[R];
    int q = 0;
    int cmax = 0;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int32_t wr = first + r;
        const int32_t g = __builtin_amdgcn_readfirstlane(wr / P.wpg);
        const int lr = (wr - g * P.wpg) * 64 + lane;
        const GroupMeta m = group_meta_uniform(P, g);
        const int t = lr / T;
        q = lr % T;
        ok[r] = t < m.sg;
        rowi[r] = (int32_t)m.row0 + t;
        // unconditional loads at a clamped index (no branch around them);
        // the output row is fetched now so the final store does not wait.
        // PAD 2 and 3 read no row lengths.
        if constexpr (PAD < 2) len[r] = P.short_len[ok[r] ? rowi[r] : 0];
        else len[r] = 0;
        orow[r] = P.perm ? P.short_row[ok[r] ? rowi[r] : 0] : rowi[r];
        stride[r] = m.sg * T;
        const bool has = m.g1 > m.g0;
        // a group without slots points at slot 0 (read only when the loop runs)
        const int64_t gb = has ? m.g0 : 0;
        vb[r] = (const S *)P.slot_val + gb;
        cb[r] = P.slot_col + gb;
        off0[r] = t * T + q;
        if constexpr (PAD) {
            const int32_t wc = has ? (int32_t)((uint32_t)(m.g1 - m.g0) / (uint32_t)stride[r]) : 0;
            nl[r] = ok[r] ? wc : 0;
            cmax = max(cmax, nl[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++) len[r] = ok[r] ? len[r] : 0;
    if constexpr (!PAD) {
        cmax = 0;
#pragma unroll
        for (int r = 0; r < R; r++) {
            nl[r] = len[r] > q ? (len[r] - q + T - 1) / T : 0;
            cmax = max(cmax, nl[r]);
        }
    }
    A acc[R][K];
#pragma unroll
    for (int r = 0; r < R; r++)
#pragma unroll
        for (int k = 0; k < K; k++) acc[r][k] = A(0);
    // steps per pass: SB / R (the host's rows-per-lane choice uses the same
    // step budget); several right-hand sides: the X-row budget over R rows
    constexpr int U = K == 1 ? SB / R : (R == 1 ? unroll_for<K>() : (multi_steps<K>() / R > 0 ? multi_steps<K>() / R : 1));
    // Inside the unrolled body every load is issued unconditionally (steps past
    // the bound read the group's first slot and x[0], in bounds whenever the
    // loop runs) and results are masked with selects, so the loads of a phase
    // are not split by branches and are in flight together.
    int32_t prevc[R];  // PAD == 3: column of the previous step
#pragma unroll
    for (int r = 0; r < R; r++) prevc[r] = -1;
    for (int c0 = 0; c0 < cmax; c0 += U) {
        S v[R][U];
        int32_t ci[R][U];
        A xv[R][U][K];
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint32_t o = c0 + u < nl[r] ? (uint32_t)(off0[r] + (c0 + u) * stride[r]) : 0u;
                v[r][u] = ld_stream<LP>((const S *)((const char *)vb[r] + o * (uint32_t)sizeof(S)));
                ci[r][u] = ld_stream<LP>((const int32_t *)((const char *)cb[r] + o * 4u));
            }
        // steps multiplied: up to the row length, or (PAD == 2) every slot of
        // the group width, padding included
        int n[R];
#pragma unroll
        for (int r = 0; r < R; r++) n[r] = PAD >= 2 ? nl[r] : (len[r] > q ? (len[r] - q + T - 1) / T : 0);
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                // PAD == 3: a padding step (column not above the previous one)
                // gathers x[0] like a step past the row length, not x at the
                // row's last column
                bool g = c0 + u < n[r];
                if constexpr (PAD == 3) g = g && ci[r][u] > (u == 0 ? prevc[r] : ci[r][u - 1]);
                const int32_t c = g ? ci[r][u] : 0;
                if constexpr (K == 1) xv[r][u][0] = ldx32<LP>(X, c, xrow);
                else load_row<A, K>(X + (int64_t)c * P.ldx, xv[r][u]);
            }
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                bool on = c0 + u < n[r];
                if constexpr (PAD == 3) {
                    on = on && ci[r][u] > prevc[r];
                    prevc[r] = ci[r][u];
                }
                const A a = V::template cvt<A>(v[r][u]);
#pragma unroll
                for (int k = 0; k < K; k++) {
                    const A f = fmaA(a, xv[r][u][k], acc[r][k]);
                    acc[r][k] = on ? f : acc[r][k];
                }
            }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        if constexpr (T > 1) {
#pragma unroll
            for (int off = T / 2; off > 0; off >>= 1)
#pragma unroll
                for (int k = 0; k < K; k++) acc[r][k] += __shfl_xor(acc[r][k], off);
        }
        if (ok[r] && q == 0) store_row<A, K>(out_row<K>(Y, P.ldy, P.pan_y, P.pan_ld, orow[r]), acc[r]);
    }
}

// Row groups of fewer than 64 lanes (several groups per wavefront): one row
// per lane, per-lane group metadata.
template <int VD, class A, int K, int T, int LP>
__device__ __forceinline__ void spmv_groups_lane(const SpmvParams &P, int32_t w, int lane) {
    using V = Val<VD>;
    using S = typename V::S;
    const S *vals = (const S *)P.slot_val;
    const A *X = (const A *)P.x;
    A *Y = (A *)P.y;
    const LaneRow L = lane_row<T>(P, w, lane);
    const int n = L.len > L.q ? (L.len - L.q + T - 1) / T : 0;
    A acc[K];
#pragma unroll
    for (int k = 0; k < K; k++) acc[k] = A(0);
    constexpr int U = K == 1 ? 8 : unroll_for<K>();
    for (int c0 = 0; c0 < n; c0 += U) {
        S v[U];
        int32_t ci[U];
        A xv[U][K];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t s = c0 + u < n ? L.base + (int64_t)(c0 + u) * L.stride : L.base;
            v[u] = ld_stream<LP>(vals + s);
            ci[u] = ld_stream<LP>(P.slot_col + s);
        }
#pragma unroll
        for (int u = 0; u < U; u++) load_row<A, K>(X + (int64_t)ci[u] * P.ldx, xv[u]);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const bool on = c0 + u < n;
            const A a = V::template cvt<A>(v[u]);
#pragma unroll
            for (int k = 0; k < K; k++) {
                const A f = fmaA(a, xv[u][k], acc[k]);
                acc[k] = on ? f : acc[k];
            }
        }
    }
    if constexpr (T > 1) {
#pragma unroll
        for (int off = T / 2; off > 0; off >>= 1)
#pragma unroll
            for (int k = 0; k < K; k++) acc[k] += __shfl_xor(acc[k], off);
    }
    if (L.ok && L.q == 0) {
        const int32_t row = P.perm ? P.short_row[L.i] : (int32_t)L.i;
        store_row<A, K>(out_row<K>(Y, P.ldy, P.pan_y, P.pan_ld, row), acc);
    }
}

template <int VD, class A, int K, int T, int R, int LP, int SB>
__device__ __forceinline__ void spmv_groups_fixed(const SpmvParams &P, int32_t first, int lane) {
    if (P.pad == 3) {
        if constexpr (T == 1) spmv_groups_uniform<VD, A, K, T, R, 3, LP, SB>(P, first, lane);
    } else if (P.pad == 2) spmv_groups_uniform<VD, A, K, T, R, 2, LP, SB>(P, first, lane);
    else if (P.pad) spmv_groups_uniform<VD, A, K, T, R, 1, LP, SB>(P, first, lane);
    else spmv_groups_uniform<VD, A, K, T, R, 0, LP, SB>(P, first, lane);
}

// R > 0: every wavefront takes R consecutive wave items.  R = 0: wavefront w
// takes the run of wave items that item word w names (first item << 2 |
// log2 of the run length), so narrow groups are packed several to a
// wavefront and wide ones run alone.
template <int VD, class A, int K, int T, int R, int LP>
__device__ __forceinline__ void spmv_short(const SpmvParams &P, int32_t w, int lane) {
    if constexpr (R == 0) {
        const int32_t it = ldc(P.short_items, w);
        const int32_t first = it >> 2;
        switch (it & 3) {
            case 0: spmv_groups_fixed<VD, A, K, T, 1, LP, kLaneSteps>(P, first, lane); break;
            case 1: spmv_groups_fixed<VD, A, K, T, 2, LP, kLaneSteps>(P, first, lane); break;
            case 2: spmv_groups_fixed<VD, A, K, T, 4, LP, kLaneSteps>(P, first, lane); break;
            default: spmv_groups_fixed<VD, A, K, T, 8, LP, kLaneSteps>(P, first, lane); break;
        }
    } else if (P.wpg > 0) {
        // one rows-per-lane count for every wavefront (uniform widths): 8-byte
        // values take half the step budget, whose loads and x gathers need
        // twice the registers
        spmv_groups_fixed<VD, A, K, T, R, LP, VD == RGCSR_F64 ? kLaneSteps / 2 : kLaneSteps>(P, w * R, lane);
    } else if constexpr (R == 1) {
        spmv_groups_lane<VD, A, K, T, LP>(P, w, lane);
    }
}

// Elements o, o + stride, ... < e of one lane, where offsets are 32-bit and
// relative to uniform bases vb/cb (scalar base + vector offset addressing).
// Branch-free unrolled body as in the row groups: out-of-range steps re-read
// the lane's first element (valid whenever the loop runs) and are masked.
template <int VD, class A, int K, int U, int LP>
__device__ __forceinline__ void strided_dot32(const typename Val<VD>::S *vb, const int32_t *cb, const A *X,
                                              int64_t ldx, uint32_t xrow, int32_t o, int32_t e, int32_t stride,
                                              A (&acc)[K], int32_t lo = 0) {
    using V = Val<VD>;
    using S = typename V::S;
    for (int32_t o0 = o; o0 < e; o0 += stride * U) {
        S v[U];
        int32_t ci[U];
        A xv[U][K];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t oo = (uint32_t)(o0 + u * stride < e ? o0 + u * stride : o);
            v[u] = ld_stream<LP>((const S *)((const char *)vb + oo * (uint32_t)sizeof(S)));
            ci[u] = ld_stream<LP>((const int32_t *)((const char *)cb + oo * 4u));
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            if constexpr (K == 1) xv[u][0] = ldx32<LP>(X, ci[u], xrow);
            else load_row<A, K>(X + (int64_t)ci[u] * ldx, xv[u]);
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const bool on = o0 + u * stride < e && o0 + u * stride >= lo;
            const A a = V::template cvt<A>(v[u]);
#pragma unroll
            for (int k = 0; k < K; k++) {
                const A f = fmaA(a, xv[u][k], acc[k]);
                acc[k] = on ? f : acc[k];
            }
        }
    }
}

// Long rows of at most kWaveRowMax nonzeros: it.b consecutive rows of the
// long list with it.c lanes each.  Their nonzeros are contiguous, so offsets
// are taken from the item's first nonzero (a scalar load).
template <int VD, class A, int K, int LP>
__device__ __forceinline__ void spmv_wave_long(const SpmvParams &P, int32_t w, int lane) {
    using S = typename Val<VD>::S;
    A *Y = (A *)P.y;
    const A *X = (const A *)P.x;
    const LongItem it = ldc(P.wave_work, w);
    const int TL = it.c;
    const int sh = 31 - __builtin_clz(TL);
    const int r = lane >> sh, q = lane & (TL - 1);
    const bool ok = r < it.b;
    const int64_t item0 = ldc(P.long_ptr, (int64_t)it.a);
    const int64_t li = (int64_t)it.a + (ok ? r : 0);
    const int32_t b = (int32_t)(P.long_ptr[li] - item0), e = ok ? (int32_t)(P.long_ptr[li + 1] - item0) : 0;
    const int32_t orow = P.long_row[li];  // fetched early, stored at the end
    const S *vb = (const S *)P.long_val + item0;
    const int32_t *cb = P.long_col + item0;
    A acc[K];
#pragma unroll
    for (int k = 0; k < K; k++) acc[k] = A(0);
    // a lane's (at most kWaveUnroll) nonzeros in one pass while their X rows
    // fit the multi-column register budget
    constexpr int U = K == 1 ? kWaveUnroll : (multi_steps<K>() >= kWaveUnroll ? kWaveUnroll : unroll_for<K>());
    strided_dot32<VD, A, K, U, LP>(vb, cb, X, P.ldx, (uint32_t)(P.ldx * (int64_t)sizeof(A)), b + q, e, TL, acc);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        if (off < TL)
#pragma unroll
            for (int k = 0; k < K; k++) acc[k] += __shfl_xor(acc[k], off);
    if (ok && q == 0) store_row<A, K>(out_row<K>(Y, P.ldy, P.pan_y, P.pan_ld, orow), acc);
}

// Same work item, single right-hand side: the item's nonzeros (at most
// kWaveRowMax, contiguous) are loaded element-parallel, lane l taking elements
// l, l + 64, ..., so the value/column loads need no row bounds and every lane
// is busy; the products (in the accumulation type A) go to this wavefront's
// LDS slice and the item's lane-per-row mapping then sums them in the same
// strided order as spmv_wave_long.
template <int VD, class A, int LP>
__device__ __forceinline__ void spmv_wave_long_lds(const SpmvParams &P, int32_t w, int lane, A *buf) {
    using V = Val<VD>;
    using S = typename V::S;
    // the load window starts at the 32-element boundary below the item (d
    // elements early), so each load instruction covers the fewest cache lines
    constexpr int U = (kWaveRowMax + 31 + 63) / 64;
    A *Y = (A *)P.y;
    const A *X = (const A *)P.x;
    const uint32_t xrow = (uint32_t)(P.ldx * (int64_t)sizeof(A));
    const LongItem it = ldc(P.wave_work, w);
    const int64_t item0 = ldc(P.long_ptr, (int64_t)it.a);
    const int32_t n = (int32_t)(ldc(P.long_ptr, (int64_t)it.a + it.b) - item0);
    const int32_t d = (int32_t)(item0 & 31);
    const S *vb = (const S *)P.long_val + (item0 - d);
    const int32_t *cb = P.long_col + (item0 - d);
    S v[U];
    int32_t ci[U];
    A xv[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int32_t p = lane + 64 * u;
        const uint32_t o = p < n + d ? (uint32_t)p : (uint32_t)d;
        v[u] = ld_stream<LP>((const S *)((const char *)vb + o * (uint32_t)sizeof(S)));
        ci[u] = ld_stream<LP>((const int32_t *)((const char *)cb + o * 4u));
    }
    // row bounds and output row of this lane, needed only after the gathers
    const int TL = it.c;
    const int sh = 31 - __builtin_clz(TL);
    const int r = lane >> sh, q = lane & (TL - 1);
    const bool ok = r < it.b;
    const int64_t li = (int64_t)it.a + (ok ? r : 0);
    const int32_t b = (int32_t)(P.long_ptr[li] - item0), e = (int32_t)(P.long_ptr[li + 1] - item0);
    const int32_t orow = P.long_row[li];
#pragma unroll
    for (int u = 0; u < U; u++) xv[u] = ldx32<LP>(X, ci[u], xrow);
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int32_t e = lane + 64 * u - d;  // element of the item
        if (e >= 0 && e < n) buf[e] = V::template cvt<A>(v[u]) * xv[u];
    }
    if (lane == 0) buf[kWaveRowMax] = A(0);  // terms past a row read this slot
    // the slice is private to this wavefront: LDS accesses of one wavefront
    // complete in order, only the compiler must not move the reads up
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int32_t nj = ok && e - b > q ? (e - b - q + TL - 1) >> sh : 0;
    A acc = A(0);
#pragma nounroll
    for (int j0 = 0; j0 < kWaveUnroll; j0 += 4)
#pragma unroll
        for (int j = j0; j < j0 + 4; j++) acc += buf[j < nj ? b + q + j * TL : kWaveRowMax];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        if (off < TL) acc += __shfl_xor(acc, off);
    if (ok && q == 0) Y[(int64_t)orow * P.ldy] = acc;
}

// One chunk (at most kBlockChunk nonzeros) of a very long row, reduced by the
// whole workgroup in LDS.
template <int VD, class A, int K, int LP>
__device__ __forceinline__ void spmv_block_item(const SpmvParams &P, int32_t u, A (*red)[K]) {
    using S = typename Val<VD>::S;
    A *Y = (A *)P.y;
    const A *X = (const A *)P.x;
    const LongItem it = ldc(P.block_work, u);
    const int64_t li = it.a;
    const int64_t beg = ldc(P.long_ptr, li) + (int64_t)it.b * kBlockChunk;
    const int32_t n = (int32_t)min(ldc(P.long_ptr, li + 1) - beg, kBlockChunk);
    A acc[K];
#pragma unroll
    for (int k = 0; k < K; k++) acc[k] = A(0);
    constexpr int U = K == 1 || multi_steps<K>() >= 16 ? 16 : unroll_for<K>();
    // start the threads' walk at the 32-element boundary below the chunk, so
    // each wavefront's 64 consecutive loads cover the fewest cache lines; the
    // d elements before the chunk are loaded but not multiplied
    const int32_t d = (int32_t)(beg & 31);
    strided_dot32<VD, A, K, U, LP>((const S *)P.long_val + (beg - d), P.long_col + (beg - d), X, P.ldx,
                                   (uint32_t)(P.ldx * (int64_t)sizeof(A)), (int32_t)threadIdx.x, n + d,
                                   kBlockThreads, acc, d);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < K; k++) acc[k] += __shfl_xor(acc[k], off);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < K; k++) red[wv][k] = acc[k];
    __syncthreads();
    if (threadIdx.x < K) {
        const int k = threadIdx.x;
        A tot = A(0);
        for (int i = 0; i < kBlockWaves; i++) tot += red[i][k];
        if (it.c == 1)
            out_row<K>(Y, P.ldy, P.pan_y, P.pan_ld, ldc(P.long_row, li))[k] = tot;
        else
            ((A *)P.partial)[((int64_t)it.d + it.b) * K + k] = tot;
    }
    __syncthreads();
}

// Combine unit of the column-tiled rows (tiles.h): the workgroup's 64 rows,
// one per lane, so each load reads 64 consecutive partial sums; wavefront w
// adds tiles [w * q, (w + 1) * q) in tile order, then one wavefront adds the
// four sums in wavefront order (a fixed order; chains of q + 4 additions).
// A is the vector type (FP64 partial sums for F64 storage, else FP32).
template <class A>
__device__ __forceinline__ void tile_combine_unit(const SpmvParams &P, int32_t ui, int lane, int wv, A *lds) {
    const int32_t k = ui * 64 + lane;
    const int q = (P.n_tiles + kBlockWaves - 1) / kBlockWaves;
    const int t0 = min(wv * q, P.n_tiles), t1 = min(t0 + q, P.n_tiles);
    const int64_t nt = P.n_trows;
    A run = A(0);
    if (k < P.n_trows) {
        const A *p = (const A *)P.tile_partial + k;
        int t = t0;
        for (; t + 16 <= t1; t += 16) {
            A v[16];
#pragma unroll
            for (int j = 0; j < 16; j++) v[j] = p[(int64_t)(t + j) * nt];
#pragma unroll
            for (int j = 0; j < 16; j++) run += v[j];
        }
        for (; t < t1; t++) run += p[(int64_t)t * nt];
    }
    lds[wv * 64 + lane] = run;
    __syncthreads();
    if (wv == 0 && k < P.n_trows) {
        A acc = A(0);
#pragma unroll
        for (int w = 0; w < kBlockWaves; w++) acc += lds[w * 64 + lane];
        ((A *)P.y)[(int64_t)P.tile_orow[k] * P.ldy] = acc;
    }
}

template <int VD, class A, int K, int T, int R, bool LONG, int LP>
__device__ __forceinline__ void spmv_unit(const SpmvParams &P, int32_t u, int lane, int wv, A (*red)[K], A *lbuf) {
    constexpr bool kLdsLong = LONG && K == 1;
    // combine units of the column-tiled rows: one right-hand side, the
    // default load policy, partial sums in the vector type (FP64 vectors
    // only with F64 storage); they use the workgroup's LDS buffer (lbuf of
    // wavefront 0 starts it)
    if constexpr (kLdsLong && LP == 0 && (sizeof(A) == 4 || VD == RGCSR_F64)) {
        if (u < P.n_comb_units) {
            tile_combine_unit<A>(P, u, lane, wv, lbuf - wv * (kWaveRowMax + 1));
            return;
        }
        u -= P.n_comb_units;
    }
    if (LONG && u < P.n_block_items) {
        spmv_block_item<VD, A, K, LP>(P, u, red);
        return;
    }
    const int32_t w = __builtin_amdgcn_readfirstlane((u - (LONG ? P.n_block_items : 0)) * kBlockWaves + wv);
    if (w >= P.n_wave_items) return;
    if (LONG && w < P.n_wave_long) {
        if constexpr (kLdsLong) spmv_wave_long_lds<VD, A, LP>(P, w, lane, lbuf);
        else spmv_wave_long<VD, A, K, LP>(P, w, lane);
    } else {
        spmv_short<VD, A, K, T, R, LP>(P, w - (LONG ? P.n_wave_long : 0), lane);
    }
}

// A single right-hand side runs one unit per workgroup (the grid covers every
// unit, so nothing stays live across units); several right-hand sides may run
// a persistent grid that strides over the units.  Four columns in runs of rows
// are held to four wavefronts per SIMD, which they miss by two registers
// otherwise (300,000 rows of 4 nonzeros, sorted: 10.5 -> 9.6 us).
template <int VD, class A, int K, int T, int R, bool LONG, int LP>
__global__ __launch_bounds__(kBlockThreads, K == 4 && R == 0 && !LONG ? 4 : 1) void rgcsr_spmv_k(SpmvParams P) {
    constexpr bool kLdsLong = LONG && K == 1;
    __shared__ A red[kBlockWaves][K];
    __shared__ A lbuf[kLdsLong ? kBlockWaves : 1][kLdsLong ? kWaveRowMax + 1 : 1];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int nwg = gridDim.x;
    // column panels: the host's table (unit_map) places each panel's units
    // on one XCD; -1 entries run nothing.  With one right-hand side the grid
    // is the table's length.
    if constexpr (K == 1) {
        int32_t u = first_unit(blockIdx.x, nwg, P.n_long_units);
        if (P.unit_map) u = ldc(P.unit_map, blockIdx.x);
        if (u >= 0 && u < P.total_units)
            spmv_unit<VD, A, K, T, R, LONG, LP>(P, u, lane, wv, red, lbuf[kLdsLong ? wv : 0]);
    } else {
        int32_t u = first_unit(blockIdx.x, nwg, P.n_long_units);
        for (int32_t j = blockIdx.x; P.unit_map ? j < P.n_map : u < P.total_units; j += nwg, u += nwg) {
            const int32_t v = P.unit_map ? ldc(P.unit_map, j) : u;
            if (v >= 0) spmv_unit<VD, A, K, T, R, LONG, LP>(P, v, lane, wv, red, lbuf[0]);
        }
    }
}

// Column panels: each split row crow[i] adds its pieces' sums yv[vidx[s]]
// for s in [cptr[i], cptr[i + 1]), in panel order.  The sums are stored by
// piece, in panel order, so each XCD writes whole lines of its own.
template <class A, int K>
__global__ __launch_bounds__(256) void panel_combine_k(const int32_t *crow, const int32_t *cptr, int64_t n,
                                                       const int32_t *vidx, const A *yv, A *Y, int64_t ldy) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t r = crow[i];
    const int32_t s0 = cptr[i], m = cptr[i + 1] - s0;  // pieces of this row
    A acc[K];
#pragma unroll
    for (int k = 0; k < K; k++) acc[k] = A(0);
    // a split row has about one piece per panel: eight pieces per pass, their
    // indices and then their sums loaded together (steps past the row's
    // pieces re-read its first piece, which exists whenever the loop runs),
    // added in panel order
    constexpr int U = 8;
    for (int32_t b = 0; b < m; b += U) {
        int32_t id[U];
#pragma unroll
        for (int u = 0; u < U; u++) id[u] = vidx[s0 + (b + u < m ? b + u : 0)];
        A v[U][K];
#pragma unroll
        for (int u = 0; u < U; u++) load_row<A, K>(yv + (int64_t)id[u] * K, v[u]);
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int k = 0; k < K; k++) acc[k] = b + u < m ? acc[k] + v[u][k] : acc[k];
    }
    store_row<A, K>(Y + r * ldy, acc);
}

// Rows split over several block items: add the chunk partial sums in order.
template <class A, int K>
__global__ __launch_bounds__(256) void combine_k(const LongItem *items, int32_t n, const int32_t *long_row,
                                                 const A *partial, A *Y, int64_t ldy, void *pan_y, int64_t pan_ld) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const LongItem it = items[i];
    A tot[K];
#pragma unroll
    for (int k = 0; k < K; k++) tot[k] = A(0);
    for (int c = 0; c < it.c; c++)
#pragma unroll
        for (int k = 0; k < K; k++) tot[k] += partial[((int64_t)it.d + c) * K + k];
    store_row<A, K>(out_row<K>(Y, ldy, pan_y, pan_ld, long_row[it.a]), tot);
}

// ---------------------------------------------------------------------------
// Value update: slots <- convert(theta[csr index]) for A, then A^T by map
// ---------------------------------------------------------------------------
template <int VD, class SRC>
__device__ __forceinline__ typename Val<VD>::S to_store(SRC v) {
    if constexpr (VD == RGCSR_F64) return (double)v;
    else if constexpr (VD == RGCSR_F32) return (float)v;
    else if constexpr (VD == RGCSR_F16) return f32_to_f16_rne((float)v);
    else return f32_to_bf16_rne((float)v);
}

// Value update over the SpMV work split (workgroup chunks of the longest
// rows, wavefront items of long rows, then row groups one row per lane); each
// lane loads up to U source values before it stores them.
// tdst (nullable): position of each element in the column-tiled copy of the
// long rows, -1 when its row is not tiled; tv: the tiled values.
template <int VD, class SRC, int U>
__device__ __forceinline__ void copy_elems(const SRC *src, typename Val<VD>::S *dst, int32_t o, int32_t e,
                                           int32_t stride, const int32_t *tdst = nullptr,
                                           typename Val<VD>::S *tv = nullptr) {
    for (int32_t o0 = o; o0 < e; o0 += stride * U) {
        SRC t[U];
        int32_t d[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int32_t i = o0 + u * stride < e ? o0 + u * stride : o;
            t[u] = src[i];
            d[u] = tdst ? tdst[i] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (o0 + u * stride < e) {
                const typename Val<VD>::S v = to_store<VD>(t[u]);
                dst[o0 + u * stride] = v;
                if (d[u] >= 0) tv[d[u]] = v;
            }
    }
}

template <int VD, class SRC, int T>
__global__ __launch_bounds__(256) void setval_k(SpmvParams P, const SRC *theta, const int64_t *row_ptr) {
    using S = typename Val<VD>::S;
    const int lane = threadIdx.x & 63;
    S *lv = (S *)P.long_val;
    const int32_t u = blockIdx.x;
    if (u < P.n_block_items) {
        const LongItem it = ldc(P.block_work, u);
        const int64_t li = it.a;
        const int64_t lb = ldc(P.long_ptr, li);
        const int64_t beg = lb + (int64_t)it.b * kBlockChunk;
        const int32_t n = (int32_t)min(ldc(P.long_ptr, li + 1) - beg, kBlockChunk);
        const int64_t row = ldc(P.long_row, li);
        copy_elems<VD, SRC, 16>(theta + (row_ptr[row] + (beg - lb)), lv + beg, (int32_t)threadIdx.x, n,
                                kBlockThreads, P.tile_dst ? P.tile_dst + beg : nullptr, (S *)P.tile_vals);
        return;
    }
    const int32_t w = __builtin_amdgcn_readfirstlane((u - P.n_block_items) * 4 + (int)(threadIdx.x >> 6));
    if (w < P.n_wave_long) {
        const LongItem it = ldc(P.wave_work, w);
        const int TL = it.c;
        const int sh = 31 - __builtin_clz(TL);
        const int r = lane >> sh, q = lane & (TL - 1);
        if (r >= it.b) return;
        const int64_t li = (int64_t)it.a + r;
        const int64_t beg = P.long_ptr[li];
        const int32_t n = (int32_t)(P.long_ptr[li + 1] - beg);
        const int64_t row = P.long_row[li];
        copy_elems<VD, SRC, kWaveUnroll>(theta + row_ptr[row], lv + beg, q, n, TL,
                                         P.tile_dst ? P.tile_dst + beg : nullptr, (S *)P.tile_vals);
        return;
    }
    const int32_t ws = w - P.n_wave_long;
    if (ws >= P.total_waves - P.n_long_waves) return;
    const LaneRow L = lane_row<T>(P, ws, lane);
    if (!L.ok || L.len <= L.q) return;
    S *sv = (S *)const_cast<void *>(P.slot_val);
    const int64_t row = P.perm ? (int64_t)P.short_row[L.i] : L.i;
    const SRC *src = theta + row_ptr[row] + L.q;
    const int32_t nl = (L.len - L.q + T - 1) / T;
    constexpr int US = 8;
    for (int32_t c0 = 0; c0 < nl; c0 += US) {
        SRC t[US];
#pragma unroll
        for (int u = 0; u < US; u++) t[u] = src[(int64_t)(c0 + u < nl ? c0 + u : 0) * T];
#pragma unroll
        for (int u = 0; u < US; u++)
            if (c0 + u < nl) sv[L.base + (int64_t)(c0 + u) * L.stride] = to_store<VD>(t[u]);
    }
}

template <int VD, class SRC>
__global__ __launch_bounds__(256) void gather_map_k(int64_t n, const int32_t *map, const SRC *theta, void *dst) {
    using S = typename Val<VD>::S;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int32_t m = map[i];
    ((S *)dst)[i] = m >= 0 ? to_store<VD>(theta[m]) : S(0);
}

// ---------------------------------------------------------------------------
// Backward: dvals[k] = dy[row(k)] * x[col(k)]; optionally dx += v * dy (atomic)
//
// The work is split as in the SpMV (workgroup chunks of the longest rows,
// wavefront items of long rows, then row groups), and every lane issues the
// column (and value) loads of up to U elements before their x gathers, so a
// row costs a few dependent memory levels, not one per element.  Each output
// is a single product, so the order of the work does not change dvals.
// ---------------------------------------------------------------------------
template <int VD, class A, bool DVALS, bool ATOMIC_DX, int U>
__device__ __forceinline__ void grad_elems(const typename Val<VD>::S *vb, const int32_t *cb, const A *X, A d,
                                           A *dv, A *dx, int32_t o, int32_t e, int32_t stride) {
    using V = Val<VD>;
    using S = typename V::S;
    for (int32_t o0 = o; o0 < e; o0 += stride * U) {
        int32_t ci[U];
        S v[U];
        A xv[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int32_t oo = o0 + u * stride < e ? o0 + u * stride : o;
            ci[u] = cb[oo];
            if constexpr (ATOMIC_DX) v[u] = vb[oo];
        }
        if constexpr (DVALS) {
#pragma unroll
            for (int u = 0; u < U; u++) xv[u] = X[ci[u]];
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            if (o0 + u * stride < e) {
                if constexpr (DVALS) dv[o0 + u * stride] = d * xv[u];
                if constexpr (ATOMIC_DX) atomicAdd(dx + ci[u], V::template cvt<A>(v[u]) * d);
            }
        }
    }
}

template <int VD, class A, int T, bool DVALS, bool ATOMIC_DX>
__global__ __launch_bounds__(256) void grad_k(SpmvParams P, const A *dy, A *dvals, A *dx, const int64_t *row_ptr) {
    using V = Val<VD>;
    using S = typename V::S;
    const int lane = threadIdx.x & 63;
    const A *X = (const A *)P.x;
    const S *lv = (const S *)P.long_val;
    const int32_t u = blockIdx.x;
    if (u < P.n_block_items) {
        // a chunk of at most kBlockChunk nonzeros of one long row
        const LongItem it = ldc(P.block_work, u);
        const int64_t li = it.a;
        const int64_t lb = ldc(P.long_ptr, li);
        const int64_t beg = lb + (int64_t)it.b * kBlockChunk;
        const int32_t n = (int32_t)min(ldc(P.long_ptr, li + 1) - beg, kBlockChunk);
        const int64_t row = ldc(P.long_row, li);
        const A d = dy[row];
        A *dv = DVALS ? dvals + (row_ptr[row] + (beg - lb)) : nullptr;
        grad_elems<VD, A, DVALS, ATOMIC_DX, 16>(lv + beg, P.long_col + beg, X, d, dv, dx, (int32_t)threadIdx.x, n,
                                                 kBlockThreads);
        return;
    }
    const int32_t w = __builtin_amdgcn_readfirstlane((u - P.n_block_items) * 4 + (int)(threadIdx.x >> 6));
    if (w < P.n_wave_long) {
        // consecutive long rows of at most kWaveRowMax nonzeros, it.c lanes each
        const LongItem it = ldc(P.wave_work, w);
        const int TL = it.c;
        const int sh = 31 - __builtin_clz(TL);
        const int r = lane >> sh, q = lane & (TL - 1);
        if (r >= it.b) return;
        const int64_t li = (int64_t)it.a + r;
        const int64_t beg = P.long_ptr[li];
        const int32_t n = (int32_t)(P.long_ptr[li + 1] - beg);
        const int64_t row = P.long_row[li];
        const A d = dy[row];
        A *dv = DVALS ? dvals + row_ptr[row] : nullptr;
        grad_elems<VD, A, DVALS, ATOMIC_DX, kWaveUnroll>(lv + beg, P.long_col + beg, X, d, dv, dx, q, n, TL);
        return;
    }
    const int32_t ws = w - P.n_wave_long;
    if (ws >= P.total_waves - P.n_long_waves) return;
    const LaneRow L = lane_row<T>(P, ws, lane);
    if (!L.ok || L.len <= L.q) return;
    const S *sv = (const S *)P.slot_val;
    const int64_t row = P.perm ? (int64_t)P.short_row[L.i] : L.i;
    const A d = dy[row];
    const int32_t nl = (L.len - L.q + T - 1) / T;  // this lane's elements
    constexpr int US = 8;
    for (int32_t c0 = 0; c0 < nl; c0 += US) {
        int32_t ci[US];
        S v[US];
        A xv[US];
#pragma unroll
        for (int u = 0; u < US; u++) {
            const int64_t s = L.base + (int64_t)(c0 + u < nl ? c0 + u : 0) * L.stride;
            ci[u] = P.slot_col[s];
            if constexpr (ATOMIC_DX) v[u] = sv[s];
        }
        if constexpr (DVALS) {
#pragma unroll
            for (int u = 0; u < US; u++) xv[u] = X[ci[u]];
        }
        const int64_t k0 = DVALS ? row_ptr[row] + L.q : 0;
#pragma unroll
        for (int u = 0; u < US; u++) {
            if (c0 + u < nl) {
                if constexpr (DVALS) dvals[k0 + (int64_t)(c0 + u) * T] = d * xv[u];
                if constexpr (ATOMIC_DX) atomicAdd(dx + ci[u], V::template cvt<A>(v[u]) * d);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Hybrid ELL + COO
// ---------------------------------------------------------------------------
template <int VD, class A>
__global__ __launch_bounds__(256) void hyb_ell_k(int64_t n, int64_t n_pad, int32_t K1, const int32_t *ecol,
                                                 const void *evals, const A *x, A *y) {
    using V = Val<VD>;
    using S = typename V::S;
    const int64_t i = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const S *ev = (const S *)evals;
    A acc = A(0);
    constexpr int U = 8;
    for (int j0 = 0; j0 < K1; j0 += U) {
        S v[U];
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            if (j0 + u < K1) {
                const int64_t e = (int64_t)(j0 + u) * n_pad + i;
                c[u] = ldnt(ecol + e);
                v[u] = ldnt(ev + e);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (j0 + u < K1 && c[u] >= 0) acc = fmaA(V::template cvt<A>(v[u]), x[c[u]], acc);
    }
    y[i] = acc;
}

// Each wavefront owns 512 consecutive COO entries, 8 per lane (rows are
// non-decreasing).  A lane sums its runs of equal row.  Runs strictly inside
// a lane belong to no other lane and are added with a plain read-modify-write.
// The lane's last run is carried across following lanes with a segmented
// scan, so a row spanning many lanes costs one addition; that addition, and
// the first run of lane 0, are atomic because they may meet another
// wavefront's entries of the same row.
template <int VD, class A>
__global__ __launch_bounds__(256) void hyb_coo_k(int64_t m, const int32_t *crow, const int32_t *ccol,
                                                 const void *cvals, const A *x, A *y) {
    using V = Val<VD>;
    using S = typename V::S;
    const S *cv = (const S *)cvals;
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6);
    const int64_t base = wave * 512;
    if (base >= m) return;
    const int64_t e0 = base + (int64_t)lane * 8;
    S v[8];
    int32_t r[8], c[8];
    if (e0 + 8 <= m) {
        // a lane's 8 consecutive entries as 16-byte loads (the arrays are
        // 256-byte aligned and e0 is a multiple of 8), so each load
        // instruction of the wavefront covers whole cache lines once
        i32x4 rv[2], cw[2];
        i32x4 vv[(8 * sizeof(S)) / 16];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            rv[h] = ldnt(reinterpret_cast<const i32x4 *>(crow + e0) + h);
            cw[h] = ldnt(reinterpret_cast<const i32x4 *>(ccol + e0) + h);
        }
#pragma unroll
        for (int h = 0; h < (int)((8 * sizeof(S)) / 16); h++) vv[h] = ldnt(reinterpret_cast<const i32x4 *>(cv + e0) + h);
        __builtin_memcpy(r, rv, sizeof(r));
        __builtin_memcpy(c, cw, sizeof(c));
        __builtin_memcpy(v, vv, sizeof(v));
    } else {
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int64_t e = e0 + u;
            r[u] = -1;
            c[u] = 0;
            v[u] = S(0);
            if (e < m) {
                r[u] = ldnt(crow + e);
                c[u] = ldnt(ccol + e);
                v[u] = ldnt(cv + e);
            }
        }
    }
    A p[8];
#pragma unroll
    for (int u = 0; u < 8; u++) p[u] = r[u] >= 0 ? V::template cvt<A>(v[u]) * x[c[u]] : A(0);
    // lane-local runs: head run, interior runs (flushed here), tail run
    const int32_t head = r[0];
    int32_t cur = r[0];
    A run = p[0], head_sum = A(0);
    bool single = true;
#pragma unroll
    for (int u = 1; u < 8; u++) {
        if (r[u] >= 0 && r[u] != cur) {
            if (single) head_sum = run;   // the lane's first run
            else y[cur] += run;           // interior run: no other lane has this row
            single = false;
            cur = r[u];
            run = A(0);
        }
        if (r[u] >= 0) run += p[u];
    }
    const int32_t tail = cur;  // -1 for a lane without entries
    // Segmented inclusive scan of tail runs over the lanes.  A lane starts a new
    // segment unless it is a single-run lane continuing the previous lane's tail.
    const int32_t tail_prev = __shfl_up(tail, 1);
    const bool have_prev = lane > 0 && head >= 0 && tail_prev == head;
    int flag = (single && have_prev) ? 0 : 1;
    A carry = run;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const A v_up = __shfl_up(carry, off);
        const int f_up = __shfl_up(flag, off);
        if (lane >= off && !flag) {
            carry += v_up;
            flag = f_up;
        }
    }
    const A carry_prev = __shfl_up(carry, 1);
    const int32_t head_next = __shfl_down(head, 1);
    if (!single && head >= 0) {
        // the head run ends inside this lane; it includes the carried run of
        // the previous lanes when they end on the same row
        const A tot = head_sum + (have_prev ? carry_prev : A(0));
        if (lane == 0 || have_prev) atomicAdd(y + head, tot);
        else y[head] += tot;
    }
    // the tail run ends here unless the next lane starts with the same row
    if (tail >= 0 && (lane == 63 || head_next != tail)) atomicAdd(y + tail, carry);
}

// ---------------------------------------------------------------------------
// Conjugate-gradient vector kernels of a solve's start and end (those of an
// iteration: cg.hip).  Dot products accumulate in FP64 into a fixed number of
// block partials and are finished by one block, so every reduction has a fixed
// order (bit-reproducible runs).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double block_sum(double v, double *sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    const int wv = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[wv] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); i++) t += sh[i];
    return t;
}

// Grid-stride loop over [0, n) taking four independent elements per pass, so
// each lane has four loads in flight; f(i) is applied in a fixed order for a
// fixed grid, which keeps the partial sums deterministic.
template <class F> __device__ __forceinline__ void grid_loop4(int64_t n, F f) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n; i += 4 * stride) {
        f(i);
        f(i + stride);
        f(i + 2 * stride);
        f(i + 3 * stride);
    }
    for (; i < n; i += stride) f(i);
}

template <class TA, class TB>
__global__ __launch_bounds__(256) void dot_partial_k(int64_t n, const TA *a, const TB *b, double *part) {
    __shared__ double sh[4];
    double acc = 0.0;
    grid_loop4(n, [&](int64_t i) { acc += (double)a[i] * (double)b[i]; });
    const double t = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// One block: sum the partials, then apply `mode` to the scalar slots.
__global__ __launch_bounds__(256) void cg_scalar_k(const double *part, int nb, double *scal, int mode) {
    __shared__ double sh[4];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nb; i += 256) acc += part[i];
    const double s = block_sum(acc, sh);
    if (threadIdx.x != 0) return;
    switch (mode) {
    case kScalRRInit: scal[kRR] = s; scal[kRR0] = s; break;
    default: scal[kOut] = s; break;
    }
}

// r64 = b - q64 ; partial sums of r64.r64
__global__ __launch_bounds__(256) void resid_k(int64_t n, const double *b, const double *q, double *r, double *part) {
    __shared__ double sh[4];
    double acc = 0.0;
    grid_loop4(n, [&](int64_t i) {
        const double ri = b[i] - q[i];
        r[i] = ri;
        acc += ri * ri;
    });
    const double t = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// r32 = r64 * s ; d32 = 0 ; p32 = r32 ; partial sums of r32.r32
__global__ __launch_bounds__(256) void refine_start_k(int64_t n, const double *r64, double s, float *r, float *d,
                                                      float *p, double *part) {
    __shared__ double sh[4];
    double acc = 0.0;
    grid_loop4(n, [&](int64_t i) {
        const float ri = (float)(r64[i] * s);
        r[i] = ri;
        p[i] = ri;
        d[i] = 0.0f;
        acc += (double)ri * (double)ri;
    });
    const double t = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// x64 += d32 * inv_s
__global__ __launch_bounds__(256) void refine_add_k(int64_t n, double *x, const float *d, double inv_s) {
    grid_loop4(n, [&](int64_t i) { x[i] += (double)d[i] * inv_s; });
}

template <class VT>
__global__ __launch_bounds__(256) void copy_k(int64_t n, const VT *a, VT *b) {
    grid_loop4(n, [&](int64_t i) { b[i] = a[i]; });
}

template <class VT>
__global__ __launch_bounds__(256) void fill_k(int64_t n, VT *a, VT v) {
    grid_loop4(n, [&](int64_t i) { a[i] = v; });
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static hipError_t check_launch() { return hipGetLastError(); }

template <int VD, class A, int K, int T, int R, int LP = 0>
static hipError_t launch_spmv_t(const SpmvParams &P, int nwg, hipStream_t st) {
    if (P.n_block_items + P.n_wave_long + P.n_comb_units > 0)
        hipLaunchKernelGGL((rgcsr_spmv_k<VD, A, K, T, R, true, LP>), dim3(nwg), dim3(kBlockThreads), 0, st, P);
    else
        hipLaunchKernelGGL((rgcsr_spmv_k<VD, A, K, T, R, false, LP>), dim3(nwg), dim3(kBlockThreads), 0, st, P);
    return check_launch();
}

// Load policies other than the default: FP32 values and vectors, one
// right-hand side, one lane per row.
template <int LP>
static hipError_t launch_spmv_lp(const SpmvParams &P, int R, int nwg, hipStream_t st) {
    switch (R) {
    case 0: return launch_spmv_t<RGCSR_F32, float, 1, 1, 0, LP>(P, nwg, st);
    case 1: return launch_spmv_t<RGCSR_F32, float, 1, 1, 1, LP>(P, nwg, st);
    case 2: return launch_spmv_t<RGCSR_F32, float, 1, 1, 2, LP>(P, nwg, st);
    case 4: return launch_spmv_t<RGCSR_F32, float, 1, 1, 4, LP>(P, nwg, st);
    case 8: return launch_spmv_t<RGCSR_F32, float, 1, 1, 8, LP>(P, nwg, st);
    }
    return hipErrorInvalidValue;
}

// One lane per row (T = 1) takes R in {1, 2, 4, 8} rows per lane, or R = 0
// for rows per lane chosen per wavefront; T > 1 and several right-hand sides
// take one row per lane.
template <int VD, class A>
static hipError_t launch_spmv_vk(const SpmvParams &P, int T, int K, int R, int nwg, hipStream_t st) {
    if (K == 1) {
        if (T == 1) {
            switch (R) {
            case 0: return launch_spmv_t<VD, A, 1, 1, 0>(P, nwg, st);
            case 1: return launch_spmv_t<VD, A, 1, 1, 1>(P, nwg, st);
            case 2: return launch_spmv_t<VD, A, 1, 1, 2>(P, nwg, st);
            case 4: return launch_spmv_t<VD, A, 1, 1, 4>(P, nwg, st);
            case 8: return launch_spmv_t<VD, A, 1, 1, 8>(P, nwg, st);
            }
            return hipErrorInvalidValue;
        }
        if (R != 1) return hipErrorInvalidValue;
        switch (T) {
        case 2: return launch_spmv_t<VD, A, 1, 2, 1>(P, nwg, st);
        case 4: return launch_spmv_t<VD, A, 1, 4, 1>(P, nwg, st);
        case 8: return launch_spmv_t<VD, A, 1, 8, 1>(P, nwg, st);
        }
        return hipErrorInvalidValue;
    }
    // several right-hand sides (on a column-panel copy; otherwise spmm.h) of at
    // most 16 bytes per row: one row per lane, or the runs of rows per lane
    // (R = 0); wider ones one row per lane
    if (T != 1 || (R != 1 && (R != 0 || K * (int)sizeof(A) > kRunsRowBytes))) return hipErrorInvalidValue;
    switch (K) {
    case 2: return R ? launch_spmv_t<VD, A, 2, 1, 1>(P, nwg, st) : launch_spmv_t<VD, A, 2, 1, 0>(P, nwg, st);
    case 4:
        if constexpr (sizeof(A) == 4) {
            if (!R) return launch_spmv_t<VD, A, 4, 1, 0>(P, nwg, st);
        }
        return launch_spmv_t<VD, A, 4, 1, 1>(P, nwg, st);
    case 8:
        if constexpr (sizeof(A) == 4) return launch_spmv_t<VD, A, 8, 1, 1>(P, nwg, st);
    }
    return hipErrorInvalidValue;
}

template <class A, int K>
static hipError_t launch_combine_k(const LongItem *items, int32_t n, const int32_t *long_row, const void *partial,
                                   void *Y, int64_t ldy, void *pan_y, int64_t pan_ld, hipStream_t st) {
    hipLaunchKernelGGL((combine_k<A, K>), dim3((n + 255) / 256), dim3(256), 0, st, items, n, long_row,
                       (const A *)partial, (A *)Y, ldy, pan_y, pan_ld);
    return check_launch();
}

template <class A>
static hipError_t launch_combine_a(const LongItem *items, int32_t n, const int32_t *long_row, const void *partial,
                                   void *Y, int64_t ldy, void *pan_y, int64_t pan_ld, int K, hipStream_t st) {
    switch (K) {
    case 1: return launch_combine_k<A, 1>(items, n, long_row, partial, Y, ldy, pan_y, pan_ld, st);
    case 2: return launch_combine_k<A, 2>(items, n, long_row, partial, Y, ldy, pan_y, pan_ld, st);
    case 4: return launch_combine_k<A, 4>(items, n, long_row, partial, Y, ldy, pan_y, pan_ld, st);
    case 8: return launch_combine_k<A, 8>(items, n, long_row, partial, Y, ldy, pan_y, pan_ld, st);
    }
    return hipErrorInvalidValue;
}

template <class A>
static hipError_t launch_panel_combine_a(const int32_t *crow, const int32_t *cptr, int64_t n, const int32_t *vidx,
                                         const A *yv, A *Y, int64_t ldy, int K, hipStream_t st) {
    const dim3 g((unsigned)((n + 255) / 256)), b(256);
    switch (K) {
    case 1: hipLaunchKernelGGL((panel_combine_k<A, 1>), g, b, 0, st, crow, cptr, n, vidx, yv, Y, ldy); break;
    case 2: hipLaunchKernelGGL((panel_combine_k<A, 2>), g, b, 0, st, crow, cptr, n, vidx, yv, Y, ldy); break;
    case 4: hipLaunchKernelGGL((panel_combine_k<A, 4>), g, b, 0, st, crow, cptr, n, vidx, yv, Y, ldy); break;
    case 8: hipLaunchKernelGGL((panel_combine_k<A, 8>), g, b, 0, st, crow, cptr, n, vidx, yv, Y, ldy); break;
    default: return hipErrorInvalidValue;
    }
    return check_launch();
}

hipError_t launch_panel_combine(const int32_t *crow, const int32_t *cptr, int64_t n, const int32_t *vidx,
                                const void *yv, void *Y, int64_t ldy, int vec_f64, int K, hipStream_t st) {
    if (n == 0) return hipSuccess;
    if (vec_f64)
        return launch_panel_combine_a<double>(crow, cptr, n, vidx, (const double *)yv, (double *)Y, ldy, K, st);
    return launch_panel_combine_a<float>(crow, cptr, n, vidx, (const float *)yv, (float *)Y, ldy, K, st);
}

hipError_t launch_combine(const LongItem *items, int32_t n, const int32_t *long_row, const void *partial, void *Y,
                          int64_t ldy, void *pan_y, int64_t pan_ld, int vec_f64, int K, hipStream_t st) {
    if (n == 0) return hipSuccess;
    if (vec_f64) return launch_combine_a<double>(items, n, long_row, partial, Y, ldy, pan_y, pan_ld, K, st);
    return launch_combine_a<float>(items, n, long_row, partial, Y, ldy, pan_y, pan_ld, K, st);
}

hipError_t launch_spmv(const SpmvParams &P, int vdt, int vec_f64, int T, int K, int R, int load_policy, int nwg,
                       hipStream_t st) {
    if (load_policy != 0) {
        if (vec_f64 || vdt != RGCSR_F32 || K != 1 || T != 1) return hipErrorNotSupported;
        if (load_policy == 1) return launch_spmv_lp<1>(P, R, nwg, st);
        if (load_policy == 2) return launch_spmv_lp<2>(P, R, nwg, st);
        return hipErrorInvalidValue;
    }
    if (vec_f64) {
        if (vdt == RGCSR_F64) return launch_spmv_vk<RGCSR_F64, double>(P, T, K, R, nwg, st);
        if (vdt == RGCSR_F32) return launch_spmv_vk<RGCSR_F32, double>(P, T, K, R, nwg, st);
    } else {
        if (vdt == RGCSR_F32) return launch_spmv_vk<RGCSR_F32, float>(P, T, K, R, nwg, st);
        if (K == 1 && vdt == RGCSR_F16) return launch_spmv_vk<RGCSR_F16, float>(P, T, 1, R, nwg, st);
        if (K == 1 && vdt == RGCSR_BF16) return launch_spmv_vk<RGCSR_BF16, float>(P, T, 1, R, nwg, st);
    }
    return hipErrorInvalidValue;
}

template <int VD, class SRC>
static hipError_t launch_setval_s(const SpmvParams &P, int T, const SRC *theta, const int64_t *rp, hipStream_t st) {
    const int64_t waves = (int64_t)P.n_wave_long + (P.total_waves - P.n_long_waves);
    const int nwg = (int)(P.n_block_items + (waves + 3) / 4);
    if (nwg == 0) return hipSuccess;
    switch (T) {
    case 1: hipLaunchKernelGGL((setval_k<VD, SRC, 1>), dim3(nwg), dim3(256), 0, st, P, theta, rp); break;
    case 2: hipLaunchKernelGGL((setval_k<VD, SRC, 2>), dim3(nwg), dim3(256), 0, st, P, theta, rp); break;
    case 4: hipLaunchKernelGGL((setval_k<VD, SRC, 4>), dim3(nwg), dim3(256), 0, st, P, theta, rp); break;
    case 8: hipLaunchKernelGGL((setval_k<VD, SRC, 8>), dim3(nwg), dim3(256), 0, st, P, theta, rp); break;
    default: return hipErrorInvalidValue;
    }
    return check_launch();
}

template <class SRC>
static hipError_t launch_setval_src(const SpmvParams &P, int vdt, int T, const SRC *theta, const int64_t *rp,
                                    hipStream_t st) {
    switch (vdt) {
    case RGCSR_F64: return launch_setval_s<RGCSR_F64, SRC>(P, T, theta, rp, st);
    case RGCSR_F32: return launch_setval_s<RGCSR_F32, SRC>(P, T, theta, rp, st);
    case RGCSR_F16: return launch_setval_s<RGCSR_F16, SRC>(P, T, theta, rp, st);
    case RGCSR_BF16: return launch_setval_s<RGCSR_BF16, SRC>(P, T, theta, rp, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_setval(const SpmvParams &P, int vdt, int T, const void *theta, int theta_f64, const int64_t *rp,
                         hipStream_t st) {
    if (theta_f64) return launch_setval_src<double>(P, vdt, T, (const double *)theta, rp, st);
    return launch_setval_src<float>(P, vdt, T, (const float *)theta, rp, st);
}

template <class SRC>
static hipError_t launch_gather_src(int64_t n, int vdt, const int32_t *map, const SRC *theta, void *dst, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const int nwg = (int)((n + 255) / 256);
    switch (vdt) {
    case RGCSR_F64: hipLaunchKernelGGL((gather_map_k<RGCSR_F64, SRC>), dim3(nwg), dim3(256), 0, st, n, map, theta, dst); break;
    case RGCSR_F32: hipLaunchKernelGGL((gather_map_k<RGCSR_F32, SRC>), dim3(nwg), dim3(256), 0, st, n, map, theta, dst); break;
    case RGCSR_F16: hipLaunchKernelGGL((gather_map_k<RGCSR_F16, SRC>), dim3(nwg), dim3(256), 0, st, n, map, theta, dst); break;
    case RGCSR_BF16: hipLaunchKernelGGL((gather_map_k<RGCSR_BF16, SRC>), dim3(nwg), dim3(256), 0, st, n, map, theta, dst); break;
    default: return hipErrorInvalidValue;
    }
    return check_launch();
}

hipError_t launch_gather_map(int64_t n, int vdt, const int32_t *map, const void *theta, int theta_f64, void *dst,
                             hipStream_t st) {
    if (theta_f64) return launch_gather_src<double>(n, vdt, map, (const double *)theta, dst, st);
    return launch_gather_src<float>(n, vdt, map, (const float *)theta, dst, st);
}

template <int VD, class A, int T>
static hipError_t launch_grad_t(const SpmvParams &P, const A *dy, A *dvals, A *dx, const int64_t *rp, bool want_dvals,
                                bool atomic_dx, hipStream_t st) {
    // block items, then wavefront items (long-row items, then the row groups
    // one row per lane)
    const int64_t waves = (int64_t)P.n_wave_long + (P.total_waves - P.n_long_waves);
    const int nwg = (int)(P.n_block_items + (waves + 3) / 4);
    if (nwg == 0) return hipSuccess;
    if (want_dvals && atomic_dx)
        hipLaunchKernelGGL((grad_k<VD, A, T, true, true>), dim3(nwg), dim3(256), 0, st, P, dy, dvals, dx, rp);
    else if (want_dvals)
        hipLaunchKernelGGL((grad_k<VD, A, T, true, false>), dim3(nwg), dim3(256), 0, st, P, dy, dvals, dx, rp);
    else if (atomic_dx)
        hipLaunchKernelGGL((grad_k<VD, A, T, false, true>), dim3(nwg), dim3(256), 0, st, P, dy, dvals, dx, rp);
    return check_launch();
}

template <int VD, class A>
static hipError_t launch_grad_v(const SpmvParams &P, int T, const A *dy, A *dvals, A *dx, const int64_t *rp,
                                bool want_dvals, bool atomic_dx, hipStream_t st) {
    switch (T) {
    case 1: return launch_grad_t<VD, A, 1>(P, dy, dvals, dx, rp, want_dvals, atomic_dx, st);
    case 2: return launch_grad_t<VD, A, 2>(P, dy, dvals, dx, rp, want_dvals, atomic_dx, st);
    case 4: return launch_grad_t<VD, A, 4>(P, dy, dvals, dx, rp, want_dvals, atomic_dx, st);
    case 8: return launch_grad_t<VD, A, 8>(P, dy, dvals, dx, rp, want_dvals, atomic_dx, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_grad(const SpmvParams &P, int vdt, int vec_f64, int T, const void *dy, void *dvals, void *dx,
                       const int64_t *rp, bool want_dvals, bool atomic_dx, hipStream_t st) {
    if (vec_f64) {
        if (vdt == RGCSR_F64)
            return launch_grad_v<RGCSR_F64, double>(P, T, (const double *)dy, (double *)dvals, (double *)dx, rp,
                                                    want_dvals, atomic_dx, st);
        if (vdt == RGCSR_F32)
            return launch_grad_v<RGCSR_F32, double>(P, T, (const double *)dy, (double *)dvals, (double *)dx, rp,
                                                    want_dvals, atomic_dx, st);
        return hipErrorInvalidValue;
    }
    switch (vdt) {
    case RGCSR_F32:
        return launch_grad_v<RGCSR_F32, float>(P, T, (const float *)dy, (float *)dvals, (float *)dx, rp, want_dvals,
                                               atomic_dx, st);
    case RGCSR_F16:
        return launch_grad_v<RGCSR_F16, float>(P, T, (const float *)dy, (float *)dvals, (float *)dx, rp, want_dvals,
                                               atomic_dx, st);
    case RGCSR_BF16:
        return launch_grad_v<RGCSR_BF16, float>(P, T, (const float *)dy, (float *)dvals, (float *)dx, rp, want_dvals,
                                                atomic_dx, st);
    }
    return hipErrorInvalidValue;
}

template <int VD, class A>
static hipError_t launch_hyb_v(const HybParams &H, const A *x, A *y, hipStream_t st) {
    const int nwg_e = (int)((H.n + 255) / 256);
    if (nwg_e > 0)
        hipLaunchKernelGGL((hyb_ell_k<VD, A>), dim3(nwg_e), dim3(256), 0, st, H.n, H.n_pad, H.K1, H.ell_col,
                           H.ell_val, x, y);
    hipError_t e = check_launch();
    if (e != hipSuccess) return e;
    if (H.m > 0) {
        const int64_t waves = (H.m + 511) / 512;
        const int nwg_c = (int)((waves + 3) / 4);
        hipLaunchKernelGGL((hyb_coo_k<VD, A>), dim3(nwg_c), dim3(256), 0, st, H.m, H.coo_row, H.coo_col,
                           H.coo_val, x, y);
        e = check_launch();
    }
    return e;
}

hipError_t launch_hyb(const HybParams &H, int vdt, int vec_f64, const void *x, void *y, hipStream_t st) {
    if (vec_f64) {
        if (vdt == RGCSR_F64) return launch_hyb_v<RGCSR_F64, double>(H, (const double *)x, (double *)y, st);
        if (vdt == RGCSR_F32) return launch_hyb_v<RGCSR_F32, double>(H, (const double *)x, (double *)y, st);
        return hipErrorInvalidValue;
    }
    switch (vdt) {
    case RGCSR_F32: return launch_hyb_v<RGCSR_F32, float>(H, (const float *)x, (float *)y, st);
    case RGCSR_F16: return launch_hyb_v<RGCSR_F16, float>(H, (const float *)x, (float *)y, st);
    case RGCSR_BF16: return launch_hyb_v<RGCSR_BF16, float>(H, (const float *)x, (float *)y, st);
    }
    return hipErrorInvalidValue;
}

// CG helpers ---------------------------------------------------------------
hipError_t launch_dot(int64_t n, const double *a, const double *b, double *part, int nb, hipStream_t st) {
    hipLaunchKernelGGL((dot_partial_k<double, double>), dim3(nb), dim3(256), 0, st, n, a, b, part);
    return check_launch();
}

hipError_t launch_scalar(const double *part, int nb, double *scal, int mode, hipStream_t st) {
    hipLaunchKernelGGL(cg_scalar_k, dim3(1), dim3(256), 0, st, part, nb, scal, mode);
    return check_launch();
}

hipError_t launch_resid(int64_t n, const double *b, const double *q, double *r, double *part, int nb, hipStream_t st) {
    hipLaunchKernelGGL(resid_k, dim3(nb), dim3(256), 0, st, n, b, q, r, part);
    return check_launch();
}

hipError_t launch_refine_start(int64_t n, const double *r64, double s, float *r, float *d, float *p, double *part,
                               int nb, hipStream_t st) {
    hipLaunchKernelGGL(refine_start_k, dim3(nb), dim3(256), 0, st, n, r64, s, r, d, p, part);
    return check_launch();
}

hipError_t launch_refine_add(int64_t n, double *x, const float *d, double inv_s, int nb, hipStream_t st) {
    hipLaunchKernelGGL(refine_add_k, dim3(nb), dim3(256), 0, st, n, x, d, inv_s);
    return check_launch();
}

hipError_t launch_copy(int64_t n, const void *a, void *b, int f64, int nb, hipStream_t st) {
    if (f64)
        hipLaunchKernelGGL((copy_k<double>), dim3(nb), dim3(256), 0, st, n, (const double *)a, (double *)b);
    else
        hipLaunchKernelGGL((copy_k<float>), dim3(nb), dim3(256), 0, st, n, (const float *)a, (float *)b);
    return check_launch();
}

// Streaming read of n 16-byte words with the matrix streams' nontemporal
// loads; the sum is stored only in a case no data reaches in practice, which
// keeps every load live.
__global__ __launch_bounds__(256) void stream_read_k(const i32x4 *a, int64_t n, int32_t *sink) {
    i32x4 acc = {0, 0, 0, 0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        acc ^= __builtin_nontemporal_load(a + i);
    const int32_t v = acc.x ^ acc.y ^ acc.z ^ acc.w;
    if (v == 0x5bd1e995) sink[0] = v;
}

// Gather floor: the (column, value) stream of a matrix in CSR order with one
// x gather per entry and nothing else (no rows, no reduction across lanes):
// lane l of the grid takes entries l, l + S, ..., l + 7S (S = grid size) and
// writes one partial sum.  Its time bounds what any SpMV over the same entries
// can reach when x gathers dominate.
__global__ __launch_bounds__(256) void gather_floor_k(const int32_t *col, const float *val, int64_t n,
                                                      const float *x, float *out) {
    const int64_t S = (int64_t)gridDim.x * 256;
    const int64_t l = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int32_t c[8];
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) {
        const int64_t e = l + u * S < n ? l + u * S : 0;
        c[u] = __builtin_nontemporal_load(col + e);
        v[u] = __builtin_nontemporal_load(val + e);
    }
    float acc = 0.f;
#pragma unroll
    for (int u = 0; u < 8; u++) {
        const float xv = x[c[u]];
        acc = l + u * S < n ? __builtin_fmaf(v[u], xv, acc) : acc;
    }
    if (l < (n + 7) / 8) out[l] = acc;
}

hipError_t launch_gather_floor(const int32_t *col, const float *val, int64_t n, const float *x, float *out,
                               hipStream_t st) {
    if (n == 0) return hipSuccess;
    const int64_t threads = (n + 7) / 8;
    hipLaunchKernelGGL(gather_floor_k, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, col, val, n, x,
                       out);
    return check_launch();
}

hipError_t launch_stream_read(const void *a, int64_t n16, int32_t *sink, int nb, hipStream_t st) {
    if (n16 == 0) return hipSuccess;
    hipLaunchKernelGGL(stream_read_k, dim3(nb), dim3(256), 0, st, (const i32x4 *)a, n16, sink);
    return check_launch();
}

hipError_t launch_zero(int64_t n, void *a, int esz, int nb, hipStream_t st) {
    if (n == 0) return hipSuccess;
    if (esz == 8)
        hipLaunchKernelGGL((fill_k<double>), dim3(nb), dim3(256), 0, st, n, (double *)a, 0.0);
    else if (esz == 4)
        hipLaunchKernelGGL((fill_k<float>), dim3(nb), dim3(256), 0, st, n, (float *)a, 0.0f);
    else
        return hipErrorInvalidValue;
    return check_launch();
}

// ---------------------------------------------------------------------------
// Workspace of the allocation-free CG: a file-scope device array, so no call
// allocates.  Each device holds its own copy at its own address; host code
// must use that address (from hipGetSymbolAddress with the device current),
// never the array's name, which on the host is only a stand-in.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kNoAllocCgBytes];

hipError_t noalloc_cg_workspace(void **base) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *base = addr[dev];
    return hipSuccess;
}

}  // namespace rg
