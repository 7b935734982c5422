// Device helpers shared by the kernel sources.  Internal; HIP only.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"
#include "kernels.h"

namespace rg {

// Workgroups are dispatched round robin over the 8 XCDs; remap so each XCD
// gets a contiguous range of logical blocks and neighbouring row groups share
// that XCD's L2 (the x windows of banded matrices then hit in L2).
__device__ __forceinline__ int xcd_remap(int bid, int nwg) {
    const int xcd = bid & 7, idx = bid >> 3;
    const int per = nwg >> 3, rem = nwg & 7;
    return (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
}

// First unit of workgroup bid.  Long-row units (the first n_long of the
// list, heaviest first) keep the dispatch order, so consecutive ones land on
// different XCDs and their work is spread evenly over the chip; the row-group
// units after them are remapped so each XCD gets a contiguous range.
__device__ __forceinline__ int first_unit(int bid, int nwg, int n_long) {
    const int h = min((n_long + 7) & ~7, nwg);
    return bid < h ? bid : h + xcd_remap(bid - h, nwg - h);
}

template <int VD> struct Val;
template <> struct Val<RGCSR_F64> {
    using S = double;
    template <class A> __device__ static A cvt(S v) { return (A)v; }
};
template <> struct Val<RGCSR_F32> {
    using S = float;
    template <class A> __device__ static A cvt(S v) { return (A)v; }
};
template <> struct Val<RGCSR_F16> {
    using S = uint16_t;
    template <class A> __device__ static A cvt(S v) { return (A)(float)__builtin_bit_cast(_Float16, v); }
};
template <> struct Val<RGCSR_BF16> {
    using S = uint16_t;
    template <class A> __device__ static A cvt(S v) { return (A)bf16_to_f32(v); }
};

template <class T> __device__ __forceinline__ T ldnt(const T *p) { return __builtin_nontemporal_load(p); }

// Load policy of the SpMV, an ablation of where x and the matrix streams live
// (after the paper's texture-cache study): 0 = value/column streams
// nontemporal, x gathers cached (the default); 1 = every load cached;
// 2 = x gathers nontemporal as well.
template <int LP, class T> __device__ __forceinline__ T ld_stream(const T *p) {
    if constexpr (LP == 1) return *p;
    else return __builtin_nontemporal_load(p);
}
template <int LP, class T> __device__ __forceinline__ T ld_x(const T *p) {
    if constexpr (LP == 2) return __builtin_nontemporal_load(p);
    else return *p;
}

// Read-only metadata through the constant address space: with a uniform index
// the compiler issues scalar loads, which need no vector registers and do not
// wait on outstanding vector loads.
typedef int i32x4 __attribute__((ext_vector_type(4)));

template <class T> __device__ __forceinline__ T ldc(const T *p, int64_t i) {
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (sizeof(T) == 16) {
        const i32x4 v = ((const __attribute__((address_space(4))) i32x4 *)(p))[i];
        T r;
        __builtin_memcpy(&r, &v, 16);
        return r;
    } else {
        return ((const __attribute__((address_space(4))) T *)(p))[i];
    }
#else
    return p[i];
#endif
}

// K consecutive vector entries starting at p (16-byte aligned when K > 1 is a
// multiple of the vector width; checked on the host).
template <class A, int K> __device__ __forceinline__ void load_row(const A *p, A (&v)[K]) {
    if constexpr (K == 1) {
        v[0] = p[0];
    } else if constexpr (sizeof(A) == 4 && K % 4 == 0) {
#pragma unroll
        for (int i = 0; i < K / 4; i++) {
            const float4 t = reinterpret_cast<const float4 *>(p)[i];
            v[4 * i] = t.x; v[4 * i + 1] = t.y; v[4 * i + 2] = t.z; v[4 * i + 3] = t.w;
        }
    } else if constexpr (sizeof(A) == 8 && K % 2 == 0) {
#pragma unroll
        for (int i = 0; i < K / 2; i++) {
            const double2 t = reinterpret_cast<const double2 *>(p)[i];
            v[2 * i] = t.x; v[2 * i + 1] = t.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < K; i++) v[i] = p[i];
    }
}

template <class A, int K> __device__ __forceinline__ void store_row(A *p, const A (&v)[K]) {
    if constexpr (sizeof(A) == 4 && K % 4 == 0) {
#pragma unroll
        for (int i = 0; i < K / 4; i++)
            reinterpret_cast<float4 *>(p)[i] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    } else if constexpr (sizeof(A) == 8 && K % 2 == 0) {
#pragma unroll
        for (int i = 0; i < K / 2; i++) reinterpret_cast<double2 *>(p)[i] = make_double2(v[2 * i], v[2 * i + 1]);
    } else {
#pragma unroll
        for (int i = 0; i < K; i++) p[i] = v[i];
    }
}

// Output of a row code: a row of Y when the code is >= 0; a negative code
// -1 - s names slot s of the per-piece sums of a column-panel copy, which
// only launches with several right-hand sides use (single-vector kernels
// store to Y without the select).
template <int K, class A>
__device__ __forceinline__ A *out_row(A *Y, int64_t ldy, void *pan, int64_t pan_ld, int32_t code) {
    if constexpr (K == 1) return Y + (int64_t)code * ldy;
    else return code >= 0 ? Y + (int64_t)code * ldy : (A *)pan + (int64_t)(-1 - code) * pan_ld;
}

__device__ __forceinline__ float fmaA(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaA(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Group metadata of group g (row0, row count, first and end slot).
struct GroupMeta {
    int64_t row0, g0, g1;
    int sg;
};

// Uniform group index: scalar loads.
__device__ __forceinline__ GroupMeta group_meta_uniform(const SpmvParams &P, int64_t g) {
    GroupMeta m{0, 0, 0, 0};
    if (g < P.ng) {
        if (P.ragged) {
            m.row0 = ldc(P.grp_row0, g);
            m.sg = ldc(P.grp_row0, g + 1) - (int32_t)m.row0;
        } else {
            m.row0 = g * P.G;
            m.sg = (int)min((int64_t)P.G, P.ns - m.row0);
        }
        m.g0 = ldc(P.gp, g);
        m.g1 = ldc(P.gend ? P.gend : P.gp + 1, g);
    }
    return m;
}

// Geometry of the row a lane owns in the grouped part.
struct LaneRow {
    int64_t i;       // index into short_len / short_row
    int64_t base;    // first slot of this lane
    int64_t stride;  // slots between this lane's consecutive elements
    int len;         // row length
    int q;           // sub-lane within the row (0 .. T-1)
    int wc;          // steps of the group (its width / T); 0 when the lane has no row
    bool ok;
};

// Per-lane group index (several groups per wavefront): vector loads.
__device__ __forceinline__ GroupMeta group_meta_lane(const SpmvParams &P, int64_t g) {
    GroupMeta m{0, 0, 0, 0};
    if (g < P.ng) {
        if (P.ragged) {
            m.row0 = P.grp_row0[g];
            m.sg = P.grp_row0[g + 1] - (int32_t)m.row0;
        } else {
            m.row0 = g * P.G;
            m.sg = (int)min((int64_t)P.G, P.ns - m.row0);
        }
        m.g0 = P.gp[g];
        m.g1 = (P.gend ? P.gend : P.gp + 1)[g];
    }
    return m;
}

template <int T>
__device__ __forceinline__ LaneRow lane_row_of(const SpmvParams &P, const GroupMeta &m, int lr) {
    LaneRow L;
    const int t = lr / T;
    L.q = lr % T;
    L.ok = t < m.sg;
    L.i = m.row0 + t;
    L.len = L.ok ? P.short_len[L.i] : 0;
    L.base = L.ok ? m.g0 + (int64_t)t * T + L.q : 0;
    L.stride = (int64_t)m.sg * T;
    // slots of a group are fewer than 2^31 (G rows of int32 length)
    L.wc = L.ok ? (int)((uint32_t)(m.g1 - m.g0) / (uint32_t)L.stride) : 0;
    return L;
}

// Row of wave-item w owned by this lane.
template <int T>
__device__ __forceinline__ LaneRow lane_row(const SpmvParams &P, int32_t w, int lane) {
    if (P.wpg > 0) {  // G*T >= 64: wpg wavefronts per group, group index uniform
        const int32_t g = w / P.wpg;
        const int lr = (w - g * P.wpg) * 64 + lane;
        return lane_row_of<T>(P, group_meta_uniform(P, g), lr);
    }
    // G*T divides 64: gpw groups per wavefront
    const int GT = P.G * T;
    const int64_t g = (int64_t)w * P.gpw + lane / GT;
    return lane_row_of<T>(P, group_meta_lane(P, g), lane % GT);
}

template <int K> constexpr int unroll_for() { return K == 1 ? 8 : (K <= 4 ? 4 : (K <= 8 ? 2 : 1)); }
// Steps in flight per lane of a several-rows-per-lane pass with K right-hand
// sides: the gathered X rows take about 64 registers (16 steps up to K = 4).
template <int K> constexpr int multi_steps() { return K <= 4 ? 16 : 64 / K; }

// X[c * ldx] for one right-hand side with a 32-bit byte offset from the
// uniform base (scalar base + vector offset addressing; the host checks
// n_cols * ldx * size < 4 GiB for single right-hand-side launches).
template <int LP, class A> __device__ __forceinline__ A ldx32(const A *X, int32_t c, uint32_t row_bytes) {
    return ld_x<LP>((const A *)((const char *)X + (uint32_t)c * row_bytes));
}

}  // namespace rg
