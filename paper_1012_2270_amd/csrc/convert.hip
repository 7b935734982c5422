// Device-side CSR -> RgCSR conversion for gfx950: the layout of Section 3.4
// with the sort-window, long-row and lanes-per-row readings, built where the
// CSR arrays already live.  Ordering and offsets use rocPRIM primitives
// (stable radix sort, stable selection, scans); the scatter writes each
// group's slots with consecutive lanes on consecutive rows, so a wavefront
// writes 64 consecutive slots per step.  The result equals the host
// converter's arrays bit for bit.
#include <hip/hip_runtime.h>

#include <cstring>
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "compact.h"
#include "convert.h"

namespace rg {

void DevScratch::reserve(size_t bytes) {
    void *p = nullptr;
    bufs.reserve(bufs.size() + 1);
    if (hipMalloc(&p, bytes ? bytes : 1) != hipSuccess) fail(RGCSR_ENOMEM, "device scratch allocation failed");
    bufs.push_back(p);
    at = (char *)p;
    left = bytes;
}

void *DevScratch::get(size_t bytes) {
    bytes = (bytes + 255) / 256 * 256;
    if (bytes > left) reserve(bytes > (size_t(1) << 20) ? bytes : size_t(1) << 20);
    void *p = at;
    at += bytes;
    left -= bytes;
    return p;
}

DevScratch::~DevScratch() {
    (void)hipStreamSynchronize(st);
    for (void *p : bufs) (void)hipFree(p);
}

namespace {

#define CHK(x)                                                                                             \
    do {                                                                                                   \
        hipError_t e_ = (x);                                                                               \
        if (e_ != hipSuccess) fail(RGCSR_EHIP, std::string("device conversion: ") + hipGetErrorString(e_)); \
    } while (0)

int nblocks(int64_t n, int per = 256) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + per - 1) / per, 65536)); }

// bit 0: row_ptr[0] != 0; bit 1: decreasing or beyond nnz; bit 2: column out
// of range; bit 4: row_ptr[n] != nnz; bit 5: a row longer than int32.
//
// Columns ascend strictly within the rows exactly when every position whose
// column does not exceed the one before it is a row's first: *excess counts
// such positions among all elements, minus those at a row's first (it means
// something when the row pointers are in order).  So no lane walks a row, and
// the elements are read once, four a lane (1.0 ms before, where a lane walked
// the longest of 500,009 rows; under 20 us now).
constexpr int kValidateThreads = 1024;
__global__ __launch_bounds__(kValidateThreads) void validate_k(const int64_t *rp, const int32_t *col, int64_t n,
                                                               int64_t n_cols, int64_t nnz, int32_t *err,
                                                               unsigned long long *excess) {
    typedef int32_t i4 __attribute__((ext_vector_type(4)));
    typedef i4 i4a __attribute__((aligned(4)));
    int32_t e = 0;
    int64_t d = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t; i < n; i += stride) {
        const int64_t b = rp[i], en = rp[i + 1];
        if (b < 0 || en < b || en > nnz) {
            e |= 2;
            continue;
        }
        if (en - b > INT32_MAX) e |= 32;
        if (b > 0 && b < en) d -= col[b] <= col[b - 1];
    }
    const int64_t m = std::max<int64_t>(0, std::min<int64_t>(rp[n], nnz));
    for (int64_t k = 4 * t; k < m; k += 4 * stride) {
        int32_t prev = col[k > 0 ? k - 1 : 0];
        if (k == 0) prev = -1;
        i4 c;
        if (k + 4 <= m) {
            c = *(const i4a *)(col + k);
        } else {
            // past the end: the last column, once more and not counted
            for (int j = 0; j < 4; j++) c[j] = col[k + j < m ? k + j : m - 1];
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (c[j] < 0 || c[j] >= n_cols) e |= 4;
            d += k + j < m && c[j] <= prev;
            prev = c[j];
        }
    }
    if (t == 0) {
        if (rp[0] != 0) e |= 1;
        if (rp[n] != nnz) e |= 16;
    }
    // one atomic per workgroup: an address takes one in about 12 ns
    __shared__ int64_t sd[kValidateThreads / 64];
    __shared__ int32_t se[kValidateThreads / 64];
    for (int off = 32; off > 0; off >>= 1) {
        d += __shfl_xor(d, off);
        e |= __shfl_xor(e, off);
    }
    if ((threadIdx.x & 63) == 0) {
        sd[threadIdx.x >> 6] = d;
        se[threadIdx.x >> 6] = e;
    }
    __syncthreads();
    if (threadIdx.x) return;
    for (int w = 1; w < kValidateThreads / 64; w++) {
        d += sd[w];
        e |= se[w];
    }
    if (d) atomicAdd(excess, (unsigned long long)d);
    if (e) atomicOr(err, e);
}

// lengths and the sort keys of the window step: (window, longest first),
// row index as the value; rows of equal key keep their order (stable sort)
__global__ void keys_k(const int64_t *rp, int64_t n, int64_t sigma, int32_t *len, uint64_t *key, int32_t *row) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int32_t l = (int32_t)(rp[i + 1] - rp[i]);
        len[i] = l;
        row[i] = (int32_t)i;
        if (key) key[i] = ((uint64_t)(i / sigma) << 31) | (uint64_t)(0x7fffffffu - (uint32_t)l);
    }
}

// Row lengths and the window order of the sort step: a workgroup sorts the rows
// of one window of up to kWindowSort in LDS, longest first, rows of equal
// length by index (the index is part of the key, so the order is the stable
// sort's).  One launch where a radix sort over all rows took 22, each about as
// long as the work in it (500,009 rows in windows of 512: 230 us, now 15).
//
// Windows of up to half of kWindowRows share a workgroup (the window leads the
// key), so a launch never has more threads than rows: a workgroup per window
// would pass the 2^32 threads of a grid at 2^27 rows in windows of two.
constexpr int kWindowSort = 4096;
constexpr int kWindowRows = 128;
__global__ __launch_bounds__(1024) void window_sort_k(const int64_t *rp, int64_t n, int32_t sigma, int32_t rows,
                                                      int32_t size, int32_t *len, int32_t *ord) {
    extern __shared__ uint64_t wkey[];  // [size], a power of two of at least `rows`, whole windows
    const int64_t w0 = (int64_t)blockIdx.x * rows;
    const int32_t m = (int32_t)std::min<int64_t>(rows, n - w0);
    for (int32_t t = threadIdx.x; t < size; t += blockDim.x) {
        uint64_t k = ~uint64_t(0);
        if (t < m) {
            const int32_t l = (int32_t)(rp[w0 + t + 1] - rp[w0 + t]);
            len[w0 + t] = l;
            k = (uint64_t)(uint32_t)(t / sigma) << 44 | (uint64_t)(0x7fffffffu - (uint32_t)l) << 12 | (uint32_t)t;
        }
        wkey[t] = k;
    }
    __syncthreads();
    for (int32_t k = 2; k <= size; k *= 2)
        for (int32_t j = k / 2; j > 0; j /= 2) {
            for (int32_t t = threadIdx.x; t < size / 2; t += blockDim.x) {
                const int32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                const uint64_t x = wkey[i], y = wkey[i + j];
                if ((x > y) == ((i & k) == 0)) {
                    wkey[i] = y;
                    wkey[i + j] = x;
                }
            }
            __syncthreads();
        }
    for (int32_t t = threadIdx.x; t < m; t += blockDim.x) ord[w0 + t] = (int32_t)w0 + (int32_t)(wkey[t] & (kWindowSort - 1));
}

// Long-row split: the rows in window order go to the grouped rows (at most
// tau elements) or to the long rows, each in that order.  Counts per tile of
// kSplitTile rows, their prefix sums (one workgroup), then the lists; three
// launches where flags, two selections and two gathers of lengths took eleven
// (500,009 rows: 230 us with the gaps between them, now 33).
constexpr int kSplitTile = 1024;
__global__ __launch_bounds__(kSplitTile) void split_count_k(const int32_t *ord, const int32_t *len, int64_t n,
                                                            int64_t tau, int32_t *cnt) {
    __shared__ int32_t c;
    if (threadIdx.x == 0) c = 0;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kSplitTile + threadIdx.x;
    const uint64_t b = __ballot(i < n && len[ord[i < n ? i : n - 1]] <= tau);
    if ((threadIdx.x & 63) == 0) atomicAdd(&c, __popcll(b));
    __syncthreads();
    if (threadIdx.x == 0) cnt[blockIdx.x] = c;
}

// cnt becomes its exclusive prefix sum; counts: grouped rows, long rows
__global__ __launch_bounds__(1024) void split_scan_k(int32_t *cnt, int32_t tiles, int64_t n, int64_t *counts) {
    __shared__ int32_t sum[16];
    int32_t before = 0;
    for (int32_t t0 = 0; t0 < tiles; t0 += 1024) {
        const int32_t t = t0 + (int)threadIdx.x;
        const int32_t v = t < tiles ? cnt[t] : 0;
        int32_t x = v;
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t up = __shfl_up(x, off);
            if ((threadIdx.x & 63) >= off) x += up;
        }
        if ((threadIdx.x & 63) == 63) sum[threadIdx.x >> 6] = x;
        __syncthreads();
        int32_t total = 0;
        for (int w = 0; w < 16; w++) {
            if (w < (int)(threadIdx.x >> 6)) x += sum[w];
            total += sum[w];
        }
        if (t < tiles) cnt[t] = before + x - v;
        before += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        counts[0] = before;
        counts[1] = n - before;
    }
}

// lens_s, flags: as gather_len_k; key: of the long rows, longest first
__global__ __launch_bounds__(kSplitTile) void split_write_k(const int32_t *ord, const int32_t *len, int64_t n,
                                                            int64_t tau, const int32_t *cnt, int32_t *sv,
                                                            int32_t *lens_s, int32_t *lv, uint32_t *key,
                                                            int32_t *flags) {
    __shared__ int32_t sum[kSplitTile / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * kSplitTile, i = i0 + threadIdx.x;
    const int32_t row = ord[i < n ? i : n - 1], l = len[row];
    const bool is_short = i < n && l <= tau;
    const uint64_t b = __ballot(is_short);
    if (lane == 0) sum[wv] = __popcll(b);
    __syncthreads();
    int32_t s = cnt[blockIdx.x] + __popcll(b & ((uint64_t(1) << lane) - 1));
    for (int w = 0; w < kSplitTile / 64; w++) s += w < wv ? sum[w] : 0;
    int32_t f = 0;
    if (is_short) {
        sv[s] = row;
        lens_s[s] = l;
        f = (row != s ? 1 : 0) | (l == 0 ? 2 : 0);
    } else if (i < n) {
        lv[i - s] = row;
        key[i - s] = 0x7fffffffu - (uint32_t)l;
    }
    f = (__any(f & 1) ? 1 : 0) | (__any(f & 2) ? 2 : 0);
    if (lane == 0 && f && (__hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & f) != f)
        atomicOr(flags, f);
}

// lengths of the grouped rows where none are long; flags for the plan: bit 0 =
// some grouped row is out of place, bit 1 = some grouped row is empty
__global__ void gather_len_k(const int32_t *rows, const int32_t *len, int64_t n, int32_t *out, int32_t *flags) {
    int32_t f = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int32_t l = len[rows[i]];
        out[i] = l;
        if (rows[i] != i) f |= 1;
        if (l == 0) f |= 2;
    }
    // one atomic per wavefront at most: nearly every lane of a permuted layout
    // has a flag to set (47 us before, for 500,009 rows)
    f = (__any(f & 1) ? 1 : 0) | (__any(f & 2) ? 2 : 0);
    if ((threadIdx.x & 63) == 0 && f && (__hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & f) != f)
        atomicOr(flags, f);
}

// slots of each group: rows x (widest row rounded up to T)
__global__ void group_slots_k(const int32_t *lens_s, int64_t ns, int32_t G, int32_t T, int64_t ng, int64_t *cnt) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < ng; g += stride) {
        const int64_t r0 = g * G, r1 = std::min<int64_t>(ns, r0 + G);
        int64_t w = 0;
        for (int64_t r = r0; r < r1; r++) w = std::max<int64_t>(w, lens_s[r]);
        w = (w + T - 1) / T * T;
        cnt[g] = (r1 - r0) * w;
    }
}

__global__ void long_len_k(const int32_t *lv, const int32_t *len, int64_t nl, int64_t *out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nl; i += stride) out[i] = len[lv[i]];
}

// ---- value conversion, same rules as the host (convert_values) ------------
__device__ __forceinline__ float f16_to_f32_exact(uint16_t h) {
    const uint32_t sign = (uint32_t)(h & 0x8000u) << 16, e = (h >> 10) & 0x1fu, m = h & 0x3ffu;
    if (e == 0x1f) return bits_f32(sign | 0x7f800000u | (m << 13));
    if (e == 0) return (sign ? -1.0f : 1.0f) * ((float)m * 0x1p-24f);
    return bits_f32(sign | ((e + 112u) << 23) | (m << 13));
}

template <int SD> struct In;
template <> struct In<RGCSR_F64> { using T = double; __device__ static float f32(T v) { return (float)v; } };
template <> struct In<RGCSR_F32> { using T = float; __device__ static float f32(T v) { return v; } };
template <> struct In<RGCSR_F16> { using T = uint16_t; __device__ static float f32(T v) { return f16_to_f32_exact(v); } };
template <> struct In<RGCSR_BF16> { using T = uint16_t; __device__ static float f32(T v) { return bf16_to_f32(v); } };

template <int DD> struct Out;
template <> struct Out<RGCSR_F64> { using T = double; };
template <> struct Out<RGCSR_F32> { using T = float; };
template <> struct Out<RGCSR_F16> { using T = uint16_t; };
template <> struct Out<RGCSR_BF16> { using T = uint16_t; };

template <int SD, int DD> __device__ __forceinline__ typename Out<DD>::T cvt(typename In<SD>::T v) {
    if constexpr (SD == DD) return v;
    else if constexpr (DD == RGCSR_F64) return (double)In<SD>::f32(v);
    else if constexpr (DD == RGCSR_F32) return In<SD>::f32(v);
    else if constexpr (DD == RGCSR_F16) return f32_to_f16_rne(In<SD>::f32(v));
    else return f32_to_bf16_rne(In<SD>::f32(v));
}

// one lane per grouped row: nonzero j of local row t of group g goes to
// gp[g] + (j/T)*(s*T) + t*T + j%T; slots past the row's length are padding
// (value bits 0, the row's last column, or 0 for an empty row)
template <int SD, int DD>
__global__ void scatter_k(const int32_t *sv, const int32_t *lens_s, const int64_t *rp, const int32_t *col,
                          const typename In<SD>::T *vals, const int64_t *gp, int64_t ns, int32_t G, int32_t T,
                          int32_t *short_len, int32_t *short_row, int32_t *slot_col, typename Out<DD>::T *slot_val) {
    using O = typename Out<DD>::T;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < ns; s += stride) {
        const int64_t g = s / G, t = s - g * G;
        const int64_t sg = std::min<int64_t>(G, ns - g * G);
        const int64_t g0 = gp[g], W = (gp[g + 1] - g0) / sg;
        const int32_t r = sv[s];
        const int64_t b = rp[r];
        const int64_t len = lens_s[s];
        short_len[s] = (int32_t)len;
        if (short_row) short_row[s] = r;
        const int32_t ghost = len ? col[b + len - 1] : 0;
        for (int64_t j = 0; j < W; j++) {
            const int64_t slot = g0 + (j / T) * (sg * T) + t * T + (j % T);
            if (j < len) {
                slot_col[slot] = col[b + j];
                slot_val[slot] = cvt<SD, DD>(vals[b + j]);
            } else {
                slot_col[slot] = ghost;
                slot_val[slot] = (O)0;
            }
        }
    }
}

// A wavefront per long row (longest first) and piece of kLongPiece elements:
// contiguous copy into the long-row segment, kLongSteps loads in flight.  A
// wavefront that copied its row alone was 61 us for the longest of 500,009.
constexpr int64_t kLongPiece = 2048;
constexpr int kLongSteps = 8;
template <int SD, int DD>
__global__ void long_copy_k(const int32_t *lv, const int64_t *lp, const int64_t *rp, const int32_t *col,
                            const typename In<SD>::T *vals, int64_t first, int64_t end, int32_t *long_row,
                            int32_t *long_col, typename Out<DD>::T *long_val) {
    const int lane = threadIdx.x & 63;
    const int64_t wstride = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t i = first + (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); i < end; i += wstride) {
        const int32_t r = lv[i];
        const int64_t b = rp[r], o = lp[i], len = lp[i + 1] - o;
        if (lane == 0 && blockIdx.y == 0) long_row[i] = r;
        for (int64_t p0 = blockIdx.y * kLongPiece; p0 < len; p0 += gridDim.y * kLongPiece) {
            const int64_t p1 = std::min(len, p0 + kLongPiece);
            for (int64_t j0 = p0; j0 < p1; j0 += 64 * kLongSteps) {
                int32_t c[kLongSteps];
                typename In<SD>::T v[kLongSteps];
#pragma unroll
                for (int u = 0; u < kLongSteps; u++) {
                    const int64_t j = std::min(j0 + 64 * u + lane, p1 - 1);
                    c[u] = col[b + j];
                    v[u] = vals[b + j];
                }
#pragma unroll
                for (int u = 0; u < kLongSteps; u++) {
                    const int64_t j = j0 + 64 * u + lane;
                    if (j < p1) {
                        long_col[o + j] = c[u];
                        long_val[o + j] = cvt<SD, DD>(v[u]);
                    }
                }
            }
        }
    }
}

// ---- rocPRIM calls with scratch from DevScratch ------------------------------
template <class F> void with_temp(DevScratch &S, F f) {
    size_t bytes = 0;
    CHK(f(nullptr, bytes));
    void *tmp = S.get(bytes);
    CHK(f(tmp, bytes));
}

}  // namespace

void device_plan(DevPlan &P, const LayoutParams &p, int64_t n_rows, int64_t n_cols, int64_t nnz,
                 const int64_t *rp, const int32_t *col, bool validate, bool patterns, hipStream_t st) {
    if (n_rows < 0 || n_cols < 0 || nnz < 0) fail(RGCSR_EINVAL, "negative size");
    if (n_rows > INT32_MAX || n_cols > INT32_MAX)
        fail(RGCSR_EOVERFLOW, "n_rows and n_cols must fit int32 column/row indices");
    if (!rp || (nnz > 0 && !col)) fail(RGCSR_EINVAL, "null CSR array");
    P.n_rows = n_rows;
    P.n_cols = n_cols;
    P.nnz = nnz;
    DevScratch &S = P.scratch;
    const int64_t n = n_rows;
    // about what the steps below take: row arrays and the groups', the sort
    // keys, the split lists (the long rows' own arrays come on top)
    const bool sorted = p.sigma > 1, split = p.tau >= 0;
    const int64_t window = std::min(p.sigma, n);
    const bool in_lds = sorted && window <= kWindowSort;
    S.reserve((size_t)n * (18 + (sorted && !in_lds ? 40 : 0) + (split ? 14 : 0)) + (size_t(1) << 17));
    // one block of what starts at zero: error and layout flags, the row counts
    // of the split, the pattern search's state and hash table
    int32_t *flags = (int32_t *)S.get(64 + kPatHash * sizeof(uint64_t));
    int32_t *pat_state = flags + 4;
    int64_t *counts = (int64_t *)(flags + 8);
    uint64_t *pat_key = (uint64_t *)(flags + 16);
    CHK(hipMemsetAsync(flags, 0, 64 + (patterns ? kPatHash * sizeof(uint64_t) : 0), st));
    if (validate) {
        const int nwg = std::min(512, std::max(nblocks(n, kValidateThreads), nblocks(nnz, 4 * kValidateThreads)));
        hipLaunchKernelGGL(validate_k, dim3(nwg), dim3(kValidateThreads), 0, st, rp, col, n, n_cols, nnz, flags,
                           (unsigned long long *)(flags + 2));
        CHK(hipGetLastError());
    }
    int32_t hf[16];
    auto read_flags = [&] {
        CHK(hipMemcpyAsync(hf, flags, sizeof(hf), hipMemcpyDeviceToHost, st));
        CHK(hipStreamSynchronize(st));
        if (!validate) return;
        const int32_t e = hf[0] | (hf[2] || hf[3] ? 8 : 0);
        if (e & 32) fail(RGCSR_EOVERFLOW, "row longer than int32");
        if (e & 1) fail(RGCSR_ECSR, "row_ptr[0] != 0");
        if (e & 2) fail(RGCSR_ECSR, "row_ptr decreases or exceeds nnz");
        if (e & 4) fail(RGCSR_ECSR, "column out of range");
        if (e & 8) fail(RGCSR_ECSR, "columns not strictly ascending");
        if (e & 16) fail(RGCSR_ECSR, "row_ptr[n_rows] != nnz");
    };
    // (the split reads row lengths alone, so its counts come with the errors)
    if (n == 0 || (validate && !split)) read_flags();
    if (n == 0) {
        P.gp_host.assign(1, 0);
        P.long_ptr_host.assign(1, 0);
        P.gp = (const int64_t *)S.get(8);
        CHK(hipMemsetAsync((void *)P.gp, 0, 8, st));
        P.long_ptr = P.gp;
        CHK(hipStreamSynchronize(st));
        return;
    }
    // window order: stable radix sort of (window, longest first)
    int32_t *len = (int32_t *)S.get(n * 4);
    int32_t *ord = (int32_t *)S.get(n * 4);
    // (one window: the key is the length alone)
    uint64_t *key = sorted && !in_lds ? (uint64_t *)S.get(n * 8) : nullptr;
    int32_t *row_tmp = key ? (int32_t *)S.get(n * 4) : ord;
    if (in_lds) {
        const int64_t rows = std::max<int64_t>(1, kWindowRows / window) * window;
        int32_t size = 2;
        while (size < rows) size *= 2;
        hipLaunchKernelGGL(window_sort_k, dim3((unsigned)((n + rows - 1) / rows)), dim3(std::clamp(size / 2, 64, 1024)),
                           size * sizeof(uint64_t), st, rp, n, (int32_t)window, (int32_t)rows, size, len, ord);
    } else {
        hipLaunchKernelGGL(keys_k, dim3(nblocks(n)), dim3(256), 0, st, rp, n, p.sigma, len, key, row_tmp);
    }
    CHK(hipGetLastError());
    if (key) {
        uint64_t *key_out = (uint64_t *)S.get(n * 8);
        const int64_t windows = (n + p.sigma - 1) / p.sigma;
        unsigned int wbits = 0;
        while (wbits < 32 && (int64_t(1) << wbits) < windows) wbits++;
        const unsigned int end_bit = 31 + wbits;
        with_temp(S, [&](void *t, size_t &b) {
            return rocprim::radix_sort_pairs(t, b, key, key_out, row_tmp, ord, (size_t)n, 0u, end_bit, st);
        });
    }
    // long-row split, both lists in window order; lengths, order and emptiness
    // flags of the grouped rows
    int32_t *sv = ord, *lv0 = nullptr;
    uint32_t *lk = nullptr;
    int32_t *lens_s = (int32_t *)S.get(n * 4);
    P.ns = n;
    P.nl = 0;
    if (split) {
        const int32_t tiles = (int32_t)((n + kSplitTile - 1) / kSplitTile);
        int32_t *cnt = (int32_t *)S.get((size_t)tiles * 4);
        sv = (int32_t *)S.get(n * 4);
        lv0 = (int32_t *)S.get(n * 4);
        lk = (uint32_t *)S.get(n * 4);
        hipLaunchKernelGGL(split_count_k, dim3(tiles), dim3(kSplitTile), 0, st, ord, len, n, p.tau, cnt);
        hipLaunchKernelGGL(split_scan_k, dim3(1), dim3(1024), 0, st, cnt, tiles, n, counts);
        hipLaunchKernelGGL(split_write_k, dim3(tiles), dim3(kSplitTile), 0, st, ord, len, n, p.tau, cnt, sv, lens_s, lv0,
                           lk, flags + 1);
        CHK(hipGetLastError());
        read_flags();
        int64_t hc[2];
        memcpy(hc, hf + 8, sizeof(hc));
        P.ns = hc[0];
        P.nl = hc[1];
    } else {
        hipLaunchKernelGGL(gather_len_k, dim3(std::min(nblocks(n), 512)), dim3(256), 0, st, sv, len, n, lens_s, flags + 1);
        CHK(hipGetLastError());
    }
    const int64_t ns = P.ns, nl = P.nl;
    // group widths, offsets
    P.ng = (ns + p.G - 1) / p.G;
    int64_t *gp = (int64_t *)S.get((P.ng + 1) * 8);
    CHK(hipMemsetAsync(gp, 0, 8, st));
    if (P.ng) {
        int64_t *cnt = (int64_t *)S.get(P.ng * 8);
        hipLaunchKernelGGL(group_slots_k, dim3(nblocks(P.ng)), dim3(256), 0, st, lens_s, ns, p.G, p.T, P.ng, cnt);
        CHK(hipGetLastError());
        with_temp(S, [&](void *t, size_t &b) {
            return rocprim::inclusive_scan(t, b, cnt, gp + 1, (size_t)P.ng, rocprim::plus<int64_t>(), st);
        });
    }
    // long rows: longest first, ties in window order; their offsets
    int32_t *lv = lv0;
    int64_t *lp = (int64_t *)S.get((nl + 1) * 8);
    CHK(hipMemsetAsync(lp, 0, 8, st));
    if (nl) {
        uint32_t *lk2 = (uint32_t *)S.get(nl * 4);
        lv = (int32_t *)S.get(nl * 4);
        with_temp(S, [&](void *t, size_t &b) {
            return rocprim::radix_sort_pairs(t, b, lk, lk2, lv0, lv, (size_t)nl, 0u, 31u, st);
        });
        int64_t *ll = (int64_t *)S.get(nl * 8);
        hipLaunchKernelGGL(long_len_k, dim3(nblocks(nl)), dim3(256), 0, st, lv, len, nl, ll);
        CHK(hipGetLastError());
        with_temp(S, [&](void *t, size_t &b) {
            return rocprim::inclusive_scan(t, b, ll, lp + 1, (size_t)nl, rocprim::plus<int64_t>(), st);
        });
    }
    patterns = patterns && nl == 0;
    if (patterns) {
        uint8_t *id = (uint8_t *)S.get(n);
        int32_t *tab = (int32_t *)S.get(kPatTab * sizeof(int32_t));
        CHK(launch_find_patterns(rp, col, n, pat_key, (int32_t *)S.get(2 * kPatHash * sizeof(int32_t)), pat_state,
                                 (uint16_t *)S.get(n * 2), id, tab, st));
        P.pat_id = id;
        P.pat_tab = tab;
    }
    P.gp_host.resize(P.ng + 1);
    P.long_ptr_host.assign(nl + 1, 0);
    int32_t small[8];
    if (patterns) {
        P.pat_host.resize(kPatTab);
        CHK(hipMemcpyAsync(P.pat_host.data(), P.pat_tab, kPatTab * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    }
    CHK(hipMemcpyAsync(P.gp_host.data(), gp, (P.ng + 1) * 8, hipMemcpyDeviceToHost, st));
    if (nl) CHK(hipMemcpyAsync(P.long_ptr_host.data(), lp, (nl + 1) * 8, hipMemcpyDeviceToHost, st));
    CHK(hipMemcpyAsync(small, flags, sizeof(small), hipMemcpyDeviceToHost, st));
    CHK(hipStreamSynchronize(st));
    P.slots = P.gp_host[P.ng];
    P.long_nnz = P.long_ptr_host[nl];
    P.perm = (small[1] & 1) != 0;
    P.no_empty = (small[1] & 2) == 0;
    P.sv = sv;
    P.lv = lv;
    P.lens_s = lens_s;
    P.gp = gp;
    P.long_ptr = lp;
    if (patterns && !small[4 + 1] && pat_pays(small[4], small[4 + 2], P.slots)) {
        P.n_pat = small[4];
        P.pat_stride = small[4 + 2];
    }
}

namespace {

template <int SD, int DD>
void fill_t(const DevPlan &P, const LayoutParams &p, const int64_t *rp, const int32_t *col, const void *vals,
            int32_t *short_len, int32_t *short_row, void *slot_val, int32_t *slot_col, int32_t *long_row,
            void *long_val, int32_t *long_col, hipStream_t st) {
    using IT = typename In<SD>::T;
    using OT = typename Out<DD>::T;
    if (P.ns) {
        hipLaunchKernelGGL((scatter_k<SD, DD>), dim3(nblocks(P.ns)), dim3(256), 0, st, P.sv, P.lens_s, rp, col,
                           (const IT *)vals, P.gp, P.ns, p.G, p.T, short_len, short_row, slot_col, (OT *)slot_val);
        CHK(hipGetLastError());
    }
    // rows of several pieces, then the rest
    int64_t big = 0;
    while (big < P.nl && P.long_ptr_host[big + 1] - P.long_ptr_host[big] > kLongPiece) big++;
    if (big) {
        const int64_t pieces = (P.long_ptr_host[1] - P.long_ptr_host[0] + kLongPiece - 1) / kLongPiece;
        hipLaunchKernelGGL((long_copy_k<SD, DD>), dim3(std::min(nblocks(big, 4), 1024), (unsigned)std::min<int64_t>(pieces, 256)),
                           dim3(256), 0, st, P.lv, P.long_ptr, rp, col, (const IT *)vals, (int64_t)0, big, long_row,
                           long_col, (OT *)long_val);
        CHK(hipGetLastError());
    }
    if (P.nl > big) {
        hipLaunchKernelGGL((long_copy_k<SD, DD>), dim3(nblocks(P.nl - big, 4)), dim3(256), 0, st, P.lv, P.long_ptr, rp,
                           col, (const IT *)vals, big, P.nl, long_row, long_col, (OT *)long_val);
        CHK(hipGetLastError());
    }
}

template <int SD>
void fill_s(int vdt, const DevPlan &P, const LayoutParams &p, const int64_t *rp, const int32_t *col, const void *vals,
            int32_t *short_len, int32_t *short_row, void *slot_val, int32_t *slot_col, int32_t *long_row,
            void *long_val, int32_t *long_col, hipStream_t st) {
    switch (vdt) {
    case RGCSR_F64: return fill_t<SD, RGCSR_F64>(P, p, rp, col, vals, short_len, short_row, slot_val, slot_col, long_row, long_val, long_col, st);
    case RGCSR_F32: return fill_t<SD, RGCSR_F32>(P, p, rp, col, vals, short_len, short_row, slot_val, slot_col, long_row, long_val, long_col, st);
    case RGCSR_F16: return fill_t<SD, RGCSR_F16>(P, p, rp, col, vals, short_len, short_row, slot_val, slot_col, long_row, long_val, long_col, st);
    case RGCSR_BF16: return fill_t<SD, RGCSR_BF16>(P, p, rp, col, vals, short_len, short_row, slot_val, slot_col, long_row, long_val, long_col, st);
    }
    fail(RGCSR_EINVAL, "bad value dtype");
}

}  // namespace

void device_fill(const DevPlan &P, const LayoutParams &p, const int64_t *rp, const int32_t *col, const void *vals,
                 int vals_dt, int vdt, int64_t *gp, int32_t *short_len, int32_t *short_row, void *slot_val,
                 int32_t *slot_col, int32_t *long_row, int64_t *long_ptr, void *long_val, int32_t *long_col,
                 hipStream_t st) {
    if (P.nnz > 0 && !vals) fail(RGCSR_EINVAL, "vals is null");
    CHK(hipMemcpyAsync(gp, P.gp, (P.ng + 1) * 8, hipMemcpyDeviceToDevice, st));
    CHK(hipMemcpyAsync(long_ptr, P.long_ptr, (P.nl + 1) * 8, hipMemcpyDeviceToDevice, st));
    switch (vals_dt) {
    case RGCSR_F64: return fill_s<RGCSR_F64>(vdt, P, p, rp, col, vals, short_len, short_row, slot_val, slot_col, long_row, long_val, long_col, st);
    case RGCSR_F32: return fill_s<RGCSR_F32>(vdt, P, p, rp, col, vals, short_len, short_row, slot_val, slot_col, long_row, long_val, long_col, st);
    case RGCSR_F16: return fill_s<RGCSR_F16>(vdt, P, p, rp, col, vals, short_len, short_row, slot_val, slot_col, long_row, long_val, long_col, st);
    case RGCSR_BF16: return fill_s<RGCSR_BF16>(vdt, P, p, rp, col, vals, short_len, short_row, slot_val, slot_col, long_row, long_val, long_col, st);
    }
    fail(RGCSR_EINVAL, "bad input dtype");
}

DevCompact device_compact(DevPlan &P, const LayoutParams &p, int esz, const int64_t *rp, const int32_t *col,
                          hipStream_t st) {
    DevCompact C;
    if (P.n_pat) {
        C.mode = kCompactPattern;
        C.n_pat = P.n_pat;
        C.stride = P.pat_stride;
        C.segs = pattern_segments(P.pat_host.data(), C.n_pat, C.stride);
        C.width = C.stride - 1;
        C.rows = compact_rows(C.width, esz);
        return C;
    }
    if (p.G != 64 || P.slots < kWinMinSlots || !win_pays(0, P.slots, P.nnz)) return C;
    const int32_t rows = compact_rows(P.slots / P.ns, esz), per = kBlockWaves * rows;
    const int64_t units = (P.ng + per - 1) / per;
    int32_t *win = (int32_t *)P.scratch.get(2 * units * sizeof(int32_t));
    unsigned long long *count = (unsigned long long *)P.scratch.get(2 * sizeof(unsigned long long));
    unsigned long long h[2];
    CHK(hipMemsetAsync(count, 0, sizeof(h), st));
    CHK(launch_windows(P.sv, rp, col, P.ns, per * 64, units, win, count, st));
    CHK(hipMemcpyAsync(h, count, sizeof(h), hipMemcpyDeviceToHost, st));
    CHK(hipStreamSynchronize(st));
    if (h[1] > (unsigned long long)kWinCols || !win_pays((int64_t)h[0], P.slots, P.nnz)) return C;
    C.mode = kCompactWindow;
    C.rows = rows;
    C.units = units;
    C.win = win;
    return C;
}

void device_compact_fill(const DevPlan &P, const DevCompact &C, const int64_t *gp, const int32_t *slot_col,
                         uint8_t *pat_id, int32_t *pat_tab, int32_t *win, uint16_t *col16, hipStream_t st) {
    if (C.mode == kCompactPattern) {
        CHK(launch_gather_id(P.sv, P.pat_id, P.ns, pat_id, st));
        CHK(hipMemcpyAsync(pat_tab, P.pat_tab, (size_t)C.n_pat * C.stride * 4, hipMemcpyDeviceToDevice, st));
    } else if (C.mode == kCompactWindow) {
        CHK(hipMemcpyAsync(win, C.win, (size_t)C.units * 8, hipMemcpyDeviceToDevice, st));
        CHK(launch_col16(gp, P.ng, kBlockWaves * C.rows, C.units, C.win, slot_col, col16, st));
    }
}

}  // namespace rg
