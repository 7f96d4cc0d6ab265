// Stand-alone recovery/imputation pass (paper Sec. 3.1: the missing slices of a
// result are added back and filled by one of three policies: Zero, Same,
// Average).  HBM-bound: only the dropped slices are written (Zero), read and
// written (Same), or the kept ones read once and the dropped ones written
// (Average).  Kept slices are never touched.
#include "zr_common.h"

namespace zr {

namespace {

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Elem<uint16_t> {   // bf16 storage
    static __device__ __forceinline__ float load(const uint16_t* p) { return bf16_bits_to_f32(*p); }
    static __device__ __forceinline__ void store(uint16_t* p, float v) { *p = (uint16_t)f32_to_bf16_bits(v); }
};

// true if p is in the ascending list keep[0..n_keep)
__device__ __forceinline__ bool is_kept(const int32_t* __restrict__ keep, int n_keep, int p)
{
    int lo = 0, hi = n_keep;          // first position with keep[pos] >= p
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (keep[mid] < p) lo = mid + 1; else hi = mid;
    }
    return lo < n_keep && keep[lo] == p;
}

constexpr int FILL_ROWS = 32;   // rows per workgroup of the column-fill kernel

// axis 1, ZERO / SAME: thread <-> one column, loops over a stripe of rows.
// Raw copies (bit-exact), so the element type is only a width.
template <typename T, bool SAME>
__global__ __launch_bounds__(256) void fill_cols_kernel(
    T* __restrict__ out, const T* __restrict__ prev, int64_t ld, int rows, int cols,
    const int32_t* __restrict__ keep, int n_keep)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= cols) return;
    if (is_kept(keep, n_keep, p)) return;
    const int r0 = blockIdx.y * FILL_ROWS;
    const int r1 = min(rows, r0 + FILL_ROWS);
    for (int r = r0; r < r1; ++r) {
        const size_t off = (size_t)r * (size_t)ld + (size_t)p;
        out[off] = SAME ? prev[off] : T(0);
    }
}

// axis 0, ZERO / SAME: one workgroup per row; kept rows exit at once.
template <typename T, bool SAME>
__global__ __launch_bounds__(256) void fill_rows_kernel(
    T* __restrict__ out, const T* __restrict__ prev, int64_t ld, int rows, int cols,
    const int32_t* __restrict__ keep, int n_keep)
{
    const int r = blockIdx.x;
    if (is_kept(keep, n_keep, r)) return;
    T* o = out + (size_t)r * (size_t)ld;
    const T* q = SAME ? prev + (size_t)r * (size_t)ld : nullptr;
    for (int c = threadIdx.x; c < cols; c += 256) o[c] = SAME ? q[c] : T(0);
}

constexpr int MARKS = 8192;          // positions marked at a time

// flags[p] <- whether c0 + p is in the list, for p < width <= MARKS (the whole workgroup calls it; two
// barriers).  Bytes: bits would be atomic additions of neighbours to one word.
__device__ __forceinline__ void mark_kept(const int32_t* __restrict__ keep, int n_keep, int c0, int width, uint8_t* flags)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int w = tid; w < (width + 15) / 16; w += nt) *(uint4*)(flags + 16 * w) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    // (from the first entry that is not below c0: the list is ascending)
    const int first = c0 == 0 ? 0 : lower_bound_wave(keep, n_keep, c0, tid & 63);
    for (int q = first + tid; q < n_keep; q += nt) {
        const int p = keep[q] - c0;
        if (p >= width) break;
        if (p >= 0) flags[p] = 1;
    }
    __syncthreads();
}

// axis 1, AVERAGE: one workgroup per RB rows.  Sum of the kept columns in a fixed
// order (per-thread strided partial sums, then a fixed tree), so the result is
// deterministic; then the dropped columns receive the mean.
// Bound by the loads of single elements that are in flight (a thread has RB rows of four list entries)
// and by the stores: a wavefront takes 64 neighbouring columns, whatever the list looks like (a thread to a
// gap, one row to a workgroup: 8192 x 3072 bf16, 0.75 kept 51 us, only the first 0.75 kept 76, now 23 and 15;
// one row of 100000 columns behind the last kept one 2000 -> 39).
template <typename T, int RB>
__global__ __launch_bounds__(256) void average_cols_kernel(
    T* __restrict__ out, int64_t ld, int rows, int cols,
    const int32_t* __restrict__ keep, int n_keep)
{
    __shared__ float part[RB][256];
    __shared__ __align__(16) uint8_t flags[MARKS];
    const int tid = threadIdx.x;
    const int r0 = blockIdx.x * RB;
    T* o[RB];                                  // rows past the last one repeat it and are not written
#pragma unroll
    for (int r = 0; r < RB; ++r) o[r] = out + (size_t)min(r0 + r, rows - 1) * (size_t)ld;
    float acc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) acc[r] = 0.f;
    constexpr int U = 4;
    for (int q0 = tid; q0 < n_keep; q0 += U * 256) {
        int at[U];
        float v[U][RB];
#pragma unroll
        for (int u = 0; u < U; ++u) at[u] = keep[min(q0 + u * 256, n_keep - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < RB; ++r) v[u][r] = Elem<T>::load(o[r] + clamp_idx(at[u], cols));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (q0 + u * 256 < n_keep) {
#pragma unroll
                for (int r = 0; r < RB; ++r) acc[r] += v[u][r];
            }
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) part[r][tid] = acc[r];
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) {
#pragma unroll
            for (int r = 0; r < RB; ++r) part[r][tid] += part[r][tid + s];
        }
        __syncthreads();
    }
    float mean[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) mean[r] = part[r][0] / (float)n_keep;
    for (int c0 = 0; c0 < cols; c0 += MARKS) {
        mark_kept(keep, n_keep, c0, min(MARKS, cols - c0), flags);
        for (int c = c0 + tid; c < min(cols, c0 + MARKS); c += 256) {
            if (flags[c - c0]) continue;
#pragma unroll
            for (int r = 0; r < RB; ++r)
                if (r0 + r < rows) Elem<T>::store(o[r] + c, mean[r]);
        }
        __syncthreads();
        if (cols - c0 <= MARKS) break;
    }
}

// axis 0, AVERAGE: one workgroup per COLS columns; its 1024 / COLS parts take the kept rows h, h + parts,
// ... and their sums are added in that order: a fixed order, so the result is deterministic.
// Bound by latency at a weight shard's sizes: with one thread walking all kept
// rows of its column every load waited for the list entry in front of it (299 us for 768 kept of
// 1024 rows, 1024 bf16 columns); here a part asks for eight rows at a time while the next eight
// list entries are on their way (9 us).  (Gaps walked by the wavefront that finds them, however long: the
// first twentieth of 8192 rows kept 169 us, now 19.)
// COLS: 32 for as many workgroups and rows in flight as possible, 256 where there are columns enough for the chip
// or too few kept rows for 32 parts (100 x 100000, 5 kept: 16 -> 9 us, 75 kept: 28 -> 12).
template <typename T, int COLS>
__global__ __launch_bounds__(1024) void average_rows_kernel(
    T* __restrict__ out, int64_t ld, int rows, int cols,
    const int32_t* __restrict__ keep, int n_keep, int first_block)
{
    constexpr int PARTS = 1024 / COLS;
    // narrow: sixteen wavefronts, each 64 / COLS rows at a time; wide: groups of COLS / 64 wavefronts
    constexpr bool WIDE = COLS >= 64;
    constexpr int GROUPS = WIDE ? PARTS : 16, ROWS = WIDE ? 1 : 64 / COLS, LONGS = 128;
    __shared__ int longs[LONGS][2], n_long;
    __shared__ float part[PARTS][COLS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = threadIdx.x % COLS, h = threadIdx.x / COLS, group = WIDE ? h : wave;
    const int cb = first_block + blockIdx.x;
    const int c = min(cb * COLS + col, cols - 1);                   // lanes past the edge repeat the last column
    const bool mine = cols - cb * COLS > col;
    constexpr int U = 8;
    int next[U];
#pragma unroll
    for (int u = 0; u < U; ++u) next[u] = keep[min(h + u * PARTS, n_keep - 1)];
    float acc = 0.f;
    for (int q0 = h; q0 < n_keep; q0 += U * PARTS) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = Elem<T>::load(out + (size_t)clamp_idx(next[u], rows) * (size_t)ld + c);
#pragma unroll
        for (int u = 0; u < U; ++u) next[u] = keep[min(q0 + (U + u) * PARTS, n_keep - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) acc += q0 + u * PARTS < n_keep ? v[u] : 0.f;
    }
    part[h][col] = acc;
    if (threadIdx.x == 0) n_long = 0;
    __syncthreads();
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < PARTS; ++w) sum += part[w][col];
    const float mean = sum / (float)n_keep;
    // gap q lies before kept row keep[q]; gap n_keep lies after the last one.  A wavefront looks
    // 64 gaps up at once and walks the short ones that hold a row; the long ones (fewer than
    // LONGS can be longer than rows / LONGS) are dealt out to all wavefronts afterwards.
    for (int q0 = group * 64; q0 <= n_keep; q0 += GROUPS * 64) {
        const int q = q0 + lane;
        int lo = 0, hi = 0;
        if (q <= n_keep) {
            lo = q == 0 ? 0 : clamp_idx(keep[q - 1], rows) + 1;
            hi = q == n_keep ? rows : clamp_idx(keep[q], rows);
        }
        const bool is_long = hi - lo > max(8, rows / LONGS);
        if (is_long && (!WIDE || col < 64)) {
            const int slot = atomicAdd(&n_long, 1);
            if (slot < LONGS) { longs[slot][0] = lo; longs[slot][1] = hi; }
        }
        unsigned long long todo = __ballot(hi > lo && !is_long);
        while (todo) {
            const int src = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            const int p1 = __builtin_amdgcn_readlane(hi, src);
            for (int p = __builtin_amdgcn_readlane(lo, src) + (WIDE ? 0 : lane / COLS); p < p1; p += ROWS)
                if (mine) Elem<T>::store(out + (size_t)p * (size_t)ld + c, mean);
        }
    }
    __syncthreads();
    for (int g = 0; g < min(n_long, LONGS); ++g) {
        const int p1 = longs[g][1];
        for (int p = longs[g][0] + group * ROWS + (WIDE ? 0 : lane / COLS); p < p1; p += GROUPS * ROWS)
            if (mine) Elem<T>::store(out + (size_t)p * (size_t)ld + c, mean);
    }
}

// ---- Average from the per-tile sums of the product's epilogue ----------------
__global__ __launch_bounds__(256) void zero_f32_kernel(float* __restrict__ p, size_t count)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = 0.f;
}

// mean over the kept slices, slots added in slot order; left in slot 0
__global__ __launch_bounds__(256) void mean_finish_kernel(float* __restrict__ partial, int slots, int len, int n_keep)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= len) return;
    float sum = 0.f;
    for (int s = 0; s < slots; ++s) sum += partial[(size_t)s * (size_t)len + i];
    partial[i] = sum / (float)n_keep;
}

// axis 1: dropped column p of row r receives mean[r]
template <typename T>
__global__ __launch_bounds__(256) void mean_fill_cols_kernel(
    T* __restrict__ out, int64_t ld, int rows, int cols, const int32_t* __restrict__ keep, int n_keep,
    const float* __restrict__ mean)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= cols) return;
    if (is_kept(keep, n_keep, p)) return;
    const int r0 = blockIdx.y * FILL_ROWS;
    const int r1 = min(rows, r0 + FILL_ROWS);
    for (int r = r0; r < r1; ++r) Elem<T>::store(out + (size_t)r * (size_t)ld + (size_t)p, mean[r]);
}

// axis 0: dropped row r receives mean[c] in column c
template <typename T>
__global__ __launch_bounds__(256) void mean_fill_rows_kernel(
    T* __restrict__ out, int64_t ld, int rows, int cols, const int32_t* __restrict__ keep, int n_keep,
    const float* __restrict__ mean)
{
    const int r = blockIdx.x;
    if (is_kept(keep, n_keep, r)) return;
    T* o = out + (size_t)r * (size_t)ld;
    for (int c = threadIdx.x; c < cols; c += 256) Elem<T>::store(o + c, mean[c]);
}

template <typename T>
int mean_fill_typed(T* out, int64_t ld, int rows, int cols, int axis, const int32_t* keep, int n_keep,
                    float* partial, int slots, hipStream_t stream)
{
    const int len = axis == 1 ? rows : cols;
    hipLaunchKernelGGL(mean_finish_kernel, dim3((len + 255) / 256), dim3(256), 0, stream, partial, slots, len, n_keep);
    if (axis == 1) {
        dim3 grid((cols + 255) / 256, (rows + FILL_ROWS - 1) / FILL_ROWS);
        hipLaunchKernelGGL(mean_fill_cols_kernel<T>, grid, dim3(256), 0, stream, out, ld, rows, cols, keep, n_keep,
                           (const float*)partial);
    } else {
        hipLaunchKernelGGL(mean_fill_rows_kernel<T>, dim3(rows), dim3(256), 0, stream, out, ld, rows, cols, keep,
                           n_keep, (const float*)partial);
    }
    return hip_status(hipGetLastError());
}

template <typename T>
int impute_typed(T* out, int64_t ld, int rows, int cols, int axis, const int32_t* keep, int n_keep,
                 int policy, const T* prev, hipStream_t stream)
{
    const int n = axis == 0 ? rows : cols;
    if (n_keep == n) return ZR_OK;                       // nothing is missing
    if (policy == ZR_IMPUTE_SAME && prev == out) return ZR_OK;
    if (policy == ZR_IMPUTE_AVERAGE) {
        if (axis == 1) {
            if (rows >= 1024)
                hipLaunchKernelGGL((average_cols_kernel<T, 4>), dim3((rows + 3) / 4), dim3(256), 0, stream, out, ld, rows, cols, keep, n_keep);
            else
                hipLaunchKernelGGL((average_cols_kernel<T, 1>), dim3(rows), dim3(256), 0, stream, out, ld, rows, cols, keep, n_keep);
        } else {
            const int wide = (cols + 255) / 256;
            if (wide >= 256 || (n_keep <= 128 && wide >= 64)) {
                constexpr int AT_ONCE = 1 << 21;             // (a launch has fewer than 2^32 threads)
                for (int first = 0; first < wide; first += AT_ONCE)
                    hipLaunchKernelGGL((average_rows_kernel<T, 256>), dim3(std::min(wide - first, AT_ONCE)), dim3(1024), 0, stream, out, ld,
                                       rows, cols, keep, n_keep, first);
            } else {
                hipLaunchKernelGGL((average_rows_kernel<T, 32>), dim3((cols + 31) / 32), dim3(1024), 0, stream, out, ld, rows, cols, keep,
                                   n_keep, 0);
            }
        }
    } else {
        const bool same = policy == ZR_IMPUTE_SAME;
        if (axis == 1) {
            dim3 grid((cols + 255) / 256, (rows + FILL_ROWS - 1) / FILL_ROWS);
            if (same) hipLaunchKernelGGL((fill_cols_kernel<T, true>), grid, dim3(256), 0, stream,
                                         out, prev, ld, rows, cols, keep, n_keep);
            else hipLaunchKernelGGL((fill_cols_kernel<T, false>), grid, dim3(256), 0, stream,
                                    out, prev, ld, rows, cols, keep, n_keep);
        } else {
            if (same) hipLaunchKernelGGL((fill_rows_kernel<T, true>), dim3(rows), dim3(256), 0, stream,
                                         out, prev, ld, rows, cols, keep, n_keep);
            else hipLaunchKernelGGL((fill_rows_kernel<T, false>), dim3(rows), dim3(256), 0, stream,
                                    out, prev, ld, rows, cols, keep, n_keep);
        }
    }
    return hip_status(hipGetLastError());
}

}  // namespace

int launch_zero_f32(float* p, size_t count, hipStream_t stream)
{
    if (count == 0) return ZR_OK;
    hipLaunchKernelGGL(zero_f32_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, p, count);
    return hip_status(hipGetLastError());
}

int launch_mean_fill(void* out, int64_t ld, int rows, int cols, int axis, const int32_t* keep_idx, int n_keep,
                     float* partial, int slots, int dtype, hipStream_t stream)
{
    if (dtype == ZR_F32)
        return mean_fill_typed<float>((float*)out, ld, rows, cols, axis, keep_idx, n_keep, partial, slots, stream);
    return mean_fill_typed<uint16_t>((uint16_t*)out, ld, rows, cols, axis, keep_idx, n_keep, partial, slots, stream);
}

int launch_impute(void* out, int64_t ld, int rows, int cols, int axis,
                  const int32_t* keep_idx, int n_keep, int policy, const void* prev,
                  int dtype, hipStream_t stream)
{
    if (dtype == ZR_F32)
        return impute_typed<float>((float*)out, ld, rows, cols, axis, keep_idx, n_keep, policy,
                                   (const float*)prev, stream);
    return impute_typed<uint16_t>((uint16_t*)out, ld, rows, cols, axis, keep_idx, n_keep, policy,
                                  (const uint16_t*)prev, stream);
}

}  // namespace zr
