// Priority bookkeeping of ZERO-resizing (paper Sec. 3.2 and Algorithm 1, the
// per-layer block that precedes the top-L_pri select):
//   delta_i = (1/R) * sum_j |w_ji^t - w_ji^(t-1)|   weight variation of slice i
//   an index pruned in the previous epoch keeps its previous score (incremental update)
//   L_uni   = #{ i : delta_i > theta }                (differentiated per-layer ratio)
// HBM-bound reductions over the two weight snapshots; every sum is taken in a
// fixed order (no floating-point atomics), so results are bitwise repeatable.
#include <atomic>

#include "zr_common.h"

namespace zr {

namespace {

// Scratch of zr_priority_scores_static: the per-row-range column sums that the ordinary
// entry point keeps in the caller's workspace.  One copy per GPU the library runs on, held
// until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; kernels are always given the address that call returned.
constexpr size_t kStaticScratchBytes = (size_t)1 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 16;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device (looked up once per device).
int static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ZR_ERR_HIP;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ZR_ERR_HIP;
        g_scratch_ptr[dev].store(p, std::memory_order_release);     // every thread finds the same address
    }
    *out = p;
    return ZR_OK;
}

template <typename T, int V> struct Vec;
template <> struct Vec<float, 1>    { using type = float; };
template <> struct Vec<float, 4>    { using type = float4; };
template <> struct Vec<uint16_t, 1> { using type = uint16_t; };
template <> struct Vec<uint16_t, 4> { using type = uint2; };
template <> struct Vec<uint16_t, 8> { using type = uint4; };

__device__ __forceinline__ float absdiff(float a, float b) { return fabsf(a - b); }

// |a - b| of V consecutive elements, added element-wise into acc[V]
template <typename T, int V>
__device__ __forceinline__ void accum(const T* __restrict__ a, const T* __restrict__ b, float* acc)
{
    using VT = typename Vec<T, V>::type;
    const VT va = *reinterpret_cast<const VT*>(a);
    const VT vb = *reinterpret_cast<const VT*>(b);
    if constexpr (sizeof(T) == 4) {
        const float* pa = reinterpret_cast<const float*>(&va);
        const float* pb = reinterpret_cast<const float*>(&vb);
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] += absdiff(pa[i], pb[i]);
    } else if constexpr (V == 1) {
        acc[0] += absdiff(bf16_bits_to_f32(va), bf16_bits_to_f32(vb));
    } else {
        const uint32_t* pa = reinterpret_cast<const uint32_t*>(&va);
        const uint32_t* pb = reinterpret_cast<const uint32_t*>(&vb);
#pragma unroll
        for (int i = 0; i < V / 2; ++i) {
            acc[2 * i]     += absdiff(__uint_as_float(pa[i] << 16), __uint_as_float(pb[i] << 16));
            acc[2 * i + 1] += absdiff(__uint_as_float(pa[i] & 0xffff0000u), __uint_as_float(pb[i] & 0xffff0000u));
        }
    }
}

// flags[0..width) <- whether column c0 + i is in the list, for i < width <= 256 (the whole
// workgroup calls it; wavefront 0 searches).  `first` is a word of LDS.  Two barriers.
__device__ __forceinline__ void mark_kept(const int32_t* __restrict__ keep, int n_keep, int c0, int width,
                                          uint8_t* flags, int* first)
{
    const int tid = threadIdx.x;
    if (tid < 64) {
        const int lo = lower_bound_wave(keep, n_keep, c0, tid);
        if (tid == 0) *first = lo;
    }
    if (tid < width) flags[tid] = 0;
    __syncthreads();
    const int i = *first + tid;
    if (tid < width && i < n_keep) {
        const int p = keep[i] - c0;
        if (p >= 0 && p < width) flags[p] = 1;
    }
    __syncthreads();
}

// Column sums of |W_t - W_prev| over the rows [blockIdx.y * rows_per, +rows_per).
// A lane owns V adjacent columns, LPR lanes a row, so a workgroup has LPR * V columns and
// 1024 / LPR rows in flight; the rows' sums are added by a fixed shuffle tree, those of the 16
// wavefronts in wavefront order.
// FINAL: the grid has one row range and writes the scores; otherwise it writes the range's sums to
// partial[blockIdx.y][N].
// What bounds it: how much the chip has in flight.  With scratch, pieces of 512 bytes and more
// by as many row ranges as give every compute unit a workgroup; without (or with few rows) a
// workgroup reads all rows of a piece, of 64 bytes so that there are as many as possible, or of 512 and
// more where those are enough: 4096 x 2752 bf16 without scratch 74 -> 15 us, with it (in a sequence
// of calls) 12 + 9 -> 12.7 + 3.9.  (Pieces of 64 bytes with scratch too, to save the second launch: 15 us
// against 17 on matrices in the last-level cache, but 22 to 33 against 12 + 9 from memory.)
template <typename T, int V, int LPR, bool FINAL>
__global__ __launch_bounds__(1024) void col_sums_kernel(
    const T* __restrict__ Wt, const T* __restrict__ Wp, int64_t ld, int K, int N, int rows_per,
    const float* __restrict__ prev_scores, const int32_t* __restrict__ prev_keep, int n_prev_keep,
    float* __restrict__ out)
{
    constexpr int CW = LPR * V, RSTEP = 1024 / LPR;
    constexpr bool NARROW = LPR * V * sizeof(T) <= 128 && LPR <= 32;
    constexpr int UNROLL = NARROW ? 8 : 4;
    using VT = typename Vec<T, V>::type;
    __shared__ float part[16][CW];
    __shared__ uint8_t kept[CW];
    __shared__ int first;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int c0 = (int)blockIdx.x * CW;
    if constexpr (CW * sizeof(T) < 128) {
        // neighbouring pieces share lines of memory: every XCD gets a contiguous range of them
        // (the host pads this grid to a multiple of 8)
        c0 = ((int)(blockIdx.x % 8) * ((int)gridDim.x / 8) + (int)blockIdx.x / 8) * CW;
        if (c0 >= N) return;
    }
    if (FINAL && prev_keep) mark_kept(prev_keep, n_prev_keep, c0, CW, kept, &first);
    const int col = c0 + (tid % LPR) * V;
    const int r0 = blockIdx.y * rows_per;
    const int r1 = min(K, r0 + rows_per);
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.f;
    if (col < N) {                      // V > 1 is only launched with N % V == 0
        int r = r0 + tid / LPR;
        // all loads of a batch before its sums; in narrow pieces rows past the range repeat the last one
        // and are left out, in wide ones they are added one by one
        for (; r + (NARROW ? 0 : (UNROLL - 1) * RSTEP) < r1; r += UNROLL * RSTEP) {
            VT a[UNROLL], b[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int row = NARROW ? min(r + u * RSTEP, r1 - 1) : r + u * RSTEP;
                const size_t off = (size_t)row * (size_t)ld + (size_t)col;
                a[u] = *reinterpret_cast<const VT*>(Wt + off);
                b[u] = *reinterpret_cast<const VT*>(Wp + off);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                if (!NARROW || r + u * RSTEP < r1) accum<T, V>(reinterpret_cast<const T*>(&a[u]), reinterpret_cast<const T*>(&b[u]), acc);
        }
        for (; r < r1; r += RSTEP) {
            const size_t off = (size_t)r * (size_t)ld + (size_t)col;
            accum<T, V>(Wt + off, Wp + off, acc);
        }
    }
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] += __shfl_xor(acc[i], o, 64);
    if (lane < LPR) {
#pragma unroll
        for (int i = 0; i < V; ++i) part[wave][lane * V + i] = acc[i];
    }
    __syncthreads();
    for (int t = tid; t < CW; t += 1024) {
        const int c = c0 + t;
        if (c >= N) continue;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 16; ++w) sum += part[w][t];
        if (FINAL) out[c] = prev_keep && !kept[t] ? prev_scores[c] : sum / (float)K;
        else       out[(size_t)blockIdx.y * (size_t)N + c] = sum;
    }
}

// scores[c] from the per-range sums partial[n_split][N]: 64 columns a workgroup, each wavefront
// adds every sixteenth range, then their sums in wavefront order
__global__ __launch_bounds__(1024) void col_finish_kernel(
    const float* __restrict__ partial, int n_split, int K, int N,
    const float* __restrict__ prev_scores, const int32_t* __restrict__ prev_keep, int n_prev_keep,
    float* __restrict__ scores)
{
    __shared__ float part[16][64];
    __shared__ uint8_t kept[64];
    __shared__ int first;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = blockIdx.x * 64, c = c0 + lane;
    float sum = 0.f;
    for (int s = wave; s < n_split; s += 16) sum += partial[(size_t)s * (size_t)N + min(c, N - 1)];
    part[wave][lane] = sum;
    if (prev_keep) mark_kept(prev_keep, n_prev_keep, c0, 64, kept, &first);
    else __syncthreads();
    if (wave > 0 || c >= N) return;
    sum = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) sum += part[w][lane];
    scores[c] = prev_keep && !kept[lane] ? prev_scores[c] : sum / (float)K;
}

// Scores of the ROWS of W[K x N] (pruned axis = K): one wavefront per row, a
// lane adds its elements in column order, then a fixed shuffle tree.  A row that
// was pruned keeps its score and is not read.  SHORT: rows of at most three steps (without the
// batches' registers twice as many wavefronts are resident: 100000 x 16 bf16 18.1 -> 15.1 us).  A batch
// is requested before the sums of the one in front of it (64 x 32768 fp32 13.6 -> 11.2).
template <typename T, int V, bool SHORT>
__global__ __launch_bounds__(256) void row_scores_kernel(
    const T* __restrict__ Wt, const T* __restrict__ Wp, int64_t ld, int K, int N,
    const float* __restrict__ prev_scores, const int32_t* __restrict__ prev_keep, int n_prev_keep,
    float* __restrict__ scores)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= K) return;
    if (prev_keep) {
        const int at = lower_bound_wave(prev_keep, n_prev_keep, row, lane);
        if (at >= n_prev_keep || prev_keep[at] != row) {        // uniform
            if (lane == 0) scores[row] = prev_scores[row];
            return;
        }
    }
    const T* a = Wt + (size_t)row * (size_t)ld;
    const T* b = Wp + (size_t)row * (size_t)ld;
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.f;
    using VT = typename Vec<T, V>::type;
    int c = lane * V;                   // V > 1 is only launched with N % V == 0
    if constexpr (!SHORT) {
        // batches of loads, the next one requested before the sums of this one; steps past the row's end
        // repeat its last elements and are left out
        constexpr int U = V == 1 ? 8 : 4, STEP = U * 64 * V;
        VT x[2][U], y[2][U];
        auto request = [&](int buf, int64_t from) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int cc = (int)min<int64_t>(from + u * 64 * V, N - V);
                x[buf][u] = *reinterpret_cast<const VT*>(a + cc);
                y[buf][u] = *reinterpret_cast<const VT*>(b + cc);
            }
        };
        auto add = [&](int buf, int64_t from) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (from + u * 64 * V < N) accum<T, V>(reinterpret_cast<const T*>(&x[buf][u]), reinterpret_cast<const T*>(&y[buf][u]), acc);
        };
        request(0, c);
        for (int64_t at = c, base = 0; base < N; base += 2 * STEP, at += 2 * STEP) {
            request(1, at + STEP);
            __builtin_amdgcn_sched_barrier(0);
            add(0, at);
            request(0, at + 2 * STEP);
            __builtin_amdgcn_sched_barrier(0);
            add(1, at + STEP);
        }
        c = N;
    }
    for (; SHORT && c < N; c += 64 * V) accum<T, V>(a + c, b + c, acc);
    float sum = acc[0];
#pragma unroll
    for (int i = 1; i < V; ++i) sum += acc[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
    if (lane == 0) scores[row] = sum / (float)N;
}

__global__ __launch_bounds__(1024) void count_above_kernel(const float* __restrict__ scores, int n, float theta,
                                                           int32_t* __restrict__ count)
{
    __shared__ int wsum[16];
    int c = 0;
    for (int i = threadIdx.x; i < n; i += 1024) c += scores[i] > theta ? 1 : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < 16; ++w) t += wsum[w];
        *count = t;
    }
}

// Row ranges: of at least 256 rows, until there is one workgroup (of 64 times V columns) per
// compute unit.  Also what the scratch that callers are told to bring is sized by.
constexpr int kTargetBlocks = 256;
constexpr int kMinRowsPerSplit = 256;

template <int V> int col_splits(int K, int N)
{
    const int chunks = (N + 64 * V - 1) / (64 * V);
    const int by_rows = (K + kMinRowsPerSplit - 1) / kMinRowsPerSplit;
    const int want = (kTargetBlocks + chunks - 1) / chunks;
    return std::max(1, std::min(by_rows, want));
}

template <typename T, int V>
int cols_typed(const T* Wt, const T* Wp, int64_t ld, int K, int N, const float* prev_scores,
               const int32_t* prev_keep, int n_prev_keep, float* scores, void* workspace, size_t workspace_bytes,
               hipStream_t stream)
{
    int splits = V == 1 ? col_splits<1>(K, N) : col_splits<4>(K, N);
    const size_t fit = workspace ? workspace_bytes / ((size_t)N * sizeof(float)) : 0;   // row ranges the scratch holds
    if ((size_t)splits > fit) splits = fit < 2 ? 1 : (int)fit;
    // up to 4 MB a snapshot the second launch costs more than it gains (1024 x 1024 bf16 12.2 us, one launch 9.5)
    if (K <= 2048 && (int64_t)K * N * (int64_t)sizeof(T) <= (4 << 20)) splits = 1;
    constexpr int WIDE = V == 8 ? 32 : 64, NARROW = V == 1 ? 32 : 64 / (V * (int)sizeof(T));       // lanes to a row
    constexpr int WIDE_COLS = WIDE * V, NARROW_COLS = NARROW * V;
    const int chunks = (N + WIDE_COLS - 1) / WIDE_COLS;
    if (splits == 1) {
        // The narrow pieces while the wide ones are too few for the chip (us on 64 bytes / on 512 and more,
        // bf16: 4096 rows, 96 wide pieces 97 / 105, 125 120 / 105, 256 222 / 183; few rows are over at once: 16 rows,
        // 16384 pieces 912 / 67; fp32 300 rows, 64 pieces 12.7 / 9.4).  In wide pieces batches of four keep two workgroups
        // on a unit, and the range's last rows one by one.
        if (chunks >= 112 || (chunks >= 32 && K <= 512))
            hipLaunchKernelGGL((col_sums_kernel<T, V, WIDE, true>), dim3(chunks, 1), dim3(1024), 0, stream,
                               Wt, Wp, ld, K, N, K, prev_scores, prev_keep, n_prev_keep, scores);
        else
            hipLaunchKernelGGL((col_sums_kernel<T, V, NARROW, true>), dim3(((N + NARROW_COLS - 1) / NARROW_COLS + 7) / 8 * 8, 1),
                               dim3(1024), 0, stream, Wt, Wp, ld, K, N, K, prev_scores, prev_keep, n_prev_keep, scores);
        return hip_status(hipGetLastError());
    }
    const int rows_per = (((K + splits - 1) / splits) + 15) & ~15;
    splits = (K + rows_per - 1) / rows_per;
    float* partial = (float*)workspace;
    hipLaunchKernelGGL((col_sums_kernel<T, V, WIDE, false>), dim3(chunks, splits), dim3(1024), 0, stream,
                       Wt, Wp, ld, K, N, rows_per, prev_scores, prev_keep, n_prev_keep, partial);
    hipLaunchKernelGGL(col_finish_kernel, dim3((N + 63) / 64), dim3(1024), 0, stream,
                       partial, splits, K, N, prev_scores, prev_keep, n_prev_keep, scores);
    return hip_status(hipGetLastError());
}

template <typename T, int V>
int rows_typed(const T* Wt, const T* Wp, int64_t ld, int K, int N, const float* prev_scores,
               const int32_t* prev_keep, int n_prev_keep, float* scores, hipStream_t stream)
{
    auto fn = N <= 3 * 64 * V ? row_scores_kernel<T, V, true> : row_scores_kernel<T, V, false>;
    hipLaunchKernelGGL(fn, dim3((K + 3) / 4), dim3(256), 0, stream,
                       Wt, Wp, ld, K, N, prev_scores, prev_keep, n_prev_keep, scores);
    return hip_status(hipGetLastError());
}

// widest vector (in elements) both snapshots allow for every row start
template <typename T> int vec_width(const T* Wt, const T* Wp, int64_t ld, int N, int vmax)
{
    for (int v = vmax; v > 1; v >>= 1) {
        const uintptr_t bytes = (uintptr_t)v * sizeof(T);
        if (N % v == 0 && ld % v == 0 && (uintptr_t)Wt % bytes == 0 && (uintptr_t)Wp % bytes == 0) return v;
    }
    return 1;
}

}  // namespace

size_t priority_workspace_bytes(int K, int N, int mode)
{
    if (mode != ZR_DROP_N) return 0;
    // the widest column chunk leaves the fewest chunks, hence the most row ranges
    return (size_t)std::max(col_splits<1>(K, N), col_splits<4>(K, N)) * (size_t)N * sizeof(float);
}

int launch_priority_scores(const void* Wt, const void* Wp, int64_t ld, int K, int N, int mode,
                           const float* prev_scores, const int32_t* prev_keep, int n_prev_keep,
                           float* scores, int dtype, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
#define ZR_ARGS(T) (const T*)Wt, (const T*)Wp, ld, K, N, prev_scores, prev_keep, n_prev_keep, scores
    if (dtype == ZR_F32) {
        const int v = vec_width((const float*)Wt, (const float*)Wp, ld, N, 4);
        if (mode == ZR_DROP_N)
            return v == 4 ? cols_typed<float, 4>(ZR_ARGS(float), workspace, workspace_bytes, stream)
                          : cols_typed<float, 1>(ZR_ARGS(float), workspace, workspace_bytes, stream);
        return v == 4 ? rows_typed<float, 4>(ZR_ARGS(float), stream) : rows_typed<float, 1>(ZR_ARGS(float), stream);
    }
    const int v = vec_width((const uint16_t*)Wt, (const uint16_t*)Wp, ld, N, 8);
    if (mode == ZR_DROP_N)
        return v == 8 ? cols_typed<uint16_t, 8>(ZR_ARGS(uint16_t), workspace, workspace_bytes, stream)
             : v == 4 ? cols_typed<uint16_t, 4>(ZR_ARGS(uint16_t), workspace, workspace_bytes, stream)
                      : cols_typed<uint16_t, 1>(ZR_ARGS(uint16_t), workspace, workspace_bytes, stream);
    return v == 8 ? rows_typed<uint16_t, 8>(ZR_ARGS(uint16_t), stream)
         : v == 4 ? rows_typed<uint16_t, 4>(ZR_ARGS(uint16_t), stream)
                  : rows_typed<uint16_t, 1>(ZR_ARGS(uint16_t), stream);
#undef ZR_ARGS
}

int launch_priority_scores_static(const void* Wt, const void* Wp, int64_t ld, int K, int N, int mode,
                                  const float* prev_scores, const int32_t* prev_keep, int n_prev_keep,
                                  float* scores, int dtype, hipStream_t stream)
{
    if (priority_workspace_bytes(K, N, mode) > kStaticScratchBytes) return ZR_ERR_LIMIT;
    void* ws = nullptr;
    if (mode == ZR_DROP_N) {                    // row scores use no scratch
        const int st = static_scratch(&ws);
        if (st != ZR_OK) return st;
    }
    // every slot of the scratch that the finishing kernel reads is written by the summing
    // kernel of the same call first: nothing has to be cleared between calls
    return launch_priority_scores(Wt, Wp, ld, K, N, mode, prev_scores, prev_keep, n_prev_keep, scores, dtype,
                                  ws, ws ? kStaticScratchBytes : 0, stream);
}

size_t priority_static_scratch_bytes() { return kStaticScratchBytes; }

int launch_count_above(const float* scores, int n, float theta, int32_t* count, hipStream_t stream)
{
    hipLaunchKernelGGL(count_above_kernel, dim3(1), dim3(1024), 0, stream, scores, n, theta, count);
    return hip_status(hipGetLastError());
}

}  // namespace zr
