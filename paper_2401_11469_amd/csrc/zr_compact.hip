// Extraction of the kept columns of an ACTIVATION tensor into a caller-provided
// workspace (the pruned input / pruned upstream gradient of paper Sec. 3.1: the
// kept columns side by side, in ascending index order).  Only activations are ever
// extracted; the weight shard is always gathered in flight by the GEMM loaders.
//
//   out[m, q] = in[m, S[q]]   for q <  n_keep
//   out[m, q] = +0            for n_keep <= q < width   (width = n_keep rounded up to 64)
//
// bf16 only (the fp32 path does not use it).  HBM-bound: reads M x n, writes
// M x width.  Main kernel: a workgroup brings a few whole rows into LDS with
// 16-byte loads (every byte of a touched line is fetched anyway: at the pruning
// ratios of interest the kept columns touch every 128-byte line), picks the kept
// elements out of LDS two at a time and stores dwords, 256 contiguous bytes per
// wavefront.  Fallback (rows that are not 16-byte aligned, or too long for LDS):
// one output dword is assembled from the two aligned input dwords that hold its
// elements with one byte permute.
#include "zr_common.h"

namespace zr {

namespace {

constexpr int CROWS = 8;   // rows per workgroup

__global__ __launch_bounds__(256) void compact_cols_kernel(
    const uint16_t* __restrict__ in, int64_t ld, int rows, int n,
    const int32_t* __restrict__ keep, int n_keep,
    uint16_t* __restrict__ out, int64_t ldo, int width)
{
    const int r0 = blockIdx.x * CROWS;
    const int nr = min(CROWS, rows - r0);
    for (int q = threadIdx.x; q < width / 2; q += 256) {
        const int c = 2 * q;
        const int a = clamp_idx(keep[min(c, n_keep - 1)], n);
        const int b = clamp_idx(keep[min(c + 1, n_keep - 1)], n);
        // byte selectors of v_perm: 0-3 from the first dword, 4-7 from the second, 0x0c -> 0x00
        const uint32_t lo = c < n_keep ? ((a & 1) ? 0x0302u : 0x0100u) : 0x0c0cu;
        const uint32_t hi = c + 1 < n_keep ? ((b & 1) ? 0x0706u : 0x0504u) : 0x0c0cu;
        const uint32_t sel = lo | (hi << 16);
        const uint16_t* p = in + (size_t)r0 * (size_t)ld;
        uint32_t* o = (uint32_t*)(out + (size_t)r0 * (size_t)ldo) + q;
        for (int r = 0; r < nr; ++r) {
            const uint32_t d0 = *(const uint32_t*)(p + (a & ~1));
            const uint32_t d1 = *(const uint32_t*)(p + (b & ~1));
            *o = __builtin_amdgcn_perm(d1, d0, sel);
            p += ld;
            o += ldo / 2;
        }
    }
}

// Rows staged through LDS: RB rows to a workgroup, up to 256 * KL chunks of 16 bytes each (rows 16-byte
// aligned).  Thread t owns the output dwords t, t + 256, ... of every row: a wavefront stores 256
// contiguous bytes and its LDS reads are ~5 bytes apart from lane to lane (8-byte stores with 4 reads per
// lane measured 15 % slower: more bank conflicts).  A copy in all but name, so what counts is that nothing
// stands between the requests: list entries and rows go out together, addresses need no division,
// and what lies past the kept count is read from a zero behind each row instead of under a branch.
// (8192 rows, us before and now: 2752 of which 2064 are kept 24.7 and 20.6, 4096 of 3072 31.7 and 25.7, 12288 of 7000
// 107 and 86; 65536 x 8192 all kept 599 and 437, 4.9 TB/s)
// QN: output dwords of a thread and row, for which it holds the list entries.
template <int KL, int RB, int QN>
__global__ __launch_bounds__(256) void compact_rows_lds_kernel(
    const uint16_t* __restrict__ in, int64_t ld, int rows, int n,
    const int32_t* __restrict__ keep, int n_keep,
    uint16_t* __restrict__ out, int64_t ldo, int width)
{
    extern __shared__ __align__(16) uint16_t stage[];
    const int tid = threadIdx.x, wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    const int r0 = blockIdx.x * RB;
    const int chunks = n >> 3, pitch = n + 8, nq = width >> 1;
    int a[QN], b[QN];
#pragma unroll
    for (int i = 0; i < QN; ++i) {
        const int c = 2 * (tid + 256 * i);
        a[i] = keep[min(c, n_keep - 1)];
        b[i] = keep[min(c + 1, n_keep - 1)];
    }
    uint4 v[RB][KL];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int k = 0; k < KL; ++k)
            v[r][k] = *(const uint4*)(in + (size_t)min(r0 + r, rows - 1) * (size_t)ld + min(tid + 256 * k, chunks - 1) * 8);
#pragma unroll
    for (int i = 0; i < QN; ++i) {
        const int c = 2 * (tid + 256 * i);
        a[i] = c < n_keep ? clamp_idx(a[i], n) : n;
        b[i] = c + 1 < n_keep ? clamp_idx(b[i], n) : n;
    }
    if (tid < RB) *(uint4*)(stage + tid * pitch + n) = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int k = 0; k < KL; ++k)
            if (tid + 256 * k < chunks) *(uint4*)(stage + r * pitch + (tid + 256 * k) * 8) = v[r][k];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        if (r0 + r >= rows) break;
        uint32_t* o = (uint32_t*)(out + (size_t)(r0 + r) * (size_t)ldo) + tid;
#pragma unroll
        for (int i = 0; i < QN; ++i) {
            if (wave0 + 256 * i >= nq) break;
            const uint32_t lo = stage[r * pitch + a[i]], hi = stage[r * pitch + b[i]];
            if (tid + 256 * i < nq) o[256 * i] = lo | (hi << 16);
        }
    }
}

}  // namespace

// width: multiple of 64, <= ldo; ld, ldo even; in/out 4-byte aligned; n even.
int launch_compact_cols(const void* in, int64_t ld, int rows, int n, const int32_t* keep, int n_keep,
                        void* out, int64_t ldo, int width, hipStream_t stream)
{
    // LDS-staged rows when every row can be read in 16-byte chunks and a few rows fit
    if ((uintptr_t)in % 16 == 0 && ld % 8 == 0 && n % 8 == 0 && n <= 12288) {
        // few rows to a workgroup, so that thousands of workgroups even out over the units
#define ZR_COMPACT(KL, RB, QN)                                                                                          \
        hipLaunchKernelGGL((compact_rows_lds_kernel<KL, RB, QN>), dim3((rows + RB - 1) / RB), dim3(256), (size_t)RB * (n + 8) * 2, stream, \
                           (const uint16_t*)in, ld, rows, n, keep, n_keep, (uint16_t*)out, ldo, width)
        // (of long rows that keep at most half, half the list: 3062 rows of 6360, 2448 kept, 13.3 us with all of it, 10.5 now)
        const int kl = (n / 8 + 255) / 256;
        const bool half = width <= 1024 * kl;
        if (kl <= 1) ZR_COMPACT(1, 4, 4); else if (kl == 2) ZR_COMPACT(2, 2, 8);
        else if (kl == 3) { if (half) ZR_COMPACT(3, 2, 6); else ZR_COMPACT(3, 2, 12); }
        else if (kl == 4) { if (half) ZR_COMPACT(4, 2, 8); else ZR_COMPACT(4, 2, 16); }
        else if (width <= 6144) ZR_COMPACT(6, 2, 12); else ZR_COMPACT(6, 2, 24);
#undef ZR_COMPACT
        return hip_status(hipGetLastError());
    }
    hipLaunchKernelGGL(compact_cols_kernel, dim3((rows + CROWS - 1) / CROWS), dim3(256), 0, stream,
                       (const uint16_t*)in, ld, rows, n, keep, n_keep, (uint16_t*)out, ldo, width);
    return hip_status(hipGetLastError());
}

}  // namespace zr
