// Priority selection: the n' highest-score indices, emitted ascending
// (Algorithm 1 of the paper: top-L_pri select, then ascending sort), plus the
// complementary pruned set P of the lineage tuple (Sec. 3.1).
//
// No sort is needed: a 4-pass MSB radix select finds the n'-th largest order
// key T and how many keys are strictly greater; one ordered pass over the
// indices then keeps every index whose key is > T and the first (by index) of
// those equal to T, writing kept and pruned indices by prefix position, which
// makes both lists ascending by construction.
//
// One workgroup per score vector.  Vectors of up to 32768 scores are turned into order keys once and kept in
// registers (select_regs), with as many threads as its length and the number of vectors ask for; longer ones
// re-read from memory, or go to many workgroups where the caller has scratch.
#include "zr_common.h"

namespace zr {

namespace {

constexpr int SEL_THREADS = 1024;      // a vector that no registers hold

// Monotone map fp32 -> uint32: larger score <=> larger key.  NaN -> 0 (lowest,
// below -inf); -0.0 and +0.0 share one key.
__device__ __forceinline__ uint32_t order_key(float s)
{
    uint32_t u = __float_as_uint(s);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;   // NaN
    if ((u & 0x7fffffffu) == 0u) u = 0u;              // -0.0 -> +0.0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int SEL_REG_KEYS = 32768;    // order keys in the registers of 1024 threads (twice as many spill)

// One workgroup of NT threads selects one score vector of up to NT * K scores, whose order keys it holds in
// registers.  What bounds it: barriers, and LDS counters that many lanes hit at once (the scores of one
// layer share their leading bits).  So
//   * the digits start at the highest bit in which any two keys differ, found with one reduction: they spread
//     over the 256 bins from the first one on, and the bits that all keys share take no pass;
//   * every pass has counters of its own, cleared at the start, and every wavefront picks the digit for
//     itself: one barrier a pass;
//   * the ordered pass counts all of its chunks before one barrier instead of two barriers a chunk.
// us a launch, before and now (norms of a layer's columns; 256-thread workgroups, keys in LDS before): 256 scores 5.2 and
// 4.5, four vectors of up to 1024 6.7 and 5.0, five of up to 3072 11.6 and 6.4, 12000 and 8000 33.7 and 12.6;
// 4096 vectors of 4096 112 and 46, of 700 26 and 15, 1000 of 9000 82 and 36.
template <int K, int NT>
__device__ __forceinline__ void select_regs(const float* __restrict__ s, int n, int n_keep,
                                            int32_t* __restrict__ keep, int32_t* __restrict__ drop)
{
    constexpr int WAVES = NT / 64, CH = 64 / WAVES;     // CH: chunks whose counts one wavefront adds up at a time
    static_assert(1024 % NT == 0 && NT >= 64, "the counters are cleared 1024 / NT words a thread");
    __shared__ __align__(16) uint32_t hist[4][256];
    __shared__ uint32_t wave_lo[WAVES], wave_hi[WAVES];
    __shared__ uint32_t counts[2][K * WAVES];           // greater, equal: chunk by chunk, wavefront by wavefront
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    uint32_t key[K];
#pragma unroll
    for (int q = 0; q < 1024 / NT; ++q) ((uint32_t*)hist)[tid + NT * q] = 0;
    uint32_t lo = 0xffffffffu, hi = 0;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += 16) {
        float v[16];
#pragma unroll
        for (int k = k0; k < k0 + 16 && k < K; ++k) v[k - k0] = s[min(tid + NT * k, n - 1)];
#pragma unroll
        for (int k = k0; k < k0 + 16 && k < K; ++k) {
            key[k] = order_key(v[k - k0]);               // (past the end: the last key again)
            lo = min(lo, key[k]);
            hi = max(hi, key[k]);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off, 64));
    }
    if (lane == 0) { wave_lo[wave] = lo; wave_hi[wave] = hi; }
    __syncthreads();
    lo = wave_lo[lane & (WAVES - 1)];
    hi = wave_hi[lane & (WAVES - 1)];
#pragma unroll
    for (int off = WAVES / 2; off > 0; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off, 64));
    }
    // ---- radix select of the n_keep-th largest key over the bits below `top` ----
    const int top = 32 - __clz((int)(lo ^ hi));          // 0: all keys are equal
    uint32_t prefix = top >= 32 ? 0u : hi >> top << top, mask = top >= 32 ? 0u : ~0u << top;
    uint32_t remaining = (uint32_t)n_keep;
    int shift = top;
    for (int pass = 0; shift > 0; ++pass) {              // (at most four)
        shift = max(shift - 8, 0);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (tid + NT * k < n && (key[k] & mask) == prefix) atomicAdd(&hist[pass][(key[k] >> shift) & 255u & ~(mask >> shift)], 1u);
        __syncthreads();
        // lane l owns bins 4l .. 4l + 3; suffix sums give, for each bin, the number of candidates in
        // strictly higher bins
        const uint4 h4 = *(const uint4*)&hist[pass][4 * lane];
        const uint32_t h[4] = {h4.x, h4.y, h4.z, h4.w};
        const uint32_t mine = h[0] + h[1] + h[2] + h[3];
        uint32_t incl = mine;                            // inclusive suffix sum over lanes
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t x = __shfl_down(incl, off, 64);
            if (lane + off < 64) incl += x;
        }
        uint32_t above = incl - mine, digit = 0xffffffffu, rem = 0;
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            if (above < remaining && remaining <= above + h[q]) { digit = (uint32_t)(4 * lane + q); rem = remaining - above; }
            above += h[q];
        }
        const uint64_t who = __ballot(digit != 0xffffffffu);       // exactly one lane
        const int src = who ? (int)(__ffsll((long long)who) - 1) : 0;
        prefix |= (uint32_t)__shfl((int)digit, src, 64) << shift;
        remaining = (uint32_t)__shfl((int)rem, src, 64);
        mask = ~0u << shift;
    }
    const uint32_t T = prefix;          // the n_keep-th largest key
    const uint32_t need_eq = remaining; // how many of the keys == T are kept (>= 1)

    // ---- ordered compaction -----------------------------------------------
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool in = tid + NT * k < n;
        const uint32_t gt = (uint32_t)__popcll(__ballot(in && key[k] > T)), eq = (uint32_t)__popcll(__ballot(in && key[k] == T));
        if (lane == 0) { counts[0][k * WAVES + wave] = gt; counts[1][k * WAVES + wave] = eq; }
    }
    __syncthreads();
    // what lies before this wavefront's part of each chunk: 64 entries to a step, prefix sums over the lanes
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t run_gt = 0, run_eq = 0;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += CH) {
        const bool in = k0 * WAVES + lane < K * WAVES;
        const uint32_t g = in ? counts[0][k0 * WAVES + lane] : 0u, e = in ? counts[1][k0 * WAVES + lane] : 0u;
        uint32_t sg = g, se = e;                         // inclusive
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t a = __shfl_up(sg, off, 64), b = __shfl_up(se, off, 64);
            if (lane >= off) { sg += a; se += b; }
        }
#pragma unroll
        for (int k = k0; k < k0 + CH && k < K; ++k) {
            const int at = (k - k0) * WAVES + wave;
            const int i = tid + NT * k;
            const uint64_t bgt = __ballot(i < n && key[k] > T), beq = __ballot(i < n && key[k] == T);
            const uint32_t pg = run_gt + (uint32_t)__shfl((int)(sg - g), at, 64) + (uint32_t)__popcll(bgt & below);
            const uint32_t pe = run_eq + (uint32_t)__shfl((int)(se - e), at, 64) + (uint32_t)__popcll(beq & below);
            if (i < n) {
                const bool kept = key[k] > T || (key[k] == T && pe < need_eq);
                // kept indices before i: all greater ones plus the first need_eq equal ones
                const uint32_t kept_before = pg + (pe < need_eq ? pe : need_eq);
                // positions are in range by construction; the comparisons only make an
                // out-of-range store impossible whatever the scores hold
                if (kept) {
                    if (kept_before < (uint32_t)n_keep) keep[kept_before] = i;
                } else if (drop) {
                    const uint32_t pos = (uint32_t)i - kept_before;
                    if (pos < (uint32_t)(n - n_keep)) drop[pos] = i;
                }
            }
        }
        run_gt += (uint32_t)__shfl((int)sg, 63, 64);
        run_eq += (uint32_t)__shfl((int)se, 63, 64);
    }
}

// The same for a vector of any length, read from memory in every pass.
template <int NT>
__device__ __forceinline__ void select_body(const float* __restrict__ s, int n, int n_keep,
                                            int32_t* __restrict__ keep, int32_t* __restrict__ drop)
{
    constexpr int SEL_WAVES = NT / 64;
    static_assert(NT >= 256 && NT % 64 == 0, "the histogram is cleared by the first 256 threads");
    __shared__ uint32_t hist[256];
    __shared__ uint32_t s_digit, s_remaining;
    __shared__ uint32_t wave_gt[SEL_WAVES], wave_eq[SEL_WAVES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;

    auto key_at = [&](int i) -> uint32_t { return order_key(s[i]); };

    // ---- radix select of the n_keep-th largest key -------------------------
    uint32_t prefix = 0, mask = 0, remaining = (uint32_t)n_keep;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int i = tid; i < n; i += NT) {
            const uint32_t k = key_at(i);
            if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (wave == 0) {
            // lane l owns bins 4l..4l+3; suffix sums give, for each bin, the
            // number of candidates in strictly higher bins
            uint32_t h[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) h[q] = hist[4 * lane + q];
            const uint32_t mine = h[0] + h[1] + h[2] + h[3];
            uint32_t incl = mine;                       // inclusive suffix sum over lanes
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t v = __shfl_down(incl, off, 64);
                if (lane + off < 64) incl += v;
            }
            uint32_t above = incl - mine;               // candidates in lanes > this one
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                if (above < remaining && remaining <= above + h[q]) {
                    s_digit = (uint32_t)(4 * lane + q);
                    s_remaining = remaining - above;
                }
                above += h[q];
            }
        }
        __syncthreads();
        prefix |= s_digit << shift;
        mask |= 0xffu << shift;
        remaining = s_remaining;
        __syncthreads();
    }
    const uint32_t T = prefix;          // the n_keep-th largest key
    const uint32_t need_eq = remaining; // how many of the keys == T are kept (>= 1)

    // ---- ordered compaction -----------------------------------------------
    uint32_t run_gt = 0, run_eq = 0;    // totals over all earlier chunks
    for (int base = 0; base < n; base += NT) {
        const int i = base + tid;
        bool gt = false, eq = false;
        if (i < n) {
            const uint32_t k = key_at(i);
            gt = k > T;
            eq = k == T;
        }
        const uint64_t bgt = __ballot(gt);
        const uint64_t beq = __ballot(eq);
        const uint64_t below = (1ull << lane) - 1ull;
        if (lane == 0) {
            wave_gt[wave] = (uint32_t)__popcll(bgt);
            wave_eq[wave] = (uint32_t)__popcll(beq);
        }
        __syncthreads();
        uint32_t pre_gt = run_gt + (uint32_t)__popcll(bgt & below);
        uint32_t pre_eq = run_eq + (uint32_t)__popcll(beq & below);
        uint32_t tot_gt = 0, tot_eq = 0;
#pragma unroll
        for (int w = 0; w < SEL_WAVES; ++w) {
            const uint32_t g = wave_gt[w], e = wave_eq[w];
            if (w < wave) { pre_gt += g; pre_eq += e; }
            tot_gt += g;
            tot_eq += e;
        }
        if (i < n) {
            const bool kept = gt || (eq && pre_eq < need_eq);
            // kept indices before i: all greater ones plus the first need_eq equal ones
            const uint32_t kept_before = pre_gt + (pre_eq < need_eq ? pre_eq : need_eq);
            // positions are in range by construction; the comparisons only make
            // an out-of-range store impossible whatever the scores hold
            if (kept) {
                if (kept_before < (uint32_t)n_keep) keep[kept_before] = i;
            } else if (drop) {
                const uint32_t pos = (uint32_t)i - kept_before;
                if (pos < (uint32_t)(n - n_keep)) drop[pos] = i;
            }
        }
        run_gt += tot_gt;
        run_eq += tot_eq;
        __syncthreads();
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void select_kernel(
    const float* __restrict__ scores, int n, int n_keep,
    int32_t* __restrict__ keep_idx, int32_t* __restrict__ drop_idx, int64_t ld_idx)
{
    select_body<NT>(scores + (size_t)blockIdx.x * (size_t)n, n, n_keep,
                        keep_idx + (size_t)blockIdx.x * (size_t)ld_idx,
                        drop_idx ? drop_idx + (size_t)blockIdx.x * (size_t)ld_idx : nullptr);
}

template <int K, int NT>
__global__ __launch_bounds__(NT) void select_regs_kernel(
    const float* __restrict__ scores, int n, int n_keep,
    int32_t* __restrict__ keep_idx, int32_t* __restrict__ drop_idx, int64_t ld_idx)
{
    select_regs<K, NT>(scores + (size_t)blockIdx.x * (size_t)n, n, n_keep, keep_idx + (size_t)blockIdx.x * (size_t)ld_idx,
                   drop_idx ? drop_idx + (size_t)blockIdx.x * (size_t)ld_idx : nullptr);
}

// Several vectors of different lengths in one launch (the projections of a layer
// shard): workgroup b takes descriptor b.  The descriptors travel as a kernel
// argument, no device memory is involved.  K: chunks of NT scores of the longest; 0: longer than registers hold.
template <int K, int NT>
__global__ __launch_bounds__(NT) void select_multi_kernel(const SelectMulti m)
{
    const int b = blockIdx.x;
    if constexpr (K == 0) select_body<NT>(m.scores[b], m.n[b], m.n_keep[b], m.keep[b], m.drop[b]);
    else select_regs<K, NT>(m.scores[b], m.n[b], m.n_keep[b], m.keep[b], m.drop[b]);
}

// ---------------------------------------------------------------------------
// One long vector on many workgroups (with scratch from the caller).  The same
// selection as select_body, cut into launches; every launch reads the vector once:
//   clear     the global histograms of three digits (11, 11 and 10 bits of the key)
//   hist p    (p = 0..2) each workgroup histograms digit p of the keys of its share that
//             match the digits chosen so far, in LDS, then adds its counters to the global
//             histogram of the pass; the digit of the pass before is chosen first, by every
//             workgroup for itself, from that pass's global histogram
//   count     the last digit gives T and how many keys equal to T are kept; each
//             WAVEFRONT counts the keys > T and == T of its slice
//   write     each workgroup adds up the counts before its own; then the ordered pass, each
//             wavefront on its own slice with no barrier: position = the counts before it + the
//             position inside it
// All counters are integers (order-free); the lists are the same, bit for bit, as
// those of the single-workgroup kernel.
// What bounds it: launches of a few microseconds that wait for memory, so the vector is cut into
// as many slices as there is room for counts (256 scores and more), and a digit is as wide as its
// histogram in LDS allows.  395264 scores, against four 8-bit digits, slices of 4096 scores and a
// launch for the prefix sums: 50 -> 24 us (write 19.4 -> 5.4); 2^24 scores: 115 -> 99 us.
// Scratch (uint32 words): [0, 5120) histograms; [5120, 5128) {prefix, wanted} after each digit;
// then gt count, eq count: 2 x WIDE_MAX_GROUPS.
// ---------------------------------------------------------------------------
constexpr int WIDE_THREADS = 256;
constexpr int WIDE_SLICE = 16384;                              // scores that make a vector worth these launches, an eighth
constexpr int WIDE_MAX_GROUPS = 4096;                          // wavefronts with counts
constexpr int WIDE_UNIT = 256;                                 // scores per wavefront: multiples of this
constexpr int WIDE_STATE = 5120;
constexpr int WIDE_COUNTS = 5128;
constexpr size_t WIDE_WORDS = 1032 + 4 * (size_t)WIDE_MAX_GROUPS;      // (more than is used; callers keep such buffers)
static_assert(WIDE_COUNTS + 2 * WIDE_MAX_GROUPS <= WIDE_WORDS, "the scratch");
constexpr int WIDE_COPIES = 4;                                 // copies of the LDS histogram
typedef uint32_t u4_words __attribute__((ext_vector_type(4), aligned(4)));      // 16 bytes at any word

__host__ __device__ constexpr int wide_bits(int pass) { return pass < 2 ? 11 : 10; }
__host__ __device__ constexpr int wide_shift(int pass) { return pass == 0 ? 21 : pass == 1 ? 10 : 0; }

// The first wavefront of a workgroup picks the digit of a pass from its global counters: the bin
// that holds the `remaining`-th largest candidate (bins taken from the top), and how many
// candidates of that bin are still wanted.  Every lane returns the result.
template <int BINS>
__device__ __forceinline__ void wide_pick(const uint32_t* __restrict__ hist, uint32_t remaining, int lane,
                                          uint32_t& digit, uint32_t& remaining_out)
{
    constexpr int PER = BINS / 64;
    uint32_t h[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < PER; q += 4) {
        const u4_words v = *(const u4_words*)(hist + PER * lane + q);
        h[q] = v.x; h[q + 1] = v.y; h[q + 2] = v.z; h[q + 3] = v.w;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) mine += h[q];
    uint32_t incl = mine;                       // inclusive suffix sum over lanes
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = __shfl_down(incl, off, 64);
        if (lane + off < 64) incl += v;
    }
    uint32_t above = incl - mine;
    uint32_t d = 0xffffffffu, r = 0;
#pragma unroll
    for (int q = PER - 1; q >= 0; --q) {
        if (above < remaining && remaining <= above + h[q]) { d = (uint32_t)(PER * lane + q); r = remaining - above; }
        above += h[q];
    }
    // exactly one lane found it
    const uint64_t who = __ballot(d != 0xffffffffu);
    const int src = who ? (int)(__ffsll((long long)who) - 1) : 0;
    digit = __shfl(d, src, 64);
    remaining_out = __shfl(r, src, 64);
}

// Prefix of the wanted key and candidates still wanted before pass PASS (3: T itself and how many
// keys equal to it are kept), for the whole workgroup; block 0 leaves them for the next launch.
template <int PASS>
__device__ __forceinline__ void wide_state(uint32_t* __restrict__ ws, uint32_t n_keep, uint32_t* shared2,
                                           uint32_t& prefix, uint32_t& remaining)
{
    prefix = 0; remaining = n_keep;
    if constexpr (PASS > 0) {
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            uint32_t before = 0, wanted = n_keep;
            if constexpr (PASS > 1) { before = ws[WIDE_STATE + 2 * (PASS - 1)]; wanted = ws[WIDE_STATE + 2 * (PASS - 1) + 1]; }
            uint32_t digit, rem;
            wide_pick<1 << wide_bits(PASS - 1)>(ws + 2048 * (PASS - 1), wanted, lane, digit, rem);
            before |= digit << wide_shift(PASS - 1);
            if (lane == 0) {
                shared2[0] = before; shared2[1] = rem;
                if (blockIdx.x == 0) { ws[WIDE_STATE + 2 * PASS] = before; ws[WIDE_STATE + 2 * PASS + 1] = rem; }
            }
        }
        __syncthreads();
        prefix = shared2[0]; remaining = shared2[1];
    }
}

__global__ __launch_bounds__(1024) void wide_clear_kernel(uint32_t* __restrict__ ws)
{
#pragma unroll
    for (int q = 0; q < 5; ++q) ws[threadIdx.x + 1024 * q] = 0;
}

// At most one workgroup of 1024 threads per compute unit, each on a contiguous share of the vector
// (every workgroup adds its counters to the global ones: more of them, more atomic additions).
constexpr int WIDE_HIST_THREADS = 1024;
constexpr int WIDE_HIST_GROUPS = 256;

template <int PASS>
__global__ __launch_bounds__(WIDE_HIST_THREADS) void wide_hist_kernel(const float* __restrict__ s, int n, int n_keep,
                                                                      uint32_t* __restrict__ ws, int share)
{
    // WIDE_COPIES counters per bin, side by side: lanes that hit the same bin (scores cluster in a
    // few exponents, so the first digit has a handful of busy bins) spread over as many addresses
    constexpr int BINS = 1 << wide_bits(PASS);
    __shared__ __align__(16) uint32_t hist[BINS * WIDE_COPIES];
    __shared__ uint32_t state[2];
    const int tid = threadIdx.x, lane = tid & 63;
    for (int q = tid; q < BINS * WIDE_COPIES; q += WIDE_HIST_THREADS) hist[q] = 0;
    uint32_t prefix, remaining;
    wide_state<PASS>(ws, (uint32_t)n_keep, state, prefix, remaining);
    __syncthreads();
    constexpr int shift = wide_shift(PASS);
    constexpr uint32_t mask = PASS == 0 ? 0u : ~0u << wide_shift(PASS > 0 ? PASS - 1 : 0);
    const int copy = lane & (WIDE_COPIES - 1);
    const int64_t lo64 = (int64_t)blockIdx.x * share;
    const int lo = (int)min<int64_t>(lo64, n), hi = (int)min<int64_t>(lo64 + share, n);
    for (int i0 = lo + tid; i0 < hi; i0 += 8 * WIDE_HIST_THREADS) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = s[min(i0 + q * WIDE_HIST_THREADS, hi - 1)];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t k = order_key(v[q]);
            if (i0 + q * WIDE_HIST_THREADS < hi && (k & mask) == prefix)
                atomicAdd(&hist[((k >> shift) & (BINS - 1)) * WIDE_COPIES + copy], 1u);
        }
    }
    __syncthreads();
    for (int b = tid; b < BINS; b += WIDE_HIST_THREADS) {
        const uint4 c = *(const uint4*)(hist + b * WIDE_COPIES);
        const uint32_t mine = c.x + c.y + c.z + c.w;
        if (mine) atomicAdd(&ws[2048 * PASS + b], mine);
    }
}

__global__ __launch_bounds__(WIDE_THREADS) void wide_count_kernel(const float* __restrict__ s, int n, int n_keep,
                                                                  uint32_t* __restrict__ ws, int slice)
{
    __shared__ uint32_t state[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t T, need_eq;
    wide_state<3>(ws, (uint32_t)n_keep, state, T, need_eq);
    const int group = blockIdx.x * (WIDE_THREADS / 64) + wave;
    const int lo = (int)min<int64_t>((int64_t)group * slice, n), hi = (int)min<int64_t>((int64_t)lo + slice, n);
    uint32_t gt = 0, eq = 0;
    for (int i0 = lo + lane; i0 < hi; i0 += 4 * 64) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = s[min(i0 + q * 64, hi - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t k = order_key(v[q]);
            if (i0 + q * 64 < hi) { gt += k > T; eq += k == T; }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { gt += __shfl_down(gt, off, 64); eq += __shfl_down(eq, off, 64); }
    if (lane == 0 && lo < n) {
        ws[WIDE_COUNTS + group] = gt;
        ws[WIDE_COUNTS + WIDE_MAX_GROUPS + group] = eq;
    }
}

__global__ __launch_bounds__(WIDE_THREADS) void wide_write_kernel(const float* __restrict__ s, int n, int n_keep,
                                                                  const uint32_t* __restrict__ ws, int slice,
                                                                  int32_t* __restrict__ keep, int32_t* __restrict__ drop)
{
    constexpr int WAVES = WIDE_THREADS / 64;
    __shared__ uint32_t sum_gt[WAVES], sum_eq[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the counts of all wavefronts before this workgroup's
    const int first = blockIdx.x * WAVES;
    uint32_t bg = 0, be = 0;
    for (int j = tid; j < first; j += WIDE_THREADS) {
        bg += ws[WIDE_COUNTS + j];
        be += ws[WIDE_COUNTS + WIDE_MAX_GROUPS + j];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { bg += __shfl_down(bg, off, 64); be += __shfl_down(be, off, 64); }
    if (lane == 0) { sum_gt[wave] = bg; sum_eq[wave] = be; }
    __syncthreads();
    const int group = first + wave;
    const int64_t lo64 = (int64_t)group * slice;
    if (lo64 >= n) return;
    const int lo = (int)lo64, hi = (int)min<int64_t>(lo64 + slice, n);
    const uint32_t T = ws[WIDE_STATE + 6], need_eq = ws[WIDE_STATE + 7];
    uint32_t run_gt = 0, run_eq = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { run_gt += sum_gt[w]; run_eq += sum_eq[w]; }
    for (int w = 0; w < wave; ++w) {
        run_gt += ws[WIDE_COUNTS + first + w];
        run_eq += ws[WIDE_COUNTS + WIDE_MAX_GROUPS + first + w];
    }
    const uint64_t below = (1ull << lane) - 1ull;
    for (int base = lo; base < hi; base += 4 * 64) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = s[min(base + q * 64 + lane, hi - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = base + q * 64 + lane;
            const uint32_t k = order_key(v[q]);
            const bool in = i < hi;
            const bool gt = in && k > T, eq = in && k == T;
            const uint64_t bgt = __ballot(gt);
            const uint64_t beq = __ballot(eq);
            const uint32_t pre_gt = run_gt + (uint32_t)__popcll(bgt & below);
            const uint32_t pre_eq = run_eq + (uint32_t)__popcll(beq & below);
            if (in) {
                const bool kept = gt || (eq && pre_eq < need_eq);
                const uint32_t kept_before = pre_gt + (pre_eq < need_eq ? pre_eq : need_eq);
                // (in range by construction; the comparisons make an out-of-range store impossible)
                if (kept) {
                    if (kept_before < (uint32_t)n_keep) keep[kept_before] = i;
                } else if (drop) {
                    const uint32_t pos = (uint32_t)i - kept_before;
                    if (pos < (uint32_t)(n - n_keep)) drop[pos] = i;
                }
            }
            run_gt += (uint32_t)__popcll(bgt);
            run_eq += (uint32_t)__popcll(beq);
        }
    }
}

__global__ void clear_flag_kernel(int32_t* flag) { *flag = 0; }

__global__ void validate_kernel(const int32_t* __restrict__ keep_idx, int n_keep, int n,
                                int32_t* __restrict__ flag)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_keep) return;
    const int v = keep_idx[i];
    bool bad = v < 0 || v >= n;
    if (i > 0 && keep_idx[i - 1] >= v) bad = true;
    if (bad) atomicOr(flag, 1);
}

}  // namespace

int launch_select(const float* scores, int n, int batch, int n_keep,
                  int32_t* keep_idx, int32_t* drop_idx, int64_t ld_idx, hipStream_t stream)
{
    if (n > SEL_REG_KEYS)
        hipLaunchKernelGGL((select_kernel<SEL_THREADS>), dim3(batch), dim3(SEL_THREADS), 0, stream,
                           scores, n, n_keep, keep_idx, drop_idx, ld_idx);
    else {
#define ZR_SELECT(K, NT) hipLaunchKernelGGL((select_regs_kernel<K, NT>), dim3(batch), dim3(NT), 0, stream, scores, n, n_keep, keep_idx, drop_idx, ld_idx)
        // few wavefronts for short vectors: each of them repeats the pick of a digit
        // (and, where the chip is full, little more room than the vector fills: what lies past its end costs as much as
        // scores.  3104 vectors of 4397 on 512 threads of 24 108 us, on 256 of 24 64; 2366 of 1339 on 256 of 16 27, of 8 21)
        if (batch >= 512) {
            if (n <= 1024) ZR_SELECT(16, 64); else if (n <= 2048) ZR_SELECT(8, 256); else if (n <= 4096) ZR_SELECT(16, 256); else if (n <= 6144) ZR_SELECT(24, 256);
            else if (n <= 8192) ZR_SELECT(16, 512); else if (n <= 12288) ZR_SELECT(24, 512); else ZR_SELECT(32, 1024);
        }
        else if (n <= 1024) ZR_SELECT(4, 256); else if (n <= 4096) ZR_SELECT(8, 512); else if (n <= 12288) ZR_SELECT(12, 1024); else ZR_SELECT(32, 1024);
#undef ZR_SELECT
    }
    return hip_status(hipGetLastError());
}

size_t select_wide_workspace_bytes() { return WIDE_WORDS * sizeof(uint32_t); }

// shortest vector that goes to the many-workgroup path (below it the launches cost more
// than the single workgroup's passes)
int select_wide_min_n() { return 8 * WIDE_SLICE; }

int launch_select_wide(const float* scores, int n, int n_keep, int32_t* keep_idx, int32_t* drop_idx,
                       void* workspace, hipStream_t stream)
{
    uint32_t* ws = (uint32_t*)workspace;
    // scores per wavefront of the last two launches
    const int slice = (int)(((int64_t)n + (int64_t)WIDE_MAX_GROUPS * WIDE_UNIT - 1) / ((int64_t)WIDE_MAX_GROUPS * WIDE_UNIT)) * WIDE_UNIT;
    const int groups = (n + slice - 1) / slice, blocks = (groups + WIDE_THREADS / 64 - 1) / (WIDE_THREADS / 64);
    if (groups > WIDE_MAX_GROUPS) return ZR_ERR_LIMIT;
    hipLaunchKernelGGL(wide_clear_kernel, dim3(1), dim3(1024), 0, stream, ws);
    // (shares of 4096 scores and more)
    const int hist_groups = std::min(WIDE_HIST_GROUPS, (n + 4095) / 4096);
    const int share = (n + hist_groups - 1) / hist_groups;
    hipLaunchKernelGGL(wide_hist_kernel<0>, dim3(hist_groups), dim3(WIDE_HIST_THREADS), 0, stream, scores, n, n_keep, ws, share);
    hipLaunchKernelGGL(wide_hist_kernel<1>, dim3(hist_groups), dim3(WIDE_HIST_THREADS), 0, stream, scores, n, n_keep, ws, share);
    hipLaunchKernelGGL(wide_hist_kernel<2>, dim3(hist_groups), dim3(WIDE_HIST_THREADS), 0, stream, scores, n, n_keep, ws, share);
    hipLaunchKernelGGL(wide_count_kernel, dim3(blocks), dim3(WIDE_THREADS), 0, stream, scores, n, n_keep, ws, slice);
    hipLaunchKernelGGL(wide_write_kernel, dim3(blocks), dim3(WIDE_THREADS), 0, stream, scores, n, n_keep,
                       (const uint32_t*)ws, slice, keep_idx, drop_idx);
    return hip_status(hipGetLastError());
}

int launch_select_multi(const SelectMulti& m, int count, hipStream_t stream)
{
    int longest = 0;
    for (int b = 0; b < count; ++b) longest = std::max(longest, m.n[b]);
#define ZR_SELECT(K, NT) hipLaunchKernelGGL((select_multi_kernel<K, NT>), dim3(count), dim3(NT), 0, stream, m)
    if (longest <= 1024) ZR_SELECT(4, 256); else if (longest <= 4096) ZR_SELECT(8, 512); else if (longest <= 12288) ZR_SELECT(12, 1024); else if (longest <= SEL_REG_KEYS) ZR_SELECT(32, 1024);
    else ZR_SELECT(0, 1024);
#undef ZR_SELECT
    return hip_status(hipGetLastError());
}

int launch_validate(const int32_t* keep_idx, int n_keep, int n, int32_t* flag, hipStream_t stream)
{
    // the flag is cleared by a kernel, not by a memset node
    hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, stream, flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return ZR_ERR_HIP;
    const int threads = 256;
    hipLaunchKernelGGL(validate_kernel, dim3((n_keep + threads - 1) / threads), dim3(threads), 0,
                       stream, keep_idx, n_keep, n, flag);
    e = hipGetLastError();
    if (e != hipSuccess) return ZR_ERR_HIP;
    int32_t host = 0;
    e = hipMemcpyAsync(&host, flag, sizeof(int32_t), hipMemcpyDeviceToHost, stream);
    if (e != hipSuccess) return ZR_ERR_HIP;
    e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return ZR_ERR_HIP;
    return host ? ZR_ERR_INDEX : ZR_OK;
}

}  // namespace zr
