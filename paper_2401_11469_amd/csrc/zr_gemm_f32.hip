// Gather-fused MFMA products of fp32 tensors (gfx950): the resized layer's forward, dX and dW
// (paper Sec. 3.1) in the canonical form
//     D[i, j] = sum_c A(i, c) * B(j, c)
// with v_mfma_f32_32x32x2f32, for tensors of any alignment and any extents.
//
// What bounds it.  The fp32 matrix rate is 256 FLOP per clock and compute unit, a sixteenth of
// the bf16 rate, so even a 64 x 64 tile asks for only 16 bytes per clock from L2 and its LDS
// reads are a small fraction of the LDS rate.  What costs time is a chip that is not full and
// loads that are waited for.  Hence small tiles, deep stages and several workgroups to a unit:
//   R = 128: 128 x 128 tiles, 32 contraction indices a stage, a 64 x 64 result per wavefront: for
//           products with many tiles (half the LDS reads and half the operand bytes per FLOP);
//   R = 64: 64 x 64 tiles, 64 contraction indices a stage, a 32 x 32 result per wavefront;
//   R = 32: 32 x 32 tiles, 128 contraction indices a stage, of which each of the four
//           wavefronts multiplies a quarter; their four sums are added in wavefront order in
//           LDS.  For products with few tiles: four times as many workgroups, half the stages.
// All bring 16 KB of each operand per stage (four 16-byte loads or sixteen element loads a
// thread, in flight for a whole stage of multiplications) and use 72 KB of LDS, so that two
// workgroups share a compute unit.
// Measured against the kernel before this one (128 x 128 tiles, 32 deep, element loads under
// branches): 1576 x 1024 x 1640 plain 94 -> 66 us, with the kept list on the contraction
// 222 -> 72 us, 256 x 512 x 192 in four launches 132 -> 30 us.  Products with many tiles, 8192 x 4096
// results (us before / on 64 x 64 tiles / on 128 x 128): contraction 1024, dW 633 / 683 / 580, forward
// 599 / 619 / 553; contraction 64, kept columns of W gathered 83 / 121 / 79; contraction 8, accumulating
// 62 / 88 / 56.  4096^3 takes 998 us on P x P and 1090 on P x Q (1074 and
// 1220 on 64 x 64 tiles; 138 and 126 TFLOP/s, 0.88 and 0.80 of the fp32 matrix peak).  Of a launch
// 10-13 us are start and end (all tiles of a round end together); a chip full of tiles keeps the
// matrix pipes at 0.9 in between, so what is left is that, and the rounding of the tile count to
// the compute units.
//
// LDS formats (32-bit words):
//   P  [row][contraction]  tensors whose contiguous axis is the contraction axis
//   Q  [contraction][row]  tensors whose contiguous axis is the other one
// The order in which the contraction is added up is free as long as both operands agree: of a
// block of 8 indices, lanes 0-31 take indices 0-3 and lanes 32-63 indices 4-7, so a P operand
// is read with one ds_read_b128 per four MFMAs.
#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "zr_common.h"

namespace zr {

namespace {

constexpr int NT = 256;
constexpr int NP = 4;            // pieces a stage is brought in: 16 bytes of each operand per thread

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));     // 16 bytes at any element address

template <int R> struct Geo {
    static constexpr int BK = 16 * NT / R;                // contraction depth of a stage: 32, 64 or 128
    static constexpr int PP = BK + 4;                     // row pitch of format P: 16 rows of a fragment read on 16 bank groups
    static constexpr int PQ = R == 32 ? 36 : R + 8;       // row pitch of format Q: rows 4 apart (the two lane halves) on other banks
    static constexpr int WORDS = R * PP > BK * PQ ? R * PP : BK * PQ;      // LDS words of one operand's stage
};

struct View {
    const float* base;
    int64_t ld;
    const int32_t* map_s;       // row list on the strided axis or nullptr
    const int32_t* map_c;       // kept list on the contiguous axis or nullptr (the gathering loaders)
    int n_s, n_c;               // memory extents
};

struct Args {
    View A, B;
    int I, J, C;
    float* out;
    int64_t ldo;
    int epilogue;
    const int32_t* keep;
    int out_full;
    int tiles_i, tiles_j;
    const float* prev;          // Same imputation source (layout of out) or nullptr
    int accumulate;             // add the old contents of out (plain epilogue)
};

// ---------------------------------------------------------------------------
// Loaders.  Each keeps one stage of its operand in registers (begin, then fetch of four pieces)
// and writes it to LDS a stage later (commit, piece by piece).  Rows of the tile beyond the
// operand's extent repeat its last row (they only feed results that are never stored);
// contraction indices past C become zero (commit with TAIL, which only the last stage needs).
// No load of tile elements stands under a branch: at a join the compiler waits for every load in flight
// (with branches for the last stage and the edges the loop ran at half of this one's speed; lists are
// read under uniform branches, a stage ahead).
// ---------------------------------------------------------------------------
// element e of the result is element e + sh of v, 0 past its end
__device__ __forceinline__ f4 shifted(f4 v, int sh)
{
    f4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float x = 0.f;
#pragma unroll
        for (int q = 3; q >= e; --q) x = sh == q - e ? v[q] : x;
        r[e] = x;
    }
    return r;
}

// Contraction axis contiguous (C >= 4), optional row list.
template <int R> struct PlainP {
    static constexpr const char* NAME = "P";
    static constexpr bool P = true;
    static constexpr int BK = Geo<R>::BK, CPR = BK / 4, RPP = NT / CPR;
    const float* ptr[NP];
    int off_;
    f4 v[NP];
    __device__ __forceinline__ void init(const View& op, int r0, int rlim, int, int tid)
    {
        int row[NP];
#pragma unroll
        for (int it = 0; it < NP; ++it) row[it] = min(r0 + tid / CPR + RPP * it, rlim - 1);
        if (op.map_s) {
#pragma unroll
            for (int it = 0; it < NP; ++it) row[it] = op.map_s[row[it]];
#pragma unroll
            for (int it = 0; it < NP; ++it) row[it] = clamp_idx(row[it], op.n_s);
        }
#pragma unroll
        for (int it = 0; it < NP; ++it) ptr[it] = op.base + (size_t)row[it] * (size_t)op.ld;
    }
    // a chunk that would reach past the contraction range is read from its last four elements
    // and shifted into place by commit
    __device__ __forceinline__ void begin(const View&, int c0, int C, int tid) { off_ = min(c0 + (tid % CPR) * 4, C - 4); }
    template <int PC> __device__ __forceinline__ void fetch(const View&, int, int, int)
    {
        v[PC] = *(const f4_any*)(ptr[PC] + off_);
    }
    template <int PC, bool TAIL> __device__ __forceinline__ void commit(float* lds, int c0, int C, int tid) const
    {
        f4 x = v[PC];
        if constexpr (TAIL) {
            const int c = c0 + (tid % CPR) * 4;
            x = shifted(x, c - min(c, C - 4));
        }
        *(f4*)(lds + (tid / CPR + RPP * PC) * Geo<R>::PP + (tid % CPR) * 4) = x;
    }
};

// Contraction axis contiguous with the kept list on it: a thread owns one contraction index of
// the stage, so a wavefront's load runs along the (ascending) list in one memory row, or two.
template <int R> struct GatherP {
    static constexpr const char* NAME = "Pg";
    static constexpr bool P = true;
    static constexpr int BK = Geo<R>::BK, RSTEP = NT / BK, N = R / RSTEP;
    static constexpr int RPW = BK < 64 ? 64 / BK : 1;                    // memory rows per wavefront load
    const float* base_;
    int64_t ld_;
    int row0_, rlast_;      // uniform: first row of this wavefront, last row of the operand
    int second_;            // 1 in the half of a wavefront that takes the second row
    const int32_t* list_;
    int col_, next_;        // column of the stage being fetched, list entry of the one after
    float v[N];
    __device__ __forceinline__ void init(const View& op, int r0, int rlim, int C, int tid)
    {
        base_ = op.base; ld_ = op.ld;
        row0_ = r0 + (RPW == 1 ? __builtin_amdgcn_readfirstlane(tid / BK) : RPW * __builtin_amdgcn_readfirstlane(tid / 64));
        second_ = RPW == 1 ? 0 : (tid % 64) / BK;
        rlast_ = rlim - 1;
        list_ = op.map_c;
        next_ = list_[min(tid % BK, C - 1)];
    }
    __device__ __forceinline__ void begin(const View& op, int c0, int C, int tid)
    {
        col_ = clamp_idx(next_, op.n_c);
        next_ = list_[min(c0 + BK + tid % BK, C - 1)];
    }
    template <int PC> __device__ __forceinline__ void fetch(const View&, int, int, int)
    {
#pragma unroll
        for (int it = 4 * PC; it < 4 * PC + 4; ++it) {
            const int r = min(row0_ + RSTEP * it, rlast_);                       // uniform
            const float* row = base_ + (int64_t)r * ld_;
            if constexpr (RPW == 1) v[it] = row[(uint32_t)col_];
            else {
                const int64_t more = r < rlast_ ? ld_ : 0;                       // uniform
                v[it] = row[(int64_t)second_ * more + col_];
            }
        }
    }
    template <int PC, bool TAIL> __device__ __forceinline__ void commit(float* lds, int c0, int C, int tid) const
    {
#pragma unroll
        for (int it = 4 * PC; it < 4 * PC + 4; ++it)
            lds[(tid / BK + RSTEP * it) * Geo<R>::PP + tid % BK] = !TAIL || c0 + tid % BK < C ? v[it] : 0.f;
    }
};

// Contraction axis strided (stored rows of at least 4 elements), optional row list on it.
template <int R> struct PlainQ {
    static constexpr const char* NAME = "Q";
    static constexpr bool P = false;
    static constexpr int BK = Geo<R>::BK, CPR = R / 4, RPP = NT / CPR;
    const float* colp;      // base + this thread's (clamped) column
    int sh_;                // how far the clamp moved it
    bool edge_;             // uniform: the tile reaches past the stored rows' end
    int row_[NP];           // memory rows of the next stage
    const float* p_[NP];
    f4 v[NP];
    __device__ __forceinline__ void rows_for(const View& op, int c0, int C, int tid)
    {
#pragma unroll
        for (int it = 0; it < NP; ++it) row_[it] = min(c0 + tid / CPR + RPP * it, C - 1);
        if (op.map_s) {
#pragma unroll
            for (int it = 0; it < NP; ++it) row_[it] = op.map_s[row_[it]];
        }
    }
    __device__ __forceinline__ void init(const View& op, int r0, int, int C, int tid)
    {
        const int col = r0 + (tid % CPR) * 4, cc = min(col, op.n_c - 4);
        edge_ = r0 + R > op.n_c;
        sh_ = col - cc;
        colp = op.base + cc;
        rows_for(op, 0, C, tid);
    }
    __device__ __forceinline__ void begin(const View& op, int c0, int C, int tid)
    {
#pragma unroll
        for (int it = 0; it < NP; ++it) p_[it] = colp + (size_t)clamp_idx(row_[it], op.n_s) * (size_t)op.ld;
        rows_for(op, c0 + BK, C, tid);
    }
    template <int PC> __device__ __forceinline__ void fetch(const View&, int, int, int) { v[PC] = *(const f4_any*)p_[PC]; }
    template <int PC, bool TAIL> __device__ __forceinline__ void commit(float* lds, int c0, int C, int tid) const
    {
        f4 x = v[PC];
        if (edge_) x = shifted(x, sh_);
        if constexpr (TAIL) {
            const bool ok = c0 + tid / CPR + RPP * PC < C;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = ok ? x[e] : 0.f;
        }
        *(f4*)(lds + (tid / CPR + RPP * PC) * Geo<R>::PQ + (tid % CPR) * 4) = x;
    }
};

// Contraction axis strided, kept list on the other axis: a thread owns one kept column, and a
// wavefront's load covers 64 of them in one memory row (32 in each of two rows for R = 32).
template <int R> struct GatherQ {
    static constexpr const char* NAME = "Qg";
    static constexpr bool P = false;
    static constexpr int BK = Geo<R>::BK, CSTEP = NT / R, N = BK / CSTEP;
    static constexpr int RPW = R < 64 ? 64 / R : 1;                      // memory rows per wavefront load
    const float* base_;
    int64_t ld_;
    int c0_, clast_;        // uniform: first contraction index of this wavefront, last one of all
    uint32_t col_, second_; // column; 1 in the half of a wavefront that takes the second row
    float v[N];
    __device__ __forceinline__ void init(const View& op, int r0, int rlim, int C, int tid)
    {
        col_ = (uint32_t)clamp_idx(op.map_c[min(r0 + tid % R, rlim - 1)], op.n_c);
        base_ = op.base; ld_ = op.ld; clast_ = C - 1; c0_ = 0;
        second_ = RPW == 1 ? 0 : (tid % 64) / R;
    }
    __device__ __forceinline__ void begin(const View&, int c0, int, int tid)
    {
        c0_ = c0 + (RPW == 1 ? __builtin_amdgcn_readfirstlane(tid / R) : RPW * __builtin_amdgcn_readfirstlane(tid / 64));
    }
    template <int PC> __device__ __forceinline__ void fetch(const View&, int, int, int)
    {
#pragma unroll
        for (int it = 4 * PC; it < 4 * PC + 4; ++it) {
            const int c = min(c0_ + CSTEP * it, clast_);                         // uniform
            const float* row = base_ + (int64_t)c * ld_;
            if constexpr (RPW == 1) v[it] = row[col_];
            else {
                const int64_t more = c < clast_ ? ld_ : 0;                       // uniform
                v[it] = row[(int64_t)second_ * more + col_];
            }
        }
    }
    template <int PC, bool TAIL> __device__ __forceinline__ void commit(float* lds, int c0, int C, int tid) const
    {
#pragma unroll
        for (int it = 4 * PC; it < 4 * PC + 4; ++it)
            lds[(tid / R + CSTEP * it) * Geo<R>::PQ + tid % R] = !TAIL || c0 + tid / R + CSTEP * it < C ? v[it] : 0.f;
    }
};

// Element by element through whatever lists there are: for products with a contiguous extent
// below the four elements that the plain loaders read at a time.  A thread owns one element of every
// line it visits; lists are read once per tile (tile rows) or per stage (contraction indices).
template <int R, bool P_> struct AnyPQ {
    static constexpr const char* NAME = P_ ? "Pe" : "Qe";
    static constexpr bool P = P_;
    static constexpr int BK = Geo<R>::BK, LEN = P ? BK : R, LPI = NT / LEN, N = 16;      // a line's elements, lines per step
    static_assert(LPI * N * LEN == R * BK, "the stage");
    const float* line_[N];  // lines of the stage being fetched
    int col_;               // column of the stage being fetched
    float v[N];
    __device__ __forceinline__ void lines(const View& op, int first, int last, int tid)
    {
        int at[N];
#pragma unroll
        for (int it = 0; it < N; ++it) at[it] = min(first + tid / LEN + LPI * it, last);
        if (op.map_s) {
#pragma unroll
            for (int it = 0; it < N; ++it) at[it] = op.map_s[at[it]];
#pragma unroll
            for (int it = 0; it < N; ++it) at[it] = clamp_idx(at[it], op.n_s);
        }
#pragma unroll
        for (int it = 0; it < N; ++it) line_[it] = op.base + (size_t)at[it] * (size_t)op.ld;
    }
    __device__ __forceinline__ void column(const View& op, int first, int last, int tid)
    {
        col_ = min(first + tid % LEN, last);
        if (op.map_c) col_ = clamp_idx(op.map_c[col_], op.n_c);
    }
    __device__ __forceinline__ void init(const View& op, int r0, int rlim, int, int tid)
    {
        if constexpr (P) lines(op, r0, rlim - 1, tid);
        else column(op, r0, rlim - 1, tid);
    }
    __device__ __forceinline__ void begin(const View& op, int c0, int C, int tid)
    {
        if constexpr (P) column(op, c0, C - 1, tid);
        else lines(op, c0, C - 1, tid);
    }
    template <int PC> __device__ __forceinline__ void fetch(const View&, int, int, int)
    {
#pragma unroll
        for (int it = 4 * PC; it < 4 * PC + 4; ++it) v[it] = line_[it][col_];
    }
    template <int PC, bool TAIL> __device__ __forceinline__ void commit(float* lds, int c0, int C, int tid) const
    {
#pragma unroll
        for (int it = 4 * PC; it < 4 * PC + 4; ++it) {
            const int line = tid / LEN + LPI * it, e = tid % LEN;
            lds[line * (P ? Geo<R>::PP : Geo<R>::PQ) + e] = !TAIL || c0 + (P ? e : line) < C ? v[it] : 0.f;
        }
    }
};
template <int R> struct AnyP : AnyPQ<R, true> {};
template <int R> struct AnyQ : AnyPQ<R, false> {};

// four contraction indices of a block of eight: 0-3 for lanes 0-31, 4-7 for lanes 32-63
template <bool P, int R>
__device__ __forceinline__ f4 fragment(const float* lds, int row, int block, int grp)
{
    if constexpr (P) return *(const f4*)(lds + row * Geo<R>::PP + block * 8 + grp * 4);
    f4 x;
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = lds[(block * 8 + grp * 4 + s) * Geo<R>::PQ + row];
    return x;
}

// One workgroup's tile `lin` of a product.
template <template <int> class LA_, template <int> class LB_, int R>
__device__ __forceinline__ void f32_body(const Args& g, float* smem, const int lin)
{
    typedef LA_<R> LA;
    typedef LB_<R> LB;
    constexpr int BK = Geo<R>::BK;
    constexpr int OP_WORDS = Geo<R>::WORDS, STAGE = 2 * OP_WORDS;
    constexpr int WAVES = NT / 64;
    constexpr int T = R == 128 ? 2 : 1;                               // 32 x 32 results per wavefront and direction
    constexpr int BLOCKS = R == 32 ? BK / 8 / WAVES : BK / 8;         // blocks of 8 per wavefront and stage
    constexpr int CP = R + 4;                                         // row pitch of the result tile
    constexpr int TAB = 512;                                          // original columns per pass of the column scatter
    constexpr int PART = R == 32 ? 4 * 32 * 36 : 0;                   // the wavefronts' sums
    static_assert(R * CP + PART + 2 * R + TAB <= 2 * STAGE, "the epilogue fits the stages");

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, grp = lane >> 5;

    if (lin >= g.tiles_i * g.tiles_j) return;
    const int grp_sz = 4 * g.tiles_j;
    const int first_i = lin / grp_sz * 4, within = lin % grp_sz;
    const int rows_in = min(4, g.tiles_i - first_i);
    const int i0 = (first_i + within % rows_in) * R, j0 = within / rows_in * R;

    const int wr0 = R == 32 ? 0 : (wave >> 1) * (R / 2), wc0 = R == 32 ? 0 : (wave & 1) * (R / 2);
    const int blk0 = R == 32 ? wave * BLOCKS : 0;

    f32x16 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // While stage k is multiplied, stage k + 1 (requested during stage k - 1) goes from registers
    // to the other LDS buffer and stage k + 2 is requested, a piece at a time between the blocks
    // of MFMAs.  (Written at the end of the stage instead, after its MFMAs, a lone workgroup on a
    // compute unit took 1.5 us per stage of R = 64 where the MFMAs take 0.85; now 1.1.)
    LA la;
    LB lb;
    const int KT = (g.C + BK - 1) / BK;
    la.init(g.A, i0, g.I, g.C, tid);
    lb.init(g.B, j0, g.J, g.C, tid);
    auto begin = [&](int kt) { la.begin(g.A, kt * BK, g.C, tid); lb.begin(g.B, kt * BK, g.C, tid); };
    auto fetch = [&](int kt, auto piece) {
        la.template fetch<decltype(piece)::value>(g.A, kt * BK, g.C, tid);
        lb.template fetch<decltype(piece)::value>(g.B, kt * BK, g.C, tid);
    };
    auto commit = [&](float* stage, int kt, auto piece, auto tail) {
        la.template commit<decltype(piece)::value, decltype(tail)::value>(stage, kt * BK, g.C, tid);
        lb.template commit<decltype(piece)::value, decltype(tail)::value>(stage + OP_WORDS, kt * BK, g.C, tid);
    };
    auto all = [](auto f) {
        f(std::integral_constant<int, 0>());
        f(std::integral_constant<int, 1>());
        f(std::integral_constant<int, 2>());
        f(std::integral_constant<int, 3>());
    };
    begin(0);
    all([&](auto p) { fetch(0, p); });
    begin(1);                            // (past the end of a short contraction: valid addresses, zeros)
    all([&](auto p) { commit(smem, 0, p, std::true_type()); fetch(1, p); });
    __syncthreads();

    // fetches: there is a stage k + 2; else stage k + 1, if there is one, is the last
    auto step = [&](int kt, auto commits, auto fetches) {
        const float* as = smem + (kt & 1) * STAGE;
        const float* bs = as + OP_WORDS;
        float* nx = smem + ((kt + 1) & 1) * STAGE;
        if constexpr (decltype(fetches)::value) begin(kt + 2);
        f4 a[T], b[T];
#pragma unroll
        for (int i = 0; i < T; ++i) {
            a[i] = fragment<LA::P, R>(as, wr0 + 32 * i + l32, blk0, grp);
            b[i] = fragment<LB::P, R>(bs, wc0 + 32 * i + l32, blk0, grp);
        }
        all([&](auto piece) {
            constexpr int PC = decltype(piece)::value;
            if constexpr (decltype(commits)::value)
                commit(nx, kt + 1, piece, std::integral_constant<bool, !decltype(fetches)::value>());
            if constexpr (decltype(fetches)::value) fetch(kt + 2, piece);
#pragma unroll
            for (int k = PC * BLOCKS / NP; k < (PC + 1) * BLOCKS / NP; ++k) {
                // (blocks past the end of the contraction hold zeros)
                if constexpr (!decltype(commits)::value && R == 128)
                    if (kt * BK + 8 * k >= g.C) break;
                f4 an[T], bn[T];
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    an[i] = a[i]; bn[i] = b[i];
                    if (k + 1 < BLOCKS) {
                        an[i] = fragment<LA::P, R>(as, wr0 + 32 * i + l32, blk0 + k + 1, grp);
                        bn[i] = fragment<LB::P, R>(bs, wc0 + 32 * i + l32, blk0 + k + 1, grp);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);       // the next block's reads stay above this block's MFMAs
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < T; ++i) { a[i] = an[i]; b[i] = bn[i]; }
            }
        });
        __syncthreads();
    };
    int kt = 0;
    for (; kt + 2 < KT; ++kt) step(kt, std::true_type(), std::true_type());
    if (kt + 1 < KT) step(kt++, std::true_type(), std::false_type());
    step(kt, std::false_type(), std::false_type());

    // ---- result tile in LDS ---------------------------------------------------
    float* Cs = smem;
    if constexpr (R != 32) {
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    Cs[(wr0 + 32 * i + (r >> 2) * 8 + grp * 4 + (r & 3)) * CP + wc0 + 32 * j + l32] = acc[i][j][r];
    } else {
        float* part = smem + R * CP;
#pragma unroll
        for (int r = 0; r < 16; ++r) part[(wave * 32 + (r >> 2) * 8 + grp * 4 + (r & 3)) * 36 + l32] = acc[0][0][r];
        __syncthreads();
        const int row = tid >> 3, col = (tid & 7) * 4;
        f4 sum = *(const f4*)(part + row * 36 + col);
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            const f4 x = *(const f4*)(part + (w * 32 + row) * 36 + col);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += x[e];
        }
        *(f4*)(Cs + row * CP + col) = sum;
    }
    int* sidx = (int*)(smem + R * CP + PART);
    const int rows_valid = min(R, g.I - i0), cols_valid = min(R, g.J - j0);
    const bool scatter_c = g.epilogue == EPI_COL_SCATTER, scatter_r = g.epilogue == EPI_ROW_SCATTER;
    if (scatter_c && tid < cols_valid) sidx[tid] = clamp_idx(g.keep[j0 + tid], g.out_full);
    if (scatter_r && tid < rows_valid) sidx[tid] = clamp_idx(g.keep[i0 + tid], g.out_full);
    __syncthreads();

    if (scatter_c) {
        // The tile owns the original columns from its first kept column (0 for the first tile) up to
        // the next tile's first kept column (the full width for the last tile).  A table says which
        // result column, if any, belongs to each; then whole rows of owned columns leave, kept and
        // imputed ones together, 256 contiguous bytes per wavefront.
        int* tab = sidx + 2 * R;
        const int start = j0 == 0 ? 0 : sidx[0];
        const int end = j0 + R >= g.J ? g.out_full : clamp_idx(g.keep[j0 + R], g.out_full);
        // a long range behind the tile's last kept column needs no table
        const int last = max(start, sidx[cols_valid - 1] + 1), mid = end - last >= 256 ? last : end;
        for (int base = start; base < mid; base += TAB) {
            const int width = min(TAB, mid - base);
            for (int q = tid; q < width; q += NT) tab[q] = -1;
            __syncthreads();
            if (tid < cols_valid) {
                const int p = sidx[tid] - base;
                if (p >= 0 && p < width) tab[p] = tid;
            }
            __syncthreads();
            for (int q = lane; q < width; q += 64) {
                const int jj = tab[q];
                float* o = g.out + (size_t)i0 * (size_t)g.ldo + base + q;
                const float* pv = g.prev ? g.prev + (size_t)i0 * (size_t)g.ldo + base + q : nullptr;
                constexpr int UB = R == 32 ? 4 : 8;
                for (int r0 = wave; r0 < rows_valid; r0 += WAVES * UB) {
                    float x[UB];
#pragma unroll
                    for (int u = 0; u < UB; ++u) {
                        const int row = min(r0 + WAVES * u, rows_valid - 1);
                        x[u] = jj >= 0 ? Cs[row * CP + jj] : 0.f;
                        if (jj < 0 && pv) x[u] = pv[(size_t)row * (size_t)g.ldo];
                    }
#pragma unroll
                    for (int u = 0; u < UB; ++u)
                        if (r0 + WAVES * u < rows_valid) o[(size_t)(r0 + WAVES * u) * (size_t)g.ldo] = x[u];
                }
            }
            __syncthreads();
        }
        // and leaves 16 bytes a lane
        for (int r0 = wave; r0 < rows_valid && mid < end; r0 += 4 * WAVES) {
            for (int p = mid + lane * 4; p < end; p += 256) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int row = r0 + WAVES * u;
                    if (row >= rows_valid) break;
                    const size_t off = (size_t)(i0 + row) * (size_t)g.ldo + p;
                    if (p + 4 <= end) {
                        f4 v = f4{0.f, 0.f, 0.f, 0.f};
                        if (g.prev) v = *(const f4_any*)(g.prev + off);
                        *(f4_any*)(g.out + off) = v;
                    } else {
                        for (int e = 0; e < end - p; ++e) g.out[off + e] = g.prev ? g.prev[off + e] : 0.f;
                    }
                }
            }
        }
        return;
    }

    constexpr int CPR = R / 4, CHUNKS = R * CPR / NT;
    if (rows_valid == R && cols_valid == R) {
        // a whole tile: the old values of eight chunks are requested together (8192 x 4096, 8 deep: 64 -> 56 us)
        constexpr int UB = CHUNKS < 8 ? CHUNKS : 8;
        const int j = tid % CPR * 4;
        for (int it = 0; it < CHUNKS; it += UB) {
            float* o[UB];
            f4 old[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int row = tid / CPR + NT / CPR * (it + u);
                o[u] = g.out + (size_t)(scatter_r ? sidx[row] : i0 + row) * (size_t)g.ldo + j0 + j;
            }
            if (g.accumulate) {
#pragma unroll
                for (int u = 0; u < UB; ++u) old[u] = *(const f4_any*)o[u];
            } else {
#pragma unroll
                for (int u = 0; u < UB; ++u) old[u] = f4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                f4 x = *(const f4*)(Cs + (tid / CPR + NT / CPR * (it + u)) * CP + j);
                if (g.accumulate) x += old[u];
                *(f4_any*)o[u] = x;
            }
        }
    } else
#pragma unroll
    for (int it = 0; it < CHUNKS; ++it) {
        const int q = tid + NT * it;
        const int row = q / CPR, j = (q % CPR) * 4;
        if (row >= rows_valid || j >= cols_valid) continue;
        float* o = g.out + (size_t)(scatter_r ? sidx[row] : i0 + row) * (size_t)g.ldo + j0 + j;
        f4 x = *(const f4*)(Cs + row * CP + j);
        if (j + 4 <= cols_valid) {
            if (g.accumulate) x += *(const f4_any*)o;
            *(f4_any*)o = x;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j + e < cols_valid) o[e] = g.accumulate ? o[e] + x[e] : x[e];
        }
    }
    if (scatter_r) {
        // the dropped rows this tile owns (same ownership rule as above): every lane looks one row
        // up, the wavefront then writes the dropped ones together
        const int start = i0 == 0 ? 0 : sidx[0];
        const int end = i0 + R >= g.I ? g.out_full : clamp_idx(g.keep[i0 + R], g.out_full);
        for (int base = start + wave * 64; base < end; base += NT) {
            const int mine = base + lane;
            bool dropped = false;
            if (mine < end) {
                const int ii = lower_bound_lds(sidx, rows_valid, mine);
                dropped = !(ii < rows_valid && sidx[ii] == mine);
            }
            unsigned long long todo = __ballot(dropped);
            while (todo) {
                // a row to every CPR lanes, 16 bytes a lane
                int p = -1;
#pragma unroll
                for (int u = 0; u < 64 / CPR; ++u) {
                    if (todo && u == lane / CPR) p = base + (__ffsll((long long)todo) - 1);
                    todo &= todo - 1;                         // (0 stays 0)
                }
                const int j = lane % CPR * 4;
                if (p < 0 || j >= cols_valid) continue;
                const size_t off = (size_t)p * (size_t)g.ldo + j0 + j;
                if (j + 4 <= cols_valid) {
                    f4 v = f4{0.f, 0.f, 0.f, 0.f};
                    if (g.prev) v = *(const f4_any*)(g.prev + off);
                    *(f4_any*)(g.out + off) = v;
                } else {
                    for (int e = 0; e < cols_valid - j; ++e) g.out[off + e] = g.prev ? g.prev[off + e] : 0.f;
                }
            }
        }
    }
}

// every XCD gets a contiguous range of tiles, ordered in groups of 4 tile rows
template <template <int> class LA, template <int> class LB, int R>
__global__ __launch_bounds__(NT) void f32_kernel(const Args g)
{
    extern __shared__ __align__(16) float smem[];
    f32_body<LA, LB, R>(g, smem, (int)((blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8));
}

// dX and dW of one backward call: the first per_w workgroups of every XCD are dW's, or with x_first the last ones.
template <template <int> class XA, template <int> class XB, int XR, template <int> class WA, template <int> class WB, int WR>
__global__ __launch_bounds__(NT) void f32_pair_kernel(const Args gx, const Args gw, const int per_x, const int per_w, const int x_first)
{
    extern __shared__ __align__(16) float smem[];
    const int xcd = blockIdx.x % 8, q = blockIdx.x / 8;
    const int qx = x_first ? q : q - per_w, qw = x_first ? q - per_x : q;
    if (qw >= 0 && qw < per_w) f32_body<WA, WB, WR>(gw, smem, xcd * per_w + qw);
    else f32_body<XA, XB, XR>(gx, smem, xcd * per_x + qx);
}

template <template <int> class LA, template <int> class LB, int R>
int launch_inst(const Args& a, hipStream_t stream)
{
    constexpr int smem = 2 * 2 * Geo<R>::WORDS * 4;
    auto fn = f32_kernel<LA, LB, R>;
    static AttrFlags attr_set;      // per instantiation and device
    if (!ensure_max_dynamic_lds((const void*)fn, smem, &attr_set)) return ZR_ERR_HIP;
    if (debug_names_wanted())
        snprintf(g_debug.last_kernel, sizeof(g_debug.last_kernel), "f32_kernel<%s, %s, %d>", LA<R>::NAME, LB<R>::NAME, R);
    Args k = a;
    k.tiles_i = (a.I + R - 1) / R;
    k.tiles_j = (a.J + R - 1) / R;
    const int64_t tiles = (int64_t)k.tiles_i * k.tiles_j;
    if (tiles > 0x7ffffff0) return ZR_ERR_LIMIT;
    hipLaunchKernelGGL(fn, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(NT), smem, stream, k);
    return hip_status(hipGetLastError());
}

// Extent of the tiles of a product on its own.
int tile_of(const Args& a)
{
    const int64_t t64 = (int64_t)((a.I + 63) / 64) * ((a.J + 63) / 64), t128 = (int64_t)((a.I + 127) / 128) * ((a.J + 127) / 128);
    // 128 x 128 tiles where they fill their rounds of 256: per area they are 4 to 24 % faster (contraction 256,
    // P x Q: 512 tiles 43 us against 48 on 64 x 64, 384 tiles 42 against 37, 256 tiles 25 against 26).  Short
    // contractions are all epilogue and half empty 64-deep stages: contraction 8, 192 tiles 9 against 10,
    // 2048 tiles 39 against 72; contraction 64, 192 tiles 11 against 10, 384 tiles 16 against 17.
    const int64_t rounds64 = (t64 + 255) / 256, rounds128 = t128 <= 256 ? 1 : 2 * ((t128 + 511) / 512);
    const bool big = a.C <= 32 ? t128 >= 192 : a.C <= 96 ? t128 >= 256 : 0.92 * 4 * (double)rounds128 < (double)rounds64;
    if (big) return 128;
    // 64 x 64 tiles once there is one for most compute units (contraction 1024: 128 tiles 22.0 us
    // against 15.2 on 32 x 32, 192 tiles 22.7 against 21.8, 256 tiles 23.3 against 27.8, 512 tiles
    // 41.1 against 52.1)
    return t64 < 192 ? 32 : 64;
}

template <template <int> class LA, template <int> class LB>
int launch_shape(const Args& a, hipStream_t stream)
{
    switch (tile_of(a)) {
        case 128: return launch_inst<LA, LB, 128>(a, stream);
        case 64: return launch_inst<LA, LB, 64>(a, stream);
        default: return launch_inst<LA, LB, 32>(a, stream);
    }
}

// The element loaders: a contraction of less than four is one stage of any tile shape; otherwise the
// result has less than four rows or columns, and the narrowest tiles waste least.
template <template <int> class LA, template <int> class LB>
int launch_short(const Args& a, hipStream_t stream)
{
    return a.C < 4 ? launch_shape<LA, LB>(a, stream) : launch_inst<LA, LB, 32>(a, stream);
}

// ---------------------------------------------------------------------------
// dX and dW in one launch
// ---------------------------------------------------------------------------
// Tiles by a model of the schedule: every XCD takes its tiles in order, each on the first of 32 units that is
// through with its own (two tiles share a unit and its matrix pipes, which takes as long as one after the
// other); a tile takes a start and an end, and a time per stage, longer where kept columns are gathered, and a launch a start
// and an end.  Fitted to 7328 backward calls (32 to 16384 tokens, 64 to 5120 wide), each in all forms and in two launches, for the time of what
// they pick: 0.800 of that of two launches on average (the best form of each would be 0.795), 16 of them more than 8 % slower.  us in two
// launches and now: 1576 x 2048 x 1024 of 1638 kept rows 151 -> 117, 609 x 1414 x 247 31 -> 20, 256 x 512 x 256
// 14.7 -> 11.6.  A product that takes 32 x 32 tiles on its own keeps them: their four partial sums are the more
// exact.  128 x 128 tiles are outside the model: see one_round.
struct Plan { int xr, wr; bool x_first; };
struct Cost { double start, stage; };
constexpr Cost kCost32 = {1.55, 0.7}, kCost64 = {1.38, 1.11}, kCost128 = {1.4, 2.06};     // us, us per stage of 128, 64 and 32
constexpr double kGathered = 0.18, kAlone = 9.2, kPair = 8.6;                             // per gathered operand; us a launch of one, of both

int64_t tiles_of(const Args& a, int r) { return (int64_t)((a.I + r - 1) / r) * ((a.J + r - 1) / r); }
bool may_take(const Args& a, int r) { return r == 32 || tiles_of(a, 64) >= 192; }

double tile_us(const Args& a, int r)
{
    const Cost c = r == 32 ? kCost32 : r == 64 ? kCost64 : kCost128;
    const int bk = 16 * NT / r;
    return c.start + c.stage * ((a.C + bk - 1) / bk) * (1 + kGathered * ((a.A.map_c != nullptr) + (a.B.map_c != nullptr)));
}

double alone_us(const Args& a)
{
    const int r = tile_of(a);
    const int64_t n = (tiles_of(a, r) + 7) / 8;
    return (double)((n + 31) / 32) * tile_us(a, r) + kAlone;
}

// Both products on 128 x 128 tiles: only where every tile has a unit to itself, 64 x 64 ones take more than three rounds, and both
// products gather and are about as deep, so that all tiles end together.  4846 backward calls whose products may take such tiles:
// there they take 0.94 of the time of what the model picks (36 calls, 0.85 to 1.05; 1576 x 1024 x 2048 of 1638 kept columns
// 165 us, now 149), without the gathers 1.08 and more, over all of them 1.47 (13120 x 704 x 2599 963 us in two launches, 1360 in one).
bool one_round(const Args& x, const Args& w)
{
    auto gathers = [](const Args& a) { return a.A.map_c || a.B.map_c; };
    auto per_xcd = [&](int r) { return (tiles_of(x, r) + 7) / 8 + (tiles_of(w, r) + 7) / 8; };
    return may_take(x, 128) && may_take(w, 128) && gathers(x) && gathers(w) && per_xcd(128) <= 32 && per_xcd(64) > 3 * 32 &&
           std::max(x.C, w.C) <= 1.2 * std::min(x.C, w.C);
}

// false: two launches
bool plan_pair(const Args& x, const Args& w, Plan& p)
{
    if (one_round(x, w)) { p = Plan{128, 128, tile_us(x, 128) > tile_us(w, 128)}; return true; }
    double best = alone_us(x) + alone_us(w);
    bool found = false;
    for (int xr : {32, 64})
        for (int wr : {32, 64}) {
            if (!may_take(x, xr) || !may_take(w, wr)) continue;
            const int64_t nx = (tiles_of(x, xr) + 7) / 8, nw = (tiles_of(w, wr) + 7) / 8;
            if (nx + nw > 1 << 20) continue;
            const double tx = tile_us(x, xr), tw = tile_us(w, wr);
            const bool x_first = tx > tw;                   // the long tiles first
            const double us = kPair + (x_first ? two_groups((int)nx, tx, (int)nw, tw, 32) : two_groups((int)nw, tw, (int)nx, tx, 32));
            if (us < best) { best = us; p = Plan{xr, wr, x_first}; found = true; }
        }
    return found;
}

template <template <int> class XA, template <int> class XB, int XR, template <int> class WA, template <int> class WB, int WR>
int launch_pair_inst(const Args& x, const Args& w, bool x_first, hipStream_t stream)
{
    constexpr int words = Geo<XR>::WORDS > Geo<WR>::WORDS ? Geo<XR>::WORDS : Geo<WR>::WORDS;
    constexpr int smem = 2 * 2 * words * 4;
    auto fn = f32_pair_kernel<XA, XB, XR, WA, WB, WR>;
    static AttrFlags attr_set;      // per instantiation and device
    if (!ensure_max_dynamic_lds((const void*)fn, smem, &attr_set)) return ZR_ERR_HIP;
    if (debug_names_wanted())
        snprintf(g_debug.last_kernel, sizeof(g_debug.last_kernel), "f32_kernel<%s, %s, %d> beside <%s, %s, %d>", WA<WR>::NAME, WB<WR>::NAME, WR,
                 XA<XR>::NAME, XB<XR>::NAME, XR);
    Args kx = x, kw = w;
    kx.tiles_i = (x.I + XR - 1) / XR; kx.tiles_j = (x.J + XR - 1) / XR;
    kw.tiles_i = (w.I + WR - 1) / WR; kw.tiles_j = (w.J + WR - 1) / WR;
    const int64_t px = ((int64_t)kx.tiles_i * kx.tiles_j + 7) / 8, pw = ((int64_t)kw.tiles_i * kw.tiles_j + 7) / 8;
    hipLaunchKernelGGL(fn, dim3((unsigned)(px + pw) * 8), dim3(NT), smem, stream, kx, kw, (int)px, (int)pw, x_first ? 1 : 0);
    return hip_status(hipGetLastError());
}

template <template <int> class XA, template <int> class XB, template <int> class WA, template <int> class WB>
int launch_pair(const Args& x, const Args& w, const Plan& p, hipStream_t stream)
{
    // (pairs of gathering products only, see one_round)
    if constexpr (std::is_same_v<XA<32>, GatherP<32>> || std::is_same_v<XB<32>, GatherQ<32>>)
        if (p.xr == 128) return launch_pair_inst<XA, XB, 128, WA, WB, 128>(x, w, p.x_first, stream);
    if (p.xr == 64 && p.wr == 64) return launch_pair_inst<XA, XB, 64, WA, WB, 64>(x, w, p.x_first, stream);
    if (p.xr == 64) return launch_pair_inst<XA, XB, 64, WA, WB, 32>(x, w, p.x_first, stream);
    if (p.wr == 64) return launch_pair_inst<XA, XB, 32, WA, WB, 64>(x, w, p.x_first, stream);
    return launch_pair_inst<XA, XB, 32, WA, WB, 32>(x, w, p.x_first, stream);
}

Args args_of(const GemmDesc& d)
{
    Args a;
    a.A = View{(const float*)d.A.base, d.A.ld, d.A.map_strided, d.A.map_contig, d.A.n_strided, d.A.n_contig};
    a.B = View{(const float*)d.B.base, d.B.ld, d.B.map_strided, d.B.map_contig, d.B.n_strided, d.B.n_contig};
    a.I = d.I; a.J = d.J; a.C = d.C;
    a.out = (float*)d.out; a.ldo = d.ldo; a.epilogue = d.epilogue; a.keep = d.keep_idx; a.out_full = d.out_full;
    a.tiles_i = a.tiles_j = 0;
    a.prev = (const float*)d.prev; a.accumulate = d.accumulate ? 1 : 0;
    return a;
}

bool too_short(const GemmDesc& d, const Operand& o) { return !o.map_contig && (o.c_contig ? d.C : o.n_contig) < 4; }

}  // namespace

int launch_gemm_f32_pair(const GemmDesc& dx, const GemmDesc& dw, hipStream_t stream)
{
    if (dx.I < 1 || dx.J < 1 || dx.C < 1 || dw.I < 1 || dw.J < 1 || dw.C < 1) return -1;
    for (const GemmDesc* d : {&dx, &dw})
        if (too_short(*d, d->A) || too_short(*d, d->B)) return -1;
    if (!dx.A.c_contig || dw.A.c_contig || dw.B.c_contig) return -1;
    const Args x = args_of(dx), w = args_of(dw);
    Plan p;
    if (!plan_pair(x, w, p)) return -1;
    const bool xa = dx.A.map_contig, xb = dx.B.map_contig, wa = dw.A.map_contig, wb = dw.B.map_contig;
    if (dx.B.c_contig) {                    // weight stored [K x N]
        if (xa && xb && !wa && wb) return launch_pair<GatherP, GatherP, PlainQ, GatherQ>(x, w, p, stream);
        if (!xa && !xb && wa && !wb) return launch_pair<PlainP, PlainP, GatherQ, PlainQ>(x, w, p, stream);
        if (!xa && !xb && !wa && !wb) return launch_pair<PlainP, PlainP, PlainQ, PlainQ>(x, w, p, stream);
        return -1;
    }
    if (xa && !xb && wa && !wb) return launch_pair<GatherP, PlainQ, GatherQ, PlainQ>(x, w, p, stream);
    if (!xa && xb && !wa && wb) return launch_pair<PlainP, GatherQ, PlainQ, GatherQ>(x, w, p, stream);
    if (!xa && !xb && !wa && !wb) return launch_pair<PlainP, PlainQ, PlainQ, PlainQ>(x, w, p, stream);
    return -1;
}

int launch_gemm_f32(const GemmDesc& d, hipStream_t stream)
{
    if (d.I < 1 || d.J < 1 || d.C < 1) return ZR_ERR_SHAPE;
    const Args a = args_of(d);
    const bool ag = d.A.map_contig != nullptr, bg = d.B.map_contig != nullptr;
    if (too_short(d, d.A) || too_short(d, d.B)) {
        if (d.A.c_contig) return d.B.c_contig ? launch_short<AnyP, AnyP>(a, stream) : launch_short<AnyP, AnyQ>(a, stream);
        return d.B.c_contig ? ZR_ERR_MODE : launch_short<AnyQ, AnyQ>(a, stream);
    }
    if (d.A.c_contig && !d.B.c_contig) {            // forward, weight stored [K x N]
        if (ag) return bg ? ZR_ERR_MODE : launch_shape<GatherP, PlainQ>(a, stream);
        return bg ? launch_shape<PlainP, GatherQ>(a, stream) : launch_shape<PlainP, PlainQ>(a, stream);
    }
    if (d.A.c_contig && d.B.c_contig) {
        // (a list on the contraction is on both operands: nothing is extracted in fp32)
        if (ag != bg) return ZR_ERR_MODE;
        return ag ? launch_shape<GatherP, GatherP>(a, stream) : launch_shape<PlainP, PlainP>(a, stream);
    }
    if (!d.A.c_contig && !d.B.c_contig) {           // dW
        if (ag) return bg ? ZR_ERR_MODE : launch_shape<GatherQ, PlainQ>(a, stream);
        return bg ? launch_shape<PlainQ, GatherQ>(a, stream) : launch_shape<PlainQ, PlainQ>(a, stream);
    }
    return ZR_ERR_MODE;
}

}  // namespace zr
