// dX and dW of one backward call in one launch (bf16, 16-byte aligned rows).
//
// What it is for: the rounding of each product's tiles to whole rounds of the 256 compute units.  On
// a Llama-2-7B shard of which a quarter is pruned, dX is two rounds of 256 x 256 tiles and dW 176 tiles
// of 192 x 256 four times as long, so a third of the chip waits for dW; on a 13B shard on eight tasks
// both leave a part of their last round empty.  In one launch the long tiles of dW start first, one to a
// unit, and the tiles of dX fill the units beside and after them.  Every XCD gets its contiguous share of
// each product's tiles, so the operand slices that its L2 serves stay those of neighbouring tiles.
#include <algorithm>
#include <cmath>

#include "zr_gemm_fast.h"

namespace zr {

namespace {

// A tile shape with its loaders, as a type.
template <int PART, template <int, int> class LA_, template <int, int> class LB_, int BM_, int BN_, int WM, int WN, int PHASE_>
struct Shape {
    static constexpr int BM = BM_, BN = BN_, NT = 64 * WM * WN, PHASE = PHASE_;
    typedef LA_<BM, NT> LA;
    typedef LB_<BN, NT> LB;
    static constexpr int LDS = fast_smem_bytes<LA::WORDS, LB::WORDS, BM, BN, LA::RING>() +
                               [] { if constexpr (LA::RING) return LB::MAPPED ? ring_list_max<BM, BN>() * 4 : 0; else return 0; }();
    static __device__ __forceinline__ void run(const FArgs& g, uint32_t* smem, int lin)
    {
        fast_body<LA_, LB_, BM_, BN_, WM, WN, PHASE_, PART>(g, smem, lin);
    }
};

// The first per_w workgroups of every XCD are dW's, or with x_first the last ones.
template <class SX, class SW>
__global__ __launch_bounds__(SX::NT) void pair_kernel(const FArgs gx, const FArgs gw, const int per_x, const int per_w, const int x_first)
{
    static_assert(SX::NT == SW::NT, "one launch, one workgroup size");
    extern __shared__ __align__(16) uint32_t smem[];
    const int xcd = blockIdx.x % 8, q = blockIdx.x / 8;
    const int qx = x_first ? q : q - per_w, qw = x_first ? q - per_x : q;
    if (qw >= 0 && qw < per_w) SW::run(gw, smem, xcd * per_w + qw);
    else SX::run(gx, smem, xcd * per_x + qx);
}

inline void whole_grid(FArgs& k, int bm, int bn)
{
    k.i_base = k.j_base = 0; k.i_end = k.I; k.j_end = k.J;
    k.tiles_i = (k.I + bm - 1) / bm; k.tiles_j = (k.J + bn - 1) / bn;
    k.split = 1; k.kt_per = 0; k.avg_slot_base = 0;
}

// ---------------------------------------------------------------------------
// The schedule.  A launch is modelled as what it is: every XCD takes its tiles in order, each as soon
// as one of its 32 units (or of 64 halves, with tiles of 128 x 128 and less) is free.  A tile takes a
// start and an end, and a time per 64-deep step of its contraction.  All shapes, with dW's contraction in
// one piece or in several, are put through the model and the shortest wins; where two products on their own
// are estimated shorter (dX of few tiles and a long contraction, which other kernels add up in groups)
// they stay alone.  The constants are fitted to 90 backward calls (64 to 16384 tokens, 128 to 4800 wide),
// each timed in 40 forms: the form that the model picks is 2.7 % slower than the best of them on average.
// ---------------------------------------------------------------------------
enum { B256, B192, B128, B64 };
struct Cost { double start, step; };               // us, us per 64 of the contraction
constexpr Cost kCost[4] = {{10.3, 1.48}, {8.6, 1.36}, {5.7, 1.12}, {6.4, 0.84}};
constexpr double kLaunch = 3.0;                     // what the models of the other kernels count for a launch, and this one does not
constexpr double kHalfFree = 0.81;                 // time per step of a small tile that has its unit to itself
constexpr double kSliceBig = 2.0, kSliceSmall = 0.5;       // a slice of a split contraction stores its sums,
constexpr double kCopiedRow = 0.08;                // us
constexpr double kReduce = 8.2, kReduceTile = 0.013;       // and a second launch adds them: us, and us per 256 x 256 sums

struct Plan { int sx, sw, slices; bool x_first; double us; };

inline int steps_of(int C) { return (C + BK - 1) / BK; }
inline int64_t per_xcd(int64_t tiles) { return (tiles + 7) / 8; }
inline void shape_of(int s, bool x, int& bm, int& bn)
{
    bm = s == B256 ? 256 : s == B192 ? (x ? 256 : 192) : s == B128 ? 128 : 64;
    bn = s == B256 ? 256 : s == B192 ? (x ? 192 : 256) : 128;
}
inline int64_t shape_tiles(int I, int J, int s, bool x)
{
    int bm, bn;
    shape_of(s, x, bm, bn);
    return tiles_of(I, J, bm, bn);
}

// One product in launches of its own, on the direct-to-LDS kernels.
double fast_alone_us(int I, int J, int C, bool may_split)
{
    double best = 1e30;
    for (int s = B256; s <= B64; ++s) {
        const int64_t n = per_xcd(shape_tiles(I, J, s, false));
        const int slots = s <= B192 ? 32 : 64;
        const double f = slots == 64 && n <= 32 ? kHalfFree : 1.0;
        best = std::min(best, (double)((n + slots - 1) / slots) * (kCost[s].start + f * kCost[s].step * steps_of(C)));
        const int64_t t = tiles_of(I, J, 128, 128);
        const int sp = (int)std::min<int64_t>(std::min<int64_t>(512 / t, 8), steps_of(C) / 8);
        if (s == B128 && sp >= 2 && may_split) {
            const double g = per_xcd(t * sp) <= 32 ? kHalfFree : 1.0;
            best = std::min(best, kCost[s].start + g * kCost[s].step * ((steps_of(C) + sp - 1) / sp) + kSliceSmall + kReduce + kReduceTile * (double)(t * sp) / 4);
        }
    }
    return best;
}

// ... or on the kernel for any alignment, whichever is the shorter.
double alone_us(int I, int J, int C)
{
    return std::min(4.6 + 0.36 * steps_of(C) * std::max(1.0, (double)tiles_of(I, J, 64, 64) / 256), fast_alone_us(I, J, C, true));
}

// (A clear gain only with a row list on the contraction of small tiles and dW in one piece: 41 calls of those took 0.85 of the time of two
// launches on average, but 6 of them more than 1.08, 3584 x 472 x 4432 of 3408 kept columns 94 us for 75.)
Plan plan_pair(const FArgs& x, const FArgs& w, bool x_rows, bool mapped, bool big_ok)
{
    Plan best{0, 0, 0, false, alone_us(x.I, x.J, x.C) + alone_us(w.I, w.J, w.C)};
    // Products that the kernel for any alignment adds up in groups of the contraction keep that order, unless they are split.
    if (adds_in_groups(x.I, x.J, x.C)) return best;
    const bool w_grouped = adds_in_groups(w.I, w.J, w.C);
    for (int sx = big_ok ? B256 : B128; sx <= (x_rows ? B64 : B128); ++sx) {
        const bool small = sx >= B128;
        const int slots = small ? 64 : 32;
        const int64_t nx = per_xcd(shape_tiles(x.I, x.J, sx, true));
        for (int sw = small ? B128 : B256; sw <= (small ? B128 : B192); ++sw) {
            const int64_t tw = shape_tiles(w.I, w.J, sw, false);
            int bm, bn;
            shape_of(sw, false, bm, bn);
            const size_t tile_bytes = (size_t)bm * bn * 4;
            for (int sl : {1, 2, 3, 4, 6, 8}) {
                if (sl > 1 && (sl > steps_of(w.C) || !split_enabled() || !w.partial || (size_t)tw * tile_bytes * sl > w.partial_bytes)) break;
                if (sl == 1 && w_grouped) continue;
                const int64_t nw = per_xcd(tw * sl);
                if (nx + nw > 1 << 20) break;
                const double f = small && nx + nw <= 32 ? kHalfFree : 1.0;
                const double tx = kCost[sx].start + f * kCost[sx].step * steps_of(x.C);
                double tp = kCost[sw].start + f * kCost[sw].step * ((steps_of(w.C) + sl - 1) / sl) + (sl > 1 ? (small ? kSliceSmall : kSliceBig) : 0.0);
                // rows that Same copies between a tile's kept ones (192 x 2288 x 608 of 248 kept rows 18 us in two launches, 33 in one)
                if (sl == 1 && w.prev && w.epilogue == EPI_ROW_SCATTER) tp += kCopiedRow * bm * (w.out_full - w.I) / w.I;
                const bool x_first = tx > tp;               // the long pieces first
                double us = x_first ? two_groups((int)nx, tx, (int)nw, tp, slots) : two_groups((int)nw, tp, (int)nx, tx, slots);
                if (sl > 1) us += kReduce + kReduceTile * (double)(tw * sl) * tile_bytes / (65536.0 * 4);
                if (mapped && small && sl == 1) us *= 1.09;
                if (us < best.us) best = Plan{sx, sw, sl, x_first, us};
            }
        }
    }
    return best;
}

template <class SX, class SW>
int launch_pair_inst(const FArgs& x, const FArgs& w, const Plan& p, hipStream_t stream)
{
    constexpr int smem = SX::LDS > SW::LDS ? SX::LDS : SW::LDS;
    static_assert(smem <= 160 * 1024, "LDS of a workgroup");
    auto fn = pair_kernel<SX, SW>;
    static AttrFlags attr_set;      // per instantiation and device
    if (!ensure_max_dynamic_lds((const void*)fn, smem, &attr_set)) return ZR_ERR_HIP;
    FArgs kx = x, kw = w;
    whole_grid(kx, SX::BM, SX::BN);
    whole_grid(kw, SW::BM, SW::BN);
    if (SW::PHASE == 1) {
        const int KT = (w.C + BK - 1) / BK;
        kw.kt_per = (KT + p.slices - 1) / p.slices;
        kw.split = (KT + kw.kt_per - 1) / kw.kt_per;                      // no empty slice
    }
    const int64_t tx = (int64_t)kx.tiles_i * kx.tiles_j, tw = (int64_t)kw.tiles_i * kw.tiles_j;
    const int64_t px = (tx + 7) / 8, pw = (tw * kw.split + 7) / 8;
    if (px + pw > 0x0ffffff0) return ZR_ERR_LIMIT;
    if (debug_names_wanted())
        snprintf(g_debug.last_kernel, sizeof(g_debug.last_kernel), "fast_kernel<%s, %s, %d, %d> beside <%s, %s, %d, %d>%s", SW::LA::NAME,
                 SW::LB::NAME, SW::BM, SW::BN, SX::LA::NAME, SX::LB::NAME, SX::BM, SX::BN, SW::PHASE == 1 ? " split" : "");
    hipLaunchKernelGGL(fn, dim3((unsigned)(px + pw) * 8), dim3(SX::NT), smem, stream, kx, kw, (int)px, (int)pw, p.x_first ? 1 : 0);
    if (SW::PHASE == 1) {
        if (hipGetLastError() != hipSuccess) return ZR_ERR_HIP;
        hipLaunchKernelGGL((split_reduce_kernel<1, SW::BM / 32, SW::BN / 64>), dim3((unsigned)(tw * (SW::BM / 32))), dim3(SW::NT), 0, stream, kw);
    }
    return hip_status(hipGetLastError());
}

template <template <int, int> class LB, int XM, int XN, int XWM, int XWN>
int launch_pair_w(const FArgs& x, const FArgs& w, const Plan& p, hipStream_t stream)
{
    typedef Shape<PART_DX, RingP, LB, XM, XN, XWM, XWN, 0> SX;
    if (p.slices > 1) {
        if (p.sw == B256) return launch_pair_inst<SX, Shape<PART_DW, RingQ, RingQ, 256, 256, 2, 4, 1>>(x, w, p, stream);
        return launch_pair_inst<SX, Shape<PART_DW, RingQ, RingQ, 192, 256, 2, 4, 1>>(x, w, p, stream);
    }
    if (p.sw == B256) return launch_pair_inst<SX, Shape<PART_DW, RingQ, RingQ, 256, 256, 2, 4, 0>>(x, w, p, stream);
    return launch_pair_inst<SX, Shape<PART_DW, RingQ, RingQ, 192, 256, 2, 4, 0>>(x, w, p, stream);
}

template <template <int, int> class LB, int XM, int XWM, int XWN>
int launch_pair_small(const FArgs& x, const FArgs& w, const Plan& p, hipStream_t stream)
{
    typedef Shape<PART_DX, DmaP, LB, XM, 128, XWM, XWN, 0> SX;
    if (p.slices > 1) return launch_pair_inst<SX, Shape<PART_DW, DmaQ, DmaQ, 128, 128, 2, 2, 1>>(x, w, p, stream);
    return launch_pair_inst<SX, Shape<PART_DW, DmaQ, DmaQ, 128, 128, 2, 2, 0>>(x, w, p, stream);
}

template <template <int, int> class LB>
int launch_pair_x(const FArgs& x, const FArgs& w, const Plan& p, hipStream_t stream)
{
    if (p.sx == B256) return launch_pair_w<LB, 256, 256, 2, 4>(x, w, p, stream);
    return launch_pair_w<LB, 256, 192, 4, 2>(x, w, p, stream);
}

}  // namespace

// A product with a gather in flight takes a time per 64-deep step that grows with what is read and left
// out (whole rows are, of which the kept columns go on).  Fitted to 1278 products of 64 to 16384 tokens, 64 to 5120
// wide, within 15 % (us: dW of 192 tiles, 2000 of 2048 kept columns, 16384 tokens 316, of 1024 of 2048 818), and 10 % less than that,
// so that it errs on the side of two launches.
double gemm_fast_us(const GemmDesc& d)
{
    const Operand* gathered = d.A.map_contig ? &d.A : d.B.map_contig ? &d.B : nullptr;
    if (!gathered) return fast_alone_us(d.I, d.J, d.C, d.split_scratch != nullptr) + kLaunch;
    const double steps = steps_of(d.C), span = (double)gathered->n_contig / (gathered->c_contig ? d.C : gathered == &d.A ? d.I : d.J);
    const int64_t t = tiles_of(d.I, d.J, 128, 128);
    const double pairs = (double)((t + 511) / 512), big = (double)((tiles_of(d.I, d.J, 256, 256) + 255) / 256);
    if (!d.A.c_contig) return 11.3 + 0.68 * steps * span * std::sqrt(span) * pairs;
    if (gathered == &d.A) return 9.1 + 3.28 * steps * big;
    if (!gathered->c_contig) return std::min(12.9 + steps * span * (t <= 256 ? 0.77 : 1.16 * pairs), 20.7 + 1.77 * steps * span * big);
    return std::min(9.2 + 2.18 * steps * std::sqrt(span) * pairs, 13.3 + 3.45 * steps * big);
}

int launch_gemm_pair(const GemmDesc& dx, const GemmDesc& dw, hipStream_t stream)
{
    if (forced_tiles() || !ring_enabled()) return -1;
    if (!gemm_fast_can(dx) || !gemm_fast_can(dw)) return -1;
    // operands as they lie, or by rows; no sums of Average imputation
    if (dx.A.map_contig || dx.B.map_contig || dw.A.map_contig || dw.B.map_contig) return -1;
    if (!dx.A.c_contig || dx.A.map_strided || dw.A.c_contig || dw.B.c_contig || dx.avg_partial || dw.avg_partial) return -1;
    // (a dW that scatters columns comes with kept columns of W in dX, which are refused above)
    if (dx.epilogue == EPI_ROW_SCATTER || dw.epilogue == EPI_COL_SCATTER) return -1;
    const bool rows = dx.B.c_contig, mapped = !rows && dx.B.map_strided;
    const FArgs x = fargs_of(dx), w = fargs_of(dw);
    const Plan p = plan_pair(x, w, rows, mapped, !mapped || dx.C <= ring_list_max<256, 256>());
    if (p.slices == 0) return -1;
    if (p.sx == B64) return launch_pair_small<DmaP, 64, 1, 4>(x, w, p, stream);
    if (p.sx == B128) {
        if (rows) return launch_pair_small<DmaP, 128, 2, 2>(x, w, p, stream);
        if (mapped) return launch_pair_small<DmaQM, 128, 2, 2>(x, w, p, stream);
        return launch_pair_small<DmaQ, 128, 2, 2>(x, w, p, stream);
    }
    if (rows) return launch_pair_x<RingP>(x, w, p, stream);
    if (mapped) return launch_pair_x<RingQM>(x, w, p, stream);
    return launch_pair_x<RingQ>(x, w, p, stream);
}

}  // namespace zr
