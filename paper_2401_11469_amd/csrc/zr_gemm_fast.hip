// Launches of the fast path: which tile shapes and loaders a bf16 product of 16-byte aligned rows takes
// (the kernels stand in zr_gemm_fast.h).
#include "zr_gemm_fast.h"

namespace zr {

namespace {

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
template <template <int, int> class LA, template <int, int> class LB, int BM, int BN, int WM, int WN>
int launch_inst(const FArgs& a, int i_base, int i_end, int j_base, int j_end, hipStream_t stream, int slot_base)
{
    typedef LA<BM, 64 * WM * WN> A;
    typedef LB<BN, 64 * WM * WN> B;
    constexpr bool ring = A::RING;
    constexpr int list_bytes = [] { if constexpr (ring) return (A::MAPPED || B::MAPPED) ? ring_list_max<BM, BN>() * 4 : 0; else return 0; }();
    constexpr int smem = fast_smem_bytes<A::WORDS, B::WORDS, BM, BN, ring>() + list_bytes;
    static_assert(smem <= 160 * 1024, "LDS of a workgroup");
    auto fn = fast_kernel<LA, LB, BM, BN, WM, WN>;
    static AttrFlags attr_set;      // per instantiation and device
    if (!ensure_max_dynamic_lds((const void*)fn, smem, &attr_set)) return ZR_ERR_HIP;
    if (debug_names_wanted())
        snprintf(g_debug.last_kernel, sizeof(g_debug.last_kernel), "fast_kernel<%s, %s, %d, %d, %d, %d>",
                 A::NAME, B::NAME, BM, BN, WM, WN);
    FArgs k = a;
    k.i_base = i_base; k.i_end = i_end; k.j_base = j_base; k.j_end = j_end;
    k.avg_slot_base = slot_base;
    k.tiles_i = (i_end - i_base + BM - 1) / BM;
    k.tiles_j = (j_end - j_base + BN - 1) / BN;
    const int64_t tiles = (int64_t)k.tiles_i * k.tiles_j;
    if (tiles > 0x7ffffff0) return ZR_ERR_LIMIT;
    k.split = 1; k.kt_per = 0;
    // Split contraction: when this launch has too few tiles for the chip and a long contraction,
    // s slices per tile (s * tiles workgroups), then a launch that adds the slices and runs the
    // epilogue.  Needs scratch for the slices (the caller's workspace).
    // (Tried on the big ring tiles of the dW products at high pruning ratios as well, 128 tiles
    // of 192 x 256 in two slices each: the slices are 50 MB of fp32 that leave the chip at the
    // end of the first launch and come back in the second, ~35 us per product, which is all
    // that the better fill of the chip gains.  A product on its own has no such form; a dW in one
    // launch with its dX has, see zr_gemm_pair.hip: there the slices run beside the tiles of dX.)
    constexpr bool can_split = A::DMA && B::DMA && !ring && BM == 128 && BN == 128;
    if constexpr (can_split) {
        const int sp = slices_for(a.C, tiles, a.partial, a.partial_bytes, a.accumulate != 0);
        if (sp >= 2) {
            const int KT = (a.C + BK - 1) / BK;
            k.kt_per = (KT + sp - 1) / sp;
            k.split = (KT + k.kt_per - 1) / k.kt_per;                      // no empty slice
            auto fn1 = fast_kernel<LA, LB, BM, BN, WM, WN, 1>;
            static AttrFlags attr1;
            if (!ensure_max_dynamic_lds((const void*)fn1, smem, &attr1)) return ZR_ERR_HIP;
            const int64_t g1 = (tiles * k.split + 7) / 8 * 8;
            hipLaunchKernelGGL(fn1, dim3((unsigned)g1), dim3(64 * WM * WN), smem, stream, k);
            if (hipGetLastError() != hipSuccess) return ZR_ERR_HIP;
            if (a.avg_partial && a.epilogue == EPI_ROW_SCATTER)
                hipLaunchKernelGGL(split_reduce_kernel<4>, dim3((unsigned)tiles), dim3(1024), 0, stream, k);
            else
                hipLaunchKernelGGL(split_reduce_kernel<1>, dim3((unsigned)(tiles * 4)), dim3(256), 0, stream, k);
            if (debug_names_wanted()) {
                char nm[128];
                snprintf(nm, sizeof(nm), "%.90s split %d", g_debug.last_kernel, k.split);
                snprintf(g_debug.last_kernel, sizeof(g_debug.last_kernel), "%s", nm);
            }
            return hip_status(hipGetLastError());
        }
    }
    const int64_t grid = (tiles + 7) / 8 * 8;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(64 * WM * WN), smem, stream, k);
    return hip_status(hipGetLastError());
}

template <template <int, int> class LA, template <int, int> class LB, int BM, int BN, int WM, int WN>
int launch_tile(const FArgs& a, int i_base, int i_end, int j_base, int j_end, hipStream_t stream, int slot_base = 0)
{
    if (i_end <= i_base || j_end <= j_base) return ZR_OK;
    if constexpr (RingOf<LA>::has && RingOf<LB>::has) {
        constexpr int NT = 64 * WM * WN;
        typedef typename RingOf<LA>::template type<BM, NT> RA;
        typedef typename RingOf<LB>::template type<BN, NT> RB;
        constexpr int TM = BM / (16 * WM), TN = BN / (16 * WN);
        constexpr int ring_a = TM % 4 == 0 ? 4 : 3;
        // the ring schedule needs whole load instructions per wavefront and enough MFMA slots
        // (and tiles above 128 x 128: the small tiles, four wavefronts and two workgroups to a compute
        // unit, measured 10-25 % slower with a barrier every 32 instead of every 64)
        constexpr bool fits = RA::FITS && RB::FITS && TM % ring_a == 0 && TM >= 4 && TN >= 4 && RA::NI + RB::NI <= TM &&
                              (TN <= TM - 1 || 2 * (TM - 1) >= TN) && BM * BN > 128 * 128;
        if constexpr (fits) {
            const bool list_ok = !(RA::MAPPED || RB::MAPPED) || a.C <= ring_list_max<BM, BN>();
            if (ring_enabled() && list_ok) {
                // (named directly, so that a profiler prints the loaders' own names)
                constexpr bool ap = std::is_same<RA, RingP<BM, NT>>::value, aq = std::is_same<RA, RingQ<BM, NT>>::value;
                constexpr bool bp = std::is_same<RB, RingP<BN, NT>>::value, bq = std::is_same<RB, RingQ<BN, NT>>::value;
                constexpr bool bm = std::is_same<RB, RingQM<BN, NT>>::value;
                static_assert((ap && (bp || bq || bm)) || (aq && bq), "loader pair without a ring instantiation");
                if constexpr (ap && bp) return launch_inst<RingP, RingP, BM, BN, WM, WN>(a, i_base, i_end, j_base, j_end, stream, slot_base);
                else if constexpr (ap && bq) return launch_inst<RingP, RingQ, BM, BN, WM, WN>(a, i_base, i_end, j_base, j_end, stream, slot_base);
                else if constexpr (ap && bm) return launch_inst<RingP, RingQM, BM, BN, WM, WN>(a, i_base, i_end, j_base, j_end, stream, slot_base);
                else return launch_inst<RingQ, RingQ, BM, BN, WM, WN>(a, i_base, i_end, j_base, j_end, stream, slot_base);
            }
        }
    }
    return launch_inst<LA, LB, BM, BN, WM, WN>(a, i_base, i_end, j_base, j_end, stream, slot_base);
}

template <template <int, int> class LA, template <int, int> class LB>
int launch_shape(const FArgs& a, hipStream_t stream)
{
    if (const int f = forced_tiles()) {
        if constexpr (LA<256, 512>::DMA && LB<256, 512>::DMA) {
            if (f == 2) return launch_tile<LA, LB, 192, 256, 2, 4>(a, 0, a.I, 0, a.J, stream);
            if (f == 3) return launch_tile<LA, LB, 256, 192, 4, 2>(a, 0, a.I, 0, a.J, stream);
        }
        if constexpr (std::is_same<LA<64, 256>, DmaP<64, 256>>::value && std::is_same<LB<128, 256>, DmaP<128, 256>>::value)
            if (f == 5) return launch_tile<LA, LB, 64, 128, 1, 4>(a, 0, a.I, 0, a.J, stream);
        if (f >= 4) return launch_tile<LA, LB, 128, 128, 2, 2>(a, 0, a.I, 0, a.J, stream);
        return launch_tile<LA, LB, 256, 256, ZR_BIG_WM, ZR_BIG_WN>(a, 0, a.I, 0, a.J, stream);
    }
    const Sched sc = plan_tiles(a.I, a.J);
    if constexpr (LA<256, 512>::DMA && LB<256, 512>::DMA) {
        const int64_t tj = tiles_of(a.I, a.J, 256, 192), ti = tiles_of(a.I, a.J, 192, 256);
        const double cj = cost_192(tj), ci = cost_192(ti);
        if (std::min(cj, ci) < sc.cost - 1e-9) {
            // equal rounds: the grid with fewer tiles has less padding
            if (cj < ci || (cj == ci && tj <= ti)) return launch_tile<LA, LB, 256, 192, 4, 2>(a, 0, a.I, 0, a.J, stream);
            return launch_tile<LA, LB, 192, 256, 2, 4>(a, 0, a.I, 0, a.J, stream);
        }
    }
    if constexpr (std::is_same<LA<64, 256>, DmaP<64, 256>>::value && std::is_same<LB<128, 256>, DmaP<128, 256>>::value) {
        // 64 x 128 tiles, three to a compute unit, while 128 x 128 ones would leave units with one
        // (1024 deep: 192 tiles 19.8 -> 15.7 us, 384 tiles 25 -> 22.7; 2048 deep 384 tiles 36.1 -> 36.7,
        // 480 tiles 38.5 -> 53).  With a row list on the contraction they are slower (512 tiles 24 -> 33).
        const int64_t t = tiles_of(a.I, a.J, 128, 128);
        if (sc.big_i_end == 0 && (t <= 256 || (t <= 384 && a.C <= 1024)) &&
            slices_for(a.C, t, a.partial, a.partial_bytes, a.accumulate != 0) < 2)
            return launch_tile<LA, LB, 64, 128, 1, 4>(a, 0, a.I, 0, a.J, stream);
    }
    if (sc.big_i_end == 0)                     // everything on small tiles
        return launch_tile<LA, LB, 128, 128, 2, 2>(a, 0, a.I, 0, a.J, stream);
    int st = launch_tile<LA, LB, 256, 256, ZR_BIG_WM, ZR_BIG_WN>(a, 0, sc.big_i_end, 0, sc.big_j_end, stream);
    if (st != ZR_OK || (sc.big_i_end >= a.I && sc.big_j_end >= a.J)) return st;
    char big[128];
    if (debug_names_wanted()) snprintf(big, sizeof(big), "%s", g_debug.last_kernel);
    // Average sums: the remainder panel's tiles continue the slot numbering of the big
    // panel along the summed axis when the cut runs across that axis; panels that
    // cover different output rows (columns) never meet in a slot
    const bool sums_over_j = a.epilogue == EPI_COL_SCATTER;
    if (sc.cut_rows) st = launch_tile<LA, LB, 128, 128, 2, 2>(a, sc.big_i_end, a.I, 0, a.J, stream,
                                                              sums_over_j ? 0 : sc.big_i_end / 256);
    else st = launch_tile<LA, LB, 128, 128, 2, 2>(a, 0, a.I, sc.big_j_end, a.J, stream,
                                                  sums_over_j ? sc.big_j_end / 256 : 0);
    if (debug_names_wanted())
        snprintf(g_debug.last_kernel, sizeof(g_debug.last_kernel), "%.60s + 128x128 remainder panel", big);
    return st;
}

}  // namespace

// Whether this path has a kernel for the product: rows of 16-byte chunks, and loaders for the pair of operands.
bool gemm_fast_can(const GemmDesc& d)
{
    if (d.dtype != ZR_BF16) return false;
    auto aligned = [](const void* p, int64_t ld) { return ((uintptr_t)p % 16 == 0) && (ld % 8 == 0); };
    if (!aligned(d.A.base, d.A.ld) || !aligned(d.B.base, d.B.ld) || !aligned(d.out, d.ldo)) return false;
    // every memory row that is walked in 16-byte chunks must be a multiple of 8 long
    auto chunked_ok = [](const Operand& o) {
        if (o.map_contig) {
            if (o.map_strided) return false;
            return o.c_contig ? o.n_contig % 2 == 0 : o.n_contig % 8 == 0;   // PG reads aligned dwords, QG chunks
        }
        return o.n_contig % 8 == 0;
    };
    if (!chunked_ok(d.A) || !chunked_ok(d.B)) return false;
    if (d.epilogue != EPI_COL_SCATTER && d.J % 8 != 0) return false;
    if (d.I < 1 || d.J < 1 || d.C < 1) return false;
    if (d.prev && (uintptr_t)d.prev % 16 != 0) return false;
    if (d.accumulate && d.epilogue != EPI_PLAIN) return false;
    // which pairs of operands there are loaders for
    const bool ag = d.A.map_contig != nullptr, bg = d.B.map_contig != nullptr;
    const bool ap = d.A.c_contig, bp = d.B.c_contig;
    if ((!ap && bp) || (ag && bg)) return false;
    if (ap && bp && ag) return false;
    if (!ap && (d.A.map_strided || d.B.map_strided)) return false;
    return true;
}

// contractions of whole 64-deep stages, or with an operand that is padded to them
static bool whole_stages(const GemmDesc& d)
{
    return d.C % BK == 0 || (d.A.c_contig && d.A.zero_padded) || (d.B.c_contig && d.B.zero_padded);
}

// Slices of the contraction that its launch on 128 x 128 tiles will make.  (Two slices of a contraction of no whole stages
// below 1344 gain nothing: 216 tiles, 1264 deep 26 us in one piece, 30 in two.)
static bool short_for_slices(const GemmDesc& d) { return !whole_stages(d) && d.C < 1344; }
static int slices_of(const GemmDesc& d, int64_t t128)
{
    return short_for_slices(d) ? 1 : slices_for(d.C, t128, d.split_scratch, d.split_scratch_bytes, d.accumulate);
}

// Whether this path takes the product (else the kernel for any alignment does).
bool gemm_fast_takes(const GemmDesc& d)
{
    if (!gemm_fast_can(d)) return false;
    if (forced_tiles()) return true;
    const bool ag = d.A.map_contig != nullptr, bg = d.B.map_contig != nullptr;
    const bool ap = d.A.c_contig, bp = d.B.c_contig;

    // Where the kernel for any alignment is the faster one, although this path could run: its tiles
    // are smaller, and so are its stages, which is what counts while the chip is not full.  By the
    // number of 128 x 128 tiles (us on this path / on the other one, 1024 deep unless given):
    // (Column scatters of plain activations into rows whose width is no multiple of 8 although their pitch is
    // stay here at any size, where the parity tests expect them: 1000 x 1024 x 780 15.5 / 10.1, 270 x 520 x 300
    // 20.9 / 9.9, 2000 x 1024 x 1500 18.2 / 18.1.)
    const int64_t t128 = tiles_of(d.I, d.J, 128, 128);
    if (ap && d.epilogue == EPI_COL_SCATTER && d.out_full % 8 != 0) return true;
    const bool whole = whole_stages(d);
    const bool split = !ag && !bg && slices_of(d, t128) >= 2;
    if (split && whole) return true;                // (48 tiles, 4096 tokens: 21 / 30)
    // Products that the other kernel adds up in groups of the contraction are all its own, so that a
    // result has the same bits whichever of its operands were extracted beforehand (64 x 8192, 4096 deep: 38 / 18).
    if (adds_in_groups(d.I, d.J, d.C)) return false;
    if (ap && ag) return t128 > 512;                // X[:,S] in flight: 160 tiles 36 / 27, 512 44 / 36, 800 (768 deep) 53 / 64
    if (ap && bp && bg) return t128 > 256;          // W[:,S] along the contraction: 128 tiles 27 / 20, 256 28.5 / 25, 792 91 / 126
    if (ap && bg) return t128 > 128;                // W[:,S] across it: 100 tiles 28.2 / 25.5 (256 deep 16.1 / 13.3, 4096 81 / 74), 128 28.7 / 25.7, 192 30 / 37
    if (ag || bg) return t128 > 96;                 // dW, a gather in flight, 4096 tokens: 48 tiles 84 / 47, 192 84 / 115
    if (!whole) {
        // The last stage is the same work for less, and rows of such a length straddle cache lines.  2518 products of 60 to
        // 260 tiles, 8 to 6000 deep, time on this path by that on the other one, by depth; split: all of W in two or more
        // slices, 128 tiles 1.34 (1600 deep) 1.12 (2048) 0.95 (3200), 160 tiles 1.05 (1600) 0.88 (2048), 192 tiles 0.96 (1600);
        if (ap && !bp) return split ? t128 > 160 || d.C > (t128 > 128 ? 1600 : 2304)
        //   in one piece, 192 tiles 0.78 (1152) 0.86 (1600); 129 to 160 tiles would be the faster here to 1152 deep (776 deep
        //   15.3 us / 17.9), and from 769 deep stay where tests/test_gpu_dispatch_rules.py has them;
                                    : t128 > (d.B.map_strided ? 256 : d.C <= 768 ? 128 : 160);
        // rows of W: split, 128 tiles 1.31 (1600) 1.10 (2560) 0.91 (above 3200); in one piece below three stages (LdPV) 1.06 to
        // 1.17 at any number of tiles to 128, to 1152 deep 0.87 to 0.98, above 1.2 to 1.3;
        if (ap) return t128 > 128 || (split ? d.C > 2560 : t128 > 64 && d.C >= 3 * BK && d.C <= 1152);
        // dW: split, 128 tiles 1.11 (1600 tokens) 1.01 (2048) 0.89 (2560), 160 tiles 1.2 (1152) 0.9 (1600), 192 tiles 0.84; in one
        // piece 0.7 to 1.0, but where dropped rows are copied 144 tiles 1.09 to 1.23, 176 tiles 1.05, 192 tiles 0.98, half
        // of them dropped 180 tiles 1.25, 198 tiles 1.5
        return split ? t128 > 128 || d.C > 1664
                     : t128 > (d.prev && d.epilogue == EPI_ROW_SCATTER ? 256 : 128);
    }
    // rows of W: 64 tiles 18 / 9, 256 19 / 17, 512 (1536 deep) 43 / 38, 1600 53 / 68; all of W: 128 13.6 / 11.8, 160 14 / 18,
    // 256 14.8 / 19.5
    if (ap && !bp) return t128 > (d.B.map_strided ? 256 : 128);
    if (ap) return t128 > 64;                       // 48 tiles 12.5 / 11, 96 14 / 16.5
    return t128 > 128;                              // dW: 48 tiles 18 / 12.6
}

// Whether the product leaves the sums of Average imputation in avg_partial.  One that is split as a whole
// has a result that the stand-alone pass reads from the caches, in one launch instead of three; many kept rows are a
// long chain there (us with the sums / with that pass: dW 768 x 4096 of 576 kept rows 74 / 71, 1024 x 2048 of 1536
// kept columns 86 / 82, 4096 x 768 of 3072 kept rows 93 / 103).  The sums need three launches (clear, finish, fill: 13 us)
// where the pass over the columns of a small result is one of 6 to 12 (880 x 2568 26 / 21, 1500 x 2568 27 / 24; 8192 x 3072 240 / 263).
bool gemm_leaves_sums(const GemmDesc& d)
{
    if (d.epilogue == EPI_PLAIN || !gemm_fast_takes(d)) return false;
    if (d.epilogue == EPI_COL_SCATTER && (int64_t)d.I * d.out_full < 8 << 20 && !forced_tiles()) return false;
    const bool split = slices_of(d, tiles_of(d.I, d.J, 128, 128)) >= 2;
    return !split || (d.epilogue == EPI_ROW_SCATTER && d.I > 1536);
}

// Returns -1 when the problem is not eligible, else a zr_status.
int launch_gemm_fast(const GemmDesc& d, hipStream_t stream)
{
    if (!gemm_fast_takes(d)) return -1;
    FArgs a = fargs_of(d);
    if (short_for_slices(d)) { a.partial = nullptr; a.partial_bytes = 0; }
    const bool ag = d.A.map_contig != nullptr, bg = d.B.map_contig != nullptr;
    if (d.A.c_contig && !d.B.c_contig) {            // forward: X rows, W columns
        const bool bm = d.B.map_strided != nullptr;        // W[S[c], :]: the row list is on the contraction axis
        if (!ag && !bg) {
            return bm ? launch_shape<DmaP, DmaQM>(a, stream) : launch_shape<DmaP, DmaQ>(a, stream);
        }
        if (ag && !bg) return launch_shape<LdPG, DmaQM>(a, stream);
        if (!ag && bg) return launch_shape<DmaP, LdQG>(a, stream);
        return -1;
    }
    if (d.A.c_contig && d.B.c_contig) {             // dX
        if (!ag && !bg) {
            // two stages and a part of one take the same time on the register-staged loaders (136 deep 11.3 / 11.2 us,
            // 72 deep 25.8 / 25.2; 200 deep 12.2 / 11.8, 1000 deep 25.6 / 23.4)
            if (d.C % BK != 0 && d.C < 3 * BK && !d.A.zero_padded && !d.B.zero_padded) return launch_shape<LdPV, LdPV>(a, stream);
            return launch_shape<DmaP, DmaP>(a, stream);
        }
        if (!ag && bg) return launch_shape<DmaP, LdPG>(a, stream);
        return -1;
    }
    if (!d.A.c_contig && !d.B.c_contig) {           // dW: the contraction runs over the tokens, never through a list
        if (d.A.map_strided || d.B.map_strided) return -1;
        if (!ag && !bg) return launch_shape<DmaQ, DmaQ>(a, stream);
        if (ag && !bg) return launch_shape<LdQG, DmaQ>(a, stream);
        if (!ag && bg) return launch_shape<DmaQ, LdQG>(a, stream);
        return -1;
    }
    return -1;
}

}  // namespace zr
