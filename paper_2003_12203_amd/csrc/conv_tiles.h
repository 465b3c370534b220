// The tiles of the convolution kernel (conv_kernel.h) and the arguments of their launches.
#pragma once

#include <type_traits>

#include "ftcnn_internal.h"
#include "encode_block.h"
#include "coc_tile.h"

namespace ftcnn {
namespace convk {

// Element-type traits: fp32 uses v_mfma_f32_32x32x2_f32 (2 k per instruction),
// bf16 uses v_mfma_f32_32x32x16_bf16 (16 k per instruction).  TK_ is the k
// extent of one LDS chunk; rows are padded by 16 bytes against bank conflicts.
template <int TK_> struct F32T {
    using T = float;
    static constexpr int TK = TK_;
    static constexpr int LDK = TK_ + 4;
    static constexpr int VEC = 4;      // elements per 16-byte load
    static constexpr int NP = 1;
};
template <int TK_> struct BF16T {
    using T = uint16_t;
    static constexpr int TK = TK_;
    static constexpr int LDK = TK_ + 8;
    static constexpr int VEC = 8;
    static constexpr int NP = 1;       // bf16 planes of an operand in the direct-to-LDS loop
};
// fp32 layers on split copies (Geom::split): 32-channel chunks of three bf16 planes.
template <int TK_> struct S3T {
    using T = float;
    static constexpr int TK = TK_;
    static constexpr int LDK = TK_ + 4;
    static constexpr int VEC = 4;
    static constexpr int NP = 3;
};

// DSTAGES > 0: the direct-to-LDS loop with that many stages of (TM + TP) rows of ROWB bytes.
template <typename Tr, int WM, int WP, int FM, int FP, bool KVEC_ = true, int DSTAGES = 0>
struct Cfg {
    using T = typename Tr::T;
    static constexpr bool KVEC = KVEC_;   // W rows 16-byte aligned: whole-slot weight loads
    static constexpr int NT = 64 * WM * WP;
    static constexpr int TM = WM * FM * 32;
    static constexpr int TP = WP * FP * 32;
    static constexpr int TK = Tr::TK;
    static constexpr int LDK = Tr::LDK;
    static constexpr int VEC = Tr::VEC;
    static constexpr int A_SLOTS = TM * TK / VEC;                    // 16-byte slots of the A tile
    static constexpr int A_PER = (A_SLOTS + NT - 1) / NT;
    static constexpr int KG = NT / TP;                               // threads per pixel along k
    static constexpr int KR = TK / KG;                               // k per thread in the gather
    static_assert(NT % TP == 0 && TK % KG == 0 && KR % VEC == 0, "tile shape");
    static_assert(KR <= 64 && A_PER * VEC <= 64, "gather masks are at most 64-bit");
    // one bit per gathered element of a thread
    using Mask = typename std::conditional<(KR > 32 || A_PER * VEC > 32), uint64_t, uint32_t>::type;
    static constexpr int ROWB = TK * 2 * Tr::NP;
    static constexpr size_t LDS_BYTES = DSTAGES > 0 ? (size_t)DSTAGES * (TM + TP) * ROWB
                                                    : 2ull * (TM + TP) * LDK * sizeof(T);
    static_assert(LDS_BYTES <= 160 * 1024, "tile exceeds the LDS of a CU");
};

// Epilogue arguments.  EPI 0: plain store.  EPI 1: the CoC-D summations of
// every stored value as well (Sec. 3.6): for each pixel p of the tile, the tile's
// rows give sum O, sum (m + wbase) O, (n + wbase) sum O and sum O^2, written as
// slice (tile_m * N + n) of a [slices][4][E*F] float64 array; block 0 resets the
// report.  EPI 2: EPI 1 with faults planted in the stored values first.
// With EPI 1 and 2, aux_groups groups of eight consecutive workgroup ids (one per
// XCD) may do other work of the protected layer instead of a tile, memory-bound work
// that runs beside the matrix-bound tiles of the same launch:
//   aux_kind 1: encode the input checksums Cd1, Cd2 of D (Sec. 3.2), in the first
//               groups of the grid (they read D as the first tiles do);
//   aux_kind 2: the Co5..Co7 partial products (coc_tile.h) of Cd1, Cd2 left by the
//               launch of the copies, in the last groups, after the tile_groups
//               groups of tiles, where they fill the slots the tiles' last round
//               leaves.
struct NoFaults {};
// D and (dense) W as given, for the outputs that a tile of split or packed copies computes again from them
struct Given {
    const void *d, *w;
};
// Stream-K schedule of the channels-last loops (S > 0): the launch has S workgroups (after the
// extra ones), as many as are resident at once.  The first dp_waves x S tiles run whole, tile
// r S + w being workgroup w's r-th, so that the workgroups resident together work on neighbouring
// tiles, as in the plain grid.  The last one to two waves' tiles (T of them) are shared evenly:
// workgroup w runs their iterations [w U / S, (w + 1) U / S) of the U = T x nch (tile, chunk)
// pairs in tile order.  A tile whose chunks span several workgroups is summed by the last of them
// to arrive: each writes its partial accumulators to a slot (0: the workgroup's first shared
// segment, 1: its last), counts itself in cnt[tile], and the last adds the slots in chunk order (a
// fixed order, whichever workgroup is last) before the epilogue.
struct SkArgs {
    float *part;    // [S][2][TM * TP]
    int *cnt;       // [tiles], zero at the launch (the channels-last copy clears it); left zero
    int S;          // 0: one tile per workgroup
    int nch;        // chunks per tile
    int dp_waves;   // waves of whole tiles before the shared ones
};
template <int EPI> struct Epi {
    double *part;
    ftcnn_report *rep;
    int cap;
    int aux_kind, aux_blocks, aux_groups;
    int tile_groups;     // groups of eight tile workgroups in front of the aux_kind 2 ones
    double *cd1, *cd2;   // kind 1: encoded here; kind 2: read
    int enc_vec;         // kind 1: 16-byte loads
    const double *cw1, *cw2;   // kind 2
    double *copart;
    CocTile co;
    int co_slices;       // Co partial slices this launch writes (recorded in rep->reserved[1])
    typename std::conditional<EPI == 2, FaultList, NoFaults>::type fl;
    const float *bias;   // NULL, or [M] added to every stored value of filter m (Sec. 5.1)
    Given src_dw;
};
template <> struct Epi<0> {
    const float *bias;
    Given src_dw;
};

// Main loops from 3 on load straight to LDS: 3 and 4 through a ring of two and three stages, 5 and 6 the
// same on packed copies (Geom::pk), 7 as 3 for kernels above 32 rows or columns.
constexpr bool packed_loop(int weave) { return weave == 5 || weave == 6; }
constexpr int dma_stages(int weave) { return weave >= 3 ? (weave == 4 || weave == 6 ? 3 : 2) : 0; }
// One tile configuration.  WEAVE: the main loop (0 register-staged, 1 gather woven between the
// MFMAs, 2 two chunks in flight, 3 to 7 direct-to-LDS).  run() and stream_k() are instantiated per tile
// in the conv_*.hip files.
template <typename Tr, int WM, int WP, int FM, int FP, int WEAVE> struct Tile {
    static constexpr int TM = WM * FM * 32;
    static constexpr int TP = WP * FP * 32;
    static constexpr int TK = Tr::TK;
    static constexpr int WEAVE_KIND = WEAVE;
    static constexpr int NT = Cfg<Tr, WM, WP, FM, FP>::NT;
    static constexpr size_t LDS_BYTES = Cfg<Tr, WM, WP, FM, FP, true, dma_stages(WEAVE)>::LDS_BYTES;
    static constexpr bool SK_FORM = (WEAVE == 3 || WEAVE == 4) && sizeof(typename Tr::T) == 4;
    // stream-K workgroups of the channels-last form on the current device (0: whole tiles)
    static int stream_k(const Geom &g, int smax);
    // NCHW: D and W as given; NHWC: the channels-last copies Dt and Wt (always aligned, K % VEC == 0)
    template <int EPI>
    static hipError_t run(const Geom &g, const void *D, const void *W, void *O, hipStream_t st, const Epi<EPI> &ep,
                          bool nhwc = false, const void *zp = nullptr, const SkArgs &sk = SkArgs{nullptr, nullptr, 0, 0, 0});
};

using F32_M32 = Tile<F32T<16>, 1, 4, 1, 2, true>;
using F32_M64 = Tile<F32T<16>, 2, 2, 1, 2, true>;
using F32_64x256 = Tile<F32T<16>, 1, 4, 2, 2, true>;   // channels-last M <= 64: 64 x 64 a wave
using F32_M96 = Tile<F32T<16>, 1, 4, 3, 1, true>;   // 96 x 128: AlexNet conv1 gets 1513 tiles, 3 full rounds
using F32_128x128 = Tile<F32T<16>, 2, 2, 2, 2, true>;
using F32_128x64 = Tile<F32T<32>, 2, 2, 2, 1, true>;
using F32_64x64 = Tile<F32T<32>, 2, 2, 1, 1, true>;
// fp32 on split copies.  128 x 256: eight waves of 64 x 64, a two-stage ring of 72 KB stages; 128 x 128:
// eight waves of 64 x 32, three stages of 48 KB (with two a chunk's loads have one short chunk to land: Darknet-19 1x1 43.4 -> 44.0 us
// protected, AlexNet conv4 163 in both); 64 x 64, three stages: layers of few tiles; 64 x 128 and 32 x 128: few
// filters.
using S3_128x256 = Tile<S3T<32>, 2, 4, 2, 2, 3>;
using S3_128x128 = Tile<S3T<32>, 2, 4, 2, 1, 4>;
using S3_64x64 = Tile<S3T<32>, 2, 2, 1, 1, 4>;
using S3_64x128 = Tile<S3T<32>, 1, 4, 2, 1, 3>;
using S3_32x128 = Tile<S3T<32>, 1, 4, 1, 1, 3>;
// kernels above 32 rows or columns
using S3W_64x128 = Tile<S3T<32>, 1, 4, 2, 1, 7>;
using S3W_128x128 = Tile<S3T<32>, 2, 4, 2, 1, 7>;
using BF16W_64x128 = Tile<BF16T<64>, 1, 4, 2, 1, 7>;
using BF16W_128x128 = Tile<BF16T<64>, 2, 2, 2, 2, 7>;
// packed copies
using S3P_32x128 = Tile<S3T<32>, 1, 4, 1, 1, 5>;
using S3P_64x128 = Tile<S3T<32>, 1, 4, 2, 1, 5>;
using S3P_96x256 = Tile<S3T<32>, 1, 8, 3, 1, 5>;
using S3P_128x128 = Tile<S3T<32>, 2, 4, 2, 1, 6>;
using S3P_64x64 = Tile<S3T<32>, 2, 2, 1, 1, 6>;
using BF16P_64x128 = Tile<BF16T<64>, 1, 4, 2, 1, 5>;
using BF16P_64x256 = Tile<BF16T<64>, 1, 8, 2, 1, 5>;
using BF16P_128x128 = Tile<BF16T<64>, 2, 2, 2, 2, 5>;
using BF16P_64x64 = Tile<BF16T<64>, 2, 2, 1, 1, 5>;
using BF16_M32 = Tile<BF16T<32>, 1, 4, 1, 2, 0>;
using BF16_M64 = Tile<BF16T<32>, 1, 4, 2, 2, 2>;
using BF16_128x128_K64 = Tile<BF16T<64>, 2, 2, 2, 2, 2>;
using BF16_256x256 = Tile<BF16T<32>, 2, 2, 4, 4, 2>;
using BF16_DMA_128x128 = Tile<BF16T<64>, 2, 2, 2, 2, 3>;
// Three stages, for layers whose tiles are about one a compute unit, where a chunk's loads have only the
// tile's own matrix work to land behind: eight waves of 64 x 32 (against the 128 x 64 tile of four waves
// and two stages that these layers ran: VGG-19 v14 46.7 -> 41.5 us for the convolution, ResNet-18 l4
// 47.4 -> 42.0, VGG-19 v10 at batch 8 46.6 -> 40.7; with two tiles a compute unit two stages are the
// faster, ResNet-18 l3 39.0 against 45.6), and 64 x 64 where even those are few (VGG-19 v14 at batch 8
// 41.6 -> 26.5 us, at batch 1 41.6 -> 25.0; shared by stream-K workgroups at batch 8 32.4).
using BF16_DMA_128x128_3 = Tile<BF16T<64>, 2, 4, 2, 1, 4>;
using BF16_DMA_64x64_3 = Tile<BF16T<64>, 2, 2, 1, 1, 4>;
// M <= 64: four waves of 64 x 32, a 48 KB ring, three workgroups a compute unit (against 64 x 256
// tiles of four 64 x 64 waves, two a compute unit: ResNet-18 l1 89 -> 79 us, VGG-19 v2 299 -> 287 us
// with the channels-last copy; 64 x 64 tiles of two waves, 64 x 128 of two waves and deeper rings
// were slower)
using BF16_DMA_64x128 = Tile<BF16T<64>, 1, 4, 2, 1, 3>;
// eight waves of 128 x 64 (two a SIMD, accumulators in 128 registers a lane): against four waves
// of 128 x 128 (one a SIMD) 5-8 % faster on VGG-19 bf16 v5-v12, which also beat 128 x 128 tiles
using BF16_DMA_256x256 = Tile<BF16T<64>, 2, 4, 4, 2, 3>;

// What a split layer's tiles take (us), as measured on one MI355X: chunk_idle + chunk_busy * (share of the
// chip's slots in use) a chunk, since busy matrix cores lower the clock, `tile` a tile beyond its
// chunks, and `shared` more where tiles are shared (publishing a workgroup's part and summing a
// tile's parts).  Fitted for the least time lost to the choice over 399 layers (the workloads' and drawn ones of 33
// and more filters, each on every tile): 1.0 % on average, 12 of them lose more than 10 %; constants fitted to
// half of them lose 1.0 and 1.5 % on the other half, those of the kernels that added their products to the
// accumulators themselves lost 2.1 %, 33 layers more than 10 %.
struct TileCost {
    int resident;   // workgroups on the chip at once
    double chunk_idle, chunk_busy, tile, shared;
};
// Stream-K pays where whole tiles leave the last round of workgroups partly idle, or never fill the
// chip, by more than sharing costs; a workgroup keeps at least kSkMinChunks chunks, and tiles of few
// chunks are not shared (1 x 1 layers of 128 to 256 channels: 4 to 8 chunks, shared tiles 28-50 % slower).
constexpr int kSkMinChunks = 16, kSkMinTile = 24;
inline int stream_k_size(long long tiles, int resident, int nch) {
    const long long fill = tiles * nch / kSkMinChunks;
    if (nch < kSkMinTile) return 0;
    if (fill >= resident) return resident;
    return fill / 8 * 8 > tiles ? (int)(fill / 8 * 8) : 0;
}
inline double whole_cost(const TileCost &t, long long tiles, int resident, double nch) {
    const long long full = tiles / resident, rem = tiles % resident;
    const double busy = (double)rem / resident;
    return full * (nch * (t.chunk_idle + t.chunk_busy) + t.tile) +
           (rem ? nch * (t.chunk_idle + t.chunk_busy * busy) + t.tile : 0.0);
}
inline double shared_cost(const TileCost &t, long long tiles, int resident, int nch, int S) {
    return (double)(tiles * nch) / S * (t.chunk_idle + t.chunk_busy * S / resident) + t.tile + t.shared;
}
// Stream-K workgroups of a layer on this tile, 0 for one workgroup per tile.
inline int stream_k_workgroups(const TileCost &t, long long tiles, int resident, int nch) {
    const int S = stream_k_size(tiles, resident, nch);
    return S > 0 && shared_cost(t, tiles, resident, nch, S) < whole_cost(t, tiles, resident, nch) ? S : 0;
}
template <typename Tl> constexpr TileCost tile_cost() { return TileCost{kComputeUnits, 1.0, 0.0, 4.0, 20.0}; }
template <> constexpr TileCost tile_cost<S3_128x256>() { return TileCost{kComputeUnits, 1.32, 0.82, 5.5, 23.0}; }
template <> constexpr TileCost tile_cost<S3_128x128>() { return TileCost{kComputeUnits, 0.62, 0.51, 4.5, 20.0}; }
template <> constexpr TileCost tile_cost<S3_64x64>() { return TileCost{2 * kComputeUnits, 0.56, 0.17, 2.2, 13.5}; }
template <> constexpr TileCost tile_cost<S3_64x128>() { return TileCost{2 * kComputeUnits, 0.80, 0.20, 2.0, 16.0}; }
template <> constexpr TileCost tile_cost<S3_32x128>() { return TileCost{2 * kComputeUnits, 0.60, 0.10, 2.0, 14.0}; }

}  // namespace convk
}  // namespace ftcnn
