// The layer's convolution, eq. (1): the choice of its tile, and its launches (the kernel is in
// conv_kernel.h, its tiles in conv_tiles.h, their instantiations in the conv_*.hip files).
#include <algorithm>

#include "conv_tiles.h"

namespace ftcnn {
using namespace convk;
namespace {

// Tile choice per layer, from sweeps over the workload shapes and drawn layers on MI355X.  The filter tile
// follows M so small-M layers waste no MFMA rows.
//
// fp32 layers of 32-channel multiples run on split copies (three bf16 planes a value, six products) where
// that is predicted to be the faster (split_pays): the bf16 matrix cores do six products in 3/8 of the time
// the fp32 ones take for one, and errors are smaller (VGG-19 v6 protected: 1010 -> 647 us, distance from
// float64 7.7e-7 -> 2.1e-7 of the norm).  Their tile and its schedule are the ones with the least
// predicted time (split_cost).  The others take fp32 copies: 64 x 256 tiles for M <= 64, else 128 x 128,
// 128 x 64 or 64 x 64.
//
// bf16 layers of 64-channel multiples take direct-to-LDS loads from channels-last copies (WEAVE 3, 4): 64 x 128
// tiles for M <= 64, 256 x 256 tiles (eight waves of 128 x 64) for M >= 256 where there are enough of them,
// 128 x 128 elsewhere, through three stages where they would not fill the compute units, and 64 x 64
// where those are few.
//
// Layers of other channel counts run on packed copies through the same loops (WEAVE 5, 6) where that is
// predicted to be the faster (pack_pays).  The rest (most short sums and small layers, copies past 32-bit
// offsets) load through registers: bf16 64 x 256, 256 x 256 or 128 x 128 tiles with two chunks in flight
// (WEAVE 2), from channels-last copies (32-channel multiples) or D and W as given; fp32 tiles as above.
long long n_tiles(const Geom &g, int tm, int tp) {
    return ((g.P_total + tp - 1) / tp) * (long long)((g.M + tm - 1) / tm);
}

// The channels that a tile of tm filters walks: the 32-channel blocks that its filters' groups reach into, on
// average (tiles that straddle two groups walk both).
double mean_channels(const Geom &g, int tm) {
    if (g.G == 1) return g.C;
    long long blocks = 0, tiles = 0;
    for (int m0 = 0; m0 < g.M; m0 += tm, ++tiles) {
        const int last = (std::min(m0 + tm, g.M) - 1) / g.Mg;
        blocks += ((last + 1) * g.Cg + 31) / 32 - group_first_channel(g, m0) / 32;
    }
    return 32.0 * (double)blocks / (double)tiles;
}

// The predicted time of a split layer's convolution on a tile, on whole tiles or shared ones; with_fetch: no less
// than its operands take to arrive.
template <typename Tl> double split_cost(const Geom &g, bool with_fetch) {
    constexpr TileCost c = tile_cost<Tl>();
    const long long tiles = n_tiles(g, Tl::TM, Tl::TP);
    const double whole = whole_cost(c, tiles, c.resident, g.R * g.S * mean_channels(g, Tl::TM) / 32);
    const int nch = g.R * g.S * (g.C / 32), S = g.G > 1 || !g.sk ? 0 : stream_k_size(tiles, c.resident, nch);
    if (S <= 0) return whole;
    double shared = shared_cost(c, tiles, c.resident, nch, S);
    if (with_fetch) {
        // Workgroups that share tiles are at chunks of their own, and no L2 serves two of them: the operands' bytes
        // bound the shared tiles, at about 14 TB/s from the Infinity Cache and half of that past its size, and
        // such a layer takes a larger tile (protected, 16 x 512 x 14^2, 512 filters of 3 x 3: 64 x 64 tiles 141 us,
        // 128 x 128 116; 3 x 608 x 43^2, 448 of 11 x 11 at stride 4: 438 and 363; 9 x 352 x 74^2, 320 of 11 x 11 at
        // stride 4: 1031, 128 x 256 697)
        const long long waves = (tiles + S - 1) / S, rest = tiles - (waves > 2 ? waves - 2 : 0) * S;
        const double copies = 6.0 * ((double)g.N * (double)g.CHW + (double)g.M * g.K);
        const double fetch = (double)rest * nch * (Tl::TM + Tl::TP) * 192 / (copies < 128e6 ? 14e6 : 7e6);
        const double busy = (double)rest * nch / S * (c.chunk_idle + c.chunk_busy * S / c.resident);
        shared += std::max(fetch - busy, 0.0);
        // and the last workgroup of a tile adds all its parts, at about 90 GB/s, which counts where they are many (6 x
        // 960 x 58 x 19, 160 filters of 11 x 11 at stride 4: 254 us for the convolution on two 128 x 256 tiles of 113
        // parts, 167 on twelve 64 x 64 ones)
        shared += std::max((double)S / tiles - 32.0, 0.0) * Tl::TM * Tl::TP * 4 / 9e4;
    }
    return std::min(whole, shared);
}

// Calls f(TileType{}) for the tile this layer uses (nhwc: the launch reads the
// channels-last copies).
template <typename Fn>
auto with_tile(const Geom &g, bool nhwc, Fn &&f) {
    if (nhwc && g.pk) {
        if (g.dtype == FTCNN_BF16) {
            if (g.M <= 64) return n_tiles(g, 64, 256) >= 512 ? f(BF16P_64x256{}) : f(BF16P_64x128{});
            return n_tiles(g, 128, 128) >= kComputeUnits ? f(BF16P_128x128{}) : f(BF16P_64x64{});
        }
        if (g.M <= 32) return f(S3P_32x128{});
        if (g.M <= 64) return f(S3P_64x128{});
        if (g.M <= 96 && n_tiles(g, 96, 256) >= kComputeUnits) return f(S3P_96x256{});
        return n_tiles(g, 128, 128) >= 128 ? f(S3P_128x128{}) : f(S3P_64x64{});
    }
    const bool wide = g.R > 32 || g.S > 32;
    if (nhwc && g.split) {
        if (wide) return g.M <= 64 ? f(S3W_64x128{}) : f(S3W_128x128{});
        if (g.M <= 32) return f(S3_32x128{});
        // the tile with the least predicted time
        auto cost = [&](auto t) { return split_cost<decltype(t)>(g, true); };
        const double c64 = cost(S3_64x64{});
        if (g.M <= 64) return c64 <= cost(S3_64x128{}) ? f(S3_64x64{}) : f(S3_64x128{});
        const double c128 = cost(S3_128x128{}), c256 = cost(S3_128x256{});
        if (c256 <= c128 && c256 <= c64) return f(S3_128x256{});
        return c128 <= c64 ? f(S3_128x128{}) : f(S3_64x64{});
    }
    if (g.dtype == FTCNN_F32) {
        if (g.M <= 32) return f(F32_M32{});
        // on channels-last layers a wave of the 64 x 256 tile holds 64 x 64 outputs, as in the
        // 128 x 128 tile (VGG-19 v2 1309 -> 1284 us, Darknet-19 c2 349 -> 334 us protected)
        if (g.M <= 64) return nhwc ? f(F32_64x256{}) : f(F32_M64{});
        if (g.M <= 96) return f(F32_M96{});
        // grouped layers: rows of tiles inside one group, so that every tile skips the other
        // groups' channels (192 filters a group: 64-row tiles)
        if (g.G > 1 && g.Mg % 128 != 0 && g.Mg % 64 == 0) return f(F32_64x64{});
        // the tile with the least predicted time: the padded outputs (tiles x TM x TP), plus half of
        // the idle slots in the last round of a tile a compute unit, at the tile's own rate per output
        // (128 x 128 : 128 x 64 : 64 x 64 = 1 : 0.972 : 0.925).  The one-half and the rates are
        // fitted to VGG-19 (224^2 .. 14^2, batch 32) and Darknet-19 (104^2 .. 13^2, batch 16),
        // where they pick the fastest of the three on every layer or one within 1%; 128 x 128
        // needs at least 600 tiles and 128 x 64 one a compute unit (fewer hide too little latency)
        const auto cost = [](long long tiles, double tile_outputs, double rate) {
            const long long slots = (tiles + kComputeUnits - 1) / kComputeUnits * kComputeUnits;
            return ((double)tiles + 0.5 * (double)(slots - tiles)) * tile_outputs / rate;
        };
        const long long t128 = n_tiles(g, 128, 128), t12864 = n_tiles(g, 128, 64);
        const double c64 = cost(n_tiles(g, 64, 64), 64.0 * 64.0, 0.925);
        const double c12864 = t12864 >= kComputeUnits ? cost(t12864, 128.0 * 64.0, 0.972) : 1e300;
        const double c128 = t128 >= 600 ? cost(t128, 128.0 * 128.0, 1.0) : 1e300;
        if (c128 <= c12864 && c128 <= c64) return f(F32_128x128{});
        if (c12864 <= c64) return f(F32_128x64{});
        return f(F32_64x64{});
    }
    const bool dma = nhwc && g.C % 64 == 0 && dma_layer(g, 2);
    if (g.M <= 32) return f(BF16_M32{});
    if (dma && wide) return g.M <= 64 ? f(BF16W_64x128{}) : f(BF16W_128x128{});
    // at most two 64 x 64 tiles a compute unit: nothing larger would fill it
    if (dma && n_tiles(g, 64, 64) <= 2 * kComputeUnits) return f(BF16_DMA_64x64_3{});
    // M <= 64 with 64-channel multiples: direct-to-LDS 64 x 128 (against register-staged loads,
    // VGG-19 v2 384 -> 308 us and ResNet-18 l1 109 -> 90 us for the convolution alone, before the
    // tile went from 64 x 256 to 64 x 128)
    if (g.M <= 64) return dma ? f(BF16_DMA_64x128{}) : f(BF16_M64{});
    if (dma) {
        // 256 x 256 where M is large and there are enough such tiles
        if (g.M >= 256 && n_tiles(g, 256, 256) >= 192) return f(BF16_DMA_256x256{});
        if (n_tiles(g, 128, 128) < kComputeUnits) return f(BF16_DMA_128x128_3{});
        return f(BF16_DMA_128x128{});
    }
    if (g.M >= 256 && n_tiles(g, 256, 256) >= 192) return f(BF16_256x256{});
    return f(BF16_128x128_K64{});
}

}  // namespace

namespace {
// What a protected layer takes (us) on a route is a sum of these, with coefficients fitted to layers drawn over the
// workloads' ranges (840 fp32 ones of 32, 64, ... channels; 373 of other counts in each type; 200 bf16 ones of 32,
// 96, ...), batch 1 to 128: rms 8 to 14 % for the copies, 19 to 32 % for the gathers.
struct Work {
    double d, w, o, cd;  // MB of D, W and O as given, and of Cd1 and Cd2
    double mac;          // 10^9 multiply-adds of the padded tiles
    double fetch;        // 10^6 input values, once a filter tile
    double cols;         // 10^6 output pixels, once a filter tile
    double k;            // terms a tile walks
};
Work work_of(const Geom &g, bool nhwc, double k) {
    const double es = g.dtype == FTCNN_F32 ? 4e-6 : 2e-6;
    Work w{es * g.N * (double)g.CHW, es * g.M * (double)g.K, es * g.M * (double)g.P_total, 16e-6 * (double)g.CHW, 0, 0, 0, k};
    with_tile(g, nhwc, [&](auto t) {
        using Tl = decltype(t);
        const double tiles = (double)n_tiles(g, Tl::TM, Tl::TP);
        w.mac = 1e-9 * tiles * Tl::TM * Tl::TP * k;
        w.fetch = 1e-6 * tiles * Tl::TP * k;
        w.cols = 1e-6 * (double)g.P_total * ((g.M + Tl::TM - 1) / Tl::TM);
        return 0;
    });
    return w;
}
}  // namespace

bool split_pays(const Geom &g) {
    if (g.R > 32 || g.S > 32) return true;
    Geom sp = g, f32 = g;
    sp.split = 1;
    f32.split = 0;
    double conv = 0;
    with_tile(sp, true, [&](auto t) {
        using Tl = decltype(t);
        if constexpr (Tl::SK_FORM) conv = split_cost<Tl>(sp, false);
        return 0;
    });
    double k = 0;
    with_tile(f32, true, [&](auto t) {
        k = g.R * g.S * mean_channels(g, decltype(t)::TM);
        return 0;
    });
    const Work w = work_of(f32, true, k);
    // rounds of eight images past the last one read it again
    const double again = w.d * ((g.N + 7) / 8 * 8 - g.N) / g.N;
    const double split = 10.9 + 0.77 * w.d + 0.37 * again + 0.89 * w.w + 0.27 * w.o + 0.99 * conv;
    const double whole = 16.3 + 0.48 * w.d + 0.28 * again + 0.19 * w.o + std::max(20.0 * w.mac, 0.047 * w.k);
    return split < 1.1 * whole;   // (1.05 and 1.1: the least mean time over the drawn layers)
}

bool pack_pays(const Geom &g) {
    Geom as_given = g;
    as_given.pk = as_given.split = 0;
    // (bf16 layers of 32-channel blocks go back to channels-last copies instead of D and W as given)
    const bool nhwc = nhwc_layer(g), one = g.R * g.S == 1;
    const Work p = work_of(g, true, g.pkk), q = work_of(as_given, nhwc, g.K);
    const auto most = [](double matrix, double chain) { return std::max(matrix, chain); };   // throughput, or one tile's K
    if (g.dtype == FTCNN_F32) {
        const double copy = 6e-6 * g.N * (double)g.H * g.pw * g.pcs;
        const double packed = 15.1 + 0.13 * copy + 0.78 * p.d + 0.51 * p.cd + 119 * p.cols + most(13.0 * p.mac, 0.0198 * p.k);
        const double gather = 10.5 + 0.37 * q.d + 0.42 * q.o + 0.61 * q.cd + (one ? 0.16 : 0.97) * q.fetch +
                              most(15.4 * q.mac, 0.082 * q.k);
        // (small layers come out up to 8 us either side of the fit: of 158 drawn ones under 45 us, 0.85 leaves 6 more
        // than 3 % slower than on the gather and takes 0.86 of its time on average; 0.75: 4 and 0.90; 0.95: 8 and 0.84)
        return packed < (gather < 45.0 ? 0.85 : 0.95) * gather;
    }
    if (nhwc) {
        const double packed = 13.2 + 0.70 * p.d + 0.10 * p.o + 0.53 * p.cd + 38.3 * p.cols + most(3.67 * p.mac, 0.0085 * p.k);
        const double copies = 14.4 + 0.43 * q.d + 0.70 * q.o + 1.05 * q.cd + most(2.86 * q.mac, 0.0162 * q.k);
        return packed < 1.05 * copies;
    }
    const double packed = 15.1 + 0.72 * p.d + 0.19 * p.o + 0.51 * p.cd + 58 * p.cols + most(2.50 * p.mac, 0.0081 * p.k);
    const double gather = 14.6 + 0.22 * q.d + 0.63 * q.o + 0.63 * q.cd + (one ? 0.0 : 0.56) * q.fetch +
                          most(8.84 * q.mac, 0.0655 * q.k);
    return packed < 0.95 * gather;
}

void conv_tile_info(const Geom &g, bool nhwc, int out[6]) {
    with_tile(g, nhwc, [&](auto t) {
        using Tt = decltype(t);
        out[0] = Tt::TM;
        out[1] = Tt::TP;
        out[2] = Tt::TK;
        out[3] = Tt::WEAVE_KIND;
        out[4] = nhwc ? 1 : 0;
        out[5] = (nhwc && g.G > 1 && Tt::WEAVE_KIND != 2 && !packed_loop(Tt::WEAVE_KIND)) ? 1 : 0;
        return 0;
    });
}

int conv_tile_m(const Geom &g, bool nhwc) {
    return with_tile(g, nhwc, [](auto t) { return decltype(t)::TM; });
}

hipError_t launch_conv(const Plan &pl, const void *D, const void *W, void *O, hipStream_t st, const float *bias) {
    const Epi<0> ep{bias, {}};
    return with_tile(pl.g, false, [&](auto t) { return decltype(t)::run(pl.g, D, W, O, st, ep); });
}

void conv_sk_space(const Geom &g, bool nhwc, int *smax, size_t *part_bytes, long long *counters) {
    *smax = 0;
    *part_bytes = 0;
    *counters = 0;
    if (!nhwc || g.G > 1) return;
    with_tile(g, true, [&](auto t) {
        using Tt = decltype(t);
        if constexpr (Tt::SK_FORM) {
            // as many as the schedule would use on a whole device (none: no scratch)
            constexpr TileCost c = tile_cost<Tt>();
            const long long tiles = n_tiles(g, Tt::TM, Tt::TP);
            *smax = stream_k_workgroups(c, tiles, c.resident, g.R * g.S * (g.C / Tt::TK));
            *part_bytes = (size_t)*smax * 2 * Tt::TM * Tt::TP * sizeof(float);
            *counters = *smax > 0 ? tiles : 0;
        }
        return 0;
    });
}

int conv_stream_k(const Plan &pl) {
    if (!pl.nhwc || pl.sk_smax <= 0) return 0;
    return with_tile(pl.g, true, [&](auto t) { return decltype(t)::stream_k(pl.g, pl.sk_smax); });
}

void conv_tile_shape(const Geom &g, bool nhwc, int *threads, size_t *lds_bytes) {
    with_tile(g, nhwc, [&](auto t) {
        *threads = decltype(t)::NT;
        *lds_bytes = decltype(t)::LDS_BYTES;
        return 0;
    });
}

// The stream-K scratch of the plan (none when the plan has no room for it).
SkArgs sk_args(const Plan &pl, void *ws) {
    if (pl.sk_smax <= 0) return SkArgs{nullptr, nullptr, 0, 0, 0};
    char *w = static_cast<char *>(ws);
    return SkArgs{reinterpret_cast<float *>(w + pl.off_skpart), reinterpret_cast<int *>(w + pl.off_skcnt), pl.sk_smax, 0,
                  0};
}

hipError_t launch_conv_sums(const Plan &pl, const void *D, const void *W, void *O, const ftcnn_checksums *ck,
                            ftcnn_report *rep, int cap, const ftcnn_fault *faults, int nf, void *ws,
                            hipStream_t st, bool cd_given) {
    char *w = static_cast<char *>(ws);
    double *cd1 = ck ? ck->cd1 : nullptr, *cd2 = ck ? ck->cd2 : nullptr;
    const void *Dc = D, *Wc = W;
    const void *zp = pl.copies ? w + pl.off_zero : nullptr;   // zeroed by the copy
    int aux_kind = 0, aux_blocks = 0, co_slices = 0;
    if (pl.copies) {
        // the copy of D also encodes Cd1, Cd2 (if asked and not given)
        double *e1 = cd_given ? nullptr : cd1, *e2 = cd_given ? nullptr : cd2;
        const hipError_t e = pl.nhwc ? launch_prep(pl, D, W, e1, e2, ws, st) : launch_pack(pl, D, W, e1, e2, ws, st);
        if (e != hipSuccess) return e;
        Dc = w + pl.off_dt;
        Wc = w + pl.off_wt;
        if (cd1 && pl.co_in_conv && ck->cw1 && ck->cw2) {
            aux_kind = 2;
            aux_blocks = pl.co.tiles * pl.co.groups;
            co_slices = pl.co.groups;
        }
    } else if (cd1 && !cd_given) {
        aux_kind = 1;   // encode workgroups; their count follows the tile's threads
    }
    double *part = reinterpret_cast<double *>(w + pl.off_sums);
    double *copart = reinterpret_cast<double *>(w + pl.off_copart);
    const double *cw1 = ck ? ck->cw1 : nullptr, *cw2 = ck ? ck->cw2 : nullptr;
    const float *bias = ck ? ck->bias : nullptr;
    if (nf == 0) {
        Epi<1> ep{part, rep, cap, aux_kind, aux_blocks, 0, 0, cd1, cd2, 0, cw1, cw2, copart, pl.co, co_slices, {}, bias, {D, W}};
        return with_tile(pl.g, pl.copies,
                         [&](auto t) { return decltype(t)::run(pl.g, Dc, Wc, O, st, ep, pl.copies, zp, sk_args(pl, ws)); });
    }
    Epi<2> ep{part, rep, cap, aux_kind, aux_blocks, 0, 0, cd1, cd2, 0, cw1, cw2, copart, pl.co, co_slices, {}, bias, {D, W}};
    for (int i = 0; i < nf; ++i) ep.fl.f[i] = faults[i];
    ep.fl.n = nf;
    return with_tile(pl.g, pl.copies,
                     [&](auto t) { return decltype(t)::run(pl.g, Dc, Wc, O, st, ep, pl.copies, zp, sk_args(pl, ws)); });
}

hipError_t launch_conv_ws(const Plan &pl, const void *D, const void *W, void *O, void *ws, hipStream_t st,
                          const float *bias) {
    if (!pl.copies) return launch_conv(pl, D, W, O, st, bias);
    const hipError_t e = pl.nhwc ? launch_prep(pl, D, W, nullptr, nullptr, ws, st) : launch_pack(pl, D, W, nullptr, nullptr, ws, st);
    if (e != hipSuccess) return e;
    char *w = static_cast<char *>(ws);
    const Epi<0> ep{bias, {D, W}};
    return with_tile(pl.g, true, [&](auto t) {
        return decltype(t)::run(pl.g, w + pl.off_dt, w + pl.off_wt, O, st, ep, true, w + pl.off_zero, sk_args(pl, ws));
    });
}

}  // namespace ftcnn
