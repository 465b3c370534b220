// Launches of the convolution kernel's tiles, instantiated by the conv_*.hip files.
#pragma once

#include "conv_kernel.h"

namespace ftcnn {
namespace convk {

// Stream-K workgroups of a tile configuration on the current device: the workgroups that are
// resident at once (the least over the three epilogues, so that the protected kernel and its
// plain twin split K at the same places and store the same bits), at most smax, a multiple of 8.
template <typename Tr, int WM, int WP, int FM, int FP, int WEAVE, bool KVEC, bool NHWC>
int sk_workgroups(int smax) {
    using C = Cfg<Tr, WM, WP, FM, FP, KVEC, dma_stages(WEAVE)>;
    static const int per_cu = [] {
        int lo = 1 << 30;
        const void *k[3] = {
            reinterpret_cast<const void *>(conv_kernel<Tr, WM, WP, FM, FP, WEAVE, KVEC, 0, NHWC, false, true>),
            reinterpret_cast<const void *>(conv_kernel<Tr, WM, WP, FM, FP, WEAVE, KVEC, 1, NHWC, false, true>),
            reinterpret_cast<const void *>(conv_kernel<Tr, WM, WP, FM, FP, WEAVE, KVEC, 2, NHWC, false, true>)};
        const void *w[3] = {
            reinterpret_cast<const void *>(conv_kernel<Tr, WM, WP, FM, FP, WEAVE, KVEC, 0, NHWC>),
            reinterpret_cast<const void *>(conv_kernel<Tr, WM, WP, FM, FP, WEAVE, KVEC, 1, NHWC>),
            reinterpret_cast<const void *>(conv_kernel<Tr, WM, WP, FM, FP, WEAVE, KVEC, 2, NHWC>)};
        int whole = 1 << 30;
        size_t spill = 0, spill_whole = 0;
        for (int i = 0; i < 6; ++i) {
            const void *f = i < 3 ? k[i] : w[i - 3];
            if (C::LDS_BYTES > 65536 &&
                hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES) != hipSuccess)
                return 0;
            int nb = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, C::NT, C::LDS_BYTES) != hipSuccess) return 0;
            hipFuncAttributes fa;
            if (hipFuncGetAttributes(&fa, f) != hipSuccess) return 0;
            if (i < 3) {
                lo = nb < lo ? nb : lo;
                spill = fa.localSizeBytes > spill ? fa.localSizeBytes : spill;
            } else {
                whole = nb < whole ? nb : whole;
                spill_whole = fa.localSizeBytes > spill_whole ? fa.localSizeBytes : spill_whole;
            }
        }
        if (spill > spill_whole) return 0;   // registers spilled to scratch: slower than any balance
        // the stream-K kernels hold more registers; where that costs resident workgroups, the
        // balance they bring does not pay for it
        if (lo < whole) return 0;
        return lo;
    }();
    int dev = 0, cus = 0;
    if (per_cu <= 0 || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    long long S = (long long)per_cu * cus;
    S = S < smax ? S : smax;
    return (int)(S / 8 * 8);
}

// The stream-K workgroups of a layer's channels-last fp32 convolution on the current device, or 0
// for one workgroup per tile.  The bf16 loops run whole tiles: on VGG-19 bf16 the stream-K form of
// the direct-to-LDS 128 x 128 tile was 5-8 % slower where its balance should have helped, and the
// 256 x 256 tile (eight waves, at most 256 registers each) spills in that form.
template <typename Tr, int WM, int WP, int FM, int FP, int WEAVE, bool KVEC, bool NHWC>
int sk_decide(const Geom &g, int smax) {
    using C = Cfg<Tr, WM, WP, FM, FP, KVEC, dma_stages(WEAVE)>;
    if constexpr (!(NHWC && (WEAVE == 3 || WEAVE == 4) && sizeof(typename C::T) == 4)) {
        return 0;
    } else {
        if (smax <= 0 || g.G > 1) return 0;
        const int nch = g.R * g.S * (g.C / C::TK);
        const long long tiles = ((g.P_total + C::TP - 1) / C::TP) * (long long)((g.M + C::TM - 1) / C::TM);
        const int S = sk_workgroups<Tr, WM, WP, FM, FP, WEAVE, KVEC, NHWC>(smax);
        // the plan's own count, or what the schedule comes to on a device that holds fewer
        return S == smax || S <= 0 ? S
                                   : stream_k_workgroups(tile_cost<Tile<Tr, WM, WP, FM, FP, WEAVE>>(), tiles, S, nch);
    }
}

template <typename Tr, int WM, int WP, int FM, int FP, int WEAVE, bool KVEC, int EPI, bool NHWC, bool GRP = false>
hipError_t launch_one(const Geom &g, const void *D, const void *W, void *O, hipStream_t st, int m_major,
                      const void *zp, const Epi<EPI> &ep, const SkArgs &skin) {
    using C = Cfg<Tr, WM, WP, FM, FP, KVEC, dma_stages(WEAVE)>;
    using T = typename C::T;
    static_assert(EPI == 0 || (size_t)WM * 3 * C::TP * sizeof(double) <= C::LDS_BYTES, "epilogue fold fits LDS");
    const int tiles_m = (g.M + C::TM - 1) / C::TM;
    const long long tiles_p = (g.P_total + C::TP - 1) / C::TP;
    const long long total = tiles_p * tiles_m;
    Epi<EPI> e = ep;
    SkArgs sk{nullptr, nullptr, 0, 0, 0};
    constexpr bool SKF = NHWC && (WEAVE == 3 || WEAVE == 4) && sizeof(T) == 4;   // has a stream-K form
    if constexpr (SKF) {
        if (skin.S > 0 && skin.part && skin.cnt) {
            const int S = sk_decide<Tr, WM, WP, FM, FP, WEAVE, KVEC, NHWC>(g, skin.S);
            if (S > 0) {
                // whole-tile waves but for the last one to two, whose tiles are shared
                const long long waves = (total + S - 1) / S;
                sk = SkArgs{skin.part, skin.cnt, S, g.R * g.S * (g.C / C::TK), (int)(waves > 2 ? waves - 2 : 0)};
            }
        }
    }
    long long grid = sk.S > 0 ? sk.S : total;
    if constexpr (EPI != 0) {
        if (e.aux_kind == 1) {
            e.enc_vec = g.CHW % kEncVec == 0 && reinterpret_cast<uintptr_t>(D) % (kEncVec * sizeof(T)) == 0;
            const long long per = (long long)C::NT * (e.enc_vec ? kEncVec : 1);
            const long long eb = (g.CHW + per - 1) / per;
            if (eb > 0x7FFFFFFFLL) return hipErrorInvalidValue;
            e.aux_blocks = (int)eb;
        }
        if (e.aux_kind == 2 && e.co_slices > 0 && (size_t)e.co.cc * coc_channel_bytes(g, e.co.ty, e.co.tx) > C::LDS_BYTES)
            return hipErrorInvalidValue;   // the plan sized the CoC window for this tile's LDS
        if (e.aux_kind != 0 && e.aux_blocks > 0) {
            // the encode first (it reads D beside the first tiles); the Co5..Co7 work after the
            // tiles, in the slots their last round leaves (in front of them it held back the first
            // tiles: VGG-19 bf16 v6 197 -> 190 us, VGG-19 fp32 overhead 4.4 -> 3.2 %)
            e.aux_groups = (e.aux_blocks + 7) / 8;
            e.tile_groups = (int)((grid + 7) / 8);
            grid = 8 * (e.aux_groups + (grid + 7) / 8);
        } else {
            e.aux_groups = 0;
        }
    }
    if (grid > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    auto kern = conv_kernel<Tr, WM, WP, FM, FP, WEAVE, KVEC, EPI, NHWC, GRP>;
    if constexpr (C::LDS_BYTES > 65536) {
        static const hipError_t attr = hipFuncSetAttribute(
            reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES);
        if (attr != hipSuccess) return attr;
    }
    if constexpr (SKF) {
        if (sk.S > 0) {
            kern = conv_kernel<Tr, WM, WP, FM, FP, WEAVE, KVEC, EPI, NHWC, GRP, true>;
            if constexpr (C::LDS_BYTES > 65536) {
                static const hipError_t attr_sk = hipFuncSetAttribute(
                    reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                    (int)C::LDS_BYTES);
                if (attr_sk != hipSuccess) return attr_sk;
            }
        }
    }
    KernelEvents &ev = kernel_events();
    if (ev.before) {
        const hipError_t r = hipEventRecord(ev.before, st);
        if (r != hipSuccess) return r;
    }
    kern<<<(unsigned)grid, C::NT, C::LDS_BYTES, st>>>(static_cast<const T *>(D),
                                                               static_cast<const T *>(W), static_cast<T *>(O), g,
                                                               tiles_m, (int)total, m_major, zp, e, sk);
    const hipError_t r = hipGetLastError();
    if (r != hipSuccess) return r;
    if (ev.after) {
        const hipError_t r2 = hipEventRecord(ev.after, st);
        if (r2 != hipSuccess) return r2;
    }
    ev.before = ev.after = nullptr;
    return hipSuccess;
}

template <typename Tr, int WM, int WP, int FM, int FP, int WEAVE>
int Tile<Tr, WM, WP, FM, FP, WEAVE>::stream_k(const Geom &g, int smax) {
    if constexpr (!SK_FORM) return 0;
    else return sk_decide<Tr, WM, WP, FM, FP, WEAVE, true, true>(g, smax);
}

// Dispatched on the operands' layout, the weight alignment and the epilogue.
template <typename Tr, int WM, int WP, int FM, int FP, int WEAVE>
template <int EPI>
hipError_t Tile<Tr, WM, WP, FM, FP, WEAVE>::run(const Geom &g, const void *D, const void *W, void *O, hipStream_t st,
                                                const Epi<EPI> &ep, bool nhwc, const void *zp, const SkArgs &sk) {
    const SkArgs none{nullptr, nullptr, 0, 0};
    if constexpr (WEAVE >= 3) {
        // direct-to-LDS tiles exist for channels-last operands only, with the copy of D right
        // behind the zero page (one buffer descriptor reaches both)
        if (!nhwc || !zp || static_cast<const char *>(zp) + 256 != static_cast<const char *>(D))
            return hipErrorInvalidValue;
        // (the kernel's D is the input as given, for the encode workgroups)
        return launch_one<Tr, WM, WP, FM, FP, WEAVE, true, EPI, true>(g, ep.src_dw.d, W, O, st, 0, zp, ep, sk);
    } else {
        if constexpr (WEAVE != 2) {
            if (nhwc && g.G > 1)   // grouped: the loop that skips other groups' channels
                return launch_one<Tr, WM, WP, FM, FP, WEAVE, true, EPI, true, true>(g, D, W, O, st, 0, zp, ep,
                                                                                    none);
        }
        if (nhwc) return launch_one<Tr, WM, WP, FM, FP, WEAVE, true, EPI, true>(g, D, W, O, st, 0, zp, ep, sk);
        const bool kvec = g.K % Tr::VEC == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0;
        if (kvec) return launch_one<Tr, WM, WP, FM, FP, WEAVE, true, EPI, false>(g, D, W, O, st, 0, zp, ep, none);
        return launch_one<Tr, WM, WP, FM, FP, WEAVE, false, EPI, false>(g, D, W, O, st, 0, zp, ep, none);
    }
}

// Instantiates one tile's launches (one conv_*.hip file per family, compiled in parallel).
#define FTCNN_CONV_TILE(T)                                                                                           \
    template int T::stream_k(const Geom &, int);                                                                     \
    template hipError_t T::run<0>(const Geom &, const void *, const void *, void *, hipStream_t, const Epi<0> &,     \
                                  bool, const void *, const SkArgs &);                                               \
    template hipError_t T::run<1>(const Geom &, const void *, const void *, void *, hipStream_t, const Epi<1> &,     \
                                  bool, const void *, const SkArgs &);                                               \
    template hipError_t T::run<2>(const Geom &, const void *, const void *, void *, hipStream_t, const Epi<2> &,     \
                                  bool, const void *, const SkArgs &);

}  // namespace convk
}  // namespace ftcnn
