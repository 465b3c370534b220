// The layer's convolution, eq. (1), as an implicit GEMM on the CDNA4 matrix cores.
//
//   C[m][p] = sum_k A[m][k] * B[k][p]
//   A = W viewed as [M][K] (already row-major, K = C*R*S ordered (c, r, s)),
//   B = im2col(D): B[k][p] = D[n][c][U*x + r - P][U*y + s - P] (zero outside),
//   p = (n, x, y) runs over the N*E*F output pixels, and C[m][p] is O[n][m][x][y].
//
// A workgroup computes a TM x TP tile of C with WM x WP waves; every wave owns
// FM x FP blocks of 32x32 accumulators.  The K loop walks chunks of TK: the next
// chunk is fetched from global memory into registers (A with 16-byte loads, B as
// a per-pixel im2col gather whose addresses are coalesced along p) while the
// matrix cores work on the current chunk from LDS; LDS is double buffered, so one
// barrier per chunk suffices.  Lanes of a 32x32 MFMA own one output pixel each,
// so the epilogue writes whole 128-byte runs of O.  Workgroup ids are remapped so
// that the M tiles of one pixel tile land on the same XCD (its L2 then serves the
// repeated im2col reads of D).
#pragma once

#include <type_traits>

#include "conv_tiles.h"

namespace ftcnn {
namespace convk {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// A 16-byte unit, or zeros: the selects work on whole 32-bit words.
__device__ inline uint4 keep_or_zero(bool ok, uint4 v) {
    return make_uint4(ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u);
}

// Map the hardware workgroup id onto a logical tile so that each XCD (ids are
// dealt round-robin over 8 XCDs) receives a contiguous run of logical tiles.
__device__ inline int xcd_tile(int bid, int total) {
    const int q = total / 8, rem = total % 8, x = bid % 8;
    return x * q + (x < rem ? x : rem) + bid / 8;
}

// 16 bytes of elements, moved between global memory, registers and LDS as one unit.
template <typename T, int VEC> union Pack {
    uint4 q;
    T e[VEC];
};

// Per-lane constants of the A (weights) gather: which 16-byte slots of the
// TM x TK tile this lane moves, and where each slot's row starts in W.
template <typename C> struct ASlots {
    int base[C::A_PER];   // element offset of the slot's first k in W, -1 if the row is past M
    int kq[C::A_PER];     // k offset of the slot inside the chunk
};

template <typename C>
__device__ inline void a_slots(const Geom &g, int m0, int tid, ASlots<C> &as) {
#pragma unroll
    for (int i = 0; i < C::A_PER; ++i) {
        const int slot = tid + i * C::NT;
        const int row = slot / (C::TK / C::VEC);
        const int m = m0 + row;
        as.kq[i] = (slot % (C::TK / C::VEC)) * C::VEC;
        as.base[i] = (slot < C::A_SLOTS && m < g.M) ? m * g.K + as.kq[i] : -1;
    }
}

// Loads are unconditional (a masked lane reads element 0 and discards it), so
// the whole gather is straight-line code the scheduler can interleave with MFMAs.
// The masks are applied only when the registers go to LDS (after the MFMAs of
// the current chunk), so no wait for these loads sits in front of the MFMAs.
template <typename C>
__device__ inline typename C::Mask load_a(const typename C::T *__restrict__ Wt, const Geom &g, int kbase, bool,
                                          const ASlots<C> &as, Pack<typename C::T, C::VEC> (&ra)[C::A_PER]) {
    using M = typename C::Mask;
    M mask = 0;
#pragma unroll
    for (int i = 0; i < C::A_PER; ++i) {
        const int k = kbase + as.kq[i];
        if constexpr (C::KVEC) {
            // W rows start on 16-byte boundaries (K % VEC == 0, aligned base): index
            // through a uint4 pointer so the load is one global_load_dwordx4
            const bool ok = (as.base[i] >= 0) & (k < g.K);
            const uint4 *w4 = reinterpret_cast<const uint4 *>(Wt);
            // an invalid slot (k >= K or a row past M) reads element 0 and keeps zeros
            ra[i].q = keep_or_zero(ok, w4[ok ? (as.base[i] + kbase) / C::VEC : 0]);
            mask |= (ok ? ((M(1) << C::VEC) - M(1)) : M(0)) << (i * C::VEC);
        } else {
#pragma unroll
            for (int v = 0; v < C::VEC; ++v) {
                const bool ok = (as.base[i] >= 0) & (k + v < g.K);
                ra[i].e[v] = Wt[ok ? as.base[i] + kbase + v : 0];
                mask |= (ok ? M(1) : M(0)) << (i * C::VEC + v);
            }
        }
    }
    return mask;
}

// The im2col gather of B: this lane's pixel is fixed (lane_base = n*C*H*W +
// ih0*W + iw0); the run of KR consecutive k is the same for the whole wave, so
// (c, r, s) and the k part of the offset live in scalar registers.
template <typename C>
__device__ inline typename C::Mask load_b(const typename C::T *__restrict__ Dt, const Geom &g, int kstart_lane,
                                          bool pvalid, int lane_base, int ih0, int iw0,
                                          Pack<typename C::T, C::VEC> (&rb)[C::KR / C::VEC]) {
    using M = typename C::Mask;
    M mask = 0;
    using T = typename C::T;
    const int kstart = __builtin_amdgcn_readfirstlane(kstart_lane);
    const int RS = g.R * g.S;
    int c = kstart / RS;
    const int rem = kstart - c * RS;
    int r = rem / g.S;
    int s = rem - r * g.S;
    const int HW = g.H * g.W;
    int koff = c * HW + r * g.W + s;
    const int wrap_s = g.W - g.S, wrap_r = HW - g.R * g.W;
    // bf16: the loads go through a buffer descriptor of D, and an element outside the image, past K
    // or of a pixel past the end takes an offset past the buffer, whose load returns zero: no
    // validity bits and no 64-bit address per element (2 N C H W bytes < 2^32: make_plan keeps
    // N C H W below 2^31)
    [[maybe_unused]] __amdgpu_buffer_rsrc_t rd;
    if constexpr (sizeof(T) == 2)
        rd = __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(Dt), (short)0,
                                               (int)(unsigned)(2ull * (unsigned long long)g.N * (unsigned long long)g.CHW),
                                               0x00020000);
#pragma unroll
    for (int j = 0; j < C::KR; ++j) {
        const int ih = ih0 + r, iw = iw0 + s;
        // bitwise, not short-circuit: no branches in the gather
        const bool ok = pvalid & (kstart + j < g.K) & ((unsigned)ih < (unsigned)g.H) &
                        ((unsigned)iw < (unsigned)g.W);
        if constexpr (sizeof(T) == 2) {
            rb[j / C::VEC].e[j % C::VEC] =
                __builtin_amdgcn_raw_buffer_load_b16(rd, ok ? 2u * (unsigned)(lane_base + koff) : 0xFFFFFFFEu, 0, 0);
        } else {
            rb[j / C::VEC].e[j % C::VEC] = Dt[ok ? lane_base + koff : 0];
            mask |= (ok ? M(1) : M(0)) << j;
        }
        // advance (c, r, s) by one k with selects (scalar registers)
        ++s;
        ++koff;
        const bool ws = s == g.S;
        s = ws ? 0 : s;
        koff += ws ? wrap_s : 0;
        r += ws ? 1 : 0;
        const bool wr = r == g.R;
        r = wr ? 0 : r;
        koff += wr ? wrap_r : 0;
        c += wr ? 1 : 0;
    }
    if constexpr (sizeof(T) == 2) return ~M(0);   // every invalid element is a zero already
    return mask;
}

// NOMASK: the gathers zeroed every invalid element already (channels-last layers
// with 16-byte weight rows), so the registers go to LDS as they are.
template <typename C, bool NOMASK = false>
__device__ inline void store_lds(typename C::T *As, typename C::T *Bs, int tid,
                                 Pack<typename C::T, C::VEC> (&ra)[C::A_PER], typename C::Mask amask,
                                 Pack<typename C::T, C::VEC> (&rb)[C::KR / C::VEC], typename C::Mask bmask,
                                 int bp, int bkg) {
    using T = typename C::T;
#pragma unroll
    for (int i = 0; i < C::A_PER; ++i) {
        const int slot = tid + i * C::NT;
        if (C::A_SLOTS % C::NT == 0 || slot < C::A_SLOTS) {
            if constexpr (!NOMASK) {
#pragma unroll
                for (int v = 0; v < C::VEC; ++v)
                    ra[i].e[v] = ((amask >> (i * C::VEC + v)) & 1) ? ra[i].e[v] : T(0);
            }
            const int row = slot / (C::TK / C::VEC);
            const int kq = slot % (C::TK / C::VEC);
            *reinterpret_cast<uint4 *>(&As[row * C::LDK + kq * C::VEC]) = ra[i].q;
        }
    }
    if constexpr (!NOMASK) {
#pragma unroll
        for (int j = 0; j < C::KR; ++j)
            rb[j / C::VEC].e[j % C::VEC] = ((bmask >> j) & 1) ? rb[j / C::VEC].e[j % C::VEC] : T(0);
    }
#pragma unroll
    for (int j = 0; j < C::KR; j += C::VEC)
        *reinterpret_cast<uint4 *>(&Bs[bp * C::LDK + bkg * C::KR + j]) = rb[j / C::VEC].q;
}

// One chunk of MFMAs from LDS.  Within a chunk, lanes 0-31 take the first half
// of the k range and lanes 32-63 the second half; A and B use the same
// assignment, so every k of the chunk is summed exactly once.
template <int TK, int FM, int FP>
__device__ inline void mma_f32(const float *As, const float *Bs, int lane, int arow0, int brow0,
                               floatx16 (&acc)[FM][FP]) {
    constexpr int LDK = F32T<TK>::LDK;
    const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
    for (int q = 0; q < TK / 8; ++q) {
        floatx4 a[FM], b[FP];
#pragma unroll
        for (int i = 0; i < FM; ++i)
            a[i] = *reinterpret_cast<const floatx4 *>(&As[(arow0 + i * 32 + l32) * LDK + h * (TK / 2) + q * 4]);
#pragma unroll
        for (int j = 0; j < FP; ++j)
            b[j] = *reinterpret_cast<const floatx4 *>(&Bs[(brow0 + j * 32 + l32) * LDK + h * (TK / 2) + q * 4]);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FP; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][t], b[j][t], acc[i][j], 0, 0, 0);
    }
}

template <int TK, int FM, int FP>
__device__ inline void mma_bf16(const uint16_t *As, const uint16_t *Bs, int lane, int arow0, int brow0,
                                floatx16 (&acc)[FM][FP]) {
    constexpr int LDK = BF16T<TK>::LDK;
    const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
    for (int q = 0; q < TK / 16; ++q) {
        bf16x8 a[FM], b[FP];
#pragma unroll
        for (int i = 0; i < FM; ++i)
            a[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(
                                                  &As[(arow0 + i * 32 + l32) * LDK + h * (TK / 2) + q * 8]));
#pragma unroll
        for (int j = 0; j < FP; ++j)
            b[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(
                                                  &Bs[(brow0 + j * 32 + l32) * LDK + h * (TK / 2) + q * 8]));
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FP; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
}

// One chunk of MFMAs from LDS for either element type.
template <typename C, int FM, int FP>
__device__ inline void mma_chunk(const typename C::T *As, const typename C::T *Bs, int lane, int arow0, int brow0,
                                 floatx16 (&acc)[FM][FP]) {
    if constexpr (sizeof(typename C::T) == 4)
        mma_f32<C::TK, FM, FP>(reinterpret_cast<const float *>(As), reinterpret_cast<const float *>(Bs), lane, arow0,
                               brow0, acc);
    else
        mma_bf16<C::TK, FM, FP>(reinterpret_cast<const uint16_t *>(As), reinterpret_cast<const uint16_t *>(Bs), lane,
                                arow0, brow0, acc);
}

// The B gather from channels-last Dt[n][h][w][c] with K in (r, s, c) order: a
// thread's run of KR consecutive k lies inside one (r, s) (Ch is a multiple of
// the chunk), so it is KR contiguous elements of one input pixel, loaded as
// 16-byte units; the padding test is one test for the whole run.
template <typename C>
__device__ inline typename C::Mask load_b_nhwc(const typename C::T *__restrict__ Dt, const Geom &g, int kstart_lane,
                                       bool pvalid, int img_base, int ih0, int iw0,
                                       Pack<typename C::T, C::VEC> (&rb)[C::KR / C::VEC]) {
    const int kstart = __builtin_amdgcn_readfirstlane(kstart_lane);
    const int rs = kstart / g.C, c0 = kstart - rs * g.C;
    const int r = rs / g.S, s = rs - r * g.S;
    const int ih = ih0 + r, iw = iw0 + s;
    const bool ok = pvalid & (kstart < g.K) & ((unsigned)ih < (unsigned)g.H) & ((unsigned)iw < (unsigned)g.W);
    // a multiple of KR: 16-byte aligned; a run outside the image reads element 0 and keeps zeros
    const uint4 *src = reinterpret_cast<const uint4 *>(Dt + (ok ? img_base + (ih * g.W + iw) * g.C + c0 : 0));
#pragma unroll
    for (int i = 0; i < C::KR / C::VEC; ++i) rb[i].q = keep_or_zero(ok, src[i]);
    using M = typename C::Mask;
    constexpr M all = C::KR == 8 * (int)sizeof(M) ? ~M(0) : ((M(1) << C::KR) - M(1));
    return ok ? all : 0u;
}

// Chunks of K on channels-last operands, each TK consecutive channels of one tap (r, s), walked
// with the channel blocks outer and the taps inner: the input window of one block of channels is
// read for all R*S taps of a tile while it is still in the L2 of the tile's XCD (with the taps
// outer, a tile's window over all channels was evicted before the next tap came back to it).
// The state is wave-uniform and advances by additions only (scalar registers, no divisions).
struct TapWalk {
    int r, s, c0;        // the chunk: tap (r, s), channels [c0, c0 + TK)
    __device__ inline void next(const Geom &g, int tk) {
        ++s;
        if (s == g.S) {
            s = 0;
            ++r;
            if (r == g.R) {
                r = 0;
                c0 += tk;
            }
        }
    }
    __device__ inline int kb(const Geom &g) const { return (r * g.S + s) * g.C + c0; }
};
// The TapWalk state of chunk j (chunks of tk channels, channel blocks outer, taps inner).
__device__ inline TapWalk tap_at(const Geom &g, int j, int tk) {
    const int rs_n = g.R * g.S, blk = j / rs_n, rs = j - blk * rs_n, r = rs / g.S;
    return TapWalk{r, rs - r * g.S, blk * tk};
}

// A 16-byte unit in global memory (address space 1): loads through it are global loads that the
// compiler knows cannot alias the thread's private arrays, which then stay in registers.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 glb_u32x4;
__device__ inline uint4 load16(uintptr_t a) {
    return __builtin_bit_cast(uint4, *reinterpret_cast<const glb_u32x4 *>(a));
}

// The gathers of one chunk for the TapWalk loops, as raw 16-byte loads: a slot outside the
// operands (a weight row past M, a tap in the zero padding) loads from the 256-byte zero page
// instead, so no select waits on the loaded data and the loads stay in flight across the MFMAs
// of the current chunk.  Addresses are selected as integers (a pointer select becomes a branch).
template <typename C>
__device__ inline void load_a_tap(const typename C::T *__restrict__ Wt, int kb, const ASlots<C> &as, uintptr_t zpa,
                                  Pack<typename C::T, C::VEC> (&ra)[C::A_PER]) {
#pragma unroll
    for (int i = 0; i < C::A_PER; ++i) {
        const uintptr_t src = as.base[i] >= 0 ? reinterpret_cast<uintptr_t>(Wt + as.base[i] + kb) : zpa;
        ra[i].q = load16(src);
    }
}

// The B gather: the thread's KR channels of its pixel's input at tap (r, s).  pix_off = image
// base + (ih0 W + iw0) C + the thread's channel offset in the chunk.
template <typename C>
__device__ inline void load_b_tap(const typename C::T *__restrict__ Dt, const Geom &g, const TapWalk &t, bool pvalid,
                                  int pix_off, int ih0, int iw0, uintptr_t zpa,
                                  Pack<typename C::T, C::VEC> (&rb)[C::KR / C::VEC]) {
    const bool ok = pvalid & ((unsigned)(ih0 + t.r) < (unsigned)g.H) & ((unsigned)(iw0 + t.s) < (unsigned)g.W);
    const int off = pix_off + (t.r * g.W + t.s) * g.C + t.c0;
    const uintptr_t src = ok ? reinterpret_cast<uintptr_t>(Dt + off) : zpa;
#pragma unroll
    for (int i = 0; i < C::KR / C::VEC; ++i) rb[i].q = load16(src + 16 * i);
}

// Stateful form of the B gather, so that its elements can be issued one at a
// time between MFMAs: (c, r, s) and the k offset advance in scalar registers.
template <typename C> struct BGather {
    int kstart, c, r, s, koff;
    typename C::Mask mask;
    __device__ inline void begin(const Geom &g, int kstart_lane) {
        kstart = __builtin_amdgcn_readfirstlane(kstart_lane);
        const int RS = g.R * g.S;
        c = kstart / RS;
        const int rem = kstart - c * RS;
        r = rem / g.S;
        s = rem - r * g.S;
        koff = c * g.H * g.W + r * g.W + s;
        mask = 0;
    }
    __device__ inline void element(const typename C::T *__restrict__ Dt, const Geom &g, int j, bool pvalid,
                                   int lane_base, int ih0, int iw0, Pack<typename C::T, C::VEC> (&rb)[C::KR / C::VEC]) {
        const int ih = ih0 + r, iw = iw0 + s;
        const bool ok = pvalid & (kstart + j < g.K) & ((unsigned)ih < (unsigned)g.H) &
                        ((unsigned)iw < (unsigned)g.W);
        rb[j / C::VEC].e[j % C::VEC] = Dt[ok ? lane_base + koff : 0];
        mask |= (ok ? typename C::Mask(1) : typename C::Mask(0)) << j;
        ++s;
        ++koff;
        const bool ws = s == g.S;
        s = ws ? 0 : s;
        koff += ws ? g.W - g.S : 0;
        r += ws ? 1 : 0;
        const bool wr = r == g.R;
        r = wr ? 0 : r;
        koff += wr ? g.H * g.W - g.R * g.W : 0;
        c += wr ? 1 : 0;
    }
};

// One fp32 chunk with the next chunk's gather woven in: after every k-step
// (FM x FP MFMAs) the wave issues its share of the gather, so the vector ALU
// and the load pipeline run while the matrix core works.  sched_barrier(0)
// keeps the compiler from regrouping the two streams.
template <typename C, int FM, int FP, bool NEXT>
__device__ inline void chunk_f32(const float *As, const float *Bs, int lane, int arow0, int brow0,
                                 floatx16 (&acc)[FM][FP], const typename C::T *__restrict__ Dt,
                                 const typename C::T *__restrict__ Wt, const Geom &g, int kb_next, bool kvec,
                                 const ASlots<C> &as, Pack<typename C::T, C::VEC> (&ra)[C::A_PER], typename C::Mask &amask,
                                 BGather<C> &bg, int bkg, bool pvalid, int lane_base, int ih0, int iw0,
                                 Pack<typename C::T, C::VEC> (&rb)[C::KR / C::VEC]) {
    constexpr int TK = C::TK, LDK = C::LDK, STEPS = TK / 2;
    const int l32 = lane & 31, h = lane >> 5;
    floatx4 a[TK / 8][FM], b[TK / 8][FP];
#pragma unroll
    for (int q = 0; q < TK / 8; ++q) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
            a[q][i] = *reinterpret_cast<const floatx4 *>(&As[(arow0 + i * 32 + l32) * LDK + h * (TK / 2) + q * 4]);
#pragma unroll
        for (int j = 0; j < FP; ++j)
            b[q][j] = *reinterpret_cast<const floatx4 *>(&Bs[(brow0 + j * 32 + l32) * LDK + h * (TK / 2) + q * 4]);
    }
    if constexpr (NEXT) {
        amask = load_a<C>(Wt, g, kb_next, kvec, as, ra);
        bg.begin(g, kb_next + bkg * C::KR);
    }
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
        const int q = t / 4, tt = t % 4;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FP; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][i][tt], b[q][j][tt], acc[i][j], 0, 0, 0);
        if constexpr (NEXT) {
            __builtin_amdgcn_sched_barrier(0);
            const int E0 = t * C::KR / STEPS, E1 = (t + 1) * C::KR / STEPS;  // folded by unrolling
#pragma unroll
            for (int e = E0; e < E1; ++e) bg.element(Dt, g, e, pvalid, lane_base, ih0, iw0, rb);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// ---- direct-to-LDS main loop (channels-last) --------------------------------
//
// Operands in memory are rows of CH channels of one tap, ROWB bytes each: 64 bf16 (128 bytes), or
// for a split fp32 layer 32 channels as three bf16 planes (high, middle, low: 192 bytes).  buffer_load_dwordx4
// ... lds moves 16 bytes per lane straight into LDS: lane L of a wave lands at the instruction's LDS
// base + 16*L (the base is wave-uniform), while every lane picks its own global address, so an
// instruction fills 64 consecutive 16-byte units of the tile's rows.
//
// Bank conflicts: a 16-byte fragment read of 16 consecutive rows is what the LDS serves in one
// cycle (256 bytes over 64 banks).  128-byte rows: unit c of row r lies at c ^ ((r >> 1) & 7), so
// rows 2i and 2i + 1 share a position but lie in different halves of a 256-byte line.  192-byte
// rows start 12 units apart, four distinct positions modulo 16; unit c of row r lies at
// c ^ ((r >> 2) & 3), which spreads each of the four over its own four positions.

typedef __attribute__((address_space(3))) void lds_void_t;

// Cache policy of buffer loads and stores that other XCDs' workgroups must see (the sc1 bit: device
// scope, past this XCD's L2).
constexpr int kDeviceCoherent = 16;

// s_waitcnt: at most V vector-memory operations of this wave outstanding.
template <int V> __device__ inline void wait_vmcnt() {
    static_assert(V >= 0 && V < 64, "vmcnt is six bits");
    __builtin_amdgcn_s_waitcnt((V & 15) | (0x7 << 4) | (0xF << 8) | ((V >> 4) << 14));
}
// s_waitcnt: no LDS operation of this wave outstanding.
__device__ inline void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }
// Workgroup barrier that orders LDS accesses around it in the compiler only.
__device__ inline void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A raw buffer descriptor over [base, base + bytes) (stride 0, the data-format word of gfx9
// buffer resources), and a 16-byte load through it straight into LDS: lane L writes lds + 16 L.
__device__ inline __amdgpu_buffer_rsrc_t buffer_rsrc(const void *base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}
__device__ inline void buffer_load_lds16(__amdgpu_buffer_rsrc_t r, unsigned char *lds, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t *)lds, 16, voff, soff, 0, 0);
}

// The taps (at most 32) of one output pixel along one side of the map that fall inside it: bit t for the tap at
// row or column first + t.
__device__ inline unsigned tap_mask(int first, int extent, int taps) {
    const int lo = first < 0 ? -first : 0;
    const int hi = extent - first < taps ? extent - first : taps;
    return lo < hi ? (~0u >> (32 - hi)) & ~((1u << lo) - 1u) : 0u;
}

// The same for any kernel the copies take (at most 4096 taps): the run's first tap and its last one's distance
// from it, or a first one past them all.
__device__ inline uint2 tap_run(int first, int extent, int taps) {
    const int lo = first < 0 ? -first : 0;
    const int hi = extent - first < taps ? extent - first : taps;
    return lo < hi ? make_uint2(lo, hi - 1 - lo) : make_uint2(taps, 0);
}

// The K loop of one tile (or of chunks [k0, k0 + kn) of it; kn < 0: all), through a ring of STAGES LDS
// stages.  Chunks follow TapWalk over the channel blocks [c_lo, c_hi) (outer) and the taps (inner).
//
// What bounds it: the matrix cores, as long as nothing sits between their instructions.  So
//  - the fragments of step q + 1 are read from LDS between the MFMAs of step q, across the chunk
//    boundary too: the barrier of a chunk sits before its last step's MFMAs, which then cover the
//    latency of the next chunk's first reads;
//  - the loads of the chunk after next are issued between the MFMAs of that last step, into the
//    stage whose last fragments every wave has just read, and have a whole chunk to land;
//  - a load costs five vector instructions (an input slot) or none (a weight slot): each slot keeps
//    one byte offset and the masks of its pixel's taps inside the map, the tap's own offset is scalar,
//    and a tap in the padding reads offset 0, the 256-byte zero page in front of the input (no branch,
//    no select).  Masks hold 32 rows and columns; kernels past that test runs of taps by saturating 16-bit
//    differences (WIDE), one instruction more: on all layers VGG-19 bf16 v10 128.3 -> 130.2 us, ResNet-18
//    l3 56.0 -> 57.2.
// With bounds tests (branches) at every load, all of them before a chunk's first read and the reads
// after the barrier, the convolution kernel of VGG-19 bf16 v10 (256 x 256 tiles, 196 of them) took
// 125 us; so it takes 110 us, 1075 TFLOP/s on 77 % of the compute units (torch.mm on 8192^3 random
// bf16 operands: 1205 TFLOP/s).  Spreading a chunk's loads over two or three steps: 107-111 us there,
// 1-5 % slower on the 128 x 128 and smaller tiles.
template <typename C, int NP, int STAGES, bool PACK, bool WIDE, int FM, int FP>
__device__ inline void dma_mainloop(const void *__restrict__ Wt, const Geom &g, int m0, long long p0,
                                    const unsigned char *zp_dt, unsigned char *smem, floatx16 (&acc)[FM][FP],
                                    int tid, int arow0, int brow0, int k0, int kn, int c_lo, int c_hi) {
    constexpr int NW = C::NT / 64;
    constexpr int ROWL = C::ROWB / 16;               // 16-byte units per row
    constexpr int CH = C::TK, Q = CH / 16;           // channels per chunk, MFMA steps per chunk
    constexpr unsigned EB = 2 * NP;                  // bytes per channel of an operand
    // wave loads (64 units) of a chunk's weight and input rows, and the most of them one wave issues
    constexpr int NLA = C::TM * ROWL / 64, NLB = C::TP * ROWL / 64;
    constexpr int NIA = (NLA + NW - 1) / NW, NIB = NLB / NW, NI = NIA + NIB;
    static_assert(C::TM * ROWL % 64 == 0 && NLB % NW == 0 && STAGES * NI < 64, "DMA tile shape");
    static_assert(STAGES == 2 || NLA % NW == 0, "every wave counts the same loads");
    static_assert(Q % 2 == 0 && (NP == 1 || Q == 2), "fragment sets alternate");
    constexpr int STAGE_A = C::TM * C::ROWB, STAGE = (C::TM + C::TP) * C::ROWB;
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the unit of row r that LDS position c holds (the map is its own inverse)
    auto unit = [](int r, int c) { return NP == 1 ? c ^ ((r >> 1) & 7) : c ^ ((r >> 2) & 3); };
    const unsigned kk = PACK ? (unsigned)g.pkk : (unsigned)g.K;   // values of a filter's row
    const unsigned px_v = PACK ? (unsigned)g.pcs : (unsigned)g.C;  // values of a pixel, a row, an image
    const unsigned row_v = (PACK ? (unsigned)g.pw : (unsigned)g.W) * px_v;
    const unsigned img_v = PACK ? (unsigned)g.H * row_v : (unsigned)g.CHW;
    const __amdgpu_buffer_rsrc_t rw = buffer_rsrc(Wt, (unsigned)g.M * kk * EB);
    const __amdgpu_buffer_rsrc_t rd = buffer_rsrc(zp_dt, 256u + (unsigned)g.N * img_v * EB);
    unsigned a_off[NIA];
#pragma unroll
    for (int j = 0; j < NIA; ++j) {
        const int s = (j * NW + w) * 64 + lane, row = s / ROWL;
        const int m = m0 + row < g.M ? m0 + row : g.M - 1;   // rows past M are never stored
        a_off[j] = (unsigned)m * kk * EB + 16u * (unsigned)unit(row, s % ROWL);
    }
    // packed copies: a slot's unit of eight channels of a chunk belongs to a tap of its own.  The walk holds
    // the chunk's first unit (unit o of tap (r, s)), and a slot counts on from it by its own unit of the
    // chunk (unit0, four bits a slot), with carries by multiplication (exact: pack_geom)
    constexpr int UPC = CH / 8;
    const int p_s = PACK ? (g.prun ? 1 : g.S) : 1;
    const int d_t = PACK ? UPC / g.pupt : 0, d_o = PACK ? UPC - d_t * g.pupt : 0, d_r = PACK ? d_t / p_s : 0,
              d_s = PACK ? d_t - d_r * p_s : 0;
    const unsigned inv_o = PACK ? ((1u << kUnitShift) + g.pupt - 1) / g.pupt : 0u,
                   inv_s = PACK ? ((1u << kUnitShift) + p_s - 1) / p_s : 0u;
    unsigned unit0 = 0;
    static_assert(!PACK || (NIB <= 8 && UPC <= 8), "four bits a slot");
    // load j of a chunk: the weight slots, then the input slots.  b_row, b_col: the masks of a pixel's rows
    // and columns of taps inside the map (packed copies: both in b_row, 16 bits each; WIDE: the runs' first
    // row and column, 16 bits each, and their lengths less one)
    unsigned b_off[NIB], b_row[NIB], b_col[PACK ? 1 : NIB];
    struct Walk {
        TapWalk t;    // packed: c0 is the unit o
        unsigned k;   // packed: the chunk's first byte in a filter's row
    };
    auto issue = [&](const Walk &wk, unsigned char *base, int j) {
        const TapWalk &t = wk.t;
        if (j < NIA) {
            if (NLA % NW != 0 && j * NW + w >= NLA) return;
            buffer_load_lds16(rw, base + (j * NW + w) * 1024, a_off[j], PACK ? wk.k : EB * (unsigned)t.kb(g));
        } else if constexpr (PACK) {
            const int i = j - NIA;
            const unsigned x = (unsigned)t.c0 + __builtin_amdgcn_ubfe(unit0, 4 * i, 3);
            const unsigned co = __umul24(x, inv_o) >> kUnitShift, o = x - __umul24(co, (unsigned)g.pupt);
            const unsigned xs = (unsigned)t.s + co;
            const unsigned cs = __umul24(xs, inv_s) >> kUnitShift, ts = xs - __umul24(cs, (unsigned)p_s);
            const unsigned tr = min((unsigned)t.r + cs, 15u);   // taps past the last: bit 15 is never set, R <= 15
            const int in = __builtin_amdgcn_sbfe((int)b_row[i], tr, 1) & __builtin_amdgcn_sbfe((int)b_row[i], ts + 16, 1);
            const unsigned tap = EB * (tr * row_v + ts * px_v + 8u * o);
            buffer_load_lds16(rd, base + STAGE_A + (i * NW + w) * 1024, (b_off[i] + tap) & (unsigned)in, 0u);
        } else {
            const int i = j - NIA;
            const unsigned tap = EB * (unsigned)((t.r * g.W + t.s) * g.C + t.c0);
            unsigned in;
            if constexpr (WIDE) {
                // a tap outside its runs leaves something of a saturating difference
                const u16x2 at = __builtin_bit_cast(u16x2, (unsigned)t.r | (unsigned)t.s << 16) - __builtin_bit_cast(u16x2, b_row[i]);
                in = min(__builtin_bit_cast(unsigned, __builtin_elementwise_sub_sat(at, __builtin_bit_cast(u16x2, b_col[i]))), 1u) - 1u;
            } else {
                in = (unsigned)(__builtin_amdgcn_sbfe((int)b_row[i], t.r, 1) & __builtin_amdgcn_sbfe((int)b_col[i], t.s, 1));
            }
            buffer_load_lds16(rd, base + STAGE_A + (i * NW + w) * 1024, (b_off[i] + tap) & in, 0u);
        }
    };
    auto advance = [&](Walk &wk) {
        if constexpr (PACK) {
            TapWalk &t = wk.t;
            wk.k += CH * EB;
            t.c0 += d_o;
            const int co = t.c0 >= g.pupt;
            t.c0 -= co ? g.pupt : 0;
            t.s += d_s + co;
            const int cs = t.s >= p_s;
            t.s -= cs ? p_s : 0;
            t.r += d_r + cs;
        } else {
            wk.t.next(g, CH);
        }
    };
    const int nch = kn >= 0 ? kn : (PACK ? g.pkk / CH : g.R * g.S * ((c_hi - c_lo) / CH));
    Walk ti{PACK ? TapWalk{0, 0, 0} : tap_at(g, k0, CH), 0u};   // the chunk whose loads are issued next
    if constexpr (!PACK) ti.t.c0 += c_lo;
    // the first chunk's weights are on their way while the pixels are worked out
#pragma unroll
    for (int j = 0; j < NIA; ++j) issue(ti, smem, j);
#pragma unroll
    for (int j = 0; j < NIB; ++j) {
        const int s = (j * NW + w) * 64 + lane, row = s / ROWL, u = unit(row, s % ROWL);
        // columns past the end are never stored; P_total < 2^31 on these layers
        const unsigned pg = (unsigned)p0 + row < (unsigned)g.P_total ? (unsigned)p0 + row : (unsigned)g.P_total - 1;
        const unsigned n = pg / (unsigned)g.EF, pix = pg - n * (unsigned)g.EF;
        const unsigned x = pix / (unsigned)g.F, y = pix - x * (unsigned)g.F;
        const int ih0 = g.U * (int)x - g.P;
        int iw0 = g.U * (int)y - g.P;
        if constexpr (WIDE) {
            const uint2 rows = tap_run(ih0, g.H, g.R), cols = tap_run(iw0, g.W, g.S);
            b_row[j] = rows.x | cols.x << 16;
            b_col[j] = rows.y | cols.y << 16;
        } else if constexpr (PACK) {
            b_row[j] = tap_mask(ih0, g.H, g.R) | (g.prun ? 1u : tap_mask(iw0, g.W, g.S)) << 16;
            if (g.prun) iw0 += g.P;   // the copy has the padding's columns
            unit0 |= (unsigned)(u / NP) << (4 * j);
        } else {
            b_row[j] = tap_mask(ih0, g.H, g.R);
            b_col[j] = tap_mask(iw0, g.W, g.S);
        }
        // 32-bit wrap-around arithmetic: the sum with a valid tap's offset is the element's offset
        b_off[j] = 256u + EB * (n * img_v + (unsigned)ih0 * row_v + (unsigned)iw0 * px_v) +
                   16u * (unsigned)(PACK ? u % NP : u);
    }
#pragma unroll
    for (int st = 0; st < STAGES; ++st)
        if (st < nch) {
#pragma unroll
            for (int j = st == 0 ? NIA : 0; j < NI; ++j) issue(ti, smem + st * STAGE, j);
            advance(ti);
        }
    // (a wave with fewer weight loads than NIA must not leave one of its first chunk's behind)
    if (nch >= STAGES) wait_vmcnt<(STAGES - 1) * (NLA % NW ? NI - 1 : NI)>();
    else wait_vmcnt<0>();
    lds_barrier();
    // fragment reads: lanes 0-31 take the first half of the chunk's units of a plane, lanes 32-63 the second
    const int l32 = lane & 31, h = lane >> 5;
    constexpr int PU = ROWL / NP;                     // groups of eight channels, NP units (planes) each
    const int sw = NP == 1 ? (l32 >> 1) & 7 : (l32 >> 2) & 3;
    int fpos[Q][NP];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) {
            // split blocks hold plane after plane, packed ones group after group
            const int grp = (PU / 2) * h + q;
            fpos[q][pl] = ((PACK ? grp * NP + pl : pl * PU + grp) ^ sw) * 16;
        }
    const int arow = (arow0 + l32) * C::ROWB, brow = STAGE_A + (brow0 + l32) * C::ROWB;
    bf16x8 fa[2][NP][FM], fb[2][NP][FP];
    // reads per step: bf16 the input fragments, then the weights'; split a fragment's planes one after the
    // other, input and weight fragments in turn, so that the first block's come first
    constexpr int NR = NP * (FM + FP), NPAIR = NP == 1 ? 0 : (FM < FP ? FM : FP);
    auto read = [&](const unsigned char *stage, int q, int set, int i) {
        const int pl = i % NP, f = i / NP;
        const bool input = f < 2 * NPAIR ? f % 2 == 0 : (NP == 1 ? f < FP : FP > FM);
        const int k = f < 2 * NPAIR ? f / 2 : (NP == 1 ? (input ? f : f - FP) : f - NPAIR);
        if (input)
            fb[set][pl][k] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u16x8 *>(stage + brow + fpos[q][pl] + k * 32 * C::ROWB));
        else
            fa[set][pl][k] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u16x8 *>(stage + arow + fpos[q][pl] + k * 32 * C::ROWB));
    };
    // the products of one step: all of bf16; of a split layer the six whose planes' orders sum to at
    // most two (the other three are below 2^-24 of the product)
    constexpr int NPROD = NP == 1 ? 1 : 6, NB = FM * FP, NM = NPROD * NB;
    // A split layer's step starts every block's six products from zero, the smallest first, and adds their
    // sum to the accumulator with ordinary (nearest) additions.  The matrix instruction drops its addends'
    // bits far below the largest one's, towards one side: adding the products to the accumulators
    // themselves left errors of up to 9.8e-7 of the norm (K = 4608, one filter; fp32 instructions 8.7e-7), all
    // leaning to one side.  So: 3.0e-7 there, VGG-19 v6 at batch 32 2.1e-7 (before 7.1e-7, fp32 instructions
    // 7.9e-7), means within 2e-9 (the weights' signs, split_weight_scale).  It costs 3 to 7 % of a split
    // layer's time (protected: v6 617 -> 630 us, v2 969 -> 1003, v4 693 -> 732, AlexNet conv4 159 -> 167,
    // conv1 158 -> 165, Darknet-19 1x1 42.8 -> 44.1), of layers of a few 64 x 64 tiles, whose waves run alone, up
    // to 16 % (packed 30 %).
    // part holds NBUF blocks' sums in turn; with two, a block's additions go between the next one's products
    // (one: 2 % slower; three filter blocks a wave leave no registers for two).
    constexpr int NBUF = NP == 1 ? 1 : (FM > 2 ? 1 : 2);
    floatx16 part[NBUF];
    if constexpr (NBUF > 1)
        for (int e = 0; e < 16; ++e) part[1][e] = 0.0f;   // nothing before the first block
    // step q's part of block b; its sign follows the weights' (split_weight_scale)
    auto add = [&](int q, int b, int from, int to) {
#pragma unroll
        for (int e = from; e < to; ++e) {
            const float v = part[(q * NB + b) % NBUF][e];
            if ((q + e) & 1) acc[b / FP][b % FP][e] -= v;
            else acc[b / FP][b % FP][e] += v;
        }
    };
    auto mfma = [&](int q, int k) {
        const int set = q & 1;
        if constexpr (NP == 1) {
            const int i = k / FP, j = k % FP;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][0][i], fb[set][0][j], acc[i][j], 0, 0, 0);
        } else {
            constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
            const floatx16 zero = {};
            const int b = k / 6, pr = k % 6, i = b / FP, j = b % FP, buf = (q * NB + b) % NBUF;
            part[buf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][PA[pr]][i], fb[set][PB[pr]][j],
                                                                pr ? part[buf] : zero, 0, 0, 0);
            if (NBUF == 1 && pr == 5) add(q, b, 0, 16);
            if (NBUF == 2 && pr) add(b ? q : (q + 1) % 2, b ? b - 1 : NB - 1, (pr - 1) * 16 / 5, pr * 16 / 5);
        }
    };

#pragma unroll
    for (int i = 0; i < NR; ++i) read(smem, 0, 0, i);
    // one chunk, in stage cur; next: another chunk follows, in stage oth; more: and the one STAGES
    // after this one too, whose loads are issued here
    auto chunk = [&](unsigned char *cur, unsigned char *oth, auto next, auto more) {
        constexpr bool NEXT = decltype(next)::value, MORE = decltype(more)::value;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool last = q == Q - 1;
            if (last && NEXT) {
                // the next chunk's loads have landed (the later chunks' may be in flight) and this wave
                // has its last fragments of this chunk; after the barrier that holds for every wave
                wait_vmcnt<MORE ? (STAGES - 2) * NI : 0>();
                wait_lgkm0();
                lds_barrier();
            }
            const int nside = last ? (NEXT ? NR + (MORE ? NI : 0) : 0) : NR;
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                mfma(q, k);
#pragma unroll
                for (int e = k * nside / NM; e < (k + 1) * nside / NM; ++e) {
                    if (e < NR) read(last ? oth : cur, last ? 0 : q + 1, (q + 1) & 1, e);
                    else issue(ti, cur, e - NR);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (MORE) advance(ti);
    };
    using std::integral_constant;
    using yes = integral_constant<bool, true>;
    using no = integral_constant<bool, false>;
    int kc = 0;
    unsigned char *cur = smem;
    auto after = [&](unsigned char *p) { return p == smem + (STAGES - 1) * STAGE ? smem : p + STAGE; };
    for (; kc + STAGES < nch; ++kc) {
        chunk(cur, after(cur), yes{}, yes{});
        cur = after(cur);
    }
    for (; kc + 1 < nch; ++kc) {
        chunk(cur, after(cur), yes{}, no{});
        cur = after(cur);
    }
    chunk(cur, cur, no{}, no{});
    if constexpr (NBUF > 1) add(1, NB - 1, 0, 16);
    wait_lgkm0();
}

// One 32 x 32 block of outputs from D and W as given (W dense, [M][K]): filters m_lo .. m_lo + 31 (past
// the last: any) at the pixel of this lane, over channels [c0, c0 + g.Cg), the accumulators laid out as the
// main loops'.  Each half of the wave takes eight consecutive k of a 16-deep step, straight from memory,
// the next step's while the matrix cores work on this one's.
template <typename T>
__device__ inline floatx16 block_as_given(const Geom &g, const T *__restrict__ D, const T *__restrict__ W, int m_lo,
                                          long long pg, int c0, int lane) {
    const int h = lane >> 5, m = min(m_lo + (lane & 31), g.M - 1), RS = g.R * g.S, HW = g.H * g.W;
    const bool pvalid = pg < g.P_total;
    int n = 0, x = 0, y = 0;
    if (pvalid) {
        n = (int)(pg / g.EF);
        const int pix = (int)(pg - (long long)n * g.EF);
        x = pix / g.F;
        y = pix - x * g.F;
    }
    const int ih0 = g.U * x - g.P, iw0 = g.U * y - g.P;
    const T *d = D + n * g.CHW + (long long)c0 * HW;
    const T *w = W + (long long)m * g.K + (long long)c0 * RS;
    const int kn = g.Cg * RS;
    // this lane's k of a step: element (r, s) of the channel at offset off, eight a step, then eight past
    // the other half's
    const int c8 = 8 / RS, r8 = (8 - c8 * RS) / g.S, s8 = 8 - c8 * RS - r8 * g.S;
    int r = 0, s = 0, off = 0, k = 0;   // off: the channel's first element
    auto skip8 = [&] {
        s += s8;
        r += r8 + (s >= g.S ? 1 : 0);
        s -= s >= g.S ? g.S : 0;
        off += (c8 + (r >= g.R ? 1 : 0)) * HW;
        r -= r >= g.R ? g.R : 0;
        k += 8;
    };
    if (h) skip8();
    T a[8], b[8];
    auto fetch = [&](bool whole) {   // whole: both halves' k lie below kn
        // a filter's eight values in 16-byte loads, where value by value the loads of 64 rows' lines bound the
        // step (VGG-19 v6 with one value of 3e38: 1.77 ms, so 1.21 ms)
        if (whole) __builtin_memcpy(a, w + k, sizeof(a));
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const bool ok = k + v < kn;   // past the last k: zeros on both sides
            const int ih = ih0 + r, iw = iw0 + s;
            const bool in = ok & pvalid & ((unsigned)ih < (unsigned)g.H) & ((unsigned)iw < (unsigned)g.W);
            const T dv = d[in ? off + ih * g.W + iw : 0];
            b[v] = in ? dv : T(0);        // a tap in the padding is a product with zero
            if (!whole) {
                const T wv = w[ok ? k + v : 0];
                a[v] = ok ? wv : T(0);
            }
            const bool ws = ++s == g.S;
            s = ws ? 0 : s;
            r += ws ? 1 : 0;
            const bool wr = r == g.R;
            r = wr ? 0 : r;
            off += wr ? HW : 0;
        }
        k += 8;
        skip8();
    };
    floatx16 acc = {};
    fetch(kn >= 16);
    for (int kb = 0; kb < kn; kb += 16) {
        T ca[8], cb[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            ca[v] = a[v];
            cb[v] = b[v];
        }
        if (kb + 16 < kn) fetch(kb + 32 <= kn);
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int v = 0; v < 8; ++v) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ca[v], cb[v], acc, 0, 0, 0);
        } else {
            u16x8 va, vb;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                va[v] = ca[v];
                vb[v] = cb[v];
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va), __builtin_bit_cast(bf16x8, vb),
                                                          acc, 0, 0, 0);
        }
    }
    return acc;
}

// The outputs of a split or packed tile that came out non-finite, again from D and W as given, on the
// instructions of the operands' own type (eq. (1), the filter's own channels).  On packed copies the zeros
// that fill a filter's row meet input values beyond the tap, which must not count even when they are
// infinite.  On split copies an infinite, NaN or nearly overflowing operand has no split whose planes
// multiply to what fp32 gives (its lower planes are NaN or of either sign), so such an output says only
// that it must be redone.  A wave redoes its 32 x 32 blocks that hold such outputs, one after another.  The
// accumulators pass through LDS so that the loop over them is not unrolled; a finite tile pays one
// multiply-add an accumulator and a barrier.
template <typename C, int FM, int FP>
__device__ inline void redo_nonfinite(const Geom &g, const typename C::T *__restrict__ D,
                                      const typename C::T *__restrict__ W, int m0,
                                      long long p0, unsigned char *smem, floatx16 (&acc)[FM][FP], int tid, int arow0,
                                      int brow0) {
    constexpr int NA = FM * FP * 16;
    static_assert((size_t)C::NT * NA * sizeof(float) <= C::LDS_BYTES, "accumulators fit LDS");
    float t = 0.0f;   // 0 while every accumulator is finite, else NaN
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FP; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) t = fmaf(acc[i][j][e], 0.0f, t);
    __syncthreads();   // every wave is done with the operand tiles
    if (__ballot(!(t == 0.0f)) == 0) return;
    float *mine = reinterpret_cast<float *>(smem) + tid;
#pragma unroll
    for (int k = 0; k < NA; ++k) mine[k * C::NT] = acc[k / 16 / FP][k / 16 % FP][k % 16];
    const int lane = tid & 63, h = lane >> 5;
    for (int b = 0; b < FM * FP; ++b) {
        float *blk = mine + b * 16 * C::NT;
        const int m_lo = __builtin_amdgcn_readfirstlane(m0 + arow0) + b / FP * 32;
        const long long pg = p0 + brow0 + b % FP * 32 + (lane & 31);
        bool bad = false;   // an output of this lane that is not finite
        for (int e = 0; e < 16; ++e)
            bad |= !isfinite(blk[e * C::NT]) && m_lo + 8 * (e >> 2) + 4 * h + (e & 3) < g.M && pg < g.P_total;
        if (__ballot(bad) == 0) continue;
        const int g_hi = min(m_lo + 31, g.M - 1) / g.Mg;
        for (int gi = m_lo / g.Mg; gi <= g_hi; ++gi) {
            const floatx16 v = block_as_given(g, D, W, m_lo, pg, gi * g.Cg, lane);
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (!isfinite(blk[e * C::NT]) && (m_lo + 8 * (e >> 2) + 4 * h + (e & 3)) / g.Mg == gi)
                    blk[e * C::NT] = v[e];
        }
    }
#pragma unroll
    for (int k = 0; k < NA; ++k) acc[k / 16 / FP][k / 16 % FP][k % 16] = mine[k * C::NT];
    // the next use of LDS in this workgroup is behind a barrier
}

template <typename T> struct Bits;
template <> struct Bits<float> {
    using B = float;   // an fp32 output is stored as computed
    __device__ static B make(float v) { return v; }
    __device__ static float value(B b) { return b; }
};
template <> struct Bits<uint16_t> {
    using B = uint16_t;
    __device__ static B make(float v) { return f32_to_bf16_rne(v); }
    __device__ static float value(B b) { return bf16_bits_to_f32(b); }
};

// Two waves a SIMD at least on split tiles, as their LDS has room for: with up to 256 registers a lane the
// compiler keeps the steps' sums (dma_mainloop) in VGPRs, with more in AGPRs, from where every value takes a copy
// before its addition (protected: VGG-19 v2 1038 us, so 1003; 2 x 288 x 13^2 in two groups, 80 filters of 7 x 7, 64 x
// 64 tiles 223, so 192; fp32 instructions 877).
template <typename Tr, int WM, int WP, int FM, int FP, int WEAVE, bool KVEC, int EPI, bool NHWC, bool GRP = false,
          bool SK = false>
__global__ __launch_bounds__(64 * WM * WP, Tr::NP == 3 || WM * WP > 4 ? 2 : 1)
void conv_kernel(const typename Tr::T *__restrict__ D, const typename Tr::T *__restrict__ Wt,
                 typename Tr::T *__restrict__ O, Geom g, int tiles_m, int tiles_total, int m_major, const void *zp,
                 Epi<EPI> ep, SkArgs sk) {
    using C = Cfg<Tr, WM, WP, FM, FP, KVEC, dma_stages(WEAVE)>;
    using T = typename C::T;
    extern __shared__ __align__(16) unsigned char smem[];
    T *As0 = reinterpret_cast<T *>(smem);
    T *Bs0 = As0 + 2 * C::TM * C::LDK;

    const int tid = threadIdx.x;
    int bid = blockIdx.x;
    if constexpr (EPI != 0) {
        if (bid == 0 && tid == 0) {
            reset_report(ep.rep, ep.cap);
            ep.rep->reserved[1] = ep.co_slices;
        }
        if (ep.aux_groups > 0) {
            int ab = -1;   // this workgroup's index among the extra ones
            if (ep.aux_kind == 2) {
                if ((bid >> 3) >= ep.tile_groups) ab = bid - 8 * ep.tile_groups;
            } else if ((bid >> 3) < ep.aux_groups) {
                ab = bid;
            } else {
                bid -= 8 * ep.aux_groups;   // keeps bid % 8, hence the XCD the tile order assumes
            }
            if (ab >= 0) {
                const int bid = ab;
                if (bid < ep.aux_blocks) {
                    if (ep.aux_kind == 1) {
                        if (ep.enc_vec) encode_block<T, C::NT, kEncVec>(D, g, bid, ep.cd1, ep.cd2);
                        else encode_block<T, C::NT, 1>(D, g, bid, ep.cd1, ep.cd2);
                    } else {
                        coc_block<C::NT>(g, ep.co, ep.cd1, ep.cd2, ep.cw1, ep.cw2, ep.copart, bid,
                                         reinterpret_cast<double *>(smem));
                    }
                }
                return;
            }
        }
    }
    constexpr bool DMA = NHWC && WEAVE >= 3;
    // the stream-K form (a separate kernel: the whole-tile kernels keep their registers) of the
    // loops that can run a range of a tile's chunks (channels-last, dense)
    constexpr bool SKOK = SK && NHWC && WEAVE >= 3;
    constexpr bool skm = SKOK;
    long long sk_it = 0, sk_end = 0, sk_u = 0, sk_i0 = 0;
    int wl = 0, dp = 0;
    if (skm) {
        if (bid >= sk.S) return;
        // contiguous tiles and iteration ranges per XCD, as the tile order below
        wl = xcd_tile(bid, sk.S);
        sk_i0 = (long long)sk.dp_waves * sk.S * sk.nch;   // the first shared iteration
        sk_u = (long long)tiles_total * sk.nch - sk_i0;
        sk_it = sk_i0 + (long long)wl * sk_u / sk.S;
        sk_end = sk_i0 + (long long)(wl + 1) * sk_u / sk.S;
    } else if (bid >= tiles_total) {
        return;
    }
    bool first_seg = true;    // the next shared segment is this workgroup's first
    bool first_iter = true;
    const Geom &g_all = g;
    for (;;) {
    // In the stream-K kernel the thread index and the geometry are passed through empty asm at
    // every segment, so that nothing derived from them is hoisted out of the segment loop and
    // held (in registers, or spilled) across the main loop and the epilogue.
    int tid;
    Geom g = g_all;
    if constexpr (SK) {
        asm volatile("v_mov_b32 %0, %1" : "=v"(tid) : "v"((int)threadIdx.x));
        asm volatile("" : "+s"(g.N), "+s"(g.C), "+s"(g.H), "+s"(g.W), "+s"(g.M), "+s"(g.R), "+s"(g.S));
        asm volatile("" : "+s"(g.U), "+s"(g.P), "+s"(g.E), "+s"(g.F), "+s"(g.K), "+s"(g.EF));
        asm volatile("" : "+s"(g.CHW), "+s"(g.P_total), "+s"(g.wbase));
    } else {
        tid = threadIdx.x;
    }
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wp = wave / WM;
    // the segment: chunks [k0, k0 + kn) of one tile (kn < 0: the whole tile)
    int tile, k0 = 0, kn = -1;
    if (skm) {
        if (dp < sk.dp_waves) {
            tile = dp * sk.S + wl;
            kn = sk.nch;
        } else {
            if (sk_it >= sk_end) break;
            tile = (int)(sk_it / sk.nch);
            k0 = (int)(sk_it - (long long)tile * sk.nch);
            kn = (int)(sk_end - sk_it < (long long)(sk.nch - k0) ? sk_end - sk_it : (long long)(sk.nch - k0));
        }
        if (!first_iter) __syncthreads();   // every wave is done with the last segment's LDS
    } else {
        // logical tile order: pixel-major keeps the M tiles of one pixel tile on one
        // XCD (its L2 serves the repeated D reads); M-major keeps one slab of W
        // resident per XCD instead (preferred when W is larger than an XCD's L2)
        tile = xcd_tile(bid, tiles_total);
    }
    const int tiles_p = tiles_total / tiles_m;
    const int mt = m_major ? tile / tiles_p : tile % tiles_m;
    const int pt = m_major ? tile % tiles_p : tile / tiles_m;
    const int m0 = mt * C::TM;
    const long long p0 = (long long)pt * C::TP;

    // this thread's im2col pixel (fixed over the K loop)
    const int bp = tid % C::TP, bkg = tid / C::TP;
    const long long pg = p0 + bp;
    const bool pvalid = pg < g.P_total;
    int lane_base = 0, ih0 = 0, iw0 = 0;
    if (pvalid) {
        const int n = (int)(pg / g.EF);
        const int pix = (int)(pg - (long long)n * g.EF);
        const int x = pix / g.F, y = pix - (pix / g.F) * g.F;
        ih0 = g.U * x - g.P;
        iw0 = g.U * y - g.P;
        // channels-last: the image's base in Dt; otherwise the pixel's first tap in D
        lane_base = NHWC ? n * (int)g.CHW : n * (int)g.CHW + ih0 * g.W + iw0;
    }
    ASlots<C> as;
    a_slots<C>(g, m0, tid, as);

    floatx16 acc[FM][FP];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FP; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    const int arow0 = wm * FM * 32, brow0 = wp * FP * 32;
    Pack<T, C::VEC> ra[C::A_PER];
    Pack<T, C::VEC> rb[C::KR / C::VEC];
    const int nchunks = (g.K + C::TK - 1) / C::TK;
    // grouped layers (Sec. 5.2) run on the block-diagonal expansion of W: a tile whose filters all
    // lie in one group needs only the chunks of K = (r, s, c) with c in that group's channels (the
    // others multiply zeros), and the channels-last loop below walks just those
    constexpr bool KSKIP = GRP && NHWC && !DMA && WEAVE != 2;   // a separate kernel: dense loops unchanged
    int nch = nchunks, cpr = 0, cg0 = 0;
    if constexpr (KSKIP) {
        const int mlast = (m0 + C::TM < g.M ? m0 + C::TM : g.M) - 1;
        if (g.G > 1 && g.Cg % C::TK == 0 && m0 / g.Mg == mlast / g.Mg) {
            cpr = g.Cg / C::TK;
            cg0 = group_first_channel(g, m0);
            nch = g.R * g.S * cpr;
        }
    }
    auto kbase = [&](int j) {
        if (KSKIP && cpr > 0) {
            const int rs = j / cpr;
            return rs * g.C + cg0 + (j - rs * cpr) * C::TK;
        }
        return j * C::TK;
    };
    typename C::Mask amask = 0, bmask = 0;
    // channels-last loops other than the two-in-flight one: chunks walked by TapWalk, channel
    // blocks [cg0, cg0 + TK * (nch / (R S))) outer, taps inner
    constexpr bool TAPS = NHWC && !DMA && WEAVE != 2;
    TapWalk tw{0, 0, 0};
    int pix_off = 0;
    const uintptr_t zpa = reinterpret_cast<uintptr_t>(zp);   // 256 zero bytes (channels-last layers)
    if constexpr (TAPS) {
        tw.c0 = cg0;
        if (!(KSKIP && cpr > 0)) nch = g.R * g.S * (g.C / C::TK);
        pix_off = lane_base + (ih0 * g.W + iw0) * g.C + bkg * C::KR;
    }
    if constexpr (!DMA) {
        if constexpr (TAPS) {
            load_a_tap<C>(Wt, tw.kb(g), as, zpa, ra);
            load_b_tap<C>(D, g, tw, pvalid, pix_off, ih0, iw0, zpa, rb);
        } else {
            amask = load_a<C>(Wt, g, kbase(0), KVEC, as, ra);
            bmask = NHWC ? load_b_nhwc<C>(D, g, kbase(0) + bkg * C::KR, pvalid, lane_base, ih0, iw0, rb)
                         : load_b<C>(D, g, bkg * C::KR, pvalid, lane_base, ih0, iw0, rb);
        }
        store_lds<C, NHWC>(As0, Bs0, tid, ra, amask, rb, bmask, bp, bkg);
        __syncthreads();
    }

    if constexpr (DMA) {
        // D is the channels-last copy, which the workspace keeps right behind the zero page zp
        // grouped layers run on the block-diagonal expansion of W: the tile walks the channel blocks
        // its filters' groups reach into (all of them when G = 1)
        const int mlast = (m0 + C::TM < g.M ? m0 + C::TM : g.M) - 1;
        const int c_lo = group_first_channel(g, m0) / C::TK * C::TK;
        const int c_hi = (group_first_channel(g, mlast) + g.Cg + C::TK - 1) / C::TK * C::TK;
        dma_mainloop<C, Tr::NP, dma_stages(WEAVE), packed_loop(WEAVE), WEAVE == 7, FM, FP>(Wt, g, m0, p0, static_cast<const unsigned char *>(zp), smem, acc, tid, arow0,
                                        brow0, k0, kn, c_lo, c_hi);
    } else if constexpr (NHWC && WEAVE == 2) {
        // channels-last, two chunks in flight: chunk kc + 2 is loaded into one register set
        // while chunk kc is consumed from LDS, and chunk kc + 1 (loaded a whole chunk earlier,
        // in the other set) then goes to the other LDS buffer, so the stores wait only on loads
        // issued two chunks back.  Unrolled by two so that each register set keeps its
        // registers; loads past the last chunk are fully masked (in-bounds, no effect).
        Pack<T, C::VEC> ra2[C::A_PER];
        Pack<T, C::VEC> rb2[C::KR / C::VEC];
        typename C::Mask amask2 = load_a<C>(Wt, g, C::TK, KVEC, as, ra2);
        typename C::Mask bmask2 = load_b_nhwc<C>(D, g, C::TK + bkg * C::KR, pvalid, lane_base, ih0, iw0, rb2);
        T *A0 = As0, *A1 = As0 + C::TM * C::LDK, *B0 = Bs0, *B1 = Bs0 + C::TP * C::LDK;
        // no exit inside the body (a chunk past the end is stored as zeros and never used), so the
        // accumulators stay in one set of registers
        int kc = 0;
        for (; kc + 1 < nchunks; kc += 2) {
            amask = load_a<C>(Wt, g, (kc + 2) * C::TK, KVEC, as, ra);
            bmask = load_b_nhwc<C>(D, g, (kc + 2) * C::TK + bkg * C::KR, pvalid, lane_base, ih0, iw0, rb);
            mma_chunk<C, FM, FP>(A0, B0, lane, arow0, brow0, acc);
            store_lds<C, NHWC>(A1, B1, tid, ra2, amask2, rb2, bmask2, bp, bkg);
            __syncthreads();
            amask2 = load_a<C>(Wt, g, (kc + 3) * C::TK, KVEC, as, ra2);
            bmask2 = load_b_nhwc<C>(D, g, (kc + 3) * C::TK + bkg * C::KR, pvalid, lane_base, ih0, iw0, rb2);
            mma_chunk<C, FM, FP>(A1, B1, lane, arow0, brow0, acc);
            store_lds<C, NHWC>(A0, B0, tid, ra, amask, rb, bmask, bp, bkg);
            __syncthreads();
        }
        if (kc < nchunks) mma_chunk<C, FM, FP>(A0, B0, lane, arow0, brow0, acc);   // odd count: the last chunk
    } else if constexpr (NHWC) {
        // channels-last: a whole chunk's gather is a few 16-byte loads per thread, issued
        // before this chunk's MFMAs and stored after them.  The scheduling fences keep the
        // compiler from sinking the loads next to their stores: they then have the whole
        // chunk of MFMAs to land instead of a few.
        for (int kc = 0; kc + 1 < nch; ++kc) {
            const int buf = kc & 1;
            tw.next(g, C::TK);
            load_a_tap<C>(Wt, tw.kb(g), as, zpa, ra);
            load_b_tap<C>(D, g, tw, pvalid, pix_off, ih0, iw0, zpa, rb);
            __builtin_amdgcn_sched_barrier(0);
            mma_chunk<C, FM, FP>(As0 + buf * C::TM * C::LDK, Bs0 + buf * C::TP * C::LDK, lane, arow0, brow0, acc);
            __builtin_amdgcn_sched_barrier(0);
            store_lds<C, NHWC>(As0 + (buf ^ 1) * C::TM * C::LDK, Bs0 + (buf ^ 1) * C::TP * C::LDK, tid, ra, amask, rb,
                         bmask, bp, bkg);
            __syncthreads();
        }
        mma_chunk<C, FM, FP>(As0 + ((nch - 1) & 1) * C::TM * C::LDK, Bs0 + ((nch - 1) & 1) * C::TP * C::LDK,
                             lane, arow0, brow0, acc);
    } else if constexpr (WEAVE == 2 && sizeof(T) == 4) {
        // two chunks in flight: while a chunk is consumed from one LDS buffer, the gather of the
        // chunk two ahead is woven between its MFMAs into one register set, and the other set
        // (the next chunk, loaded a whole chunk earlier) goes to the other buffer at the end, so
        // no load latency is waited on.  The loop is unrolled by two so that each register set
        // keeps its registers; chunks past the last one are fully masked (zeros, no effect).
        Pack<T, C::VEC> ra2[C::A_PER];
        Pack<T, C::VEC> rb2[C::KR / C::VEC];
        typename C::Mask amask2 = load_a<C>(Wt, g, C::TK, KVEC, as, ra2);
        BGather<C> bg, bg2;
        bg2.mask = load_b<C>(D, g, C::TK + bkg * C::KR, pvalid, lane_base, ih0, iw0, rb2);
        const float *A0 = reinterpret_cast<const float *>(As0), *A1 = A0 + C::TM * C::LDK;
        const float *B0 = reinterpret_cast<const float *>(Bs0), *B1 = B0 + C::TP * C::LDK;
        for (int kc = 0; kc < nchunks; kc += 2) {
            chunk_f32<C, FM, FP, true>(A0, B0, lane, arow0, brow0, acc, D, Wt, g, (kc + 2) * C::TK, KVEC, as, ra,
                                       amask, bg, bkg, pvalid, lane_base, ih0, iw0, rb);
            store_lds<C>(As0 + C::TM * C::LDK, Bs0 + C::TP * C::LDK, tid, ra2, amask2, rb2, bg2.mask, bp, bkg);
            __syncthreads();
            chunk_f32<C, FM, FP, true>(A1, B1, lane, arow0, brow0, acc, D, Wt, g, (kc + 3) * C::TK, KVEC, as, ra2,
                                       amask2, bg2, bkg, pvalid, lane_base, ih0, iw0, rb2);
            if (kc + 2 >= nchunks) break;
            store_lds<C>(As0, Bs0, tid, ra, amask, rb, bg.mask, bp, bkg);
            __syncthreads();
        }
    } else if constexpr (WEAVE == 1 && sizeof(T) == 4) {
        // every chunk but the last: the next chunk's gather is woven between this chunk's MFMAs
        BGather<C> bg;
        for (int kc = 0; kc + 1 < nchunks; ++kc) {
            const int buf = kc & 1;
            chunk_f32<C, FM, FP, true>(reinterpret_cast<const float *>(As0 + buf * C::TM * C::LDK),
                                       reinterpret_cast<const float *>(Bs0 + buf * C::TP * C::LDK), lane, arow0,
                                       brow0, acc, D, Wt, g, (kc + 1) * C::TK, KVEC, as, ra, amask, bg, bkg,
                                       pvalid, lane_base, ih0, iw0, rb);
            store_lds<C>(As0 + (buf ^ 1) * C::TM * C::LDK, Bs0 + (buf ^ 1) * C::TP * C::LDK, tid, ra, amask, rb,
                         bg.mask, bp, bkg);
            __syncthreads();
        }
        chunk_f32<C, FM, FP, false>(reinterpret_cast<const float *>(As0 + ((nchunks - 1) & 1) * C::TM * C::LDK),
                                    reinterpret_cast<const float *>(Bs0 + ((nchunks - 1) & 1) * C::TP * C::LDK),
                                    lane, arow0, brow0, acc, D, Wt, g, 0, KVEC, as, ra, amask, bg, bkg, pvalid,
                                    lane_base, ih0, iw0, rb);
    } else {
        auto mma = [&](int buf) {
            const T *As = As0 + buf * C::TM * C::LDK;
            const T *Bs = Bs0 + buf * C::TP * C::LDK;
            if constexpr (sizeof(T) == 4)
                mma_f32<C::TK, FM, FP>(reinterpret_cast<const float *>(As), reinterpret_cast<const float *>(Bs),
                                       lane, arow0, brow0, acc);
            else
                mma_bf16<C::TK, FM, FP>(reinterpret_cast<const uint16_t *>(As),
                                        reinterpret_cast<const uint16_t *>(Bs), lane, arow0, brow0, acc);
        };
        // every chunk but the last: fetch the next one while the MFMAs consume this one
        for (int kc = 0; kc + 1 < nchunks; ++kc) {
            const int buf = kc & 1;
            const int kb = (kc + 1) * C::TK;
            amask = load_a<C>(Wt, g, kb, KVEC, as, ra);
            bmask = load_b<C>(D, g, kb + bkg * C::KR, pvalid, lane_base, ih0, iw0, rb);
            mma(buf);
            store_lds<C>(As0 + (buf ^ 1) * C::TM * C::LDK, Bs0 + (buf ^ 1) * C::TP * C::LDK, tid, ra, amask, rb,
                         bmask, bp, bkg);
            __syncthreads();
        }
        mma((nchunks - 1) & 1);
    }

    if constexpr (SKOK) {
        if (kn >= 0 && kn < sk.nch) {
            // a part of the tile: publish it; the last of the tile's workgroups sums them all
            const long long ib = (long long)tile * sk.nch;
            // the workgroup whose range holds iteration i
            auto owner = [&](long long i) { return (int)(((i - sk_i0 + 1) * sk.S - 1) / sk_u); };
            const int w0 = owner(ib), w1 = owner(ib + sk.nch - 1);
            // a slot: FM * FP * 4 rows of NT 16-byte units, four accumulators of a thread each
            static_assert(FM * FP * 16 * C::NT == C::TM * C::TP, "slot size");
            const __amdgpu_buffer_rsrc_t rp = buffer_rsrc(sk.part, (unsigned)sk.S * 2u * (C::TM * C::TP * 4u));
            auto slot_at = [&](int w, int slot) { return ((unsigned)w * 2u + (unsigned)slot) * (C::TM * C::TP * 4u); };
            const unsigned mine = slot_at(wl, first_seg ? 0 : 1);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FP; ++j) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const floatx4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2],
                                           acc[i][j][4 * q + 3]};
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rp,
                                                               (((i * FP + j) * 4 + q) * C::NT + tid) * 16, mine,
                                                               kDeviceCoherent);
                    }
                    __builtin_amdgcn_sched_barrier(0);   // a few units live at a time
                }
            // The parts go to memory with device-coherent stores (they bypass the XCD's L2), so
            // once every wave has seen its stores complete, one device-scope count publishes the
            // whole part: no L2 write-back is needed.  Every wave is past the main loop: the first
            // word of LDS carries the verdict.
            int *sk_last = reinterpret_cast<int *>(smem);
            wait_vmcnt<0>();
            __syncthreads();
            if (tid == 0)
                *sk_last = __hip_atomic_fetch_add(sk.cnt + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                           w1 - w0;
            __syncthreads();
            const bool last = *sk_last != 0;
            if (!last) {
                sk_it += kn;
                first_seg = false;
                first_iter = false;
                continue;
            }
            // the other parts, read with device-coherent loads after the count said they are all there
            if (tid == 0) __hip_atomic_store(sk.cnt + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // the tile's parts in chunk order (this workgroup's own from its slot too): part w lies
            // in slot 0 of workgroup w when its range starts inside this tile, else in its slot 1
            // (its last segment).  A block of 32 x 32 at a time, four parts of it in flight.
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FP; ++j) {
                    for (int w = w0; w <= w1; w += 4) {
                        floatx4 v[4][4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int wu = w + u <= w1 ? w + u : w1;   // past the last: read again, not added
                            const unsigned src = slot_at(wu, sk_i0 + (long long)wu * sk_u / sk.S >= ib ? 0 : 1);
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                v[u][q] = __builtin_bit_cast(
                                    floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                                                 rp, (((i * FP + j) * 4 + q) * C::NT + tid) * 16, src, kDeviceCoherent));
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (w + u <= w1)
#pragma unroll
                                for (int e = 0; e < 16; ++e)
                                    acc[i][j][e] = w + u == w0 ? v[u][e / 4][e % 4] : acc[i][j][e] + v[u][e / 4][e % 4];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
    }

    if constexpr (DMA && Tr::NP == 3) {
        // the copies' scale out
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FP; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] *= kSplitUnscale;
    }
    if constexpr (DMA && (Tr::NP == 3 || packed_loop(WEAVE)))
        redo_nonfinite<C, FM, FP>(g, static_cast<const T *>(ep.src_dw.d), static_cast<const T *>(ep.src_dw.w), m0, p0,
                                  smem, acc, tid, arow0, brow0);

    // epilogue: lane owns pixel (lane & 31) of each 32-wide block; register e of
    // block (i, j) is row 8*(e/4) + 4*(lane/32) + e%4 of that block
    const int l32 = lane & 31, h = lane >> 5;
    // the tile's bias rows (Sec. 5.1), staged in LDS once the main loop is done: read in the store
    // loops below from LDS, whose wait never holds on the tile's own output stores
    const bool hb = ep.bias != nullptr;
    constexpr size_t kBiasOff = EPI == 0 ? 0 : (size_t)WM * 3 * C::TP * sizeof(double);
    static_assert(kBiasOff + C::TM * sizeof(float) <= C::LDS_BYTES, "bias rows fit LDS");
    float *bias_s = reinterpret_cast<float *>(smem + kBiasOff);
    if (hb) {
        __syncthreads();   // every wave is done with the operand tiles
        for (int t = tid; t < C::TM; t += C::NT) bias_s[t] = m0 + t < g.M ? ep.bias[m0 + t] : 0.0f;
        __syncthreads();
    }
    if constexpr (EPI == 0) {
        if (!hb) {
#pragma unroll
            for (int j = 0; j < FP; ++j) {
                const long long pgo = p0 + brow0 + j * 32 + l32;
                if (pgo >= g.P_total) continue;
                const long long n = pgo / g.EF;
                const long long ob = n * g.M * (long long)g.EF + (pgo - n * g.EF);
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int m = m0 + arow0 + i * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
                        if (m < g.M) Elem<T>::store(O, ob + (long long)m * g.EF, acc[i][j][e]);
                    }
            }
        } else {
#pragma unroll
            for (int j = 0; j < FP; ++j) {
                const long long pgo = p0 + brow0 + j * 32 + l32;
                if (pgo >= g.P_total) continue;
                const long long n = pgo / g.EF;
                const long long ob = n * g.M * (long long)g.EF + (pgo - n * g.EF);
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int mt_row = arow0 + i * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
                        const int m = m0 + mt_row;
                        if (m < g.M) Elem<T>::store(O, ob + (long long)m * g.EF, acc[i][j][e] + bias_s[mt_row]);
                    }
            }
        }
    } else {
        using Bt = Bits<T>;
        // faults inside this tile (a uniform test; usually none)
        bool planted = false;
        if constexpr (EPI == 2) {
            for (int f = 0; f < ep.fl.n; ++f) {
                const ftcnn_fault &q = ep.fl.f[f];
                const long long pf = (long long)q.n * g.EF + (long long)q.x * g.F + q.y;
                planted |= q.m >= m0 && q.m < m0 + C::TM && pf >= p0 && pf < p0 + C::TP;
            }
        }
        if constexpr (WM > 1) __syncthreads();  // the LDS tiles are free: reuse them for the cross-wave fold
        double *red = reinterpret_cast<double *>(smem);   // [WM][3][TP]
        const double wb = (double)g.wbase;
        // per-column state; rows are visited one register at a time (row-dependent
        // values are then live only briefly, which keeps the kernel's register
        // budget, and so the main loop's occupancy, close to the plain store's)
        const int mrow = m0 + arow0 + 4 * h;
        T *obase[FP];
        long long pcol[FP];
        bool cval[FP];
        double s1[FP], s6[FP], sq[FP];
#pragma unroll
        for (int j = 0; j < FP; ++j) {
            const long long pgo = p0 + brow0 + j * 32 + l32;
            cval[j] = pgo < g.P_total;
            const long long n = cval[j] ? pgo / g.EF : 0;
            pcol[j] = pgo;
            obase[j] = O + (n * g.M + mrow) * (long long)g.EF + (pgo - n * g.EF);
            s1[j] = s6[j] = sq[j] = 0.0;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            if constexpr (sizeof(T) == 2) {
                // bf16 outputs: the 16 rows of a block are first summed in fp32, then added in
                // fp64.  Every term is exact in fp32 (8-bit values, weights m + wbase below 2^16),
                // so the only roundings are the 15 additions of a run: at most 15 * 2^-24 of the
                // run's sum of magnitudes, far inside the bf16 tolerance (whose output unit is
                // 2^-8), and none at all while the partial sums stay integers below 2^24.  The
                // fp64 arithmetic per element would otherwise cost as much as a third of the
                // matrix-core time on short-K layers.
                float f1[FP], f6[FP], fq[FP];
#pragma unroll
                for (int j = 0; j < FP; ++j) f1[j] = f6[j] = fq[j] = 0.0f;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int mo = i * 32 + 8 * (e >> 2) + (e & 3);   // row offset from mrow
                    const int m = mrow + mo;
                    const bool mok = m < g.M;
                    const float wm = (float)(m + g.wbase);
                    const float bm = hb ? bias_s[m - m0] : 0.0f;
#pragma unroll
                    for (int j = 0; j < FP; ++j) {
                        const typename Bt::B b = Bt::make(hb ? acc[i][j][e] + bm : acc[i][j][e]);
                        if (cval[j] && mok) {
                            const float v = Bt::value(b);
                            f1[j] += v;
                            f6[j] = fmaf(wm, v, f6[j]);
                            fq[j] = fmaf(v, v, fq[j]);
                            obase[j][(long long)mo * g.EF] = b;
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < FP; ++j) {
                    s1[j] += (double)f1[j];
                    s6[j] += (double)f6[j];
                    sq[j] += (double)fq[j];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int mo = i * 32 + 8 * (e >> 2) + (e & 3);   // row offset from mrow
                    const int m = mrow + mo;
                    const bool mok = m < g.M;
                    const double wm = (double)m + wb;
                    const float bm = hb ? bias_s[m - m0] : 0.0f;
#pragma unroll
                    for (int j = 0; j < FP; ++j) {
                        const typename Bt::B b = Bt::make(hb ? acc[i][j][e] + bm : acc[i][j][e]);
                        if (cval[j] && mok) {
                            const double v = (double)Bt::value(b);
                            s1[j] += v;
                            s6[j] = fma(wm, v, s6[j]);
                            sq[j] = fma(v, v, sq[j]);
                            obase[j][(long long)mo * g.EF] = b;
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < FP; ++j) {
            // rows 4..7 of every 8 sit in the other half-wave: both halves end with the same sums
            const double a1 = s1[j] + __shfl_xor(s1[j], 32, 64);
            const double a6 = s6[j] + __shfl_xor(s6[j], 32, 64);
            const double aq = sq[j] + __shfl_xor(sq[j], 32, 64);
            const int cl = brow0 + j * 32 + l32;
            if (WM == 1) {
                if (h == 0 && cval[j]) {
                    const long long pgo = pcol[j];
                    const long long n = pgo / g.EF;
                    double *dst = ep.part + ((size_t)mt * g.N + n) * 4 * g.EF + (pgo - n * g.EF);
                    dst[0] = a1;
                    dst[g.EF] = a6;
                    dst[2 * (size_t)g.EF] = ((double)n + wb) * a1;
                    dst[3 * (size_t)g.EF] = aq;
                }
            } else if (h == 0) {
                red[(wm * 3 + 0) * C::TP + cl] = a1;
                red[(wm * 3 + 1) * C::TP + cl] = a6;
                red[(wm * 3 + 2) * C::TP + cl] = aq;
            }
        }
        if constexpr (WM > 1) {
            __syncthreads();
            for (int cl = tid; cl < C::TP; cl += C::NT) {
                const long long pgo = p0 + cl;
                if (pgo >= g.P_total) continue;
                double s1 = 0.0, s6 = 0.0, sq = 0.0;
#pragma unroll
                for (int w = 0; w < WM; ++w) {
                    s1 += red[(w * 3 + 0) * C::TP + cl];
                    s6 += red[(w * 3 + 1) * C::TP + cl];
                    sq += red[(w * 3 + 2) * C::TP + cl];
                }
                const long long n = pgo / g.EF;
                double *dst = ep.part + ((size_t)mt * g.N + n) * 4 * g.EF + (pgo - n * g.EF);
                dst[0] = s1;
                dst[g.EF] = s6;
                dst[2 * (size_t)g.EF] = ((double)n + wb) * s1;
                dst[3 * (size_t)g.EF] = sq;
            }
        }
        if constexpr (EPI == 2) {
            // the planted faults of this tile, in list order, on the values as stored: each one
            // rewrites its element of O and moves the tile's partial sums of that pixel by the
            // change it made (one thread, after every store of the tile is done)
            if (planted) {
                __syncthreads();
                if (tid == 0) {
                    for (int f = 0; f < ep.fl.n; ++f) {
                        const ftcnn_fault &q = ep.fl.f[f];
                        const long long pf = (long long)q.n * g.EF + (long long)q.x * g.F + q.y;
                        if (!(q.m >= m0 && q.m < m0 + C::TM && pf >= p0 && pf < p0 + C::TP)) continue;
                        const long long pos = pf - (long long)q.n * g.EF;
                        T *o = O + ((long long)q.n * g.M + q.m) * g.EF + pos;
                        const typename Bt::B b = *o, b2 = fault_apply(b, q);
                        *o = b2;
                        const double v = (double)Bt::value(b), v2 = (double)Bt::value(b2), d = v2 - v;
                        double *dst = ep.part + ((size_t)mt * g.N + q.n) * 4 * g.EF + pos;
                        dst[0] += d;
                        dst[g.EF] += ((double)q.m + wb) * d;
                        dst[2 * (size_t)g.EF] += ((double)q.n + wb) * d;
                        dst[3 * (size_t)g.EF] += v2 * v2 - v * v;
                    }
                }
            }
        }
    }
    if (!skm) break;
    first_iter = false;
    if (dp < sk.dp_waves) {
        ++dp;
    } else {
        sk_it += kn;
        first_seg = false;
    }
    }   // segments
}

}  // namespace convk
}  // namespace ftcnn
