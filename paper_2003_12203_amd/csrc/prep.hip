// Channels-last copies for the convolution's vector-gather path: the same
// tensors as eq. (1) uses, in another order,
//   Dt[n][h][w][c] = D[n][c][h][w],   Wt[m][r][s][c] = W[m][c][r][s],
// so that the K = (r, s, c) run of one pixel is contiguous in memory and the
// im2col gather becomes 16-byte loads.
//
// The copy of D also encodes the input checksums of Sec. 3.2,
//   Cd1 = sum_n D_n,   Cd2 = sum_n (n + wbase) D_n,
// from the values it moves, so D is read once for both.  A workgroup owns a
// tile of 32 (or 64) channels x TH positions of the feature maps and walks the
// images in order, keeping the running float64 sums of its tile in registers.
// On layers with few tiles (Plan::enc_apart) other workgroups of the launch
// encode, and each round of images of a tile is a workgroup.
//
// Every global access is a 16-byte vector.  A channel row of the tile is read
// as eight aligned vectors.  When H*W is a multiple of the vector the row
// segment starts on a vector and the tile is eight vectors wide; otherwise it
// starts s elements into its first vector (s depends on the channel and the
// tile, not on the image, because Ch*H*W is a multiple of the vector) and the
// tile is seven vectors wide, the eighth covering the shift.
#include "encode_block.h"
#include "ftcnn_internal.h"

namespace ftcnn {
namespace {

// Transpose tile: TC channels x TH positions per image.  ROW = 8 vectors are
// loaded per channel row; TC = 32 channels, or 64 for bf16 when the channel
// count allows (a stored position is then one 128-byte line).  Every thread
// loads TC/32 vectors (one channel row each) per image and stores TC/32 vectors
// of channels (one position each).
template <typename T, int TC_, bool SHIFT_> struct PrepT {
    static constexpr int TC = TC_;
    static constexpr bool SHIFT = SHIFT_;
    static constexpr int VEC = 16 / sizeof(T);          // elements per 16-byte vector
    static constexpr int ROW = 8 * VEC;                  // elements loaded per channel row
    static constexpr int TH = (SHIFT ? 7 : 8) * VEC;     // positions per tile
    static constexpr int LDT = ROW + 4 / sizeof(T);      // LDS row, padded by one word
    static constexpr int RPT = TC / 32;                  // channel rows per thread
    static constexpr int BATCH = kPrepBatch * 32 / TC;   // images per round (one LDS tile each)
    static constexpr int LDS_ELEMS = BATCH * TC * LDT;
};

template <typename T> __device__ inline double widen(T v) {
    if constexpr (sizeof(T) == 4) return (double)v;
    else return (double)bf16_bits_to_f32(v);
}

template <typename T, int V> union VecT {
    uint4 q;
    T e[V];
};

// Eight values split into three bf16 planes whose sum they are: each plane the nearest bf16 of what
// the ones before left over (8 + 8 + 8 significand bits hold all 24; every difference is exact).
// Plane pl goes to dst + STEP pl.
template <int STEP> __device__ inline void store_split8(const float (&x)[8], uint16_t *dst) {
    union { uint4 q; uint16_t e[8]; } pl[3];
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        pl[0].e[v] = f32_to_bf16_rne(x[v]);
        const float r1 = x[v] - bf16_bits_to_f32(pl[0].e[v]);
        pl[1].e[v] = f32_to_bf16_rne(r1);
        pl[2].e[v] = f32_to_bf16_rne(r1 - bf16_bits_to_f32(pl[1].e[v]));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<uint4 *>(dst + STEP * k) = pl[k].q;
}

// Workgroup b's tile of `total`: each XCD (ids are dealt round-robin over 8) takes a run of neighbouring
// tiles, whose reads and stores then share lines in one L2.  The copies are bound by memory; with tiles
// dealt out by id, protected layers took longer: VGG-19 v2 fp32 1062 us (in runs 1038), v4 733 (715), Darknet-19
// 1x1 45.3 (43.4), AlexNet conv4 165.8 (163.2); bf16 VGG-19 v2 359 (351), ResNet-18 l3 57.4 (55.2), its
// projection 31.0 (28.9); VGG-19 v6 the same in both types, Darknet-19 c4 87.7 (89).  Channel blocks before
// positions within a run: v2 1 % faster, 1x1 4 % slower.  Packed copies keep the id order (with runs AlexNet
// conv1 was 3 % slower, 160 channels 1x1 5 % faster).
__device__ inline int xcd_run(int b, int total) {
    const int q = total / 8, rem = total % 8, x = b % 8;
    return x * q + (x < rem ? x : rem) + b / 8;
}

// vec_d / vec_w: D / W is 16-byte aligned (else element loads; the layout is
// the same with shift 0, which a tile of seven vectors also covers).
// SPLIT (fp32): the copies hold blocks of 32 channels as three bf16 planes of 32 (192 bytes): four
// threads then store 64 bytes that run on (groups of eight channels, plane after plane: Darknet-19 1x1 13.6 -> 17.8 us).
template <typename T, bool ENC, int TC, bool SHIFT, bool SPLIT>
__global__ __launch_bounds__(kThreads) void prep_kernel(const T *__restrict__ D, const T *__restrict__ W,
                                                        T *__restrict__ Dt, T *__restrict__ Wt, Geom g,
                                                        double *cd1, double *cd2, int tr_blocks, int hw_tiles, int c_tiles, int ns, int vec_d,
                                                        int vec_w, uint4 *__restrict__ zero16, int *__restrict__ skcnt,
                                                        int skcnt_n, int enc_blocks, int enc_vec) {
    using P = PrepT<T, TC, SHIFT>;
    constexpr int VEC = P::VEC, TH = P::TH, LDT = P::LDT, RPT = P::RPT, BATCH = P::BATCH;
    __shared__ T tile[BATCH][TC][LDT];
    int b = blockIdx.x;
    if constexpr (!ENC) {
        // the encode in workgroups of its own (pl.enc_apart), first: they walk all images
        if (b < enc_blocks) {
            if (enc_vec) encode_block<T, kThreads, kEncVec>(D, g, b, cd1, cd2);
            else encode_block<T, kThreads, 1>(D, g, b, cd1, cd2);
            return;
        }
        b -= enc_blocks;
    }
    const int HW = g.H * g.W;
    if (b < tr_blocks) {
        const int tiles = hw_tiles * c_tiles;
        b = xcd_run(b, tr_blocks);
        const int split = b / tiles, rest = b - split * tiles;
        const int ht = rest % hw_tiles, ct = rest / hw_tiles;
        const int n0 = (int)((long long)split * g.N / ns), n1 = (int)((long long)(split + 1) * g.N / ns);
        const int p0 = ht * TH;
        const int pend = p0 + TH < HW ? p0 + TH : HW;   // the tile's positions are [p0, pend)
        const int hmod = HW & (VEC - 1);
        // shift of channel row r of the tile: where position p0 sits in its vector
        auto shift = [&](int r) { return vec_d ? ((r & (VEC - 1)) * hmod + p0) & (VEC - 1) : 0; };
        // load role: channel rows cr + 32 q, vector vq of the row; its first element is at
        // position rel[q] of the row
        const int cr = threadIdx.x / 8, vq = threadIdx.x % 8;
        int rel[RPT];
        const T *src[RPT];
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            rel[q] = p0 - shift(cr + 32 * q) + vq * VEC;
            src[q] = D + (long long)(ct * TC + cr + 32 * q) * HW + rel[q];
        }
        // store role: positions hs + HS i of the tile, channels cg*VEC .. cg*VEC + VEC
        constexpr int CG = TC / VEC;
        constexpr int HS = kThreads / CG;                  // positions stored per pass
        const int hs = threadIdx.x / CG, cg = threadIdx.x % CG;
        int sv[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) sv[v] = shift(v);
        double a1[RPT][VEC], a2[RPT][VEC];
#pragma unroll
        for (int q = 0; q < RPT; ++q)
#pragma unroll
            for (int v = 0; v < VEC; ++v) a1[q][v] = a2[q][v] = 0.0;
        // one round: BATCH images, one LDS tile each; the loads of the next round are issued
        // before this round goes through LDS, so two rounds of loads are in flight
        auto load_round = [&](int nb, VecT<T, VEC>(&x)[BATCH][RPT]) {
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                const int n = nb + j < n1 ? nb + j : n1 - 1;   // past the range: re-read a row, ignored
#pragma unroll
                for (int q = 0; q < RPT; ++q) {
                    const T *p = src[q] + (long long)n * g.CHW;
                    if (vec_d) {
                        // an aligned vector that overlaps the tile's part of the row lies inside D
                        x[j][q].q = rel[q] < pend ? *reinterpret_cast<const uint4 *>(p) : make_uint4(0, 0, 0, 0);
                    } else {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) x[j][q].e[v] = rel[q] + v < pend ? p[v] : T(0);
                    }
                }
            }
        };
        auto do_round = [&](int nb, VecT<T, VEC>(&x)[BATCH][RPT]) {
            __syncthreads();   // the previous round's tiles are read
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                if (nb + j >= n1) break;
#pragma unroll
                for (int q = 0; q < RPT; ++q) {
                    if constexpr (ENC) {
                        const double wgt = (double)(nb + j + g.wbase);
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            const double xv = widen(x[j][q].e[v]);
                            a1[q][v] += xv;
                            a2[q][v] = fma(wgt, xv, a2[q][v]);
                        }
                    }
                    uint32_t *row = reinterpret_cast<uint32_t *>(&tile[j][cr + 32 * q][vq * VEC]);
                    row[0] = x[j][q].q.x;
                    row[1] = x[j][q].q.y;
                    row[2] = x[j][q].q.z;
                    row[3] = x[j][q].q.w;
                }
            }
            __syncthreads();
            if constexpr (SPLIT) {
                // eight channels of one position a thread, two images at a time
                static_assert(TC == 32 && TH <= 32 && kThreads == 256 && BATCH % 2 == 0, "split store roles");
                const int cq = threadIdx.x & 3, hp = (threadIdx.x >> 2) & 31, jo = threadIdx.x >> 7;
                uint16_t *out = reinterpret_cast<uint16_t *>(Dt);
#pragma unroll
                for (int j = 0; j < BATCH; j += 2) {
                    const int n = nb + j + jo;
                    if (n >= n1 || hp >= TH || p0 + hp >= HW) continue;
                    float x8[8];
#pragma unroll
                    for (int v = 0; v < 8; ++v) x8[v] = kSplitScale * tile[j + jo][cq * 8 + v][hp + sv[v % VEC]];
                    store_split8<32>(x8, out + (((long long)n * HW + p0 + hp) * g.C + ct * TC) * 3 + cq * 8);
                }
                return;
            }
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                if (nb + j >= n1) break;
#pragma unroll
                for (int h = hs; h < TH; h += HS) {
                    if (p0 + h >= HW) break;
                    VecT<T, VEC> y;
#pragma unroll
                    for (int v = 0; v < VEC; ++v) y.e[v] = tile[j][cg * VEC + v][h + sv[v]];
                    *reinterpret_cast<uint4 *>(Dt + ((long long)(nb + j) * HW + p0 + h) * g.C + ct * TC + cg * VEC) = y.q;
                }
            }
        };
        VecT<T, VEC> xa[BATCH][RPT], xb[BATCH][RPT];
        if (n0 < n1) load_round(n0, xa);
        for (int nb = n0; nb < n1; nb += 2 * BATCH) {
            if (nb + BATCH < n1) load_round(nb + BATCH, xb);
            do_round(nb, xa);
            if (nb + BATCH >= n1) break;
            if (nb + 2 * BATCH < n1) load_round(nb + 2 * BATCH, xa);
            do_round(nb + BATCH, xb);
        }
        if constexpr (ENC) {
            // element v of the thread's vector is position rel + v of its row; each position of the
            // tile is in exactly one vector of the row
            double *o1 = cd1, *o2 = cd2;
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const long long row = (long long)(ct * TC + cr + 32 * q) * HW;
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    const int p = rel[q] + v;
                    if (p >= p0 && p < pend) {
                        o1[row + p] = a1[q][v];
                        o2[row + p] = a2[q][v];
                    }
                }
            }
        }
        return;
    }
    // weights: one workgroup per filter m; its [C][R*S] row goes through LDS in channel chunks
    // (whole-vector loads of W) and comes out as [R*S][C] (vectors of VEC channels written to Wt)
    const int m = b - tr_blocks;
    if (m >= g.M) return;
    if (m == 0 && threadIdx.x < 16) zero16[threadIdx.x] = make_uint4(0, 0, 0, 0);
    // the convolution's stream-K arrival counts, spread over the weight workgroups
    for (int i = m * kThreads + threadIdx.x; i < skcnt_n; i += g.M * kThreads) skcnt[i] = 0;
    T *stage = &tile[0][0][0];
    const int RS = g.R * g.S;
    const T *wm = W + (long long)m * g.K;
    T *wtm = Wt + (long long)m * g.K;
    constexpr int CG = SPLIT ? 8 : VEC;   // channels stored as one unit
    if (vec_w && CG * RS <= P::LDS_ELEMS) {
        // chunks of a multiple of CG channels: every chunk starts on a vector of W and of Wt
        int cch = (P::LDS_ELEMS / RS) / CG * CG;
        cch = cch > g.C ? g.C : cch;
        for (int c0 = 0; c0 < g.C; c0 += cch) {
            const int nc = cch < g.C - c0 ? cch : g.C - c0;
            const int nvec = nc * RS / VEC;
            const uint4 *wv = reinterpret_cast<const uint4 *>(wm + (long long)c0 * RS);
            __syncthreads();
            for (int i0 = 0; i0 < nvec; i0 += 4 * kThreads) {
                uint4 x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u * kThreads + threadIdx.x;
                    x[u] = i < nvec ? wv[i] : make_uint4(0, 0, 0, 0);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u * kThreads + threadIdx.x;
                    if (i < nvec) *reinterpret_cast<uint4 *>(stage + (long long)i * VEC) = x[u];
                }
            }
            __syncthreads();
            if constexpr (SPLIT) {
                // C and the chunk are multiples of 8 channels
                const int c8_n = nc / 8;
                uint16_t *out = reinterpret_cast<uint16_t *>(Wt) + (long long)m * g.K * 3;
                for (int o = threadIdx.x; o < RS * c8_n; o += kThreads) {
                    const int rs = o / c8_n, cl = (o - rs * c8_n) * 8, c = c0 + cl;
                    float x8[8];
#pragma unroll
                    for (int v = 0; v < 8; ++v) x8[v] = split_weight_scale(m, c / 8) * stage[(cl + v) * RS + rs];
                    store_split8<32>(x8, out + ((long long)rs * g.C + c / 32 * 32) * 3 + c % 32);
                }
                continue;
            }
            const int cv_n = nc / VEC;
            for (int o = threadIdx.x; o < nvec; o += kThreads) {
                const int rs = o / cv_n, cv = o - (o / cv_n) * cv_n;
                VecT<T, VEC> y;
#pragma unroll
                for (int v = 0; v < VEC; ++v) y.e[v] = stage[(cv * VEC + v) * RS + rs];
                *reinterpret_cast<uint4 *>(wtm + (long long)rs * g.C + c0 + cv * VEC) = y.q;
            }
        }
        return;
    }
    const int cch = P::LDS_ELEMS / RS < g.C ? (P::LDS_ELEMS / RS > 0 ? P::LDS_ELEMS / RS : 1) : g.C;
    for (int c0 = 0; c0 < g.C; c0 += cch) {
        const int nc = cch < g.C - c0 ? cch : g.C - c0;
        __syncthreads();
        for (int e = threadIdx.x; e < nc * RS; e += kThreads) stage[e] = wm[(long long)c0 * RS + e];
        __syncthreads();
        for (int e = threadIdx.x; e < nc * RS; e += kThreads) {
            const int rs = e / nc, c = e - (e / nc) * nc;
            if constexpr (SPLIT) {
                const float x = split_weight_scale(m, (c0 + c) / 8) * stage[c * RS + rs];
                const uint16_t hi = f32_to_bf16_rne(x);
                const float r1 = x - bf16_bits_to_f32(hi);
                const uint16_t mi = f32_to_bf16_rne(r1);
                uint16_t *dst = reinterpret_cast<uint16_t *>(Wt) + (long long)m * g.K * 3 +
                                ((long long)rs * g.C + (c0 + c) / 32 * 32) * 3 + (c0 + c) % 32;
                dst[0] = hi;
                dst[32] = mi;
                dst[64] = f32_to_bf16_rne(r1 - bf16_bits_to_f32(mi));
            } else {
                wtm[(long long)rs * g.C + c0 + c] = stage[c * RS + rs];
            }
        }
    }
}

template <typename T, int TC, bool SHIFT, bool SPLIT>
hipError_t run_tc(const Plan &pl, const void *D, const void *W, double *cd1, double *cd2, void *ws, hipStream_t st) {
    using P = PrepT<T, TC, SHIFT>;
    const Geom &g = pl.g;
    char *w = static_cast<char *>(ws);
    T *Dt = reinterpret_cast<T *>(w + pl.off_dt);
    T *Wt = reinterpret_cast<T *>(w + pl.off_wt);
    uint4 *zero16 = reinterpret_cast<uint4 *>(w + pl.off_zero);
    int *skcnt = reinterpret_cast<int *>(w + pl.off_skcnt);
    if (pl.sk_counters > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    const int skcnt_n = (int)pl.sk_counters;
    const long long HW = (long long)g.H * g.W;
    const long long hw_tiles = (HW + P::TH - 1) / P::TH, c_tiles = g.C / TC;
    // without the encode in the copying workgroups every round of images is a workgroup of its own
    const bool apart = cd1 && pl.enc_apart;
    const int ns = cd1 && !apart ? 1 : (g.N + P::BATCH - 1) / P::BATCH;
    const int enc_vec = reinterpret_cast<uintptr_t>(D) % (kEncVec * sizeof(T)) == 0;
    const long long per = (long long)kThreads * (enc_vec ? kEncVec : 1);
    const long long enc_blocks = apart ? (g.CHW + per - 1) / per : 0;
    // Ch*H*W and K are multiples of 32 on these layers, so aligned bases keep every vector aligned
    const int vec_d = reinterpret_cast<uintptr_t>(D) % 16 == 0;
    const int vec_w = reinterpret_cast<uintptr_t>(W) % 16 == 0;
    const long long tr = (long long)ns * c_tiles * hw_tiles;
    const long long grid = enc_blocks + tr + g.M;
    if (grid > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    if (cd1 && !apart)
        prep_kernel<T, true, TC, SHIFT, SPLIT><<<(unsigned)grid, kThreads, 0, st>>>(
            static_cast<const T *>(D), static_cast<const T *>(W), Dt, Wt, g, cd1, cd2, (int)tr, (int)hw_tiles,
            (int)c_tiles, ns, vec_d, vec_w, zero16, skcnt, skcnt_n, 0, 0);
    else
        prep_kernel<T, false, TC, SHIFT, SPLIT><<<(unsigned)grid, kThreads, 0, st>>>(
            static_cast<const T *>(D), static_cast<const T *>(W), Dt, Wt, g, cd1, cd2, (int)tr,
            (int)hw_tiles, (int)c_tiles, ns, vec_d, vec_w, zero16, skcnt, skcnt_n, (int)enc_blocks, enc_vec);
    return hipGetLastError();
}

template <typename T, int TC, bool SPLIT = false>
hipError_t run_shift(const Plan &pl, const void *D, const void *W, double *cd1, double *cd2, void *ws,
                     hipStream_t st) {
    if (((long long)pl.g.H * pl.g.W) % (16 / sizeof(T)) == 0) return run_tc<T, TC, false, SPLIT>(pl, D, W, cd1, cd2, ws, st);
    return run_tc<T, TC, true, SPLIT>(pl, D, W, cd1, cd2, ws, st);
}

// The copies of a packed layer (Geom::pk): a thread a group of eight values.  D: 32 columns by eight
// groups a workgroup (prun: 256 groups of a row run), so that the lines it writes are whole and its
// loads of a channel run along the row; W: a workgroup a filter; then enc_blocks workgroups that encode
// Cd1, Cd2 (they read D beside the others).
template <typename T>
__global__ __launch_bounds__(kThreads) void pack_kernel(const T *__restrict__ D, const T *__restrict__ W,
                                                        uint16_t *__restrict__ Dt, uint16_t *__restrict__ Wt, Geom g,
                                                        int d_blocks, int pos_blocks, int enc_blocks, int enc_vec,
                                                        double *cd1, double *cd2, uint4 *__restrict__ zero16) {
    constexpr int NP = sizeof(T) == 4 ? 3 : 1;
    auto put = [&](const T (&x)[8], float scale, uint16_t *dst) {
        if constexpr (NP == 3) {
            float y[8];
#pragma unroll
            for (int v = 0; v < 8; ++v) y[v] = scale * x[v];
            store_split8<8>(y, dst);   // packed copies: groups of eight channels, plane after plane
        } else {
            VecT<uint16_t, 8> y;
#pragma unroll
            for (int v = 0; v < 8; ++v) y.e[v] = x[v];
            *reinterpret_cast<uint4 *>(dst) = y.q;
        }
    };
    int b = blockIdx.x;
    const int t = threadIdx.x;
    // the encode first: its workgroups walk all images
    if (b < enc_blocks) {
        if (enc_vec) encode_block<T, kThreads, kEncVec>(D, g, b, cd1, cd2);
        else encode_block<T, kThreads, 1>(D, g, b, cd1, cd2);
        return;
    }
    b -= enc_blocks;
    T x[8];
    if (b < d_blocks) {
        if (g.prun) {
            const int upr = g.pw * g.pcs / 8;                    // groups of a row
            const long long i = (long long)b * kThreads + t, rows = (long long)g.N * g.H;
            if (i >= rows * upr) return;
            const long long row = i / upr;                       // n H + h
            const int u = (int)(i - row * upr), n = (int)(row / g.H), h = (int)(row - (long long)n * g.H);
            const int col0 = u * 8 / g.pcs - g.P;
            const T *src = D + n * g.CHW + (long long)h * g.W;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const int c = v & (g.pcs - 1), col = col0 + v / g.pcs;   // pcs is 4 or 8
                const bool ok = c < g.C && (unsigned)col < (unsigned)g.W;
                const T val = src[ok ? (long long)c * g.H * g.W + col : 0];
                x[v] = ok ? val : T(0);
            }
            put(x, kSplitScale, Dt + i * 8 * NP);
            return;
        }
        const int HW = g.H * g.W;
        const int pb = b % pos_blocks, ub = b / pos_blocks;
        const long long pos = (long long)pb * 32 + (t & 31), all = (long long)g.N * HW;
        const int u = ub * 8 + (t >> 5);
        if (pos >= all || u >= g.pupt) return;
        const int n = (int)(pos / HW), q = (int)(pos - (long long)n * HW);
        const T *src = D + n * g.CHW + q;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int c = u * 8 + v;
            const T val = src[c < g.C ? (long long)c * HW : 0];
            x[v] = c < g.C ? val : T(0);
        }
        put(x, kSplitScale, Dt + (pos * g.pcs + u * 8) * NP);
        return;
    }
    const int m = b - d_blocks;
    if (m == 0 && t < 16) zero16[t] = make_uint4(0, 0, 0, 0);
    const int p_s = g.prun ? 1 : g.S, taps = g.R * p_s;
    const T *wm = W + (long long)m * g.K;
    for (int i = t; i < g.pkk / 8; i += kThreads) {
        const int tap = i / g.pupt, o = i - tap * g.pupt, r = tap / p_s;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int e = o * 8 + v;                             // value of the tap's run
            const int c = g.prun ? e & (g.pcs - 1) : e, s = g.prun ? e / g.pcs : tap - r * p_s;
            const bool ok = tap < taps && c < g.C && s < g.S;
            const T val = wm[ok ? ((long long)c * g.R + r) * g.S + s : 0];
            x[v] = ok ? val : T(0);
        }
        put(x, split_weight_scale(m, i), Wt + ((long long)m * g.pkk + i * 8) * NP);
    }
}

template <typename T>
hipError_t run_pack(const Plan &pl, const void *D, const void *W, double *cd1, double *cd2, void *ws, hipStream_t st) {
    const Geom &g = pl.g;
    char *w = static_cast<char *>(ws);
    const long long all = (long long)g.N * g.H * g.W;
    const long long pos_blocks = (all + 31) / 32;
    const long long d_blocks = g.prun ? ((long long)g.N * g.H * (g.pw * g.pcs / 8) + kThreads - 1) / kThreads
                                      : pos_blocks * ((g.pupt + 7) / 8);
    const int enc_vec = g.CHW % kEncVec == 0 && reinterpret_cast<uintptr_t>(D) % (kEncVec * sizeof(T)) == 0;
    const long long per = (long long)kThreads * (enc_vec ? kEncVec : 1);
    const long long enc_blocks = cd1 ? (g.CHW + per - 1) / per : 0;
    if (enc_blocks + d_blocks + g.M > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    pack_kernel<T><<<(unsigned)(enc_blocks + d_blocks + g.M), kThreads, 0, st>>>(
        static_cast<const T *>(D), static_cast<const T *>(W), reinterpret_cast<uint16_t *>(w + pl.off_dt),
        reinterpret_cast<uint16_t *>(w + pl.off_wt), g, (int)d_blocks, (int)pos_blocks,
        (int)enc_blocks, enc_vec, cd1, cd2, reinterpret_cast<uint4 *>(w + pl.off_zero));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_pack(const Plan &pl, const void *D, const void *W, double *cd1, double *cd2, void *ws,
                       hipStream_t st) {
    return pl.g.dtype == FTCNN_F32 ? run_pack<float>(pl, D, W, cd1, cd2, ws, st)
                                   : run_pack<uint16_t>(pl, D, W, cd1, cd2, ws, st);
}

hipError_t launch_prep(const Plan &pl, const void *D, const void *W, double *cd1, double *cd2, void *ws,
                       hipStream_t st) {
    if (pl.g.split) return run_shift<float, 32, true>(pl, D, W, cd1, cd2, ws, st);
    if (pl.g.dtype == FTCNN_F32) return run_shift<float, 32>(pl, D, W, cd1, cd2, ws, st);
    if (prep_tile_channels(pl.g) == 64) return run_shift<uint16_t, 64>(pl, D, W, cd1, cd2, ws, st);
    return run_shift<uint16_t, 32>(pl, D, W, cd1, cd2, ws, st);
}

}  // namespace ftcnn
