// rmsnorm.hip -- RMSNorm over the feature axis of (batch, dim, seqlen) activations,
// forward and backward, for the packed Mamba block.  RMSNorm is token-wise, so
// packing leaves it unchanged (§3.2); it is here so that every step of the block
// runs in this library's kernels or in plain GEMMs.
//
// A block owns a tile of consecutive tokens of one batch row: GROUPS lanes side by side,
// each with one 16-byte vector of tokens, so that every feature row gives GROUPS x 16
// contiguous bytes, and THREADS / GROUPS slices of the features.  A thread keeps the
// vectors of its first KEPT features in registers from the sum over the features to the
// second sweep; features beyond those are read again.
// Bound by HBM where there are tiles enough for the GPU.  Us, forward and backward, against
// 1024 threads that keep nothing and 8 tokens per lane in both types:
//   8 x 4096 x 2048 bf16 (67 M elements)  49, 133   before 60, 165
//   8 x 4096 x 2048 fp32                  96, 257   before 166, 349
//   2 x 3001 x 2560 bf16                  44,  87   before 134, 273
#include "common.hpp"
#include "launch.hpp"

namespace pm {
namespace {

constexpr int64_t kCus = 256;

// Forward: (batch row) x (tiles per row) + tile of this block.  Blocks go to the 8 XCDs in
// turn; with 64-byte rows of a tile, the two tiles that share 128-byte lines go to the same one.
template <int GROUPS>
__device__ __forceinline__ int64_t tile_id() {
    const int64_t id = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t g = id / 16 * 16, r = id - g;
    if (GROUPS >= 8 || g + 16 > (int64_t)gridDim.x * gridDim.y) return id;
    return g + (r % 8) * 2 + r / 8;
}

template <int GROUPS, int THREADS, int TOK>
struct __attribute__((aligned(16))) RmsSmem {
    static constexpr int kSlices = THREADS / GROUPS, kTile = GROUPS * TOK;
    static constexpr int kParts = THREADS / kTile;       // first-level sums of each token
    float red[kSlices][kTile];   // per-slice values of each token
    float part[kParts][kTile];
    float tot[kTile];            // their sums
};

// Sum over the slices of each token's per-slice value, in a fixed order; every thread gets
// its own tokens' totals.
template <int GROUPS, int THREADS, int TOK>
__device__ __forceinline__ void slice_sum(float (&v)[TOK], RmsSmem<GROUPS, THREADS, TOK>& sm, int sl, int grp) {
    using S = RmsSmem<GROUPS, THREADS, TOK>;
#pragma unroll
    for (int k = 0; k < TOK; k += 4)
        *reinterpret_cast<f32x4*>(&sm.red[sl][grp * TOK + k]) = f32x4{v[k], v[k + 1], v[k + 2], v[k + 3]};
    __syncthreads();
    constexpr int kPer = S::kSlices / S::kParts;
    const int tok = threadIdx.x % S::kTile, q = threadIdx.x / S::kTile;
    float a = sm.red[q * kPer][tok];
#pragma unroll
    for (int i = 1; i < kPer; ++i) a += sm.red[q * kPer + i][tok];
    sm.part[q][tok] = a;
    __syncthreads();
    if (threadIdx.x < S::kTile) {
        a = sm.part[0][tok];
#pragma unroll
        for (int i = 1; i < S::kParts; ++i) a += sm.part[i][tok];
        sm.tot[tok] = a;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TOK; k += 4) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(&sm.tot[grp * TOK + k]);
        v[k] = t.x; v[k + 1] = t.y; v[k + 2] = t.z; v[k + 3] = t.w;
    }
}

template <typename T, typename TO, int GROUPS, int THREADS, int KEPT>
__global__ __launch_bounds__(THREADS) void rmsnorm_fwd_kernel(const T* __restrict__ x, const float* __restrict__ w,
                                                              float eps, TO* __restrict__ out,
                                                              float* __restrict__ rstd, int64_t dim, int64_t L) {
    constexpr int TOK = Storage<T>::kPerVec;
    using Smem = RmsSmem<GROUPS, THREADS, TOK>;
    constexpr int SL = Smem::kSlices;
    __shared__ Smem sm;
    const int grp = threadIdx.x % GROUPS, sl = threadIdx.x / GROUPS;
    const int64_t id = tile_id<GROUPS>();
    const int64_t b = id / gridDim.x;
    const int64_t t0 = (id - b * gridDim.x) * Smem::kTile;
    const bool whole = t0 + Smem::kTile <= L || L % TOK == 0;      // no vector crosses the row end
    const bool live = t0 + grp * TOK < L;
    const int64_t l0 = whole && !live ? t0 : t0 + grp * TOK;
    const T* xb = x + b * dim * L;
    TO* ob = out + b * dim * L;
    // FULL (block-uniform): no vector crosses the row end; lanes past it repeat the tile's
    // first and store nothing
    const auto body = [&](auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        constexpr int C = FULL ? KEPT : 0;                      // features kept in registers
        const int64_t lane = sl * L + l0;                    // this lane's vector of feature sl
        RawRun<T, TOK> xr[KEPT];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            xr[i] = RawRun<T, TOK>{};
            if (sl + i * SL < dim) xr[i] = load_raw<T, TOK>(xb + i * SL * L + lane, 0);
        }
        float s[TOK] = {};
        const auto square = [&](const float (&v)[TOK]) {
#pragma unroll
            for (int k = 0; k < TOK; ++k) s[k] = fmaf(v[k], v[k], s[k]);
        };
#pragma unroll
        for (int i = 0; i < C; ++i) {
            float v[TOK];
            unpack_run(xr[i], v);
            square(v);
        }
        for (int64_t f = sl + C * SL; f < dim; f += SL) {
            float v[TOK];
            load_run<T, TOK, FULL>(xb + f * L, l0, L, v);
            square(v);
        }
        slice_sum(s, sm, sl, grp);
        float r[TOK];
#pragma unroll
        for (int k = 0; k < TOK; ++k) r[k] = 1.0f / sqrtf(s[k] / (float)dim + eps);
        if (sl == 0) {
#pragma unroll
            for (int k = 0; k < TOK; ++k)
                if (FULL ? live : l0 + k < L) rstd[b * L + l0 + k] = r[k];
        }
        const auto scale = [&](float (&v)[TOK], int64_t fb) {      // feature fb + sl
            const int64_t f = fb + sl;
            const float wv = w[f];
#pragma unroll
            for (int k = 0; k < TOK; ++k) v[k] = v[k] * r[k] * wv;
            if constexpr (FULL) { if (live) store_run<TO, TOK, true>(ob + fb * L + lane, 0, L, v); }
            else store_run<TO, TOK>(ob + f * L, l0, L, v);
        };
#pragma unroll
        for (int i = 0; i < C; ++i) {
            float v[TOK];
            unpack_run(xr[i], v);
            if (sl + i * SL < dim) scale(v, i * SL);
        }
        for (int64_t f = sl + C * SL; f < dim; f += SL) {
            float v[TOK];
            load_run<T, TOK, FULL>(xb + f * L, l0, L, v);
            scale(v, f - sl);
        }
    };
    if (whole) body(std::true_type{});
    else body(std::false_type{});
}

// dx = r (dh w - x r^2 s / dim) (+ dres), s = sum_f dh w x at each token;
// partial[b, tile, f] = sum over the tile's tokens of dh x r.
// A tile is 64 tokens: one partial row per 64 tokens is what the workspace holds, whatever the
// launch.  Where that leaves CUs idle, gridDim.z blocks (a power of two) share a tile: each
// sums over all features and writes the gradients of its part of them, every gridDim.z-th of
// a slice's.  The sum's loads are repeated, from the XCD's L2 that the blocks of a tile share.
// One block a tile where dx takes the place of x or dh, which the others would still read.
template <typename T, typename TO, int THREADS, int KEPT>
__global__ __launch_bounds__(THREADS) void rmsnorm_bwd_kernel(
    const T* __restrict__ x, const float* __restrict__ w, const float* __restrict__ rstd,
    const T* __restrict__ dh, const T* __restrict__ dres, TO* __restrict__ dx,
    float* __restrict__ partial, int64_t dim, int64_t L) {
    constexpr int TOK = Storage<T>::kPerVec, GROUPS = kRmsTile / TOK;
    using Smem = RmsSmem<GROUPS, THREADS, TOK>;
    constexpr int SL = Smem::kSlices;
    __shared__ Smem sm;
    const int grp = threadIdx.x % GROUPS, sl = threadIdx.x / GROUPS;
    // blocks go to the 8 XCDs in turn: the parts of a tile are 8 blocks apart
    const int64_t tiles = (int64_t)gridDim.x * gridDim.y;
    const int64_t blk = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const int parts = (int)gridDim.z, parts_log2 = __builtin_ctz(gridDim.z);
    const int64_t first = blk / (8 * parts) * 8;
    const int in = (int)(blk - first * parts), wide = (int)min(tiles - first, (int64_t)8);
    const int64_t id = first + in % wide;
    const int part = in / wide;
    const int64_t b = id / gridDim.x;
    const int64_t t0 = (id - b * gridDim.x) * Smem::kTile;
    const bool whole = t0 + Smem::kTile <= L || L % TOK == 0;      // as in the forward
    const bool live = t0 + grp * TOK < L;
    const int64_t l0 = whole && !live ? t0 : t0 + grp * TOK;
    const int64_t off = b * dim * L;
    const T* xb = x + off;
    const T* gb = dh + off;
    float* pb = partial + id * dim;
    const auto body = [&](auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        constexpr int C = FULL ? KEPT : 0;                      // features kept in registers
        const int64_t lane = sl * L + l0;                    // this lane's vector of feature sl
        const int64_t own = (int64_t)part * SL, step = (int64_t)parts * SL;   // the block's features: sl + own + i step
        RawRun<T, TOK> xr[KEPT], gr[KEPT];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            xr[i] = gr[i] = RawRun<T, TOK>{};
            const int64_t fb = own + i * step;
            if (sl + fb < dim) {
                xr[i] = load_raw<T, TOK>(xb + fb * L + lane, 0);
                gr[i] = load_raw<T, TOK>(gb + fb * L + lane, 0);
            }
        }
        float s[TOK] = {};
        const auto dot = [&](const float (&xv)[TOK], const float (&gv)[TOK], float wv) {
#pragma unroll
            for (int k = 0; k < TOK; ++k) s[k] = fmaf(gv[k] * wv, xv[k], s[k]);
        };
#pragma unroll
        for (int i = 0; i < C; ++i) {
            float xv[TOK], gv[TOK];
            unpack_run(xr[i], xv);
            unpack_run(gr[i], gv);
            const int64_t f = sl + own + i * step;
            if (f < dim) dot(xv, gv, w[f]);
        }
        const auto sweep = [&](int64_t f) {
            float xv[TOK], gv[TOK];
            load_run<T, TOK, FULL>(xb + f * L, l0, L, xv);
            load_run<T, TOK, FULL>(gb + f * L, l0, L, gv);
            dot(xv, gv, w[f]);
        };
        if (parts == 1) {
            for (int64_t f = sl + C * SL; f < dim; f += SL) sweep(f);
        } else {
            int i = 0;
            for (int64_t f = sl; f < dim; f += SL, ++i)
                if ((i & (parts - 1)) != part || (i >> parts_log2) >= C) sweep(f);
        }
        float r[TOK], c[TOK];
#pragma unroll
        for (int k = 0; k < TOK; ++k) r[k] = (FULL || l0 + k < L) ? rstd[b * L + l0 + k] : 0.0f;
        slice_sum(s, sm, sl, grp);
#pragma unroll
        for (int k = 0; k < TOK; ++k) c[k] = r[k] * r[k] * s[k] / (float)dim;
        const auto grad = [&](const float (&xv)[TOK], const float (&gv)[TOK], int64_t fb) {      // feature fb + sl
            const int64_t f = fb + sl;
            float o[TOK], pw = 0.0f;
            if (dres) {
                if constexpr (FULL) load_run<T, TOK, true>(dres + off + fb * L + lane, 0, L, o);
                else load_run<T, TOK>(dres + off + f * L, l0, L, o);
            }
            const float wv = w[f];
#pragma unroll
            for (int k = 0; k < TOK; ++k) {
                const float v = r[k] * (gv[k] * wv - xv[k] * c[k]);
                o[k] = dres ? o[k] + v : v;
                pw = fmaf(gv[k] * xv[k], r[k], pw);      // 0 past the row end: loads read 0
            }
            if (FULL && !live) pw = 0.0f;
            if constexpr (FULL) { if (live) store_run<TO, TOK, true>(dx + off + fb * L + lane, 0, L, o); }
            else store_run<TO, TOK>(dx + off + f * L, l0, L, o);
            // over the groups of the slice (consecutive lanes), in a fixed order
#pragma unroll
            for (int m = 1; m < GROUPS; m *= 2) pw += __shfl_xor(pw, m, GROUPS);
            if (grp == 0) pb[f] = pw;
        };
#pragma unroll
        for (int i = 0; i < C; ++i) {
            float xv[TOK], gv[TOK];
            unpack_run(xr[i], xv);
            unpack_run(gr[i], gv);
            const int64_t fb = own + i * step;
            if (sl + fb < dim) grad(xv, gv, fb);
        }
        for (int64_t f = sl + own + C * step; f < dim; f += step) {
            float xv[TOK], gv[TOK];
            load_run<T, TOK, FULL>(xb + f * L, l0, L, xv);
            load_run<T, TOK, FULL>(gb + f * L, l0, L, gv);
            grad(xv, gv, f - sl);
        }
    };
    if (whole) body(std::true_type{});
    else body(std::false_type{});
}

// dw[f] = sum over the (batch, tile) rows of partial[., f], in a fixed order: a block owns
// 32 features (128 bytes of each row), each of its 32 row groups sums every 32nd row, eight
// loads in flight, and the groups' sums are added in order.  One launch in place of two
// (slabs, then slabs' sums), 5 us less; a thread per feature chained 512 loads (156 us at
// the Mamba-1.4B block's shape).
constexpr int kFinFeat = 32, kFinRows = 32;
__global__ __launch_bounds__(kFinFeat * kFinRows) void rmsnorm_bwd_finalize(const float* __restrict__ partial,
                                                                          float* __restrict__ dw, int64_t rows,
                                                                          int64_t dim) {
    __shared__ float part[kFinRows][kFinFeat];
    const int fo = threadIdx.x % kFinFeat, rg = threadIdx.x / kFinFeat;
    const int64_t f = (int64_t)blockIdx.x * kFinFeat + fo;
    float a = 0.0f;
    if (f < dim) {
        int64_t i = rg;
        for (; i + 7 * kFinRows < rows; i += 8 * kFinRows) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = partial[(i + q * kFinRows) * dim + f];
#pragma unroll
            for (int q = 0; q < 8; ++q) a += v[q];
        }
        for (; i < rows; i += kFinRows) a += partial[i * dim + f];
    }
    part[rg][fo] = a;
    __syncthreads();
    if (rg == 0 && f < dim) {
#pragma unroll
        for (int q = 1; q < kFinRows; ++q) a += part[q][fo];
        dw[f] = a;
    }
}

template <typename T, typename TO, int GROUPS, int THREADS, int KEPT>
hipError_t fwd_g(const RmsArgs& a, hipStream_t s) {
    constexpr int64_t kTile = GROUPS * Storage<T>::kPerVec;
    hipLaunchKernelGGL((rmsnorm_fwd_kernel<T, TO, GROUPS, THREADS, KEPT>),
                       dim3((unsigned)((a.seqlen + kTile - 1) / kTile), (unsigned)a.batch), dim3(THREADS), 0, s,
                       static_cast<const T*>(a.x), a.w, a.eps, static_cast<TO*>(a.out), a.rstd_out, a.dim, a.seqlen);
    return hipGetLastError();
}

// 8 groups where tiles of 8 give each CU a block, else 4 (us, 8 and 4 groups, bf16: 256 tiles
// of 8, 4 x 4096 x 768: 8.1, 11.5; 8 x 2048 x 2048: 26.7, 30.1; 128 tiles, 8 x 1024 x 2048:
// 14.8, 13.7; 32 tiles, 1 x 2048 x 4096: 19.8, 12.6).  1024 threads; fewer where most slices
// would have few features or none: up to 256 of them 512 threads (16 x 4096 x 256: bf16 10.4
// against 12.5 with 256, fp32 20.9 against 26) and 256 up to 128 (16 x 8192 x 128 bf16: 10.6
// against 15.5 with 512 and 33 with 1024) and in narrow tiles (1 x 4096 x 32: 3.1 against 5.6);
// in bf16 also up to 512 (5 x 2816 x 512: 7.1 against 11.5; 8 x 4096 x 384 7.9, 11.4; 1 x 2048 x
// 300 4.1, 5.9; fp32 64 x 256 x 512 11.4, 9.9).
// Rows that end inside a 64-byte piece of a line share their lines between tiles, which go to
// different XCDs: tiles of 64 tokens from 96 of them on in bf16, in fp32, whose 64 tokens are two
// lines, from 64 (us, against the other tiles: bf16 96 tiles, 6 x 1000 x 2048 25.0, 27.4; 94,
// 2 x 3001 x 2560 47.6, 44.6; fp32 84, 21 x 216 x 5120 71.6, 92.4; 64, 4 x 1000 x 2048 28.8, 28.6;
// up to 256 features 20 x 12712 x 256: bf16 76 against 105, fp32 111 against 162).
// Eight kept features leave a CU one block of 1024 threads in bf16, four two: four where tiles
// just over one round leave the second nearly empty (270 tiles, 30 x 576 x 2560: 44.5 against
// 49.4; x 1024 15.1, 19.2; 320 tiles, 40 x 512 x 2560 50.6, 50.8; 352 52.6, 51.9), in narrow tiles
// up to 2048 features (264, 33 x 256 x 768 9.1, 11.7; 384, 12 x 1024 x 2048 21.9, 24.7; x 4096 51.5,
// 47.2), or where the kept four are all (8 x 1024 x 768 6.7, 7.1).
constexpr int kSmallDim = 256;

template <typename T, typename TO>
hipError_t fwd_t(const RmsArgs& a, hipStream_t s) {
    constexpr bool kBf16 = Storage<T>::kPerVec == 8;
    constexpr int64_t kTile = 8 * Storage<T>::kPerVec;
    constexpr int kG64 = 64 / Storage<T>::kPerVec;               // groups of a tile of 64 tokens
    const bool wide = a.batch * ((a.seqlen + kTile - 1) / kTile) >= kCus;
    const bool split_lines = a.seqlen * (int64_t)sizeof(T) % 64 != 0;
    const int64_t tiles64 = a.batch * ((a.seqlen + 63) / 64);
    const bool by64 = split_lines && tiles64 >= (kBf16 ? kCus * 3 / 8 : kCus / 4);
    if (a.dim <= kSmallDim) {
        if (!wide) return fwd_g<T, TO, 4, 256, 4>(a, s);
        if (split_lines) return fwd_g<T, TO, kG64, 512, 8>(a, s);
        return a.dim <= kSmallDim / 2 ? fwd_g<T, TO, 8, 256, 4>(a, s) : fwd_g<T, TO, 8, 512, 4>(a, s);
    }
    if constexpr (kBf16) {
        if (a.dim <= 2 * kSmallDim && !by64)
            return wide ? fwd_g<T, TO, 8, 512, 8>(a, s) : fwd_g<T, TO, 4, 512, 4>(a, s);
        if (a.dim > 2 * kSmallDim && tiles64 > kCus && tiles64 <= kCus * 5 / 4) return fwd_g<T, TO, 8, 1024, 4>(a, s);
    }
    if (by64) return fwd_g<T, TO, kG64, 1024, 8>(a, s);
    if (wide) return fwd_g<T, TO, 8, 1024, 8>(a, s);
    if constexpr (kBf16) {
        const int64_t tiles32 = a.batch * ((a.seqlen + 31) / 32);
        if (a.dim <= 1024 || (a.dim <= 2048 && tiles32 > kCus)) return fwd_g<T, TO, 4, 1024, 4>(a, s);
    }
    return fwd_g<T, TO, 4, 1024, 8>(a, s);
}

template <typename T, typename TO, int THREADS, int KEPT>
hipError_t bwd_g(const RmsArgs& a, hipStream_t s) {
    constexpr int64_t kSlices = THREADS * (int64_t)Storage<T>::kPerVec / kRmsTile;
    const int64_t row_tiles = (a.seqlen + kRmsTile - 1) / kRmsTile;
    // Blocks that share a tile: as many as leave no CU two, each with features of its own (us,
    // 1, 2, 4, 8 blocks, bf16, 32 tiles, 1 x 2048 x 4096: 57, 40, 31, 27; 64 tiles, 8 x 512 x
    // 2048: 32, 24, 21, 27; 128 tiles, 4 x 2048 x 768: 16.6, 14.8, 19.9; 256 tiles, 8 x 2048 x
    // 2048: 58, 61; fp32, 128 tiles, 8 x 1024 x 2048: 63, 61, 65).
    unsigned parts = 1;
    const bool in_place = a.out == a.x || a.out == a.dout;
    while (!in_place && parts < 8 && a.batch * row_tiles * parts * 2 <= kCus && a.dim > kSlices * parts) parts *= 2;
    hipLaunchKernelGGL((rmsnorm_bwd_kernel<T, TO, THREADS, KEPT>), dim3((unsigned)row_tiles, (unsigned)a.batch, parts),
                       dim3(THREADS), 0, s, static_cast<const T*>(a.x), a.w, a.rstd, static_cast<const T*>(a.dout),
                       static_cast<const T*>(a.dres), static_cast<TO*>(a.out), a.partial, a.dim, a.seqlen);
    if (hipError_t e = hipGetLastError()) return e;
    hipLaunchKernelGGL(rmsnorm_bwd_finalize, dim3((unsigned)((a.dim + kFinFeat - 1) / kFinFeat)),
                       dim3(kFinFeat * kFinRows), 0, s, a.partial, a.dw, a.batch * row_tiles, a.dim);
    return hipGetLastError();
}

// 1024 threads, 512 where that leaves a thread at most two features (16 x 8192 x 128: 31 us
// against 42 in bf16, 45 against 51 in fp32; 4 x 4096 x 768 bf16: 27.5 against 22.5).  At 1024
// threads a bf16 lane holds 4 features (8 spill 67 VGPRs: 160 us against 129 at 8 x 4096 x
// 2048), an fp32 lane, with half the tokens, 8 (257 against 281 there with 4).
template <typename T, typename TO>
hipError_t bwd_t(const RmsArgs& a, hipStream_t s) {
    constexpr int64_t kSlices = 1024 * (int64_t)Storage<T>::kPerVec / kRmsTile;
    if (a.dim <= 2 * kSlices) return bwd_g<T, TO, 512, 4>(a, s);
    return bwd_g<T, TO, 1024, Storage<T>::kPerVec == 8 ? 4 : 8>(a, s);
}

}  // namespace

hipError_t launch_rmsnorm_fwd(const RmsArgs& a, hipStream_t s) {
    switch (a.dtype) {
        case 1: return fwd_t<bf16_t, bf16_t>(a, s);
        case 2: return fwd_t<bf16_t, float>(a, s);
        default: return fwd_t<float, float>(a, s);
    }
}

hipError_t launch_rmsnorm_bwd(const RmsArgs& a, hipStream_t s) {
    switch (a.dtype) {
        case 1: return bwd_t<bf16_t, bf16_t>(a, s);
        case 2: return bwd_t<bf16_t, float>(a, s);
        default: return bwd_t<float, float>(a, s);
    }
}

}  // namespace pm
