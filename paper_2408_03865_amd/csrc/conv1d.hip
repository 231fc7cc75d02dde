// conv1d.hip -- packed causal depthwise conv1d, forward and backward (Alg. 1, §3.3, §3.5).
//
// HBM-bound streaming kernels.  The tap mask uses only integer compares against
// the token's position index, read with the same coalesced vector loads (§3.5):
// the forward keeps the tap reaching k tokens back iff k <= pos[l]; the
// backward's dx takes the next width-1 tokens' indices ("reverse indices") and
// keeps tap k iff pos[j+k] >= k.
//  - Forward: one wave per (tile of tokens, channels) or a block per row, described at their
//    kernels.
//  - Backward: one wave per (row, segment), described at its kernel.
#include "common.hpp"
#include "launch.hpp"

namespace pm {
namespace {

constexpr int kTok = 8;        // the halo vector of the backward and of the forward by rows
constexpr int kTokBwd = 8;     // tokens per thread per step (backward)
constexpr int kThreads = 256;
constexpr int kConvBwdParts = 16;     // most waves of one channel that the backward gathers in a block

// N position indices from l0 (N a multiple of 4); beyond L they read 0.  FULL: the
// caller guarantees l0 + N <= L
template <int N = kTok, bool FULL = false>
__device__ __forceinline__ void load_pos(const int32_t* __restrict__ pr, int64_t l0, int64_t L, int* p) {
    u32x4 a[N / 4] = {};
#pragma unroll
    for (int i = 0; i < N / 4; ++i)
        if (FULL || l0 + 4 * i + 4 <= L) a[i] = *reinterpret_cast<const u32x4_a4*>(pr + l0 + 4 * i);
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        int* q = p + 4 * i;
        q[0] = (int)a[i].x; q[1] = (int)a[i].y; q[2] = (int)a[i].z; q[3] = (int)a[i].w;
        const int64_t l = l0 + 4 * i;
        if (!FULL && l < L && l + 4 > L) {                     // the row ends inside the vector
#pragma unroll
            for (int t = 0; t < 4; ++t) q[t] = l + t < L ? pr[l + t] : 0;
        }
    }
}

// Per-row states of a sequence cut at a row end (§5): (batch*dim, W-1) arrays, or
// null.  xinit holds the W-1 inputs before the row (token -1 last), xfinal the
// row's last W-1 inputs; dxfinal and dxinit are their gradients.
template <typename T, typename TO>
struct ConvStates {
    const T* xinit;
    T* xfinal;
    const T* dxfinal;
    TO* dxinit;
};

// The W-1 tokens before the row into xs[kTok-W+1 .. kTok-1] (zeros without xinit).
template <typename T, int W>
__device__ __forceinline__ void load_row_halo(const T* __restrict__ xinit, int64_t row, float* xs) {
#pragma unroll
    for (int i = 0; i < kTok; ++i) xs[i] = 0.0f;
    if (xinit) {
#pragma unroll
        for (int t = 0; t < W - 1; ++t) xs[kTok - (W - 1) + t] = Storage<T>::load1(xinit + row * (W - 1) + t);
    }
}

// The row's last W-1 inputs, copied as stored (reaching into xinit for short rows).
template <typename T, typename TO, int W>
__device__ __forceinline__ void store_xfinal(const T* __restrict__ x, const ConvStates<T, TO>& st, int64_t row, int64_t L) {
    constexpr int H = W - 1;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const int64_t m = L - H + i;
        T v{};
        if (m >= 0) v = x[row * L + m];
        else if (st.xinit) v = st.xinit[row * H + H + m];
        st.xfinal[row * H + i] = v;
    }
}

// Forward: one wave per (tile of tokens, R channels).  Each lane owns KT consecutive
// tokens (one 16-byte vector of x), a row takes 2^lanes_log2 lanes of a wave, and a wave
// holds 64 >> lanes_log2 rows at once, so that rows shorter than a wave's span (one token
// in a decode step) fill it too; rows longer than a wave's span (LONG) are cut into tiles,
// one wave each, which then has a channel's weights in scalar registers.  The wave walks R such sets of rows of one batch row, all loads first: the
// position indices are read and their tap masks compared once for the R, and R vectors
// per lane are in flight.  The W-1 tokens before a lane's come from the lane before it by
// a lane shift, only lane 0 of a later tile reads them from memory: a pass reads x once
// and writes out once.  Bound by HBM at long rows (8 x 4096 x 4096 fp32: 182 us, 5.9 TB/s,
// against 223 us with 8 tokens a lane); one token of 64 x 4096 channels takes 4 us against 153
// with a block per row.
template <typename T, typename TO, int W, int R, bool LONG>
__global__ __launch_bounds__(kThreads) void conv1d_fwd_kernel(
    const T* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias,
    const int32_t* __restrict__ pos, TO* __restrict__ out, ConvStates<T, TO> st, int64_t dim,
    int64_t L, int silu, int lanes_log2, uint32_t ntiles, uint32_t waves) {
    constexpr int KT = Storage<T>::kPerVec;
    constexpr int H = W - 1;
    const int lane = (int)(threadIdx.x & 63);
    const uint32_t wave = blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (wave >= waves) return;
    const int64_t b = blockIdx.y;
    const uint32_t group = LONG ? wave / ntiles : wave;
    const int tile = LONG ? (int)(wave - group * ntiles) : 0;
    const int rows = LONG ? 1 : 64 >> lanes_log2;       // rows a wave holds at once
    const int vec = LONG ? lane : lane & ((1 << lanes_log2) - 1);
    const int64_t l0 = ((int64_t)tile * 64 + vec) * KT;
    const int64_t d0 = (int64_t)group * (R * rows) + (LONG ? 0 : lane >> lanes_log2);
    const int32_t* pr = pos + b * L;
    const bool first = vec == 0;

    // every load of the R rows first
    RawRun<T, KT> raw[R];
    float halo[R][H], wk[R][W], b0[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t d = d0 + r * rows;
        const int64_t row = b * dim + (d < dim ? d : dim - 1);
        const T* xr = x + row * L;
        raw[r] = RawRun<T, KT>{};
        if (l0 + KT <= L) raw[r] = load_raw<T, KT>(xr, l0);
#pragma unroll
        for (int t = 0; t < H; ++t) halo[r][t] = 0.0f;
        if (first) {
            if (tile > 0) {
                float v[4];
                unpack_run(load_raw<T, 4>(xr, l0 - 4), v);
#pragma unroll
                for (int t = 0; t < H; ++t) halo[r][t] = v[4 - H + t];
            } else if (st.xinit) {
#pragma unroll
                for (int t = 0; t < H; ++t) halo[r][t] = Storage<T>::load1(st.xinit + row * H + t);
            }
        }
#pragma unroll
        for (int k = 0; k < W; ++k) wk[r][k] = w[(row - b * dim) * W + k];
        b0[r] = bias ? bias[row - b * dim] : 0.0f;
    }
    int p[KT];
    load_pos<KT>(pr, l0, L, p);
    const bool full = LONG && ((int64_t)tile + 1) * 64 * KT <= L;
    int pmin = W - 1;                                   // lowest index of the lane's tokens inside the row
    if (full) {
#pragma unroll
        for (int t = 0; t < KT; ++t) pmin = min(pmin, p[t]);
    } else {
#pragma unroll
        for (int t = 0; t < KT; ++t) pmin = l0 + t < L ? min(pmin, p[t]) : pmin;
    }
    const bool all_live = __all(pmin >= W - 1);          // no tap of the wave is cut off

    auto channel = [&](auto live_tag, auto silu_tag, const int r) {
        constexpr bool LIVE = decltype(live_tag)::value, SILU = decltype(silu_tag)::value;
        const int64_t d = d0 + r * rows;
        const int64_t row = b * dim + (d < dim ? d : dim - 1);
        float xs[H + KT];
        unpack_run(raw[r], xs + H);
        if (l0 < L && l0 + KT > L) {                    // the row ends inside this lane's vector
#pragma unroll
            for (int t = 0; t < KT; ++t) xs[H + t] = l0 + t < L ? Storage<T>::load1(x + row * L + l0 + t) : 0.0f;
        }
#pragma unroll
        for (int t = 0; t < H; ++t) {
            const float prev = dpp<kWaveShr1>(0.0f, xs[KT + t]);     // the same token of the lane before
            xs[t] = first ? halo[r][t] : prev;
        }
        if (KT == 8) {
            // 24 masks are compared again for each channel: kept for the next, they spill from
            // the scalar registers, at two instructions a mask
#pragma unroll
            for (int t = 0; t < KT; ++t) asm volatile("" : "+v"(p[t]));
        }
        float o[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            float v = fmaf(wk[r][W - 1], xs[H + t], b0[r]);           // tap 0: position indices are >= 0
#pragma unroll
            for (int k = 1; k < W; ++k) {
                const float u = fmaf(wk[r][W - 1 - k], xs[H + t - k], v);
                v = (LIVE || k <= p[t]) ? u : v;
            }
            o[t] = SILU ? v * sigmoid_f(v) : v;
        }
        if (d >= dim) return;
        TO* orow = out + row * L;
        if (full) store_run<TO, KT, true>(orow, l0, L, o);
        else if (l0 < L) store_run<TO, KT>(orow, l0, L, o);
        if (st.xfinal && first && tile == 0) store_xfinal<T, TO, W>(x, st, row, L);
    };
    const auto channels = [&](auto live_tag, auto silu_tag) {
#pragma unroll
        for (int r = 0; r < R; ++r) channel(live_tag, silu_tag, r);
    };
    if (silu) {
        if (all_live) channels(std::true_type{}, std::true_type{});
        else channels(std::false_type{}, std::true_type{});
    } else {
        if (all_live) channels(std::true_type{}, std::false_type{});
        else channels(std::false_type{}, std::false_type{});
    }
}

// Forward of bf16 rows of a few thousand tokens, aligned to vectors (conv_fwd_by_row): a block
// per row, which it walks 2048 tokens at a time, each lane reading its vector and the one before
// it, which the lane or block before it has brought into the cache.
template <typename T, typename TO, int W>
__global__ __launch_bounds__(kThreads) void conv1d_fwd_row_kernel(
    const T* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias,
    const int32_t* __restrict__ pos, TO* __restrict__ out, ConvStates<T, TO> st, int64_t dim,
    int64_t L, int silu) {
    constexpr int KT = Storage<T>::kPerVec;
    static_assert(KT == kTok, "the halo is the vector before");
    const int64_t row = blockIdx.x;
    const int64_t b = row / dim, d = row - b * dim;
    const T* xr = x + row * L;
    TO* orow = out + row * L;
    const int32_t* pr = pos + b * L;
    float wk[W];
#pragma unroll
    for (int k = 0; k < W; ++k) wk[k] = w[d * W + k];
    const float b0 = bias ? bias[d] : 0.0f;

    for (int64_t l0 = (int64_t)threadIdx.x * KT; l0 < L; l0 += (int64_t)kThreads * KT) {
        const RawRun<T, KT> rx = load_raw<T, KT>(xr, l0);
        RawRun<T, KT> rh{};
        if (l0 > 0) rh = load_raw<T, KT>(xr, l0 - KT);
        int p[KT];
        load_pos<KT, true>(pr, l0, L, p);
        float xs[2 * KT], o[KT];
        if (l0 > 0) unpack_run(rh, xs);
        else load_row_halo<T, W>(st.xinit, row, xs);
        unpack_run(rx, xs + KT);
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            float v = fmaf(wk[W - 1], xs[KT + t], b0);               // tap 0: position indices are >= 0
#pragma unroll
            for (int k = 1; k < W; ++k)
                if (k <= p[t]) v = fmaf(wk[W - 1 - k], xs[KT + t - k], v);
            o[t] = silu ? v * sigmoid_f(v) : v;
        }
        store_run<TO, KT, true>(orow, l0, L, o);
    }
    if (st.xfinal && threadIdx.x == 0) store_xfinal<T, TO, W>(x, st, row, L);
}

// Backward: one wave per (row, segment), walking the segment from its end in steps
// of 64*KT tokens (long rows with few channels are cut into segments of whole steps,
// so that the grid has enough waves).
// Each lane owns KT consecutive tokens per step and computes their activation
// gradient g once.  dx of a token needs g of the next W-1 tokens (the reverse-index
// halo): they belong to the next lane, which hands over their masked values with a
// lane shift, and for lane 63 to lane 0 of the previous (later) step, whose values
// are carried.
// A step that crosses the row end loads the vectors inside the row, all of them before the first
// wait; with a branch per run, each run waited for the one before (35 x 84 x 5120 fp32: 180 ->
// 130 us, bf16 244 -> 199).
// DXF: a final-input gradient is given (a separate instantiation, so that the
// common path keeps its register count).
// ALL: a block holds all waves of one channel, batch row by batch row and segment by segment
// (up to kConvBwdParts of them), and sums their parameter gradients in that order itself;
// without it a block is one wave, which leaves its part in `partial` for the finalize.
template <typename T, typename TO, int W, int KT, bool DXF, bool ALL>
__global__ __launch_bounds__(ALL ? 64 * kConvBwdParts : 64) void conv1d_bwd_kernel(
    const T* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias,
    const int32_t* __restrict__ pos, const T* __restrict__ dout, TO* __restrict__ dx,
    float* __restrict__ partial, float* __restrict__ dw, float* __restrict__ dbias, ConvStates<T, TO> st,
    int64_t dim, int64_t L, int nseg, int silu) {
    static_assert(KT >= W - 1 && KT % 4 == 0, "the halo lies in the next lane's tokens");
    const int wave = ALL ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const int64_t b = ALL ? wave / nseg : blockIdx.x / dim;
    const int64_t d = ALL ? blockIdx.x : blockIdx.x - b * dim;
    const int seg = ALL ? wave - (int)b * nseg : blockIdx.y;
    const int64_t row = b * dim + d;
    const int lane = (int)(threadIdx.x & 63);
    const T* xr = x + row * L;
    const T* gr = dout + row * L;
    TO* dxr = dx + row * L;
    const int32_t* pr = pos + b * L;
    float wk[W];
#pragma unroll
    for (int k = 0; k < W; ++k) wk[k] = w[d * W + k];
    const float b0 = bias ? bias[d] : 0.0f;
    constexpr int64_t kSpan = 64 * KT;
    static_assert(kSpan == kConvBwdSpan, "segments hold whole steps");
    const int64_t nsteps = (L + kSpan - 1) / kSpan;
    const int64_t seg_steps = (nsteps + nseg - 1) / nseg;
    const int64_t s0 = (int64_t)seg * seg_steps;
    const int64_t s1 = min(nsteps, s0 + seg_steps);
    float acc[W + 1];   // dw[0..W-1], dbias
#pragma unroll
    for (int j = 0; j <= W; ++j) acc[j] = 0.0f;
    // masked activation gradients gm[k][t] (k > t, t < W-1) of the first W-1 tokens of
    // lane 0 in the step to the right: 0 past the row end; at the end of a segment that
    // is not the row's last, recomputed here (the same value in every lane)
    float cgm[W][W - 1];
#pragma unroll
    for (int k = 0; k < W; ++k) {
#pragma unroll
        for (int t = 0; t < W - 1; ++t) cgm[k][t] = 0.0f;
    }
    if (s1 * kSpan < L) {
        const int64_t e = s1 * kSpan;               // first token after the segment
#pragma unroll
        for (int t = 0; t < W - 1; ++t) {
            const int64_t l = e + t;
            if (l >= L) break;
            const int p = pr[l];
            float g = Storage<T>::load1(gr + l);
            if (silu) {
                float v = b0;
#pragma unroll
                for (int k = 0; k < W; ++k)
                    if (k <= p) v = fmaf(wk[W - 1 - k], Storage<T>::load1(xr + l - k), v);
                const float sg = sigmoid_f(v);
                g *= sg * (1.0f + v * (1.0f - sg));
            }
#pragma unroll
            for (int k = t + 1; k < W; ++k) cgm[k][t] = k <= p ? g : 0.0f;
        }
    }
    // One step; FULL (wave-uniform) means the step lies inside the row, so the loads and
    // stores need no bounds checks.
    auto step = [&](auto full_tag, const int64_t sidx) {
        constexpr bool FULL = decltype(full_tag)::value;
        const int64_t l0 = sidx * kSpan + (int64_t)lane * KT;
        // every load first.  x of tokens l0-8 .. l0+KT-1 (pre-activations of this lane's tokens)
        RawRun<T, kTok> rh{};
        if (l0 > 0) rh = load_part<T, kTok, FULL>(xr, l0 - kTok, L);
        const RawRun<T, KT> rx = load_part<T, KT, FULL>(xr, l0, L);
        const RawRun<T, KT> rg = load_part<T, KT, FULL>(gr, l0, L);
        int p[KT];
        load_pos<KT, FULL>(pr, l0, L, p);
        float xs[kTok + KT];
        if (l0 > 0) unpack_part<T, kTok, FULL>(rh, xr, l0 - kTok, L, xs);
        else load_row_halo<T, W>(st.xinit, row, xs);
        unpack_part<T, KT, FULL>(rx, xr, l0, L, xs + kTok);
        float gs[KT];
        unpack_part<T, KT, FULL>(rg, gr, l0, L, gs);   // 0 beyond L, so g = 0 there
        // gm[k][t] = g[t] if tap k of token t is live (k <= pos[t]) else 0, with g the
        // activation gradient.  The same masked values give dx through the reverse
        // indices (tap k of token j is live iff pos[j+k] >= k) and dw.  Tap 0 is always
        // live (position indices are >= 0).
        float gm[W][KT + W - 1];
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            bool live[W];
#pragma unroll
            for (int k = 1; k < W; ++k) live[k] = k <= p[t];
            float gt = gs[t];
            if (silu) {
                float v = fmaf(wk[W - 1], xs[kTok + t], b0);
#pragma unroll
                for (int k = 1; k < W; ++k)
                    if (live[k]) v = fmaf(wk[W - 1 - k], xs[kTok + t - k], v);
                const float sg = sigmoid_f(v);
                gt *= sg * (1.0f + v * (1.0f - sg));
            }
            gm[0][t] = gt;
#pragma unroll
            for (int k = 1; k < W; ++k) gm[k][t] = live[k] ? gt : 0.0f;
        }
        // the next W-1 tokens (only the taps that reach back into this lane): from the
        // next lane, or for lane 63 from the carry; then lane 0's become the carry
#pragma unroll
        for (int t = 0; t < W - 1; ++t) {
#pragma unroll
            for (int k = t + 1; k < W; ++k) {
                const float h = __shfl_down(gm[k][t], 1, 64);
                gm[k][KT + t] = lane == 63 ? cgm[k][t] : h;
                cgm[k][t] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, gm[k][t])));
            }
        }
        float o[KT];
#pragma unroll
        for (int i = 0; i < KT; ++i) {
            float a = wk[W - 1] * gm[0][i];
#pragma unroll
            for (int k = 1; k < W; ++k) a = fmaf(wk[W - 1 - k], gm[k][i + k], a);
            o[i] = a;
        }
        // the final inputs are copies of the last W-1 inputs: their gradient adds in
        if (DXF && l0 + KT > L - (W - 1)) {
#pragma unroll
            for (int i = 0; i < KT; ++i) {
                const int64_t j = l0 + i - (L - (W - 1));
                if (j >= 0 && l0 + i < L) o[i] += Storage<T>::load1(st.dxfinal + row * (W - 1) + j);
            }
        }
        store_run<TO, KT, FULL>(dxr, l0, L, o);
        // parameter gradients from this lane's own tokens
#pragma unroll
        for (int i = 0; i < KT; ++i) {
#pragma unroll
            for (int k = 0; k < W; ++k) acc[W - 1 - k] = fmaf(gm[k][i], xs[kTok + i - k], acc[W - 1 - k]);
            acc[W] += gm[0][i];
        }
    };
    for (int64_t sidx = s1 - 1; sidx >= s0; --sidx) {
        if ((sidx + 1) * kSpan <= L) step(std::true_type{}, sidx);
        else step(std::false_type{}, sidx);
    }
    // gradient of the inputs before the row: initial input j (token j-W+1) meets output
    // token t <= j through tap k = t-j+W-1 > t (weight w[j-t]); the carry now holds the
    // masked gradients of tokens 0..W-2
    if (st.dxinit && seg == 0 && lane == 0) {
#pragma unroll
        for (int j = 0; j < W - 1; ++j) {
            float a = 0.0f;
#pragma unroll
            for (int t = 0; t <= j; ++t) a = fmaf(wk[j - t], cgm[t - j + W - 1][t], a);
            // a row shorter than W-1 copies initial input j >= L to final input j - L
            if (st.dxfinal && j >= L) a += Storage<T>::load1(st.dxfinal + row * (W - 1) + (j - L));
            Storage<TO>::store1(st.dxinit + row * (W - 1) + j, a);
        }
    }
#pragma unroll
    for (int j = 0; j <= W; ++j) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc[j] += __shfl_xor(acc[j], off, 64);
    }
    if constexpr (ALL) {
        __shared__ float part[kConvBwdParts][W + 1];
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j <= W; ++j) part[wave][j] = acc[j];
        }
        __syncthreads();
        if (threadIdx.x <= W) {
            const int j = (int)threadIdx.x, parts = (int)(blockDim.x >> 6);
            float s = 0.0f;
            for (int r = 0; r < parts; ++r) s += part[r][j];
            if (j < W) dw[d * W + j] = s;
            else if (dbias) dbias[d] = s;
        }
    } else if (lane == 0) {
        float* pp = partial + ((b * nseg + seg) * dim + d) * (W + 1);
#pragma unroll
        for (int j = 0; j <= W; ++j) pp[j] = acc[j];
    }
}

// dw[d,k] = sum_r partial[r,d,k]; dbias[d] = sum_r partial[r,d,W] over the (batch row,
// segment) pairs r, in a fixed order
__global__ void conv1d_bwd_finalize(const float* __restrict__ partial, float* __restrict__ dw,
                                    float* __restrict__ dbias, int64_t batch, int64_t dim, int W) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= dim * (W + 1)) return;
    const int64_t d = i / (W + 1);
    const int j = (int)(i - d * (W + 1));
    float s = 0.0f;
    for (int64_t b = 0; b < batch; ++b) s += partial[(b * dim + d) * (W + 1) + j];
    if (j < W) dw[d * W + j] = s;
    else if (dbias) dbias[d] = s;
}

// bf16 rows that a block each walks.  Us, one wave per tile against a block per row:
// 2 x 6208 x 5120 52, 43; 1 x 7872 x 5120 34, 27; 2 x 16192 x 2048 53, 43; 1 x 21704 x 1536 29,
// 24; 4 x 3072 x 2048 22, 19; 5 x 7104 x 192 9.4, 7.3; 8 x 4096 x 4096 103, 95.  Beyond the limits, the second measured
// with row ends looked for: 12 x 1088 x 5120 62, 68 (a block's 2048 tokens are half empty);
// 1 x 32768 x 5120 141, 190 and 2 x 65536 x 1024 95, 123; 1 x 16384 x 256 5.1, 7.3 (too few
// rows); unaligned rows, 8 x 4095 x 4096 119, 121, 2 x 12289 x 2048 43, 46.  In fp32 a lane's 8
// tokens are two vectors, 32 bytes apart from the next lane's: 182, 223 at 8 x 4096 x 4096.
// (A launch holds fewer than 2^32 threads.)
bool conv_fwd_by_row(const ConvArgs& a) {
    const int64_t rows = a.batch * a.dim;
    return a.seqlen % kTok == 0 && a.seqlen > 2048 && a.seqlen < 32768 && rows >= 768 && rows < (int64_t)1 << 24;
}

// Rows per lane of the tiled forward where that leaves 8 waves for each of the 1024 SIMDs, else 1.
// Rows of several tiles: 16 tokens a lane (2 and 4 rows, us: fp32 15 x 1152 x 768 19.3, 18.3;
// 4 x 2304 x 1024 13.6, 12.4; 4 x 2048 x 1536 17.7, 16.6; 8 x 4096 x 4096 175, 179; bf16 15 x 1152 x
// 768 13.8, 14.7; 4 x 2048 x 1536 9.9, 10.7; 12 x 1088 x 5120 54, 52).  Shorter rows: 2 (fp32
// 16 x 250 x 2048 12.5, 13.1; 64 x 100 x 1024 9.6, 10.6).
template <typename T>
constexpr int kFwdRowsLong = 16 / Storage<T>::kPerVec;
constexpr int kFwdRows = 2;
constexpr int64_t kFwdWaves = 8192;

template <typename T, typename TO, int W, int R, bool LONG>
hipError_t conv_fwd_r(const ConvArgs& a, hipStream_t s, int lanes_log2, int64_t ntiles) {
    const int64_t set = (int64_t)R * (64 >> lanes_log2);           // channels of a wave
    const int64_t waves = (a.dim + set - 1) / set * ntiles;
    const ConvStates<T, TO> st{static_cast<const T*>(a.xinit), static_cast<T*>(a.xfinal), nullptr, nullptr};
    hipLaunchKernelGGL((conv1d_fwd_kernel<T, TO, W, R, LONG>),
                       dim3((unsigned)((waves + kThreads / 64 - 1) / (kThreads / 64)), (unsigned)a.batch), dim3(kThreads),
                       0, s, static_cast<const T*>(a.x), a.w, a.bias, a.pos, static_cast<TO*>(a.out), st, a.dim,
                       a.seqlen, a.silu, lanes_log2, (uint32_t)ntiles, (uint32_t)waves);
    return hipGetLastError();
}

template <typename T, typename TO, int W>
hipError_t conv_fwd_w(const ConvArgs& a, hipStream_t s) {
    constexpr int KT = Storage<T>::kPerVec;
    if constexpr (KT == kTok) {
        if (conv_fwd_by_row(a)) {
            const ConvStates<T, TO> st{static_cast<const T*>(a.xinit), static_cast<T*>(a.xfinal), nullptr, nullptr};
            hipLaunchKernelGGL((conv1d_fwd_row_kernel<T, TO, W>), dim3((unsigned)(a.batch * a.dim)), dim3(kThreads), 0, s,
                               static_cast<const T*>(a.x), a.w, a.bias, a.pos, static_cast<TO*>(a.out), st, a.dim,
                               a.seqlen, a.silu);
            return hipGetLastError();
        }
    }
    const int64_t nvec = (a.seqlen + KT - 1) / KT;
    int lanes_log2 = 0;
    while (lanes_log2 < 6 && ((int64_t)1 << lanes_log2) < nvec) ++lanes_log2;
    const int64_t ntiles = (nvec + 63) / 64;
    const auto many = [&](int64_t set) { return (a.dim + set - 1) / set * ntiles * a.batch >= kFwdWaves; };
    if (lanes_log2 == 6)
        return many(kFwdRowsLong<T>) ? conv_fwd_r<T, TO, W, kFwdRowsLong<T>, true>(a, s, 6, ntiles)
                                     : conv_fwd_r<T, TO, W, 1, true>(a, s, 6, ntiles);
    return many(kFwdRows * (64 >> lanes_log2)) ? conv_fwd_r<T, TO, W, kFwdRows, false>(a, s, lanes_log2, 1)
                                               : conv_fwd_r<T, TO, W, 1, false>(a, s, lanes_log2, 1);
}

template <typename T, typename TO>
hipError_t conv_fwd_t(const ConvArgs& a, hipStream_t s) {
    switch (a.width) {
        case 2: return conv_fwd_w<T, TO, 2>(a, s);
        case 3: return conv_fwd_w<T, TO, 3>(a, s);
        default: return conv_fwd_w<T, TO, 4>(a, s);
    }
}

// Whether a block takes all `parts` waves (batch rows x segments) of a channel.  It sums the
// parameter gradients and saves the finalize's launch, 2.5 us; but it needs that many of a CU's 20
// places at once, which costs where blocks queue, the more so where they load its four SIMDs
// unevenly or leave many places empty (12), and its waves read batch rows far apart.  Us, a wave per block against gathered, bf16
// rows of 500 tokens (fp32 and 64 tokens lie within a few percent):
//   4 waves x 3072 channels 19.9, 17.9; x 5120 28, 27;  5 x 1024 11.5, 10.9; x 1536 14.6, 15.3
//   6 x 1024 13.3, 12.2; x 1536 16.2, 17.5;  8 x 1024 15.7, 12.7; x 2048 26, 25; x 5120 51, 57
//   9 x 512 12.2, 11.4; x 1024 16.7, 21.4;  12 x 512 14.6, 12; x 1024 21.8, 23.1
//   16 x 512 17.4, 13.2; x 1024 28, 27; x 2048 45, 52;  9 x 704 x 5120: 61, 111; 12, 4 x 7488 x 403
//   23.5, 28.8
// Longer waves: 6 of them, 1 x 4096 x 700 10.8, 8.3; 1 x 8192 x 700 15.5, 15.6; 2 x 3648 x 768 15.7,
//   18; 10, 5 x 1088 x 512 13.2, 14.4; 14, 7 x 1280 x 347 14.1, 16.3; 1 x 16384 x 300 14.9, 17.8;
//   16, 16 x 2048 x 256 18.6, 13.3; 8, 8 x 4096 x 512 27, 24.
// Most elements: 2 x 8192 x 2048 45.3, 41.7, fp32 92, 89; 2^26 of them, 4 x 8192 x 2048 77, 79, fp32 177,
// 182; 8 x 4096 x 4096 157, 188.
bool conv_bwd_gathers(const ConvArgs& a, int64_t parts) {
    if (parts > kConvBwdParts || a.batch * a.dim * a.seqlen > (int64_t)1 << 25) return false;
    if (parts <= 4) return true;
    if (parts % 8 == 0) return parts * a.dim <= 8192;
    return parts * a.dim <= (parts < 8 ? 6144 : 4096) && a.batch * a.dim * a.seqlen <= (int64_t)1 << 22;
}

template <typename T, typename TO, int W, bool DXF>
hipError_t conv_bwd_w(const ConvArgs& a, hipStream_t s) {
    const ConvStates<T, TO> st{static_cast<const T*>(a.xinit), nullptr, static_cast<const T*>(a.dxfinal),
                               static_cast<TO*>(a.dxinit)};
    const T* x = static_cast<const T*>(a.x);
    const T* g = static_cast<const T*>(a.dout);
    TO* dx = static_cast<TO*>(a.out);
    const int64_t nseg = conv_bwd_segments(a.batch, a.dim, a.seqlen), parts = a.batch * nseg;
    if (conv_bwd_gathers(a, parts)) {
        hipLaunchKernelGGL((conv1d_bwd_kernel<T, TO, W, kTokBwd, DXF, true>), dim3((unsigned)a.dim),
                           dim3((unsigned)(64 * parts)), 0, s, x, a.w, a.bias, a.pos, g, dx, a.partial, a.dw, a.dbias,
                           st, a.dim, a.seqlen, (int)nseg, a.silu);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((conv1d_bwd_kernel<T, TO, W, kTokBwd, DXF, false>),
                       dim3((unsigned)(a.batch * a.dim), (unsigned)nseg), dim3(64), 0, s, x, a.w, a.bias, a.pos, g, dx,
                       a.partial, a.dw, a.dbias, st, a.dim, a.seqlen, (int)nseg, a.silu);
    if (hipError_t e = hipGetLastError()) return e;
    // the partials of every (batch row, segment) are summed like batch rows
    const int64_t n = a.dim * (a.width + 1);
    hipLaunchKernelGGL(conv1d_bwd_finalize, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       a.partial, a.dw, a.dbias, parts, a.dim, (int)a.width);
    return hipGetLastError();
}

template <typename T, typename TO>
hipError_t conv_bwd_t(const ConvArgs& a, hipStream_t s) {
    const bool dxf = a.dxfinal != nullptr;
    switch (a.width) {
        case 2: return dxf ? conv_bwd_w<T, TO, 2, true>(a, s) : conv_bwd_w<T, TO, 2, false>(a, s);
        case 3: return dxf ? conv_bwd_w<T, TO, 3, true>(a, s) : conv_bwd_w<T, TO, 3, false>(a, s);
        default: return dxf ? conv_bwd_w<T, TO, 4, true>(a, s) : conv_bwd_w<T, TO, 4, false>(a, s);
    }
}

}  // namespace

hipError_t launch_conv1d_fwd(const ConvArgs& a, hipStream_t s) {
    switch (a.dtype) {
        case 1: return conv_fwd_t<bf16_t, bf16_t>(a, s);
        case 2: return conv_fwd_t<bf16_t, float>(a, s);
        default: return conv_fwd_t<float, float>(a, s);
    }
}

hipError_t launch_conv1d_bwd(const ConvArgs& a, hipStream_t s) {
    switch (a.dtype) {
        case 1: return conv_bwd_t<bf16_t, bf16_t>(a, s);
        case 2: return conv_bwd_t<bf16_t, float>(a, s);
        default: return conv_bwd_t<float, float>(a, s);
    }
}

}  // namespace pm
