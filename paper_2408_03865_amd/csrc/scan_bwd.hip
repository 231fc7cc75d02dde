// scan_bwd.hip -- packed selective scan, backward (§3.4), and the second-pass
// reductions of its parameter gradients.
//
// Same work layout as the forward (16-lane DPP rows = channels, K consecutive
// tokens per lane, a block = 16 channels of one batch row), with chunks of
// 16*K = 128 tokens = the saved-state stride, walked from the last to the first:
//  1. stage B, C and the reset mask of the chunk in LDS;
//  2. per state n: replay the forward inside the chunk from the saved state h at
//     the chunk start (fold, row scan, replay), keeping Abar and Abar*h_{l-1};
//  3. run the reverse recurrence dh_l = Abar_{l+1} dh_{l+1} + C_l dy_l as a
//     reverse fold + reverse DPP row scan (row_shl), entering with the carry from
//     the chunk to the right.  Abar_{l+1} of a token whose successor starts a
//     sequence is 0 (the matching reset, §3.4): it is the very Abar the replay
//     computed, shifted by one token;
//  4. accumulate du, ddelta per token, dA per lane, and write the dB, dC
//     contributions; these are summed over the block's 16 channels in LDS and
//     written as one partial per block (part_bc), summed over blocks by
//     scan_bwd_finalize in a fixed order.
// dz needs y, which the forward has computed already: it saves the factor
// (y + D u) d(z sigmoid(z))/dz of dout beside the chunk states, and dz is written at
// the start of each chunk, so the state loop does not rebuild y.
// Long rows with few channels are split into segments scanned by different blocks
// (as in the forward): an aggregate pass folds each segment's reverse recurrence
// into dh_first = Q x + H, where x is dh at the first token of the next segment,
// and the main pass chains the maps to the right of its segment from the row end and
// enters with that x.
#include "common.hpp"
#include "launch.hpp"

namespace pm {
namespace {

constexpr int kN = 16;
constexpr int kRows = 16;
constexpr int kThreads = 256;
constexpr int kK = 8;               // tokens per lane
constexpr int kCH = 16 * kK;        // tokens per chunk == saved-state stride
static_assert(kCH == 128, "chunk must equal the saved-state stride");
static_assert(kRows == kScanBwdChannels, "partials are per 16 channels");

constexpr int kWaves = kThreads / 64;
constexpr int kSeg = kK + 4;        // padded lane segment: conflict-free 16-byte LDS reads

struct __attribute__((aligned(16))) BwdSmem {
    float red[2][kWaves][2][2][kCH];   // [state parity][wave][row pair][dB|dC][token]: sums of
                                       // two channels
                                    // (first: its addresses need no constant offset)
    // [state][lane's half][lane][token]: consecutive lanes read consecutive 16-byte words
    float B[kN][kK / 4][16][4];
    float C[kN][kK / 4][16][4];
    float M[kK / 4][16][4];         // 0, or -inf on a sequence start
    // one 16-byte read per (channel, state): A * log2(e), and the carries of the row's ends,
    // zeros in the other lanes.  Three copies: the middle lanes'; lane 0's with the state at
    // the chunk start (saved by the forward); lane 15's with dh and Abar at the first token
    // of the chunk to the right
    f32x4 tab[3][kRows][kN];
    float dA[kRows][kN];            // per-channel dA accumulators
};

struct BwdParams {
    const void* u;
    const void* delta;
    const float* A;
    const void* B;
    const void* C;
    const float* D;
    const void* z;
    const float* delta_bias;
    const int32_t* pos;
    const void* dout;
    const float* states;
    const float* dzf;     // (batch, dim, L): factor of dout in dz, saved by the forward
    const float* h0;      // state before each row (batch, dim, kN), or null
    const float* dhfinal; // gradient of the state after each row, or null; the main pass of split
                          // rows reads `entry`
    float* entry;         // split rows: copy of dhfinal, by the aggregate pass
    float* dh0;           // gradient of h0, or null; may be dhfinal's buffer
    void* du;
    void* ddelta;
    void* dz;
    float* part_bc;       // (batch, groups, 2, kN, L)
    float* part_chan;     // (batch, nseg, dim, kN + 2): dA[n], dD, ddelta_bias
    float2* agg;          // the segments' maps (batch, dim, nseg, kN) = (Q, H): written by the
                          // aggregate pass, chained by the main pass
    int64_t dim, L;
    int64_t seg_chunks;   // chunks per segment
    int nseg;
    int nchunk_states;
    int groups;
    int softplus;
};

// dh at the first token after segment `seg`: the maps x -> Q x + H of the segments to its
// right, from the last to the next, applied to x (the final state's gradient, or 0).  Each
// block chains its own: a few loads that do not wait for one another, against a launch of
// its own for a carry pass (5 us).
__device__ __forceinline__ float chain_maps(const float2* __restrict__ maps, int last, int seg, float x) {
    int s = last;
    for (; s - 8 >= seg; s -= 8) {
        float2 m[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) m[i] = maps[(int64_t)(s - i) * kN];
#pragma unroll
        for (int i = 0; i < 8; ++i) x = fmaf(m[i].x, x, m[i].y);
    }
    for (; s > seg; --s) {
        const float2 m = maps[(int64_t)s * kN];
        x = fmaf(m.x, x, m.y);
    }
    return x;
}

// Step and reset mask of token l of a row (the first token after a segment), or
// (0, 0) past the row end.
template <typename T>
__device__ __forceinline__ void token_step(const T* __restrict__ dr, const int32_t* __restrict__ pr,
                                           int64_t l, int64_t L, float dbias, int softplus,
                                           float& dt, float& m) {
    dt = 0.0f;
    m = 0.0f;
    if (l < L) {
        const float s = Storage<T>::load1(dr + l) + dbias;
        dt = softplus ? softplus_f(s) : s;
        m = pr[l] == 0 ? -INFINITY : 0.0f;
    }
}

// Main pass.  Bound by the VALU issue rate (at 8 x 4096 x 4096 92% busy counted at 2.4 GHz, 98%
// of the cycles that the clock gave), so what counts is instructions per (token, channel, state): one 16-byte table read per (channel, state)
// with one address to step, carries that enter the scans at the row's ends, and the dA
// sums of two states at once took the call from 1920 to 1815 us there (fp32 2120 to 2035).
// Two channels per lane need 10% fewer instructions and half the dB/dC partials, but 213
// VGPRs: two waves per SIMD keep the VALU 84% busy, 1870 us.  Three waves per SIMD (at most 168 VGPRs):
// three blocks share a CU, so one block's barrier waits are covered by the other two.
template <typename T, typename TO>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
void scan_bwd_kernel(BwdParams p) {
    constexpr int PV = Storage<T>::kPerVec;
    constexpr int K = kK;
    __shared__ BwdSmem sm;

    const int64_t b = blockIdx.y;
    const int64_t grp = blockIdx.x;
    const int seg = blockIdx.z;
    const int64_t L = p.L;
    const int64_t nchunk = (L + kCH - 1) / kCH;
    const int64_t c0 = (int64_t)seg * p.seg_chunks;
    const int64_t c1 = min(nchunk, c0 + p.seg_chunks);
    // Addresses are a block-uniform base (scalar registers) plus a lane's offset, the same for
    // all activations, so that the rows' pointers take no vector registers over the state
    // loop (a pointer per tensor spilled 9 of them: 1915 us at 8 x 4096 x 4096, 1870 this way).
    const int64_t d0 = grp * kRows;                       // the block's first channel
    const int64_t row0 = b * p.dim + d0;
    const int left = (int)min(p.dim - d0, (int64_t)kRows);   // channels of the block
    const T* Bb = static_cast<const T*>(p.B) + b * kN * L;
    const T* Cb = static_cast<const T*>(p.C) + b * kN * L;
    const int32_t* pr = p.pos + b * L;

    const int tid = threadIdx.x;
    const int j = tid & 15, r = tid >> 4;
    const bool active = r < left;                           // rows past the last channel repeat it, inactive
    const int64_t rc = min(r, left - 1);                   // channel, from d0
    const int64_t rl = rc * L + j * K;              // the lane's first token
    const float Dd = p.D ? p.D[d0 + rc] : 0.0f;
    const float dbias = p.delta_bias ? p.delta_bias[d0 + rc] : 0.0f;
    float dDacc = 0.0f, dbacc = 0.0f;
    float dt_next, m_next;     // step and mask of the first token of the chunk to the right
    // at the row end the carry is the final state's gradient, entering h_{L-1} with
    // multiplier 1
    const bool row_end = c1 == nchunk;
    {   // per-channel tables: lane j of row r fills state j
        const int64_t d = d0 + rc;
        token_step<T>(static_cast<const T*>(p.delta) + (b * p.dim + d) * L, pr, c1 * kCH, L, dbias, p.softplus, dt_next, m_next);
        const float A2n = p.A[d * kN + j] * kLog2e;
        float xc0 = 0.0f;
        if (p.dhfinal) xc0 = p.dhfinal[(b * p.dim + d) * kN + j];
        xc0 = chain_maps(p.agg + (b * p.dim + d) * p.nseg * kN + j, p.nseg - 1, seg, xc0);
        sm.tab[0][r][j] = f32x4{A2n, 0.0f, 0.0f, 0.0f};
        sm.tab[1][r][j] = f32x4{A2n, 0.0f, 0.0f, 0.0f};
        sm.tab[2][r][j] = f32x4{A2n, 0.0f, xc0, !row_end ? fast_exp2(fmaf(dt_next, A2n, m_next)) : (p.dhfinal ? 1.0f : 0.0f)};
        sm.dA[r][j] = 0.0f;
    }
    // One chunk; FULL (block-uniform) means the chunk lies inside the row, so every load
    // and store is unconditional.
    auto chunk = [&](auto full_tag, const int64_t c) {
        constexpr bool FULL = decltype(full_tag)::value;
        const int64_t lb = c * kCH;
        const int64_t l0 = lb + (int64_t)j * K;
        const int64_t base = row0 * L + lb;
        const T* const ub = static_cast<const T*>(p.u) + base;
        const T* const db = static_cast<const T*>(p.delta) + base;
        const T* const gb = static_cast<const T*>(p.dout) + base;
        const T* const zb = static_cast<const T*>(p.z) + base;
        // this lane's inputs, loaded first in a full chunk so that their latency
        // overlaps the staging below; u and delta stay in registers, as stored, for the
        // chunk end
        RawRun<T, K> wu, wd, wg, wz;
        f32x4 wf[2];
        if constexpr (FULL) {
            wu = load_raw_nt<T, K>(ub + rl, 0);
            wd = load_raw_nt<T, K>(db + rl, 0);
            wg = load_raw_nt<T, K>(gb + rl, 0);
            if (p.z) wz = load_raw_nt<T, K>(zb + rl, 0);
        }
        if (p.z) {
            // this lane's 8 tokens of the dz factor: vectors 2 (j & 1) and 2 (j & 1) + 1 of
            // the forward's lane 8 (c & 1) + j / 2 in forward chunk c / 2 (padded row, so
            // whole vectors even past the row end)
            const float* const fb = p.dzf + row0 * dzf_row_len(L) + dzf_vec(c >> 1, 0, 8 * (int)(c & 1));
            const float* const fr = fb + rc * dzf_row_len(L) + dzf_vec(0, 2 * (j & 1), j >> 1);
            wf[0] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(fr));
            wf[1] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(fr + dzf_vec(0, 1, 0)));
        }
        // ---- stage B, C, the reset mask and the chunk-start states in LDS ----
        // The addresses are computed again for each chunk from an index that the compiler cannot
        // see through: kept over the state loop they would take vector registers that it needs.
        int tids = tid;
        asm volatile("" : "+v"(tids));
        for (int idx = tids * PV; idx < kN * kCH; idx += kThreads * PV) {
            const int n = idx / kCH, t = idx - n * kCH;
            float vb[PV], vc[PV];
            load_run<T, PV, FULL>(Bb + (int64_t)n * L, lb + t, L, vb);
            load_run<T, PV, FULL>(Cb + (int64_t)n * L, lb + t, L, vc);
#pragma unroll
            for (int i = 0; i < PV; i += 4) {
                const int h = (t % K + i) / 4;
                *reinterpret_cast<f32x4*>(sm.B[n][h][t / K]) = f32x4{vb[i], vb[i + 1], vb[i + 2], vb[i + 3]};
                *reinterpret_cast<f32x4*>(sm.C[n][h][t / K]) = f32x4{vc[i], vc[i + 1], vc[i + 2], vc[i + 3]};
            }
        }
        if (tids < kCH) {
            const int64_t l = lb + tids;
            sm.M[tids % K / 4][tids / K][tids % 4] = ((FULL || l < L) && pr[l] == 0) ? -INFINITY : 0.0f;
        }
        {   // state at the chunk start (h after token lb-1), saved by the forward
            float h = 0.0f;
            if (c > 0) h = p.states[((row0 + rc) * p.nchunk_states + (c - 1)) * kN + j];
            else if (p.h0) h = p.h0[(row0 + rc) * kN + j];
            sm.tab[1][r][j].y = h;
        }
        __syncthreads();

        // ---- per-token inputs ----
        float dt[K], dlu[K], dyD[K], sdhB[K], sdA[K];
        float S = 0.0f, Sr, M[K], Mf = 0.0f, Mr = 0.0f, m0 = 0.0f;
#pragma unroll
        for (int k = 0; k < K; k += 4) {
            const f32x4 m = *reinterpret_cast<const f32x4*>(sm.M[k / 4][j]);
            M[k] = m.x; M[k + 1] = m.y; M[k + 2] = m.z; M[k + 3] = m.w;
            if (k == 0) m0 = m.x;
            Mf += (m.x + m.y) + (m.z + m.w);
            Mr += ((k > 0 ? m.x : 0.0f) + m.y) + (m.z + m.w);
        }
        {
            float dl[K], uv[K];
            if constexpr (FULL) {
                unpack_run(wu, uv);
                unpack_run(wd, dl);
                unpack_run(wg, dyD);                          // dout for now
            } else {
                load_run<T, K, FULL>(ub + rl, 0, L - l0, uv);
                load_run<T, K, FULL>(db + rl, 0, L - l0, dl);
                load_run<T, K, FULL>(gb + rl, 0, L - l0, dyD);
            }
            if (p.z) {
                // dz = dout (y + D u) d(z sigmoid(z))/dz: the forward saved every factor
                // but dout, so dz is final here; dy = dout SiLU(z) enters the recurrence
                float zv[K];
                if constexpr (FULL) unpack_run(wz, zv);
                else load_run<T, K, FULL>(zb + rl, 0, L - l0, zv);
                float fz[K] = {wf[0].x, wf[0].y, wf[0].z, wf[0].w, wf[1].x, wf[1].y, wf[1].z, wf[1].w};
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    fz[k] *= dyD[k];
                    dyD[k] *= zv[k] * sigmoid_f(zv[k]);
                }
                if (active) store_run<TO, K, FULL, true>(static_cast<TO*>(p.dz) + base + rl, 0, L - l0, fz);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float s = dl[k] + dbias;
                float v = s;
                if (p.softplus) v = softplus_f(s);
                if (!FULL) v = (l0 + k < L) ? v : 0.0f;   // identity past the row end
                dt[k] = v;
                dlu[k] = v * uv[k];
                sdhB[k] = 0.0f;
                sdA[k] = 0.0f;
                S += v;
            }
            if (left < kRows) {                            // padding rows contribute nothing to dB, dC
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    dyD[k] = active ? dyD[k] : 0.0f;
                    dlu[k] = active ? dlu[k] : 0.0f;
                }
            }
#pragma unroll
            for (int k = 0; k < K; ++k) dDacc = fmaf(dyD[k], uv[k], dDacc);
        }
        // Lane products of Abar as one exp2 each: prod_k exp2(dt_k A2) = exp2(A2 sum_k dt_k),
        // forced to 0 when a reset falls inside the product range.
        Sr = S - dt[0] + dpp<kRowShl1>(dt_next, dt[0]);    // the next token's step, across the lane edge
        dt_next = dpp<kNewBcast0>(0.0f, dt[0]);
        Mr += dpp<kRowShl1>(m_next, m0);
        m_next = dpp<kNewBcast0>(0.0f, m0);

        // per-thread LDS addresses
        const f32x4* const tab_r = sm.tab[j == 0 ? 1 : j == 15 ? 2 : 0][r];
        // dB/dC sums: where this thread writes, and the offset of its partial (token red_t of
        // dB or dC) inside the block's state-0 partials
        const int wr = r & 3;                        // row inside the wave
        float* const red_w = &sm.red[0][tid >> 6][wr & 1][wr >> 1][j * K];
        const int red_which = __builtin_amdgcn_readfirstlane(tid >> 7);   // 0: dB, 1: dC (per wave)
        const int red_t = tid & (kCH - 1);
        const float* const red_r = &sm.red[0][0][0][red_which][red_t];
        float* const part_n = p.part_bc + ((b * p.groups + grp) * 2 + red_which) * kN * L + lb;
        float dA_even = 0.0f;
        // one state; the odd one of a pair also sums the dA of both
#pragma unroll 1
        for (int n = 0; n < kN; ++n) {
            const f32x4 tb = tab_r[n];
            const float A2n = tb.x, hin = tb.y, xc = tb.z, an = tb.w;
            float a[K], ah[K], bv[K], cdy[K], bx[K];
            // ---- fold the lane's tokens both ways, then both row scans at once ----
#pragma unroll
            for (int k = 0; k < K; k += 4) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(sm.B[n][k / 4][j]);
                bv[k] = v.x; bv[k + 1] = v.y; bv[k + 2] = v.z; bv[k + 3] = v.w;
                const f32x4 cv = *reinterpret_cast<const f32x4*>(sm.C[n][k / 4][j]);
                cdy[k] = cv.x * dyD[k]; cdy[k + 1] = cv.y * dyD[k + 1];
                cdy[k + 2] = cv.z * dyD[k + 2]; cdy[k + 3] = cv.w * dyD[k + 3];
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                a[k] = fast_exp2(fmaf(dt[k], A2n, M[k]));
                bx[k] = dlu[k] * bv[k];
            }
            // forward: h -> P h + H over the lane's tokens
            float H = bx[0];
#pragma unroll
            for (int k = 1; k < K; ++k) H = fmaf(a[k], H, bx[k]);
            // reverse: dh_l = Abar_{l+1} dh_{l+1} + C_l dy_l over the lane's tokens
            float Hr = cdy[K - 1];
#pragma unroll
            for (int k = K - 2; k >= 0; --k) Hr = fmaf(a[k + 1], Hr, cdy[k]);
            float P = fast_exp2(fmaf(S, A2n, Mf));
            float Pr = fast_exp2(fmaf(Sr, A2n, Mr));
            // the carries enter at the row's ends, so the scans give the states themselves
            H = fmaf(P, hin, H);
            Hr = fmaf(Pr, xc, Hr);
            // Wave priority (s_setprio, per wave, relative to the other waves of the SIMD):
            // raised over this DPP latency chain, and from the reverse recurrence to the
            // state's barrier, so that the block's waves reach the barrier sooner; the
            // other blocks' waves fill the issue slots meanwhile (-4% at 8 x 4096 x 4096).
            __builtin_amdgcn_s_setprio(1);
            row_scan_up_down(P, H, Pr, Hr);
            __builtin_amdgcn_s_setprio(0);
            // ---- replay the forward inside the chunk ----
            float hprev = dpp<kRowShr1>(hin, H);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                ah[k] = a[k] * hprev;
                const float h = ah[k] + bx[k];
                bx[k] = dyD[k] * h;                          // dC contribution (reuses bx)
                hprev = h;
            }
            // ---- reverse recurrence, entering with the carry from the right ----
            const float alast = dpp<kRowShl1>(an, a[0]);      // Abar of the next lane's first token
            float dh = dpp<kRowShl1>(xc, Hr);                   // dh at the next lane's first token
            if (j == 0) *(reinterpret_cast<float2*>(&sm.tab[2][r][n]) + 1) = float2{Hr, a[0]};
            __builtin_amdgcn_s_setprio(2);
            float dAl = 0.0f;
            float dBp[K];
#pragma unroll
            for (int k = K - 1; k >= 0; --k) {
                const float am = (k == K - 1) ? alast : a[k + 1];
                dh = fmaf(am, dh, cdy[k]);
                sdhB[k] = fmaf(dh, bv[k], sdhB[k]);
                const float q = dh * ah[k];
                sdA[k] = fmaf(q, A2n, sdA[k]);
                dAl = fmaf(q, dt[k], dAl);
                dBp[k] = dh * dlu[k];
            }
            // dA: the row sums of two states at once
            if (n & 1) {
                const float s = row_sum2_to_7_15(dA_even, dAl);
                if ((j & 7) == 7) sm.dA[r][n - 1 + (j >> 3)] += s;
            } else {
                dA_even = dAl;
            }
            // ---- dB, dC: sum over the block's channels ----
            // First over pairs of the wave's 4 rows (channels) in registers:
            // permlane32_swap pairs rows {0,1} with {2,3} and leaves dB sums on rows 0-1
            // and dC sums on rows 2-3 (one swap and one add per pair of values; a second
            // swap stage over even and odd rows measured slower than summing eight
            // partials instead of four from LDS).
            float R[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const auto s2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(dBp[k]),
                                                                 __float_as_uint(bx[k]), false, false);
                R[k] = __uint_as_float(s2[0]) + __uint_as_float(s2[1]);
            }
            const int par = (n & 1) * (kWaves * 4 * kCH);
            *reinterpret_cast<f32x4*>(red_w + par) = f32x4{R[0], R[1], R[2], R[3]};
            *reinterpret_cast<f32x4*>(red_w + par + 4) = f32x4{R[4], R[5], R[6], R[7]};
            __syncthreads();
            __builtin_amdgcn_s_setprio(0);
            {   // then over the block's waves x 2 row pairs, in a fixed order
                float s = red_r[par];
#pragma unroll
                for (int q = 1; q < 2 * kWaves; ++q) s += red_r[par + q * 2 * kCH];
                if (FULL || lb + red_t < L)
                    __builtin_nontemporal_store(s, part_n + n * L + red_t);   // read once, by the finalize
            }
            // no second barrier: the next state writes the other buffer, and this one is
            // rewritten only after every thread has passed the next state's barrier
        }

        // ---- per-token gradients ----
        {
            float o_du[K], o_dd[K];
            float uv[K], dl[K];
            if constexpr (FULL) {
                unpack_run(wu, uv);
                unpack_run(wd, dl);
            } else {
                load_run<T, K, FULL>(ub + rl, 0, L - l0, uv);
                load_run<T, K, FULL>(db + rl, 0, L - l0, dl);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                o_du[k] = fmaf(dyD[k], Dd, dt[k] * sdhB[k]);
                const float ddt = fmaf(uv[k], sdhB[k], sdA[k] * kLn2);   // sdA was built with A*log2e
                const float s = dl[k] + dbias;
                o_dd[k] = p.softplus ? ddt * softplus_grad_f(s, dt[k]) : ddt;
                dbacc += (FULL || l0 + k < L) ? o_dd[k] : 0.0f;
            }
            if (active) {
                store_run<TO, K, FULL, true>(static_cast<TO*>(p.du) + base + rl, 0, L - l0, o_du);
                store_run<TO, K, FULL, true>(static_cast<TO*>(p.ddelta) + base + rl, 0, L - l0, o_dd);
            }
        }
        __syncthreads();     // LDS is restaged for the next chunk
    };
    for (int64_t c = c1 - 1; c >= c0; --c) {
        if ((c + 1) * kCH <= L) chunk(std::true_type{}, c);
        else chunk(std::false_type{}, c);
    }

    // ---- per-channel partials ----
    dDacc = row_sum_to_15(dDacc);
    dbacc = row_sum_to_15(dbacc);
    if (!active) return;
    const int64_t d = d0 + r;
    // gradient of the initial state: dh at token 0 times Abar at token 0 (0 at a start),
    // both left in LDS by lane 0 after the first chunk
    if (p.dh0 && c0 == 0) p.dh0[(b * p.dim + d) * kN + j] = sm.tab[2][r][j].w * sm.tab[2][r][j].z;
    float* pc = p.part_chan + ((b * p.nseg + seg) * p.dim + d) * (kN + 2);
    pc[j] = sm.dA[r][j];
    if (j == 15) {
        pc[kN] = dDacc;
        pc[kN + 1] = dbacc;
    }
}

// Aggregate pass of one segment (blockIdx.z + 1; the first segment needs none): the
// reverse recurrence over the segment with x = 0 gives H = dh at its first token,
// and Q = the product of the multipliers Abar_{l+1} over its tokens l, so that
// dh_first = Q x + H.  Same arithmetic as the main pass, without the forward replay
// and the gradients.
struct __attribute__((aligned(16))) AggSmem {
    float C[kN][16][kSeg];
    float M[16][kSeg];
    float A2[kRows][kN];
    float xc[kRows][kN];
    float q[kRows][kN];
};

template <typename T>
__global__ __launch_bounds__(kThreads) void scan_bwd_agg_kernel(BwdParams p) {
    constexpr int PV = Storage<T>::kPerVec;
    constexpr int K = kK;
    __shared__ AggSmem sm;

    const int tid = threadIdx.x;
    const int j = tid & 15;
    const int r = tid >> 4;
    const int64_t b = blockIdx.y;
    const int64_t g = blockIdx.x;
    const int seg = blockIdx.z + 1;
    const int64_t d = min(g * kRows + r, p.dim - 1);
    const int64_t L = p.L;
    const int64_t rowoff = (b * p.dim + d) * L;
    const int64_t nchunk = (L + kCH - 1) / kCH;
    const int64_t c0 = (int64_t)seg * p.seg_chunks;
    const int64_t c1 = min(nchunk, c0 + p.seg_chunks);

    const T* dr = static_cast<const T*>(p.delta) + rowoff;
    const T* zr = p.z ? static_cast<const T*>(p.z) + rowoff : nullptr;
    const T* gr = static_cast<const T*>(p.dout) + rowoff;
    const T* Cb = static_cast<const T*>(p.C) + b * kN * L;
    const int32_t* pr = p.pos + b * L;

    const float dbias = p.delta_bias ? p.delta_bias[d] : 0.0f;
    {
        const int rr = tid >> 4, n = tid & 15;
        const int64_t dd = min(g * kRows + rr, p.dim - 1);
        sm.A2[rr][n] = p.A[dd * kN + n] * kLog2e;
        sm.xc[rr][n] = 0.0f;
        sm.q[rr][n] = 1.0f;
        // The main pass's blocks each start from dhfinal, and the first segment's write dh0,
        // which may be the same memory.
        if (seg == 1 && p.dhfinal) p.entry[(b * p.dim + dd) * kN + n] = p.dhfinal[(b * p.dim + dd) * kN + n];
    }

    auto chunk = [&](auto full_tag, const int64_t c) {
        constexpr bool FULL = decltype(full_tag)::value;
        const int64_t lb = c * kCH;
        float dt_next, m_next;     // step and mask of the first token after the chunk
        token_step<T>(dr, pr, lb + kCH, L, dbias, p.softplus, dt_next, m_next);
        for (int idx = tid * PV; idx < kN * kCH; idx += kThreads * PV) {
            const int n = idx / kCH, t = idx - n * kCH;
            float vc[PV];
            load_run<T, PV, FULL>(Cb + (int64_t)n * L, lb + t, L, vc);
            float* dc = &sm.C[n][t / K][t % K];
#pragma unroll
            for (int i = 0; i < PV; ++i) dc[i] = vc[i];
        }
        for (int t = tid; t < kCH; t += kThreads) {
            const int64_t l = lb + t;
            sm.M[t / K][t % K] = ((FULL || l < L) && pr[l] == 0) ? -INFINITY : 0.0f;
        }
        __syncthreads();

        const int64_t l0 = lb + (int64_t)j * K;
        float dt[K], dyD[K], M[K];
        float S = 0.0f, Mr = 0.0f;
        {
            float dl[K];
            load_run<T, K, FULL>(dr, l0, L, dl);
            load_run<T, K, FULL>(gr, l0, L, dyD);
            if (zr) {
                float zv[K];
                load_run<T, K, FULL>(zr, l0, L, zv);
#pragma unroll
                for (int k = 0; k < K; ++k) dyD[k] *= zv[k] * sigmoid_f(zv[k]);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float s = dl[k] + dbias;
                float v = s;
                if (p.softplus) v = softplus_f(s);
                if (!FULL) v = (l0 + k < L) ? v : 0.0f;
                dt[k] = v;
            }
#pragma unroll
            for (int k = 0; k < K; k += 4) {
                const f32x4 m = *reinterpret_cast<const f32x4*>(&sm.M[j][k]);
                M[k] = m.x; M[k + 1] = m.y; M[k + 2] = m.z; M[k + 3] = m.w;
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                S += dt[k];
                if (k > 0) Mr += M[k];
            }
        }
        const float dt0n = dpp<kRowShl1>(dt_next, dt[0]);
        const float m0n = dpp<kRowShl1>(m_next, M[0]);
        const float Sr = S - dt[0] + dt0n;
        Mr += m0n;

#pragma unroll 1
        for (int n = 0; n < kN; ++n) {
            // a (channel, state) whose multiplier product is already exactly 0 is final;
            // the wave skips the state when that holds for its 4 channels
            if (__all(sm.q[r][n] == 0.0f)) continue;
            const float A2n = sm.A2[r][n];
            float cdy[K];
#pragma unroll
            for (int k = 0; k < K; k += 4) {
                const f32x4 cv = *reinterpret_cast<const f32x4*>(&sm.C[n][j][k]);
                cdy[k] = cv.x * dyD[k]; cdy[k + 1] = cv.y * dyD[k + 1];
                cdy[k + 2] = cv.z * dyD[k + 2]; cdy[k + 3] = cv.w * dyD[k + 3];
            }
            float Hr = cdy[K - 1];
#pragma unroll
            for (int k = K - 2; k >= 0; --k)
                Hr = fmaf(fast_exp2(fmaf(dt[k + 1], A2n, M[k + 1])), Hr, cdy[k]);
            float Pr = fast_exp2(fmaf(Sr, A2n, Mr));
            row_scan_down(Pr, Hr);
            // lane 0's (Pr, Hr) is the chunk's map from dh after the chunk to dh at its
            // first token; the chunks before it are already composed in (q, xc), which
            // becomes (q Pr, q Hr + xc)
            if (j == 0) {
                const float qa = sm.q[r][n];
                sm.xc[r][n] = fmaf(qa, Hr, sm.xc[r][n]);
                sm.q[r][n] = qa * Pr;
            }
        }
        __syncthreads();
    };
    // The chunk maps are composed from the segment's start forwards.  Once the product
    // of the multipliers is exactly 0 for every channel and state of the block (the
    // token before a sequence start, or underflow of a long decay), the later chunks
    // contribute exactly nothing, and the walk stops.
    for (int64_t c = c0; c < c1; ++c) {
        if ((c + 1) * kCH <= L) chunk(std::true_type{}, c);
        else chunk(std::false_type{}, c);
        if (!__syncthreads_or(sm.q[tid >> 4][tid & 15] != 0.0f)) break;
    }
    {
        const int rr = tid >> 4, n = tid & 15;
        const int64_t dd = g * kRows + rr;
        if (dd < p.dim) {
            p.agg[((b * p.dim + dd) * p.nseg + seg) * kN + n] = float2{sm.q[rr][n], sm.xc[rr][n]};
        }
    }
}

// The second-pass sums, one launch: the first `chan_blocks` blocks sum the per-channel
// partials, the others dB and dC.
//  - dA[d,n], dD[d], ddelta_bias[d] = sum over batch rows and segments (fixed order).
//  - dB[b,n,l] / dC[b,n,l] = sum over groups of the per-block partials.  Each thread owns
//    four consecutive tokens and keeps four running sums over interleaved groups
//    (q mod 4), added at the end: a fixed order, so the result is reproducible.
__global__ __launch_bounds__(kThreads) void scan_bwd_finalize(
    const float* __restrict__ part_bc, float* __restrict__ dB, float* __restrict__ dC, int64_t batch,
    int64_t L, int groups, const float* __restrict__ part_chan, float* __restrict__ dA,
    float* __restrict__ dD, float* __restrict__ ddb, int64_t nparts, int64_t dim, int chan_blocks) {
    if ((int)blockIdx.x < chan_blocks) {
        const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;   // over dim*(kN+2)
        if (i >= dim * (kN + 2)) return;
        const int64_t d = i / (kN + 2);
        const int q = (int)(i - d * (kN + 2));
        float s = 0.0f;
#pragma unroll 4
        for (int64_t b = 0; b < nparts; ++b) s += part_chan[b * dim * (kN + 2) + i];
        if (q < kN) dA[d * kN + q] = s;
        else if (q == kN) { if (dD) dD[d] = s; }
        else if (ddb) ddb[d] = s;
        return;
    }
    const int64_t NL = (int64_t)kN * L;
    const int64_t i4 = ((int64_t)(blockIdx.x - chan_blocks) * kThreads + threadIdx.x) * 4;   // over batch*2*NL
    if (i4 >= batch * 2 * NL) return;
    const int64_t b = i4 / (2 * NL);
    const int64_t rem = i4 - b * 2 * NL;
    const int which = (int)(rem / NL);
    const int64_t nl = rem - which * NL;
    const float* src = part_bc + ((b * groups) * 2 + which) * NL + nl;
    const int64_t stride = 2 * NL;
    float* dst = (which ? dC : dB) + b * NL + nl;
    // NL = 16 L, so a group of four never crosses a (b, dB|dC) boundary and every
    // offset is a multiple of four floats (16-byte aligned).
    f32x4 acc[4] = {};
    int q = 0;
    for (; q + 4 <= groups; q += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            acc[u] += *reinterpret_cast<const f32x4*>(src + (int64_t)(q + u) * stride);
    }
    for (; q < groups; ++q) acc[q & 3] += *reinterpret_cast<const f32x4*>(src + (int64_t)q * stride);
    *reinterpret_cast<f32x4*>(dst) = (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

template <typename T, typename TO>
hipError_t launch_t(const ScanArgs& a, hipStream_t s) {
    static_assert(kK == 8 && 2 * kCH == kDzfChunk, "the dz factor layout follows the forward's chunk");
    BwdParams p;
    p.u = a.u; p.delta = a.delta; p.A = a.A; p.B = a.B; p.C = a.C; p.D = a.D; p.z = a.z;
    p.delta_bias = a.delta_bias; p.pos = a.pos; p.dout = a.dout; p.states = a.states;
    p.dzf = a.z ? a.dzf : nullptr;
    if (a.z && !a.dzf) return hipErrorInvalidValue;
    p.h0 = a.h0; p.dhfinal = a.dhfinal; p.dh0 = a.dh0;
    p.du = a.du; p.ddelta = a.ddelta; p.dz = a.dz; p.part_bc = a.part_bc; p.part_chan = a.part_chan;
    p.dim = a.dim; p.L = a.seqlen;
    p.nchunk_states = (int)((a.seqlen + kCH - 1) / kCH);
    p.groups = (int)((a.dim + kRows - 1) / kRows);
    p.softplus = a.softplus;
    const SegPlan sp = scan_segments(a.batch, a.dim, a.seqlen, kSegTargetBwd);
    static_assert(kSegUnit % kCH == 0, "segments hold whole chunks");
    p.seg_chunks = sp.seg_len / kCH;
    p.nseg = (int)sp.nseg;
    p.entry = a.ws_entry;
    p.agg = reinterpret_cast<float2*>(a.ws_agg);
    const dim3 groups((unsigned)p.groups, (unsigned)a.batch);
    if (sp.nseg > 1) {
        hipLaunchKernelGGL((scan_bwd_agg_kernel<T>), dim3(groups.x, groups.y, (unsigned)(sp.nseg - 1)), dim3(kThreads),
                           0, s, p);
        if (hipError_t e = hipGetLastError()) return e;
        if (p.dhfinal) p.dhfinal = p.entry;
    }
    hipLaunchKernelGGL((scan_bwd_kernel<T, TO>), dim3(groups.x, groups.y, (unsigned)sp.nseg), dim3(kThreads), 0, s, p);
    if (hipError_t e = hipGetLastError()) return e;
    const int64_t nch = a.dim * (kN + 2), chan_blocks = (nch + kThreads - 1) / kThreads;
    const int64_t nbc4 = a.batch * 2 * kN * a.seqlen / 4, bc_blocks = (nbc4 + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(scan_bwd_finalize, dim3((unsigned)(chan_blocks + bc_blocks)), dim3(kThreads), 0, s, a.part_bc,
                       a.dB, a.dC, a.batch, a.seqlen, p.groups, a.part_chan, a.dA, a.dD, a.ddelta_bias,
                       a.batch * sp.nseg, a.dim, (int)chan_blocks);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_scan_bwd(const ScanArgs& a, hipStream_t s) {
    switch (a.dtype) {
        case 1: return launch_t<bf16_t, bf16_t>(a, s);
        case 2: return launch_t<bf16_t, float>(a, s);
        default: return launch_t<float, float>(a, s);
    }
}

}  // namespace pm
