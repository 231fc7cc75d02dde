// scan_fwd.hip -- packed selective scan, forward (Eqs. 1a, 1b, 2a; Alg. 2; §3.4).
//
// Layout of the work (gfx950, wave64):
//  - a block is 4 waves; a group of LANES lanes (16, 32 or 64: whole DPP rows) owns one
//    channel d of one batch row b, so a block covers 256 / LANES channels of one b;
//  - each lane owns K = 256 / LANES consecutive tokens, a group owns a chunk of 256
//    tokens, and the block walks the sequence chunk by chunk, carrying the state h[n] of
//    every channel from one chunk to the next in LDS.  16 lanes need the fewest
//    instructions (fold and scans are shared by 16 tokens), 32 and 64 give two and four
//    times the waves and shorter chains where 16 leave SIMDs idle (scan_fwd_plan);
//  - B and C of the chunk (shared by the block's channels) and the reset mask derived
//    from the position indices are staged once per chunk in LDS as fp32 (conflict-free
//    16-byte reads), read from HBM with coalesced vector loads (§3.5);
//  - per state n the pair (Abar, Bbar x) = (exp(dt*A), dt*B*u) is folded over the
//    lane's K tokens, the lane aggregates are combined by an inclusive DPP scan over the
//    group, the chunk carry is applied, and the lane replays its K tokens from its start
//    state to form h and y += C h.
//  - Reset (Alg. 2): Abar = exp2(dt * A*log2e + M) with M = -inf on a token whose
//    position index is 0, so the multiplier is exactly 0 there at no extra cost;
//    a product range that contains a start is therefore 0 inside the fold and the
//    scan alike (§3.4).
//  - Tokens past the row end get dt = 0 and u = 0, i.e. the identity (1, 0).
//  - When the states are saved for the backward and z is given, the kernel also
//    writes the factor (y + D u) d(z sigmoid(z))/dz of dout in dz (fp32), so that
//    the backward does not rebuild y.
//  - Long rows with few channels are split into segments scanned by different
//    blocks: an aggregate pass folds each segment into one map h -> P h + H per
//    (channel, state), and the main pass chains the maps before its segment and
//    starts from that state.
#include "common.hpp"
#include "launch.hpp"

namespace pm {
namespace {

constexpr int kN = 16;              // d_state
constexpr int kThreads = 256;
constexpr int kStride = 128;        // saved-state token stride (PACKMAMBA_STATE_STRIDE)

constexpr int kCH = 256;                // tokens per chunk

template <int LANES>
struct __attribute__((aligned(16))) FwdSmem {
    // [state][four of the lane's tokens][lane][token]: consecutive lanes read consecutive
    // 16-byte words.  The padding puts the words that 8 neighbouring threads stage, those of
    // the same lanes among them, into different banks (4 x 2048 x 1536 fp32: 110 -> 108 us).
    static constexpr int K = kCH / LANES, kRows = kThreads / LANES;
    static constexpr int kStride4 = LANES + (LANES == 16 ? 2 : LANES == 32 ? 4 : 0);
    float B[kN][K / 4][kStride4][4];
    float C[kN][K / 4][kStride4][4];
    float M[K / 4][kStride4][4];   // 0, or -inf on a sequence start
    float A2[kRows][kN];        // A * log2(e)
    float carry[kRows][kN];     // state after the previous chunk
    float pseg[kRows][kN];      // aggregate pass: product of the multipliers so far
};

struct FwdParams {
    const void* u;
    const void* delta;
    const float* A;
    const void* B;
    const void* C;
    const float* D;
    const void* z;
    const float* delta_bias;
    const int32_t* pos;
    void* out;
    float* states;
    float* dzf;               // (batch, dim, L): factor of dout in dz, or null
    const float* h0;          // state before each row (batch, dim, kN), or null; the main pass of
                              // split rows reads `entry`
    float* entry;             // split rows: copy of h0, by the aggregate pass
    float* hfinal;            // state after each row (batch, dim, kN), or null; may be h0's buffer
    float2* agg;              // the segments' maps (batch, dim, nseg, kN) = (P, H): written by the
                              // aggregate pass, chained by the main pass
    int64_t dim, L;
    int64_t seg_chunks;       // chunks per segment
    int nseg;
    int nchunk_states;
    int softplus;
};

// The state before segment `seg`: the maps h -> P h + H of the segments before it applied
// to h, the row's initial state.  Each block chains its own: a few loads that do not wait
// for one another, against a launch of its own for a carry pass (5 us).
__device__ __forceinline__ float chain_maps(const float2* __restrict__ maps, int seg, float h) {
    int s = 0;
    for (; s + 8 <= seg; s += 8) {
        float2 m[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) m[i] = maps[(int64_t)(s + i) * kN];
#pragma unroll
        for (int i = 0; i < 8; ++i) h = fmaf(m[i].x, h, m[i].y);
    }
    for (; s < seg; ++s) {
        const float2 m = maps[(int64_t)s * kN];
        h = fmaf(m.x, h, m.y);
    }
    return h;
}

// AGG: aggregate pass over one segment (no C, no outputs), writes its map (P, H).
template <typename T, typename TO, int LANES, bool AGG>
__global__ __launch_bounds__(kThreads, LANES == 16 ? 3 : 1) void scan_fwd_kernel(FwdParams p) {
    constexpr int PV = Storage<T>::kPerVec;
    using Smem = FwdSmem<LANES>;
    constexpr int K = Smem::K, kRows = Smem::kRows, CH = kCH;
    constexpr bool AHEAD = LANES > 16;            // registers to spare: load a chunk ahead
    __shared__ Smem sm;

    const int tid = threadIdx.x;
    const int j = tid & (LANES - 1);              // lane position inside the channel's group
    const int r = tid / LANES;                    // channel inside the block
    const int64_t b = blockIdx.y;
    const int seg = blockIdx.z;
    const int64_t d_raw = (int64_t)blockIdx.x * kRows + r;
    const bool active = d_raw < p.dim;
    const int64_t d = active ? d_raw : p.dim - 1;
    const int64_t L = p.L;
    const int64_t rowoff = (b * p.dim + d) * L;

    const T* ur = static_cast<const T*>(p.u) + rowoff;
    const T* dr = static_cast<const T*>(p.delta) + rowoff;
    const T* zr = p.z ? static_cast<const T*>(p.z) + rowoff : nullptr;
    TO* orow = p.out ? static_cast<TO*>(p.out) + rowoff : nullptr;
    const T* Bb = static_cast<const T*>(p.B) + b * kN * L;
    const T* Cb = static_cast<const T*>(p.C) + b * kN * L;
    const int32_t* pr = p.pos + b * L;

    if (tid < kRows * kN) {
        const int rr = tid >> 4, n = tid & 15;
        const int64_t dd = min((int64_t)blockIdx.x * kRows + rr, p.dim - 1);
        sm.A2[rr][n] = p.A[dd * kN + n] * kLog2e;
        float c0v = 0.0f;
        if (!AGG) {
            if (p.h0) c0v = p.h0[(b * p.dim + dd) * kN + n];
            c0v = chain_maps(p.agg + (b * p.dim + dd) * p.nseg * kN + n, seg, c0v);
        } else if (seg == 0 && p.h0) {
            // The main pass's blocks each start from h0, and the last segment's write hfinal,
            // which may be the same memory (a serving loop that updates its states in place).
            p.entry[(b * p.dim + dd) * kN + n] = p.h0[(b * p.dim + dd) * kN + n];
        }
        sm.carry[rr][n] = c0v;
        sm.pseg[rr][n] = 1.0f;
    }
    const float Dd = p.D ? p.D[d] : 0.0f;
    const float dbias = p.delta_bias ? p.delta_bias[d] : 0.0f;

    const int64_t nchunk = (L + CH - 1) / CH;
    // The inputs of one chunk that this thread loads, as stored: its own tokens of u, delta and
    // z, its part of the block's B and C, and a position index.  A chunk that crosses the row
    // end is loaded so too where there are registers for it (!AHEAD).
    constexpr int NB = kN * CH / (kThreads * PV);
    constexpr bool EARLY = AHEAD || NB == 2;      // B and C too before anything is staged
    struct Inputs {
        RawRun<T, K> u, d, z;
        RawRun<T, PV> b[NB], c[NB];
        int pos;
    } in;
    const auto load_inputs = [&](auto full_tag, int64_t c) {
        constexpr bool FULL = decltype(full_tag)::value;
        const int64_t lb = c * CH, l0 = lb + (int64_t)j * K;
        in.u = load_part<T, K, FULL>(ur, l0, L);
        in.d = load_part<T, K, FULL>(dr, l0, L);
        if (AHEAD && !AGG && zr) in.z = load_part<T, K, FULL>(zr, l0, L);
#pragma unroll
        for (int i = 0; i < (EARLY ? NB : 0); ++i) {
            const int idx = (i * kThreads + tid) * PV, n = idx / CH, t = idx - n * CH;
            in.b[i] = load_part<T, PV, FULL>(Bb + (int64_t)n * L, lb + t, L);
            if (!AGG) in.c[i] = load_part<T, PV, FULL>(Cb + (int64_t)n * L, lb + t, L);
        }
        in.pos = FULL || lb + tid < L ? pr[lb + tid] : 1;
    };
    // One chunk; FULL (block-uniform) means the chunk lies inside the row, so every load
    // and store is unconditional.  `next`: the chunk to load ahead of the state loop, or -1.
    auto chunk = [&](auto full_tag, const int64_t c, const int64_t next) {
        constexpr bool FULL = decltype(full_tag)::value;
        const int64_t lb = c * CH;
        const int64_t l0 = lb + (int64_t)j * K;
        constexpr bool RAW = FULL || !AHEAD;      // the inputs are in `in`
        // this lane's inputs, loaded first so that their latency overlaps the staging below
        if constexpr (!AHEAD) load_inputs(full_tag, c);
        // ---- stage B, C and the reset mask of this chunk in LDS ----
        static_assert(kThreads == CH, "a thread stages one position index");
#pragma unroll(EARLY ? NB : 1)
        for (int i = 0; i < NB; ++i) {
            const int idx = (i * kThreads + tid) * PV, n = idx / CH, t = idx - n * CH;
            float vb[PV], vc[PV];
            const T* const br = Bb + (int64_t)n * L;
            const T* const cr = Cb + (int64_t)n * L;
            RawRun<T, PV> rb, rc;
            if constexpr (RAW && EARLY) {
                rb = in.b[i];
                rc = in.c[i];
            } else {
                rb = load_part<T, PV, FULL>(br, lb + t, L);
                if (!AGG) rc = load_part<T, PV, FULL>(cr, lb + t, L);
            }
            unpack_part<T, PV, FULL>(rb, br, lb + t, L, vb);
            if (!AGG) unpack_part<T, PV, FULL>(rc, cr, lb + t, L, vc);
#pragma unroll
            for (int q = 0; q < PV; q += 4) {
                const int h = (t + q) % K / 4, l = (t + q) / K;
                *reinterpret_cast<f32x4*>(sm.B[n][h][l]) = f32x4{vb[q], vb[q + 1], vb[q + 2], vb[q + 3]};
                if (!AGG) *reinterpret_cast<f32x4*>(sm.C[n][h][l]) = f32x4{vc[q], vc[q + 1], vc[q + 2], vc[q + 3]};
            }
        }
        const int ps = RAW ? in.pos : lb + tid < L ? pr[lb + tid] : 1;
        sm.M[tid % K / 4][tid / K][tid % 4] = ps == 0 ? -INFINITY : 0.0f;
        __syncthreads();

        // ---- per-token inputs of this lane ----
        float dt[K], du[K], y[K], M[K];
        {
            float uv[K];
            if constexpr (RAW) {
                unpack_part<T, K, FULL>(in.u, ur, l0, L, uv);
                unpack_part<T, K, FULL>(in.d, dr, l0, L, dt);
            } else {
                const RawRun<T, K> ru = load_part<T, K, FULL>(ur, l0, L), rd = load_part<T, K, FULL>(dr, l0, L);
                unpack_part<T, K, FULL>(ru, ur, l0, L, uv);
                unpack_part<T, K, FULL>(rd, dr, l0, L, dt);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float s = dt[k] + dbias;
                float v = p.softplus ? softplus_f(s) : s;
                if (!FULL) v = (l0 + k < L) ? v : 0.0f;   // identity past the row end
                dt[k] = v;
                du[k] = v * uv[k];
                y[k] = Dd * uv[k];
            }
#pragma unroll
            for (int k = 0; k < K; k += 4) {
                const f32x4 m = *reinterpret_cast<const f32x4*>(sm.M[k / 4][j]);
                M[k] = m.x; M[k + 1] = m.y; M[k + 2] = m.z; M[k + 3] = m.w;
            }
        }
        // the next chunk's inputs, on their way while this one's states are worked through
        const RawRun<T, K> wz = in.z;
        if (AHEAD && next >= 0) load_inputs(std::true_type{}, next);
        // product of the lane's multipliers as one exp2 (0 if the lane holds a start)
        float S = 0.0f, Mf = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) { S += dt[k]; Mf += M[k]; }

        // ---- states ----
#pragma unroll 1
        for (int n = 0; n < kN; ++n) {
            // aggregate: a (channel, state) whose multiplier product is already exactly 0
            // is final; the wave skips the state when that holds for all its channels
            if (AGG && __all(sm.pseg[r][n] == 0.0f)) continue;
            const float A2n = sm.A2[r][n];
            const float cin = sm.carry[r][n];
            float a[K], bx[K];
            f32x4 bv[K / 4];
#pragma unroll
            for (int k = 0; k < K / 4; ++k) bv[k] = *reinterpret_cast<const f32x4*>(sm.B[n][k][j]);
            // all four reads first: left to itself, the scheduler issues the last two after the
            // first two have been used (8 x 200 x 4096, fp32 54 -> 49 us, bf16 54 -> 41)
            if (LANES == 16) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < K; k += 4) {
                const float bb[4] = {bv[k / 4].x, bv[k / 4].y, bv[k / 4].z, bv[k / 4].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    a[k + q] = fast_exp2(fmaf(dt[k + q], A2n, M[k + q]));
                    bx[k + q] = du[k + q] * bb[q];
                }
            }
            // fold the lane's K tokens into one affine map h -> P h + H
            float H = bx[0];
#pragma unroll
            for (int k = 1; k < K; ++k) H = fmaf(a[k], H, bx[k]);
            float P = fast_exp2(fmaf(S, A2n, Mf));
            lane_scan_up<LANES>(P, H);
            if (AGG) {
                // the last lane's (P, H) is the chunk's map; the chunks after it are already
                // composed in (pseg, carry), which becomes (pseg P, pseg H + carry)
                if (j == LANES - 1) {
                    const float pa = sm.pseg[r][n];
                    sm.carry[r][n] = fmaf(pa, H, sm.carry[r][n]);
                    sm.pseg[r][n] = pa * P;
                }
                continue;
            }
            const float hend = fmaf(P, cin, H);               // state after this lane's last token
            float h = dpp<LANES == 16 ? kRowShr1 : kWaveShr1>(cin, hend);   // state before this lane's first token
            if (LANES == 32) h = j == 0 ? cin : h;            // lane 32's came from the other channel
            if (j == LANES - 1) sm.carry[r][n] = hend;               // state after the chunk
#pragma unroll
            for (int k = 0; k < K; k += 4) {
                const f32x4 cv = *reinterpret_cast<const f32x4*>(sm.C[n][k / 4][j]);
                const float cc[4] = {cv.x, cv.y, cv.z, cv.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    h = fmaf(a[k + q], h, bx[k + q]);
                    y[k + q] = fmaf(cc[q], h, y[k + q]);
                }
            }
            // saved states: h after every kStride-th token
            if (p.states && active && (((j + 1) * K) % kStride) == 0) {
                const int64_t sc = (l0 + K) / kStride - 1;
                if (sc < p.nchunk_states)
                    p.states[((b * p.dim + d) * p.nchunk_states + sc) * kN + n] = hend;
            }
        }

        // ---- gate and store; for the backward, the factor of dout in dz ----
        if (!AGG && active && (orow || p.dzf)) {
            if (zr) {
                float zv[K], g[K];
                if constexpr (FULL && AHEAD) unpack_run(wz, zv);
                else unpack_part<T, K, FULL>(load_part<T, K, FULL>(zr, l0, L), zr, l0, L, zv);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const float sz = sigmoid_f(zv[k]);
                    g[k] = y[k] * sz * (1.0f + zv[k] * (1.0f - sz));   // y d(z sigmoid(z))/dz
                    y[k] = y[k] * zv[k] * sz;
                }
                if (p.dzf) {
                    // padded row: whole vectors, also in a chunk that crosses the row end
                    float* fr = p.dzf + (b * p.dim + d) * dzf_row_len(L);
#pragma unroll
                    for (int i = 0; i < K / 4; ++i)
                        __builtin_nontemporal_store(f32x4{g[4 * i], g[4 * i + 1], g[4 * i + 2], g[4 * i + 3]},
                                                    reinterpret_cast<f32x4*>(fr + dzf_vec(c, (j * K + 4 * i) % 16 / 4, (j * K + 4 * i) / 16)));
                }
            }
            if (orow) store_run<TO, K, FULL>(orow, l0, L, y);
        }
        __syncthreads();      // LDS is restaged for the next chunk
    };
    const int64_t c0 = (int64_t)seg * p.seg_chunks;
    const int64_t c1 = min(nchunk, c0 + p.seg_chunks);
    if (AGG) {
        // The aggregate composes the chunk maps from the segment's end backwards.  Once
        // the product of the multipliers is exactly 0 for every channel and state of the
        // block (a sequence start, or underflow of a long decay), the earlier chunks
        // contribute exactly nothing, and the walk stops.
        if (AHEAD) load_inputs(std::true_type{}, c1 - 1);   // (a segment that is aggregated lies inside the row)
        for (int64_t c = c1 - 1; c >= c0; --c) {
            chunk(std::true_type{}, c, c > c0 ? c - 1 : -1);
            if (!__syncthreads_or(tid < kRows * kN && sm.pseg[0][tid] != 0.0f)) break;
        }
    } else {
        const int64_t full = L / CH;              // chunks that lie inside the row
        if (AHEAD && c0 < full) load_inputs(std::true_type{}, c0);
        for (int64_t c = c0; c < c1; ++c) {
            if (c < full) chunk(std::true_type{}, c, c + 1 < min(c1, full) ? c + 1 : -1);
            else chunk(std::false_type{}, c, -1);
        }
    }
    if (AGG) {
        __syncthreads();
        const int rr = tid >> 4, n = tid & 15;
        const int64_t dd = (int64_t)blockIdx.x * kRows + rr;
        if (rr < kRows && dd < p.dim) {
            p.agg[((b * p.dim + dd) * p.nseg + seg) * kN + n] = float2{sm.pseg[rr][n], sm.carry[rr][n]};
        }
    } else if (p.hfinal && c1 == nchunk) {
        // the carry after the row's last chunk is h after its last token (tokens past
        // the row end are identities)
        const int rr = tid >> 4, n = tid & 15;
        const int64_t dd = (int64_t)blockIdx.x * kRows + rr;
        if (rr < kRows && dd < p.dim) p.hfinal[(b * p.dim + dd) * kN + n] = sm.carry[rr][n];
    }
}

// Short rows (a decode step's few tokens): a lane owns 4 states of one channel and walks
// the row token by token, the 4 lanes of a channel adding their parts of y by DPP.  At one
// token the pass is its states: each is read and written once, 16 bytes a lane, a wave
// 1 KB in a row.  B, C and the reset mask of the whole row are in LDS.
// 64 x 4096 channels, bf16, one token: 313 -> 9.0 us (4.0 TB/s), the chunk kernel's work
// being a whole 256-token chunk.  The walk is serial in the tokens: the rows it takes are in
// short_row().
constexpr int64_t kShortRow = 32;
constexpr int kShortCh = kThreads / 4;       // channels per block

template <typename T, typename TO>
__global__ __launch_bounds__(kThreads) void scan_fwd_short_kernel(FwdParams p) {
    __shared__ __attribute__((aligned(16))) float sB[kShortRow][kN], sC[kShortRow][kN];
    __shared__ float sM[kShortRow];
    const int tid = threadIdx.x;
    const int q = tid & 3;                                   // states 4q .. 4q+3
    const int64_t b = blockIdx.y;
    const int64_t d_raw = (int64_t)blockIdx.x * kShortCh + (tid >> 2);
    const bool active = d_raw < p.dim;
    const int64_t d = active ? d_raw : p.dim - 1;
    const int L = (int)p.L;
    const int64_t row = b * p.dim + d;
    const T* ur = static_cast<const T*>(p.u) + row * L;
    const T* dr = static_cast<const T*>(p.delta) + row * L;
    const T* zr = p.z ? static_cast<const T*>(p.z) + row * L : nullptr;
    TO* orow = p.out ? static_cast<TO*>(p.out) + row * L : nullptr;

    f32x4 h = {};
    if (p.h0) h = *reinterpret_cast<const f32x4*>(p.h0 + row * kN + 4 * q);
    const f32x4 A2 = *reinterpret_cast<const f32x4*>(p.A + d * kN + 4 * q) * kLog2e;
    const float Dd = p.D ? p.D[d] : 0.0f;
    const float dbias = p.delta_bias ? p.delta_bias[d] : 0.0f;
    float u = Storage<T>::load1(ur), dl = Storage<T>::load1(dr), z = zr ? Storage<T>::load1(zr) : 0.0f;
    const T* Bb = static_cast<const T*>(p.B) + b * kN * L;
    const T* Cb = static_cast<const T*>(p.C) + b * kN * L;
    for (int i = tid; i < kN * L; i += kThreads) {
        const int n = i / L, l = i - n * L;
        sB[l][n] = Storage<T>::load1(Bb + i);
        sC[l][n] = Storage<T>::load1(Cb + i);
    }
    if (tid < L) sM[tid] = p.pos[b * L + tid] == 0 ? -INFINITY : 0.0f;
    __syncthreads();

    for (int l = 0; l < L; ++l) {
        const float s = dl + dbias, uv = u, zv = z;
        if (l + 1 < L) {                                     // the next token's, ahead of this one's work
            u = Storage<T>::load1(ur + l + 1);
            dl = Storage<T>::load1(dr + l + 1);
            if (zr) z = Storage<T>::load1(zr + l + 1);
        }
        const float dt = p.softplus ? softplus_f(s) : s;
        const float du = dt * uv, m = sM[l];
        const f32x4 Bv = *reinterpret_cast<const f32x4*>(&sB[l][4 * q]);
        const f32x4 Cv = *reinterpret_cast<const f32x4*>(&sC[l][4 * q]);
        float y = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h[i] = fmaf(fast_exp2(fmaf(dt, A2[i], m)), h[i], du * Bv[i]);
            y = fmaf(Cv[i], h[i], y);
        }
        y += dpp<kQuadXor1>(0.0f, y);
        y += dpp<kQuadXor2>(0.0f, y);
        if (orow && active && q == 0) {
            y = fmaf(Dd, uv, y);
            if (zr) y *= zv * sigmoid_f(zv);
            Storage<TO>::store1(orow + l, y);
        }
    }
    if (p.hfinal && active) *reinterpret_cast<f32x4*>(p.hfinal + row * kN + 4 * q) = h;
}

// Lanes per channel of the aggregate pass, whatever the main pass has: a wave of two
// channels skips a state as soon as both are done, and its chains are half as long as with
// four (1 x 65536 x 2048 with three long sequences: the whole call 1171 -> 1037 us; 64
// lanes 1121, pieces of a quarter segment 1041).
constexpr int kAggLanes = 32;

template <typename T, typename TO, int LANES>
hipError_t launch_lanes(const ScanArgs& a, FwdParams p, hipStream_t s) {
    constexpr int kRows = FwdSmem<LANES>::kRows;
    const dim3 grid((unsigned)((a.dim + kRows - 1) / kRows), (unsigned)a.batch, (unsigned)p.nseg);
    if (p.nseg > 1) {
        // aggregate every segment but the last
        constexpr int kAggRows = FwdSmem<kAggLanes>::kRows;
        hipLaunchKernelGGL((scan_fwd_kernel<T, TO, kAggLanes, true>),
                           dim3((unsigned)((a.dim + kAggRows - 1) / kAggRows), grid.y, grid.z - 1), dim3(kThreads), 0, s, p);
        if (hipError_t e = hipGetLastError()) return e;
        if (p.h0) p.h0 = p.entry;
    }
    hipLaunchKernelGGL((scan_fwd_kernel<T, TO, LANES, false>), grid, dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

// Longest rows of the short kernel, where its time meets the chunk kernel's (us, chunk kernel
// second; both are latencies where blocks are few, 16 channels each): 4 blocks, 20 tokens 8.6,
// 9.3, 24 tokens 10.1, 8.5; 192 blocks, 24 tokens 10.4, 10.2, 28 tokens 12.0, 11.4; 384 blocks,
// 32 tokens 13.5, 13.4; 2048 blocks, 32 tokens 15, 43.  Its 4-byte loads of fp32 run through a
// line a tensor and channel, 32 tokens, that very many rows evict from the caches: 64 x 4096
// channels, 28 tokens 248, 311, 32 tokens 331, 312.
template <typename T>
int64_t short_row(const ScanArgs& a) {
    const int64_t blocks = a.batch * ((a.dim + 15) / 16);
    if (blocks < 128) return 20;
    if (blocks < 384) return 24;
    return std::is_same_v<T, float> && blocks >= 8192 ? 28 : kShortRow;
}

template <typename T, typename TO>
hipError_t launch_t(const ScanArgs& a, hipStream_t s) {
    static_assert(kCH == kDzfChunk, "the dz factor layout follows the forward's chunk");
    FwdParams p;
    p.u = a.u; p.delta = a.delta; p.A = a.A; p.B = a.B; p.C = a.C; p.D = a.D; p.z = a.z;
    p.delta_bias = a.delta_bias; p.pos = a.pos; p.out = a.out; p.states = a.states;
    p.dzf = a.z ? a.dzf : nullptr;
    p.h0 = a.h0; p.hfinal = a.hfinal;
    p.dim = a.dim; p.L = a.seqlen;
    p.nchunk_states = (int)((a.seqlen + kStride - 1) / kStride);
    p.softplus = a.softplus;
    if (a.seqlen <= short_row<T>(a) && !a.states) {
        hipLaunchKernelGGL((scan_fwd_short_kernel<T, TO>),
                           dim3((unsigned)((a.dim + kShortCh - 1) / kShortCh), (unsigned)a.batch), dim3(kThreads), 0, s, p);
        return hipGetLastError();
    }
    const FwdPlan plan = scan_fwd_plan(a.batch, a.dim, a.seqlen, std::is_same_v<T, float>);
    const SegPlan sp = plan.seg;
    static_assert(kSegUnit % kCH == 0, "segments hold whole chunks");
    p.seg_chunks = sp.seg_len / kCH;
    p.nseg = (int)sp.nseg;
    p.entry = a.ws_entry;
    p.agg = reinterpret_cast<float2*>(a.ws_agg);
    switch (plan.lanes) {
        case 64: return launch_lanes<T, TO, 64>(a, p, s);
        case 32: return launch_lanes<T, TO, 32>(a, p, s);
        default: return launch_lanes<T, TO, 16>(a, p, s);
    }
}

}  // namespace

hipError_t launch_scan_fwd(const ScanArgs& a, hipStream_t s) {
    switch (a.dtype) {
        case 1: return launch_t<bf16_t, bf16_t>(a, s);
        case 2: return launch_t<bf16_t, float>(a, s);
        default: return launch_t<float, float>(a, s);
    }
}

}  // namespace pm
