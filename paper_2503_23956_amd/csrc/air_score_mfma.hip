// air_score, bf16: the window-query x visual-key product (Eq.6-7) on MFMA, heads of 64 or 128 elements.
//
// A workgroup of 4 waves owns one 256-key chunk of one unit (layer, sequence, KV head); each
// wave keeps its 64 keys (4 tiles of 16) in registers as MFMA B operands, loaded straight from
// global memory: lane (n = lane % 16, c = lane / 16) holds the c-th 16 bytes of every 64-byte
// slice of key n of the tile (air_tile.h).  The elite rows of the G query heads of the group are the A
// operand, 16 rows per block, so that S[row][key] comes out with lane (key n, c) holding four
// rows of key n: the sum over window rows that Eq.8 needs is then in-lane plus two cross-lane
// steps.
//
// Eq.8 needs every row's softmax normaliser before any column can be finished, and the
// normaliser needs all keys.  Three kernels:
//
//   score_stream_kernel  reads K_v ONCE.  Per (row, chunk) it leaves the chunk maximum m and
//       sum-exp z; when the unit has at most kStashRows window rows (the elite window: a few
//       rows per head) it also stashes e = exp(s - m) per (row, key) in fp32, 4 bytes per row
//       and key against the 256 bytes of the key itself.
//   score_rows_mfma_kernel  per row: M = max over chunks (and over the elite-text columns),
//       Z = sum z exp(m - M), weight w = 1 / (R_h G Z).  Launched for windows that turn their
//       whole span into rows (up to 32 of them); the elite window's rows are done inside the finish kernel.
//   score_finish_kernel  units with a stash never touch K again:
//       I[key] = sum_rows e[row][key] * (w exp(m_chunk - M)).  Units with more rows (a low threshold; windows without one
//       have a kernel of their own, air_score_window.hip) recompute their logits from K_v: I[key] = sum_rows w exp(s - M).
//       Epilogue: the workgroup's sum of I and its second and third moments about the workgroup's own
//       mean (fp64); the unit's last workgroup to finish shifts the entries to the row mean and adds them
//       up for Eq.9-10 (raw power sums would cancel on rows of little spread: S2 - S1 mu loses
//       (mu / sigma)^2 of its digits), and, where the layers fit one wave, the last unit of a sequence
//       goes on to Eq.11 and the cache layout (air_budget_dev.h).
#include "air_device.h"
#include "air_internal.h"
#include "air_score_mfma_dev.h"
#include <type_traits>

namespace air {

constexpr int kRowsLds = 512;  // rows whose (M, w) are staged in LDS at a time (recompute path)

// keys of one wave: tiles of 16, as MFMA B operands.  Keys past the end of the visual span re-read
// the last one (no predication in front of the loads); `valid` masks their logits.
template <int NS>
__device__ __forceinline__ void load_keys(const UnitCtx &u, const air_strides &st, int key0, int n, int c,
                                          uint4 (&kreg)[4][NS], bool (&valid)[4]) {
#pragma unroll
    for (int tile = 0; tile < 4; ++tile) {
        const int key = key0 + 16 * tile + n;
        valid[tile] = key < u.sq.vis_len;
        const bf16_t *src = u.k + (int64_t)(u.sq.vis_start + min(key, u.sq.vis_len - 1)) * st.kv_t + 8 * c;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) kreg[tile][sl] = *reinterpret_cast<const uint4 *>(src + 32 * sl);
    }
}

// RAW logits (dot products, before the 1/sqrt(d) scale) of a block of 16 rows against the wave's 64
// keys: lane (key n, c) gets rows rbase + 4i + c.  Maxima are taken and exchanged in raw units and
// the scale is folded into the exponential, exp((s - M) / sqrt(d)) = 2^((s - M) * kC).
template <int NS>
__device__ __forceinline__ void logits_of(const uint4 (&qa)[NS], const uint4 (&kreg)[4][NS], f32x4 (&s)[4]) {
#pragma unroll
    for (int tile = 0; tile < 4; ++tile) {
        s[tile] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) s[tile] = mma<bf16_t>(qa[sl], kreg[tile][sl], s[tile]);
    }
}

template <int NS>
__device__ __forceinline__ void block_logits(const DevTables &t, const UnitCtx &u, const air_strides &st,
                                             const int *s_pref, int rbase, int n, int c, const uint4 (&kreg)[4][NS],
                                             f32x4 (&s)[4]) {
    uint4 qa[NS];
    load_rows(t, u, st, s_pref, rbase, n, c, qa);
    logits_of(qa, kreg, s);
}

// ---------------------------------------------------------------------------------------
// One workgroup per 256-key chunk of a unit.
// Stash layout of one (unit, chunk, row): 256 floats, key 64w + 16 tile + n at position 64w + 4n + tile,
// i.e. the four tiles of a lane are one 16-byte store.
// VIS: the rows are the tokens of a visual window (all heads have the same win_len rows); row rho sits at
// visual index prow0 + rho % win_len and sees the keys up to itself.  A (row, chunk) pair that lies wholly
// behind the row leaves the partial (-inf, 0) and zeros in the stash.
template <int D, bool VIS>
__global__ __launch_bounds__(256, 4) void score_stream_kernel(Dims dm, DevTables t, int l0, LaunchLayers ll,
                                                              air_strides st, SeqArgs seqs) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, c = lane >> 4;
    constexpr int NS = D / 32;
    UnitCtx u;
    if (!unit_setup(dm, seqs, l0, ll, st, u, 1)) return;
    __shared__ int s_pref[17];
    __shared__ float s_pm[4][16], s_pz[4][16], s_mw[16];

    const int chunk = u.chunk;
    uint4 kreg[4][NS];
    bool valid[4];
    load_keys(u, st, chunk * kChunkKeys + wave * 64, n, c, kreg, valid);
    head_prefix(t, u.hrow0, u.G, s_pref);
    u.R_total = s_pref[u.G];
    const bool stash = u.R_total <= kStashRows;
    uint4 qa0[NS];
    load_rows(t, u, st, s_pref, 0, n, c, qa0);

    {
        float *stash_base = t.stash + ((u.unit * dm.n_chunks + chunk) * (int64_t)kStashRows) * kChunkKeys;
        // per (row, chunk) maximum and sum-exp of the block of 16 rows that starts at list row rb, from its logits
        auto reduce_block = [&](int rb, f32x4 (&s)[4]) __attribute__((always_inline)) {
            const int n_i = min(4, (u.R_total - rb + 3) >> 2);  // live values of i (uniform over the workgroup)
            int lim[4];  // VIS: last key of the lane's tiles that row i sees, relative to the lane's key of tile 0
#pragma unroll
            for (int i = 0; i < 4; ++i)
                lim[i] = VIS ? (u.sq.win_start - u.sq.vis_start) + (rb + 4 * i + c) % u.sq.win_len -
                                   (chunk * kChunkKeys + wave * 64 + n)
                             : 0;
            auto live = [&](int tile, int i) __attribute__((always_inline)) {
                return VIS ? (valid[tile] && 16 * tile <= lim[i]) : valid[tile];
            };
            float m[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                m[i] = -INFINITY;
                if (i >= n_i) continue;
                float mx = -INFINITY;
#pragma unroll
                for (int tile = 0; tile < 4; ++tile) mx = fmaxf(mx, live(tile, i) ? s[tile][i] : -INFINITY);
                m[i] = max16(mx);
            }
            lds_barrier();
            if (n == 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) s_pm[wave][4 * i + c] = m[i];  // indexed by list row within the block
            }
            lds_barrier();
            // chunk maximum of every row: the reference of the stashed exponentials
            float z[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                z[i] = 0.f;
                if (i >= n_i) continue;
                const int r = 4 * i + c;
                const float M = fmaxf(fmaxf(s_pm[0][r], s_pm[1][r]), fmaxf(s_pm[2][r], s_pm[3][r]));
                f32x4 e;
#pragma unroll
                for (int tile = 0; tile < 4; ++tile) e[tile] = live(tile, i) ? exp_key<D>(s[tile][i] - M) : 0.f;
                float zz = (e[0] + e[1]) + (e[2] + e[3]);
                if (stash && rb + r < u.R_total)
                    // read once, by the next kernel: marked so.  us for air_score marked / plain: one layer of 576 ... 16384 tokens and
                    // one prompt of them in 28 layers no difference (29.7 / 29.7, 65.5 / 65.4, 135.0 / 134.9), four of 2304 81.2 / 81.5,
                    // eight 157 / 161, sixteen 302 / 310, four of 6272 201 / 204, two of 16384 in 32 layers of 8 KV heads
                    // 552 / 571.  Marking the key loads costs 1-11 %.
                    __builtin_nontemporal_store(e, reinterpret_cast<f32x4 *>(stash_base + (int64_t)(rb + r) * kChunkKeys + wave * 64 + 4 * n));
                z[i] = sum16(zz);
                if (wave == 0 && n == 0) s_mw[r] = M;
            }
            if (n == 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) s_pz[wave][4 * i + c] = z[i];
            }
            lds_barrier();
            if (tid < 16 && rb + tid < u.R_total) {
                const int rho = rb + tid;
                const float Z = (s_pz[0][tid] + s_pz[1][tid]) + (s_pz[2][tid] + s_pz[3][tid]);
                const int g = head_of_row(s_pref, u.G, rho);
                const int64_t slot = (u.hrow0 + g) * u.W + (rho - s_pref[g]);
                t.part[slot * dm.n_chunks + chunk] = make_float2(s_mw[tid], Z);
            }
        };
        for (int rb = 0; rb < u.R_total; rb += 16) {
            f32x4 s[4];
            if (rb == 0) logits_of(qa0, kreg, s);
            else block_logits(t, u, st, s_pref, rb, n, c, kreg, s);
            reduce_block(rb, s);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Parameters of one window row, by one wave (every lane gets the result): M = max over the chunk
// partials and the elite-text columns (raw units), Z = sum z exp(m - M) in fp64, w = 1 / (R_h G Z).
// p0 returns the lane's own partial of the first 64 chunks.  A partial with sum 0 (a chunk wholly
// behind a visual-window row; the empty text columns of such a window) has maximum -inf and takes no part.
template <int D>
__device__ __forceinline__ void row_params(const DevTables &t, int64_t slot, int nch, int n_chunks, int rows_of_head, int G,
                                           int lane, float &M, float &w, float2 &p0) {
    const float2 *p = t.part + slot * n_chunks;
    const float mt = t.row_mtext[slot], zt = t.row_ztext[slot];
    p0 = lane < nch ? p[lane] : make_float2(-INFINITY, 0.f);  // the first 64 chunks stay in registers
    M = fmaxf(mt, p0.x);
    for (int cc = lane + 64; cc < nch; cc += 64) M = fmaxf(M, p[cc].x);
    M = wave_max(M);
    double Z = lane < nch && p0.y > 0.f ? (double)(p0.y * exp_raw<D>(p0.x - M)) : 0.0;
    for (int cc = lane + 64; cc < nch; cc += 64) {
        const float2 x = p[cc];
        if (x.y > 0.f) Z += (double)(x.y * exp_raw<D>(x.x - M));
    }
    Z = wave_sum(Z);
    if (zt > 0.f) Z += (double)(zt * exp_raw<D>(mt - M));
    w = (float)(1.0 / ((double)rows_of_head * (double)G * Z));
}
// the factor that turns a stashed exponential of a chunk into its share of Eq.8
template <int D>
__device__ __forceinline__ float chunk_factor(float2 part, float M, float w) {
    return part.y > 0.f ? w * exp_raw<D>(part.x - M) : 0.f;
}

// ---------------------------------------------------------------------------------------
// Row parameters, once per unit: one wave per window row, lanes over the chunk partials.
// M = max over chunks and the elite-text columns, Z = sum z exp(m - M) in fp64,
// w = 1 / (R_h G Z).  Units with a stash also get f[row][chunk] = w exp(m_chunk - M), the factor
// that turns a stashed exponential into its share of Eq.8.
constexpr int kRowWaves = 16;  // up to one wave per row: a unit's usual dozen rows are then done in one round of loads
template <int D>
__global__ __launch_bounds__(64 * kRowWaves) void score_rows_mfma_kernel(Dims dm, DevTables t, int l0, SeqArgs seqs) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int kvh = blockIdx.x, b = blockIdx.y, l = l0 + (int)blockIdx.z;  // grid (KV head, sequence, layer)
    const int G = dm.G, W = dm.max_window;
    const int64_t hrow0 = ((int64_t)l * dm.B + b) * dm.Hq + (int64_t)kvh * G;
    const int64_t unit = ((int64_t)l * dm.B + b) * dm.Hkv + kvh;
    const int nch = (seqs.s[b].vis_len + kChunkKeys - 1) / kChunkKeys;
    __shared__ int s_pref[17];
    head_prefix(t, hrow0, G, s_pref);
    const int R_total = s_pref[G];
    const bool stash = R_total <= kStashRows;
    if (tid == 0) t.unit_R[unit] = R_total;
    for (int rho = wave; rho < R_total; rho += (int)(blockDim.x >> 6)) {
        const int g = head_of_row(s_pref, G, rho);
        const int64_t slot = (hrow0 + g) * W + (rho - s_pref[g]);
        const float2 *p = t.part + slot * dm.n_chunks;
        float M, w;
        float2 p0;
        row_params<D>(t, slot, nch, dm.n_chunks, s_pref[g + 1] - s_pref[g], G, lane, M, w, p0);
        if (lane == 0) {
            t.row_M[slot] = M;  // raw units
            t.row_w[slot] = w;
        }
        if (stash) {
            float *f = t.row_f + (unit * kStashRows + rho) * dm.n_chunks;
            if (lane < nch) f[lane] = chunk_factor<D>(p0, M, w);
            for (int cc = lane + 64; cc < nch; cc += 64) f[cc] = chunk_factor<D>(p[cc], M, w);
        }
    }
}

// ---------------------------------------------------------------------------------------
// One workgroup finishes kFinishChunks consecutive chunks of a unit and leaves one moment entry.
// INLINE: no row-parameter kernel has run; every workgroup forms the parameters of the unit's rows
// itself from the chunk partials (the elite window's handful of rows: cheaper than a launch).

template <int D, bool VIS, bool INLINE>
__global__ __launch_bounds__(256, 4) void score_finish_kernel(Dims dm, DevTables t, int l0, LaunchLayers ll,
                                                           air_strides st, SeqArgs seqs) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, c = lane >> 4;
    constexpr int NS = D / 32;
    UnitCtx u;
    if (!unit_setup(dm, seqs, l0, ll, st, u, kFinishChunks)) return;
    __shared__ int s_pref[17];
    __shared__ float s_M[kRowsLds], s_w[kRowsLds];
    __shared__ float s_f[kFinishChunks][kStashRows];
    __shared__ double s_mom[4][3];

    const int nch = (u.sq.vis_len + kChunkKeys - 1) / kChunkKeys;
    const int first = u.chunk, last = min(nch, first + kFinishChunks);
    // factor table of the stash path goes out before anything else; rows past R_total are never used
    float f_mine = 0.f;
    if (!INLINE) {
        if (tid < kFinishChunks * kStashRows && first + tid / kStashRows < last)
            f_mine = t.row_f[(u.unit * kStashRows + (tid % kStashRows)) * dm.n_chunks + first + tid / kStashRows];
        u.R_total = t.unit_R[u.unit];
    } else {
        head_prefix(t, u.hrow0, u.G, s_pref);
        u.R_total = s_pref[u.G];
    }
    const bool stash = u.R_total <= kStashRows;
    if (!INLINE && !stash) head_prefix(t, u.hrow0, u.G, s_pref);

    const int n_wg = min(u.sq.vis_len, last * kChunkKeys) - first * kChunkKeys;  // scores of this workgroup
    const int n_ent = (nch + kFinishChunks - 1) / kFinishChunks;                 // workgroups of this unit
    auto put_moments = [&](const auto &x, const auto &ok) __attribute__((always_inline)) {
        leave_moments(dm, t, u.unit, u.b, u.sq, n_wg, n_ent, x, ok, s_mom);
    };

    if (stash) {
        // factors f[chunk][row] into LDS: read from the table the row-parameter kernel left, or formed
        // here, a wave per row (rows past the list get zero)
        auto put_factors = [&]() __attribute__((always_inline)) {
            if (!INLINE) {
                if (tid < kFinishChunks * kStashRows) s_f[tid / kStashRows][tid % kStashRows] = (tid % kStashRows) < u.R_total ? f_mine : 0.f;
            } else {
                // a row of 16 lanes per window row (16 rows at a time), a lane takes every 16th chunk
                // partial: all loads of a round go out together and the reductions stay inside the row
                if (tid < kFinishChunks * kStashRows && (tid % kStashRows) >= u.R_total) s_f[tid / kStashRows][tid % kStashRows] = 0.f;
                const int grp = tid >> 4, gl = tid & 15;
                for (int r0 = 0; r0 < u.R_total; r0 += 16) {
                    const int rho = min(r0 + grp, u.R_total - 1);  // a row group past the list repeats the last row and stores nothing
                    const int g = head_of_row(s_pref, u.G, rho);
                    const int64_t slot = (u.hrow0 + g) * u.W + (rho - s_pref[g]);
                    const float2 *p = t.part + slot * dm.n_chunks;
                    const float mt = t.row_mtext[slot], zt = t.row_ztext[slot];
                    const float2 pf = p[min(first + gl, nch - 1)];  // the partial a factor is made of (lanes 0 .. 3)
                    float2 pc[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) pc[k] = gl + 16 * k < nch ? p[gl + 16 * k] : make_float2(-INFINITY, 0.f);
                    float M = mt;
#pragma unroll
                    for (int k = 0; k < 4; ++k) M = fmaxf(M, pc[k].x);
                    for (int cc = gl + 64; cc < nch; cc += 16) M = fmaxf(M, p[cc].x);
                    M = max16(M);
                    double Z = 0.0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) Z += pc[k].y > 0.f ? (double)(pc[k].y * exp_raw<D>(pc[k].x - M)) : 0.0;
                    for (int cc = gl + 64; cc < nch; cc += 16) {
                        const float2 x = p[cc];
                        if (x.y > 0.f) Z += (double)(x.y * exp_raw<D>(x.x - M));
                    }
                    Z = sum16(Z);
                    if (zt > 0.f) Z += (double)(zt * exp_raw<D>(mt - M));
                    const float w = (float)(1.0 / ((double)(s_pref[g + 1] - s_pref[g]) * (double)u.G * Z));
                    if (r0 + grp < u.R_total && gl < kFinishChunks) s_f[gl][rho] = first + gl < last ? chunk_factor<D>(pf, M, w) : 0.f;
                }
            }
            lds_barrier();
        };
        // One wave per chunk; a lane takes 16 bytes of every stashed row (four keys, 16 apart: see
        // stash_pos) and all rows of a round are requested at once, in front of the factors.  Rows past
        // the list re-read its last row against a zero factor, a wave past the last chunk re-reads the
        // last chunk and stores nothing.
        const int ci = wave, chunk = first + ci;
        const float *sb = t.stash + ((u.unit * dm.n_chunks + min(chunk, last - 1)) * (int64_t)kStashRows) * kChunkKeys + 4 * lane;
        f32x4 imp = (f32x4){0.f, 0.f, 0.f, 0.f};
        auto get_rows = [&](auto &e, int r0) __attribute__((always_inline)) {
            constexpr int RB = sizeof(e) / sizeof(e[0]);
#pragma unroll
            for (int r = 0; r < RB; ++r)
                e[r] = *reinterpret_cast<const f32x4 *>(sb + (int64_t)min(r0 + r, max(u.R_total - 1, 0)) * kChunkKeys);
        };
        auto add_rows = [&](const auto &e, int r0) __attribute__((always_inline)) {
            constexpr int RB = sizeof(e) / sizeof(e[0]);
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const float f = s_f[ci][r0 + r];
#pragma unroll
                for (int i = 0; i < 4; ++i) imp[i] = fmaf(f, e[r][i], imp[i]);
            }
        };
        static_assert(kFinishChunks == 4, "one wave of the workgroup per chunk");
        static_assert(kStashRows == 32, "rows beyond 16 are taken in a second round of 16");
        bool ok[4] = {false, false, false, false};
        if (u.R_total == 0) {  // no window row: the importance is zero (and so are its moments)
            for (int key = first * kChunkKeys + tid; key < min(last * kChunkKeys, u.sq.vis_len); key += 256)
                t.scores[u.unit * dm.max_vis + key] = 0.f;
        } else {
            // 16 rows in flight at most: 32 at once would cost the kernel half of its occupancy
            if (u.R_total <= 8) {
                f32x4 e[8];
                get_rows(e, 0);
                put_factors();
                add_rows(e, 0);
            } else {
                f32x4 e[16];
                get_rows(e, 0);
                put_factors();
                add_rows(e, 0);
                if (u.R_total > 16) {
                    get_rows(e, 16);
                    add_rows(e, 16);
                }
            }
            if (chunk < last) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int key = chunk * kChunkKeys + 64 * (lane >> 4) + 16 * i + (lane & 15);
                    ok[i] = key < u.sq.vis_len;
                    if (ok[i]) t.scores[u.unit * dm.max_vis + key] = imp[i];
                }
            }
        }
        const float xs[4] = {imp[0], imp[1], imp[2], imp[3]};
        put_moments(xs, ok);
        return;
    }
    if constexpr (VIS) return;  // not reached: visual windows of more rows go to the kernel for many rows
    // recompute path: (M, w) of a block of rows staged from the row tables
    auto stage_rows = [&](int rs, int rows) {
        __syncthreads();
        if (!INLINE) {
            for (int rr = tid; rr < rows; rr += 256) {
                const int rho = rs + rr;
                const int g = head_of_row(s_pref, u.G, rho);
                const int64_t slot = (u.hrow0 + g) * u.W + (rho - s_pref[g]);
                s_M[rr] = t.row_M[slot];
                s_w[rr] = t.row_w[slot];
            }
        } else {
            for (int rr = wave; rr < rows; rr += 4) {
                const int rho = rs + rr;
                const int g = head_of_row(s_pref, u.G, rho);
                const int64_t slot = (u.hrow0 + g) * u.W + (rho - s_pref[g]);
                float M, w;
                float2 p0;
                row_params<D>(t, slot, nch, dm.n_chunks, s_pref[g + 1] - s_pref[g], u.G, lane, M, w, p0);
                if (lane == 0) {
                    s_M[rr] = M;
                    s_w[rr] = w;
                }
            }
        }
        __syncthreads();
    };
    for (int chunk = first; chunk < last; ++chunk) {
        const int key0 = chunk * kChunkKeys + wave * 64;
        uint4 kreg[4][NS];
        bool valid[4];
        load_keys(u, st, key0, n, c, kreg, valid);
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        for (int rs = 0; rs < u.R_total; rs += kRowsLds) {
            const int rows_here = min(kRowsLds, u.R_total - rs);
            if (chunk == first || u.R_total > kRowsLds) stage_rows(rs, rows_here);
            for (int rb = 0; rb < rows_here; rb += 16) {
                f32x4 s[4];
                block_logits(t, u, st, s_pref, rs + rb, n, c, kreg, s);
                const int n_i = min(4, (rows_here - rb + 3) >> 2);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (i >= n_i) continue;
                    const int rr = rb + 4 * i + c;
                    const bool have = rr < rows_here;
                    const float M = have ? s_M[rr] : 0.f;
                    const float w = have ? s_w[rr] : 0.f;
#pragma unroll
                    for (int tile = 0; tile < 4; ++tile) acc[tile] = fmaf(w, exp_key<D>(s[tile][i] - M), acc[tile]);
                }
            }
        }
#pragma unroll
        for (int tile = 0; tile < 4; ++tile) {
            float v = acc[tile];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (c == 0 && valid[tile]) t.scores[u.unit * dm.max_vis + key0 + 16 * tile + n] = v;
        }
    }
    // the moments need every score of the workgroup at once: each lane reads back the ones it stored itself
    float xs[kFinishChunks * 4];
    bool ok[kFinishChunks * 4];
#pragma unroll
    for (int ci = 0; ci < kFinishChunks; ++ci)
#pragma unroll
        for (int tile = 0; tile < 4; ++tile) {
            const int key = (first + ci) * kChunkKeys + wave * 64 + 16 * tile + n;
            ok[4 * ci + tile] = c == 0 && first + ci < last && key < u.sq.vis_len;
            xs[4 * ci + tile] = ok[4 * ci + tile] ? t.scores[u.unit * dm.max_vis + key] : 0.f;
        }
    put_moments(xs, ok);
}

// ---------------------------------------------------------------------------------------
// Eq.4-5 for bf16.  One workgroup per (KV head, sequence, layer).
//   phase 1: raw last-row logits of the G heads against every candidate text key on MFMA
//            (fp32 accumulation), into LDS.
//   phase 2: one wave per head.  Eq.5 is decided as the fp64 test exp((a_j - a_max)/sqrt(d)) >= alpha.
//            The fp32 logits settle every candidate that is not within a margin of the
//            threshold; the maximum and the few candidates inside the margin are recomputed as
//            exact fp64 dot products (bf16 products are exact, the sum is fp64) before deciding.
//            The margin is what an fp32 sum of D products can be off by, D 2^-23 of the sum of their
//            magnitudes (the largest over the head's candidates, formed on MFMA from the operands without
//            their signs), and kEliteMargin at least.
//            Then the ordered compaction of the elite positions and the elite-text columns of Eq.7.
// ---------------------------------------------------------------------------------------
constexpr int kEliteWaves = 8;      // phase 2 takes one head per wave
// Elite-text columns of up to 16 kKept rows: tiles kept between maximum and sums, keys requested together.  (Tile by tile, twice, the
// 32 rows a head of a window of 32 tokens cost eight trips to memory one behind the other: 16.5 us for 28 x 4 units of 7 heads, 13.5 now; the
// few rows of an elite window are a path of their own: 7.7 and 7.3 for one layer.)  Three tiles take 113 registers with heads of 128 elements
// (96 without them: four waves a SIMD in place of five, which calls of many units do not show), four 131, and a workgroup a CU is lost: air_score
// of 28 x 8 x 4 units of 64 keys with two / three / four tiles, 32 rows a head 90 / 93 / 106 us, 48 rows 152 / 127 / 145, 64 rows 205 / 205 / 178,
// elite window 47.3 / 47.6 / 53.8 (47.3 without); 28 x 4 units 35.0 / 35.8 / 36.6, 52.2 / 45.8 / 46.7, 66.4 / 66.4 / 55.8.
// Heads of 64 elements take 90 registers with three tiles, 80 without: two workgroups a CU in place of three, which calls of several rounds of
// workgroups do show.  air_score of 30 x 16 x 8 units, 4 heads, 714 keys without / with: elite window 172 / 182 us (threshold 0.2: 358 / 368), 7 / 20 / 32 rows
// a head 255 / 263, 269 / 273, 307 / 314, 45 rows 416 / 411; of 28 x 8 x 4 units, 7 heads, 400 keys 52.6 / 52.9 (with 0.2 147 / 145), 59.3 / 59.4, 81.8 / 80.9,
// 98.2 / 96.1, 142.6 / 132.8.  With a threshold, where few heads have more than 16 rows, calls of less than two full rounds show it too: 24 x 3 x 8 units, 900 keys 42.1 / 44.6.
constexpr int kKept = 3;
constexpr float kEliteMargin = 4e-3f;  // raw-logit units
__device__ __forceinline__ uint4 masked(const uint4 &x, uint32_t keep) { return make_uint4(x.x & keep, x.y & keep, x.z & keep, x.w & keep); }

template <int D>
__device__ __forceinline__ double dot64_wave(const bf16_t *a, const bf16_t *b, int lane) {
    uint32_t ua = 0, ub = 0;  // two elements a lane; heads of 64 elements leave the upper half of the wave at zero
    if (D == 128 || lane < 32) {
        ua = reinterpret_cast<const uint32_t *>(a)[lane];
        ub = reinterpret_cast<const uint32_t *>(b)[lane];
    }
    const double p = (double)__uint_as_float(ua << 16) * (double)__uint_as_float(ub << 16) +
                     (double)__uint_as_float(ua & 0xffff0000u) * (double)__uint_as_float(ub & 0xffff0000u);
    return wave_sum(p);
}

template <int D, int KEPT>
__global__ __launch_bounds__(64 * kEliteWaves) void elite_mfma_kernel(Dims dm, DevTables t, int l0, LaunchLayers ll, air_strides st,
                                                         SeqArgs seqs, double alpha, double ln_alpha, int gb) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, c = lane >> 4;
    const int kvh = blockIdx.x, b = blockIdx.y, li = blockIdx.z;
    const int l = l0 + li;
    const air_seq sq = seqs.s[b];
    if (li == 0 && kvh == 0 && tid == 0) t.seq_tab[b] = sq;
    const int t0 = sq.vis_start + sq.vis_len;
    const int G = dm.G, W = dm.max_window, wl = sq.win_len;
    const bf16_t *qb = (const bf16_t *)ll.p[li].q + (int64_t)b * st.q_b;
    const bf16_t *k = (const bf16_t *)ll.p[li].k + (int64_t)b * st.kv_b + (int64_t)kvh * st.kv_h;
    const int ref = sq.win_start + wl - 1;
    extern __shared__ float s_dynf[];  // gb * max_window raw logits, then as many ints (elite lists)
    float *s_logit = s_dynf;
    int *s_elite = reinterpret_cast<int *>(s_dynf + (size_t)gb * W);
    constexpr int NS = D / 32;
    constexpr double inv_sqrt_d = D == 128 ? 0.08838834764831845 : 0.125;  // 1 / sqrt(d), correctly rounded
    constexpr float scale = (float)inv_sqrt_d;
    __shared__ float s_size[16][16 * kEliteWaves];  // per head of the round: the largest sum of magnitudes that a lane has seen

    for (int g0 = 0; g0 < G; g0 += gb) {
        const int ng = min(gb, G - g0);
        // ---- phase 1: A = reference queries of heads g0 .. g0+ng-1 (MFMA row m = head), B = candidate keys
        uint4 qa[NS];
        {
            const bf16_t *qr = qb + (int64_t)(kvh * G + g0 + (n < ng ? n : 0)) * st.q_h + (int64_t)(ref - t0) * st.q_t;
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) {
                qa[sl] = make_uint4(0, 0, 0, 0);
                if (n < ng) qa[sl] = *reinterpret_cast<const uint4 *>(qr + 32 * sl + 8 * c);
            }
        }
        f32x4 size = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int j0 = wave * 16; j0 < wl; j0 += 16 * kEliteWaves) {
            const int j = j0 + n;
            uint4 kb[NS];
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) {
                kb[sl] = make_uint4(0, 0, 0, 0);
                if (j < wl) kb[sl] = *reinterpret_cast<const uint4 *>(k + (int64_t)(sq.win_start + j) * st.kv_t + 32 * sl + 8 * c);
            }
            // the logits, then the sums of magnitudes: one copy of the code, the operands with and without their signs (a
            // kernel this short waits for its instructions)
#pragma unroll 1
            for (int turn = 0; turn < 2; ++turn) {
                const uint32_t keep = turn == 0 ? 0xffffffffu : 0x7fff7fffu;
                f32x4 s4 = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int sl = 0; sl < NS; ++sl) s4 = mma<bf16_t>(masked(qa[sl], keep), masked(kb[sl], keep), s4);
                if (turn == 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (4 * c + i < ng && j < wl) s_logit[(size_t)(4 * c + i) * W + j] = s4[i];
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) size[i] = fmaxf(size[i], s4[i]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * c + i < ng) s_size[4 * c + i][16 * wave + n] = size[i];
        __syncthreads();
        // ---- phase 2
        for (int hh = wave; hh < ng; hh += kEliteWaves) {
            const int h = kvh * G + g0 + hh;
            const int64_t hrow = ((int64_t)l * dm.B + b) * dm.Hq + h;
            const float *logit = s_logit + (size_t)hh * W;
            int *elite = s_elite + (size_t)hh * W;
            const bf16_t *q = qb + (int64_t)h * st.q_h;
            const bf16_t *qref = q + (int64_t)(ref - t0) * st.q_t;
            // What an fp32 logit of this head can be off by: infinite where operands overflow, every candidate is then decided in
            // fp64; a logit that is no number is whatever the margin (the comparisons below are negated).
            static_assert(16 * kEliteWaves == 128, "two entries a lane");
            const float err = wave_max(fmaxf(s_size[hh][lane], s_size[hh][lane + 64])) * (D * 0x1p-23f);
            const float margin = fmaxf(kEliteMargin, err), near_max = fmaxf(kEliteMargin, 2.f * err);
            float m32 = -INFINITY;
            for (int j = lane; j < wl; j += 64) m32 = fmaxf(m32, logit[j]);
            m32 = wave_max(m32);
            // exact maximum: every candidate within both logits' errors of the fp32 maximum is recomputed
            // (with a threshold of 0 every number passes, whatever the maximum is; where logits or their sums of magnitudes overflow
            // fp32 the exact maximum decides which are numbers)
            const bool any_will_do = alpha == 0.0 && fabsf(m32) < INFINITY && err < INFINITY;
            double amax = any_will_do ? (double)m32 : -INFINITY;
            for (int j0 = 0; j0 < wl && !any_will_do; j0 += 64) {
                const int j = j0 + lane;
                unsigned long long near = __ballot(j < wl && !(logit[j] < m32 - near_max));
                while (near) {
                    const int src = __ffsll(near) - 1;
                    near &= near - 1;
                    amax = fmax(amax, dot64_wave<D>(qref, k + (int64_t)(sq.win_start + j0 + src) * st.kv_t, lane));
                }
            }
            int R = 0;
            for (int j0 = 0; j0 < wl; j0 += 64) {
                const int j = j0 + lane;
                // x > 0 <=> exp((a_j - a_max) / sqrt(d)) > alpha
                const double x = j < wl ? ((double)logit[j] - amax) * inv_sqrt_d - ln_alpha : -1.0;
                bool flag = j < wl && x > 0.0;
                unsigned long long unsure = __ballot(j < wl && !(fabs(x) > (double)(margin * scale)));
                while (unsure) {
                    const int src = __ffsll(unsure) - 1;
                    unsure &= unsure - 1;
                    const double a = dot64_wave<D>(qref, k + (int64_t)(sq.win_start + j0 + src) * st.kv_t, lane);
                    const bool f = exp((a - amax) * inv_sqrt_d) >= alpha;
                    if (lane == src) flag = f;
                }
                const unsigned long long bal = __ballot(flag);
                if (flag) {
                    const int pos = R + __popcll(bal & ((1ull << lane) - 1ull));
                    elite[pos] = sq.win_start + j;
                    t.elite_idx[hrow * W + pos] = sq.win_start + j;
                }
                R += __popcll(bal);
            }
            if (lane == 0) t.elite_cnt[hrow] = R;
            // elite-text columns of Eq.7: (max, sum-exp) of every elite row over the elite text keys.  The
            // R x R logits are formed on MFMA, 16 rows against 16 keys per tile; lane (n, c) of a tile holds
            // key n and rows 4c .. 4c+3, rows and keys past R re-read the last one.  Up to 16 KEPT rows the
            // tiles are kept; longer windows (alpha = 0 turns the whole span into rows) go over the keys
            // twice (maximum, then sum).  The maximum is kept as the RAW dot product (before the
            // 1/sqrt(d) scale), the sum is of exp((a - max) / sqrt(d)).
            for (int rb = 0; rb < R; rb += 16) {
                uint4 qa2[NS];
                {
                    const bf16_t *qr = q + (int64_t)(elite[min(rb + n, R - 1)] - t0) * st.q_t;
#pragma unroll
                    for (int sl = 0; sl < NS; ++sl) qa2[sl] = *reinterpret_cast<const uint4 *>(qr + 32 * sl + 8 * c);
                }
                float m4[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY}, z4[4] = {0.f, 0.f, 0.f, 0.f};
                // key jb + n of the elite list against row rb + 4c + i; the list is in position order, so with the causal option a
                // row sees the keys up to its own place in it
                auto sees = [&](int jb, int i) { return jb + n < R && (!dm.causal_text || jb + n <= rb + 4 * c + i); };
                auto top = [&](const f32x4 &a4, int jb) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) m4[i] = fmaxf(m4[i], sees(jb, i) ? a4[i] : -INFINITY);
                };
                auto over_lanes = [&]() {
#pragma unroll
                    for (int i = 0; i < 4; ++i) m4[i] = max16(m4[i]);
                };
                auto add = [&](const f32x4 &a4, int jb) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) z4[i] += sees(jb, i) ? expf((a4[i] - m4[i]) * scale) : 0.f;
                };
                auto keys = [&](int jb, uint4(&kb2)[NS]) {
                    const bf16_t *kr = k + (int64_t)elite[min(jb + n, R - 1)] * st.kv_t;
#pragma unroll
                    for (int sl = 0; sl < NS; ++sl) kb2[sl] = *reinterpret_cast<const uint4 *>(kr + 32 * sl + 8 * c);
                };
                auto tile = [&](const uint4(&kb2)[NS]) {
                    f32x4 a4 = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int sl = 0; sl < NS; ++sl) a4 = mma<bf16_t>(qa2[sl], kb2[sl], a4);
                    return a4;
                };
                uint4 kb2[NS];
                if (R <= 16) {
                    keys(0, kb2);
                    const f32x4 a4 = tile(kb2);
                    top(a4, 0);
                    over_lanes();
                    add(a4, 0);
                } else if (KEPT > 1 && R <= 16 * KEPT) {
                    // the keys of a row block requested together, their tiles kept for the sums
                    uint4 kb[KEPT][NS];
                    f32x4 a4[KEPT];
#pragma unroll
                    for (int j = 0; j < KEPT; ++j) keys(16 * j, kb[j]);  // (past the list its last key again)
#pragma unroll
                    for (int j = 0; j < KEPT; ++j) {
                        a4[j] = tile(kb[j]);
                        top(a4[j], 16 * j);
                    }
                    over_lanes();
#pragma unroll
                    for (int j = 0; j < KEPT; ++j)
                        if (16 * j < R) add(a4[j], 16 * j);
                } else {
                    for (int jb = 0; jb < R; jb += 16) {
                        keys(jb, kb2);
                        top(tile(kb2), jb);
                    }
                    over_lanes();
                    for (int jb = 0; jb < R; jb += 16) {
                        keys(jb, kb2);
                        add(tile(kb2), jb);
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float z = sum16(z4[i]);
                    const int r = rb + 4 * c + i;
                    if (n == 0 && r < R) {
                        t.row_mtext[hrow * W + r] = m4[i];
                        t.row_ztext[hrow * W + r] = z;
                    }
                }
            }
        }
        __syncthreads();
    }
}

hipError_t launch_elite_mfma(hipStream_t s, const Dims &dm, const DevTables &t, int l0, int nl, const LaunchLayers &ll,
                             const air_strides &st, const SeqArgs &seqs, double alpha) {
    const size_t per_head = (size_t)dm.max_window * (sizeof(float) + sizeof(int));
    int gb = (int)(49152 / per_head);  // heads whose logits share the LDS
    gb = gb < 1 ? 1 : (gb > dm.G ? dm.G : gb);
    const double ln_alpha = alpha > 0.0 ? log(alpha) : -INFINITY;
    const dim3 grid(dm.Hkv, dm.B, nl), block(64 * kEliteWaves);
    const bool tiles_kept = (int64_t)nl * dm.B * dm.Hkv <= (alpha > 0.0 ? 2 : 4) * kCUs || (alpha == 0.0 && dm.max_window > 32);
    auto kernel = dm.D == 128 ? elite_mfma_kernel<128, kKept> : tiles_kept ? elite_mfma_kernel<64, kKept> : elite_mfma_kernel<64, 1>;
    hipLaunchKernelGGL(kernel, grid, block, gb * per_head, s, dm, t, l0, ll, st, seqs, alpha, ln_alpha, gb);
    return hipGetLastError();
}

template <int D>
static hipError_t score_launch(hipStream_t s, const Dims &dm, const DevTables &t, int pass, int l0, int nl,
                               const LaunchLayers &ll, const air_strides &st, const SeqArgs &seqs, int inline_rows) {
    const dim3 block(256);
    if (pass == 1) {
        const dim3 grid(dm.n_chunks, dm.Hkv, nl * dm.B);
        if (dm.vis_window) hipLaunchKernelGGL((score_stream_kernel<D, true>), grid, block, 0, s, dm, t, l0, ll, st, seqs);
        else hipLaunchKernelGGL((score_stream_kernel<D, false>), grid, block, 0, s, dm, t, l0, ll, st, seqs);
        return hipGetLastError();
    }
    const dim3 grid((dm.n_chunks + kFinishChunks - 1) / kFinishChunks, dm.Hkv, nl * dm.B);
    if (inline_rows && !dm.vis_window) {
        hipLaunchKernelGGL((score_finish_kernel<D, false, true>), grid, block, 0, s, dm, t, l0, ll, st, seqs);
        return hipGetLastError();
    }
    // a wave per row when the launch has few units; with many units, 4 waves walk the rows
    hipLaunchKernelGGL(score_rows_mfma_kernel<D>, dim3(dm.Hkv, dm.B, nl),
                       dim3(nl * dm.B * dm.Hkv >= 512 ? 256 : 64 * kRowWaves), 0, s, dm, t, l0, seqs);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (dm.vis_window) hipLaunchKernelGGL((score_finish_kernel<D, true, false>), grid, block, 0, s, dm, t, l0, ll, st, seqs);
    else hipLaunchKernelGGL((score_finish_kernel<D, false, false>), grid, block, 0, s, dm, t, l0, ll, st, seqs);
    return hipGetLastError();
}

hipError_t launch_score_mfma(hipStream_t s, const Dims &dm, const DevTables &t, int pass, int l0, int nl,
                             const LaunchLayers &ll, const air_strides &st, const SeqArgs &seqs, int inline_rows) {
    return dm.D == 128 ? score_launch<128>(s, dm, t, pass, l0, nl, ll, st, seqs, inline_rows)
                       : score_launch<64>(s, dm, t, pass, l0, nl, ll, st, seqs, inline_rows);
}

}  // namespace air
