// air_score, bf16, windows that turn their whole span into rows (a continuous, all-text or visual window of dozens to
// hundreds of rows per unit): Eq.6-8 with the ROWS kept in registers and the keys streamed past them, twice.
//
// A workgroup of four waves owns a run of a unit's keys.  Every wave holds up to 64 window rows (four MFMA A operands of 16
// rows) and all waves take the same 64 keys at a time from LDS (double-buffered, one barrier per 64 keys, the next keys
// in flight meanwhile).  Exponentials are 2^(s kC - m): one fused multiply-add and one exponential per element, with a
// reference m that is a whole number, so that references are moved and partial sums merged exactly.
//   pass 1  leaves (reference, sum) per (row, run of keys).  The reference starts at the maximum over the first 64 keys of
//           the run; a lane raises its own, and scales its sum down, after a step that left the sum above its limit: one
//           addition per element, no maximum.
//   pass 2  forms maximum, fp64 normaliser and weight of the unit's rows from the partials, a thread per row, then
//           I[key] = sum over the rows of w 2^(s kC - m): one fused add per element, the sum over the
//           lanes and waves once per 64 keys.
// Precision: the argument of an exponential is rounded, to 2^-24 of itself, and the largest terms are the ones that count, so a
// reference has to stay near the maximum; and a logit keeps its bits only if its sum starts at zero.  (With sums that
// started at minus the reference, and the lane's first logit as reference up to 2^100, the scores were 9.7e-7 off fp64 in
// place of 4.3e-7 for logits of a spread of 5, 4.0e-6 in place of 8.7e-7 for a spread of 18, heads of 128.  The limit on a sum
// weighs the error of the step that finds a logit far above the reference against doing it again: 2^12 / 2^16 / 2^24 / 2^100,
// us for 224 rows at a spread of 5: 271 / 250 / 220 / 226, at a spread of 2: 222 / 220 / 218 / 224.)
// Bound: nothing alone.  The exponentials are 19 us a pass (2.86 M of a wave, 16 clocks of a SIMD each), 33 with the three
// instructions beside each; counters: vector issue 55 % of the clocks in pass 1 and 40 % in pass 2, matrix unit 20 and 18 %.  The
// rest is waiting: a barrier per 64 keys, 57 KB of query rows and (pass 2) the rows' parameters in front of 8-16 steps, 14
// blocks dealt 3 / 4 / 3 / 4, two workgroups a CU in 3.3 rounds (pass 1, 1680 workgroups) and 1.75 (pass 2, 896).
// 224 rows per unit (7 heads x 32), 28 layers x 4 KV heads x 7290 keys, us for the two passes: 207 (102 + 105).  Before, a
// workgroup kept 256 keys and walked the rows with three barriers and two reductions over sixteen lanes per 16 rows, plus a
// kernel for the row parameters, layers in two groups: 478 (195 + 40 + 243).
#include "air_score_mfma_dev.h"

#include <type_traits>

namespace air {

constexpr int kStepKeys = 64;                 // keys in LDS at a time
// Four waves with four blocks each and two waves a SIMD: eight with two blocks, at three or four a SIMD, measured 240-277 us
// against 230 for 224 rows (a key operand read from LDS then serves half as many rows, or registers spill).
constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kWaveBlocks = 4;                 // blocks of 16 rows per wave
constexpr int kWinRows = kWaves * kWaveBlocks * 16;  // rows of a workgroup at a time

// Keys in LDS: place p of key k holds its 16-byte piece p ^ swizzle(k), so that the sixteen keys that a read of one piece
// touches lie in different banks.  They pass through registers: with loads straight into LDS the compiler waits for all of
// them in front of the first LDS read behind them, the other buffer's keys or not.
template <int D>
__device__ __forceinline__ int key_swizzle(int key) {
    return D == 128 ? key & 15 : (key >> 1) & 7;
}

__device__ __forceinline__ int ilogb_of(float x) { return (int)(__float_as_uint(x) >> 23) - 127; }  // of a normal number above 0

template <int D, int PASS>
__global__ __launch_bounds__(kThreads, 2) void window_kernel(Dims dm, DevTables t, int l0, LaunchLayers ll, air_strides st, SeqArgs seqs,
                                                        int seg_chunks) {
    constexpr int NS = D / 32;
    constexpr int kPieces = D / 8;               // 16-byte pieces of a key
    constexpr int kIt = kStepKeys * kPieces / kThreads;
    constexpr float kC = Log2Scale<D>::kHi;
    constexpr float kSumLimit = 64.0f;   // of a lane's sum in front of a step: it has at most 64 keys of a row
    constexpr float kSumMost = 0x1p24f;  // a step that leaves a sum above this is done again
    constexpr float kHigh = 4.0f;        // then with the reference raised in front of exponentials above 2^kHigh
    // Beyond 2^22 a reference and a logit no longer differ by what fp32 says they do (raw logits of 3e7: keys masked by a large
    // negative number, operands in the thousands).  References stop there; logits below weigh nothing, logits above are
    // held at the bound: in pass 1 when their step is done again, in pass 2 by a plain loop over the rows that have such a reference.
    constexpr float kFar = 0x1p22f, kFarRaw = kFar / kC;
    auto held = [](float s) __attribute__((always_inline)) { return s > kFarRaw ? kFarRaw : (s < -kFarRaw ? -kFarRaw : s); };
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, c = lane >> 4;
    const int wg_chunks = PASS == 1 ? seg_chunks : kFinishChunks;
    UnitCtx u;
    if (!unit_setup(dm, seqs, l0, ll, st, u, wg_chunks)) return;
    __shared__ int s_pref[17];
    __shared__ __align__(16) bf16_t s_k[2][kStepKeys * D];
    __shared__ float s_M[kWinRows], s_w[kWinRows];
    __shared__ int s_any_far;             // pass 2: some row has its reference at the bound
    __shared__ int s_slot[kWinRows];      // a row's place in the unit's row tables
    __shared__ int64_t s_query[kWinRows]; // and in the query tensor
    __shared__ __align__(16) float s_part[PASS == 2 ? 2 : 1][kWaves][PASS == 2 ? 4 * kStepKeys : 4];  // [lane][tile]
    __shared__ float s_imp[PASS == 2 ? kFinishChunks * kChunkKeys : 1];
    __shared__ double s_mom[kWaves][3];
    const int nch = (u.sq.vis_len + kChunkKeys - 1) / kChunkKeys;
    const int first = u.chunk, last = min(nch, first + wg_chunks);
    const int n_seg = (nch + seg_chunks - 1) / seg_chunks;
    const int key_lo = first * kChunkKeys;
    // a visual-window row at visual index p sees the keys up to p: keys behind the last row are never looked at
    const int prow0 = u.sq.win_start - u.sq.vis_start;
    const int key_end = min(last * kChunkKeys, dm.vis_window ? prow0 + u.sq.win_len : u.sq.vis_len);
    const int steps = max(0, (key_end - key_lo + kStepKeys - 1) / kStepKeys);
    if (PASS == 2 && tid == 0) s_any_far = 0;
    head_prefix(t, u.hrow0, u.G, s_pref);
    u.R_total = s_pref[u.G];
    if (PASS == 2)
        for (int i = tid; i < kFinishChunks * kChunkKeys; i += kThreads) s_imp[i] = 0.f;

    // the keys of a step; keys past the end of the span repeat the last one
    auto fetch = [&](u32x4(&kx)[kIt], int step) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int p = tid + kThreads * it;
            const int key = min(key_lo + kStepKeys * step + p / kPieces, u.sq.vis_len - 1);
            kx[it] = *reinterpret_cast<const u32x4 *>(u.k + (int64_t)(u.sq.vis_start + key) * st.kv_t + 8 * (p % kPieces));
        }
    };
    int key_at[NS];  // the lane's 16 bytes of key n of a tile, slice by slice
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) key_at[sl] = n * D + 8 * ((4 * sl + c) ^ key_swizzle<D>(n));
    auto put = [&](const u32x4(&kx)[kIt], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int p = tid + kThreads * it, k = p / kPieces;
            *reinterpret_cast<u32x4 *>(&s_k[buf][k * D + 8 * ((p % kPieces) ^ key_swizzle<D>(k))]) = kx[it];
        }
    };

    for (int r0 = 0; r0 < u.R_total; r0 += kWinRows) {
        const int rows_here = min(kWinRows, u.R_total - r0);
        const int n_blk = (rows_here + 15) >> 4;
        // the blocks are dealt evenly: 14 blocks as 3, 4, 3, 4
        const int blk0 = wave * n_blk / kWaves, nb = (wave + 1) * n_blk / kWaves - blk0;
        u32x4 kx0[kIt];
        fetch(kx0, 0);
        // a thread per row of the group: where it lives and (pass 2) its maximum, normaliser and weight
        if (tid < ((rows_here + 15) & ~15)) {
            const bool have = tid < rows_here;
            const int rho = r0 + min(tid, rows_here - 1);
            const int g = head_of_row(s_pref, u.G, rho);
            const int place = g * u.W + (rho - s_pref[g]);
            const int64_t slot = u.hrow0 * u.W + place;
            const int tok = t.elite_idx[slot];
            s_slot[tid] = place;
            s_query[tid] = (int64_t)(u.kvh * u.G + g) * st.q_h + (int64_t)(tok - u.qbase) * st.q_t;
            if (PASS == 2) {
                const float2 *p = t.part + slot * dm.n_chunks;
                const float mt = t.row_mtext[slot], zt = t.row_ztext[slot];  // of raw logits
                constexpr int kAtOnce = 16;  // partials requested together; a run of them past the end repeats the last one
                float M = mt > -INFINITY ? rintf(held(mt) * kC) : -INFINITY;
                double Z = 0.0;
                for (int pass = n_seg <= kAtOnce ? 1 : 0; pass < 2; ++pass) {
                    for (int s0 = 0; s0 < n_seg; s0 += kAtOnce) {
                        float2 x[kAtOnce];
#pragma unroll
                        for (int s = 0; s < kAtOnce; ++s) x[s] = p[min(s0 + s, n_seg - 1)];
                        if (pass == 0 || n_seg <= kAtOnce) {
#pragma unroll
                            for (int s = 0; s < kAtOnce; ++s) M = fmaxf(M, x[s].x);
                        }
                        if (pass == 1) {
#pragma unroll
                            for (int s = 0; s < kAtOnce; ++s)
                                if (s0 + s < n_seg && x[s].y > 0.f) Z += (double)ldexpf(x[s].y, (int)(x[s].x - M));
                        }
                    }
                }
                if (zt > 0.f) Z += (double)(zt * __builtin_amdgcn_exp2f(fmaf(held(mt), kC, -M)));
                if (fabsf(M) > 0.5f * kFar && M > -INFINITY) s_any_far = 1;
                s_M[tid] = have && Z > 0.0 ? M : 0.f;  // rows past the list weigh nothing, nor do rows that see no key but far ones
                s_w[tid] = have && !(Z <= 0.0) ? (float)(1.0 / ((double)(s_pref[g + 1] - s_pref[g]) * (double)u.G * Z)) : 0.f;
            }
        }
        put(kx0, 0);
        lds_barrier();
        // A operands; list row rb + 4 i + c of a block sits where the accumulator of lane group c, element i, expects it
        uint4 qa[kWaveBlocks][NS];
#pragma unroll
        for (int b = 0; b < kWaveBlocks; ++b) {
            if (b >= nb) continue;
            const int row = 16 * (blk0 + b) + 4 * (n & 3) + (n >> 2);
            const bf16_t *qr = u.q + s_query[row] + 8 * c;
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) {
                qa[b][sl] = *reinterpret_cast<const uint4 *>(qr + 32 * sl);
                if (row >= rows_here) qa[b][sl] = make_uint4(0, 0, 0, 0);
            }
        }
        // ref: minus the row's reference; sum: pass 1 the sum of the exponentials, pass 2 the row's weight
        f32x4 ref[kWaveBlocks], sum[kWaveBlocks];
        if (PASS == 1) {
#pragma unroll
            for (int b = 0; b < kWaveBlocks; ++b) {
                ref[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
                sum[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        } else {
#pragma unroll
            for (int b = 0; b < kWaveBlocks; ++b)
                if (b < nb) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float M = s_M[16 * (blk0 + b) + 4 * i + c];
                        ref[b][i] = fabsf(M) > 0.5f * kFar ? -INFINITY : -M;  // the plain loop below takes that row
                        sum[b][i] = s_w[16 * (blk0 + b) + 4 * i + c];
                    }
                }
        }
        // NB: blocks of the wave, a constant (the products of its blocks interleave, rows it does not have cost nothing).  Every
        // wave passes the same number of barriers, whichever instance it runs.
        auto stream = [&](auto nb_const) __attribute__((always_inline)) {
            constexpr int NB = decltype(nb_const)::value;
            // one step over the 64 keys of a buffer.  CHECKED (pass 1): far logits are held at the bound, and the reference is
            // raised in front of an exponential above 2^kHigh; MASKED: some keys of the step do not exist or lie behind a row.
            auto keys_of_step = [&](const bf16_t *buf, int key0, f32x4(&acc), auto checked, auto masked) __attribute__((always_inline)) {
                int lim[NB > 0 ? NB : 1][4];  // last key that a row sees
                if constexpr (decltype(masked)::value) {
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            lim[b][i] = dm.vis_window ? prow0 + (r0 + 16 * (blk0 + b) + 4 * i + c) % u.sq.win_len : u.sq.vis_len - 1;
                }
#pragma unroll
                for (int tile = 0; tile < 4; ++tile) {
                    uint4 kb[NS];
#pragma unroll
                    for (int sl = 0; sl < NS; ++sl) kb[sl] = *reinterpret_cast<const uint4 *>(buf + key_at[sl] + 16 * tile * D);
                    f32x4 s[NB > 0 ? NB : 1];
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        s[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int sl = 0; sl < NS; ++sl) s[b] = mma<bf16_t>(qa[b][sl], kb[sl], s[b]);
                    }
                    if constexpr (decltype(checked)::value) {
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int i = 0; i < 4; ++i) s[b][i] = held(s[b][i]);
                    }
                    if constexpr (decltype(masked)::value) {
                        const int key = key0 + 16 * tile + n;
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int i = 0; i < 4; ++i) s[b][i] = key > lim[b][i] ? -INFINITY : s[b][i];
                    }
                    if constexpr (decltype(checked)::value) {
#pragma unroll
                        for (int b = 0; b < NB; ++b) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const bool high = fmaf(s[b][i], kC, ref[b][i]) > kHigh;
                                if (__ballot(high) == 0ull) continue;
                                const float m = rintf(s[b][i] * kC);
                                if (high) {
                                    sum[b][i] = ldexpf(sum[b][i], (int)(-ref[b][i] - m));
                                    ref[b][i] = -m;
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float e = __builtin_amdgcn_exp2f(fmaf(s[b][i], kC, ref[b][i]));
                            if (PASS == 1) sum[b][i] += e;
                            else acc[tile] = fmaf(sum[b][i], e, acc[tile]);
                        }
                }
            };
            auto masked_from = [&](int key0) { return key0 + kStepKeys > u.sq.vis_len || (dm.vis_window && key0 + kStepKeys > prow0 + 1); };
            if (PASS == 1 && steps > 0) {  // the rows' first references: the maximum over the first keys
                const bool masked = masked_from(key_lo);
                f32x4 top[NB > 0 ? NB : 1];
#pragma unroll
                for (int b = 0; b < NB; ++b) top[b] = (f32x4){-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
                for (int tile = 0; tile < 4; ++tile) {
                    const int key = key_lo + 16 * tile + n;
                    uint4 kb[NS];
#pragma unroll
                    for (int sl = 0; sl < NS; ++sl) kb[sl] = *reinterpret_cast<const uint4 *>(s_k[0] + key_at[sl] + 16 * tile * D);
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        f32x4 s = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int sl = 0; sl < NS; ++sl) s = mma<bf16_t>(qa[b][sl], kb[sl], s);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if (masked) {
                                const int lim = dm.vis_window ? prow0 + (r0 + 16 * (blk0 + b) + 4 * i + c) % u.sq.win_len : u.sq.vis_len - 1;
                                s[i] = key > lim ? -INFINITY : s[i];
                            }
                            top[b][i] = fmaxf(top[b][i], s[i]);
                        }
                    }
                }
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float m = max16(top[b][i]);
                        if (m > -INFINITY) ref[b][i] = -rintf(held(m) * kC);  // else the row sees none of these keys, or logits of -inf
                    }
            }
            for (int step = 0; step < steps; ++step) {
                const bf16_t *buf = s_k[step & 1];
                const int key0 = key_lo + kStepKeys * step;
                u32x4 kx[kIt];
                fetch(kx, min(step + 1, steps - 1));
                const bool masked = masked_from(key0);
                f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (PASS == 1) {
                    // Steps are taken without looking at single logits; where some logit stands far above its reference the step is
                    // done again from the sums before it, with the check.
                    auto largest_sum = [&]() __attribute__((always_inline)) {
                        float x = 0.f;
#pragma unroll
                        for (int b = 0; b < NB; ++b) x = fmaxf(fmaxf(x, fmaxf(sum[b][0], sum[b][1])), fmaxf(sum[b][2], sum[b][3]));
                        return x;
                    };
                    bool again = masked;
                    if (!again) {
                        f32x4 before[NB > 0 ? NB : 1];
#pragma unroll
                        for (int b = 0; b < NB; ++b) before[b] = sum[b];
                        keys_of_step(buf, key0, acc, std::false_type(), std::false_type());
                        again = __ballot(largest_sum() >= kSumMost) != 0ull;
                        if (again) {
#pragma unroll
                            for (int b = 0; b < NB; ++b) sum[b] = before[b];
                        }
                    }
                    if (again) keys_of_step(buf, key0, acc, std::true_type(), std::true_type());
                    if (__ballot(largest_sum() >= kSumLimit) != 0ull) {  // the next steps' exponentials start from a reference that fits
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int up = sum[b][i] >= kSumLimit && sum[b][i] < INFINITY ? ilogb_of(sum[b][i]) : 0;
                                sum[b][i] = ldexpf(sum[b][i], -up);
                                ref[b][i] -= (float)up;
                            }
                    }
                } else {
                    if (masked) keys_of_step(buf, key0, acc, std::false_type(), std::true_type());
                    else keys_of_step(buf, key0, acc, std::false_type(), std::false_type());
                    *reinterpret_cast<f32x4 *>(&s_part[step & 1][wave][4 * lane]) = acc;
                }
                put(kx, (step + 1) & 1);
                lds_barrier();
                // keys of the step: summed over the lane groups and the waves by one of the waves
                if (PASS == 2 && wave == (step & (kWaves - 1))) {
                    float v = 0.f;
#pragma unroll
                    for (int w = 0; w < kWaves; ++w)
#pragma unroll
                        for (int cc = 0; cc < 4; ++cc) v += s_part[step & 1][w][4 * (16 * cc + n) + c];  // key 16 c + n
                    s_imp[kStepKeys * step + lane] += v;
                }
            }
        };
        static_assert(kWaveBlocks == 4, "instances below");
        if (nb == 4) stream(std::integral_constant<int, 4>());
        else if (nb == 3) stream(std::integral_constant<int, 3>());
        else if (nb == 2) stream(std::integral_constant<int, 2>());
        else if (nb == 1) stream(std::integral_constant<int, 1>());
        else stream(std::integral_constant<int, 0>());
        if (PASS == 2 && s_any_far) {
            lds_barrier();  // the last step's sums are in place
            for (int r = 0; r < rows_here; ++r) {
                const float M = s_M[r], w = s_w[r];
                if (fabsf(M) <= 0.5f * kFar) continue;
                const int last_key = dm.vis_window ? prow0 + (r0 + r) % u.sq.win_len : u.sq.vis_len - 1;
                for (int i = tid; i < kFinishChunks * kChunkKeys && key_lo + i <= last_key; i += kThreads) {
                    const bf16_t *kr = u.k + (int64_t)(u.sq.vis_start + key_lo + i) * st.kv_t, *qr = u.q + s_query[r];
                    float s = 0.f;
#pragma unroll 1
                    for (int e = 0; e < D; e += 8)
                        s = dot_piece<bf16_t>(*reinterpret_cast<const uint4 *>(qr + e), *reinterpret_cast<const uint4 *>(kr + e), s);
                    s_imp[i] += w * __builtin_amdgcn_exp2f(fmaf(held(s), kC, -M));
                }
            }
        }
        if (PASS == 1) {  // one (maximum, sum-exp) per row from the sixteen lanes that share it
#pragma unroll
            for (int b = 0; b < kWaveBlocks; ++b) {
                if (b >= nb) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float m = sum[b][i] > 0.f ? -ref[b][i] : -INFINITY;
                    const float M = max16(m);
                    float z = sum16(m > -INFINITY ? ldexpf(sum[b][i], (int)(m - M)) : sum[b][i]);
                    // (the sum goes out as a fraction of 1 to 2: pass 2 takes the largest reference of a row, which its terms then stay below)
                    const int up = z > 0.f && z < INFINITY ? ilogb_of(z) : 0;
                    z = ldexpf(z, -up);
                    const int rho = r0 + 16 * (blk0 + b) + 4 * i + c;
                    if (n == 0 && rho < u.R_total) {
                        const int64_t slot = u.hrow0 * u.W + s_slot[rho - r0];
                        t.part[slot * dm.n_chunks + (int)blockIdx.x] = make_float2(z > 0.f ? M + (float)up : -INFINITY, z);
                    }
                }
            }
        }
        lds_barrier();  // the buffers and the row parameters have been read: the next group of rows may come
    }
    if (PASS == 1) return;
    lds_barrier();
    constexpr int kPer = kFinishChunks * kChunkKeys / kThreads;
    float xs[kPer];
    bool ok[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = kThreads * j + tid;
        xs[j] = s_imp[i];
        ok[j] = key_lo + i < u.sq.vis_len;  // keys of chunks past the last lie behind the span as well
        if (ok[j]) t.scores[u.unit * dm.max_vis + key_lo + i] = xs[j];
    }
    const int n_wg = min(u.sq.vis_len, last * kChunkKeys) - key_lo;
    leave_moments(dm, t, u.unit, u.b, u.sq, n_wg, (nch + kFinishChunks - 1) / kFinishChunks, xs, ok, s_mom);
}

// Chunks of 256 keys per workgroup of pass 1: as many as leave a launch over all layers 1536 workgroups (three rounds of two per
// CU), so that the rows a workgroup loads (57 KB at 224 rows) serve many keys; pass 2 takes the four chunks of a
// moment entry.  The run decides references and partial sums, so it follows from the context alone, not from the layers of
// the call: the scores are the same bits however the layers are cut into calls and launches.
static int window_seg_chunks(const Dims &dm) {
    int seg = kFinishChunks;
    while (seg > 1 && (int64_t)((dm.n_chunks + seg - 1) / seg) * dm.Hkv * dm.B * dm.L < 1536) seg >>= 1;
    return seg;
}

hipError_t launch_score_window(hipStream_t s, const Dims &dm, const DevTables &t, int pass, int l0, int nl, const LaunchLayers &ll,
                               const air_strides &st, const SeqArgs &seqs) {
    const int seg = window_seg_chunks(dm);
    const int per = pass == 1 ? seg : kFinishChunks;
    const dim3 grid((dm.n_chunks + per - 1) / per, dm.Hkv, nl * dm.B), block(kThreads);
    if (dm.D == 128) {
        if (pass == 1) hipLaunchKernelGGL((window_kernel<128, 1>), grid, block, 0, s, dm, t, l0, ll, st, seqs, seg);
        else hipLaunchKernelGGL((window_kernel<128, 2>), grid, block, 0, s, dm, t, l0, ll, st, seqs, seg);
    } else {
        if (pass == 1) hipLaunchKernelGGL((window_kernel<64, 1>), grid, block, 0, s, dm, t, l0, ll, st, seqs, seg);
        else hipLaunchKernelGGL((window_kernel<64, 2>), grid, block, 0, s, dm, t, l0, ll, st, seqs, seg);
    }
    return hipGetLastError();
}

}  // namespace air
