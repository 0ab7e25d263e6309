// air_score, fp32: window logits and importance (Eq.6-8) on the fp32 matrix unit (air_tile.h), full fp32 products and sums.
//
//   score_stream_f32  reads K_v once, whatever the number of rows.  Per (row, 256-key chunk) it leaves the maximum and the
//                     sum-exp; units of at most kStashRows rows stash their logits.
//   score_finish_f32  row maximum, fp64 normaliser and weight of every row from the chunk partials, then
//                     I[key] = sum over the rows of w exp(s - M), from the stash or from K_v again, by the products of the first
//                     pass and in the same order; the moments, statistics and the allocation as in the bf16 path.
//
// A wave keeps its 32 keys in registers as matrix operands, straight from global memory (64-byte segments, all requested in front
// of the row lists), blocks of 16 window rows are the other operand.  Bound: HBM and, with the two rounds of workgroups of 2304 keys
// in 28 x 4 units, the row lists and rows that arrive behind the keys; the products of a block take 1024 clocks a tile of 16 keys, half
// of them for padding with the usual 7 to 10 rows.  First pass on that shape, heads of 128 elements: 32.5 us (132 MB, 4.1 TB/s; 35 to 36
// with the places of a lane's rows and keys held in registers across the rows); with a thread per key on the vector unit, keys and query rows through LDS (20 us of LDS time for the rows alone), 41.5;
// four waves of 64 keys 35.9, three workgroups of them a CU 45.3.  Two layers x 2 heads of 576 keys of 64 elements: 6.1 and 8.2.
// More rows than the stash holds: every wave requests the rows of a block from memory, in either pass.  air_score, 28 x 4 units of 2304 keys, 7 heads,
// 5 / 32 rows a head 200 / 1610 us, with the vector unit 262 / 2100; heads of 64 133 / 1305 and 183 / 1633; 7290 keys, 7 rows a head 514 and 790.
#include "air_device.h"
#include "air_internal.h"
#include "air_score_dev.h"
#include "air_tile.h"

#include <type_traits>

namespace air {

constexpr int kStreamWaves = 8;  // of the first pass: 32 keys a wave
constexpr int kGroupRows = 32;  // window rows whose tables are staged at a time
static_assert(kGroupRows * 8 == 256, "eight lanes to a row of the group");
static_assert(kGroupRows == kStashRows, "a unit with a stash has one group of rows");

struct F32Unit {
    int kvh, b, li, l;
    air_seq sq;
    int qbase, nch;
    const float *q, *k;
    int64_t hrow0, unit;
};

__device__ __forceinline__ void unit_of(const Dims &dm, const SeqArgs &seqs, int l0, const LaunchLayers &ll, const air_strides &st,
                                        F32Unit &u) {
    u.kvh = blockIdx.y;
    seq_layer_of(dm, (int)blockIdx.z, u.b, u.li);
    u.l = l0 + u.li;
    u.sq = seqs.s[u.b];
    u.nch = (u.sq.vis_len + kChunkKeys - 1) / kChunkKeys;
    u.qbase = dm.vis_window ? u.sq.win_start : u.sq.vis_start + u.sq.vis_len;
    u.q = (const float *)ll.p[u.li].q + (int64_t)u.b * st.q_b;
    u.k = (const float *)ll.p[u.li].k + (int64_t)u.b * st.kv_b + (int64_t)u.kvh * st.kv_h;
    u.hrow0 = ((int64_t)u.l * dm.B + u.b) * dm.Hq + (int64_t)u.kvh * dm.G;
    u.unit = ((int64_t)u.l * dm.B + u.b) * dm.Hkv + u.kvh;
}

struct F32Lds {
    int pref[17], row[kGroupRows], head[kGroupRows], lim[kGroupRows];  // of a row: its place in the query tensor, head of the group, last visual index it sees
    int64_t slot[kGroupRows];                                // place of the row in the per-row tables
};

__device__ __forceinline__ void row_prefix(const DevTables &t, int64_t hrow0, int G, int *pref) {
    if (threadIdx.x == 0) {
        int run = 0;
        for (int g = 0; g < G; ++g) {
            pref[g] = run;
            run += t.elite_cnt[hrow0 + g];
        }
        pref[G] = run;
    }
    lds_barrier();
}

// tables of list rows r0 .. r0 + nb of the unit
__device__ __forceinline__ void stage_rows(const Dims &dm, const DevTables &t, const F32Unit &u, int r0, int nb, F32Lds &s) {
    lds_barrier();  // the group before has been used
    const int tid = threadIdx.x;
    if (tid < nb) {
        int g = 0;
        while (g + 1 < dm.G && s.pref[g + 1] <= r0 + tid) ++g;
        s.slot[tid] = (u.hrow0 + g) * dm.max_window + (r0 + tid - s.pref[g]);
        const int tok = t.elite_idx[s.slot[tid]];
        s.row[tid] = tok - u.qbase;
        s.head[tid] = g;
        s.lim[tid] = dm.vis_window ? tok - u.sq.vis_start : 0x7fffffff;
    }
    lds_barrier();
}

// the wave's 16 TILES keys of a chunk as matrix operands, lane (n, c) the c-th quarter of every slice of key n of a tile (keys past the
// end repeat the last one)
template <int D, int TILES>
__device__ __forceinline__ void keys_of(const F32Unit &u, const air_strides &st, int chunk, uint4 (&k)[TILES][D / 16]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 15, c = lane >> 4;
#pragma unroll
    for (int tile = 0; tile < TILES; ++tile) {
        const int key = min(chunk * kChunkKeys + 16 * TILES * wave + 16 * tile + n, u.sq.vis_len - 1);
        const float *src = u.k + (int64_t)(u.sq.vis_start + key) * st.kv_t + 4 * c;
#pragma unroll
        for (int sl = 0; sl < D / 16; ++sl) k[tile][sl] = *reinterpret_cast<const uint4 *>(src + 16 * sl);
    }
}

// Up to four rows (one or two heads a KV head): sixteen products of 4 rows x 4 keys at a time, one for every four keys of a tile and quarter c of
// their slices, in a quarter of the clocks.  The operands are those of the large products but for the row, n % 4; lane (n, c) gets the four rows'
// sums over its quarters, and keeps row c of the sum over the quarters, in a[.][0].  (With 12 of 16 rows padding the matrix unit took what the vector unit
// did not: air_score of 28 x 2 x 4 units of 2304 keys of 128 elements, one head / two, 89.6 / 91.9 us, 83.2 / 87.1 this way, 80.3 / 85.2 on the vector unit; heads
// of 64 63.2 / 65.8, 58.6 / 61.3, 60.9 / 65.4.)  Eight sums of D / 8 products: scores 0.3 to 0.5 times as far off fp64 as on the vector unit.
template <int D, int TILES>
__device__ __forceinline__ void few_logits(const uint4 (&q)[D / 16], const uint4 (&k)[TILES][D / 16], f32x4 (&a)[TILES]) {
    // over the two halves of two registers, or over the quarters: what each has of the first in the lower (even) ones, of the second in the others
    auto halves = [](float x, float y) __attribute__((always_inline)) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    auto quarters = [](float x, float y) __attribute__((always_inline)) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
#pragma unroll
    for (int tile = 0; tile < TILES; ++tile) {
        f32x4 x = (f32x4){0.f, 0.f, 0.f, 0.f}, half = x;
#pragma unroll
        for (int sl = 0; sl < D / 16; sl += 2) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x = __builtin_amdgcn_mfma_f32_4x4x1f32(__builtin_bit_cast(f32x4, q[sl])[e], __builtin_bit_cast(f32x4, k[tile][sl])[e], x, 0, 0, 0);
                half = __builtin_amdgcn_mfma_f32_4x4x1f32(__builtin_bit_cast(f32x4, q[sl + 1])[e], __builtin_bit_cast(f32x4, k[tile][sl + 1])[e], half, 0, 0, 0);
            }
        }
        x += half;
        a[tile] = (f32x4){0.f, 0.f, 0.f, 0.f};
        a[tile][0] = quarters(halves(x[0], x[2]), halves(x[1], x[3]));
    }
}

// Logits of the staged rows rb .. rb + 15 against those keys: lane (n, c) gets rows rb + 4 i + c of key n of every tile.  (Operand row
// 4 c + i carries staged row 4 i + c, so that all lanes are done after (nb - rb + 3) / 4 values.)  Even and odd slices have a sum each: in
// one sum over the D products the scores were up to 1.17 times as far off fp64 as with a chain of multiply-adds on the vector unit (logits of
// a spread of 5, heads of 128: 1.52e-6 and 1.30e-6), in two they are 0.2 to 0.8 times as far (7.0e-7), in the same time.
template <int D, bool FEW, int TILES>
__device__ __forceinline__ void logits(const Dims &dm, const F32Unit &u, const air_strides &st, const F32Lds &s, int rb, int nb,
                                       const uint4 (&k)[TILES][D / 16], f32x4 (&a)[TILES]) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // what follows from it is formed here, not held across the rows: registers for a workgroup a CU more
    const int n = lane & 15, c = lane >> 4;
    const int r = rb + (FEW ? n & 3 : 4 * (n & 3) + (n >> 2));
    const float *src = u.q + (int64_t)(u.kvh * dm.G + s.head[min(r, nb - 1)]) * st.q_h + (int64_t)s.row[min(r, nb - 1)] * st.q_t + 4 * c;
    uint4 q[D / 16];
#pragma unroll
    for (int sl = 0; sl < D / 16; ++sl) q[sl] = *reinterpret_cast<const uint4 *>(src + 16 * sl);
    if constexpr (FEW) {
        few_logits<D, TILES>(q, k, a);
    } else {
#pragma unroll
        for (int tile = 0; tile < TILES; ++tile) {
            f32x4 half = (f32x4){0.f, 0.f, 0.f, 0.f};
            a[tile] = half;
#pragma unroll
            for (int sl = 0; sl < D / 16; sl += 2) {
                a[tile] = mma<float>(q[sl], k[tile][sl], a[tile]);
                half = mma<float>(q[sl + 1], k[tile][sl + 1], half);
            }
            a[tile] += half;
        }
    }
    {
#pragma clang fp contract(off)  // the scaled logit is rounded (it may be stashed): not fused into what follows
        const float scale = 1.0f / sqrtf((float)D);
#pragma unroll
        for (int tile = 0; tile < TILES; ++tile)
#pragma unroll
            for (int i = 0; i < 4; ++i) a[tile][i] *= scale;
    }
}

template <int D>
__global__ __launch_bounds__(64 * kStreamWaves, D == 64 ? 6 : 4) void score_stream_f32(Dims dm, DevTables t, int l0, LaunchLayers ll, air_strides st, SeqArgs seqs) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    F32Unit u;
    unit_of(dm, seqs, l0, ll, st, u);
    const int chunk = blockIdx.x;
    if (chunk >= u.nch) return;
    __shared__ F32Lds s;
    __shared__ float s_m[kStreamWaves][16], s_z[kStreamWaves][16];
    constexpr int T = 16 / kStreamWaves;  // tiles of a wave
    uint4 k[T][D / 16];
    keys_of<D, T>(u, st, chunk, k);
    row_prefix(t, u.hrow0, dm.G, s.pref);
    const int R_total = s.pref[dm.G];
    const bool stash = R_total <= dm.stash_rows;
    auto over_waves = [&](const float(&x)[kStreamWaves][16], int r, auto op) {
        float v = x[0][r];
#pragma unroll
        for (int w = 1; w < kStreamWaves; ++w) v = op(v, x[w][r]);
        return v;
    };
    float *stash_of = t.stash + ((u.unit * dm.n_chunks + chunk) * (int64_t)kStashRows) * kChunkKeys;
    for (int r0 = 0; r0 < R_total; r0 += kGroupRows) {
        const int nb = min(kGroupRows, R_total - r0);
        stage_rows(dm, t, u, r0, nb, s);
        auto block = [&](int rb, auto few) __attribute__((always_inline)) {
            constexpr int I = decltype(few)::value ? 1 : 4;  // values of a lane
            int lane = threadIdx.x & 63;
            asm volatile("" : "+v"(lane));  // (as above)
            const int n = lane & 15, c = lane >> 4, key0 = 16 * T * wave + n;
            float *stash_base = stash_of + key0;
            f32x4 a[T];
            logits<D, I == 1, T>(dm, u, st, s, rb, nb, k, a);
            const int n_i = min(4, (nb - rb + 3) >> 2);  // live values of i (uniform over the workgroup)
            int lim[I];  // last key of the chunk that row i sees, relative to the lane's first
#pragma unroll
            for (int i = 0; i < I; ++i) lim[i] = min(s.lim[min(rb + 4 * i + c, nb - 1)], u.sq.vis_len - 1) - chunk * kChunkKeys - key0;
#pragma unroll
            for (int i = 0; i < I; ++i) {
                if (i >= n_i) continue;
                const int r = 4 * i + c;
                float m = -INFINITY;
#pragma unroll
                for (int tile = 0; tile < T; ++tile) {
                    if (stash && rb + r < nb) stash_base[(rb + r) * kChunkKeys + 16 * tile] = a[tile][i];
                    m = fmaxf(m, 16 * tile <= lim[i] ? a[tile][i] : -INFINITY);
                }
                m = max16(m);
                if (n == 0) s_m[wave][r] = m;
            }
            lds_barrier();
#pragma unroll
            for (int i = 0; i < I; ++i) {
                if (i >= n_i) continue;
                const int r = 4 * i + c;
                const float m = over_waves(s_m, r, [](float x, float y) { return fmaxf(x, y); });
                float z = 0.f;
#pragma unroll
                for (int tile = 0; tile < T; ++tile) z += 16 * tile <= lim[i] ? expf(a[tile][i] - m) : 0.f;
                z = sum16(z);
                if (n == 0) s_z[wave][r] = z;
            }
            lds_barrier();
            if (tid < 16 && rb + tid < nb) {
                const float m = over_waves(s_m, tid, [](float x, float y) { return fmaxf(x, y); });
                const float z = over_waves(s_z, tid, [](float x, float y) { return x + y; });
                t.part[s.slot[rb + tid] * dm.n_chunks + chunk] = make_float2(m, z);
            }
            lds_barrier();  // the maxima have been read
        };
        for (int rb = 0; rb < nb; rb += 16) {
            if (nb - rb <= 4) block(rb, std::true_type());
            else block(rb, std::false_type());
        }
    }
}

template <int D>
__global__ __launch_bounds__(256) void score_finish_f32(Dims dm, DevTables t, int l0, LaunchLayers ll, air_strides st, SeqArgs seqs) {
    const int tid = threadIdx.x;
    F32Unit u;
    unit_of(dm, seqs, l0, ll, st, u);
    const int first = (int)blockIdx.x * kFinishChunks;
    if (first >= u.nch) return;
    const int last = min(u.nch, first + kFinishChunks);
    __shared__ F32Lds s;
    __shared__ float s_M[kGroupRows], s_w[kGroupRows];
    __shared__ double s_mom[4][3];
    row_prefix(t, u.hrow0, dm.G, s.pref);
    const int R_total = s.pref[dm.G];
    const bool stash = R_total <= dm.stash_rows;
    float imp[kFinishChunks] = {0.f, 0.f, 0.f, 0.f};
    for (int r0 = 0; r0 < R_total; r0 += kGroupRows) {
        const int nb = min(kGroupRows, R_total - r0);
        stage_rows(dm, t, u, r0, nb, s);
        // Row maximum over the chunks and the elite-text columns, normaliser in fp64, weight: eight lanes to a row, all rows of
        // the group at once; the text columns are the item in front of the chunks.  (Sixteen lanes in two rounds, and the
        // stash read chunk by chunk below: 13.1 us for the kernel on the tiny workload, where it is all latency, 24.5 on 112
        // units of 2304 keys with heads of 128 elements; so 12.3 and 21.7.)
        {
            const int r = min(tid >> 3, nb - 1), gl = tid & 7;
            const int64_t slot = s.slot[r];
            const float2 *p = t.part + slot * dm.n_chunks;
            const float2 text = make_float2(t.row_mtext[slot] * (1.0f / sqrtf((float)D)), t.row_ztext[slot]);  // stored unscaled
            auto item = [&](int c) { return c == 0 ? text : p[min(c, u.nch) - 1]; };
            const float2 x0 = item(gl), x1 = item(gl + 8);
            float M = fmaxf(text.x, fmaxf(x0.x, x1.x));  // an item past the last repeats it
            for (int c = gl + 16; c <= u.nch; c += 8) M = fmaxf(M, item(c).x);
            M = max8(M);
            double Z = gl <= u.nch ? (double)x0.y * exp((double)x0.x - (double)M) : 0.0;
            if (gl + 8 <= u.nch) Z += (double)x1.y * exp((double)x1.x - (double)M);
            for (int c = gl + 16; c <= u.nch; c += 8) {
                const float2 x = item(c);
                Z += (double)x.y * exp((double)x.x - (double)M);
            }
            Z = sum8(Z);
            const int g = s.head[r];
            if (gl == 0) {
                s_M[r] = M;
                s_w[r] = (float)(1.0 / ((double)(s.pref[g + 1] - s.pref[g]) * (double)dm.G * Z));
            }
        }
        lds_barrier();
        if (stash) {
            const float *sb = t.stash + ((u.unit * dm.n_chunks + first) * (int64_t)kStashRows) * kChunkKeys + tid;
            float acc[kFinishChunks][4] = {};  // rows by their number modulo 4, as in the products' lane groups below
            for (int rb = 0; rb < nb; rb += 8) {
                float a[kFinishChunks][8];
#pragma unroll
                for (int ci = 0; ci < kFinishChunks; ++ci)
#pragma unroll
                    for (int r = 0; r < 8; ++r)  // a chunk past the last and a row past the list re-read the last one
                        a[ci][r] = sb[min(ci, last - 1 - first) * (kStashRows * kChunkKeys) + min(rb + r, nb - 1) * kChunkKeys];
#pragma unroll
                for (int ci = 0; ci < kFinishChunks; ++ci) {
                    const int i = (first + ci) * kChunkKeys + tid;
#pragma unroll
                    for (int r = 0; r < 8; ++r)
                        if (rb + r < nb && i <= s.lim[rb + r])
                            acc[ci][r & 3] = fmaf(s_w[rb + r], expf(a[ci][r] - s_M[rb + r]), acc[ci][r & 3]);
                }
            }
#pragma unroll
            for (int ci = 0; ci < kFinishChunks; ++ci) imp[ci] += (acc[ci][0] + acc[ci][1]) + (acc[ci][2] + acc[ci][3]);
        } else {
            const int lane = tid & 63, c = lane >> 4;
            // (Unrolled, heads of 128 take 260 registers, one wave a SIMD: air_score of 28 x 4 units of 7290 keys, 7 x 7 rows, 617 us in place of 537.)
#pragma unroll 1
            for (int ci = 0; ci < kFinishChunks; ++ci) {
                if (first + ci >= last) break;
                uint4 k[4][D / 16];
                keys_of<D, 4>(u, st, first + ci, k);
                const int key0 = (first + ci) * kChunkKeys + (tid & ~63) + (lane & 15);
                float acc[4] = {0.f, 0.f, 0.f, 0.f};  // rows of the lane, key of every tile
                auto block = [&](int rb, auto few) __attribute__((always_inline)) {
                    f32x4 a[4];
                    logits<D, decltype(few)::value, 4>(dm, u, st, s, rb, nb, k, a);
#pragma unroll
                    for (int i = 0; i < (decltype(few)::value ? 1 : 4); ++i) {
                        const int r = rb + 4 * i + c;
                        if (r >= nb) continue;
#pragma unroll
                        for (int tile = 0; tile < 4; ++tile)
                            if (key0 + 16 * tile <= s.lim[r]) acc[tile] = fmaf(s_w[r], expf(a[tile][i] - s_M[r]), acc[tile]);
                    }
                };
                for (int rb = 0; rb < nb; rb += 16) {
                    if (nb - rb <= 4) block(rb, std::true_type());
                    else block(rb, std::false_type());
                }
                // over the rows of the four lane groups; lane (n, c) keeps key 16 c + n, the thread's own
#pragma unroll
                for (int tile = 0; tile < 4; ++tile) {
                    float v = acc[tile];
                    v += __shfl_xor(v, 16, 64);
                    v += __shfl_xor(v, 32, 64);
#pragma unroll
                    for (int cj = 0; cj < kFinishChunks; ++cj) imp[cj] += c == tile && cj == ci ? v : 0.f;
                }
            }
        }
    }
    bool ok[kFinishChunks];
#pragma unroll
    for (int ci = 0; ci < kFinishChunks; ++ci) {
        const int i = (first + ci) * kChunkKeys + tid;
        ok[ci] = i < u.sq.vis_len;  // keys of chunks past the last lie behind the span as well
        if (ok[ci]) t.scores[u.unit * dm.max_vis + i] = imp[ci];
    }
    const int n_wg = min(u.sq.vis_len, last * kChunkKeys) - first * kChunkKeys;
    leave_moments(dm, t, u.unit, u.b, u.sq, n_wg, (u.nch + kFinishChunks - 1) / kFinishChunks, imp, ok, s_mom);
}

hipError_t launch_score_f32(hipStream_t s, const Dims &dm, const DevTables &t, int pass, int l0, int nl, const LaunchLayers &ll,
                            const air_strides &st, const SeqArgs &seqs) {
    const dim3 stream_grid(dm.n_chunks, dm.Hkv, nl * dm.B), finish_grid(dm.n_entries, dm.Hkv, nl * dm.B);
    if (pass == 1) {
        if (dm.D == 128) hipLaunchKernelGGL(score_stream_f32<128>, stream_grid, dim3(64 * kStreamWaves), 0, s, dm, t, l0, ll, st, seqs);
        else hipLaunchKernelGGL(score_stream_f32<64>, stream_grid, dim3(64 * kStreamWaves), 0, s, dm, t, l0, ll, st, seqs);
    } else {
        if (dm.D == 128) hipLaunchKernelGGL(score_finish_f32<128>, finish_grid, dim3(256), 0, s, dm, t, l0, ll, st, seqs);
        else hipLaunchKernelGGL(score_finish_f32<64>, finish_grid, dim3(256), 0, s, dm, t, l0, ll, st, seqs);
    }
    return hipGetLastError();
}

}  // namespace air
