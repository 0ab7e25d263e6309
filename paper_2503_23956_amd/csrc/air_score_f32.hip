// air_score, fp32: window logits and importance (Eq.6-8) on the vector unit, a thread per visual key.
//
// A logit is one chain of fp32 fused multiply-adds over the head's elements in their order, then one multiplication by
// 1/sqrt(d).  (The fp32 matrix instructions have the same peak rate, add in another order, and would spend half of their
// rows on padding: a unit has 7-10 window rows.)
//
//   score_stream_f32  reads K_v once.  Per (row, 256-key chunk) it leaves the maximum and the sum-exp; units of at most
//                     kStashRows rows stash their logits.
//   score_finish_f32  row maximum, fp64 normaliser and weight of every row from the chunk partials, then
//                     I[key] = sum over the rows, in list order, of w exp(s - M), from the stash or from K_v again; the
//                     moments, statistics and the allocation as in the bf16 path.
//
// Keys reach the threads through LDS: a wave reads 128-byte slices of its 64 keys, eight lanes to a key, and a lane then
// picks up its own key's slice.  (One whole row per lane straight from global memory touches 64 lines with every
// instruction and fetches each line eight times: 28 layers of 2304 keys with heads of 128 elements took 85 + 53 us for
// the two passes, 41 + 24 us this way, with the rows' parameters, the statistics and the allocation in the second.)
#include "air_device.h"
#include "air_internal.h"
#include "air_score_dev.h"
#include "air_tile.h"

namespace air {

constexpr int kGroupRows = 32;  // window rows whose logits a thread holds at a time
constexpr int kSliceElems = 32; // elements of a key staged at a time: 128 bytes
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

template <int D>
struct F32Lds {
    __align__(16) float q[kGroupRows][D];                    // query rows of the group, read as broadcasts
    __align__(16) float key[4][64][kSliceElems + 4];         // per wave: a slice of its 64 keys
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
    __syncthreads();
}

// table places (and, with QUERIES, the query rows) of list rows r0 .. r0 + nb of the unit
template <int D, bool QUERIES>
__device__ __forceinline__ void stage_rows(const Dims &dm, const DevTables &t, const F32Unit &u, const air_strides &st, int r0, int nb,
                                           F32Lds<D> &s) {
    __syncthreads();  // the group before has been used
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
    __syncthreads();
    if (!QUERIES) return;
    for (int p = tid; p < nb * (D / 4); p += 256) {
        const int r = p / (D / 4), c = 4 * (p % (D / 4));
        *reinterpret_cast<f32x4 *>(&s.q[r][c]) =
            *reinterpret_cast<const f32x4 *>(u.q + (int64_t)(u.kvh * dm.G + s.head[r]) * st.q_h + (int64_t)s.row[r] * st.q_t + c);
    }
    __syncthreads();
}

// logits of the nb staged rows against key i = chunk * 256 + tid (keys past the end repeat the last one)
template <int D>
__device__ __forceinline__ void logits(const F32Unit &u, const air_strides &st, int chunk, int nb, F32Lds<D> &s,
                                       float (&a)[kGroupRows]) {
    constexpr int kSlices = D / kSliceElems, kPer = kSliceElems / 4;  // 16-byte pieces of a slice
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int key0 = chunk * kChunkKeys + wave * 64;
    f32x4 next[kPer];
    auto fetch = [&](int sl) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < kPer; ++it) {
            const int key = min(key0 + (lane >> 3) + 8 * it, u.sq.vis_len - 1);
            next[it] = *reinterpret_cast<const f32x4 *>(u.k + (int64_t)(u.sq.vis_start + key) * st.kv_t + kSliceElems * sl + 4 * (lane & 7));
        }
    };
#pragma unroll
    for (int r = 0; r < kGroupRows; ++r) a[r] = 0.f;
    fetch(0);
    for (int sl = 0; sl < kSlices; ++sl) {
#pragma unroll
        for (int it = 0; it < kPer; ++it) *reinterpret_cast<f32x4 *>(&s.key[wave][(lane >> 3) + 8 * it][4 * (lane & 7)]) = next[it];
        if (sl + 1 < kSlices) fetch(sl + 1);
        // a wave uses its own part of the LDS only: its accesses complete in order, no barrier
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        f32x4 k[kPer];
#pragma unroll
        for (int c = 0; c < kPer; ++c) k[c] = *reinterpret_cast<const f32x4 *>(&s.key[wave][lane][4 * c]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int rb = 0; rb < kGroupRows; rb += 4) {
            if (rb >= nb) break;  // rows past the list hold whatever was there: their logits are never used
#pragma unroll
            for (int c = 0; c < kPer; ++c) {
#pragma unroll
                for (int r = rb; r < rb + 4; ++r) {
                    const f32x4 q = *reinterpret_cast<const f32x4 *>(&s.q[r][kSliceElems * sl + 4 * c]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[r] = fmaf(q[e], k[c][e], a[r]);
                }
            }
        }
    }
    {
#pragma clang fp contract(off)  // the scaled logit is rounded (it may be stashed): not fused into what follows
        const float scale = 1.0f / sqrtf((float)D);
#pragma unroll
        for (int r = 0; r < kGroupRows; ++r) a[r] *= scale;
    }
}

template <int D>
__global__ __launch_bounds__(256) void score_stream_f32(Dims dm, DevTables t, int l0, LaunchLayers ll, air_strides st, SeqArgs seqs) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    F32Unit u;
    unit_of(dm, seqs, l0, ll, st, u);
    const int chunk = blockIdx.x;
    if (chunk >= u.nch) return;
    __shared__ F32Lds<D> s;
    __shared__ float s_red[kGroupRows][4];
    row_prefix(t, u.hrow0, dm.G, s.pref);
    const int R_total = s.pref[dm.G];
    const bool stash = R_total <= dm.stash_rows;
    const int i = chunk * kChunkKeys + tid;
    const bool valid = i < u.sq.vis_len;
    float *stash_base = t.stash + ((u.unit * dm.n_chunks + chunk) * (int64_t)kStashRows) * kChunkKeys;
    for (int r0 = 0; r0 < R_total; r0 += kGroupRows) {
        const int nb = min(kGroupRows, R_total - r0);
        stage_rows<D, true>(dm, t, u, st, r0, nb, s);
        float a[kGroupRows];
        logits<D>(u, st, chunk, nb, s, a);
        if (stash) {
#pragma unroll
            for (int r = 0; r < kGroupRows; ++r)
                if (r < nb) stash_base[r * kChunkKeys + tid] = a[r];
        }
#pragma unroll
        for (int r = 0; r < kGroupRows; ++r) {
            if (r >= nb) break;
            const float m = wave_max(valid && i <= s.lim[r] ? a[r] : -INFINITY);
            if (lane == 0) s_red[r][wave] = m;
        }
        __syncthreads();
        float mrow = 0.f;  // of row tid, for the entry
        if (tid < nb) mrow = fmaxf(fmaxf(s_red[tid][0], s_red[tid][1]), fmaxf(s_red[tid][2], s_red[tid][3]));
#pragma unroll
        for (int r = 0; r < kGroupRows; ++r) {
            if (r >= nb) break;
            const float m = fmaxf(fmaxf(s_red[r][0], s_red[r][1]), fmaxf(s_red[r][2], s_red[r][3]));
            a[r] = wave_sum(valid && i <= s.lim[r] ? expf(a[r] - m) : 0.f);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kGroupRows; ++r) {
            if (r >= nb) break;
            if (lane == 0) s_red[r][wave] = a[r];
        }
        __syncthreads();
        if (tid < nb) {
            const float z = (s_red[tid][0] + s_red[tid][1]) + (s_red[tid][2] + s_red[tid][3]);
            t.part[s.slot[tid] * dm.n_chunks + chunk] = make_float2(mrow, z);
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
    __shared__ F32Lds<D> s;
    __shared__ float s_M[kGroupRows], s_w[kGroupRows];
    __shared__ double s_mom[4][3];
    row_prefix(t, u.hrow0, dm.G, s.pref);
    const int R_total = s.pref[dm.G];
    const bool stash = R_total <= dm.stash_rows;
    float imp[kFinishChunks] = {0.f, 0.f, 0.f, 0.f};
    for (int r0 = 0; r0 < R_total; r0 += kGroupRows) {
        const int nb = min(kGroupRows, R_total - r0);
        if (stash) stage_rows<D, false>(dm, t, u, st, r0, nb, s);
        else stage_rows<D, true>(dm, t, u, st, r0, nb, s);
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
        __syncthreads();
        if (stash) {
            const float *sb = t.stash + ((u.unit * dm.n_chunks + first) * (int64_t)kStashRows) * kChunkKeys + tid;
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
                        if (rb + r < nb && i <= s.lim[rb + r]) imp[ci] = fmaf(s_w[rb + r], expf(a[ci][r] - s_M[rb + r]), imp[ci]);
                }
            }
        } else {
            float a[kGroupRows];
#pragma unroll
            for (int ci = 0; ci < kFinishChunks; ++ci) {
                if (first + ci >= last) break;
                logits<D>(u, st, first + ci, nb, s, a);
                const int i = (first + ci) * kChunkKeys + tid;
#pragma unroll
                for (int r = 0; r < kGroupRows; ++r)
                    if (r < nb && i <= s.lim[r]) imp[ci] = fmaf(s_w[r], expf(a[r] - s_M[r]), imp[ci]);
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
        if (dm.D == 128) hipLaunchKernelGGL(score_stream_f32<128>, stream_grid, dim3(256), 0, s, dm, t, l0, ll, st, seqs);
        else hipLaunchKernelGGL(score_stream_f32<64>, stream_grid, dim3(256), 0, s, dm, t, l0, ll, st, seqs);
    } else {
        if (dm.D == 128) hipLaunchKernelGGL(score_finish_f32<128>, finish_grid, dim3(256), 0, s, dm, t, l0, ll, st, seqs);
        else hipLaunchKernelGGL(score_finish_f32<64>, finish_grid, dim3(256), 0, s, dm, t, l0, ll, st, seqs);
    }
    return hipGetLastError();
}

}  // namespace air
