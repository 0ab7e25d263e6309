// What the bf16 score kernels share: the unit of a workgroup, the A operand of a block of window rows, exponentials.
#pragma once

#include "air_score_dev.h"
#include "air_tile.h"

namespace air {

struct UnitCtx {
    int kvh, b, li, l, chunk, t0, G, W, R_total;
    int qbase;  // token that row 0 of the query tensor belongs to (start of the text span, or of a visual window)
    air_seq sq;
    const bf16_t *q, *k;
    int64_t hrow0, unit;
};

// row-list offsets of the heads of the group: s_pref[g] .. s_pref[g+1] are the rows of head g
__device__ __forceinline__ void head_prefix(const DevTables &t, int64_t hrow0, int G, int *s_pref) {
    if (threadIdx.x == 0) {
        int run = 0;
        for (int g = 0; g < G; ++g) {
            s_pref[g] = run;
            run += t.elite_cnt[hrow0 + g];
        }
        s_pref[G] = run;
    }
    lds_barrier();
}

__device__ __forceinline__ int head_of_row(const int *s_pref, int G, int rho) {
    int g = 0;
    while (g + 1 < G && s_pref[g + 1] <= rho) ++g;
    return g;
}

__device__ __forceinline__ bool unit_setup(const Dims &dm, const SeqArgs &seqs, int l0, const LaunchLayers &ll,
                                           const air_strides &st, UnitCtx &u, int chunks_per_wg) {
    u.chunk = blockIdx.x * chunks_per_wg;  // first chunk of this workgroup
    u.kvh = blockIdx.y;  // grid (chunk group, KV head, sequence + B * layer)
    seq_layer_of(dm, (int)blockIdx.z, u.b, u.li);
    u.l = l0 + u.li;
    u.sq = seqs.s[u.b];  // from the kernel arguments: no table read in front of the key loads
    if (u.chunk * kChunkKeys >= u.sq.vis_len) return false;
    u.t0 = u.sq.vis_start + u.sq.vis_len;
    u.qbase = dm.vis_window ? u.sq.win_start : u.t0;
    u.G = dm.G;
    u.W = dm.max_window;
    u.q = (const bf16_t *)ll.p[u.li].q + (int64_t)u.b * st.q_b;
    u.k = (const bf16_t *)ll.p[u.li].k + (int64_t)u.b * st.kv_b + (int64_t)u.kvh * st.kv_h;
    u.hrow0 = ((int64_t)u.l * dm.B + u.b) * dm.Hq + (int64_t)u.kvh * u.G;
    u.unit = ((int64_t)u.l * dm.B + u.b) * dm.Hkv + u.kvh;
    return true;
}

// A operand of one block of 16 window rows.  MFMA row m = 4c'+i' carries list row rbase + 4i' + c'
// (c' = m / 4, i' = m % 4), so that output lane group c holds rows rbase + c, rbase + 4 + c, ...:
// with fewer than 16 rows in the block every lane group has the same number of live rows and
// loops over i stop early.
template <int NS>
__device__ __forceinline__ void load_rows(const DevTables &t, const UnitCtx &u, const air_strides &st,
                                          const int *s_pref, int rbase, int n, int c, uint4 (&qa)[NS]) {
    const int rho = rbase + 4 * (n & 3) + (n >> 2);
    const int g = head_of_row(s_pref, u.G, rho);
    const bool have = rho < u.R_total;
    int tok = u.qbase;
    if (have) tok = t.elite_idx[(u.hrow0 + g) * u.W + (rho - s_pref[g])];
    const bf16_t *qr = u.q + (int64_t)(u.kvh * u.G + g) * st.q_h + (int64_t)(tok - u.qbase) * st.q_t;
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
        qa[sl] = make_uint4(0, 0, 0, 0);
        if (have) qa[sl] = *reinterpret_cast<const uint4 *>(qr + 32 * sl + 8 * c);
    }
}

// Logits are RAW dot products until they are exponentiated: exp((s - M) / sqrt(d)) = 2^((s - M) * kC).
template <int D>
struct Log2Scale {  // log2(e) / sqrt(d), split
    static constexpr double kC = 1.4426950408889634 * (D == 128 ? 0.08838834764831845 : 0.125);
    static constexpr float kHi = (float)kC, kLo = (float)(kC - (double)kHi);
};
template <int D>
__device__ __forceinline__ float exp_raw(float d) { return exp2_scaled(d, Log2Scale<D>::kHi, Log2Scale<D>::kLo); }
// The per-key exponentials take the one-multiply form: its rounding of d * kHi costs a relative
// 0.7 * 2^-24 * |log2 of the result|, below 6e-6 down to the smallest fp32 the result can be.
template <int D>
__device__ __forceinline__ float exp_key(float d) { return __builtin_amdgcn_exp2f(d * Log2Scale<D>::kHi); }

}  // namespace air
