// air_score, the kernels in front of the window's logits:
//   elite_kernel       fp32 tensors: Eq.4 (last row) + Eq.5, elite index set of every query head (one workgroup per KV
//                      group), and the contribution of the elite text keys to each elite row's softmax.  All logits in
//                      fp64 (bf16 tensors take elite_mfma_kernel, which needs fp64 near the threshold only).
//   window_rows_kernel visual window: every token of the span is a row.
#include "air_device.h"
#include "air_internal.h"

namespace air {

// ---------------------------------------------------------------------------------------
// Eq.4-5.  One workgroup per (KV head, sequence, layer): the candidate text keys are read once
// for all G query heads of the group.  The decision of Eq.5 is taken in fp64:
// exp(s_j - max_j s) >= alpha, the form in which the softmax normaliser of Eq.4 has cancelled.
//   phase 1 (all threads): last-row logits of every head of the batch against every candidate,
//           16 lanes per candidate key (coalesced row reads), D/16 elements per lane, fp64.
//   phase 2 (one wave per head): maximum, threshold, ordered compaction of the elite positions,
//           then the elite-text columns of Eq.7 for that head's elite rows.
// Heads are processed in batches of `gb` so that gb * max_window logits fit the LDS.
// ---------------------------------------------------------------------------------------
// The kernel waits, for its keys and for one head after the other: eight waves (NW) take fewer rounds of keys and of heads than
// four, but only one such workgroup fits a CU, where two of four waves do (three with heads of 64 elements).
template <typename T, int D, int NW>
__global__ __launch_bounds__(64 * NW) void elite_kernel(Dims dm, DevTables t, int l0, LaunchLayers ll, air_strides st,
                                                    SeqArgs seqs, double alpha, int gb) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int kvh = blockIdx.x, b = blockIdx.y, li = blockIdx.z;
    const int l = l0 + li;
    const air_seq sq = seqs.s[b];
    if (li == 0 && kvh == 0 && tid == 0) t.seq_tab[b] = sq;
    const int t0 = sq.vis_start + sq.vis_len;
    const int G = dm.G, W = dm.max_window, wl = sq.win_len;
    const T *qb = (const T *)ll.p[li].q + (int64_t)b * st.q_b;
    const T *k = (const T *)ll.p[li].k + (int64_t)b * st.kv_b + (int64_t)kvh * st.kv_h;
    const int ref = sq.win_start + wl - 1;

    extern __shared__ double s_dyn[];  // gb * max_window doubles (last-row logits), then as many ints (elite lists)
    double *s_logit = s_dyn;
    int *s_elite = reinterpret_cast<int *>(s_dyn + (size_t)gb * W);

    constexpr int E = D / 16, UN = 4, HB = 8;  // elements per lane, candidate rounds in flight, heads per register batch
    constexpr int kGroups = 4 * NW;            // candidate keys read side by side
    const int sub = tid & 15, grp = tid >> 4;
    const double sqrt_d = sqrt((double)D);
    const float scale = 1.0f / sqrtf((float)D);

    for (int g0 = 0; g0 < G; g0 += gb) {
        const int ng = min(gb, G - g0);
        // ---- phase 1
        for (int hb = 0; hb < ng; hb += HB) {
            const int nh = min(HB, ng - hb);
            double qd[HB][E];
#pragma unroll
            for (int hh = 0; hh < HB; ++hh) {
                T tmp[E];
                const int h = kvh * G + g0 + hb + (hh < nh ? hh : 0);
                __builtin_memcpy(tmp, __builtin_assume_aligned(qb + (int64_t)h * st.q_h + (int64_t)(ref - t0) * st.q_t + sub * E,
                                                               sizeof(T) * E), sizeof(tmp));
#pragma unroll
                for (int e = 0; e < E; ++e) qd[hh][e] = (double)ldf(&tmp[e]);
            }
            for (int j0 = 0; j0 < wl; j0 += kGroups * UN) {
                T kv[UN][E];
#pragma unroll
                for (int un = 0; un < UN; ++un) {
                    const int j = j0 + un * kGroups + grp;
                    if (j < wl)
                        __builtin_memcpy(kv[un], __builtin_assume_aligned(k + (int64_t)(sq.win_start + j) * st.kv_t + sub * E,
                                                                          sizeof(T) * E), sizeof(kv[un]));
                }
#pragma unroll
                for (int un = 0; un < UN; ++un) {
                    const int j = j0 + un * kGroups + grp;
                    double kd[E];
#pragma unroll
                    for (int e = 0; e < E; ++e) kd[e] = j < wl ? (double)ldf(&kv[un][e]) : 0.0;
#pragma unroll
                    for (int hh = 0; hh < HB; ++hh) {
                        if (hh >= nh) break;
                        double acc = 0.0;
#pragma unroll
                        for (int e = 0; e < E; ++e) acc += qd[hh][e] * kd[e];
                        acc = sum16(acc);
                        if (sub == 0 && j < wl) s_logit[(size_t)(hb + hh) * W + j] = acc / sqrt_d;
                    }
                }
            }
        }
        __syncthreads();
        // ---- phase 2
        for (int hh = wave; hh < ng; hh += NW) {
            const int h = kvh * G + g0 + hh;
            const int64_t hrow = ((int64_t)l * dm.B + b) * dm.Hq + h;
            const double *logit = s_logit + (size_t)hh * W;
            int *elite = s_elite + (size_t)hh * W;
            double lmax = -INFINITY;
            for (int j = lane; j < wl; j += 64) lmax = fmax(lmax, logit[j]);
            const double smax = wave_max(lmax);
            int R = 0;
            for (int j0 = 0; j0 < wl; j0 += 64) {
                const int j = j0 + lane;
                const bool flag = j < wl && exp(logit[j] - smax) >= alpha;
                const unsigned long long bal = __ballot(flag);
                if (flag) {
                    const int pos = R + __popcll(bal & ((1ull << lane) - 1ull));
                    elite[pos] = sq.win_start + j;
                    t.elite_idx[hrow * W + pos] = sq.win_start + j;
                }
                R += __popcll(bal);
            }
            if (lane == 0) t.elite_cnt[hrow] = R;
            // elite-text columns of Eq.7: (max, sum-exp) of every elite row over the elite text keys; each
            // (row, key) logit is a 64-lane dot product.  Up to 8 keys are scored in one batch of loads,
            // longer rows are scored twice (maximum, then sum).  The maximum is kept as the RAW dot
            // product (before the 1/sqrt(d) scale), the sum is of exp((a - max) / sqrt(d)).
            constexpr int kPer = D / 64;  // elements per lane
            const T *q = qb + (int64_t)h * st.q_h;
            for (int r = 0; r < R; ++r) {
                const T *qr = q + (int64_t)(elite[r] - t0) * st.q_t;
                float qv[kPer];
#pragma unroll
                for (int e = 0; e < kPer; ++e) qv[e] = ldf(qr + lane * kPer + e);
                float m = -INFINITY, z = 0.f;
                const int Rr = dm.causal_text ? r + 1 : R;  // keys this row sees: the list is in position order
                if (R <= 8) {
                    float a[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        a[j] = 0.f;
                        if (j < Rr) {
                            const T *kj = k + (int64_t)elite[j] * st.kv_t;
#pragma unroll
                            for (int e = 0; e < kPer; ++e) a[j] = fmaf(qv[e], ldf(kj + lane * kPer + e), a[j]);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (j < Rr) {
                            a[j] = wave_sum(a[j]);
                            m = fmaxf(m, a[j]);
                        }
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (j < Rr) z += expf((a[j] - m) * scale);
                } else {
                    for (int j = 0; j < Rr; ++j) {
                        const T *kj = k + (int64_t)elite[j] * st.kv_t;
                        float a = 0.f;
#pragma unroll
                        for (int e = 0; e < kPer; ++e) a = fmaf(qv[e], ldf(kj + lane * kPer + e), a);
                        m = fmaxf(m, wave_sum(a));
                    }
                    for (int j = 0; j < Rr; ++j) {
                        const T *kj = k + (int64_t)elite[j] * st.kv_t;
                        float a = 0.f;
#pragma unroll
                        for (int e = 0; e < kPer; ++e) a = fmaf(qv[e], ldf(kj + lane * kPer + e), a);
                        z += expf((wave_sum(a) - m) * scale);
                    }
                }
                if (lane == 0) {
                    t.row_mtext[hrow * W + r] = m;
                    t.row_ztext[hrow * W + r] = z;
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------
// Visual observation window (the "visual window" of the ablation table, Tab.5): every token of the span
// is a row of every query head and no text key takes part, so the row lists are written out
// directly and the elite-text columns are empty (maximum -inf, sum 0).  One workgroup per
// (layer, sequence, query head).
__global__ __launch_bounds__(64) void window_rows_kernel(Dims dm, DevTables t, int l0, SeqArgs seqs) {
    const int h = blockIdx.x, b = blockIdx.y, li = blockIdx.z;
    const air_seq sq = seqs.s[b];
    if (li == 0 && h == 0 && threadIdx.x == 0) t.seq_tab[b] = sq;
    const int64_t hrow = ((int64_t)(l0 + li) * dm.B + b) * dm.Hq + h;
    const int W = dm.max_window;
    for (int j = threadIdx.x; j < sq.win_len; j += 64) {
        t.elite_idx[hrow * W + j] = sq.win_start + j;
        t.row_mtext[hrow * W + j] = -INFINITY;
        t.row_ztext[hrow * W + j] = 0.f;
    }
    if (threadIdx.x == 0) t.elite_cnt[hrow] = sq.win_len;
}

hipError_t launch_window_rows(hipStream_t s, const Dims &dm, const DevTables &t, int l0, int nl, const SeqArgs &seqs) {
    hipLaunchKernelGGL(window_rows_kernel, dim3(dm.Hq, dm.B, nl), dim3(64), 0, s, dm, t, l0, seqs);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
hipError_t launch_elite(hipStream_t s, const Dims &dm, const DevTables &t, int l0, int nl, const LaunchLayers &ll,
                        const air_strides &st, const SeqArgs &seqs, double alpha) {
    const size_t per_head = (size_t)dm.max_window * (sizeof(double) + sizeof(int));
    int gb = (int)(49152 / per_head);  // heads whose logits share the LDS
    gb = gb < 1 ? 1 : (gb > dm.G ? dm.G : gb);
    const dim3 grid(dm.Hkv, dm.B, nl);
    auto launch = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), gb * per_head, s, dm, t, l0, ll, st, seqs, alpha, gb);
    };
    // Eight waves where the launch leaves every workgroup a CU of its own and some span has more than 64 candidates (a round of
    // keys for four waves).  air_score, us, four waves / eight, 128 candidates, heads of 128 elements: 112 units of 7 heads 61 / 58, 256
    // of 7 heads 68 / 64, 256 of 1 head 42.5 / 42; 448 units of 2 heads 52 / 56, 768 of 2 heads 74 / 80, 4096 of 7 heads 448 / 491;
    // heads of 64: 256 units of 2 heads 37.5 / 37, 448 of 2 heads 45 / 48, 768 59 / 66, 4096 199 / 249.  The table entries are the
    // same bits either way.
    int most = 0;
    for (int b = 0; b < dm.B; ++b) most = seqs.s[b].win_len > most ? seqs.s[b].win_len : most;
    if (most > 64 && (int64_t)nl * dm.B * dm.Hkv <= kCUs)
        dm.D == 128 ? launch(elite_kernel<float, 128, 8>, 8) : launch(elite_kernel<float, 64, 8>, 8);
    else
        dm.D == 128 ? launch(elite_kernel<float, 128, 4>, 4) : launch(elite_kernel<float, 64, 4>, 4);
    return hipGetLastError();
}

}  // namespace air
