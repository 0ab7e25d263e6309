// What the last kernel of air_score does with the scores of a workgroup, for every storage: moments, unit statistics
// (Eq.9-10) and, from the last unit of a sequence, the allocation of Eq.11.
#pragma once

#include "air_budget_dev.h"
#include "air_device.h"
#include "air_internal.h"

namespace air {

// Eq.10 from the central sums of second and third powers
__device__ __forceinline__ double skewness(int n_vis, double mu, double c2, double c3) {
#pragma clang fp contract(off)
    const double n = (double)n_vis;
    double sk = 0.0;
    if (n_vis >= 3) {
        const double sigma = sqrt(c2 / (n - 1.0));
        // zero spread (Eq.10 undefined; taken as 0): a standard deviation at most 1e-6 of the mean
        if (sigma > 1e-6 * fabs(mu)) sk = n / ((n - 1.0) * (n - 2.0)) * (c3 / (sigma * sigma * sigma));
    }
    return sk;
}

// Eq.9-10 of one (layer, sequence, KV head) from the moment entries of its importance row, by one wave.  Entry c holds
// the sum S1_c, the mean m_c and the moments M2_c, M3_c about m_c of the n_c scores of kFinishChunks chunks.  With
// d_c = m_c - mu the central moments of the row are
//   sum (x - mu)^2 = sum_c M2_c + n_c d_c^2,   sum (x - mu)^3 = sum_c M3_c + 3 d_c M2_c + n_c d_c^3,
// sums of terms no larger than their result (raw power sums would cancel on rows of little spread).  Lane g of each row
// of sixteen lanes takes the entries g, g + 16, ... (the first two stay in registers), the sums over the entries are
// butterflies over the sixteen lanes: a fixed order, the same on every run; every operation is rounded once (no
// contraction: the budgets that follow from these numbers must not depend on how the compiler fuses them).
__device__ __forceinline__ void unit_statistics(__amdgpu_buffer_rsrc_t ers, int n_ent, int n_vis, int lane, double &st_out,
                                                double &sk_out) {
#pragma clang fp contract(off)
    constexpr int kEntryKeys = kFinishChunks * kChunkKeys;
    const int gl = lane & 15;
    auto entry = [&](int c, double (&e)[4]) __attribute__((always_inline)) {
        const int cc = min(c, n_ent - 1);
        const u32x4 lo = __builtin_amdgcn_raw_buffer_load_b128(ers, cc * 32, 0, kSysScope);
        const u32x4 hi = __builtin_amdgcn_raw_buffer_load_b128(ers, cc * 32 + 16, 0, kSysScope);
        const bool have = c < n_ent;
        e[0] = have ? __builtin_bit_cast(double, (u32x2){lo[0], lo[1]}) : 0.0;
        e[1] = have ? __builtin_bit_cast(double, (u32x2){lo[2], lo[3]}) : 0.0;
        e[2] = have ? __builtin_bit_cast(double, (u32x2){hi[0], hi[1]}) : 0.0;
        e[3] = have ? __builtin_bit_cast(double, (u32x2){hi[2], hi[3]}) : 0.0;
    };
    double e0[4], e1[4];
    entry(gl, e0);
    entry(gl + 16, e1);
    const double n = (double)n_vis;
    double s1 = e0[0] + e1[0];
    for (int c = gl + 32; c < n_ent; c += 16) {  // beyond 32768 visual tokens
        double ex[4];
        entry(c, ex);
        s1 += ex[0];
    }
    const double S1 = sum16(s1);
    const double mu = S1 / n;
    double c2 = 0.0, c3 = 0.0;
    auto add = [&](int c, const double (&e)[4]) __attribute__((always_inline)) {
        if (c < n_ent) {
            const double nc = (double)min(kEntryKeys, n_vis - c * kEntryKeys);
            const double dl = e[1] - mu, M2 = e[2], M3 = e[3];
            c2 += M2 + nc * (dl * dl);
            c3 += (M3 + 3.0 * dl * M2) + nc * (dl * dl * dl);
        }
    };
    add(gl, e0);
    add(gl + 16, e1);
    for (int c = gl + 32; c < n_ent; c += 16) {
        double ex[4];
        entry(c, ex);
        add(c, ex);
    }
    c2 = sum16(c2);
    c3 = sum16(c3);
    st_out = S1;
    sk_out = skewness(n_vis, mu, c2, c3);
}

// The statistics of a unit that is complete, by one wave; the last unit of a sequence goes on to Eq.11 (dm.fuse_budget).
__device__ __forceinline__ void leave_unit(const Dims &dm, const DevTables &t, int64_t unit, int b, const air_seq &sq, int lane,
                                           double unit_st, double unit_sk) {
    if (!dm.fuse_budget) {
        if (lane == 0) {
            t.unit_st[unit] = unit_st;
            t.unit_sk[unit] = unit_sk;
        }
        return;
    }
    // The same once more, one level up: the unit's statistics go out written through, the wave counts the unit at
    // its sequence's arrival counter, and the wave that counts the last of the L * H_kv units does Eq.11 and the
    // cache layout of the sequence (the layers fit one wave): air_budget has nothing left to launch.
    const int64_t all_units = (int64_t)dm.L * dm.B * dm.Hkv;
    const __amdgpu_buffer_rsrc_t srs = __builtin_amdgcn_make_buffer_rsrc(t.unit_st, 0, (int)(all_units * 8), 0x00020000);
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(t.unit_sk, 0, (int)(all_units * 8), 0x00020000);
    if (lane == 0) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, unit_st), srs, (int)unit * 8, 0, kSysScope);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, unit_sk), krs, (int)unit * 8, 0, kSysScope);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int prev = 0;
    if (lane == 0) prev = __hip_atomic_fetch_add(&t.seq_cnt[b], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    prev = __builtin_amdgcn_readfirstlane(prev);
    if (prev != dm.L * dm.Hkv - 1) return;
    if (lane == 0) __hip_atomic_store(&t.seq_cnt[b], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next prompt
    __shared__ double s_a0[64], s_a1[64], s_frac[64];
    __shared__ int s_i0[64], s_i1[64];
    allocate_and_lay_out<true>(dm, t, b, sq, dm.retention, dm.budget_mode, dm.min_keep, false, lane, s_a0, s_a1, s_frac,
                               s_i0, s_i1, [&](int l, double &a, double &c) __attribute__((always_inline)) {
                                   // all heads' loads go out together; the sums run left to right over the live ones
                                   u32x2 vs[16], vk[16];
#pragma unroll
                                   for (int h = 0; h < 16; ++h) {
                                       const int off = (int)((((int64_t)l * dm.B + b) * dm.Hkv + min(h, dm.Hkv - 1)) * 8);
                                       vs[h] = __builtin_amdgcn_raw_buffer_load_b64(srs, off, 0, kSysScope);
                                       vk[h] = __builtin_amdgcn_raw_buffer_load_b64(krs, off, 0, kSysScope);
                                   }
#pragma unroll
                                   for (int h = 0; h < 16; ++h) {
                                       if (h < dm.Hkv) {
                                           a += __builtin_bit_cast(double, vs[h]);
                                           c += __builtin_bit_cast(double, vk[h]);
                                       }
                                   }
                               });
}

// Moments of a workgroup's scores, every sum in a fixed order: S1 = sum x, the workgroup mean S1 / n, then
// M2 = sum (x - mean)^2 and M3 = sum (x - mean)^3 in fp64.  One entry (S1, mean, M2, M3) per workgroup (of NW waves).
// x, ok: the thread's own scores and which of them exist (n_wg in the workgroup); n_ent workgroups share the unit.
template <int NX, int NW>
__device__ __forceinline__ void leave_moments(const Dims &dm, const DevTables &t, int64_t unit, int b, const air_seq &sq, int n_wg,
                                              int n_ent, const float (&x)[NX], const bool (&ok)[NX], double (&s_mom)[NW][3]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto over_waves = [&](int slot) {
        double v = s_mom[0][slot];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += s_mom[w][slot];
        return v;
    };
    auto wg_sum = [&](double v, int slot) {
        v = wave_sum(v);
        if (lane == 0) s_mom[wave][slot] = v;
        lds_barrier();
        return over_waves(slot);
    };
    double s1 = 0.0;
#pragma unroll
    for (int i = 0; i < NX; ++i) s1 += ok[i] ? (double)x[i] : 0.0;
    const double S1 = wg_sum(s1, 0);
    const double mean = S1 / (double)n_wg;
    double m2 = 0.0, m3 = 0.0;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const double dlt = ok[i] ? (double)x[i] - mean : 0.0;
        m2 += dlt * dlt;
        m3 += dlt * dlt * dlt;
    }
    m2 = wave_sum(m2);
    m3 = wave_sum(m3);
    if (lane == 0) {
        s_mom[wave][1] = m2;
        s_mom[wave][2] = m3;
    }
    lds_barrier();
    if (wave != 0) return;
    // The entry goes out written through to memory, and the workgroup then counts itself at the unit's arrival
    // counter; the one that counts last (every entry of the unit is in memory by then: each writer waited for its
    // stores before it counted) turns the entries into the unit's strength and skewness.  The ordering is that of
    // the decode kernel's exchange of partials: write-through stores, s_waitcnt, a relaxed device-scope
    // read-modify-write, loads that bypass the caches.
    double *mo_unit = t.moments + unit * dm.n_entries * 4;
    const __amdgpu_buffer_rsrc_t ers = __builtin_amdgcn_make_buffer_rsrc(mo_unit, 0, dm.n_entries * 32, 0x00020000);
    if (lane < 4) {
        const double r = lane == 0 ? S1 : (lane == 1 ? mean : over_waves(lane - 1));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, r), ers, (int)blockIdx.x * 32 + lane * 8, 0, kSysScope);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int prev = 0;
    if (lane == 0) prev = __hip_atomic_fetch_add(&t.unit_cnt[unit], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    prev = __builtin_amdgcn_readfirstlane(prev);
    if (prev != n_ent - 1) return;
    if (lane == 0) __hip_atomic_store(&t.unit_cnt[unit], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next launch
    double unit_st, unit_sk;
    unit_statistics(ers, n_ent, sq.vis_len, lane, unit_st, unit_sk);
    leave_unit(dm, t, unit, b, sq, lane, unit_st, unit_sk);
}

// The same for a workgroup of NW waves that has written scores of its unit, through to memory (all of its waves; n_parts
// workgroups share the unit): the last of them reads the unit's scores back past the caches and forms S1, the mean and the central
// sums from them, in a fixed order, whatever the workgroups' parts were.  A workgroup that has the unit to itself takes the scores from
// s_scores, where its threads left them (thread i the scores i, i + 64 NW, ...): nothing to wait for, to count or to read back.
// s_mom: as above; s_last: an int in LDS.
template <int NW>
__device__ __forceinline__ void leave_scores(const Dims &dm, const DevTables &t, int64_t unit, int b, const air_seq &sq, int n_parts,
                                             const float *s_scores, double (&s_mom)[NW][3], int &s_last) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (n_parts > 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
        if (tid == 0) s_last = __hip_atomic_fetch_add(&t.unit_cnt[unit], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_parts - 1;
        lds_barrier();
        if (!s_last) return;
        if (tid == 0) __hip_atomic_store(&t.unit_cnt[unit], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next launch
    }
    const int n_vis = sq.vis_len;
    float *scores = t.scores + unit * dm.max_vis;
    constexpr int kAtOnce = 16, kStep = 64 * NW;  // reads past the scores give zero
    auto over_waves = [&](int slot) {
        double v = s_mom[0][slot];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += s_mom[w][slot];
        return v;
    };
    float x[kAtOnce];
    auto read = [&](int i0) {
        if (n_parts == 1) {
#pragma unroll
            for (int j = 0; j < kAtOnce; ++j)
                if (i0 + kStep * j < n_vis) x[j] = i0 + kStep * j + tid < n_vis ? s_scores[i0 + kStep * j + tid] : 0.f;
            return;
        }
        // (offsets from i0: those from the row's start leave 32 bits behind at 2^30 scores)
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(scores + i0, 0, min(n_vis - i0, kStep * kAtOnce) * 4, 0x00020000);
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j)
            x[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (kStep * j + tid) * 4, 0, kSysScope));
    };
    double s1 = 0.0;
    for (int i0 = 0; i0 < n_vis; i0 += kStep * kAtOnce) {
        read(i0);
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j)
            if (i0 + kStep * j < n_vis) s1 += (double)x[j];
    }
    s1 = wave_sum(s1);
    if (lane == 0) s_mom[wave][0] = s1;
    lds_barrier();
    const double S1 = over_waves(0), mu = S1 / (double)n_vis;
    double m2 = 0.0, m3 = 0.0;
    for (int i0 = 0; i0 < n_vis; i0 += kStep * kAtOnce) {
        if (n_vis > kStep * kAtOnce) read(i0);  // (else they are still there)
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j) {
            if (i0 + kStep * j >= n_vis) continue;
            const double dlt = i0 + kStep * j + tid < n_vis ? (double)x[j] - mu : 0.0;
            m2 += dlt * dlt;
            m3 += dlt * dlt * dlt;
        }
    }
    m2 = wave_sum(m2);
    m3 = wave_sum(m3);
    if (lane == 0) {
        s_mom[wave][1] = m2;
        s_mom[wave][2] = m3;
    }
    lds_barrier();
    if (wave == 0) leave_unit(dm, t, unit, b, sq, lane, S1, skewness(n_vis, mu, over_waves(1), over_waves(2)));
}

}  // namespace air
