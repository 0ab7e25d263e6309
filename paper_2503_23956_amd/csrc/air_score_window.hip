// air_score, bf16, windows that turn their whole span into rows (a continuous, all-text or visual window of dozens to
// hundreds of rows per unit; bf16 contexts whose workspace holds no stash come here with an elite window too): Eq.6-8 with the ROWS in
// LDS, once per workgroup, and the keys of a wave in its registers, twice.
//
// A workgroup of eight waves takes a part of a unit's keys; its waves share up to 256 window rows in LDS (loaded straight into
// it) and go their own ways: a wave loads 32 keys from memory as MFMA operands, walks the row blocks over them and
// takes its next keys, without a barrier.  Exponentials are 2^(s kC - m): one fused multiply-add and one exponential per
// element, with a reference m that is a whole number, so that references are moved and partial sums merged exactly.
//   pass 1  products of 32 keys x 32 rows: a lane holds 16 logits of ONE window row per block, so that it needs one sum and one
//           reference per block.  References start at the maximum over the first keys of all waves.  Leaves (reference, sum) per
//           (run of keys, row).  A lane whose 16 exponentials add up to more than its limit raises its reference to their
//           maximum and forms them again.
//   pass 2  forms maximum, fp64 normaliser and weight of the unit's rows from the partials, a thread per row, then
//           I[key] = sum over the rows of w 2^(s kC - m): the keys of a wave are complete after the last row block (two steps
//           across the lanes).  The unit's last workgroup forms its statistics from the scores.
// The products of the two passes differ in shape but give a logit the same bits, and have to: a weight would be off by
// 2^(difference) where a key stands above all others.
// Bound (7290 keys, 7 x 32 rows, 28 x 4 units: 448 workgroups of 1856 keys, pass 1 69 us, pass 2 82): instruction issue, 60 % of the clocks
// in pass 1 and 57 % in pass 2 (an exponential takes a SIMD 16 clocks, any other instruction 4; matrix unit 34 and 24 %), on the CUs that
// have two workgroups, by stamps close to all of it between the first keys and the last; then the quarter of the CUs that have one
// workgroup, 4 us in pass 1 and 8 in pass 2 in front of a workgroup's first keys, and 9 behind its last (statistics, allocation).
// What stands in front are dependent accesses, so there are few of them: the rows follow from the window and are requested before the
// counts of the lists are there (without a threshold), and a run's partial sums lie side by side (a thread per row used to touch a line for every one: 5 us).
// With lists read first, partial sums a line apart, references that each wave found for itself and 832 keys a run: 78.5 and 86.8 us.
// Two waves a SIMD with 64 keys each, products between exponentials, take as long for the keys and longer in front (101 and 86).
// Four waves a SIMD need 128 registers: everything in front of the loops is kept out of registers across them (`here`).
// air_score with the elite kernel (14 for 32 x 7), rows a head x heads, us now / with those and an elite kernel that kept no tiles: 7290 keys, 28
// layers x 4 KV heads, 32 x 7 rows 161 / 169, 5 x 7 95 / 97, 512 x 7 3700 / 3970, visual 152 / 159, heads of 64 117 / 128; eight layers 103 / 118;
// 16 prompts of 2304 keys 738 / 762; 65536 keys, 2 units 80 / 96; 28 x 8 x 8 units of 300 keys 183 / 197; 32 x 64 x 8 of 128 keys, 4 x 9 rows 695 /
// 764; 28 layers of 7290 keys one by one 1380 / 1645, visual 1100 / 1280, 5 x 7 rows 903 / 976 (1086 with
// 1856 keys a run, 1113 with four groups of a wave's keys on their way as well).
// Precision: the argument of an exponential is rounded, to 2^-24 of itself, and the largest terms are the ones that count, so a
// reference has to stay near the maximum; and a logit keeps its bits only if its sum starts at zero.  (With sums that
// started at minus the reference, and the lane's first logit as reference up to 2^100, the scores were 9.7e-7 off fp64 in
// place of 4.3e-7 for logits of a spread of 5, 4.0e-6 in place of 8.7e-7 for a spread of 18, heads of 128.)
#include "air_score_mfma_dev.h"

#include <type_traits>

namespace air {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kWinRows = 256;                  // rows in LDS at a time
constexpr int kPartLeast = 512, kPartMost = 2048;  // keys of a workgroup
constexpr int kTiles = 2;                      // pass 2: tiles of 16 keys in a wave's registers
// Beyond 2^22 a reference and a logit no longer differ by what fp32 says they do (raw logits of 3e7: keys masked by a large
// negative number, operands in the thousands).  References stop there; logits below weigh nothing, logits above are
// held at the bound: in pass 1 where exponentials are formed again, in pass 2 by a plain loop over the rows that have such a
// reference.  -2^22 is also where a reference starts: the first logits above it raise it.
constexpr float kFar = 0x1p22f;
template <int D>
__device__ __forceinline__ float held(float s) {
    constexpr float kFarRaw = kFar / Log2Scale<D>::kHi;
    return s > kFarRaw ? kFarRaw : (s < -kFarRaw ? -kFarRaw : s);
}

// Rows in LDS: place p of row r holds its 16-byte piece p ^ swizzle(r), so that the sixteen rows that a read of one piece
// touches lie in different banks.
template <int D>
__device__ __forceinline__ int row_swizzle(int row) {
    return D == 128 ? row & 15 : (row >> 1) & 7;
}

__device__ __forceinline__ int ilogb_of(float x) { return (int)(__float_as_uint(x) >> 23) - 127; }  // of a normal number above 0

// the lane's 16 bytes of row n of a block in LDS, slice by slice
template <int D>
__device__ __forceinline__ void row_places(int n, int c, int (&row_at)[D / 32]) {
#pragma unroll
    for (int sl = 0; sl < D / 32; ++sl) row_at[sl] = n * D + 8 * ((4 * sl + c) ^ row_swizzle<D>(n));
}

// A value that the compiler takes as new: what follows from it is formed where it is used, not in front of the loop around
// (held in registers there it was spilled, and a spill in the prologue costs microseconds).
__device__ __forceinline__ int here(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// the keys of a wave's group as MFMA operands; keys past the end of the span repeat the last one
template <int TILES, int NS>
__device__ __forceinline__ void group_keys(const UnitCtx &u, const air_strides &st, int key0, uint4 (&kreg)[TILES][NS]) {
    const int lane = here(threadIdx.x & 63), n = lane & 15, c = lane >> 4;
#pragma unroll
    for (int tile = 0; tile < TILES; ++tile) {
        const bf16_t *src = u.k + (int64_t)(u.sq.vis_start + min(key0 + 16 * tile + n, u.sq.vis_len - 1)) * st.kv_t + 8 * c;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) kreg[tile][sl] = *reinterpret_cast<const uint4 *>(src + 32 * sl);
    }
}

// a row's query: head of the group and place in the window, as one word in LDS (u.q: at the window's first token)
static_assert(AIR_MAX_TEXT <= 1 << 27, "the places of a window and sixteen heads in a word");
__device__ __forceinline__ const bf16_t *query_of(const UnitCtx &u, const air_strides &st, int word) {
    return u.q + (int64_t)(u.kvh * u.G + (int)((unsigned)word >> 27)) * st.q_h + (int64_t)(word & 0x7ffffff) * st.q_t;
}

// The unit's rows.  Without a threshold a window has every token of its span as a row of every head, but for logits that are no
// numbers (`whole`): the rows are then taken from the window itself and requested while the counts of the lists are on their way, and
// only where a count says otherwise are they taken from the lists (WHOLE).  With a threshold (contexts whose workspace holds no stash) they are a few
// of the window's, and the lists come first: air_score of 28 x 8 x 4 units, 4 heads of 64, 2304 keys, 128 text tokens, 133 us, with the window's rows
// in front of them 152; 24 x 2 units of 7 heads, 7290 keys 44.4 and 48.3.
__device__ __forceinline__ int rows_of_unit(const DevTables &t, UnitCtx &u, bool whole, int *s_pref) {  // also: rows of head `lane` of the group
    const int lane = threadIdx.x & 63;
    if (!whole) {
        head_prefix(t, u.hrow0, u.G, s_pref);
        u.R_total = s_pref[u.G];
        return 0;
    }
    u.R_total = u.G * u.sq.win_len;
    return t.elite_cnt[u.hrow0 + min(lane, u.G - 1)];
}
__device__ __forceinline__ int2 row_of(const UnitCtx &u, const int *s_pref, bool whole, int rho) {
    if (whole) {  // rho / win_len: rho < 2^16, and (rho + 1/2) / win_len is farther from a whole number than it can be off by
        const int g = (int)(((float)rho + 0.5f) * __builtin_amdgcn_rcpf((float)u.sq.win_len));
        return make_int2(g, rho - g * u.sq.win_len);
    }
    const int g = head_of_row(s_pref, u.G, rho);
    return make_int2(g, rho - s_pref[g]);
}
__device__ __forceinline__ int query_word(const DevTables &t, const UnitCtx &u, bool whole, int2 row) {
    const int tok = whole ? row.y : t.elite_idx[(u.hrow0 + row.x) * u.W + row.y] - u.sq.win_start;
    return (int)((unsigned)row.x << 27 | (unsigned)tok);
}

// The rows of a workgroup straight into LDS, n_load of them (whole blocks; those past the list repeat the last one); the
// caller waits for them.
template <int D>
__device__ __forceinline__ void load_rows_lds(const UnitCtx &u, const air_strides &st, const int *s_query, bf16_t *s_rows, int n_rows, int n_load, int wave) {
    typedef __attribute__((address_space(1))) void gptr_t;
    typedef __attribute__((address_space(3))) void lptr_t;
    constexpr int kPieces = D / 8, kRowsOfWave = 64 / kPieces, kStep = kRowsOfWave * kWaves, kIt = kWinRows / kStep;
    const int lane = here(threadIdx.x & 63);
    int word[kIt];
#pragma unroll
    for (int i = 0; i < kIt; ++i) word[i] = s_query[min(kStep * i + kRowsOfWave * wave + lane / kPieces, n_rows - 1)];
#pragma unroll
    for (int i = 0; i < kIt; ++i) {
        const int row0 = kStep * i + kRowsOfWave * wave;
        if (row0 >= n_load) break;
        const int row = row0 + lane / kPieces;  // lane i's 16 bytes land at the place of lane 0's + 16 i
        const bf16_t *src = query_of(u, st, word[i]) + 8 * ((lane % kPieces) ^ row_swizzle<D>(row));
        __builtin_amdgcn_global_load_lds((gptr_t *)src, (lptr_t *)(s_rows + row0 * D), 16, 0, 0);
    }
}
// Partial sums of a unit: a run's rows side by side (row r of head g at g W + r), so that a thread per row reads whole lines.
__device__ __forceinline__ float2 *unit_parts(const Dims &dm, const DevTables &t, const UnitCtx &u) { return t.part + u.hrow0 * u.W * dm.n_chunks; }

__device__ __forceinline__ void rows_wait_barrier() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
}

// ---------------------------------------------------------------------------------------
// Pass 1.  A workgroup takes a run of run_keys keys of a unit and one of `shares` shares of its rows.  Products of 32 keys x 32 rows: lane (n, c),
// n = lane % 32, holds sixteen logits of row n.
constexpr int kBlocks1 = kWinRows / 32;
template <int D, bool WHOLE>
__global__ __launch_bounds__(kThreads, 4) void window_sums_kernel(Dims dm, DevTables t, int l0, LaunchLayers ll, air_strides st, SeqArgs seqs,
                                                               int run_keys, int shares, uint32_t inv_shares, int share_rows) {
    constexpr int NS = D / 16, kGroup = 32;
    constexpr float kC = Log2Scale<D>::kHi;
    constexpr float kSumLimit = 64.0f;  // of a lane's exponentials of a block
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    UnitCtx u;
    const int run = inv_shares ? (int)__umulhi(blockIdx.x, inv_shares) : (int)blockIdx.x;
    if (!unit_setup(dm, seqs, l0, ll, st, u, 0) || run * run_keys >= u.sq.vis_len) return;
    u.q += (int64_t)(u.sq.win_start - u.qbase) * st.q_t;
    __shared__ int s_pref[17];
    __shared__ __align__(16) bf16_t s_rows[kWinRows * D];
    __shared__ int s_slot[kWinRows];  // a row's place in the unit's row tables
    __shared__ int s_query[kWinRows];
    __shared__ int s_last[kWinRows];  // last key that a row sees
    static_assert(kWaves * kWinRows * sizeof(float2) <= sizeof(s_rows), "the partial sums of the waves take the place of the rows");
    __shared__ int s_top[kWinRows];  // a row's first reference
    // a visual-window row at visual index p sees the keys up to p: keys behind the last row are never looked at
    const int prow0 = u.sq.win_start - u.sq.vis_start;
    const int key_first = run * run_keys + 32 * wave;
    const int key_hi = min((run + 1) * run_keys, dm.vis_window ? prow0 + u.sq.win_len : u.sq.vis_len);
    // the keys of the wave's next group, 16 elements a slice, eight of them in either half of the wave; requested at the end of
    // the group before
    uint4 kreg[NS];
    auto load_keys = [&](int key0) __attribute__((always_inline)) {
        const int lane = here(threadIdx.x & 63);
        const bf16_t *src = u.k + (int64_t)(u.sq.vis_start + min(key0 + (lane & 31), key_hi - 1)) * st.kv_t + 8 * (lane >> 5);
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) kreg[sl] = *reinterpret_cast<const uint4 *>(src + 16 * sl);
    };
    bool whole = WHOLE;
    const int count = rows_of_unit(t, u, whole, s_pref);
    // the workgroup's rows: whole blocks of 32 (a block's rows share their raised references: blocks are the same however the rows are dealt)
    const int row_lo = ((int)blockIdx.x - run * shares) * share_rows;
    int row_hi = min(u.R_total, row_lo + share_rows);
    for (int r0 = row_lo; r0 < row_hi; r0 += kWinRows) {
        int rows_here = min(kWinRows, row_hi - r0);
        const int tid = here(threadIdx.x);
        while (true) {
            if (tid < rows_here) {
                const int2 row = row_of(u, s_pref, whole, r0 + tid);
                s_slot[tid] = row.x * u.W + row.y;
                s_last[tid] = dm.vis_window ? prow0 + row.y : u.sq.vis_len - 1;
                s_query[tid] = query_word(t, u, whole, row);
            }
            lds_barrier();
            load_rows_lds<D>(u, st, s_query, s_rows, rows_here, (rows_here + 31) & ~31, wave);
            if (!whole || __ballot(count != u.sq.win_len) == 0ull) break;
            whole = false;
            rows_wait_barrier();
            head_prefix(t, u.hrow0, u.G, s_pref);
            u.R_total = s_pref[u.G];
            row_hi = min(u.R_total, row_lo + share_rows);
            rows_here = min(kWinRows, row_hi - r0);
            if (rows_here <= 0) return;
        }
        const int n_blk = (rows_here + 31) >> 5;
        if (tid < kWinRows) s_top[tid] = -(int)kFar;
        rows_wait_barrier();
        float ref[kBlocks1], sum[kBlocks1];  // of row 32 b + n
        // the logits of the wave's keys and every block of rows, and what is done with them
        auto logits = [&](int key0, auto masked, auto take) __attribute__((always_inline)) {
            asm volatile("" ::: "memory");  // the rows are read from LDS for every group: as values of the loop they would be spilled
            const int lane = here(threadIdx.x & 63), n = lane & 31, c = lane >> 5;
            int row_at[NS];  // the lane's 16 bytes of row n of a block
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) row_at[sl] = n * D + 8 * ((2 * sl + c) ^ row_swizzle<D>(n));
#pragma unroll
            for (int b = 0; b < kBlocks1; ++b) {
                if (b >= n_blk) break;
                f32x16 s = (f32x16){0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int sl = 0; sl < NS; ++sl) {
                    const uint4 qb = *reinterpret_cast<const uint4 *>(s_rows + 32 * b * D + row_at[sl]);
                    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kreg[sl]), __builtin_bit_cast(bf16x8, qb), s, 0, 0, 0);
                }
                if constexpr (decltype(masked)::value) {  // some keys do not exist or lie behind the row
                    const int lim = s_last[min(32 * b + n, rows_here - 1)] - key0 - 4 * c;
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[i] = 8 * (i >> 2) + (i & 3) > lim ? -INFINITY : s[i];  // key 8 (i / 4) + 4 c + i % 4
                }
                take(b, s);
            }
        };
        constexpr float kFarRaw = kFar / kC;
        // the largest of the lane's logits, as a reference
        auto top_of = [&](const f32x16 &s, float &m) __attribute__((always_inline)) {
            m = -kFarRaw;
#pragma unroll
            for (int i = 0; i < 16; ++i) m = fmaxf(m, s[i]);
            return rintf(fminf(m, kFarRaw) * kC);
        };
        auto for_keys = [&](int key0, auto take) __attribute__((always_inline)) {
            if (key0 + kGroup > u.sq.vis_len || (dm.vis_window && key0 + kGroup > prow0 + 1)) logits(key0, std::true_type(), take);
            else logits(key0, std::false_type(), take);
        };
        load_keys(key_first);
        // The first reference of a row: its maximum over the first keys of all waves.  (Products are cheap here, a reference that
        // turns out too low is not: the exponentials of its block are formed a second time.)  With up to two groups a wave it costs
        // more than it saves, and a lane starts from the maximum of its own first keys: 28 x 8 x 8 units of 300 keys, 8 x 20 rows, 207
        // us with shared references, 199 without; 28 x 16 x 4 units of 2304 keys, 7 x 32 rows, 751 and 773.
        const bool shared_first = key_hi - run * run_keys > 2 * kGroup * kWaves;
        if (shared_first && key_first < key_hi) {
            for_keys(key_first, [&](int b, f32x16 &s) __attribute__((always_inline)) {
                float m;
                const float top = top_of(s, m);
                atomicMax(&s_top[32 * b + (here(threadIdx.x) & 31)], (int)top);
            });
        }
        lds_barrier();
#pragma unroll
        for (int b = 0; b < kBlocks1; ++b) {
            ref[b] = (float)s_top[32 * b + (tid & 31)];
            sum[b] = 0.f;
        }
        for (int key0 = key_first; key0 < key_hi; key0 += kGroup * kWaves) {
            for_keys(key0, [&](int b, f32x16 &s) __attribute__((always_inline)) {
                auto exps = [&](float r) __attribute__((always_inline)) {
                    f32x4 z;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float e = __builtin_amdgcn_exp2f(fmaf(s[i], kC, -r));
                        z[i & 3] = i < 4 ? e : z[i & 3] + e;
                    }
                    return (z[0] + z[1]) + (z[2] + z[3]);
                };
                float z = kSumLimit;  // no reference yet: whatever the exponentials above the lowest one are
                if (shared_first || key0 != key_first) z = exps(ref[b]);
                if (__ballot(z >= kSumLimit) != 0ull) {
                    // the lane's reference becomes its largest logit, if that lies above; logits above the bound are held at it
                    float m;
                    const float up = fmaxf(ref[b], top_of(s, m));
                    if (__ballot(m > kFarRaw) != 0ull) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) s[i] = s[i] > kFarRaw ? kFarRaw : s[i];
                    }
                    sum[b] = ldexpf(sum[b], (int)(ref[b] - up));
                    ref[b] = up;
                    z = exps(up);
                }
                sum[b] += z;
            });
            load_keys(key0 + kGroup * kWaves);  // (the last key again where there are none)
        }
        // one (reference, sum) per row: over the two lanes that share it, then over the waves, a thread per row.  (A lane or wave without a term has the lowest reference.)
        auto merge = [](float &M, float &z, float m2, float z2) __attribute__((always_inline)) {
            const float top = fmaxf(M, m2);
            z = ldexpf(z, (int)(M - top)) + ldexpf(z2, (int)(m2 - top));
            M = top;
        };
        lds_barrier();  // the rows have been read: their place holds the waves' references and sums
        float2(*s_part)[kWinRows] = reinterpret_cast<float2(*)[kWinRows]>(s_rows);
        const int lane = tid & 63;
#pragma unroll
        for (int b = 0; b < kBlocks1; ++b) {
            if (b >= n_blk) break;
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(ref[b]), __float_as_uint(ref[b]), false, false);
            const auto z = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[b]), __float_as_uint(sum[b]), false, false);
            float M = __uint_as_float(r[0]), Z = __uint_as_float(z[0]);
            merge(M, Z, __uint_as_float(r[1]), __uint_as_float(z[1]));
            if (lane < 32) s_part[wave][32 * b + lane] = make_float2(M, Z);
        }
        lds_barrier();
        if (tid < rows_here) {
            // (in fp64: a lane adds up 1856 keys of a run in seven or eight steps, 832 in three or four; with that and the eight waves added up
            // in fp32 scores of logits of a spread of 1 were 2.2 % further off fp64)
            float2 x = s_part[0][tid];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) x.x = fmaxf(x.x, s_part[w][tid].x);
            double z = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) z += (double)ldexpf(s_part[w][tid].y, (int)(s_part[w][tid].x - x.x));
            x.y = (float)z;
            // (the sum goes out as a fraction of 1 to 2: pass 2 takes the largest reference of a row, which its terms then stay below)
            const int up = x.y > 0.f && x.y < INFINITY ? ilogb_of(x.y) : 0;
            unit_parts(dm, t, u)[(int64_t)run * u.G * u.W + s_slot[tid]] =
                make_float2(x.y > 0.f ? x.x + (float)up : -INFINITY, ldexpf(x.y, -up));
        }
        lds_barrier();  // the partials have been read: the next group of rows may come
    }
}

// ---------------------------------------------------------------------------------------
// Pass 2.  A workgroup takes part_keys keys of a unit.
template <int D, bool WHOLE>
__global__ __launch_bounds__(kThreads, 4) void window_scores_kernel(Dims dm, DevTables t, int l0, LaunchLayers ll, air_strides st, SeqArgs seqs,
                                                                 int run_keys, int part_keys) {
    constexpr int NS = D / 32, T = kTiles, kGroup = 16 * T;
    constexpr float kC = Log2Scale<D>::kHi;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, c = lane >> 4;
    UnitCtx u;
    if (!unit_setup(dm, seqs, l0, ll, st, u, 0) || (int)blockIdx.x * part_keys >= u.sq.vis_len) return;
    u.q += (int64_t)(u.sq.win_start - u.qbase) * st.q_t;
    __shared__ int s_pref[17];
    __shared__ __align__(16) bf16_t s_rows[kWinRows * D];
    __shared__ __align__(16) float s_M[kWinRows], s_w[kWinRows];
    __shared__ __align__(16) float s_ref[kWinRows];  // minus s_M; -inf for a row that the plain loop takes
    __shared__ __align__(16) int s_last[kWinRows];   // last key that a row sees
    __shared__ int s_query[kWinRows];
    __shared__ float s_imp[kPartMost];
    __shared__ int s_any_far;  // some row has its reference at the bound
    __shared__ double s_mom[kWaves][3];
    __shared__ int s_is_last;
    const int n_seg = (u.sq.vis_len + run_keys - 1) / run_keys;
    const int prow0 = u.sq.win_start - u.sq.vis_start;
    const int key_lo = (int)blockIdx.x * part_keys;
    const int key_hi = min(key_lo + part_keys, dm.vis_window ? prow0 + u.sq.win_len : u.sq.vis_len);
    uint4 kreg[T][NS];  // the keys of the wave's next group
    if (tid == 0) s_any_far = 0;
    if (!WHOLE)
        for (int i = tid; i < part_keys; i += kThreads) s_imp[i] = 0.f;
    // (Known to be true at first, the compiler reserves 68 bytes of scratch a lane that no instruction touches; as a value it does not know, 28 x 16 x 4
    // units of 128 keys, 4 x 9 rows take 94.5 us in place of 91.8.)
    bool whole = WHOLE;
    const int count = rows_of_unit(t, u, whole, s_pref);
    for (int r0 = 0; r0 < u.R_total; r0 += kWinRows) {
        int rows_here = min(kWinRows, u.R_total - r0);
        const int tid = here(threadIdx.x);
        int2 row = make_int2(0, 0);  // of the thread
        while (true) {
            if (tid < rows_here) {
                row = row_of(u, s_pref, whole, r0 + tid);
                s_query[tid] = query_word(t, u, whole, row);
            }
            lds_barrier();
            load_rows_lds<D>(u, st, s_query, s_rows, rows_here, (rows_here + 15) & ~15, wave);
            if (!whole || __ballot(count != u.sq.win_len) == 0ull) break;
            whole = false;
            rows_wait_barrier();
            head_prefix(t, u.hrow0, u.G, s_pref);
            u.R_total = s_pref[u.G];
            rows_here = min(kWinRows, u.R_total);
            if (rows_here <= 0) break;
        }
        if (WHOLE && r0 == 0)
            for (int i = tid; i < part_keys; i += kThreads) s_imp[i] = 0.f;
        if (rows_here <= 0) {  // no row: the scores are zero
            lds_barrier();
            break;
        }
        const int n_blk = (rows_here + 15) >> 4;
        if (tid < 16 * n_blk) {  // maximum, normaliser, weight
            float M = -INFINITY, w = 0.f;
            const int tid = here(threadIdx.x);
            if (tid < rows_here) {
                const int place = row.x * u.W + row.y;
                const int64_t slot = u.hrow0 * u.W + place, stride = (int64_t)u.G * u.W;
                const float2 *part = unit_parts(dm, t, u) + place;
                const float mt = t.row_mtext[slot], zt = t.row_ztext[slot];  // of raw logits
                constexpr int kAtOnce = 16;  // partials requested together
                float2 x[kAtOnce];
#pragma unroll
                for (int s = 0; s < kAtOnce; ++s) {
                    x[s] = make_float2(-INFINITY, 0.f);
                    if (s < n_seg) x[s] = part[s * stride];
                }
                M = mt > -INFINITY ? rintf(held<D>(mt) * kC) : -INFINITY;
#pragma unroll
                for (int s = 0; s < kAtOnce; ++s) M = fmaxf(M, x[s].x);
                constexpr int kMore = 8;  // of those behind
#pragma unroll 1
                for (int s0 = kAtOnce; s0 < n_seg; s0 += kMore) {
                    float y[kMore];
#pragma unroll
                    for (int s = 0; s < kMore; ++s) y[s] = part[min(s0 + s, n_seg - 1) * stride].x;
#pragma unroll
                    for (int s = 0; s < kMore; ++s) M = fmaxf(M, y[s]);
                }
                double Z = 0.0;
#pragma unroll
                for (int s = 0; s < kAtOnce; ++s) Z += x[s].y > 0.f ? (double)ldexpf(x[s].y, (int)(x[s].x - M)) : 0.0;
#pragma unroll 1
                for (int s0 = kAtOnce; s0 < n_seg; s0 += kMore) {
                    float2 y[kMore];
#pragma unroll
                    for (int s = 0; s < kMore; ++s) y[s] = part[min(s0 + s, n_seg - 1) * stride];
#pragma unroll
                    for (int s = 0; s < kMore; ++s) Z += s0 + s < n_seg && y[s].y > 0.f ? (double)ldexpf(y[s].y, (int)(y[s].x - M)) : 0.0;
                }
                if (zt > 0.f) Z += (double)(zt * __builtin_amdgcn_exp2f(fmaf(held<D>(mt), kC, -M)));
                if (fabsf(M) > 0.5f * kFar && M > -INFINITY) s_any_far = 1;
                w = !(Z <= 0.0) ? (float)(1.0 / ((double)(whole ? u.sq.win_len : s_pref[row.x + 1] - s_pref[row.x]) * (double)u.G * Z)) : 0.f;
                if (!(Z > 0.0)) M = 0.f;  // a row that sees no key but far ones weighs nothing
            }
            s_M[tid] = tid < rows_here ? M : 0.f;
            s_ref[tid] = fabsf(M) > 0.5f * kFar ? -INFINITY : -M;  // (so does a row past the list)
            s_w[tid] = w;
            // (a row past the list sees what the unit's last row sees: its weight is 0, but a key behind the window may be NaN or infinite)
            s_last[tid] = dm.vis_window ? prow0 + (tid < rows_here ? row.y : u.sq.win_len - 1) : u.sq.vis_len - 1;
        }
        rows_wait_barrier();
        group_keys<T, NS>(u, st, key_lo + kGroup * wave, kreg);
        auto group = [&](int key0, auto masked) __attribute__((always_inline)) {
            asm volatile("" ::: "memory");
            const int lane = here(threadIdx.x & 63), n = lane & 15, c = lane >> 4;
            int row_at[NS];
            row_places<D>(n, c, row_at);
            float acc[T] = {};  // key 16 tile + n, the rows of lane group c
            auto block = [&](int b, auto last_block, float(&out)[T]) __attribute__((always_inline)) {
                uint4 qa[NS];
#pragma unroll
                for (int sl = 0; sl < NS; ++sl) qa[sl] = *reinterpret_cast<const uint4 *>(s_rows + 16 * b * D + row_at[sl]);
                f32x4 s[T];
#pragma unroll
                for (int tile = 0; tile < T; ++tile) {
                    s[tile] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int sl = 0; sl < NS; ++sl) s[tile] = mma<bf16_t>(qa[sl], kreg[tile][sl], s[tile]);
                }
                // the next group's keys (or the first's again, for the next group of rows) behind the last products of this one
                if constexpr (decltype(last_block)::value)
                    group_keys<T, NS>(u, st, key0 + kGroup * kWaves < key_hi ? key0 + kGroup * kWaves : key_lo + kGroup * wave, kreg);
                const f32x4 ref = *reinterpret_cast<const f32x4 *>(s_ref + 16 * b + 4 * c);
                const f32x4 w = *reinterpret_cast<const f32x4 *>(s_w + 16 * b + 4 * c);
                typedef __attribute__((ext_vector_type(4))) int i32x4;
                i32x4 last;
                if constexpr (decltype(masked)::value) last = *reinterpret_cast<const i32x4 *>(s_last + 16 * b + 4 * c);
#pragma unroll
                for (int tile = 0; tile < T; ++tile) {
                    float sum = 0.f;  // of the block: one long chain of additions would be 5 % further off fp64 where all keys weigh alike
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (decltype(masked)::value)
                            if (key0 + 16 * tile + n > last[i]) s[tile][i] = -INFINITY;
                        const float e = __builtin_amdgcn_exp2f(fmaf(s[tile][i], kC, ref[i]));
                        sum = i == 0 ? w[0] * e : fmaf(w[i], e, sum);
                    }
                    out[tile] = sum;
                }
            };
            // (Blocks join the sum of a key in pairs: 14 of them one by one were 2.5 % further off fp64 where all keys weigh alike, and no faster.)
            int b = 0;
#pragma unroll 1
            for (; b + 1 < n_blk - 1; b += 2) {
                float first[T], second[T];
                block(b, std::false_type(), first);
                block(b + 1, std::false_type(), second);
#pragma unroll
                for (int tile = 0; tile < T; ++tile) acc[tile] += first[tile] + second[tile];
            }
            float rest[T] = {}, last[T];
            if (b < n_blk - 1) block(b, std::false_type(), rest);
            block(n_blk - 1, std::true_type(), last);
#pragma unroll
            for (int tile = 0; tile < T; ++tile) acc[tile] += rest[tile] + last[tile];
            // over the lane groups; lane (n, c), c < T, stores key 16 c + n
            float v = 0.f;
#pragma unroll
            for (int tile = 0; tile < T; ++tile) {
                float a = acc[tile];
                a += __shfl_xor(a, 16, 64);
                a += __shfl_xor(a, 32, 64);
                if (c == tile) v = a;
            }
            if (c < T) s_imp[key0 - key_lo + lane] += v;
        };
        for (int key0 = key_lo + kGroup * wave; key0 < key_hi; key0 += kGroup * kWaves) {
            if (key0 + kGroup > u.sq.vis_len || (dm.vis_window && key0 + kGroup > prow0 + 1)) group(key0, std::true_type());
            else group(key0, std::false_type());
        }
        lds_barrier();  // the rows and their parameters have been read, the sums are in place
        if (s_any_far) {
            for (int r = 0; r < rows_here; ++r) {
                const float M = s_M[r], w = s_w[r];
                if (fabsf(M) <= 0.5f * kFar) continue;
                const int last_key = s_last[r];
                for (int i = tid; i < part_keys && key_lo + i <= last_key; i += kThreads) {
                    const bf16_t *kr = u.k + (int64_t)(u.sq.vis_start + key_lo + i) * st.kv_t, *qr = query_of(u, st, s_query[r]);
                    float s = 0.f;
#pragma unroll 1
                    for (int e = 0; e < D; e += 8)
                        s = dot_piece<bf16_t>(*reinterpret_cast<const uint4 *>(qr + e), *reinterpret_cast<const uint4 *>(kr + e), s);
                    s_imp[i] += w * __builtin_amdgcn_exp2f(fmaf(held<D>(s), kC, -M));
                }
            }
        }
        lds_barrier();  // s_any_far and the parameters have been read: the next group of rows may come
    }
    const int n_here = min(part_keys, u.sq.vis_len - key_lo);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(t.scores + u.unit * dm.max_vis + key_lo, 0, n_here * 4, 0x00020000);
    for (int i = tid; i < n_here; i += kThreads)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, s_imp[i]), rs, i * 4, 0, kSysScope);
    leave_scores(dm, t, u.unit, u.b, u.sq, (u.sq.vis_len + part_keys - 1) / part_keys, s_imp, s_mom, s_is_last);
}

// Keys of a workgroup, a multiple of 64 from kPartLeast to kPartMost.  Two workgroups share a CU, 512 the chip: as many parts of max_vis
// as make the rounds of 512 times the work of one least.  A round costs the keys and about `extra` groups of 64 keys for what is in
// front and behind (rows into LDS, parameters, partial sums).
constexpr int kPartExtra = 8;
static int part_keys(const Dims &dm, int64_t units, int most = kPartMost, int extra = kPartExtra) {
    const int groups = (dm.max_vis + 63) / 64;
    int best = most / 64;
    int64_t best_cost = -1;
    for (int g = most / 64; g >= kPartLeast / 64; --g) {
        const int64_t cost = (units * ((groups + g - 1) / g) + 511) / 512 * (g + extra);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = g;
        }
    }
    return 64 * best;
}

// Keys of a run of pass 1.  It decides references and partial sums, so it follows from the context alone, not from the layers of the call:
// the scores are the same bits however the layers are cut into calls and launches.  Runs as long as parts suit a call of all layers (7290 keys,
// 28 x 4 units, 7 x 32 rows: pass 1 70 us with 1856 keys a run, 78 with 832).  In a call of one layer a run's rows go to several workgroups
// (below); up to three blocks of rows are too few for that: there a workgroup is bound by the keys that its CU can fetch, and runs are shorter.  air_score
// of all layers / one by one, long and shorter runs, us: 28 x 4 units of 7290 keys, 7 heads of 5 rows 93.5 / 1086 and 96.0 / 902, of 13 rows 100 /
// 1110 and 103 / 929, visual 94.5 / 980 and 98 / 797; 40 x 8 units of 16384 keys, 8 x 12 rows 568 / 1935 and 573 / 1820; with four blocks (7 x 18 rows) all
// layers take 107.9 and 113.7.  With a threshold (no stash) the rows of a unit are not known here: 28 x 8 x 4 units of 2304 keys, heads of 64, take 131 / 863
// with runs of 1152 keys, 141 / 804 with 768.
constexpr int kFewRows = 96, kRunMost = 1536, kRunExtra = 4;
static int run_keys(const Dims &dm) {
    const int64_t units = (int64_t)dm.L * dm.B * dm.Hkv;
    return dm.G * dm.max_window <= kFewRows ? part_keys(dm, units, kRunMost, kRunExtra) : part_keys(dm, units);
}

// Workgroups among which the rows of a run are dealt in pass 1, whole blocks of 32: a call of few units (a layer of a context whose runs
// are as long as a call of all layers likes them) would otherwise leave most of the chip idle.  As many as leave every workgroup a CU:
// air_score of one layer after the other, in 1 / 2 / 3 / 4 / 7 shares, 7290 keys, 28 x 4 units, 7 x 32 rows (16 runs) 1788 / 1535 / 1461 / 1425 / 1403
// us, 16384 keys, 40 x 8 units, 8 x 32 rows (64 runs) 3236 / 2693 / 2541 / 2607 / 3055.
static int rows_of_share(const Dims &dm, int64_t runs) {
    const int blocks = (dm.G * dm.max_window + 31) / 32;
    int shares = (int)(runs < kCUs ? kCUs / runs : 1);
    shares = shares < blocks ? shares : blocks;
    return 32 * ((blocks + shares - 1) / shares);
}

template <int D, bool WHOLE>
static hipError_t window_launch(hipStream_t s, const Dims &dm, const DevTables &t, int pass, int l0, int nl, const LaunchLayers &ll,
                                const air_strides &st, const SeqArgs &seqs) {
    // Pass 2 leaves whole sums of a key and the unit's statistics from whole units: its parts follow the launch.
    const int64_t units = (int64_t)nl * dm.B * dm.Hkv;
    const int run = run_keys(dm);
    const dim3 block(kThreads);
    if (pass == 1) {
        const int n_runs = (dm.max_vis + run - 1) / run, share_rows = rows_of_share(dm, units * n_runs);
        const int shares = (dm.G * dm.max_window + share_rows - 1) / share_rows;
        const uint32_t inv = shares > 1 ? (uint32_t)(0x100000000ull / (uint64_t)shares) + 1u : 0u;  // n_runs * shares is small then
        hipLaunchKernelGGL((window_sums_kernel<D, WHOLE>), dim3(n_runs * shares, dm.Hkv, nl * dm.B), block, 0, s, dm, t, l0, ll, st, seqs, run,
                           shares, inv, share_rows);
    } else {
        const int part = part_keys(dm, units);
        hipLaunchKernelGGL((window_scores_kernel<D, WHOLE>), dim3((dm.max_vis + part - 1) / part, dm.Hkv, nl * dm.B), block, 0, s, dm, t, l0, ll,
                           st, seqs, run, part);
    }
    return hipGetLastError();
}

hipError_t launch_score_window(hipStream_t s, const Dims &dm, const DevTables &t, int pass, int l0, int nl, const LaunchLayers &ll,
                               const air_strides &st, const SeqArgs &seqs, bool whole) {
    auto launch = dm.D == 128 ? (whole ? window_launch<128, true> : window_launch<128, false>) : (whole ? window_launch<64, true> : window_launch<64, false>);
    return launch(s, dm, t, pass, l0, nl, ll, st, seqs);
}

}  // namespace air
