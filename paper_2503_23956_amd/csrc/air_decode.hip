// air_decode_attn: Eq.2 append, then softmax(q K'^T / sqrt(d)) V' over the compacted cache.
//
//   decode_mfma_kernel ONE launch per call, for both storage types and head sizes: one workgroup per (split, unit), the
//                      grid laid out so that no block index needs an integer division.
//                      The tiled K' and the block-transposed V' go from global memory straight
//                      into MFMA operands, every load instruction reading 1 KB of consecutive
//                      memory; the G query heads of the group are the second MFMA dimension.
//                      The token the call appends (Eq.2) is scored from k_new / v_new by one wave
//                      of the split that owns its row, which also stores it into the cache; the
//                      workgroup of a unit that finishes last merges the unit's split-K partials.
#include "air_device.h"
#include "air_internal.h"
#include "air_tile.h"

#include <mutex>

namespace air {

constexpr int kMaxGroup = 16;

// ---------------------------------------------------------------------------------------
// Split-K exchange area of the entry point that allocates nothing (air_decode_attn_static): a fixed array in
// the library's own device image instead of the caller's workspace.  Every GPU the library runs on holds its own
// copy at its own address; host code only ever uses the address hipGetSymbolAddress returns for the current
// device (the array's name is a host-side stand-in, not a device address).
//   [arrival counters: kStaticSlots ints][(max, sum) pairs: kStaticSlots x 16][partial outputs: kStaticSlots x 16 x 128 floats]
// ---------------------------------------------------------------------------------------
constexpr size_t kStaticCntBytes = kStaticSlots * sizeof(int32_t);
constexpr size_t kStaticMlBytes = kStaticSlots * kMaxGroup * sizeof(float2);
constexpr size_t kStaticOBytes = kStaticSlots * kMaxGroup * 128 * sizeof(float);
constexpr size_t kStaticScratchBytes = kStaticCntBytes + kStaticMlBytes + kStaticOBytes;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];  // per device, filled on first use with that device current
static std::mutex g_scratch_mutex;

hipError_t static_exchange(DecodeExchange *x) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void *ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            if (!ptr) return hipErrorInvalidSymbol;
            g_scratch_ptr[dev] = ptr;
        }
        ptr = g_scratch_ptr[dev];
    }
    if (x) {
        char *base = (char *)ptr;
        x->cnt = (int32_t *)base;
        x->ml = (float2 *)(base + kStaticCntBytes);
        x->o = (float *)(base + kStaticCntBytes + kStaticMlBytes);
        x->local = 1;
        x->stride = 0;  // set per launch: the launch's own split count
    }
    return hipSuccess;
}

// counters of a launch start at zero (a kernel, not a memset: the call may be recorded into a graph)
__global__ __launch_bounds__(256) void zero_counters_kernel(int32_t *p, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}
hipError_t launch_zero_counters(hipStream_t s, int32_t *p, int n) {
    hipLaunchKernelGGL(zero_counters_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// MFMA decode attention.  Workgroup (split, unit) of NW waves; wave w takes the chunks w, w+NW, ...
// (16*KT keys each) of the split's key range.  Lane (n = lane % 16, c = lane / 16).
//   scores^T tile (16 keys x 16 heads) = K'(16 keys x 128) * q^T: A = key n, elements 8c..8c+7 of
//   each 32-element slice; B = head n, same elements; the result leaves lane (n = head, c) with
//   keys 4c..4c+3 of the tile.  Two tiles cover a 32-token block, so that lane holds 8
//   probabilities of head n: exactly the A operand of P*V for the block when the block's tokens
//   are stored in v_slot order.  B of P*V = 16 bytes of the transposed V' block per lane, and the
//   accumulator of output tile j keeps heads 4c..4c+3 of column 16j + n.
// The kernel is bound by instruction issue as much as by memory when there are few units, so the
// key loop carries no predication: tiles past the end of the range re-read the last valid tile
// (their scores are masked, in the one iteration that has a tail), and the token this call appends
// (Eq.2) is not read through the cache at all: one wave of the split that owns its row scores it
// from k_new / v_new on the vector ALU and stores it into the cache.
// Softmax runs in the base-2 domain: logits are scaled by log2(e)/sqrt(d) and exponentiated with
// exp2; running maxima and the exchanged partial maxima are in that domain.
// The waves of a workgroup merge through LDS.  With more than one split per unit the
// workgroups exchange partials through memory and the one that finishes last merges them.
// ---------------------------------------------------------------------------------------
// What the MFMA decode kernel needs of the tables and of the per-layer launch block: a short
// argument block (the kernel starts with the loads of its arguments).
struct DecodeTabs {
    // (side by side: one scalar load; a load of its own for the second, behind the first wait, cost 0.3 us a launch)
    const int2 *len_off;
    int32_t *dec_steps;  // null: the host passes the count of appended tokens (DecodeSteps)
    const int4 *by_length;  // per sequence, (length, offset, layer) of the layers by falling cache length
    void *kcache, *vcache;
    float *dec_o;
    float2 *dec_ml;
    int32_t *dec_cnt;
    int32_t n_units;     // units of the whole context: the cache-full flag lies behind their counts
    const CachePtrs *cache_ptrs;  // in-place cache: the K / V tensor of every layer (else null: the cache is the workspace's pool)
    int64_t kv_b, kv_h;           // in-place cache: element strides between sequences / KV heads of those tensors
    int32_t x_local;     // 1: the exchange slots (dec_o, dec_ml, dec_cnt) are indexed by the unit inside the launch
    int32_t x_stride;    // exchange slots per unit
};
struct DecodeSteps {
    int32_t uniform;  // >= 0: every layer of the launch has appended this many tokens (any number of layers per launch)
    int32_t appended[kMaxLayersPerLaunch];
};

// 16-key tiles of a wave's chunk in launches that are not told otherwise: 16 KB of K' and V' (32 KB of the fp32 rows).
// One launch on the matrix unit in place of three (append, attention on the vector unit with one row per thread, combine),
// us per step: bf16 d = 64, 48 units of ~870 keys 157 -> 7.5; fp32 d = 128, 112 units of ~390 keys 154 -> 12.6.
template <typename T, int D>
constexpr int kDecodeTiles = sizeof(T) == 4 && D == 128 ? 2 : 4;

// INPLACE: the cache is kept inside the layers' own K / V tensors (their addresses come from a table)
// SORTED: a launch over all layers whose grid index z is not the layer but its rank by cache length within the
// sequence (longest first); the layer comes with the table entry that carries the length
// VH > 1: VH workgroups per unit, each with its part of the columns of V' (see below); ONE_SEQ: the instance for B = 1
// STREAM: a cache several times the size of the memory-side cache: its loads are marked as used once
template <typename T, int D, int NW, int KT, bool SPLIT, bool INPLACE, bool SORTED = false, int VH = 1, bool ONE_SEQ = false,
          bool STREAM = false>
__global__ __launch_bounds__(64 * NW) void decode_mfma_kernel(Dims dm, DecodeTabs t, int l0, int lbase,
                                                              DecodeSteps ll, const T *q_new,
                                                              const T *k_new, const T *v_new, T *out,
                                                              int splits, int lg_splits) {
    constexpr int kVec = Elem<T>::kVec, kVTok = Elem<T>::kVTok;
    constexpr int NS = D / Elem<T>::kSlice;  // slices of the contraction over the head's elements
    constexpr int kPieces = D / kVec;        // 16-byte pieces of a row
    constexpr int kIter = 16 * KT;           // keys per loop iteration of one wave (KT score tiles, TB token blocks)
    constexpr int TB = kIter / kVTok;
    constexpr int NJ = D / 16 / VH;          // output tiles (16 columns each) of the workgroup
    constexpr int kCols = D / VH;            // columns of V' of the workgroup
    constexpr int kColsPer = kCols > 64 ? kCols / 64 : 1;  // columns of the appended V' row per lane (lanes < kCols)
    static_assert(kIter % kVTok == 0 && kCols >= 16, "whole V' blocks per iteration, whole output tiles");
    static_assert(VH == 1 || (!SPLIT && !SORTED), "column parts: VH workgroups per unit, no exchange");
    static_assert(kStepCopies % VH == 0, "whole copies of the step count per part");
    // Non-finite values.  A logit of -inf weighs nothing, also in a chunk that has no other (its head then has no reference
    // yet); an infinite element of V' makes its output column infinite: every factor of V' is at least kLeast, also the one
    // of the last block read again behind the last key, whose infinities are in the column anyway (0 * inf would be NaN; of
    // finite elements it adds 1e-38).  bf16 with heads of 128 elements goes without: such a chunk, or an infinite element
    // in the last block, gives NaN there.
    constexpr bool kNonFinite = sizeof(T) == 4 || D == 64;
    constexpr float kLeast = 0x1p-126f;
    const int lane = threadIdx.x & 63, n = lane & 15, c = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // a scalar: the wave's chunk walk and its branches stay off the vector unit
    // grid (split + splits * KV head, sequence, layer): the linear order of the workgroups is (split, unit) and
    // no index needs a division (the number of splits is a power of two)
    const int split = SPLIT ? (int)blockIdx.x & (splits - 1) : 0;
    int kvh = SPLIT ? (int)blockIdx.x >> lg_splits : (int)blockIdx.x;
    int b = blockIdx.y;
    int li = blockIdx.z;
    int vh = 0;
    bool live = true;
    if (VH > 1) {
        // VH workgroups per unit, each with all of K' and 1 / VH of the columns of V' and of the output: no partials to
        // exchange, and a workgroup moves (1 + 1 / VH) / 2 of the unit's bytes (a CU takes in about 140 GB/s, which is what
        // bounds a launch of few units).  A 1-D grid: the workgroups of a unit get ids 8 (VH p + part) + x, the
        // same XCD (ids are dealt round-robin over the 8 XCDs) at neighbouring dispatch slots, so that the K' tiles they all
        // stream come through that XCD's L2 once.  `splits` carries the units of the launch (the grid is rounded up to
        // whole groups of 8 units: the workgroups past the end redo the last unit and store nothing), `lg_splits` log2 of
        // the KV heads.
        const int wid = blockIdx.x, slot = wid >> 3;
        constexpr int kLgVH = VH == 8 ? 3 : (VH == 4 ? 2 : 1);
        int pair = ((slot >> kLgVH) << 3) | (wid & 7);
        vh = slot & (VH - 1);
        live = pair < splits;
        pair = min(pair, splits - 1);
        kvh = pair & (dm.Hkv - 1);
        if (ONE_SEQ) {  // one sequence: its index is a constant of the instance (every address in front of the first loads is shorter: 0.6 us per launch)
            li = pair >> lg_splits;
            b = 0;
        } else {
            seq_layer_of(dm, pair >> lg_splits, b, li);
        }
    }
    int2 len_off;
    if (SORTED) {
        const int4 e = t.by_length[(int64_t)b * dm.L + blockIdx.z];
        len_off = make_int2(e.x, e.y);
        li = e.z - l0;
    }
    const int l = l0 + li;
    const int G = dm.G;
    // the unit's cache length and offset first: everything that touches the cache waits for them
    if (!SORTED) len_off = t.len_off[(int64_t)b * dm.L + l];
    CachePtrs cp = {nullptr, nullptr};
    if (INPLACE) cp = t.cache_ptrs[l];  // requested together with the table entry
    // The token this call appends (Eq.2): every wave fetches its k_new / v_new values first thing (the
    // addresses depend on the block index only), so they are long there when the wave that owns the
    // token needs them.
    const int64_t new_src = (((int64_t)(lbase + li) * dm.B + b) * dm.Hkv + kvh) * D;
    uint4 knew[NS], krow;
    T vnew[NJ], vcol[kColsPer];
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) knew[sl] = *reinterpret_cast<const uint4 *>(k_new + new_src + Elem<T>::kSlice * sl + kVec * c);
    krow = *reinterpret_cast<const uint4 *>(k_new + new_src + kVec * (lane & (kPieces - 1)));
#pragma unroll
    for (int j = 0; j < NJ; ++j) vnew[j] = v_new[new_src + 16 * (j + NJ * vh) + n];
#pragma unroll
    for (int h2 = 0; h2 < kColsPer; ++h2) vcol[h2] = v_new[new_src + kCols * vh + 64 * h2 + (kCols < 64 ? lane & (kCols - 1) : lane)];
    const int64_t unit = ((int64_t)l * dm.B + b) * dm.Hkv + kvh;
    // tokens appended so far: from the host with the launch, or counted on the device (a recorded launch
    // that is replayed): a column part reads and advances copies of its own (count_step), of the splits of a unit the one that
    // merges them advances all copies, after every split has read the first
    int appended = ll.uniform >= 0 ? ll.uniform : ll.appended[li];
    // A workgroup past the last unit does not look at the device's count: it redoes a part that may have finished, so that
    // the count may already be the next step's, and with it a cache that only looks full.  (A pointer it does not have, not
    // a return in front of it: behind a branch the argument is fetched late, 0.15 us a launch.)
    const int32_t *const steps = VH > 1 && !live ? nullptr : t.dec_steps;
    if (steps) {
        appended = steps[unit * kStepCopies + vh];
        if (appended >= dm.max_steps) {  // cache full: nothing is appended or written
            if (threadIdx.x == 0) t.dec_steps[(int64_t)t.n_units * kStepCopies] = 1;
            return;
        }
    }
    if (VH > 1 && !live) return;
    // The next step's count: part vh of VH reads copy vh and writes the copies vh, vh + VH, ..., so that the parts of a unit need
    // not wait for one another and a launch of another shape finds every copy advanced.  (One count, advanced by the last part
    // to arrive at an atomic counter: a recorded launch of one layer took 7.7 us where the same launch called eagerly took 6.8.)
    auto count_step = [&]() {
        if (threadIdx.x < kStepCopies / VH) t.dec_steps[unit * kStepCopies + vh + VH * threadIdx.x] = appended + 1;
    };
    const int len = len_off.x + appended + 1;
    const int newrow = len - 1;  // the token appended by this call (Eq.2): scored from k_new / v_new, stored to the cache
    int k0 = 0, k1 = len;
    if (SPLIT) {  // ceil(len / splits) rounded up to whole 32-token blocks
        const int cs = (((len + splits - 1) >> lg_splits) + 31) & ~31;
        k0 = split * cs;
        k1 = min(len, k0 + cs);
    }
    const int kend = min(k1, newrow);  // the split's keys that are in the cache: [k0, kend)
    // the unit's cache: its region of the workspace pool, or (kept in place) its rows of the layer's own K / V tensors
    const int64_t row0 = INPLACE ? 0 : ((int64_t)b * dm.Hkv + kvh) * dm.pool_rows + len_off.y;
    const int64_t ip0 = INPLACE ? (int64_t)b * t.kv_b + (int64_t)kvh * t.kv_h : 0;
    T *kc = INPLACE ? (T *)cp.k + ip0 : (T *)t.kcache + row0 * D;
    T *vc = INPLACE ? (T *)cp.v + ip0 : (T *)t.vcache + row0 * D;
    T *o_unit = out + (((int64_t)(lbase + li) * dm.B + b) * dm.Hq + (int64_t)kvh * G) * D;

    uint4 qb[NS];
    {
        // MFMA columns past the group's heads re-read its last head: their results are never stored
        const T *q = q_new + (((int64_t)(lbase + li) * dm.B + b) * dm.Hq + (int64_t)kvh * G + min(n, G - 1)) * D;
#pragma unroll
        for (int s = 0; s < NS; ++s) qb[s] = *reinterpret_cast<const uint4 *>(q + Elem<T>::kSlice * s + kVec * c);
    }
    constexpr double kScale2D = (D == 128 ? 0.08838834764831845 : 0.125) * 1.4426950408889634;  // log2(e) / sqrt(d)
    // fp32 takes it to 46 bits; the second term is positive, so that a masked score stays -inf
    constexpr bool kTwoTerm = sizeof(T) == 4;
    constexpr float kScale2 = (float)(kTwoTerm ? kScale2D * (1.0 - 1.2e-7) : kScale2D);
    constexpr float kScale2Lo = (float)(kScale2D - (double)kScale2);
    static_assert(!kTwoTerm || kScale2Lo > 0.f, "sign of the second term");
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // ---- the appended token belongs to the wave of the owning split that would take the next
    // chunk.  The row goes into the cache at once, so that the stores complete behind the cache
    // loads: K' into its places of the tile, V' into its slot of the block (a token that opens a
    // block writes the block's other slots as zeros).  Other waves and splits never use these
    // places in this launch: their reads of them are masked or carry zero probability.  The
    // token's own score (vector ALU) starts the wave's running softmax: max = score, sum = its weight against that maximum,
    // formed as a cached key's is (1, but for the rounding of the maximum), accumulator = that times v_new for every head.
    const bool owns_new = newrow >= k0 && newrow < k1 && wave == ((kend - k0 + kIter - 1) / kIter) % NW;
    if (owns_new) {
        if (lane < kPieces && vh == 0)  // the new K' row: 16 bytes a lane
            *reinterpret_cast<uint4 *>(kc + k_tiled<D, kVec>(newrow, kVec * lane)) = krow;
        const int tok = newrow & (kVTok - 1);
#pragma unroll
        for (int h2 = 0; h2 < kColsPer; ++h2) {
            if (kCols < 64 && lane >= kCols) break;
            const int col = kCols * vh + 64 * h2 + lane;
            if (tok == 0) {  // a new block: the column's other slots are written as zeros
                constexpr int kGroup = 16 * kVec;  // elements from one slot group to the next
                T *vcolp = vc + (int64_t)newrow * D + (col >> 4) * (4 * kGroup) + (col & 15) * kVec;  // slot group 0
                const uint4 z = make_uint4(0, 0, 0, 0);
                *reinterpret_cast<uint4 *>(vcolp) = make_uint4(bits_of(vcol[h2]), 0, 0, 0);  // token 0 sits in slot 0
                *reinterpret_cast<uint4 *>(vcolp + kGroup) = z;
                *reinterpret_cast<uint4 *>(vcolp + 2 * kGroup) = z;
                *reinterpret_cast<uint4 *>(vcolp + 3 * kGroup) = z;
            } else {
                vc[v_tiled<D, kVec>(newrow, col)] = vcol[h2];
            }
        }
        float sn = 0.f;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) sn = dot_piece<T>(qb[sl], knew[sl], sn);
        sn += __shfl_xor(sn, 16, 64);
        sn += __shfl_xor(sn, 32, 64);
        m_run = sn * kScale2;
        float p = 1.f;
        if constexpr (sizeof(T) == 4 || D == 64) {
            const float x = fmaf(sn, kScale2, -m_run);
            p = __builtin_amdgcn_exp2f(kTwoTerm ? fmaf(sn, kScale2Lo, x) : x);
            if (m_run == -INFINITY) p = 0.f;
        }
        l_run = c == 0 ? p : 0.f;  // l_run is a per-lane partial of the head's sum: the token counts once
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const float v = ldf(&vnew[j]);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[j][i] = sizeof(T) == 4 || D == 64 ? v * __shfl(p, 4 * c + i, 64) : v;  // rows are heads 4c..4c+3
        }
    }

    const int last_tile = (kend - 1) & ~15, last_block = (kend - 1) & ~(kVTok - 1);  // last tile / block with a cached key
    // The chunks of the range are walked front to back on even steps and back to front on odd ones:
    // what a step read last is what the next step reads first, so the part of the cache that is
    // still in the L2 of the XCD (the unit-to-XCD mapping is the same every launch) gets reused
    // instead of being evicted just before its turn.
    const bool backward = (appended & 1) != 0;
    const int n_chunks = (max(kend - k0, 0) + kIter - 1) / kIter;
    const int kb_first = k0 + (backward ? n_chunks - 1 - wave : wave) * kIter;
    const int kStep = (backward ? -NW : NW) * kIter;  // distance between two chunks of one wave
    auto has = [&](int kb) { return kb >= k0 && kb < kend; };

    // all loads of a chunk: the KT score tiles of K' and the V' operands of the TB token blocks
    auto load_chunk = [&](uint4(&a)[KT][NS], uint4(&vb)[TB][NJ], int kb) {
#pragma unroll
        for (int tile = 0; tile < KT; ++tile) {
            const T *src = kc + (int64_t)min(kb + 16 * tile, last_tile) * D + Elem<T>::kSlice * n + kVec * c;
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) {
                if constexpr (STREAM) a[tile][sl] = load16<true>(src + 64 * kVec * sl);
                else a[tile][sl] = *reinterpret_cast<const uint4 *>(src + 64 * kVec * sl);
            }
        }
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            const T *src = vc + (int64_t)min(kb + kVTok * tb, last_block) * D + 16 * kVec * c + kVec * n;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if constexpr (STREAM) vb[tb][j] = load16<true>(src + 64 * kVec * (j + NJ * vh));
                else vb[tb][j] = *reinterpret_cast<const uint4 *>(src + 64 * kVec * (j + NJ * vh));
            }
        }
    };
    auto compute_chunk = [&](const uint4(&a)[KT][NS], const uint4(&vb)[TB][NJ], int kb) {
        // ---- scores^T
        f32x4 s[KT];
#pragma unroll
        for (int tile = 0; tile < KT; ++tile) {
            s[tile] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) s[tile] = mma<T>(a[tile][sl], qb[sl], s[tile]);
        }
        if (kb + kIter > kend) {  // the chunk with the tail (uniform over the wave)
#pragma unroll
            for (int tile = 0; tile < KT; ++tile)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (kb + 16 * tile + 4 * c + i >= kend) s[tile][i] = -INFINITY;
        }
        // ---- online softmax for head n over the keys this lane holds (4c+i of each tile).  The four lanes of a
        // head share one reference maximum m_run; it is raised (and the accumulators rescaled) only when some
        // score of the chunk lies more than kSlack above it, so most chunks need no cross-lane step at all:
        // probabilities may then be as large as 2^kSlack, which fp32 sums and bf16 operands hold without loss.
        // The sum l_run stays a per-lane partial and is added up over the four lanes after the last chunk.
        constexpr float kSlack = 8.0f;
        float mloc = s[0][0];
#pragma unroll
        for (int tile = 0; tile < KT; ++tile)
#pragma unroll
            for (int i = 0; i < 4; ++i) mloc = fmaxf(mloc, s[tile][i]);
        mloc *= kScale2;
        if (__ballot(mloc > m_run + kSlack) != 0ull) {  // uniform over the wave; always taken on a wave's first chunk
            float mb = fmaxf(mloc, __shfl_xor(mloc, 16, 64));
            mb = fmaxf(mb, __shfl_xor(mb, 32, 64));
            const float m_new = fmaxf(m_run, mb);  // finite for finite logits: key kb is valid
            float corr = __builtin_amdgcn_exp2f(m_run - m_new);
            if (kNonFinite && m_new == -INFINITY) corr = 1.0f;  // this head has seen logits of -inf only: its sums are zero
            l_run *= corr;
            m_run = m_new;
            // accumulator rows are heads 4c..4c+3: fetch their rescale factors from lanes 4c+i
            if ((owns_new || kb != kb_first) && __ballot(corr != 1.0f) != 0ull) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float f = __shfl(corr, 4 * c + i, 64);
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[j][i] *= f;
                }
            }
        }
        const float m_ref = kNonFinite && m_run == -INFINITY ? 0.f : m_run;
        float lb = 0.f;
#pragma unroll
        for (int tile = 0; tile < KT; ++tile)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float x = fmaf(s[tile][i], kScale2, -m_ref);
                if (kTwoTerm) x = fmaf(s[tile][i], kScale2Lo, x);
                const float p = __builtin_amdgcn_exp2f(x);
                s[tile][i] = sizeof(T) == 4 ? fmaxf(p, kLeast) : p;
                lb += p;
            }
        l_run += lb;
        // ---- P * V
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            if constexpr (sizeof(T) == 4) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[j] = mma<T>(__builtin_bit_cast(uint4, s[tb]), vb[tb][j], acc[j]);
            } else {
                // bf16 operands.  Heads of 128 elements take the probabilities rounded to bf16; with heads of 64 they keep their
                // 24 bits, as three bf16 terms of 8, cut off, not rounded, so that none is negative (the matrix unit is idle most
                // of the time: two more products a tile)
                constexpr int kTerms = D == 128 ? 1 : 3;
                bf16x8 pa[kTerms];
                if constexpr (kTerms == 1) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) pa[0][i] = (__bf16)s[2 * tb + (i >> 2)][i & 3];
                } else {
                    typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
                    constexpr uint32_t kLeast2 = 0x00800080u;  // twice kLeast in bf16; positive values order as their bits do
                    u32x4 term[kTerms];
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        float p0 = s[2 * tb + (w >> 1)][2 * (w & 1)], p1 = s[2 * tb + (w >> 1)][2 * (w & 1) + 1];
#pragma unroll
                        for (int k = 0; k < kTerms; ++k) {
                            const uint32_t t0 = __float_as_uint(p0) & 0xffff0000u, t1 = __float_as_uint(p1) & 0xffff0000u;
                            term[k][w] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, (t0 >> 16) | t1),
                                                                                                __builtin_bit_cast(u16x2, kLeast2)));
                            p0 -= __uint_as_float(t0);
                            p1 -= __uint_as_float(t1);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < kTerms; ++k) pa[k] = __builtin_bit_cast(bf16x8, term[k]);
                }
#pragma unroll
                for (int k = kTerms - 1; k >= 0; --k)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[j] = mma<T>(__builtin_bit_cast(uint4, pa[k]), vb[tb][j], acc[j]);
            }
        }
    };
    // Two chunk buffers: while one chunk is multiplied the loads of the wave's next chunk are in
    // flight.  Loads are issued only for chunks that exist, and the loop is laid out so that every
    // path reaches a compute step with the same loads behind it (the wait counts stay exact).
    if constexpr (KT * NS + TB * NJ > 24) {  // two buffers of this size do not fit the registers: load, then multiply
        for (int kb = kb_first; has(kb); kb += kStep) {
            uint4 a0[KT][NS], v0[TB][NJ];
            load_chunk(a0, v0, kb);
            compute_chunk(a0, v0, kb);
        }
    } else if (has(kb_first)) {
        uint4 a0[KT][NS], v0[TB][NJ], a1[KT][NS], v1[TB][NJ];
        int kb = kb_first;
        load_chunk(a0, v0, kb);
        if (!has(kb + kStep)) {
            compute_chunk(a0, v0, kb);
        } else {
            load_chunk(a1, v1, kb + kStep);
            while (true) {
                compute_chunk(a0, v0, kb);
                if (!has(kb + 2 * kStep)) {
                    compute_chunk(a1, v1, kb + kStep);
                    break;
                }
                load_chunk(a0, v0, kb + 2 * kStep);
                compute_chunk(a1, v1, kb + kStep);
                if (!has(kb + 3 * kStep)) {
                    compute_chunk(a0, v0, kb + 2 * kStep);
                    break;
                }
                load_chunk(a1, v1, kb + 3 * kStep);
                kb += 2 * kStep;
            }
        }
    }

    // the head's sum over the four lanes that hold its keys
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);

    // ---- merge the NW waves of the workgroup through LDS.  Every wave first rescales its partial
    // to the workgroup's maximum, so that the merge is a plain sum: wave w ends up with output
    // tiles w, w+NW, ... (heads 4c..4c+3, column 16j+n), plus the merged (max, sum) of those heads.
    constexpr int kTiles = NJ >= NW ? NJ / NW : 1;  // output tiles a wave owns after the merge: j = wave + NW*jj (of the workgroup's NJ)
    const bool owns_tiles = NJ >= NW || wave < NJ;
    __shared__ f32x4 s_acc[NW][NJ][64];
    __shared__ float s_mw[kMaxGroup][NW], s_lw[kMaxGroup][NW];
    __shared__ int s_prev;
    float mrg_m[4], mrg_l[4];  // merged max / sum of heads 4c+i
    if (NW > 1) {
        if (c == 0) s_mw[n][wave] = m_run;
        __syncthreads();
        float M = s_mw[n][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) M = fmaxf(M, s_mw[n][w]);
        const float f = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - M);
        if (c == 0) s_lw[n][wave] = l_run * f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float fi = __shfl(f, 4 * c + i, 64);
            mrg_m[i] = __shfl(M, 4 * c + i, 64);
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[j][i] *= fi;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) s_acc[wave][j][lane] = acc[j];
        __syncthreads();
#pragma unroll
        for (int jj = 0; jj < kTiles; ++jj) {
            const int j = NJ >= NW ? wave + NW * jj : min(wave, NJ - 1);  // waves without a tile (more waves than tiles) repeat the last one
            f32x4 sum = s_acc[0][j][lane];
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                const f32x4 x = s_acc[w][j][lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[i] += x[i];
            }
            acc[jj] = sum;  // tile wave + NW*jj
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float Lsum = s_lw[4 * c + i][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) Lsum += s_lw[4 * c + i][w];
            mrg_l[i] = Lsum;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            mrg_m[i] = __shfl(m_run, 4 * c + i, 64);
            mrg_l[i] = __shfl(l_run, 4 * c + i, 64);
        }
    }
    if (!SPLIT || splits == 1) {  // no partials: normalise and store
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int g = 4 * c + i;
            if (g < G && owns_tiles) {
                const float inv = __builtin_amdgcn_rcpf(mrg_l[i]);
#pragma unroll
                for (int jj = 0; jj < kTiles; ++jj)
                    stf(&o_unit[g * D + 16 * (NJ * vh + wave + NW * jj) + n], sizeof(T) == 4 ? acc[jj][i] / mrg_l[i] : acc[jj][i] * inv);
            }
        }
        if (t.dec_steps) count_step();
        return;
    }
    if (!SPLIT) return;  // the instance for one workgroup per unit carries none of what follows
    // ---- partial of this split.  Partials are exchanged between workgroups of one launch, which
    // may run on different XCDs (separate L2s).  They are written and read with system-scope
    // (write-through / L2-bypassing) 16-byte accesses in the accumulators' own lane layout, the
    // writers wait for their stores to complete before the workgroup counts itself, and the
    // workgroup that counts last reads them.  This keeps the exchange off the whole-L2 write-back
    // that a release fence would cost.  Layout of one partial: [tile j][lane][4] floats.
    const int64_t xu = t.x_local ? ((int64_t)li * dm.B + b) * dm.Hkv + kvh : unit;  // the unit's exchange slots
    const int64_t part = xu * t.x_stride + split;
    float *pu = t.dec_o + xu * t.x_stride * (int64_t)kMaxGroup * D;
    const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(pu, 0, t.x_stride * kMaxGroup * D * 4, 0x00020000);
    if (4 * c < G && owns_tiles) {
#pragma unroll
        for (int jj = 0; jj < kTiles; ++jj)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[jj]), prs,
                                                   (split * kMaxGroup * D + ((wave + NW * jj) * 64 + lane) * 4) * 4, 0,
                                                   kSysScope);
    }
    if (wave == 0 && n == 0) {  // lane (0, c) holds the merged stats of heads 4c..4c+3
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int g = 4 * c + i;
            if (g < G) {
                float *mlp = reinterpret_cast<float *>(t.dec_ml + part * G + g);
                __hip_atomic_store(mlp, mrg_m[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(mlp + 1, mrg_l[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) s_prev = __hip_atomic_fetch_add(&t.dec_cnt[xu], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_prev != splits - 1) return;
    if (threadIdx.x == 0) __hip_atomic_store(&t.dec_cnt[xu], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next launch

    // merge of the splits: every wave loads the partial tiles it owns (one round of loads), the
    // (max, sum) pairs go through LDS
    __shared__ float s_m[kMaxSplits][kMaxGroup], s_l[kMaxSplits][kMaxGroup], s_w[kMaxSplits][kMaxGroup];
    __shared__ float s_inv[kMaxGroup];
    const float *ml = reinterpret_cast<const float *>(t.dec_ml + xu * t.x_stride * G);
    f32x4 num[kTiles];
#pragma unroll
    for (int jj = 0; jj < kTiles; ++jj) num[jj] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int p = threadIdx.x; p < splits * G; p += 64 * NW) {
        s_m[p / G][p % G] = __hip_atomic_load(ml + 2 * p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_l[p / G][p % G] = __hip_atomic_load(ml + 2 * p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if ((int)threadIdx.x < G) {
        const int g = threadIdx.x;
        float M = -INFINITY;
        for (int s2 = 0; s2 < splits; ++s2) M = fmaxf(M, s_m[s2][g]);
        float den = 0.f;
        for (int s2 = 0; s2 < splits; ++s2) {
            const float wg = s_l[s2][g] > 0.f ? __builtin_amdgcn_exp2f(s_m[s2][g] - M) : 0.f;
            s_w[s2][g] = wg;
            den = fmaf(wg, s_l[s2][g], den);
        }
        s_inv[g] = 1.0f / den;
    }
    __syncthreads();
    constexpr int kRound = (32 / kTiles) < kMaxSplits ? (32 / kTiles) : kMaxSplits;  // splits loaded together
    for (int s0 = 0; s0 < splits; s0 += kRound) {
        f32x4 v[kRound][kTiles];
#pragma unroll
        for (int s2 = 0; s2 < kRound; ++s2)
#pragma unroll
            for (int jj = 0; jj < kTiles; ++jj) {
                v[s2][jj] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (s0 + s2 < splits && 4 * c < G && owns_tiles)
                    v[s2][jj] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                        prs, ((s0 + s2) * kMaxGroup * D + ((wave + NW * jj) * 64 + lane) * 4) * 4, 0, kSysScope));
            }
#pragma unroll
        for (int s2 = 0; s2 < kRound; ++s2) {
            if (s0 + s2 < splits) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float wg = s_w[s0 + s2][(4 * c + i) & (kMaxGroup - 1)];
#pragma unroll
                    for (int jj = 0; jj < kTiles; ++jj) num[jj][i] = fmaf(wg, v[s2][jj][i], num[jj][i]);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int g = 4 * c + i;
        if (g < G && owns_tiles) {
            const float inv = s_inv[g];
#pragma unroll
            for (int jj = 0; jj < kTiles; ++jj) stf(&o_unit[g * D + 16 * (wave + NW * jj) + n], num[jj][i] * inv);
        }
    }
    if (t.dec_steps) count_step();
}

// ---------------------------------------------------------------------------------------
struct DecodeLaunch {
    hipStream_t s;
    const Dims &dm;
    const DecodeTabs &dt;
    const DecodeSteps &ds;
    int l0, nl, lbase, splits, lg_splits;
    const void *q_new, *k_new, *v_new;
    void *out;
    bool stream;
};

template <typename T, int D, int NW, int KT, bool SPLIT, bool INPLACE, bool SORTED, int VH, bool ONE_SEQ, bool STREAM = false>
static void decode_launch(const DecodeLaunch &a, dim3 grid, int splits, int lg_splits) {
    hipLaunchKernelGGL((decode_mfma_kernel<T, D, NW, KT, SPLIT, INPLACE, SORTED, VH, ONE_SEQ, STREAM>), grid, dim3(64 * NW), 0, a.s, a.dm,
                       a.dt, a.l0, a.lbase, a.ds, (const T *)a.q_new, (const T *)a.k_new, (const T *)a.v_new, (T *)a.out, splits,
                       lg_splits);
}

template <typename T, int D, int NW, int KT>
static void decode_shape_launch(const DecodeLaunch &a, bool longest_first) {
    const dim3 grid(a.splits * a.dm.Hkv, a.dm.B, a.nl);
    if constexpr (sizeof(T) == 2 && D == 128) {  // the only storage that can keep its cache in place
        if (a.dt.cache_ptrs) {
            if (a.splits == 1) decode_launch<T, D, NW, KT, false, true, false, 1, false>(a, grid, 1, 0);
            else decode_launch<T, D, NW, KT, true, true, false, 1, false>(a, grid, a.splits, a.lg_splits);
            return;
        }
    }
    if constexpr (KT == kDecodeTiles<T, D> && (NW == 1 || NW == 4)) {
        if (longest_first && a.splits == 1)
            return a.stream ? decode_launch<T, D, NW, KT, false, false, true, 1, false, true>(a, grid, 1, 0)
                            : decode_launch<T, D, NW, KT, false, false, true, 1, false>(a, grid, 1, 0);
    }
    if constexpr (KT == kDecodeTiles<T, D> && NW <= 4) {
        if (a.stream && a.splits == 1) return decode_launch<T, D, NW, KT, false, false, false, 1, false, true>(a, grid, 1, 0);
    }
    if (a.splits == 1) decode_launch<T, D, NW, KT, false, false, false, 1, false>(a, grid, 1, 0);
    else decode_launch<T, D, NW, KT, true, false, false, 1, false>(a, grid, a.splits, a.lg_splits);
}

// VH workgroups per unit, each with its part of the columns of V' (the caller has checked what this variant asks for)
template <typename T, int D, int VH>
static void decode_parts_launch_(const DecodeLaunch &a) {
    constexpr int KT = kDecodeTiles<T, D>;
    const int units = a.nl * a.dm.B * a.dm.Hkv;
    int lg_h = 0;
    while ((1 << lg_h) < a.dm.Hkv) ++lg_h;
    const dim3 grid(VH * ((units + 7) & ~7));
    if constexpr (sizeof(T) == 2 && D == 128) {
        if (a.dt.cache_ptrs) {
            if (a.dm.B == 1) decode_launch<T, D, 4, KT, false, true, false, VH, true>(a, grid, units, lg_h);
            else decode_launch<T, D, 4, KT, false, true, false, VH, false>(a, grid, units, lg_h);
            return;
        }
    }
    if (a.dm.B == 1) decode_launch<T, D, 4, KT, false, false, false, VH, true>(a, grid, units, lg_h);
    else decode_launch<T, D, 4, KT, false, false, false, VH, false>(a, grid, units, lg_h);
}
template <typename T, int D>
static void decode_parts_launch(const DecodeLaunch &a, int parts) {
    if constexpr (D == 128) {
        if (parts == 8) return decode_parts_launch_<T, D, 8>(a);
    }
    if (parts >= 4) decode_parts_launch_<T, D, 4>(a);
    else decode_parts_launch_<T, D, 2>(a);
}

template <typename T, int D, int KT>
static void decode_waves_launch(const DecodeLaunch &a, int waves, bool longest_first) {
    if (waves == 8 && KT < 8) decode_shape_launch<T, D, 8, KT < 8 ? KT : 4>(a, longest_first);
    else if (waves >= 4) decode_shape_launch<T, D, 4, KT>(a, longest_first);
    else if (waves == 2) decode_shape_launch<T, D, 2, KT>(a, longest_first);
    else decode_shape_launch<T, D, 1, KT>(a, longest_first);
}

hipError_t launch_decode(hipStream_t s, const Dims &dm, const DevTables &t, const DecodeExchange &x, int dtype, int l0,
                         int nl, int lbase, const LaunchLayers &ll, const void *q_new, const void *k_new,
                         const void *v_new, void *out, int splits, int waves, int tiles, int uniform_appended,
                         bool longest_first, int column_parts, bool stream) {
    if (splits < 1 || (splits & (splits - 1)) != 0) return hipErrorInvalidValue;  // the kernel shifts by log2(splits)
    int lg_splits = 0;
    while ((1 << lg_splits) < splits) ++lg_splits;
    DecodeTabs dt;
    dt.len_off = t.len_off;
    dt.by_length = t.by_length;
    dt.kcache = t.kcache;
    dt.vcache = t.vcache;
    dt.dec_o = x.o;
    dt.dec_ml = x.ml;
    dt.dec_cnt = x.cnt;
    dt.x_local = x.local;
    dt.x_stride = x.stride;
    dt.dec_steps = t.dec_steps;
    dt.cache_ptrs = t.cache_ptrs;
    dt.kv_b = t.ip_kv_b;
    dt.kv_h = t.ip_kv_h;
    dt.n_units = dm.L * dm.B * dm.Hkv;
    DecodeSteps ds;
    ds.uniform = uniform_appended;
    for (int i = 0; i < kMaxLayersPerLaunch; ++i) ds.appended[i] = ll.appended[i];
    const DecodeLaunch a = {s, dm, dt, ds, l0, nl, lbase, splits, lg_splits, q_new, k_new, v_new, out, stream};
    if (dtype == AIR_BF16 && dm.D == 128) {
        if (column_parts > 1) decode_parts_launch<bf16_t, 128>(a, column_parts);
        else if (tiles == 4) decode_waves_launch<bf16_t, 128, 4>(a, waves, longest_first);
        else if (tiles == 2) decode_waves_launch<bf16_t, 128, 2>(a, waves, longest_first);
        else decode_waves_launch<bf16_t, 128, 8>(a, waves, longest_first);
    } else if (dtype == AIR_BF16) {  // the other storages have one chunk size each
        if (column_parts > 1) decode_parts_launch<bf16_t, 64>(a, column_parts);
        else decode_waves_launch<bf16_t, 64, kDecodeTiles<bf16_t, 64>>(a, waves, longest_first);
    } else if (dm.D == 128) {
        if (column_parts > 1) decode_parts_launch<float, 128>(a, column_parts);
        else decode_waves_launch<float, 128, kDecodeTiles<float, 128>>(a, waves, longest_first);
    } else {
        if (column_parts > 1) decode_parts_launch<float, 64>(a, column_parts);
        else decode_waves_launch<float, 64, kDecodeTiles<float, 64>>(a, waves, longest_first);
    }
    return hipGetLastError();
}

}  // namespace air
