// Forward trace with one wave per ray (BVH path).
//
// The 64 lanes of a wave share one ray, so every step of the k-buffer marching
// of Sec. 3.2 is done for many candidates at once and a ray waits for a few
// dozen memory round trips instead of several hundred:
//   NODE  up to 16 wide nodes are taken from the stack and their 64 child boxes
//         and slabs tested, one per lane; crossed inner children go back on the
//         stack, the nearest group on top, crossed clusters into a queue;
//   LEAF  up to 64 records of the queued clusters are tested, one per lane
//         (clusters are contiguous, so neighbouring lanes read neighbouring
//         records); hits between the resume key and the last key that can
//         matter collect in a pending list;
//   MERGE 64 pending keys are sorted across the lanes and merged into the
//         buffer of the 128 smallest keys, two per lane in ascending order; the
//         buffered hits' optical depth (4 bits in each key) tells behind
//         which key the transmittance is used up for certain;
//   COMP  every lane re-evaluates its buffered hit; the transmittance runs
//         through the lanes in hit order, and each composited channel is the
//         running sum of one lane (O, D, then the features), so the operations
//         and their order per ray are those of the nested form, bit for bit.
// A round whose buffer let hits go and whose transmittance stays above the
// cutoff is followed by another from the top, after the last complete key.
//
// What bounds it: VALU issue (1M surfels, 4.2M rays: 2,712 VALU and 978 scalar
// instructions per ray, a VALU instruction per SIMD every 3.3 cycles; 68% L2
// hits, 18.7 KB per ray past L2).  Against one ray per lane, whose waves
// stepped through 1,230 dependent iterations with 45% of their lanes active:
// 1M surfels, 4.2M rays 70.3 -> 34.4 ms; 200K surfels 36.6 -> 11.9 ms; launches
// smaller than the chip, whose time is one ray's chain of round trips: 4,096
// rays 580 -> 33 us (19 without the scratch that such a launch does not use),
// 2^18 rays 13.9 -> 5 ms.  Then, forward of 1M / 5M surfels:
//   34.4 / 232 -> 25.3 / 128 ms: the children's slabs cull what only crosses
//     the fat boxes of tilted patches (records tested per ray 1,206 -> 718);
//   -> 23.6 / 127 ms: corner sums and extents in the nodes, the first step at a
//     full tree level, scalar masks in the sort, immediate row offsets;
//   -> 19.8 / 82 ms: the stack ordered in two groups (below);
//   -> 16.0 / 70 ms: 128 keys and the optical-depth bound (node steps per ray
//     18.4 -> 10.9, leaf steps 12.7 -> 7.9, rounds 1.31 -> 1.00; at 5M surfels
//     110 hits per ray, rounds 2.30 -> 1.54).
//
// The complete part of the buffer after a round is the smallest keys above the
// resume key whatever the visiting order, and results do not depend on its
// size, so every requested k gives the same outputs as the per-lane form.
#pragma once

#include "irgs_internal.hpp"
#include "march.hpp"
#include "wave_ops.hpp"

namespace irgs {

constexpr int kWaveBlock = 64;   // one wave per block: no barrier anywhere
constexpr int kWaveNodes = 16;   // nodes taken from the stack per step (4 lanes each)
constexpr int kWaveStack = 512;
constexpr int kWaveQueue = 128;  // clusters: at most kLeafTrigger - 1 + 64 wait
constexpr int kWavePend = 128;   // hit keys: at most 63 + 64 wait
constexpr int kLeafTrigger = 8;  // clusters that start a leaf step (about 64 records)
constexpr int kWaveRowShort = 13;  // composite rows of up to 10 channels
constexpr int kWaveLdsWords = kWaveStack + kWaveQueue + 2 * kWavePend;
constexpr int kWaveParts = 8;         // claim counters, one per XCD ...
constexpr int kWaveClaimStride = 16;  // ... 128 bytes apart
constexpr int kWaveChunk = 256;       // consecutive slots of one part

// A node step takes one node at a time (depth first) once fewer than the
// reserve's entries are left above a full step: from any node on, depth-first
// steps add at most 3 entries per level.
inline int wave_stack_reserve(int wide_depth) { return 3 * wide_depth + 4; }
inline bool wave_stack_fits(int wide_depth)
{
    return wave_stack_reserve(wide_depth) + 3 * kWaveNodes + 64 <= kWaveStack;
}

typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) float lds_f32;

// Orders this wave's LDS accesses around it for the compiler (the hardware
// executes one wave's LDS operations in order).
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ int wave_rank(uint64_t mask)  // set bits of mask below this lane
{
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u)));
}

__device__ __forceinline__ int bcast(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float bcast(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ uint64_t bcast(uint64_t v, int lane)
{
    return (static_cast<uint64_t>(static_cast<uint32_t>(bcast(static_cast<int>(v >> 32), lane))) << 32) |
           static_cast<uint32_t>(bcast(static_cast<int>(v), lane));
}

// Lane l's value of lane l ^ X, for the X a sort of 64 needs.
template <int X>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane)
{
    if constexpr (X == 1) return dpp<0xB1>(v, v);        // quad_perm 1,0,3,2
    else if constexpr (X == 2) return dpp<0x4E>(v, v);   // quad_perm 2,3,0,1
    else if constexpr (X == 3) return dpp<0x1B>(v, v);   // quad_perm 3,2,1,0
    else if constexpr (X == 7) return dpp<0x141>(v, v);  // row_half_mirror
    else if constexpr (X == 8) return dpp<0x128>(v, v);  // row_ror:8
    else if constexpr (X == 15) return dpp<0x140>(v, v); // row_mirror
    else if constexpr (X == 4 || X == 16 || X == 31)
        return static_cast<uint32_t>(__builtin_amdgcn_ds_swizzle(static_cast<int>(v), (X << 10) | 0x1f));
    else
        return static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute((lane ^ X) << 2, static_cast<int>(v)));
}

template <int X>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v, int lane)
{
    return (static_cast<uint64_t>(lane_xor<X>(static_cast<uint32_t>(v >> 32), lane)) << 32) |
           lane_xor<X>(static_cast<uint32_t>(v), lane);
}

// Keys read as doubles are in reverse order (see hit_key), and an FP64
// compare runs at the FP32 rate.
__device__ __forceinline__ bool key_less(uint64_t a, uint64_t b)
{
    return __longlong_as_double(static_cast<long long>(a)) > __longlong_as_double(static_cast<long long>(b));
}

// Compare-exchange with lane ^ X: the lower lane keeps the smaller key.
template <int X>
__device__ __forceinline__ void key_step(uint64_t& k, int lane)
{
    // the lanes with X's top bit set, as a scalar mask
    constexpr uint64_t upper = X >= 32   ? 0xFFFFFFFF00000000ull
                               : X >= 16 ? 0xFFFF0000FFFF0000ull
                               : X >= 8  ? 0xFF00FF00FF00FF00ull
                               : X >= 4  ? 0xF0F0F0F0F0F0F0F0ull
                               : X >= 2  ? 0xCCCCCCCCCCCCCCCCull
                                         : 0xAAAAAAAAAAAAAAAAull;
    const uint64_t y = lane_xor<X>(k, lane);
    k = __builtin_amdgcn_inverse_ballot_w64(__ballot(key_less(y, k)) ^ upper) ? y : k;
}

// A hit's key here: its position is followed by 4 bits of optical depth, in
// 1/16 and rounded down (a + a^2 / 2 <= -ln(1 - a)), so that a buffer of keys
// knows where the transmittance is certainly used up.
constexpr float kDepthUnits = 16.0f;
__device__ __forceinline__ uint64_t wave_key(float tau, int pos, float a)
{
    const uint32_t q = static_cast<uint32_t>(fminf(fmaf(a, 0.5f * a, a) * kDepthUnits, 15.0f));
    return hit_key(tau, static_cast<int>(static_cast<uint32_t>(pos) << 4 | q));
}

// Ascending bitonic sort of one key per lane (mirrored first stages, so every
// exchange has the same direction).
__device__ __forceinline__ void sort_keys(uint64_t& k, int lane)
{
    key_step<1>(k, lane);
    key_step<3>(k, lane), key_step<1>(k, lane);
    key_step<7>(k, lane), key_step<2>(k, lane), key_step<1>(k, lane);
    key_step<15>(k, lane), key_step<4>(k, lane), key_step<2>(k, lane), key_step<1>(k, lane);
    key_step<31>(k, lane), key_step<8>(k, lane), key_step<4>(k, lane), key_step<2>(k, lane), key_step<1>(k, lane);
    key_step<63>(k, lane), key_step<16>(k, lane), key_step<8>(k, lane), key_step<4>(k, lane), key_step<2>(k, lane),
        key_step<1>(k, lane);
}

// Sort a bitonic sequence.
__device__ __forceinline__ void sort_bitonic(uint64_t& k, int lane)
{
    key_step<32>(k, lane), key_step<16>(k, lane), key_step<8>(k, lane), key_step<4>(k, lane);
    key_step<2>(k, lane), key_step<1>(k, lane);
}

// The k-buffer: the 128 smallest keys so far, two per lane, lane i's first the
// i-th of all, its second the (64 + i)-th.
struct WaveBuf {
    uint64_t a, b;

    __device__ __forceinline__ void clear() { a = b = kKeyNone; }

    // Merge in 64 sorted keys.
    __device__ __forceinline__ void merge(uint64_t x, int lane)
    {
        if (bcast(a, 0) == kKeyNone) {
            a = x;
            return;
        }
        const uint64_t xr = lane_xor<63>(x, lane);
        const bool less = key_less(xr, a);
        uint64_t over = less ? a : xr;
        a = less ? xr : a;
        sort_bitonic(a, lane);
        if (__ballot(over != kKeyNone) == 0) return;
        if (bcast(b, 0) == kKeyNone) {
            sort_bitonic(over, lane);
            b = over;
            return;
        }
        // `over` is bitonic: sorted the other way round, its minimum with b
        // leaves the 64 smallest of both
        sort_bitonic(over, lane);
        const uint64_t r = lane_xor<63>(over, lane);
        b = key_less(r, b) ? r : b;
        sort_bitonic(b, lane);
    }

    // The last key that can still matter: the one at which the buffered hits
    // use up `budget` units of optical depth, else the 128th (kKeyNone while
    // there is none).  Keys past it in the second half are dropped whole when
    // the first half holds it.
    __device__ __forceinline__ uint64_t last(uint32_t budget)
    {
        const uint32_t da = wave_scan(a != kKeyNone ? static_cast<uint32_t>(a) & 15u : 0u);
        const uint64_t in_a = __ballot(da >= budget);
        if (in_a) {
            b = kKeyNone;
            return bcast(a, __ffsll(static_cast<unsigned long long>(in_a)) - 1);
        }
        if (bcast(b, 0) == kKeyNone) return kKeyNone;
        const uint32_t db = wave_scan(b != kKeyNone ? static_cast<uint32_t>(b) & 15u : 0u) + bcast(static_cast<int>(da), 63);
        const uint64_t in_b = __ballot(db >= budget);
        return bcast(b, in_b ? __ffsll(static_cast<unsigned long long>(in_b)) - 1 : 63);
    }
};

// One scene, slots [0, R), taken in `order` when given.
struct WavePlain {
    SceneView sc;
    OutPtrs o;
    const float* ro;
    const float* rd;
    int64_t R;
    const uint32_t* order;

    __device__ __forceinline__ int64_t total() const { return R; }
    __device__ __forceinline__ int64_t locate(int64_t slot, int lane, int* item) const
    {
        *item = 0;
        return order ? static_cast<int64_t>(order[slot]) : slot;
    }
    __device__ __forceinline__ Ray ray(int64_t r, int) const { return load_ray(ro, rd, r); }
    __device__ __forceinline__ const OutPtrs& out(int) const { return o; }
    __device__ __forceinline__ const SceneView& view(int) const { return sc; }
};

// Several requests over several scenes: a slot indexes the concatenation of
// the items' rays.  The lanes look for the owning item, the last one whose
// first slot is not past it, in 64ths of the range left: one dependent read
// up to 64 items, three up to 262,144 (a scan from the first item, 64 at a
// time, read 60 KB of items per ray with 1,000 of them: 2.1M rays in 1,000 /
// 10,000 items 9.3 / 39.5 ms, this 7.6 / 7.7; one item 6.6).
struct WavePacked {
    const SceneView* scenes;
    const WorkItem* items;
    int n_items;
    int64_t n_rays;

    __device__ __forceinline__ int64_t total() const { return n_rays; }
    __device__ __forceinline__ int64_t locate(int64_t slot, int lane, int* item) const
    {
        int it = 0, n = n_items;  // the item is one of the n from `it` on
        while (n > 1) {
            const int step = (n + 63) >> 6;
            const int at = lane * step;
            const bool before = at < n && items[it + at].chunk_begin <= slot;
            const int skip = (__popcll(__ballot(before)) - 1) * step;  // first slots ascend; the first item's is not past it
            it += skip;
            n = min(step, n - skip);
        }
        *item = it;
        return items[it].ray_begin + (slot - items[it].chunk_begin);
    }
    __device__ __forceinline__ Ray ray(int64_t r, int item) const { return load_ray(items[item].ro, items[item].rd, r); }
    __device__ __forceinline__ const OutPtrs& out(int item) const { return items[item].out; }
    __device__ __forceinline__ const SceneView& view(int item) const { return scenes[items[item].scene]; }
};

// The F features of a surfel into its row (16-byte loads where they are aligned).
__device__ __forceinline__ void stage_features(lds_f32* row, const float* __restrict__ f, int F)
{
    if ((F & 3) == 0 && (reinterpret_cast<uintptr_t>(f) & 15) == 0) {
        for (int c = 0; c < F; c += 4) {
            const float4 v = *reinterpret_cast<const float4*>(f + c);
            row[c] = v.x, row[c + 1] = v.y, row[c + 2] = v.z, row[c + 3] = v.w;
        }
        return;
    }
    for (int c0 = 0; c0 < F; c0 += 4) {  // four loads in flight; past the end the last one again
        float v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = f[min(c0 + c, F - 1)];
#pragma unroll
        for (int c = 0; c < 4; ++c) row[min(c0 + c, F - 1)] = v[c];
    }
}

// acc plus w times column x over n rows in order (rows past n up to a multiple
// of 8 are zero); row length LC, or L when LC is 0.
template <int LC>
__device__ __forceinline__ float sum_rows(float acc, const lds_f32* rows, int x, int n, int L)
{
    const int step = LC ? LC : L;
    for (int i = 0; i < n; i += 8) {
        const lds_f32* r = rows + i * step;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc = fmaf(r[j * step], r[j * step + x], acc);
    }
    return acc;
}

// Trace ray r of `sc` with the whole wave; returns its hits.  `lds`: kWaveLdsWords words of this
// wave; `reserve`: stack entries kept for depth-first steps.
template <int CM>
__device__ __forceinline__ int trace_ray_wave(const SceneView& sc, const TraceParams& P, const Ray& ray, int64_t r,
                                               const OutPtrs& out, lds_u32* lds, int reserve, int lane)
{
    lds_u32* stk = lds;
    lds_u32* queue = lds + kWaveStack;
    lds_u32* pend = queue + kWaveQueue;  // low words, then high words
    lds_u32* pend_hi = pend + kWavePend;
    lds_f32* rows = reinterpret_cast<lds_f32*>(lds);  // composite staging (the traversal's areas are idle then)
    const int F = sc.F;
    const int FO = CM == kColSH ? 3 : (CM == kColNormal ? F + 3 : F);
    float T = 1.0f;
    float acc = 0.0f;   // lane 0: O, lane 1: D, lane 2 + c: channel c
    float acc2 = 0.0f;  // lane c: channel 62 + c
    int nh = 0;
    if (sc.n > 0 && ray_valid(ray)) {
        const BoxRay q = box_ray(ray);
        const float tmax_c = fminf(P.t_max, 3.0e38f);
        uint64_t after = 0;
        while (true) {
            WaveBuf buf;
            buf.clear();
            uint64_t kth = kKeyNone;
            const float lo = after == 0 ? P.t_min : fmaxf(P.t_min, key_tau(after));
            float hi = tmax_c;
            // optical depth (in units, with a margin over the rounding of T)
            // that takes T below the cutoff for certain
            const float left = P.T_min > 0.0f ? 0.6931472f * __log2f(T / P.T_min) + 2e-3f : 1e9f;
            const float units = ceilf(fmaxf(fminf(left * kDepthUnits, 1e9f), 1.0f));
            const uint32_t budget = __builtin_amdgcn_readfirstlane(static_cast<int>(units));
            int sp = 0, qn = 0, pn = 0;
            if (lane < sc.n_start) stk[lane] = static_cast<uint32_t>(sc.start + lane);
            sp = sc.n_start;
            lds_order();
            while (true) {
                if (qn >= kLeafTrigger || (sp == 0 && qn > 0)) {
                    // whole clusters from the queue's end, at most 64 records
                    const bool have = lane < qn;
                    const int ref = have ? static_cast<int>(queue[qn - 1 - lane]) : 0;
                    const int first = (ref & ~kLeafBit) >> 4;
                    const int cnt = have ? (ref & 15) + 1 : 0;
                    const uint32_t incl = wave_scan(static_cast<uint32_t>(cnt));
                    const bool take = have && incl <= 64u;
                    const int nt = __popcll(__ballot(take));
                    const int excl = static_cast<int>(incl) - cnt;
                    const int total = bcast(static_cast<int>(incl), nt - 1);
                    // lane -> cluster: each taken cluster marks its first lane
                    lds_u32* mark = pend + 64;  // at most 63 keys wait here
                    mark[lane] = 0u;
                    lds_order();
                    if (take) mark[excl] = 1u;
                    lds_order();
                    const uint64_t starts = __ballot(mark[lane] != 0u);
                    const int src = wave_rank(starts) - 1 + static_cast<int>((starts >> lane) & 1ull);
                    const int pos = __builtin_amdgcn_ds_bpermute(src << 2, first - excl) + lane;
                    qn -= nt;
                    bool pass = false;
                    uint64_t key = kKeyNone;
                    if (lane < total) {
                        const SurfelRec s = load_rec(sc.rec, pos);
                        float tau, rho2;
                        const bool hit = hit_test(s, ray, P.t_min, P.t_max, &tau, &rho2);
                        key = wave_key(tau, pos, alpha_of(s, rho2));
                        pass = hit && key > after && key < kth;
                    }
                    const uint64_t m = __ballot(pass);
                    lds_order();
                    if (pass) {
                        const int at = pn + wave_rank(m);
                        pend[at] = static_cast<uint32_t>(key);
                        pend_hi[at] = static_cast<uint32_t>(key >> 32);
                    }
                    lds_order();
                    pn += __popcll(m);
                    if (pn >= 64) {
                        pn -= 64;
                        uint64_t x = (static_cast<uint64_t>(pend_hi[pn + lane]) << 32) | pend[pn + lane];
                        sort_keys(x, lane);
                        buf.merge(x, lane);
                        kth = buf.last(budget);
                        if (kth != kKeyNone) hi = fminf(key_tau(kth), tmax_c);
                    }
                } else if (sp > 0) {
                    int nn = min(sp, kWaveNodes);
                    if (sp + 3 * kWaveNodes > kWaveStack - reserve) nn = 1;
                    const int ni = lane >> 2;
                    bool inner = false, leaf = false;
                    float tn = 0.0f, tf = 0.0f;
                    int ref = 0;
                    if (ni < nn) {
                        const WideChild w = load_child(sc.wnodes, static_cast<int>(stk[sp - 1 - ni]), lane & 3);
                        child_span(w, ray, q, lo, hi, &tn, &tf);
                        ref = w.ref;
                        inner = tn <= tf && ref >= 0;
                        leaf = tn <= tf && ref < 0;
                    }
                    sp -= nn;
                    lds_order();
                    const uint64_t ml = __ballot(leaf);
                    if (leaf) queue[qn + wave_rank(ml)] = static_cast<uint32_t>(ref);
                    qn += __popcll(ml);
                    // of the inner children, those entered before the nearest one
                    // is left go on top, each group the nearest node's first
                    // (measured at 1M / 5M surfels: all children in stack order
                    // 23.4 / 157 ms, every node's children by depth 21.2 / 125,
                    // each node's nearest on top 20.9 / 87, this 19.8 / 82)
                    uint32_t near = __float_as_uint(inner ? tf : __int_as_float(0x7f800000));
                    auto lower = [&](uint32_t o) {
                        near = __float_as_uint(fminf(__uint_as_float(near), __uint_as_float(o)));
                    };
                    lower(lane_xor<1>(near, lane)), lower(lane_xor<2>(near, lane)), lower(lane_xor<7>(near, lane));
                    lower(lane_xor<15>(near, lane)), lower(lane_xor<16>(near, lane)), lower(lane_xor<32>(near, lane));
                    const bool first = tn <= __uint_as_float(near);
                    const uint64_t mt = __ballot(inner && first), mb = __ballot(inner && !first);
                    const int top = __popcll(mt), below = __popcll(mb);
                    if (inner)
                        stk[sp + below - 1 + (first ? top - wave_rank(mt) : -wave_rank(mb))] = static_cast<uint32_t>(ref);
                    sp += top + below;
                    lds_order();
                } else {
                    break;
                }
            }
            if (pn > 0) {
                uint64_t x = kKeyNone;
                if (lane < pn) x = (static_cast<uint64_t>(pend_hi[lane]) << 32) | pend[lane];
                sort_keys(x, lane);
                buf.merge(x, lane);
                const uint64_t end = bcast(buf.b, 63);  // hits past it may have fallen off
                kth = end < kth ? end : kth;
            }
            lds_order();
            // composite the buffered hits, 64 at a time, lane i the i-th
            // (none past the last key that matters: of the hits there, some
            // were left out)
            uint64_t cut = 0;
            for (int half = 0; half < 2; ++half) {
                const uint64_t kb = half == 0 ? buf.a : buf.b;
                const int m = __popcll(__ballot(kb != kKeyNone && !key_less(kth, kb)));
                float tau = 0.0f, a = 0.0f;
                int id = 0;
                float4 nr = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (lane < m) {
                    const SurfelRec s = load_rec(sc.rec, key_pos(kb) >> 4);
                    float rho2;
                    plane_hit(s, ray, &tau, &rho2);
                    a = alpha_of(s, rho2);
                    id = __float_as_int(s.c.w);
                    nr = s.b;
                }
                // T before lane i's hit: T runs one lane up per step, so that the
                // products are those of the hit-by-hit form
                const float om = 1.0f - a;
                const float omp = __uint_as_float(dpp<0x138>(__float_as_uint(1.0f), __float_as_uint(om)));  // wave_shr:1
                float Tl = T;
                for (int i = 1; i < m; i += 8) {
#pragma unroll
                    for (int j = 0; j < 8; ++j)  // steps past the last hit change no lane that counts
                        Tl = __uint_as_float(dpp<0x138>(__float_as_uint(T), __float_as_uint(Tl))) * omp;
                }
                const float Ta = Tl * om;
                cut = __ballot(lane < m && Ta < P.T_min);
                const int used = cut ? __ffsll(static_cast<unsigned long long>(cut)) : m;
                const float w = Tl * a;
                if (out.hit_ids && lane < used && nh + lane < out.H_cap) {
                    const int64_t at = r * out.H_cap + nh + lane;
                    __builtin_nontemporal_store(id, out.hit_ids + at);
                    if (out.hit_T) __builtin_nontemporal_store(Tl, out.hit_T + at);
                }
                // rows of (w, 1, tau, channels) in LDS; every lane then sums its
                // own column in hit order.  An odd row length puts a column's
                // words in different banks; the short one is a constant, so that
                // the sums' addresses are immediates.
                const int L = FO <= kWaveRowShort - 3 ? kWaveRowShort : (3 + FO) | 1;
                const int nrows = min(64, (kWaveLdsWords / L) & ~7);
                float Y[16];
                if constexpr (CM == kColSH) sh_basis(ray.dx, ray.dy, ray.dz, P.sh_deg, Y);
                for (int b = 0; b < used; b += nrows) {
                    const int i = lane - b;
                    if (i >= 0 && i < nrows) {
                        lds_f32* row = rows + i * L;
                        if (lane < used) {
                            row[0] = w, row[1] = 1.0f, row[2] = tau;
                            const float* f = sc.feat + static_cast<int64_t>(id) * F;
                            if constexpr (CM == kColSH) {
                                float raw[3];
                                sh_raw(f, P.sh_deg, Y, raw);
#pragma unroll
                                for (int c = 0; c < 3; ++c) row[3 + c] = fmaxf(raw[c], 0.0f);
                            } else {
                                stage_features(row + 3, f, F);
                                if constexpr (CM == kColNormal) {
                                    const float s = dot3(nr.x, nr.y, nr.z, ray.dx, ray.dy, ray.dz) > 0.0f ? -1.0f : 1.0f;
                                    row[3 + F] = s * nr.x, row[4 + F] = s * nr.y, row[5 + F] = s * nr.z;
                                }
                            }
                        } else {
                            for (int c = 0; c < 3 + FO; ++c) row[c] = 0.0f;
                        }
                    }
                    lds_order();
                    const int n = min(used - b, nrows);
                    const int x = 1 + min(lane, FO + 1);  // this lane's column
                    if (L == kWaveRowShort)
                        acc = sum_rows<kWaveRowShort>(acc, rows, x, n, 0);
                    else
                        acc = sum_rows<0>(acc, rows, x, n, L);
                    if (FO > 62) acc2 = sum_rows<0>(acc2, rows, 3 + min(62 + lane, FO - 1), n, L);
                    lds_order();
                }
                nh += used;
                if (used > 0) T = bcast(Ta, used - 1);
                if (cut || m < 64) break;
            }
            if (cut || kth == kKeyNone) break;
            after = kth;
        }
    }
    if (lane == 0) {
        out.O[r] = acc;
        if (out.T) out.T[r] = T;
        if (out.n_hits) out.n_hits[r] = nh;
    }
    if (lane == 1) out.D[r] = acc;
    if (lane >= 2 && lane < 2 + FO) out.feat[r * FO + lane - 2] = acc;
    if (62 + lane < FO) out.feat[r * FO + 62 + lane] = acc2;
    return nh;
}

// Every wave of a launch runs this.  Without claim counters wave b traces slot
// b.  With them (a persistent grid) the slots are dealt in chunks of
// kWaveChunk to kWaveParts parts, and a wave claims one slot at a time from
// the part of its XCD (blocks are handed to the XCDs in turn), then from the
// other parts: rays next to each other in the caller's order are then traced
// at about the same time on the CUs behind one L2, and eight counters share
// the claims (a single counter takes one claim every 12 ns).  One million
// surfels, 4.2M rays, 64 per origin: one counter and 8 slots per claim 61 ms,
// this 34 ms; 2 / 4 slots per claim 40 / 46 ms; chunks of 64 to 1,024 alike.
template <int CM, class Source>
__device__ __forceinline__ void trace_waves(const Source& src, unsigned long long* next, const TraceParams& P,
                                            lds_u32* lds, int reserve)
{
    const int lane = threadIdx.x;
    const int64_t total = src.total();
    int part = blockIdx.x & (kWaveParts - 1), left = kWaveParts;
    int64_t slot = blockIdx.x;
    while (true) {
        if (next) {
            unsigned long long b = 0;
            if (lane == 0) b = atomicAdd(next + part * kWaveClaimStride, 1ull);
            const int64_t i = static_cast<int64_t>(bcast(static_cast<uint64_t>(b), 0));
            slot = (i / kWaveChunk * kWaveParts + part) * kWaveChunk + i % kWaveChunk;
        }
        if (slot >= total) {
            if (!next || --left == 0) return;
            part = (part + 1) & (kWaveParts - 1);  // this part is used up: help the next
            continue;
        }
        int item;
        int64_t r = src.locate(slot, lane, &item);
        r = static_cast<int64_t>(bcast(static_cast<uint64_t>(r), 0));  // the same in every lane: into scalars
        item = bcast(item, 0);
        const Ray v = src.ray(r, item);
        Ray ray;
        ray.ox = bcast(v.ox, 0), ray.oy = bcast(v.oy, 0), ray.oz = bcast(v.oz, 0);
        ray.dx = bcast(v.dx, 0), ray.dy = bcast(v.dy, 0), ray.dz = bcast(v.dz, 0);
        trace_ray_wave<CM>(src.view(item), P, ray, r, src.out(item), lds, reserve, lane);
        if (!next) return;
    }
}

}  // namespace irgs
