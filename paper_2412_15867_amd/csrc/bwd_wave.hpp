// Backward over hit lists with a wave's lanes over the hits.
//
// The hits of a group of rays form one stream, every ray's back to front, and
// a wave takes 64 hits of it per step, whatever ray they belong to.  The suffix
// composite S_i = alpha_i c_i + (1 - alpha_i) S_{i+1} is an affine map per hit,
// so a step runs it as an inclusive scan of maps over the lanes (FP64).  A
// ray's last hit starts it anew: lanes whose range holds one take nothing from
// the lanes before, by selection, so that what is not finite in one ray stays
// out of the others (a map with the factor 0 would make NaN of it).
//
// Per-surfel sums are collected in a hash table in LDS shared by a block's
// waves and written out when it fills: groups are taken in the order of where
// their rays land, so that a block's rays meet the same surfels (1M surfels,
// 4.2M rays: 2.0 hits per surfel and 64 rays in the caller's order, 4.8 in this,
// 6.4 per 192 rays).  LDS float atomics take 3 cycles a lane, so the table is
// updated without them: the waves of a block put their step's hits in LDS, and
// after a barrier wave w adds components w, w + W, ... of all of them, a ray's
// hits (all different surfels) at a time.  A hit that finds no slot is added to
// global memory by consecutive lanes, one component each.
//
// Against one ray per lane (64 rays stepping together, 53% of the lanes with a
// hit, two scattered list reads per hit, 96 slots): 1M surfels, F = 8 18.4 ->
// 16.4 ms, SH degree 3 58.0 -> 42.6 ms; 5M surfels 51 -> 38.6 ms and the rays
// with cut lists, re-marched by one lane each before, 219 -> 7 ms.  With LDS
// atomics: 25.1 and 67.5 ms.  Of 40,000 cycles per step of a block of 12 waves
// 14,000 went to the FP64 chain rule and its loads, so these were cut: a row's
// reciprocals are packed once per surfel, its loads are all issued at once
// (none behind a branch), the first words a step ahead: F = 8 16.3 -> 14.3 ms.
// With many components the table is what counts: groups of 3 rays leave room
// for more slots than groups of 16: SH 41.3 -> 36.8 ms, 262,144 SH rays of 1,024
// pixels 4.1 -> 2.8 ms; 24 and 64 features, groups of 8 -> 3, 10.0 -> 9.5 and
// 15.2 -> 14.3 ms; 8 and 16 features lose or are level.  Keeping the rays apart
// by selection costs 0.14 ms at F = 8.  What bounds it: F = 8 the steps' own work
// (VALU 34%, 120M atomic requests against 183M hits); SH the atomics (401M for
// 4.2M rays, 28M for 262,144: they are done in memory, 11 per ns).
#pragma once

#include "irgs_internal.hpp"
#include "march.hpp"
#include "trace_wave.hpp"

namespace irgs {

constexpr int kWalkProbes = 16;

// Per kernel: FM = features of a surfel at most.  One block of 12 waves per CU
// (3 per SIMD, what the FP64 registers allow) shares all of its LDS.
template <int FM>
struct WalkShape {
    static constexpr int waves = 12;
    static constexpr int group = FM <= 16 ? 16 : 3;  // rays per group at most
    static constexpr int slots = FM <= 8 ? 1350 : FM <= 16 ? 900 : FM <= 48 ? 476 : 350;
    static constexpr int comps = 10 + FM;
    static constexpr int per_wave = (comps + waves - 1) / waves;  // components a wave adds
    static constexpr int stride = slots | 1;      // words between components: odd, so a row's lie in different banks
    static constexpr int fill = slots * 7 / 8;    // a step that starts past this many adds no new keys (others until none is free)
    static constexpr int flush = slots * 5 / 8;   // written out when it holds more
};

// A hit as its wave stages it: ten components, T alpha (FP64), and a word of
// slot (kNoSlot: none), ray of the step, SH clamp and row.
constexpr int kStageWords = 13;
constexpr uint32_t kNoSlot = 0xffffu;

// A ray's words in LDS: origin, direction, upstream of O and D, of the
// channels, and (SH) the basis; then its list: index (2), hits, first place
// in the group's stream.
template <int FM, int CM>
struct WalkRow {
    static constexpr int up = CM == kColSH ? 3 : FM;  // upstream channels (normal mode: F + 3 <= FM)
    static constexpr int basis = 8 + up;
    static constexpr int list = basis + (CM == kColSH ? 16 : 0);
    static constexpr int words = (list + 4) | 1;
};

// Feature component k of a hit: T alpha g_F; with SH T alpha g_F,c Y_j(d)
// wherever the channel is not clamped.
template <int FM, int CM>
__device__ __forceinline__ float feature_grad(const lds_f32* row, int k, double wgt, uint32_t lit)
{
    using Row = WalkRow<FM, CM>;
    if constexpr (CM == kColSH) {
        const int j = k / 3, ch = k - 3 * j;
        const double gc = (lit >> ch) & 1u ? wgt * row[8 + ch] : 0.0;
        return static_cast<float>(gc * row[Row::basis + j]);
    } else {
        return static_cast<float>(wgt * row[8 + k]);
    }
}

// Hash table of per-surfel sums of a block (see WalkShape).
template <int FM>
struct WalkTable {
    using Sh = WalkShape<FM>;
    int* keys;    // -1 = empty
    float* vals;  // [comps][stride]
    int* filled;

    __device__ __forceinline__ int find(int id) const
    {
        uint32_t slot = __umulhi(static_cast<uint32_t>(id) * 2654435761u, static_cast<uint32_t>(Sh::slots));
        const bool may_insert = *filled < Sh::fill;
        for (int p = 0; p < kWalkProbes; ++p) {
            const int k = keys[slot];
            if (k == id) return static_cast<int>(slot);
            if (k == -1) {
                if (!may_insert) return -1;
                const int prev = atomicCAS(&keys[slot], -1, id);
                if (prev == -1) atomicAdd(filled, 1);
                if (prev == -1 || prev == id) return static_cast<int>(slot);
            }
            slot = slot + 1 == Sh::slots ? 0 : slot + 1;
        }
        return -1;
    }
    __device__ __forceinline__ void clear(int tid, int threads, int nc) const
    {
        if (tid == 0) *filled = 0;
        for (int i = tid; i < Sh::slots; i += threads) keys[i] = -1;
        for (int i = tid; i < nc * Sh::stride; i += threads) vals[i] = 0.0f;
    }
    // Consecutive lanes add consecutive components of one surfel.
    __device__ __forceinline__ void write(int tid, int threads, int nc, float* gbuf, int gs) const
    {
        const int dh = threads / nc, dc = threads - dh * nc;
        for (int slot = tid / nc, c = tid - slot * nc; slot < Sh::slots;) {
            const int id = keys[slot];
            if (id >= 0) {
                const float v = vals[c * Sh::stride + slot];
                if (v != 0.0f) atomicAdd(gbuf + static_cast<int64_t>(id) * gs + c, v);
            }
            slot += dh;
            c += dc;
            if (c >= nc) {
                c -= nc;
                ++slot;
            }
        }
    }
};

template <int Ctrl, int Rows>
__device__ __forceinline__ double dpp_f64(double old, double v)
{
    const long long o = __double_as_longlong(old), x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(static_cast<int>(o), static_cast<int>(x), Ctrl, Rows, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(static_cast<int>(o >> 32), static_cast<int>(x >> 32), Ctrl, Rows, 0xf, false);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<uint32_t>(lo));
}

__device__ __forceinline__ double bcast(double v, int lane)
{
    return __longlong_as_double(static_cast<long long>(bcast(static_cast<uint64_t>(__double_as_longlong(v)), lane)));
}

// A hit's gradient but for the features.
struct WalkHit {
    float g[10];   // mu, quaternion, scales, opacity
    double wgt;    // T alpha
    uint32_t lit;  // SH: channels that are not clamped
};

// One step: lane's hit (id, 0 if not valid, transmittance Ti before it) of the ray in row ri;
// `last`: the ray's last hit (its suffix is 0).  S carries the suffix from step
// to step.  The geometry and the chain rule are evaluated in FP64 from the
// FP32 parameters: for a grazing ray (small n.r_d) FP32 rounding of the depth
// is amplified into u, v and into dtau/dmu.  Only the per-surfel contributions
// are rounded to FP32.  With SH the hit's colour is recomputed exactly as in
// the forward.  In the normal mode the upstream holds F feature channels and
// then 3 for the hit's normal turned to face the ray, s n with s = -1 where n
// . d > 0, decided exactly as in the forward; s T alpha g_N adds to the
// gradient of n.
template <int FM, int CM>
__device__ __forceinline__ WalkHit walk_step(const RawSurfels& raw, const TraceParams& P, const lds_f32* rows, int ri,
                                             bool valid, bool last, int id, float4 mo, float Ti_f, double& S, int lane)
{
    using Row = WalkRow<FM, CM>;
    const lds_f32* row = rows + ri * Row::words;
    const int F = P.F;
    const float* prow = raw.pk + static_cast<int64_t>(id) * raw.ps;  // the packed copy of the surfel's parameters
    const float4 qf = *reinterpret_cast<const float4*>(prow + 4);
    // Every load of the hit is issued here, none behind a branch: a load in a
    // branch waits for itself before the next.
    constexpr int held = CM != kColSH && FM <= 16 ? FM : 0;  // features in the row, zeros past F
    float4 ff[held / 4 + 1];
#pragma unroll
    for (int k = 0; k < held / 4; ++k) ff[k] = *reinterpret_cast<const float4*>(prow + 12 + 4 * k);
    const float* f = raw.feat_packed ? prow + 12 : raw.feat + static_cast<int64_t>(id) * F;
    const float gO = row[6], gD_f = row[7];
    const double o = mo.w;
    const double inv = *reinterpret_cast<const double*>(prow + 10);
    double rsu, rsv;
    if (FM <= 48 || raw.recips) {
        const double2 rs = *reinterpret_cast<const double2*>(prow + raw.ps - 4);
        rsu = rs.x, rsv = rs.y;
    } else {
        const float2 sc = *reinterpret_cast<const float2*>(prow + 8);
        rsu = 1.0 / double(sc.x), rsv = 1.0 / double(sc.y);
    }
    const double w = qf.x * inv, x = qf.y * inv, y = qf.z * inv, z = qf.w * inv;
    const double tu0 = 1.0 - 2.0 * (y * y + z * z), tu1 = 2.0 * (x * y + w * z), tu2 = 2.0 * (x * z - w * y);
    const double tv0 = 2.0 * (x * y - w * z), tv1 = 1.0 - 2.0 * (x * x + z * z), tv2 = 2.0 * (y * z + w * x);
    const double n0 = 2.0 * (x * z + w * y), n1 = 2.0 * (y * z - w * x), n2 = 1.0 - 2.0 * (x * x + y * y);
    const double dx_ = row[3], dy_ = row[4], dz_ = row[5];
    const double wx = double(mo.x) - row[0], wy = double(mo.y) - row[1], wz = double(mo.z) - row[2];
    const double rden = 1.0 / (n0 * dx_ + n1 * dy_ + n2 * dz_);
    const double tau = (n0 * wx + n1 * wy + n2 * wz) * rden;
    const double px = tau * dx_ - wx, py = tau * dy_ - wy, pz = tau * dz_ - wz;
    const double u = (px * tu0 + py * tu1 + pz * tu2) * rsu;
    const double v = (px * tv0 + py * tv1 + pz * tv2) * rsv;
    const double G = exp(-0.5 * (u * u + v * v));
    const double alpha = o * G;
    const double wgt = double(Ti_f) * alpha;

    double c = gO + double(gD_f) * tau;
    WalkHit h;
    h.wgt = wgt;
    h.lit = 0;
    double sN = 0.0, gN0 = 0.0, gN1 = 0.0, gN2 = 0.0;  // normal channels: turn and upstream
    if constexpr (CM == kColSH) {
        const int nb = (P.sh_deg + 1) * (P.sh_deg + 1);
        float col[3] = {0.5f, 0.5f, 0.5f};
        int j0 = 0;
        for (; j0 + 4 <= nb; j0 += 4) {  // a dozen loads in flight
            float x[12];
#pragma unroll
            for (int i = 0; i < 12; ++i) x[i] = f[3 * j0 + i];
#pragma unroll
            for (int i = 0; i < 12; ++i) col[i % 3] = fmaf(row[Row::basis + j0 + i / 3], x[i], col[i % 3]);
        }
        for (; j0 < nb; ++j0) {
            const float Y = row[Row::basis + j0];
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) col[ch] = fmaf(Y, f[3 * j0 + ch], col[ch]);
        }
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            const float gF = row[8 + ch];
            c += double(gF) * fmaxf(col[ch], 0.0f);
            h.lit |= col[ch] > 0.0f ? 1u << ch : 0u;
        }
    } else {
        if constexpr (held > 0) {
#pragma unroll
            for (int k = 0; k < FM; ++k) {
                const float fk = reinterpret_cast<const float*>(ff)[k];
                // (the upstream past F is zero, but for the normal's channels)
                if (CM != kColNormal || k < F) c += double(row[8 + k]) * fk;
            }
        } else {
#pragma unroll
            for (int k = 0; k < FM; ++k)
                if (k < F) c += double(row[8 + k]) * f[k];
        }
        if constexpr (CM == kColNormal) {
            float tf[3], vf[3], nf[3];
            quat_frame(qf, tf, vf, nf);
            const float dn = dot3(nf[0], nf[1], nf[2], row[3], row[4], row[5]);
            sN = dn > 0.0f ? -1.0 : 1.0;
            gN0 = row[8 + F], gN1 = row[9 + F], gN2 = row[10 + F];
            c += sN * (gN0 * n0 + gN1 * n1 + gN2 * n2);
        }
    }
    // suffix composites: inclusive scan of the maps S -> A + B S over the lanes.
    // `closed`: the lanes whose range so far holds a ray's last hit; a step
    // takes in a neighbouring range, then the masks its closed lanes.
    double A = valid ? alpha * c : 0.0, B = valid ? 1.0 - alpha : 1.0;
    const double Sin = S;
    uint64_t closed = __ballot(last);
#define IRGS_AFFINE_STEP(ctrl, rows, reach)                                                               \
    {                                                                                                     \
        const double Ap = dpp_f64<ctrl, rows>(0.0, A), Bp = dpp_f64<ctrl, rows>(1.0, B);                  \
        A = __builtin_amdgcn_inverse_ballot_w64(closed) ? A : fma(B, Ap, A);                              \
        B = B * Bp; /* of no use in a closed lane */                                                      \
        closed |= reach;                                                                                  \
    }
    IRGS_AFFINE_STEP(0x111, 0xf, (closed & 0x7fff7fff7fff7fffull) << 1)  // within rows of 16 lanes
    IRGS_AFFINE_STEP(0x112, 0xf, (closed & 0x3fff3fff3fff3fffull) << 2)
    IRGS_AFFINE_STEP(0x114, 0xf, (closed & 0x0fff0fff0fff0fffull) << 4)
    IRGS_AFFINE_STEP(0x118, 0xf, (closed & 0x00ff00ff00ff00ffull) << 8)
    IRGS_AFFINE_STEP(0x142, 0xa, (closed >> 15 & 0x0000000100000001ull) * 0xffff0000ull)  // lane 15 to row 1, 47 to 3
    IRGS_AFFINE_STEP(0x143, 0xc, (closed >> 31 & 1ull) * 0xffffffff00000000ull)           // lane 31 to rows 2 and 3
#undef IRGS_AFFINE_STEP
    const double Sout = __builtin_amdgcn_inverse_ballot_w64(closed) ? A : fma(B, Sin, A);
    double Sn = dpp_f64<0x138, 0xf>(Sin, Sout);  // the suffix behind this hit: the lane before's
    Sn = last ? 0.0 : Sn;
    S = bcast(Sout, 63);

    const double dA = double(Ti_f) * (c - Sn);
    h.g[9] = static_cast<float>(dA * G);
    const double gu = -dA * alpha * u;
    const double gv = -dA * alpha * v;
    h.g[7] = static_cast<float>(-gu * u * rsu);
    h.g[8] = static_cast<float>(-gv * v * rsv);
    // p - mu = tau d - w;  du/d(p-mu) = t_u / s_u
    const double au = gu * rsu, av = gv * rsv;
    const double gpx = au * tu0 + av * tv0, gpy = au * tu1 + av * tv1, gpz = au * tu2 + av * tv2;
    const double gtau = wgt * double(gD_f) + gpx * dx_ + gpy * dy_ + gpz * dz_;
    const double gt_den = gtau * rden;
    h.g[0] = static_cast<float>(gt_den * n0 - gpx);
    h.g[1] = static_cast<float>(gt_den * n1 - gpy);
    h.g[2] = static_cast<float>(gt_den * n2 - gpz);
    // dtau/dn = -(p - mu) / den;  du/dt_u = (p - mu) / s_u; the normal
    // channels add s T alpha g_N
    const double wn = wgt * sN;
    const double gn0 = -gt_den * px + wn * gN0, gn1 = -gt_den * py + wn * gN1, gn2 = -gt_den * pz + wn * gN2;
    const double gu0 = au * px, gu1 = au * py, gu2 = au * pz;
    const double gv0 = av * px, gv1 = av * py, gv2 = av * pz;
    // derivatives of the rotation columns with respect to (w, x, y, z)
    const double dw = 2.0 * (z * gu1 - y * gu2 - z * gv0 + x * gv2 + y * gn0 - x * gn1);
    const double dx = 2.0 * (y * gu1 + z * gu2 + y * gv0 - 2.0 * x * gv1 + w * gv2 + z * gn0 - w * gn1 - 2.0 * x * gn2);
    const double dy = 2.0 * (-2.0 * y * gu0 + x * gu1 - w * gu2 + x * gv0 + z * gv2 + w * gn0 + z * gn1 - 2.0 * y * gn2);
    const double dz = 2.0 * (-2.0 * z * gu0 + w * gu1 + x * gu2 - w * gv0 - 2.0 * z * gv1 + y * gv2 + x * gn0 + y * gn1);
    const double proj = w * dw + x * dx + y * dy + z * dz;
    h.g[3] = static_cast<float>((dw - w * proj) * inv);
    h.g[4] = static_cast<float>((dx - x * proj) * inv);
    h.g[5] = static_cast<float>((dy - y * proj) * inv);
    h.g[6] = static_cast<float>((dz - z * proj) * inv);

    return h;
}

// Add the hits of `rest` to global memory: lane c adds component c.
template <int FM, int CM>
__device__ __forceinline__ void add_direct(uint64_t rest, const WalkHit& h, const TraceParams& P, const lds_f32* rows,
                                           int ri, int id, float* gbuf, int gs, int lane)
{
    using Row = WalkRow<FM, CM>;
    const int nc = 10 + P.F;
    while (rest) {
        const int L = __ffsll(static_cast<unsigned long long>(rest)) - 1;
        rest &= rest - 1;
        float* dst = gbuf + static_cast<int64_t>(bcast(id, L)) * gs;
        const lds_f32* row = rows + bcast(ri, L) * Row::words;
        const double wgt = bcast(h.wgt, L);
        const uint32_t lit = static_cast<uint32_t>(bcast(static_cast<int>(h.lit), L));
        float val = 0.0f;
#pragma unroll
        for (int k = 0; k < 10; ++k) val = lane == k ? bcast(h.g[k], L) : val;
        if (lane >= 10 && lane < nc) val = feature_grad<FM, CM>(row, lane - 10, wgt, lit);
        if (lane < nc && val != 0.0f) atomicAdd(dst + lane, val);
        if constexpr (FM > 54) {
            if (64 + lane < nc) {
                val = feature_grad<FM, CM>(row, 54 + lane, wgt, lit);
                if (val != 0.0f) atomicAdd(dst + 64 + lane, val);
            }
        }
    }
}

// A ray's inputs, in registers from their loads on (the upstream of wide
// features is loaded when the row is written).
template <int FM, int CM>
struct WalkInput {
    using Row = WalkRow<FM, CM>;
    static constexpr int held = Row::up <= 16 ? Row::up : 1;
    Ray ray;
    float gO, gD, up[held];

    __device__ __forceinline__ float upstream(const TraceParams& P, const GradIn& gin, int64_t r, int k) const
    {
        const int FO = CM == kColSH ? 3 : (CM == kColNormal ? P.F + 3 : P.F);
        return gin.gF && k < FO ? gin.gF[r * FO + k] : 0.0f;
    }
    __device__ __forceinline__ void load(const TraceParams& P, const float* __restrict__ ro,
                                         const float* __restrict__ rd, const GradIn& gin, int64_t r)
    {
        ray = load_ray(ro, rd, r);
        gO = gin.gO ? gin.gO[r] : 0.0f;
        gD = gin.gD ? gin.gD[r] : 0.0f;
        if constexpr (Row::up <= 16) {
#pragma unroll
            for (int k = 0; k < held; ++k) up[k] = upstream(P, gin, r, k);
        }
    }
    // False when the ray has nothing to do.
    __device__ __forceinline__ bool work(const TraceParams& P, const GradIn& gin, int64_t r) const
    {
        bool any = gO != 0.0f || gD != 0.0f;
        if constexpr (Row::up <= 16) {
#pragma unroll
            for (int k = 0; k < held; ++k) any = any || up[k] != 0.0f;
        } else {
            for (int k = 0; k < Row::up; ++k) any = any || upstream(P, gin, r, k) != 0.0f;
        }
        return any && ray_valid(ray);
    }
    __device__ __forceinline__ void store(lds_f32* row, const TraceParams& P, const GradIn& gin, int64_t r) const
    {
        row[0] = ray.ox, row[1] = ray.oy, row[2] = ray.oz;
        row[3] = ray.dx, row[4] = ray.dy, row[5] = ray.dz;
        row[6] = gO, row[7] = gD;
        if constexpr (Row::up <= 16) {
#pragma unroll
            for (int k = 0; k < held; ++k) row[8 + k] = up[k];
        } else {
            for (int k = 0; k < Row::up; ++k) row[8 + k] = upstream(P, gin, r, k);
        }
        if constexpr (CM == kColSH) {
            float Y[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) Y[j] = 0.0f;
            sh_basis(ray.dx, ray.dy, ray.dz, P.sh_deg, Y);
#pragma unroll
            for (int j = 0; j < 16; ++j) row[Row::basis + j] = Y[j];
        }
    }
};

// Walk over stored lists.  Blocks claim chunks of `groups` groups of `group`
// slots (of `order`, or of the launch); a block's waves take the chunk's
// groups in turn.  Rays whose list is not complete are put in rm_list.
template <int FM, int CM>
__global__ __launch_bounds__(WalkShape<FM>::waves * 64) __attribute__((amdgpu_waves_per_eu(3)))
void k_walk(RawSurfels raw, TraceParams P, int64_t R, const float* __restrict__ ro, const float* __restrict__ rd,
            OutPtrs saved, GradIn gin, float* gbuf, int gs, unsigned long long* next_chunk,
            const uint32_t* __restrict__ order, int group, int groups, int* rm_list, unsigned long long* rm_count)
{
    using Sh = WalkShape<FM>;
    using Row = WalkRow<FM, CM>;
    constexpr int threads = Sh::waves * 64;
    __shared__ int keys[Sh::slots];
    __shared__ float vals[Sh::comps * Sh::stride];
    __shared__ int filled, next, left;
    __shared__ long long chunk;
    __shared__ float ray_rows[Sh::waves * Sh::group * Row::words];
    __shared__ uint32_t marks[Sh::waves * 64];
    __shared__ float stages[Sh::waves * kStageWords * 64];
    __shared__ int n_segs[Sh::waves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nc = 10 + P.F;
    const WalkTable<FM> tb{keys, vals, &filled};
    lds_f32* rows = (lds_f32*)(ray_rows + wave * Sh::group * Row::words);
    lds_u32* mark = (lds_u32*)(marks + wave * 64);
    lds_f32* stage = (lds_f32*)(stages + wave * kStageWords * 64) + lane;
    tb.clear(tid, threads, nc);
    if (tid == 0) next = 0, left = 0;
    __syncthreads();
    int n_hits = 0, at = 0;              // hits of the wave's group, first of the next step
    int n_rays = 0, first = 0, end = 0;  // the group's rays with work; lane i: places of the i-th one's hits
    double S = 0.0;
    bool more = true;  // chunks may be left
    // The next group is loaded in three parts, a step apart: 1 its rays' ids are
    // on the way, 2 their inputs are.  (Without, some wave of the block would
    // wait out that chain in every step, and the others for it at the barrier.)
    int ahead = 0;
    int64_t next_r = 0;
    int next_n = 0;
    bool next_in = false;
    WalkInput<FM, CM> next_ray{};
    auto take_group = [&]() {
        int g = 0;
        if (lane == 0) g = atomicAdd(&next, 1);
        g = bcast(g, 0);
        if (g >= left) return;
        // the rays of `waves` groups are dealt in turn, so that waves at the
        // same place of their groups are on neighbouring rays
        const int64_t slot = (chunk * groups + g / Sh::waves * Sh::waves) * group + lane * Sh::waves + g % Sh::waves;
        next_in = lane < group && slot < R;
        next_r = 0;
        if (next_in) next_r = order ? static_cast<int64_t>(order[slot]) : slot;
        ahead = 1;
    };
    auto take_rays = [&]() {
        next_n = 0;
        if (next_in) {
            next_n = saved.n_hits[next_r];
            next_ray.load(P, ro, rd, gin, next_r);
        }
        ahead = 2;
    };
    // A step's hits, their loads issued before the barriers of the step before.
    int id = 0, ri = 0, held = 0, segs = 0;
    float Ti = 0.0f;
    bool valid = false, last = false;
    float4 mo{};
    auto take_hits = [&]() {
        // the ray of stream place at + lane: the one that holds `at`, plus the
        // rays that start between
        mark[lane] = 0u;
        lds_order();
        if (lane < n_rays && first > at && first < at + 64) mark[first - at] = 1u;
        lds_order();
        const uint64_t starts = __ballot(mark[lane] != 0u);
        held = __popcll(__ballot(lane < n_rays && end <= at));
        segs = __popcll(starts) + 1;
        const int t = at + lane;
        valid = t < n_hits;
        ri = valid ? held + wave_rank(starts) + static_cast<int>((starts >> lane) & 1ull) : 0;
        const lds_f32* l = rows + ri * Row::words + Row::list;
        const int64_t r = (static_cast<int64_t>(__float_as_int(l[1])) << 32) | static_cast<uint32_t>(__float_as_int(l[0]));
        const int h = __float_as_int(l[2]) - 1 - (t - __float_as_int(l[3]));
        last = valid && t == __float_as_int(l[3]);
        id = 0;
        Ti = 0.0f;
        if (valid) {
            id = saved.hit_ids[r * saved.H_cap + h];
            Ti = saved.hit_T[r * saved.H_cap + h];
        }
    };
    while (true) {
        if (at >= n_hits) {
            at = n_hits = n_rays = 0;
            S = 0.0;
            if (ahead == 0 && more) take_group();
            if (ahead == 1) take_rays();
            if (ahead == 2) {
                ahead = 0;
                bool work = next_in && next_n > 0 && next_n <= saved.H_cap;
                const bool cut = next_in && next_n != 0 && !work;
                const uint64_t mc = __ballot(cut);
                if (mc) {  // one atomic per wave for the rays it leaves
                    unsigned long long b = 0;
                    if (lane == 0) b = atomicAdd(rm_count, static_cast<unsigned long long>(__popcll(mc)));
                    b = bcast(static_cast<uint64_t>(b), 0);
                    if (cut) rm_list[b + wave_rank(mc)] = static_cast<int>(next_r);
                }
                work = work && next_ray.work(P, gin, next_r);
                // rows are packed: the i-th ray with work is row (and lane) i
                const uint64_t mw = __ballot(work);
                const int incl = static_cast<int>(wave_scan(static_cast<uint32_t>(work ? next_n : 0)));
                if (work) {
                    lds_f32* row = rows + wave_rank(mw) * Row::words;
                    next_ray.store(row, P, gin, next_r);
                    lds_f32* l = row + Row::list;
                    l[0] = __int_as_float(static_cast<int>(next_r));
                    l[1] = __int_as_float(static_cast<int>(next_r >> 32));
                    l[2] = __int_as_float(next_n), l[3] = __int_as_float(incl - next_n);
                }
                lds_order();
                n_rays = __popcll(mw);
                n_hits = bcast(incl, 63);
                first = end = 0;
                if (lane < n_rays) {
                    const lds_f32* l = rows + lane * Row::words + Row::list;
                    first = __float_as_int(l[3]);
                    end = first + __float_as_int(l[2]);
                }
                if (n_hits > 0) {
                    take_hits();
                    mo = *reinterpret_cast<const float4*>(raw.pk + static_cast<int64_t>(id) * raw.ps);
                }
            }
        }
        if (at < n_hits) {
            if (ahead == 1)
                take_rays();
            else if (ahead == 0 && more)
                take_group();
            const WalkHit hit = walk_step<FM, CM>(raw, P, rows, ri, valid, last, id, mo, Ti, S, lane);
            const int slot = valid ? tb.find(id) : -1;
            add_direct<FM, CM>(__ballot(valid && slot < 0), hit, P, rows, ri, id, gbuf, gs, lane);
#pragma unroll
            for (int k = 0; k < 10; ++k) stage[k * 64] = hit.g[k];
            const long long wb = __double_as_longlong(hit.wgt);
            stage[10 * 64] = __int_as_float(static_cast<int>(wb));
            stage[11 * 64] = __int_as_float(static_cast<int>(wb >> 32));
            const int seg = ri - held;  // ray of the step
            stage[12 * 64] = __uint_as_float((slot < 0 ? kNoSlot : static_cast<uint32_t>(slot)) |
                                             (static_cast<uint32_t>(seg) & 63u) << 16 | hit.lit << 22 |
                                             static_cast<uint32_t>(ri) << 25);
            if (lane == 0) n_segs[wave] = segs;
            at += 64;
            if (at < n_hits) take_hits();
        } else {
            stage[12 * 64] = __uint_as_float(kNoSlot);
            if (lane == 0) n_segs[wave] = 0;
        }
        const bool busy = __syncthreads_or(at < n_hits || ahead != 0) != 0;
        const bool full = filled > Sh::flush;
        const bool refill = more && next >= left;
        if (at < n_hits) mo = *reinterpret_cast<const float4*>(raw.pk + static_cast<int64_t>(id) * raw.ps);
        // This wave's components of every wave's hits, a ray's hits at a time
        // (rays share surfels).  With two components per wave all values are
        // loaded first, so that their latencies overlap; more do not fit the
        // registers.
        const int counts = lane < Sh::waves ? n_segs[lane] : 0;
        lds_f32* mine = (lds_f32*)vals + wave * Sh::stride;
        auto value = [&](int b, int c, uint32_t info) {
            const lds_f32* st = (const lds_f32*)stages + b * kStageWords * 64 + lane;
            if (c < 10) return st[c * 64];
            const lds_f32* row = (const lds_f32*)ray_rows + (b * Sh::group + (info >> 25)) * Row::words;
            const double wgt = __longlong_as_double((static_cast<long long>(__float_as_int(st[11 * 64])) << 32) |
                                                    static_cast<uint32_t>(__float_as_int(st[10 * 64])));
            return feature_grad<FM, CM>(row, c - 10, wgt, (info >> 22) & 7u);
        };
        auto add = [&](int b, uint32_t info, const float* v) {
            const uint32_t slot = info & 0xffffu;
            const int seg = slot == kNoSlot ? -1 : static_cast<int>((info >> 16) & 63u);
            const int count = bcast(counts, b);
            for (int g = 0; g < count; ++g) {
                if (seg == g) {
                    lds_f32* to = mine + slot;
                    float sum[Sh::per_wave];
#pragma unroll
                    for (int i = 0; i < Sh::per_wave; ++i)
                        if (wave + i * Sh::waves < nc) sum[i] = to[i * Sh::waves * Sh::stride] + v[i];
#pragma unroll
                    for (int i = 0; i < Sh::per_wave; ++i)
                        if (wave + i * Sh::waves < nc) to[i * Sh::waves * Sh::stride] = sum[i];
                }
                lds_order();
            }
        };
        const lds_f32* infos = (const lds_f32*)stages + 12 * 64 + lane;
        if constexpr (Sh::per_wave <= 2) {
            float v[Sh::waves][Sh::per_wave];
            uint32_t info[Sh::waves];
#pragma unroll
            for (int b = 0; b < Sh::waves; ++b) info[b] = __float_as_uint(infos[b * kStageWords * 64]);
#pragma unroll
            for (int i = 0; i < Sh::per_wave; ++i) {
                const int c = wave + i * Sh::waves;
                if (c < 10) {
#pragma unroll
                    for (int b = 0; b < Sh::waves; ++b) v[b][i] = value(b, c, info[b]);
                } else if (c < nc) {
#pragma unroll
                    for (int b = 0; b < Sh::waves; ++b) v[b][i] = value(b, c, info[b]);
                }
            }
#pragma unroll
            for (int b = 0; b < Sh::waves; ++b) add(b, info[b], v[b]);
        } else {
            for (int b = 0; b < Sh::waves; ++b) {
                if (bcast(counts, b) == 0) continue;
                const uint32_t info = __float_as_uint(infos[b * kStageWords * 64]);
                float v[Sh::per_wave];
#pragma unroll
                for (int i = 0; i < Sh::per_wave; ++i) {
                    const int c = wave + i * Sh::waves;
                    v[i] = c < nc ? value(b, c, info) : 0.0f;
                }
                add(b, info, v);
            }
        }
        __syncthreads();
        if (full) {
            tb.write(tid, threads, nc, gbuf, gs);
            __syncthreads();
            tb.clear(tid, threads, nc);
        }
        if (refill) {
            if (tid == 0) {
                chunk = static_cast<long long>(atomicAdd(next_chunk, 1ull));
                left = static_cast<int64_t>(chunk) * groups * group < R ? groups : 0;
                next = 0;
            }
            __syncthreads();
            more = left > 0;
        } else if (full) {
            __syncthreads();
        }
        if (!more && !busy) break;
    }
    tb.write(tid, threads, nc, gbuf, gs);
}

// Rays of rm_list (their stored list was cut), each traced again by one wave
// into a list of List hits in LDS, which the wave then walks (no table: they
// are few).  A ray with more hits is left to `rest`.
template <int FM, int CM, int List>
__global__ __launch_bounds__(kWaveBlock)
void k_remarch(SceneView sc, RawSurfels raw, TraceParams P, const float* __restrict__ ro, const float* __restrict__ rd,
               GradIn gin, float* gbuf, int gs, int reserve, const int* __restrict__ rm_list,
               const unsigned long long* rm_count, unsigned long long* next, int* rest, unsigned long long* rest_count)
{
    using Row = WalkRow<FM, CM>;
    __shared__ uint32_t lds[kWaveLdsWords];
    __shared__ int list_ids[List];
    __shared__ float list_T[List];
    __shared__ float row_mem[Row::words];
    lds_f32* row = (lds_f32*)row_mem;
    const int lane = threadIdx.x;
    const int64_t count = static_cast<int64_t>(*rm_count);
    OutPtrs out{};  // the composite goes where the traversal's areas are, idle by then
    out.O = reinterpret_cast<float*>(lds);
    out.D = out.O + 1;
    out.feat = out.O + 2;
    out.hit_ids = list_ids;
    out.hit_T = list_T;
    out.H_cap = List;
    // the first ray by the block's number, the others by claims: a launch
    // that has nothing to do touches no counter
    for (int64_t i = blockIdx.x; i < count;) {
        const int64_t r = bcast(rm_list[i], 0);
        const Ray v = load_ray(ro, rd, r);
        Ray ray;
        ray.ox = bcast(v.ox, 0), ray.oy = bcast(v.oy, 0), ray.oz = bcast(v.oz, 0);
        ray.dx = bcast(v.dx, 0), ray.dy = bcast(v.dy, 0), ray.dz = bcast(v.dz, 0);
        WalkInput<FM, CM> in;
        in.load(P, ro, rd, gin, r);
        if (in.work(P, gin, r)) {  // the same in every lane
            in.store(row, P, gin, r);
            const int n = trace_ray_wave<CM>(sc, P, ray, 0, out, (lds_u32*)lds, reserve, lane);
            // the list is read by other lanes than wrote it
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            lds_order();
            if (n > List) {
                if (lane == 0) rest[atomicAdd(rest_count, 1ull)] = static_cast<int>(r);
            } else {
                double S = 0.0;
                for (int at = 0; at < n; at += 64) {
                    const int t = at + lane;
                    const bool valid = t < n;
                    const int id = valid ? list_ids[n - 1 - t] : 0;
                    const float Ti = valid ? list_T[n - 1 - t] : 0.0f;
                    const float4 mo = *reinterpret_cast<const float4*>(raw.pk + static_cast<int64_t>(id) * raw.ps);
                    const WalkHit hit = walk_step<FM, CM>(raw, P, row, 0, valid, t == 0, id, mo, Ti, S, lane);
                    add_direct<FM, CM>(__ballot(valid), hit, P, row, 0, id, gbuf, gs, lane);
                }
            }
            lds_order();
        }
        unsigned long long b = 0;
        if (lane == 0) b = atomicAdd(next, 1ull);
        i = static_cast<int64_t>(gridDim.x) + static_cast<int64_t>(bcast(static_cast<uint64_t>(b), 0));
    }
}

}  // namespace irgs
