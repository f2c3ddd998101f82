// Adjoint of the 2D Gaussian ray trace (the paper's trace is differentiable so
// that gradients of the indirect radiance reach the surfels, Sec. 3.3).
//
// With c_i = g_O + g_F . f_i + g_D tau_i the loss seen by one ray is
// L = sum_i T_i alpha_i c_i, T_i = prod_{j<i} (1 - alpha_j) (Eq. 2).  Walking
// the ray's hits back to front with the suffix composite
//     S_i = alpha_i c_i + (1 - alpha_i) S_{i+1},   S_end = 0,
// gives, without ever dividing by (1 - alpha),
//     dL/dalpha_i = T_i (c_i - S_{i+1}),   dL/df_i = T_i alpha_i g_F,
//     dL/dtau_i (through D) = T_i alpha_i g_D.
// alpha = o exp(-(u^2+v^2)/2) with u, v, tau from Eq. 6-7 chains these to
// the centre, the raw quaternion (through its normalisation), the scales and
// the opacity; per-surfel sums use FP32 global atomics.
//
// The hit list of a ray is read back from the forward pass (ids and the
// transmittance before each hit) and walked by bwd_wave.hpp.  A ray whose list
// was cut is traced again by one wave; what does not fit that wave's list
// either (or a tree its stack does not take) is re-marched by one lane: a first
// pass lists the hits and records the state at the start of k-buffer rounds, a
// second walks the list back to front or, where it does not hold them,
// re-collects the rounds last to first and walks each one.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "irgs_internal.hpp"
#include "bwd_wave.hpp"
#include "march.hpp"

namespace irgs {

namespace {

constexpr int kBwdBlock = 64;
constexpr int kMarchK = 16;  // the re-march's k-buffer (results do not depend on it)

// Per-surfel gradient components of one hit: mu (3), raw quaternion (4),
// scales (2), opacity (1), features (F).
template <int FM>
struct HitGrad {
    float g[10 + FM];
};

// The interleaved per-surfel accumulator: gbuf[id * gs + c].
struct GradAcc {
    float* gbuf;
    int gs;  // stride in floats (a multiple of 32: one 128 B line per surfel at F <= 22)
    int F;

    template <int FM>
    __device__ __forceinline__ void direct(int id, const HitGrad<FM>& h) const
    {
        float* g = gbuf + static_cast<int64_t>(id) * gs;
#pragma unroll
        for (int c = 0; c < 10 + FM; ++c)
            if (c < 10 + F && h.g[c] != 0.0f) atomicAdd(g + c, h.g[c]);
    }
};

// Gradient of one hit.  The geometry and the chain rule are evaluated in
// FP64 from the FP32 parameters: for a grazing ray (small n.r_d) FP32
// rounding of the depth is amplified into u, v and into dtau/dmu; FP64 keeps
// every surfel's gradient at FP32 accuracy.  Only the per-surfel
// contributions are rounded to FP32 for accumulation.  The transmittance
// before the hit (Ti) is the forward pass's own.
// With SH the features are RGB coefficients: the hit's colour is recomputed
// exactly as in the forward (FP32), and the coefficient gradients are
// T alpha g_F,c Y_j(d) wherever the channel is not clamped.
// With NRM (the relighting blend) the upstream holds F feature channels and
// then 3 for the hit's normal turned to face the ray, s n with s = -1 where
// n . d > 0; the turn is decided exactly as in the forward (the FP32 frame
// of the record, the same dot product), and s T alpha g_N adds to the
// gradient of n, which the rotation chain below carries to the quaternion.
template <int FM, int FU, bool SH, bool NRM = false>
__device__ __forceinline__ void grad_hit(const RawSurfels& raw, const TraceParams& P, int id, const Ray& ray,
                                         float Ti_f, float& S_f, float gO, const float* gF, float gD,
                                         HitGrad<FM>& h)
{
    const int F = P.F;
    const int64_t i = id;
    const float* row = raw.pk + i * raw.ps;  // the packed copy of surfel i's parameters
    const float4 mo = *reinterpret_cast<const float4*>(row);
    const float4 qf = *reinterpret_cast<const float4*>(row + 4);
    const float2 sc = *reinterpret_cast<const float2*>(row + 8);
    const double mx = mo.x, my = mo.y, mz = mo.z;
    const double su = sc.x, sv = sc.y;
    const double o = mo.w;
    const double qn = sqrt(double(qf.x) * qf.x + double(qf.y) * qf.y + double(qf.z) * qf.z + double(qf.w) * qf.w);
    const double inv = 1.0 / qn;
    const double w = qf.x * inv, x = qf.y * inv, y = qf.z * inv, z = qf.w * inv;
    const double tu0 = 1.0 - 2.0 * (y * y + z * z), tu1 = 2.0 * (x * y + w * z), tu2 = 2.0 * (x * z - w * y);
    const double tv0 = 2.0 * (x * y - w * z), tv1 = 1.0 - 2.0 * (x * x + z * z), tv2 = 2.0 * (y * z + w * x);
    const double n0 = 2.0 * (x * z + w * y), n1 = 2.0 * (y * z - w * x), n2 = 1.0 - 2.0 * (x * x + y * y);
    const double dx_ = ray.dx, dy_ = ray.dy, dz_ = ray.dz;
    const double wx = mx - ray.ox, wy = my - ray.oy, wz = mz - ray.oz;
    const double den = n0 * dx_ + n1 * dy_ + n2 * dz_;
    const double tau = (n0 * wx + n1 * wy + n2 * wz) / den;
    const double px = tau * dx_ - wx, py = tau * dy_ - wy, pz = tau * dz_ - wz;
    const double u = (px * tu0 + py * tu1 + pz * tu2) / su;
    const double v = (px * tv0 + py * tv1 + pz * tv2) / sv;
    const double G = exp(-0.5 * (u * u + v * v));
    const double alpha = o * G;
    const double Ti = Ti_f;
    const double S = S_f;

    double c = gO + gD * tau;
    const float* f = raw.feat_packed ? row + 12 : raw.feat + i * F;
    const double wgt = Ti * alpha;
    if constexpr (SH) {
        float Y[16], col[3];
        sh_basis(ray.dx, ray.dy, ray.dz, P.sh_deg, Y);
        sh_raw(f, P.sh_deg, Y, col);
        const int nb = (P.sh_deg + 1) * (P.sh_deg + 1);
        double gc[3];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            c += double(gF[ch]) * fmaxf(col[ch], 0.0f);
            gc[ch] = col[ch] > 0.0f ? wgt * gF[ch] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch)
                if (3 * j + ch < FM) h.g[10 + 3 * j + ch] = j < nb ? static_cast<float>(gc[ch] * Y[j]) : 0.0f;
#pragma unroll
        for (int k = 48; k < FM; ++k) h.g[10 + k] = 0.0f;
    } else {
        static_assert(SH || FU == FM, "plain features: one upstream channel per feature");
#pragma unroll
        for (int k = 0; k < FM; ++k) {
            const float fv = k < F ? f[k] : 0.0f;
            c += double(gF[k]) * fv;
        }
#pragma unroll
        for (int k = 0; k < FM; ++k) h.g[10 + k] = (!NRM || k < F) ? static_cast<float>(wgt * gF[k]) : 0.0f;
    }
    double sN = 0.0, gN0 = 0.0, gN1 = 0.0, gN2 = 0.0;  // normal channels: turn and upstream
    if constexpr (NRM) {
        float tf[3], vf[3], nf[3];
        quat_frame(qf, tf, vf, nf);
        sN = dot3(nf[0], nf[1], nf[2], ray.dx, ray.dy, ray.dz) > 0.0f ? -1.0 : 1.0;
#pragma unroll
        for (int k = 0; k < FM; ++k) {
            gN0 += k == F ? double(gF[k]) : 0.0;
            gN1 += k == F + 1 ? double(gF[k]) : 0.0;
            gN2 += k == F + 2 ? double(gF[k]) : 0.0;
        }
        c += sN * (gN0 * n0 + gN1 * n1 + gN2 * n2);
    }
    const double dA = Ti * (c - S);
    S_f = static_cast<float>(alpha * c + (1.0 - alpha) * S);

    h.g[9] = static_cast<float>(dA * G);

    const double gu = -dA * alpha * u;
    const double gv = -dA * alpha * v;
    h.g[7] = static_cast<float>(-gu * u / su);
    h.g[8] = static_cast<float>(-gv * v / sv);
    // p - mu = tau d - w;  du/d(p-mu) = t_u / s_u
    const double au = gu / su, av = gv / sv;
    const double gpx = au * tu0 + av * tv0, gpy = au * tu1 + av * tv1, gpz = au * tu2 + av * tv2;
    const double gtau = wgt * gD + gpx * dx_ + gpy * dy_ + gpz * dz_;
    const double gt_den = gtau / den;
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
}

// alpha of the k-buffer entry at leaf position pos (the same arithmetic as
// the forward composite, so T is reproduced bit for bit).
__device__ __forceinline__ float entry_alpha(const SceneView& sc, const Ray& ray, int pos)
{
    const SurfelRec s = load_rec(sc.rec, pos);
    float tau, rho2;
    plane_hit(s, ray, &tau, &rho2);
    return alpha_of(s, rho2);
}

template <int K>
__device__ __forceinline__ void entry(const KBuf<K>& kb, const float* Tj, int j, int* pos, float* T)
{
    int ri = 0;
    float rt = 0.0f;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        ri = q == j ? kb.pos(q) : ri;
        rt = q == j ? Tj[q] : rt;
    }
    *pos = ri;
    *T = rt;
}

template <int FU>
struct LaneUp {
    float gO, gD, gF[FU];
    bool any;
};

// Upstream gradients of ray r; FO = composited channels (the g_feat stride).
template <int FU>
__device__ __forceinline__ LaneUp<FU> load_upstream(const GradIn& gin, int64_t r, int FO)
{
    const int F = FO;
    LaneUp<FU> u;
    u.gO = gin.gO ? gin.gO[r] : 0.0f;
    u.gD = gin.gD ? gin.gD[r] : 0.0f;
    u.any = u.gO != 0.0f || u.gD != 0.0f;
#pragma unroll
    for (int k = 0; k < FU; ++k) {
        u.gF[k] = (gin.gF && k < F) ? gin.gF[r * F + k] : 0.0f;
        u.any = u.any || u.gF[k] != 0.0f;
    }
    return u;
}

// Re-march one ray.  Pass 1 marches the k-buffer rounds again (the forward's
// arithmetic, so T is reproduced bit for bit), recording the hits (id and T) in
// the lane's list of `cap` while it holds them and the state at the start of
// rounds as checkpoints.  Pass 2 walks the list back to front or, for a ray
// with more hits, re-collects the rounds last to first from the nearest
// checkpoint.  Checkpoints are kept for every stride-th round:
// once all kBwdCheckpoints are taken every other one is dropped and the stride
// doubles, so pass 2 re-collects at most stride - 1 extra rounds per round.
template <int K, int FM, int FU, bool SH, bool NRM, class Acc>
__device__ __forceinline__ void bwd_remarch(const SceneView& sc, const RawSurfels& raw, const TraceParams& P,
                                            const Ray& ray, const LaneUp<FU>& up, const Acc& acc, Stack& st,
                                            float4* ck, int64_t ck_stride, int* list_ids, float* list_T, int cap)
{
    float S = 0.0f;
    Counters ct;
    const BoxRay q = box_ray(ray);
    uint64_t after = 0;
    float T = 1.0f;
    int nh = 0;
    int rounds = 0;
    int stride = 1;  // a power of two: checkpoint i holds the start of round i * stride
    int nck = 0;
    bool done = false;
    while (!done) {
        if ((rounds & (stride - 1)) == 0) {
            if (nck == kBwdCheckpoints) {
                for (int i = 1; i < kBwdCheckpoints / 2; ++i) ck[i * ck_stride] = ck[2 * i * ck_stride];
                nck = kBwdCheckpoints / 2;
                stride *= 2;
            }
            if ((rounds & (stride - 1)) == 0)
                ck[(nck++) * ck_stride] = make_float4(__uint_as_float(static_cast<uint32_t>(after >> 32)),
                                                      __uint_as_float(static_cast<uint32_t>(after)), T,
                                                      __int_as_float(nh));
        }
        KBuf<K> kb;
        kb.clear();
        collect_bvh<K>(kb, sc, ray, q, P.t_min, P.t_max, after, st, ct);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (j < kb.cnt && !done) {
                if (nh < cap) {
                    list_ids[nh] = __float_as_int(sc.rec[kb.pos(j)].c.w);
                    list_T[nh] = T;
                }
                T = T * (1.0f - entry_alpha(sc, ray, kb.pos(j)));
                ++nh;
                if (T < P.T_min) done = true;
            }
        }
        if (kb.cnt < K)
            done = true;
        else
            after = kb.last();
        ++rounds;
    }
    const int total = nh;
    if (total <= cap) {
        for (int i = total - 1; i >= 0; --i) {
            HitGrad<FM> h;
            grad_hit<FM, FU, SH, NRM>(raw, P, list_ids[i], ray, list_T[i], S, up.gO, up.gF, up.gD, h);
            acc.template direct<FM>(list_ids[i], h);
        }
        return;
    }
    for (int rr = rounds - 1; rr >= 0; --rr) {
        const int base = rr / stride;
        float4 c4 = ck[base * ck_stride];
        after = (static_cast<uint64_t>(__float_as_uint(c4.x)) << 32) | __float_as_uint(c4.y);
        T = c4.z;
        int nb = __float_as_int(c4.w);
        KBuf<K> kb;
        for (int adv = base * stride; adv < rr; ++adv) {  // rounds between the checkpoint and rr
            kb.clear();
            collect_bvh<K>(kb, sc, ray, q, P.t_min, P.t_max, after, st, ct);
#pragma unroll
            for (int j = 0; j < K; ++j) T = j < kb.cnt ? T * (1.0f - entry_alpha(sc, ray, kb.pos(j))) : T;
            nb += kb.cnt;
            after = kb.last();
        }
        kb.clear();
        collect_bvh<K>(kb, sc, ray, q, P.t_min, P.t_max, after, st, ct);
        const int m = min(kb.cnt, total - nb);
        float Tj[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            Tj[j] = T;
            T = j < m ? T * (1.0f - entry_alpha(sc, ray, kb.pos(j))) : T;
        }
        for (int j = m - 1; j >= 0; --j) {
            int pos;
            float Ti;
            entry<K>(kb, Tj, j, &pos, &Ti);
            const int id = __float_as_int(sc.rec[pos].c.w);
            HitGrad<FM> h;
            grad_hit<FM, FU, SH, NRM>(raw, P, id, ray, Ti, S, up.gO, up.gF, up.gD, h);
            acc.template direct<FM>(id, h);
        }
    }
}

// The rays of `list` re-marched by one lane each.
template <int K, int FM, int FU, bool SH, bool NRM>
__global__ __launch_bounds__(kBwdBlock) void k_remarch_lanes(SceneView sc, RawSurfels raw, TraceParams P,
                                                             const float* __restrict__ ro, const float* __restrict__ rd,
                                                             GradIn gin, float* gbuf, int gs, int* ovf, float4* ck,
                                                             int* lists, int cap, const int* __restrict__ list,
                                                             const unsigned long long* list_count,
                                                             unsigned long long* next)
{
    const int tid = threadIdx.x;
    const int64_t gtid = static_cast<int64_t>(blockIdx.x) * kBwdBlock + tid;
    const int64_t nthr = static_cast<int64_t>(gridDim.x) * kBwdBlock;
    // the stack lives entirely in the global area (0 LDS slots)
    Stack st{nullptr, as_glb(ovf + gtid), static_cast<int>(nthr), tid, 0, 0};
    const GradAcc acc{gbuf, gs, P.F};
    int* my_ids = lists + gtid * 2 * cap;
    float* my_T = reinterpret_cast<float*>(my_ids + cap);
    const int64_t count = static_cast<int64_t>(*list_count);
    while (true) {
        unsigned long long c = 0;
        if (tid == 0) c = atomicAdd(next, 1ull);
        const int64_t base = static_cast<int64_t>(bcast(static_cast<uint64_t>(c), 0)) * kBwdBlock;
        if (base >= count) return;
        if (base + tid < count) {
            const int64_t r = list[base + tid];
            const Ray ray = load_ray(ro, rd, r);
            const LaneUp<FU> up = load_upstream<FU>(gin, r, SH ? 3 : (NRM ? P.F + 3 : P.F));
            if (up.any && ray_valid(ray))
                bwd_remarch<K, FM, FU, SH, NRM>(sc, raw, P, ray, up, acc, st, ck + gtid, nthr, my_ids, my_T, cap);
        }
    }
}

// Sort key of a ray for the backward's chunks: the Morton code (10 bits per
// axis) of its mean hit point ro + (D / O) rd inside the root's box; a ray
// without a hit sorts last.
__global__ void k_ray_keys(int64_t R, const float* __restrict__ ro, const float* __restrict__ rd,
                           const float* __restrict__ O, const float* __restrict__ D, const WideNode* __restrict__ root,
                           uint64_t* __restrict__ keys, uint32_t* __restrict__ vals)
{
    const int64_t r = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (r >= R) return;
    float lo[3], hi[3];
    root_box(root, lo, hi);
    uint64_t key = 0xffffffffull;
    const float o = O[r];
    if (o > 0.0f && lo[0] <= hi[0]) {
        const float t = D[r] / o;
        const float x[3] = {fmaf(t, rd[3 * r], ro[3 * r]), fmaf(t, rd[3 * r + 1], ro[3 * r + 1]),
                            fmaf(t, rd[3 * r + 2], ro[3 * r + 2])};
        key = morton30(x, lo, hi);
    }
    keys[r] = key;
    vals[r] = static_cast<uint32_t>(r);
}

// One packed row per surfel (see RawSurfels).  A thread writes 16 bytes of a
// row, so that a wave writes whole lines.
__global__ void k_pack(int64_t n, int F, int ps, bool feats, bool recips, const float* __restrict__ mu,
                       const float* __restrict__ quat, const float* __restrict__ scale, const float* __restrict__ opac,
                       const float* __restrict__ feat, float* __restrict__ pk)
{
    const int parts = ps / 4;
    const int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    const int64_t i = t / parts;
    const int c = static_cast<int>(t - i * parts);
    if (i >= n) return;
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (c == 0) {
        v = make_float4(mu[3 * i], mu[3 * i + 1], mu[3 * i + 2], opac[i]);
    } else if (c == 1) {
        v = make_float4(quat[4 * i], quat[4 * i + 1], quat[4 * i + 2], quat[4 * i + 3]);
    } else if (c == 2) {
        v.x = scale[2 * i], v.y = scale[2 * i + 1];
        const double w = quat[4 * i], x = quat[4 * i + 1], y = quat[4 * i + 2], z = quat[4 * i + 3];
        const long long inv = __double_as_longlong(1.0 / sqrt(w * w + x * x + y * y + z * z));
        v.z = __int_as_float(static_cast<int>(inv)), v.w = __int_as_float(static_cast<int>(inv >> 32));
    } else if (recips && c == parts - 1) {
        const long long u = __double_as_longlong(1.0 / double(scale[2 * i]));
        const long long w = __double_as_longlong(1.0 / double(scale[2 * i + 1]));
        v = make_float4(__int_as_float(static_cast<int>(u)), __int_as_float(static_cast<int>(u >> 32)),
                        __int_as_float(static_cast<int>(w)), __int_as_float(static_cast<int>(w >> 32)));
    } else if (feats) {
        const int f0 = 4 * (c - 3);
        const float* f = feat + i * F;
        v.x = f0 < F ? f[f0] : 0.0f, v.y = f0 + 1 < F ? f[f0 + 1] : 0.0f;
        v.z = f0 + 2 < F ? f[f0 + 2] : 0.0f, v.w = f0 + 3 < F ? f[f0 + 3] : 0.0f;
    }
    reinterpret_cast<float4*>(pk)[t] = v;
}

// gbuf (interleaved per surfel) added into the caller's gradient arrays.
__global__ void k_grad_out(int64_t n, int F, int gs, const float* __restrict__ gbuf, GradOut go)
{
    const int nc = 10 + F;
    for (int64_t flat = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; flat < n * nc;
         flat += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t i = flat / nc;
        const int c = static_cast<int>(flat - i * nc);
        const float v = gbuf[i * gs + c];
        if (v == 0.0f) continue;
        if (c < 3) {
            if (go.mu) go.mu[3 * i + c] += v;
        } else if (c < 7) {
            if (go.quat) go.quat[4 * i + c - 3] += v;
        } else if (c < 9) {
            if (go.scale) go.scale[2 * i + c - 7] += v;
        } else if (c == 9) {
            if (go.opac) go.opac[i] += v;
        } else {
            if (go.feat) go.feat[i * F + c - 10] += v;
        }
    }
}

// Rays ordered by where they land (see k_ray_keys); *order stays null when the
// forward's O and D are not there or the launch is too large to sort.
hipError_t landing_order(const SceneView& sc, int64_t R, const float* ro, const float* rd, const OutPtrs& saved,
                         char* p, const uint32_t** order, hipStream_t st)
{
    uint64_t* k0 = reinterpret_cast<uint64_t*>(p);
    uint64_t* k1 = k0 + R;
    uint32_t* v0 = reinterpret_cast<uint32_t*>(k1 + R);
    uint32_t* v1 = v0 + R;
    uint32_t* counts = v1 + R;
    k_ray_keys<<<static_cast<unsigned>((R + 255) / 256), 256, 0, st>>>(R, ro, rd, saved.O, saved.D, sc.wnodes, k0, v0);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = sort_pairs(static_cast<int>(R), k0, v0, k1, v1, counts, 4, st);
    if (e == hipSuccess) *order = v0;
    return e;
}

template <int FM, int CM>
hipError_t launch_f(const SceneView& sc, const RawSurfels& raw, const TraceParams& P, int64_t R, const float* ro,
                    const float* rd, const OutPtrs& saved, const GradIn& gin, const GradOut& go, int wide_depth,
                    char* scratch, hipStream_t st)
{
    using Sh = WalkShape<FM>;
    const BackwardPlan pl = plan_backward(R, sc.n, P.F, wide_depth, saved.H_cap);
    const int gs = grad_stride(P.F);
    float* gbuf = reinterpret_cast<float*>(scratch);
    // a claim counter for the walk, then a count and a claim counter per re-march
    unsigned long long* claims = reinterpret_cast<unsigned long long*>(scratch + pl.claims);
    int* rm_list = reinterpret_cast<int*>(scratch + pl.rm_list);
    int* rest = reinterpret_cast<int*>(scratch + pl.rest);
    // zero the accumulator and the claim counters behind it
    hipError_t e = fill_u32(gbuf, static_cast<int64_t>(pl.rm_list / 4), 0u, st);
    if (e != hipSuccess) return e;
    const uint32_t* order = nullptr;
    if (R >= kSortWalkRays && saved.O && saved.D && ray_sort_words(R) > 0) {
        e = landing_order(sc, R, ro, rd, saved, scratch + pl.sort, &order, st);
        if (e != hipSuccess) return e;
    }
    {
        const int64_t resident = resident_blocks(k_walk<FM, CM>, Sh::waves * 64);
        const int64_t waves = (resident > 0 ? resident : 256) * Sh::waves;
        // groups of full size once every wave gets several, chunks of a few
        // groups per wave; smaller launches spread over all waves
        int64_t group = R / (2 * waves);
        group = group < 1 ? 1 : (group > Sh::group ? Sh::group : group);
        const int groups = group == Sh::group ? 2 * Sh::waves : Sh::waves;
        const int64_t chunks = (R + group * groups - 1) / (group * groups);
        k_walk<FM, CM><<<persistent_grid(chunks, resident), Sh::waves * 64, 0, st>>>(
            raw, P, R, ro, rd, saved, gin, gbuf, gs, claims, order, static_cast<int>(group), groups, rm_list, claims + 1);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // the cut lists, then what each launch leaves to the next
    int *todo = rm_list, *left = rest;
    unsigned long long *count = claims + 1, *next = claims + 2;
    auto wave_launch = [&](auto kern) {
        const unsigned grid = persistent_grid(std::min(R, kRemarchWaves), resident_blocks(kern, kWaveBlock));
        kern<<<grid, kWaveBlock, 0, st>>>(sc, raw, P, ro, rd, gin, gbuf, gs, wave_stack_reserve(wide_depth), todo, count,
                                          next, left, count + 2);
        std::swap(todo, left);
        count += 2, next += 2;
        return hipGetLastError();
    };
    if (pl.short_lists) e = wave_launch(k_remarch<FM, CM, kRemarchShort>);
    if (e == hipSuccess && pl.long_lists) e = wave_launch(k_remarch<FM, CM, kRemarchList>);
    if (e == hipSuccess && pl.lane_blocks > 0) {
        constexpr int FU = CM == kColSH ? 4 : FM;
        k_remarch_lanes<kMarchK, FM, FU, CM == kColSH, CM == kColNormal>
            <<<static_cast<unsigned>(pl.lane_blocks), kBwdBlock, 0, st>>>(
                sc, raw, P, ro, rd, gin, gbuf, gs, reinterpret_cast<int*>(scratch + pl.stacks),
                reinterpret_cast<float4*>(scratch + pl.checkpoints), reinterpret_cast<int*>(scratch + pl.lists),
                pl.lane_list, todo, count, next);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    const int64_t work = static_cast<int64_t>(sc.n) * (10 + P.F);
    const int blocks = static_cast<int>(work < 2048 * 256 ? (work + 255) / 256 : 2048);
    k_grad_out<<<blocks > 0 ? blocks : 1, 256, 0, st>>>(sc.n, P.F, gs, gbuf, go);
    return hipGetLastError();
}

}  // namespace

hipError_t pack_surfels(const RawSurfels& raw, int64_t n, int F, float* pk, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int64_t t = n * (raw.ps / 4);
    k_pack<<<static_cast<unsigned>((t + 255) / 256), 256, 0, st>>>(n, F, raw.ps, raw.feat_packed, raw.recips, raw.mu, raw.quat,
                                                                   raw.scale, raw.opac, raw.feat, pk);
    return hipGetLastError();
}

BackwardPlan plan_backward(int64_t R, int64_t N, int F, int wide_depth, int H_cap)
{
    BackwardPlan pl{};
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t here = at;
        at += (bytes + 255) & ~static_cast<size_t>(255);
        return here;
    };
    take(static_cast<size_t>(N) * grad_stride(F) * sizeof(float));
    pl.claims = take(256);
    pl.rm_list = take(static_cast<size_t>(R) * sizeof(int));
    pl.rest = take(static_cast<size_t>(R) * sizeof(int));
    pl.sort = take(R >= kSortWalkRays ? ray_sort_words(R) * sizeof(float) : 0);
    const bool cut = N > H_cap;  // a list can have been cut
    const bool wave = wave_stack_fits(wide_depth);
    pl.short_lists = cut && wave && R > kRemarchSmall;
    pl.long_lists = cut && wave && !(pl.short_lists && N <= kRemarchShort);
    if (cut && (!wave || N > kRemarchList)) {
        pl.lane_list = wave ? 0 : static_cast<int>(std::min<int64_t>(kRemarchLaneList, N));
        const size_t stack = (3 * static_cast<size_t>(wide_depth) + 1) * sizeof(int);
        const size_t checkpoints = kBwdCheckpoints * sizeof(float4);
        const size_t list = 2 * static_cast<size_t>(pl.lane_list) * sizeof(int);
        int64_t lanes = kRemarchLanes;
        if (!wave) {
            const int64_t fit = static_cast<int64_t>(kRemarchLaneBytes / (stack + checkpoints + list));
            lanes = std::max(lanes, std::min(kRemarchLanesAll, fit / kBwdBlock * kBwdBlock));
        }
        pl.lane_blocks = std::min((R + kBwdBlock - 1) / kBwdBlock, lanes / kBwdBlock);
        lanes = pl.lane_blocks * kBwdBlock;
        pl.stacks = take(lanes * stack);
        pl.checkpoints = take(lanes * checkpoints);
        pl.lists = take(lanes * list);
    }
    pl.bytes = at;
    return pl;
}

hipError_t launch_backward(const SceneView& sc, const RawSurfels& raw, const TraceParams& P, int k, int64_t R,
                           const float* ro, const float* rd, const OutPtrs& saved, const GradIn& gin,
                           const GradOut& go, int wide_depth, char* scratch, hipStream_t st)
{
    if (R <= 0) return hipSuccess;
    const bool special = P.sh_deg >= 0 || P.normals;
    if (!features_offered(k, P.F, special)) return hipErrorInvalidValue;
    if (P.sh_deg >= 0) return launch_f<48, kColSH>(sc, raw, P, R, ro, rd, saved, gin, go, wide_depth, scratch, st);
    if (P.normals) {  // F <= 5 features and 3 normal channels upstream
        if (P.F > 5) return hipErrorInvalidValue;
        return launch_f<8, kColNormal>(sc, raw, P, R, ro, rd, saved, gin, go, wide_depth, scratch, st);
    }
    if (P.F <= 8) return launch_f<8, kColPlain>(sc, raw, P, R, ro, rd, saved, gin, go, wide_depth, scratch, st);
    if (P.F <= 16) return launch_f<16, kColPlain>(sc, raw, P, R, ro, rd, saved, gin, go, wide_depth, scratch, st);
    return launch_f<64, kColPlain>(sc, raw, P, R, ro, rd, saved, gin, go, wide_depth, scratch, st);
}

}  // namespace irgs
