// Relighting variant of the trace's consumer.  To relight, the trace
// alpha-blends albedo, roughness and the normal along each incident ray
// (normalised weights T_i alpha_i / sum T_i alpha_i), and the ray's indirect
// radiance is shaded in one query with the split-sum approximation:
// L_ind = L_d + L_s, L_d = A / pi * E(N), L_s = P_R(refl) (F0 S_A + S_B),
// where E is the irradiance of the sky, P_R the sky prefiltered with the GGX
// lobe of roughness R, and (S_A, S_B) a pre-integrated BRDF table.
//
// Readings (the construction is cited, no numbers are given): the sky is a
// cubemap of 6 E x E texels, each integral a sum over texel centres with
// their exact solid angle 4 / (E^2 (1 + s^2 + t^2)^{3/2}); P_R assumes
// normal = view = reflection direction; roughness levels r_l = (l + 1) / M,
// nearest level; the table at cell centres ((i + 1/2)/S, (j + 1/2)/S) is the
// GGX-importance-sampled estimate over 256 Hammersley points; F0 = 0.04 and
// the Smith G of the shading BRDF; lookups take the nearest texel / cell;
// the surface is viewed from -d; a ray with no hit carries no indirect light.
#include <hip/hip_runtime.h>

#include "irgs_internal.hpp"

namespace irgs {

namespace {

constexpr float kPiR = 3.14159265358979323846f;
constexpr float kF0R = 0.04f;
constexpr int kHammersley = 256;

// Unnormalised direction of face coordinates (s, t) in [-1, 1]^2 on a face:
// the inverse of the nearest-texel addressing below.
__device__ __forceinline__ void face_point(int face, float s, float t, float* d)
{
    switch (face) {
        case 0: d[0] = 1.0f, d[1] = -t, d[2] = -s; break;
        case 1: d[0] = -1.0f, d[1] = -t, d[2] = s; break;
        case 2: d[0] = s, d[1] = 1.0f, d[2] = t; break;
        case 3: d[0] = s, d[1] = -1.0f, d[2] = -t; break;
        case 4: d[0] = s, d[1] = -t, d[2] = 1.0f; break;
        default: d[0] = -s, d[1] = -t, d[2] = -1.0f; break;
    }
}

// Centre direction (unit) and solid angle of texel `idx` of an E x E cube.
__device__ __forceinline__ void texel_dir(int idx, int E, float* d, float* dw)
{
    const int face = idx / (E * E);
    const int rc = idx - face * E * E;
    const int row = rc / E, col = rc - row * E;
    const float s = 2.0f * (col + 0.5f) / E - 1.0f;
    const float t = 2.0f * (row + 0.5f) / E - 1.0f;
    face_point(face, s, t, d);
    const float q = 1.0f + s * s + t * t;
    const float inv = 1.0f / sqrtf(q);
    d[0] *= inv, d[1] *= inv, d[2] *= inv;
    *dw = 4.0f / (E * E * q * sqrtf(q));
}

// Nearest texel of direction (x, y, z): the same addressing as the shading.
__device__ __forceinline__ int texel_of(float x, float y, float z, int E)
{
    const float ax = fabsf(x), ay = fabsf(y), az = fabsf(z);
    int face;
    float s, t, m;
    if (ax >= ay && ax >= az) {
        m = ax, face = x >= 0.0f ? 0 : 1, s = x >= 0.0f ? -z : z, t = -y;
    } else if (ay >= az) {
        m = ay, face = y >= 0.0f ? 2 : 3, s = x, t = y >= 0.0f ? z : -z;
    } else {
        m = az, face = z >= 0.0f ? 4 : 5, s = z >= 0.0f ? x : -x, t = -y;
    }
    s /= m;
    t /= m;
    const int col = min(max(static_cast<int>(floorf((s + 1.0f) * E * 0.5f)), 0), E - 1);
    const int row = min(max(static_cast<int>(floorf((t + 1.0f) * E * 0.5f)), 0), E - 1);
    return (face * E + row) * E + col;
}

__device__ __forceinline__ float smith(float l, float v, float r)
{
    const float k = (r + 1.0f) * (r + 1.0f) * 0.125f;
    return l / (l * (1.0f - k) + k) * (v / (v * (1.0f - k) + k));
}

// Sums over all input texels for kSkyOut output texels per block.  The
// threads of a block split the input texels kSkySplit ways (a lane's output is
// lane & 15, its part of each input tile the rest of its index), so a sky of
// 6 x 32^2 texels fills the chip where one output texel per thread left 98% of
// it idle, and the FP32 running sums are 64 times shorter.  A tile's
// directions, solid angles and radiances are put in LDS once per block.  With
// the unit half vector h of c and w, |c x h|^2 = |w - c|^2 / 4 and (c . h)^2 =
// |w + c|^2 / 4, so the lobe needs neither h nor a square root, and keeps its
// accuracy near the peak (q = |c x h|^2 + (c . h)^2 alpha^2).  VALU-bound:
// about 12 instructions per pair of texels and level; E = 32, 8 levels:
// 3,816 + 2,473 us (prefilter and irradiance, texel directions recomputed for
// every pair) -> 122 us together.
constexpr int kSkyOut = 16;
constexpr int kSkyThreads = 512;
constexpr int kSkySplit = kSkyThreads / kSkyOut;
constexpr int kSkyTile = 512;

// Levels [l0, l0 + MC) (those below M are stored) and, with IRR, the irradiance.
template <int MC, bool IRR>
__global__ __launch_bounds__(kSkyThreads) void k_sky(int E, int M, int l0, const float* __restrict__ env,
                                                     float* __restrict__ irr, float* __restrict__ pref)
{
    constexpr int kSums = 4 * MC + (IRR ? 3 : 0);
    __shared__ float4 dirs[kSkyTile];  // w, solid angle
    __shared__ float4 light[kSkyTile];
    __shared__ float red[kSkyThreads / 64][kSkyOut][kSums + 1];
    const int n = 6 * E * E;
    const int tid = threadIdx.x;
    const int o = blockIdx.x * kSkyOut + (tid & (kSkyOut - 1));
    const int part = tid / kSkyOut;
    float c[3], dwo;
    texel_dir(min(o, n - 1), E, c, &dwo);
    float a2[MC > 0 ? MC : 1];
#pragma unroll
    for (int l = 0; l < MC; ++l) {
        const float rough = static_cast<float>(min(l0 + l, M - 1) + 1) / M;
        a2[l] = (rough * rough) * (rough * rough);
    }
    float sum[kSums];
#pragma unroll
    for (int k = 0; k < kSums; ++k) sum[k] = 0.0f;
    for (int t0 = 0; t0 < n; t0 += kSkyTile) {
        __syncthreads();
        if (t0 + tid < n) {
            float w[3], dw;
            texel_dir(t0 + tid, E, w, &dw);
            dirs[tid] = make_float4(w[0], w[1], w[2], dw);
            const float* L = env + 3 * static_cast<int64_t>(t0 + tid);
            light[tid] = make_float4(L[0], L[1], L[2], 0.0f);
        }
        __syncthreads();
        const int cnt = min(kSkyTile, n - t0);
        for (int i = part; i < cnt; i += kSkySplit) {
            const float4 w = dirs[i];
            const float cs = w.x * c[0] + w.y * c[1] + w.z * c[2];
            if (cs <= 0.0f) continue;
            const float4 L = light[i];
            const float f = cs * w.w;
            if constexpr (IRR) {
                sum[4 * MC] = fmaf(f, L.x, sum[4 * MC]);
                sum[4 * MC + 1] = fmaf(f, L.y, sum[4 * MC + 1]);
                sum[4 * MC + 2] = fmaf(f, L.z, sum[4 * MC + 2]);
            }
            if constexpr (MC > 0) {
                const float dx = w.x - c[0], dy = w.y - c[1], dz = w.z - c[2];
                const float sx = w.x + c[0], sy = w.y + c[1], sz = w.z + c[2];
                const float s2 = 0.25f * fmaf(dx, dx, fmaf(dy, dy, dz * dz));  // |c x h|^2
                const float h2 = 0.25f * fmaf(sx, sx, fmaf(sy, sy, sz * sz));  // (c . h)^2
#pragma unroll
                for (int l = 0; l < MC; ++l) {
                    const float q = fmaf(h2, a2[l], s2);
                    // D up to its constant, which the quotient drops; a2 / q in
                    // [a2, 1 / a2] keeps it in range
                    const float d = a2[l] * __builtin_amdgcn_rcpf(q);
                    const float wt = d * d * f;
                    sum[4 * l] += wt;
                    sum[4 * l + 1] = fmaf(wt, L.x, sum[4 * l + 1]);
                    sum[4 * l + 2] = fmaf(wt, L.y, sum[4 * l + 2]);
                    sum[4 * l + 3] = fmaf(wt, L.z, sum[4 * l + 3]);
                }
            }
        }
    }
    // the four parts of a wave, then the waves
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
        sum[k] += __shfl_xor(sum[k], 16);
        sum[k] += __shfl_xor(sum[k], 32);
        if ((tid & 63) < kSkyOut) red[tid >> 6][tid & 63][k] = sum[k];
    }
    __syncthreads();
    for (int t = tid; t < kSkyOut * kSums; t += kSkyThreads) {
        const int oo = t / kSums, k = t - oo * kSums;
        float v = 0.0f;
        for (int w = 0; w < kSkyThreads / 64; ++w) v += red[w][oo][k];
        red[0][oo][k] = v;
    }
    __syncthreads();
    for (int t = tid; t < kSkyOut * kSums; t += kSkyThreads) {
        const int oo = t / kSums, k = t - oo * kSums;
        const int64_t out = static_cast<int64_t>(blockIdx.x) * kSkyOut + oo;
        if (out >= n) continue;
        if (k >= 4 * MC) {
            if (IRR) irr[3 * out + k - 4 * MC] = red[0][oo][k];
        } else if ((k & 3) != 0 && l0 + k / 4 < M) {
            pref[3 * ((l0 + k / 4) * static_cast<int64_t>(n) + out) + (k & 3) - 1] = red[0][oo][k] / red[0][oo][k & ~3];
        }
    }
}

// One cell per kTableLanes lanes, which split the 256 samples: the latency of
// 256 dependent samples per thread took 82 us at S = 32, this 5 us.
constexpr int kTableLanes = 32;

__global__ void k_brdf_table(int S, float* __restrict__ table)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int cell = t / kTableLanes, sub = t % kTableLanes;
    if (cell >= S * S) return;  // whole groups leave together
    const int i = cell / S, j = cell - i * S;
    const float nv = (i + 0.5f) / S, r = (j + 0.5f) / S;
    const float vx = sqrtf(1.0f - nv * nv), vz = nv;  // view in the xz plane, normal +z
    const float a2 = (r * r) * (r * r);
    float A = 0.0f, B = 0.0f;
    for (int k = sub; k < kHammersley; k += kTableLanes) {
        const float x = (k + 0.5f) / kHammersley;
        const float y = static_cast<float>(__brev(static_cast<unsigned>(k))) * 2.3283064365386963e-10f;  // 2^-32
        // cos^2 and sin^2 of the sampled half vector over one exact
        // denominator (1 - y is exact), so neither cancels at small roughness
        const float den = fmaf(a2, y, 1.0f - y);
        const float ct = sqrtf((1.0f - y) / den), st = sqrtf(a2 * y / den);
        float sp, cp;
        sincosf(2.0f * kPiR * x, &sp, &cp);
        const float hx = st * cp, hz = ct;
        const float vh = hx * vx + hz * vz;
        const float lz = 2.0f * vh * hz - vz;
        if (lz <= 0.0f) continue;
        const float g = smith(lz, nv, r) * vh / (hz * nv);
        const float om = 1.0f - vh, om2 = om * om;
        const float fc = om2 * om2 * om;
        A = fmaf(1.0f - fc, g, A);
        B = fmaf(fc, g, B);
    }
#pragma unroll
    for (int off = kTableLanes / 2; off > 0; off >>= 1) {
        A += __shfl_xor(A, off);
        B += __shfl_xor(B, off);
    }
    if (sub == 0) {
        table[2 * cell] = A / kHammersley;
        table[2 * cell + 1] = B / kHammersley;
    }
}

__global__ void k_relight_lind(RelightArgs a, float* __restrict__ lind)
{
    for (int64_t r = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; r < a.R;
         r += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const float O = a.O[r];
        float out[3] = {0, 0, 0};
        if (O > 0.0f) {
            const float* f = a.Fo + 7 * r;
            const float inv = 1.0f / O;
            const float A[3] = {f[0] * inv, f[1] * inv, f[2] * inv};
            const float Rg = fminf(fmaxf(f[3] * inv, 0.0f), 1.0f);
            float N[3] = {f[4] * inv, f[5] * inv, f[6] * inv};
            const float nn = sqrtf(N[0] * N[0] + N[1] * N[1] + N[2] * N[2]);
            if (nn > 0.0f) N[0] /= nn, N[1] /= nn, N[2] /= nn;
            float d[3] = {a.rd[3 * r], a.rd[3 * r + 1], a.rd[3 * r + 2]};
            const float dn = sqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
            d[0] /= dn, d[1] /= dn, d[2] /= dn;
            const float* E = a.irr + 3 * static_cast<int64_t>(texel_of(N[0], N[1], N[2], a.E));
            const float nv = fminf(fmaxf(-(N[0] * d[0] + N[1] * d[1] + N[2] * d[2]), 0.0f), 1.0f);
            const float dd = d[0] * N[0] + d[1] * N[1] + d[2] * N[2];
            const float refl[3] = {d[0] - 2.0f * dd * N[0], d[1] - 2.0f * dd * N[1], d[2] - 2.0f * dd * N[2]};
            const int lev = min(max(static_cast<int>(floorf(Rg * a.M + 0.5f)) - 1, 0), a.M - 1);
            const float* Pr = a.pref + 3 * (static_cast<int64_t>(lev) * 6 * a.E * a.E +
                                              texel_of(refl[0], refl[1], refl[2], a.E));
            const int ti = min(max(static_cast<int>(floorf(nv * a.S)), 0), a.S - 1);
            const int tj = min(max(static_cast<int>(floorf(Rg * a.S)), 0), a.S - 1);
            const float spec = kF0R * a.table[2 * (ti * a.S + tj)] + a.table[2 * (ti * a.S + tj) + 1];
#pragma unroll
            for (int c = 0; c < 3; ++c) out[c] = A[c] / kPiR * E[c] + Pr[c] * spec;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) lind[3 * r + c] = out[c];
    }
}

// Sampling weight of texel i: max(mean RGB, 0) times its solid angle at the
// centre, in FP64 (a NaN texel weighs 0).
__device__ __forceinline__ double texel_weight(int i, int E, const float* __restrict__ env)
{
    const int rc = i % (E * E);
    const int row = rc / E, col = rc - row * E;
    const double s = 2.0 * (col + 0.5) / E - 1.0, t = 2.0 * (row + 0.5) / E - 1.0;
    const double q = 1.0 + s * s + t * t;
    const double inten = fmax((static_cast<double>(env[3 * i]) + env[3 * i + 1] + env[3 * i + 2]) / 3.0, 0.0);
    return inten * 4.0 / (static_cast<double>(E) * E * q * sqrt(q));
}

constexpr int kCdfBlock = 1024;

// Inclusive CDF of the texel weights in texel order, one block: each thread
// sums a run of consecutive texels in FP64, a block scan offsets the runs,
// and each run is rewritten as running sums rounded once to FP32 (so the
// table never decreases).
__global__ __launch_bounds__(kCdfBlock) void k_env_cdf(int E, const float* __restrict__ env, float* __restrict__ cdf)
{
    __shared__ double part[kCdfBlock];
    const int n = 6 * E * E;
    const int per = (n + kCdfBlock - 1) / kCdfBlock;
    const int b = min(static_cast<int>(threadIdx.x) * per, n), e = min(b + per, n);
    // The first weights of a run are held in registers, the others computed
    // twice (a call at E = 32 / 48 / 128: 12 / 28 / 221 us; all twice 16 / 32 / 227).
    constexpr int kKept = 8;
    double kept[kKept];
    double run = 0.0;
#pragma unroll
    for (int j = 0; j < kKept; ++j) {
        kept[j] = b + j < e ? texel_weight(b + j, E, env) : 0.0;
        run += kept[j];
    }
    for (int i = b + kKept; i < e; ++i) run += texel_weight(i, E, env);
    part[threadIdx.x] = run;
    __syncthreads();
    for (int off = 1; off < kCdfBlock; off <<= 1) {
        const double v = threadIdx.x >= static_cast<unsigned>(off) ? part[threadIdx.x - off] : 0.0;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    run = threadIdx.x > 0 ? part[threadIdx.x - 1] : 0.0;
#pragma unroll
    for (int j = 0; j < kKept; ++j) {
        run += kept[j];
        if (b + j < e) cdf[b + j] = static_cast<float>(run);
    }
    for (int i = b + kKept; i < e; ++i) {
        run += texel_weight(i, E, env);
        cdf[i] = static_cast<float>(run);
    }
}

// One ray per sample drawn from the sky's intensity: the first texel whose
// CDF exceeds u0 * total (FP32), a point uniform in that texel's face
// coordinates, density p_j E^2 / 4 (1 + s^2 + t^2)^{3/2}, estimator weight
// 1 / (N pdf) above the horizon of n and 0 below it or for an empty sky.
__global__ void k_env_rays(EnvRayArgs a)
{
    const int nt = 6 * a.E * a.E;
    const float total = a.cdf[nt - 1];
    const float step = 2.0f / a.E;
    for (int64_t r = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; r < a.P * a.N;
         r += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t p = r / a.N;
        const float* u = a.u + 3 * r;
        float target = u[0] * total;
        if (!(target < total)) target = nextafterf(total, 0.0f);
        int lo = 0, hi = nt - 1;  // first index with cdf > target (the last one if none)
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (a.cdf[mid] > target) hi = mid;
            else lo = mid + 1;
        }
        const int face = lo / (a.E * a.E);
        const int rc = lo - face * a.E * a.E;
        const int row = rc / a.E, col = rc - row * a.E;
        const float s = (static_cast<float>(col) + u[1]) * step - 1.0f;
        const float t = (static_cast<float>(row) + u[2]) * step - 1.0f;
        float d[3];
        face_point(face, s, t, d);
        const float q = 1.0f + s * s + t * t;
        const float inv = 1.0f / sqrtf(q);
        d[0] *= inv, d[1] *= inv, d[2] *= inv;
        const float n[3] = {a.n[3 * p], a.n[3 * p + 1], a.n[3 * p + 2]};
        const float pj = (a.cdf[lo] - (lo > 0 ? a.cdf[lo - 1] : 0.0f)) / total;
        const float pdf = pj * (0.25f * a.E * a.E) * (q * sqrtf(q));
        const bool ok = d[0] * n[0] + d[1] * n[1] + d[2] * n[2] > 0.0f && pdf > 0.0f && total > 0.0f;
        a.wgt[r] = ok ? 1.0f / (static_cast<float>(a.N) * pdf) : 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            a.ro[3 * r + c] = fmaf(a.offset, n[c], a.x[3 * p + c]);
            a.rd[3 * r + c] = d[c];
        }
    }
}

unsigned grid_for(int64_t n, int block)
{
    const int64_t b = (n + block - 1) / block;
    return static_cast<unsigned>(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

}  // namespace

hipError_t launch_env_prefilter(int E, const float* env, int M, float* irr, float* pref, hipStream_t st)
{
    const int n = 6 * E * E;
    const unsigned grid = static_cast<unsigned>((n + kSkyOut - 1) / kSkyOut);
    if (!pref) M = 0;
    // eight levels per pass over the sky (four for a short rest), the
    // irradiance with the first
    int l0 = 0;
    bool first = irr != nullptr;
    while (l0 < M || first) {
        const int left = M - l0;
        if (left > 4) {
            if (first) k_sky<8, true><<<grid, kSkyThreads, 0, st>>>(E, M, l0, env, irr, pref);
            else k_sky<8, false><<<grid, kSkyThreads, 0, st>>>(E, M, l0, env, irr, pref);
            l0 += 8;
        } else if (left > 0) {
            if (first) k_sky<4, true><<<grid, kSkyThreads, 0, st>>>(E, M, l0, env, irr, pref);
            else k_sky<4, false><<<grid, kSkyThreads, 0, st>>>(E, M, l0, env, irr, pref);
            l0 += 4;
        } else {
            k_sky<0, true><<<grid, kSkyThreads, 0, st>>>(E, 1, 0, env, irr, pref);
        }
        first = false;
    }
    return hipGetLastError();
}

hipError_t launch_brdf_table(int S, float* table, hipStream_t st)
{
    const int64_t threads = static_cast<int64_t>(S) * S * kTableLanes;
    k_brdf_table<<<static_cast<unsigned>((threads + 127) / 128), 128, 0, st>>>(S, table);
    return hipGetLastError();
}

hipError_t launch_relight_lind(const RelightArgs& a, float* lind, hipStream_t st)
{
    if (a.R <= 0) return hipSuccess;
    k_relight_lind<<<grid_for(a.R, 256), 256, 0, st>>>(a, lind);
    return hipGetLastError();
}

hipError_t launch_env_cdf(int E, const float* env, float* cdf, hipStream_t st)
{
    k_env_cdf<<<1, kCdfBlock, 0, st>>>(E, env, cdf);
    return hipGetLastError();
}

hipError_t launch_env_rays(const EnvRayArgs& a, hipStream_t st)
{
    if (a.P * a.N <= 0) return hipSuccess;
    k_env_rays<<<grid_for(a.P * a.N, 256), 256, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace irgs
