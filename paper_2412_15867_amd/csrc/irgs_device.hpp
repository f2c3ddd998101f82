// Device-side building blocks of the 2D Gaussian ray tracer (gfx950).
//
// Geometry follows Sec. 3.2 of the paper:
//   * a surfel has centre mu, opacity o, a rotation quaternion q = (w,x,y,z)
//     whose rotation matrix has columns (t_u, t_v, n), and scales (s_u, s_v);
//   * Eq. 6: the ray meets the surfel plane at tau = n.(mu - r_o) / n.r_d;
//   * Eq. 7: at p = r_o + tau r_d the local coordinates are
//     u = (p - mu).t_u / s_u and v = (p - mu).t_v / s_v and the influence is
//     G = exp(-(u^2 + v^2) / 2); alpha = o G;
//   * Eq. 2 / Eq. 8: hits are alpha-blended front to back.
// Readings fixed here (the paper gives no value): a hit needs
// t_min < tau < t_max, u^2 + v^2 <= min(sigma^2, 2 ln(o / alpha_min)) (the
// support cap and the alpha_min test of Eq. 5's proxy, both inclusive);
// hits are ordered by (tau, surfel id); compositing includes a hit and then
// stops once T < T_min.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace irgs {

constexpr int kBlock = 256;          // threads per block of the trace kernels
constexpr int kStackLds = 24;        // per-lane traversal stack entries kept in LDS
constexpr int kLeafBit = 0x80000000; // child reference: leaf flag
constexpr int kNoChild = -1;         // child reference: empty slot (N == 1 root)

// 64-byte surfel record, stored in BVH leaf order.
//   a = (mu.xyz, o)            b = (n.xyz, rho2_max)
//   c = (t_u / s_u, id bits)   d = (t_v / s_v, 0)
// rho2_max = min(sigma^2, 2 ln(o / alpha_min)), or -1 for a surfel that can
// never be hit (o < alpha_min or an invalid parameter).
struct __align__(16) SurfelRec {
    float4 a, b, c, d;
};

// Internal BVH node: the boxes of both children plus their references.
// A reference r >= 0 is an internal node, r with kLeafBit set is the leaf at
// leaf position (r & ~kLeafBit), kNoChild is an empty slot.
struct __align__(16) BvhNode {
    float4 p0;  // lo0.xyz, hi0.x
    float4 p1;  // hi0.yz, lo1.xy
    float4 p2;  // lo1.z, hi1.xyz
    int4 ch;    // child0, child1, parent, unused
};

// 4-wide node used by the traversal (collapsed from the binary tree): four
// children of 32 bytes, so that a lane that tests one child reads it with two
// 16-byte loads and four neighbouring lanes read one 128-byte line.  A child
// reference r >= 0 is a wide node; r with kLeafBit set is a cluster of
// ((r & 15) + 1) surfels starting at leaf position ((r & ~kLeafBit) >> 4);
// kNoChild is an empty slot.  The box is kept as the sum of its corners
// (twice the centre) and its extent: box and slab test share the centre.  An
// empty box has the extent -inf, which no ray crosses; one that is not finite
// is taken as all of space (centre 0, extent +inf).
struct __align__(16) WideChild {
    float c2[3], ext[3];
    int32_t ref;
    uint32_t slab;  // a slab that holds the child's discs (see Slab, child_span)
};
struct __align__(128) WideNode {
    WideChild c[4];
};

__device__ __forceinline__ WideChild load_child(const WideNode* __restrict__ nodes, int node, int slot)
{
    const float4* p = reinterpret_cast<const float4*>(&nodes[node].c[slot]);
    const float4 a = p[0], b = p[1];
    WideChild w;
    w.c2[0] = a.x, w.c2[1] = a.y, w.c2[2] = a.z;
    w.ext[0] = a.w, w.ext[1] = b.x, w.ext[2] = b.y;
    w.ref = __float_as_int(b.z);
    w.slab = __float_as_uint(b.w);
    return w;
}

__device__ __forceinline__ bool child_empty(const WideChild& w) { return !(w.ext[0] >= 0.0f); }

// A child's slab: bytes 0-2 are an integer normal N (N_i + 128, largest
// component 127 in size), byte 3 its thickness H in 1/255 of the box's own
// extent along N; every disc below the child lies in the box and in
// |N.(2 x - c2)| <= H.  Surfels of one surface patch share a plane, so
// the slab is thin where the box of a tilted patch is fat.
struct Slab {
    float nx, ny, nz;
    float h;  // H
};

__device__ __forceinline__ Slab child_slab(const WideChild& w)
{
    Slab s;
    s.nx = static_cast<float>(w.slab & 0xffu) - 128.0f;
    s.ny = static_cast<float>((w.slab >> 8) & 0xffu) - 128.0f;
    s.nz = static_cast<float>((w.slab >> 16) & 0xffu) - 128.0f;
    const float ext = fmaf(fabsf(s.nx), w.ext[0], fmaf(fabsf(s.ny), w.ext[1], fabsf(s.nz) * w.ext[2]));
    s.h = ext * (static_cast<float>(w.slab >> 24) * (1.0f / 255.0f));
    return s;
}
constexpr uint32_t kSlabNone = 0xff000000u | 0xff8080u;  // N = (0, 0, 127), H = the box's extent: culls nothing

constexpr int kLeafDefault = 12;  // surfels per cluster leaf (at most 16)

__host__ __device__ __forceinline__ int cluster_ref(int first, int count)
{
    return kLeafBit | (first << 4) | (count - 1);
}

// What a trace kernel needs of one scene (passed by value).
struct SceneView {
    const SurfelRec* rec;   // N records, leaf order
    const WideNode* wnodes; // 4-wide nodes, root = 0
    const float* feat;      // N x F, caller layout (original ids)
    int32_t n;
    int32_t F;
    int32_t start, n_start; // wide nodes [start, start + n_start) hold every leaf below them: a traversal's first nodes
};

// How the composited channels are formed from a hit (template argument of
// the forward kernels).
enum ColourMode : int {
    kColPlain = 0,   // the surfel's F features
    kColSH = 1,      // view-dependent colour from RGB SH coefficients (3 channels)
    kColNormal = 2,  // the F features, then the unit normal turned to face the ray (F + 3)
};

struct TraceParams {
    float t_min, t_max, T_min;
    int32_t F;       // features per surfel
    int32_t sh_deg;  // -1: features composited as they are; 0..3: RGB SH coefficients (3 output channels)
    int32_t normals; // 1: the features, then the ray-facing unit normal (F + 3 output channels)
};

struct Ray {
    float ox, oy, oz, dx, dy, dz;
};

__device__ __forceinline__ float dot3(float ax, float ay, float az, float bx, float by, float bz)
{
    return fmaf(ax, bx, fmaf(ay, by, az * bz));
}

// Columns (t_u, t_v, n) of the rotation of q = (w,x,y,z), normalised here.
// Returns the norm of q.
__device__ __forceinline__ float quat_frame(float4 q, float* tu, float* tv, float* nn)
{
    float qn = sqrtf(q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w);
    float inv = 1.0f / qn;
    float w = q.x * inv, x = q.y * inv, y = q.z * inv, z = q.w * inv;
    tu[0] = 1.0f - 2.0f * (y * y + z * z);
    tu[1] = 2.0f * (x * y + w * z);
    tu[2] = 2.0f * (x * z - w * y);
    tv[0] = 2.0f * (x * y - w * z);
    tv[1] = 1.0f - 2.0f * (x * x + z * z);
    tv[2] = 2.0f * (y * z + w * x);
    nn[0] = 2.0f * (x * z + w * y);
    nn[1] = 2.0f * (y * z - w * x);
    nn[2] = 1.0f - 2.0f * (x * x + y * y);
    return qn;
}

// Eq. 6-7 against one record: depth tau and rho2 = u^2 + v^2 of the ray's
// crossing of the surfel plane.  Every kernel (brute force, BVH, packed,
// composite, backward re-march) evaluates a (ray, surfel) pair through this
// one function, so the pair is decided and ordered identically everywhere.
__device__ __forceinline__ void plane_hit(const SurfelRec& s, const Ray& r, float* tau_out, float* rho2_out)
{
    const float wx = s.a.x - r.ox, wy = s.a.y - r.oy, wz = s.a.z - r.oz;
    const float den = dot3(s.b.x, s.b.y, s.b.z, r.dx, r.dy, r.dz);
    const float num = dot3(s.b.x, s.b.y, s.b.z, wx, wy, wz);
    const float tau = num * __builtin_amdgcn_rcpf(den);  // den == 0: +-inf or NaN, rejected by the window
    const float px = fmaf(tau, r.dx, -wx), py = fmaf(tau, r.dy, -wy), pz = fmaf(tau, r.dz, -wz);
    const float u = dot3(px, py, pz, s.c.x, s.c.y, s.c.z);
    const float v = dot3(px, py, pz, s.d.x, s.d.y, s.d.z);
    *tau_out = tau;
    *rho2_out = fmaf(u, u, v * v);
}

// A hit: inside (t_min, t_max) (n.r_d == 0 gives +-inf or NaN, rejected) and
// inside the support rho2 <= rho2_max.
__device__ __forceinline__ bool hit_test(const SurfelRec& s, const Ray& r, float t_min, float t_max,
                                         float* tau_out, float* rho2_out)
{
    plane_hit(s, r, tau_out, rho2_out);
    return (*tau_out > t_min && *tau_out < t_max) && (*rho2_out <= s.b.w);
}

// alpha = o exp(-rho2 / 2) (Eq. 7 times the opacity).
__device__ __forceinline__ float alpha_of(const SurfelRec& s, float rho2) { return s.a.w * __expf(-0.5f * rho2); }

__device__ __forceinline__ SurfelRec load_rec(const SurfelRec* __restrict__ rec, int i)
{
    const float4* p = reinterpret_cast<const float4*>(rec + i);
    SurfelRec s;
    s.a = p[0];
    s.b = p[1];
    s.c = p[2];
    s.d = p[3];
    return s;
}

// Hit keys: (tau, leaf position) packed into one 64-bit integer whose
// unsigned order is the lexicographic order.  tau maps to a 32-bit unsigned
// m of the same order (sign-flipped when negative); the key is the top bit,
// then m, then the 31-bit position.  With the top bit set every key read as
// a double is negative, finite and normal (m's high bits equal to all ones or
// all zeros would need a NaN tau), so the FP64 order of keys is the reverse
// of their integer order: the k-buffer merges with FP64 min and max.
__device__ __forceinline__ uint64_t hit_key(float tau, int pos)
{
    const uint32_t u = __float_as_uint(tau);
    const uint32_t m = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return 0x8000000000000000ull | (static_cast<uint64_t>(m) << 31) | static_cast<uint32_t>(pos);
}

__device__ __forceinline__ float key_tau(uint64_t k)
{
    const uint32_t m = static_cast<uint32_t>(k >> 31);
    return __uint_as_float((m & 0x80000000u) ? (m & 0x7fffffffu) : ~m);
}

__device__ __forceinline__ int key_pos(uint64_t k) { return static_cast<int>(static_cast<uint32_t>(k) & 0x7fffffffu); }

// Above every key as an integer (a finite tau gives at most 0xFFBF...), and
// -inf read as a double.  Key 0 (below every key) marks a ray's first round.
constexpr uint64_t kKeyNone = 0xFFF0000000000000ull;

// The root node's box: the union of its non-empty child slots (lo > hi
// when the scene is empty).
__device__ __forceinline__ void root_box(const WideNode* __restrict__ root, float lo[3], float hi[3])
{
    const float inf = __int_as_float(0x7f800000);
    for (int a = 0; a < 3; ++a) {
        lo[a] = inf;
        hi[a] = -inf;
    }
    for (int c = 0; c < 4; ++c) {
        const WideChild& w = root->c[c];
        if (child_empty(w)) continue;
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], 0.5f * (w.c2[a] - w.ext[a]));
            hi[a] = fmaxf(hi[a], 0.5f * (w.c2[a] + w.ext[a]));
        }
    }
}

// 30-bit Morton code (10 bits per axis) of point x in the box [lo, hi],
// clamped to the box.
__device__ __forceinline__ uint32_t morton30(const float x[3], const float lo[3], const float hi[3])
{
    uint32_t code = 0;
    for (int a = 0; a < 3; ++a) {
        const float ext = hi[a] - lo[a];
        const float u = ext > 0.0f ? (x[a] - lo[a]) / ext : 0.0f;
        const uint32_t q = static_cast<uint32_t>(fminf(fmaxf(u * 1024.0f, 0.0f), 1023.0f));
        uint32_t v = q;  // spread 10 bits to every third position
        v = (v | (v << 16)) & 0x030000ffu;
        v = (v | (v << 8)) & 0x0300f00fu;
        v = (v | (v << 4)) & 0x030c30c3u;
        v = (v | (v << 2)) & 0x09249249u;
        code |= v << (2 - a);
    }
    return code;
}

// A ray as the box tests take it: half the inverse direction and twice the
// origin.  Per axis the ray is at the box's centre for t = (c2 - 2 o) i and
// within it for t +- ext |i|: the difference is taken before the product, so
// these depths are rounded by a few 1e-7 of the distance along the axis, far
// inside the padding every leaf box carries (at least 1e-5 (1 + |mu|)).
struct BoxRay {
    float ix, iy, iz;
    float ox2, oy2, oz2;
};

// Entry and exit of a ray in a child's box, clamped to [lo, hi], then narrowed
// to its slab, which the ray crosses for 2 t in (num -+ H) / den: the child is
// crossed inside the window when *tn <= *tf.  The pad on H covers the FP32
// rounding of these depths and of a hit's (both stay within a few 1e-7 of the
// distances involved off the plane; 1e-5 (1 + |w|) is taken, times twice |N| <
// 220).  A ray parallel to the plane gives infinities, which are a miss
// outside the slab and narrow nothing inside; a NaN narrows nothing.
__device__ __forceinline__ void child_span(const WideChild& w, const Ray& r, const BoxRay& q, float lo, float hi,
                                           float* tn, float* tf)
{
    const float wx = w.c2[0] - q.ox2, wy = w.c2[1] - q.oy2, wz = w.c2[2] - q.oz2;
    const float tx = wx * q.ix, ty = wy * q.iy, tz = wz * q.iz;
    const float ax = fabsf(q.ix), ay = fabsf(q.iy), az = fabsf(q.iz);
    const float bn = fmaxf(fmaxf(fmaf(-w.ext[0], ax, tx), fmaf(-w.ext[1], ay, ty)), fmaf(-w.ext[2], az, tz));
    const float bf = fminf(fminf(fmaf(w.ext[0], ax, tx), fmaf(w.ext[1], ay, ty)), fmaf(w.ext[2], az, tz));
    const Slab s = child_slab(w);
    const float num = dot3(s.nx, s.ny, s.nz, wx, wy, wz);
    const float den = dot3(s.nx, s.ny, s.nz, r.dx, r.dy, r.dz);
    const float far = fmaxf(fmaxf(fabsf(wx), fabsf(wy)), fabsf(wz));
    const float h = fmaf(far, 4.4e-3f, s.h + 4.4e-3f);
    const float inv = 0.5f * __builtin_amdgcn_rcpf(den);
    const float ta = (num - h) * inv, tb = (num + h) * inv;
    *tn = fmaxf(fmaxf(bn, lo), fminf(ta, tb));
    *tf = fminf(fminf(bf, hi), fmaxf(ta, tb));
}

// View-dependent colour (Sec. 3.1: each surfel's colour is modelled by
// spherical harmonics; the trace uses that colour).  `k` holds RGB
// coefficients of the real SH basis up to degree `deg`, coefficient-major
// (k[3 j + c], j = l^2 + l + m); the colour seen along direction (dx, dy, dz)
// (normalised here) is max(sum_j Y_j k[3 j + c] + 1/2, 0) per channel.  The
// basis is sqrt(2) Re / sqrt(2) Im of the complex harmonics with the
// Condon-Shortley phase (m > 0 / m < 0), written out as polynomials in the
// unit direction; the constants are sqrt((2l+1)/(4 pi) (l-|m|)!/(l+|m|)!)
// times the polynomial's own factor.
__device__ __forceinline__ void sh_basis(float dx, float dy, float dz, int deg, float* Y)
{
    const float inv = 1.0f / sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
    const float x = dx * inv, y = dy * inv, z = dz * inv;
    Y[0] = 0.28209479177387814f;  // 1 / (2 sqrt(pi))
    if (deg < 1) return;
    const float c1 = 0.48860251190291992f;  // sqrt(3 / (4 pi))
    Y[1] = -c1 * y;
    Y[2] = c1 * z;
    Y[3] = -c1 * x;
    if (deg < 2) return;
    const float xx = x * x, yy = y * y, zz = z * z;
    Y[4] = 1.0925484305920792f * (x * y);          // sqrt(15 / (4 pi))
    Y[5] = -1.0925484305920792f * (y * z);
    Y[6] = 0.31539156525252005f * (3.0f * zz - 1.0f);  // sqrt(5 / (16 pi))
    Y[7] = -1.0925484305920792f * (x * z);
    Y[8] = 0.54627421529603959f * (xx - yy);       // sqrt(15 / (16 pi))
    if (deg < 3) return;
    Y[9] = -0.59004358992664352f * (y * (3.0f * xx - yy));   // sqrt(35 / (32 pi))
    Y[10] = 2.8906114426405538f * (x * y * z);               // sqrt(105 / (4 pi))
    Y[11] = -0.45704579946446577f * (y * (5.0f * zz - 1.0f)); // sqrt(21 / (32 pi))
    Y[12] = 0.37317633259011540f * (z * (5.0f * zz - 3.0f));  // sqrt(7 / (16 pi))
    Y[13] = -0.45704579946446577f * (x * (5.0f * zz - 1.0f));
    Y[14] = 1.4453057213202769f * (z * (xx - yy));           // sqrt(105 / (16 pi))
    Y[15] = -0.59004358992664352f * (x * (xx - 3.0f * yy));
}

// Raw colour sum_j Y_j k[3 j + c] + 1/2 (before the clamp at 0).
__device__ __forceinline__ void sh_raw(const float* __restrict__ k, int deg, const float* Y, float* raw)
{
    const int nb = (deg + 1) * (deg + 1);
    raw[0] = raw[1] = raw[2] = 0.5f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if (j < nb) {
            raw[0] = fmaf(Y[j], k[3 * j], raw[0]);
            raw[1] = fmaf(Y[j], k[3 * j + 1], raw[1]);
            raw[2] = fmaf(Y[j], k[3 * j + 2], raw[2]);
        }
    }
}

__device__ __forceinline__ float safe_inv(float d)
{
    const float tiny = 1e-20f;
    float dd = fabsf(d) < tiny ? copysignf(tiny, d) : d;
    return 1.0f / dd;
}

__device__ __forceinline__ BoxRay box_ray(const Ray& r)
{
    BoxRay q;
    q.ix = 0.5f * safe_inv(r.dx), q.iy = 0.5f * safe_inv(r.dy), q.iz = 0.5f * safe_inv(r.dz);
    q.ox2 = 2.0f * r.ox, q.oy2 = 2.0f * r.oy, q.oz2 = 2.0f * r.oz;
    return q;
}

}  // namespace irgs
