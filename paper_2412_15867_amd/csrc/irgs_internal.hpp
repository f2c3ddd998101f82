// Host-side interfaces between the translation units of the HIP library.
#pragma once

#include <vector>

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "irgs_device.hpp"

namespace irgs {

struct BuildArgs {
    int n;
    const float* mu;
    const float* quat;
    const float* scale;
    const float* opac;
    float alpha_min;
    float sigma;
    uint32_t* order;        // leaf position -> surfel id
    uint64_t* sorted_keys;  // optional copy of the sorted Morton codes
    SurfelRec* rec;
    float* leafbox;         // 6 floats per leaf position
    BvhNode* nodes;
    int* leaf_parent;
    uint32_t* counters;     // unused by the level refit (kept for the buffer layout)
    int* level_nodes;       // internal node ids grouped by depth
    std::vector<int>* levels;  // host: level offsets into level_nodes (depth + 2 entries)
    std::vector<int>* wide_levels;  // host: first node of each level of the wide tree, then their number
    int2* brange;           // per binary node: first leaf, leaf count
    WideNode* wnodes;       // up to max(N - 1, 1) wide nodes
    int4* wsrc;             // per wide node and slot: (binary parent << 1 | side), -1 = empty
    int* wscratch;          // 3 * max(N - 1, 1) + 4 ints: collapse sources, level sizes and firsts
    int leaf_size;          // surfels per cluster leaf (1..16)
    bool ploc;              // binary tree by PLOC (else the Morton radix tree)
    int n_wide;             // out (host): wide nodes built; also the refit input
    int wide_depth;         // out (host): levels of the wide tree
    int max_depth;          // out (host): most internal ancestors of a leaf
};

hipError_t lbvh_sort_scratch_bytes(int n, size_t* bytes);
// Build: synchronises `st` (the clusters left and the levels' sizes are read back).
hipError_t lbvh_build(BuildArgs& a, void* scratch, hipStream_t st);
hipError_t lbvh_refit(const BuildArgs& a, hipStream_t st);
// The bounds of each leaf cluster's remaining records (k_cluster_slabs), which
// only the per-lane forward reads: records are built without them (no culls).
hipError_t lbvh_cluster_bounds(const BuildArgs& a, hipStream_t st);

struct OutPtrs {
    float* O;
    float* feat;
    float* D;
    float* T;
    int32_t* n_hits;
    int32_t* hit_ids;
    float* hit_T;
    int32_t H_cap;
    int32_t* counters;  // optional R x 4 work counters
};

struct GradIn {
    const float* gO;
    const float* gF;
    const float* gD;
};

struct GradOut {
    float* mu;
    float* quat;
    float* scale;
    float* opac;
    float* feat;
};

struct RawSurfels {
    const float* mu;
    const float* quat;
    const float* scale;
    const float* opac;
    const float* feat;
    // The backward's copy of the same parameters, one row of `ps` floats per
    // surfel id: (mu, o), q, (s_u, s_v, 1 / |q| in FP64), then the F features if they
    // fit one 128-byte line with these (F <= 20; a hit then reads that line
    // instead of five scattered ones); wider features stay in `feat`.  The
    // row's last four words hold 1 / s_u and 1 / s_v in FP64 where no feature
    // does (`recips`): an FP64 division or root per hit costs the walk over
    // the hits more than a row's few words.
    const float* pk;
    int ps;
    bool feat_packed, recips;
};

inline bool pack_features(int F) { return F <= 20; }
inline bool pack_recips(int F) { return F <= 16 || !pack_features(F); }
// Floats per packed row.
inline int pack_stride(int F) { return pack_features(F) ? 32 : 16; }
// Fill pk (n rows of raw.ps floats) from the raw arrays.
hipError_t pack_surfels(const RawSurfels& raw, int64_t n, int F, float* pk, hipStream_t st);

// Largest k-buffer / feature count the kernels are instantiated for.
constexpr int kMaxK = 64;
constexpr int kMaxF = 64;

// Upper bound on the persistent trace threads of a launch over R rays;
// scratch is sized per thread of this bound.
int64_t trace_threads(int64_t R);

// Blocks of `kern` (block_size threads each) that the whole device keeps
// resident at once, or 0 if the runtime cannot say.  Persistent launches use
// at most this many, so no block waits for another to finish.
template <class Kern>
int64_t resident_blocks(Kern kern, int block_size)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, block_size, 0) != hipSuccess) return 0;
    return per_cu > 0 && cus > 0 ? static_cast<int64_t>(per_cu) * cus : 0;
}

inline unsigned persistent_grid(int64_t max_blocks, int64_t resident)
{
    return static_cast<unsigned>(resident > 0 && resident < max_blocks ? resident : max_blocks);
}

// Device scratch of a persistent forward launch, sized for trace_threads(R)
// threads (the launch may use fewer).
constexpr int kDeferCap = 192;
// Deferred-list entries a lane stages in LDS before writing them as one
// group (kDeferCap and every fitted list size are multiples of it).
constexpr int kDeferStage = 8;
// Smallest deferred-list half a launch into a fixed scratch area takes
// before it gives up resident blocks instead.
constexpr int kDeferCapMin = 32;
struct FlatScratch {
    int* ovf;                      // stack overflow: ovf_slots ints per thread, or null when ovf_slots == 0
    int ovf_slots;
    int* dbuf;                     // deferred-work lists: 2 * defer_cap ints per thread (BVH launches)
    unsigned long long* next_ray;  // ray-claim counter (BVH launches); the launch zeroes it
    const uint32_t* order;         // optional claim order (slot -> ray), BVH launches over one scene
    int wide_depth;                // levels of the wide tree
    int defer_cap;                 // entries per half of a thread's deferred list
    // 0: ovf and dbuf are sized for trace_threads(R) threads at defer_cap.
    // Otherwise they share one area of this many ints (ovf first, dbuf
    // right after it, placed by the launch): the launch picks its grid and
    // the deferred-list size so that both fit (fewer resident blocks only
    // when even kDeferCapMin entries per half do not fit every one).
    size_t fixed_words;
};

// True when a launch into a fixed area of `words` ints can run at least one
// block (its threads' stack overflow and deferred-list halves of
// kDeferCapMin entries).
inline size_t fixed_scratch_block_words(int ovf_slots, int block)
{
    return static_cast<size_t>(block) * (ovf_slots + 2 * kDeferCapMin) + kDeferStage;  // + alignment of dbuf
}
inline bool fixed_scratch_fits(size_t words, int ovf_slots, int block)
{
    return words >= fixed_scratch_block_words(ovf_slots, block);
}

// Claim order of a forward trace: rays sorted by the Morton code of their
// origin in the scene's root box.  `buf` holds ray_sort_words(R) floats;
// *order points into it afterwards.  Needs R <= 2^31 - 1 and a built scene.
hipError_t ray_order_by_origin(const SceneView& sc, int64_t R, const float* ro, void* buf, const uint32_t** order,
                               hipStream_t st);

// True when a forward launch runs with one wave per ray (no per-thread scratch:
// only the claim counters); false for the plain tracer and the per-lane form
// (work counters asked for, or a wide tree deeper than the wave's stack takes).
bool use_wave_trace(bool bvh, bool counters, int wide_depth);
constexpr int kWaveClaimBytes = 1024;  // the claim counters of a wave launch
// True when a wave launch over R rays takes claim counters (more rays than
// waves fit the chip).
bool wave_claims(const TraceParams& P, int64_t R);

// Forward trace.  use_bvh = false tests every record (the plain tracer).
hipError_t launch_trace(const SceneView& sc, const TraceParams& P, int k, bool use_bvh, int64_t R,
                        const float* ro, const float* rd, const OutPtrs& out, const FlatScratch& fs,
                        hipStream_t st);

// True when the trace takes F features with a k-buffer of k (`special`: SH
// colour or normal channels).
bool features_offered(int k, int F, bool special);

// Backward over saved hit lists (ids and T).  Rays with n_hits > H_cap are
// traced again by a wave each, into a list in its LDS that the wave walks: a
// launch whose lists hold kRemarchShort hits, of which a CU keeps 12, and one
// for what it leaves with lists of kRemarchList hits, of which it keeps 8.
// Launches of at most kRemarchSmall rays take the second alone: there all lists
// can be cut, and twice the launches cost more than the waves.  Rays with more
// hits go to at most kRemarchLanes lanes.  With a tree too deep for the wave
// form all go to at most kRemarchLanesAll lanes (fewer where their stacks and
// lists take more than kRemarchLaneBytes), each with a list of kRemarchLaneList
// hits (4,000 rays with few hits each 7.5 -> 3.8 ms by the lists; 200,000 rays
// of 700 hits 936 -> 359 ms against 16,384 lanes).  Against lists in global
// memory and a wave per 64 rays to keep them small, all lists cut: 64 / 4,000
// rays of 1,500 hits 49.5 / 49.7 -> 0.9 / 1.9 ms, 1M rays of 44 hits 13.9 ->
// 13.8 ms (18.0 with the long lists alone); none cut, 262,144 rays: 1.29 ->
// 1.00 ms (68 MB less to allocate).
constexpr int kBwdCheckpoints = 16;
constexpr int kRemarchShort = 1024;
constexpr int kRemarchList = 2048;
constexpr int64_t kRemarchSmall = 32768;
constexpr int64_t kRemarchWaves = 4096;  // of a launch at most
constexpr int64_t kRemarchLanes = 16384;
constexpr int64_t kRemarchLanesAll = 131072;
constexpr int kRemarchLaneList = 512;
constexpr size_t kRemarchLaneBytes = size_t(1) << 30;
// Rays from which on the walk takes them in the order of where they land.
constexpr int64_t kSortWalkRays = 16384;
// Byte offsets in the backward's scratch: the interleaved per-surfel
// accumulator, then these.
struct BackwardPlan {
    size_t claims, rm_list, rest, sort, stacks, checkpoints, lists, bytes;
    bool short_lists, long_lists;  // wave launches over the cut lists
    int64_t lane_blocks;           // lanes' blocks of a launch over what is left (none: 0)
    int lane_list;                 // hits a lane's list holds
};
BackwardPlan plan_backward(int64_t R, int64_t N, int F, int wide_depth, int H_cap);
inline int grad_stride(int F) { return ((10 + F + 31) / 32) * 32; }
size_t sort_pairs_count_bytes(int n);
hipError_t sort_pairs(int n, uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1, uint32_t* counts, int passes,
                      hipStream_t st);
// Ray order of a launch: two key and two value buffers plus the sort's tile
// counters, in words; none for launches too large for 32-bit indices.
inline size_t ray_sort_words(int64_t R)
{
    if (R <= 0 || R > 0x7fffffffLL) return 0;
    return (static_cast<size_t>(R) * (2 * sizeof(uint64_t) + 2 * sizeof(uint32_t)) +
            sort_pairs_count_bytes(static_cast<int>(R))) / sizeof(float) + 64;
}
hipError_t launch_backward(const SceneView& sc, const RawSurfels& raw, const TraceParams& P, int k, int64_t R,
                           const float* ro, const float* rd, const OutPtrs& saved, const GradIn& gin,
                           const GradOut& gout, int wide_depth, char* scratch, hipStream_t st);

// Packed launch over work items of several scenes (serving).  Item i owns
// the slots [chunk_begin, chunk_begin + ray_count) of the concatenation of
// every item's rays.
struct WorkItem {
    int32_t scene;
    int32_t pad;
    int64_t ray_begin;
    int64_t ray_count;
    int64_t chunk_begin;
    const float* ro;
    const float* rd;
    OutPtrs out;
};

// counters: some item asks for work counters.
hipError_t launch_packed(const SceneView* scenes_dev, const WorkItem* items_dev, int n_items, int64_t n_rays,
                         const TraceParams& P, int k, const FlatScratch& fs, int grid_blocks, bool counters,
                         hipStream_t st);

// Monte Carlo rendering-equation consumer (shade.hip).
struct ShadeArgs {
    int64_t P;            // pixels
    int32_t N;            // samples per pixel
    int32_t E;            // cubemap face resolution
    const float* n;       // P x 3
    const float* wo;      // P x 3
    const float* albedo;  // P x 3
    const float* rough;   // P
    const float* wi;      // P x N x 3
    const float* O;       // P x N
    const float* Lind;    // P x N x 3
    const float* env;     // 6 x E x E x 3
    const float* wgt;     // P x N per-sample weights, or null: 2 pi / N each
};

struct ShadeGrads {
    float* albedo;  // P x 3, accumulated
    float* rough;   // P, accumulated
    float* env;     // 6 x E x E x 3, accumulated
    float* O;       // P x N, written
    float* Lind;    // P x N x 3, written
};

hipError_t launch_mc_rays(int64_t P, int St, int Sp, const float* x, const float* n, const float* u, float offset,
                          float* ro, float* rd, hipStream_t st);
hipError_t launch_mc_shade(const ShadeArgs& a, float* c, hipStream_t st);
hipError_t launch_mc_shade_backward(const ShadeArgs& a, const float* g_c, const ShadeGrads& g, hipStream_t st);

// Relighting variant (relight.hip).
struct RelightArgs {
    int64_t R;
    const float* O;      // R
    const float* Fo;     // R x 7: blended albedo (3), roughness, normal (3), all times O
    const float* rd;     // R x 3
    int32_t E, M, S;     // cube resolution, prefilter levels, table size
    const float* irr;    // 6 x E x E x 3
    const float* pref;   // M x 6 x E x E x 3
    const float* table;  // S x S x 2
};

hipError_t launch_env_prefilter(int E, const float* env, int M, float* irr, float* pref, hipStream_t st);
hipError_t launch_brdf_table(int S, float* table, hipStream_t st);
hipError_t launch_relight_lind(const RelightArgs& a, float* lind, hipStream_t st);

// Importance sampling of the sky by intensity (relight.hip).
struct EnvRayArgs {
    int64_t P;          // pixels
    int32_t N;          // samples per pixel
    int32_t E;          // cube resolution
    const float* x;     // P x 3 surface points
    const float* n;     // P x 3 unit normals
    const float* u;     // P x N x 3 uniforms in [0, 1)
    const float* cdf;   // 6 E^2 inclusive CDF of the texel weights
    float offset;       // origin offset along n
    float* ro;          // P N x 3
    float* rd;          // P N x 3
    float* wgt;         // P N estimator weights
};
hipError_t launch_env_cdf(int E, const float* env, float* cdf, hipStream_t st);
hipError_t launch_env_rays(const EnvRayArgs& a, hipStream_t st);

// Fill n 32-bit words with v (a kernel, so it can be captured in a graph).
hipError_t fill_u32(void* p, int64_t n, uint32_t v, hipStream_t st);

}  // namespace irgs
