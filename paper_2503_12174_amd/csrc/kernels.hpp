// kernels.hpp -- host-side entry points of the device kernels (one process, one device).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace dpcs {

// ------------------------------------------------------------------ BVH build
struct BvhInputs {
    const float* V;          // device vertices
    const int* F;            // device triangles
    const float* UV;         // device corner uvs
    const float* Le;         // device emission or null
    int nt;
    float lo[3], scale[3];   // centroid box origin and 1023 / extent
    float clo[3], chi[3];    // centroid box
    uint32_t* keys[2];
    uint32_t* vals[2];
    uint32_t* hist;          // 256 * ntiles
    int* child;              // 2 * (nt - 1)
    int* parent_int;         // nt - 1
    int* parent_leaf;        // nt
    int* flags;              // nt - 1, zeroed
    float* node_box;         // 6 * (nt - 1)
};
struct BvhOutputs {
    float4* nodes;           // 4 * max(nt - 1, 1)
    float4* tris;            // 4 * nt
    float4* emission;        // nt or null
    int* leaf_of_prim;       // nt
    const uint32_t* order;   // leaf -> original triangle (points into keys/vals scratch)
};
// The binary hierarchy with its bounds, then the leaf records.  LBVH: the radix tree over
// the Morton-sorted codes; PLOC: clustering over the Morton order (scratch of
// ploc_scratch_bytes); SAH: top-down binned SAH (scratch of sah_scratch_bytes).  PLOC reads
// one count per round into host_word[0..1].  child / parent_int / parent_leaf
// receive the topology (parent_int must hold -1 everywhere beforehand); out.order points
// into in.vals (LBVH, PLOC) or into the scratch (SAH).  SAH returns hipErrorNotSupported
// for a tree deeper than 64 levels.
enum class BvhBuild { LBVH, PLOC, SAH };
hipError_t build_bvh(hipStream_t st, const BvhInputs& in, BvhOutputs& out, BvhBuild kind = BvhBuild::LBVH,
                     void* scratch = nullptr, uint64_t* host_word = nullptr);
size_t ploc_scratch_bytes(int nt);
hipError_t build_ploc(hipStream_t st, const BvhInputs& in, const uint32_t* order, void* scratch, uint64_t* host_word,
                      float4* nodes);
size_t sah_scratch_bytes(int nt);
hipError_t build_sah(hipStream_t st, const BvhInputs& in, void* scratch, float4* nodes, const uint32_t** order_out);
// the 4-wide BVH of a binary one (nt >= 2) and the tree's checks, in scratch of
// wide_scratch_bytes(nt): result nodes4 (8 float4 per node) and map4 (4 ints per node)
// point into the scratch; the host reads one count per level into host_words (>= 2)
struct WideArgs {
    const float4* nodes;
    const int* parent_int;
    const int* parent_leaf;
    const uint32_t* order;
    int nt;
};
constexpr int MAX_LEVELS4 = 64;   // scenes are made of trees no deeper than that
struct WideResult {
    float4* nodes4;
    int* map4;
    int nnodes4, depth4;   // 4-wide nodes and levels
    int level_base[MAX_LEVELS4 + 1];   // first node of every level, and nnodes4
    int stack_bound;       // most stack entries a traversal holds
    int depth;             // binary depth (internal nodes on the longest root-to-leaf path)
    bool malformed;        // a leaf reached other than once, a parent chain off the root, or
                           // a leaf order that is not a permutation
};
size_t wide_scratch_bytes(int nt);
hipError_t build_wide(hipStream_t st, const WideArgs& a, void* scratch, uint64_t* host_words, WideResult& res);
// leaf-ordered triangle / emission records for a leaf order built elsewhere
hipError_t build_leaf_records(hipStream_t st, const BvhInputs& in, const uint32_t* order, BvhOutputs& out);
// new vertex positions on a fixed topology: the leaf records' vertices and the boxes of the
// binary nodes and of the 4-wide nodes, from map4 (4 per node: binary node, ~leaf, or
// INT_MIN empty) and the first node of every 4-wide level (level_base, nlevels + 1 entries).
// Without a 4-wide tree (nodes4 null) the binary boxes are climbed to with flags (ni zeroed
// ints) and node_box (6 ni floats of scratch), which are not used otherwise.
struct RefitArgs {
    const float* V;
    const int* F;
    const uint32_t* order;
    const int* child;
    const int* parent_int;
    const int* parent_leaf;
    int* flags;
    float* node_box;
    int nt;
    float4* nodes;
    float4* tris;
    float4* nodes4;
    const int* map4;
    int nnodes4;
};
hipError_t refit_bvh(hipStream_t st, const RefitArgs& a, const int* level_base, int nlevels);

// ------------------------------------------------------------------ path queues
// Structure-of-arrays queues in HBM.  Path state is FP64 position/direction (PathO,
// PathD, 32 B each) plus FP32 throughput; shadow rays only need a visibility
// decision and are FP32 (16-byte float4 fields: a wave64 touches 1 KiB per field).
struct Queues {
    PathO* po[2];      // path ray origin, slot, triangle left
    PathD* pd[2];      // path ray direction, global sample index g
    float4* pb[2];     // path throughput beta (rgb, -)
    int* hit;          // leaf-order triangle hit by the current queue (-1: escaped)
    float4* so[2];     // shadow ray origin (w: slot); [0] projector, [1] environment
    float4* sd[2];     // shadow direction (w: triangle the ray leaves)
    float4* sc[2];     // shadow contribution (w: batch sample index)
    float* st[2];      // shadow tmax
    float4* L;         // per batch sample radiance (rgb, -)
    uint32_t* cnt;     // [0], [1] path queue sizes, [4..6] the replay's path queue sizes (by
                       // depth mod 3), [8..11] shadow queue sizes (shadow_slot)
    int64_t cap;       // path capacity
    unsigned long long* stats;   // null, or [0] nodes visited, [1] triangles tested (profiling)
    int* spill;        // traversal stack overflow: SPILL ints per thread of a capped grid
    int trace_blocks;  // workgroups the spill region covers: the traversal grid cap
};

constexpr int SHORT_STACK = 8;                 // LDS stack entries per thread
constexpr int SPILL = 64 - SHORT_STACK;        // overflow entries per thread
constexpr int TRACE_TB = 128;                  // threads per workgroup of the traversal kernels
// traversal kernels are compiled for 8 waves per SIMD (at most 64 VGPRs): the loop is
// latency-bound enough that occupancy pays more than the odd spilled register costs
#define TRAVERSAL_OCCUPANCY __attribute__((amdgpu_waves_per_eu(8, 8)))
// except the forward's shadow rays: with the staged tree top their any-hit loop spills a
// few registers at 64 VGPRs; at 7 waves (72 VGPRs, 8 to 12 bytes spilled) they run ~3 % faster
#define SHADOW_OCCUPANCY __attribute__((amdgpu_waves_per_eu(7, 7)))
// and the re-tracing replay's shadow rays, whose gradient bookkeeping after the query
// spilled ~150 bytes per lane at 64 VGPRs: at 4 waves (105 VGPRs) nothing spills and
// the re-tracing step is ~1.5 % faster
#define ADJ_SHADOW_OCCUPANCY __attribute__((amdgpu_waves_per_eu(4, 4)))
constexpr int PATH_TB = 64;   // threads per workgroup of the whole-path kernel
// Waves of up to SMALL_PATHS paths run a whole path per thread (k_paths), larger ones queues and
// three launches per depth: those gather the paths that go on into full waves at 8 waves per
// SIMD; k_paths has 4 and loses the lanes whose path ended, but no launch waits for the one
// before.  Renders by queues and by k_paths, us, corner of 50k triangles at 16 k, 0.33 M and 0.66 M
// paths: depth 1 62 and 47, 96 and 73, 117 and 101; depth 2 153 and 94, 225 and 158, 287 and 246;
// depth 4 307 and 167, 402 and 269, 480 and 421; beyond, depth 4, 640 x 360 x 4 (0.92 M) 581 and
// 589, 256 x 256 x 16 598 and 675; of 200k, depth 6, lit room, 317 x 203 x 9 (0.58 M) 1086 and 829.
// A tree of a few nodes (less than TOP_NODES) has little to gather: the quad and cube at 16 k and
// 0.98 M, depth 1 38 and 25, 92 and 62; depth 4 108 and 47, 276 and 144.
constexpr int64_t SMALL_PATHS = 5 << 17, SMALL_PATHS_TINY = 1 << 20;
// Traversal grids are capped at `rounds` x grid_cap x 128 threads (grid_cap x 128 threads
// is one resident round at 8 waves per SIMD); the spill region holds SPILL ints for every
// thread of that grid.  Several rounds let workgroups that finish early be replaced
// while others still trace long paths (4 rounds: traversal -7 %), at 224 B of spill
// space per thread (never more threads than paths of a wave in the request loop, whose
// queues count against its memory budget).
constexpr int TRACE_ROUNDS = 4;
inline int trace_grid_cap(int grid_cap, int rounds) {
    const int g = grid_cap * 128 / TRACE_TB * rounds;
    return g > 0 ? g : 1;
}
inline size_t spill_ints(int grid_cap, int rounds) { return (size_t)trace_grid_cap(grid_cap, rounds) * TRACE_TB * SPILL; }

// Binned accumulation of the cotangent of one texel map (BRDF maps or E_p): the replay
// writes one record per (vertex, map) -- bilinear base texel and offsets plus the C
// cotangent values -- instead of 4 x C global atomics; a flush groups the records by
// T x T texel tile (counting sort), accumulates every tile in LDS and adds the tiles
// into the map with plain stores.
constexpr int MAP_MAX_BINS = 4096;
constexpr int MAP_MAX_T = 16;   // tile side 8 or 16: maps up to 1024 x 1024 are binned
constexpr int BIN_DEPTHS = 4;   // replay depths between flushes (record capacity follows)
constexpr int ACC_CHUNK = 4096; // most records of one tile a workgroup of the accumulation sums
                                // at once (a unit); the stage holds one block of (T + 1)^2 x C
                                // sums per unit
constexpr int ACC_TB = 1024;    // threads per workgroup of the accumulation
constexpr int BIN_CHUNK = 4096; // records per workgroup of the histogram and the placement, at
constexpr int BIN_CHUNK_MIN = 1024;   // most and at least (bin_chunk)
constexpr int BIN_BLOCKS = 2048;      // workgroups they are spread over before chunks grow
constexpr int BIN_TB = 1024;    // their threads per workgroup: 16 waves share one LDS histogram
constexpr int BIN_U = 4;        // records a thread of the placement loads at once
static_assert(BIN_CHUNK % (BIN_TB * BIN_U) == 0, "placement chunking");
constexpr long long STAGE_NAN = -0x7fffffffffffffffll - 1;   // INT64_MIN
struct MapBins {
    float* rec;          // records of rs floats (null: binning off, the replay scatters directly)
    float* sorted;       // the same records grouped by tile
    long long* stage;    // per unit (T + 1)^2 x C exact fixed-point sums (tile plus one halo
                         // row/column); STAGE_NAN marks a unit with a non-finite value
    uint32_t* count;     // records appended since the last flush (may exceed cap)
    uint32_t* bins;      // counts[nb], offsets[nb + 1], first units[nb + 1], fixed-point exponent
                         // E, largest |value| (float bits): map_bin_words(nb)
    uint32_t* unit_tile; // tile of every unit
    uint32_t* rowbase;   // per (chunk, tile): where the chunk's records start in the tile
    int64_t cap;         // record capacity
    int64_t fill;        // most records before the next flush (<= cap)
    int chunk;           // records per workgroup of the histogram and the placement
    int W, H, T, nbx, nby, nb;
};

// Records per workgroup of a flush of at most `fill` records.  A larger chunk has fewer global
// atomics and rows per record, a smaller one more workgroups and waves in flight.  Histogram +
// placement, by chunk: 64 x 64 x 32 (fill 0.4 M) 27 + 24 us at 16384, 11 + 10 at 4096, 6 + 6 at
// 1024; 256 x 256 x 16 (4.2 M) 19 + 21 at 2048, 28 + 23 at 1024; 256 x 256 x 64 (16.8 M) 51 + 126
// at 16384, 53 + 83 at 4096, 62 + 82 at 2048, 102 + 106 at 1024.
constexpr int bin_chunk(int64_t fill) {
    int c = BIN_CHUNK_MIN;
    while (c < BIN_CHUNK && fill > (int64_t)c * BIN_BLOCKS) c *= 2;
    return c;
}
constexpr int64_t bin_chunks(int64_t fill, int chunk) { return (fill + chunk - 1) / chunk; }

constexpr int64_t map_bin_words(int64_t nb) { return 3 * nb + 4; }
// most units of cap records in nb tiles
constexpr int64_t map_units(int64_t cap, int64_t nb) { return (cap + ACC_CHUNK - 1) / ACC_CHUNK + nb; }

// adjoint additions (see adjoint.hip)
struct AdjQueues {
    float4* rl[2];     // remaining radiance L_r of the path (rgb, -), follows the path queue
    float4* delta;     // re-tracing replay: per batch sample cotangent of its radiance (rgb, -);
                       // record replay: the pixel's, at its first sample
    // the re-tracing replay's shadow rays and pending bounces (null for the record replay)
    double2* sproj[2]; // shadow: projector pixel position (pu, pv) of the vertex
    double2* suv[2];   // shadow: texture coordinate (u, v) of the vertex (FP64: 1k+ maps)
    float4* sg[2];     // shadow: E_p cotangent weight per channel (w: -)
    float4* sa[2];     // shadow: albedo cotangent rgb (w: roughness cotangent)
    float* ss[2];      // shadow: specular cotangent
    double2* puv[2];   // pending bounce: texture coordinate (u, v) of the previous vertex
    float2* pend[2];   // pending bounce: (dr, dsp) cotangent scale of the previous vertex
    float4* penda[2];  // pending bounce: albedo cotangent scale rgb
    MapBins tb;        // BRDF-map cotangent records (C = 5, 8 floats per record; C = 9, 12 floats
                       // with the metallic and normal maps)
    MapBins eb;        // E_p cotangent records (C = 3, 6 floats per record)
};

constexpr int REPLAY_CNT = 4;   // first of the replay's three queue-size slots in Queues::cnt
// The shadow queues' sizes alternate by depth parity: shading at depth d appends to
// q.cnt[shadow_slot(d & 1, which)] (every depth loop starts with cur = 0, so d & 1 = cur),
// so the closest-hit launch of depth d + 1, which empties the slots shading at d + 1
// appends to, leaves intact the sizes that depth d's shadow launch reads (the two may
// run at the same time on two streams).
constexpr int SHADOW_CNT = 8;
// Launch waves of fewer paths keep their shadow rays on the main stream: their launches
// take a few microseconds, less than the two cross-stream waits per depth cost.
constexpr int64_t SIDE_MIN_PATHS = int64_t(1) << 17;
constexpr int64_t LOOP_SIDE_MIN_PATHS = int64_t(1) << 21;   // the same for the request loop's waves
__host__ __device__ constexpr int shadow_slot(int parity, int which) { return SHADOW_CNT + 2 * parity + which; }
struct Launch {
    hipStream_t st;
    int grid_cap;      // upper bound on workgroups of grid-stride kernels
};

// forward kernels; `uni` is the request descriptor when every path of the launch
// belongs to one request (table == null), else descriptors are read from `table`.
// what a render reads besides the scene, in one launch: E_p and the packed maps (tex4b:
// null without metallic and normal maps)
void launch_prepare(const Launch& l, const ReqDesc& r, float4* Ep, const float* albedo, const float* rough, float4* tex4,
                    const float* nmap = nullptr, const float* metal = nullptr, float4* tex4b = nullptr);
void launch_set_count(const Launch& l, uint32_t* cnt, int idx, uint32_t value, int zero_from, int zero_to);
// The request loop's per-request launches, for all segments of a wave at once: a segment is
// pixels [p0, p1) of the request in descriptor slot `slot` (table[slot], at spp samples a
// pixel).  Each is a few microseconds on a few hundred workgroups, most of it the launch itself
// (4,096 pixels of 32 samples: camera rays 6 us, finalize 8, pixel backward 11, finish 8 + 3), so a
// list of up to WAVE_SEGS segments shares one: workgroup b belongs to the last segment
// whose first[] is not beyond it.  A step of 8 such pairs, in three waves: 1492 us a request at a
// time, 1305 us so.
constexpr int WAVE_SEGS = 16;
struct WaveSeg {
    int32_t slot;
    uint32_t p0, p1;
    int32_t spp;
};
struct SegList {
    int32_t n;
    int32_t slot[WAVE_SEGS];
    uint32_t p0[WAVE_SEGS], p1[WAVE_SEGS], first[WAVE_SEGS];
};
// Runs go(list, workgroups) for the segments in lists of at most WAVE_SEGS; blocks(segment) is
// the number of workgroups a segment takes (0: none, left out).
template <class BLOCKS, class GO>
void for_seg_lists(const WaveSeg* segs, int n, BLOCKS blocks, GO go) {
    SegList a{};
    uint32_t g = 0;
    for (int k = 0; k < n; ++k) {
        const uint32_t b = blocks(segs[k]);
        if (b == 0) continue;
        if (a.n == WAVE_SEGS) {
            go(a, g);
            a.n = 0;
            g = 0;
        }
        a.slot[a.n] = segs[k].slot;
        a.p0[a.n] = segs[k].p0;
        a.p1[a.n] = segs[k].p1;
        a.first[a.n++] = g;
        g += b;
    }
    if (a.n > 0) go(a, g);
}
// the segment of a workgroup
template <class LIST>
__host__ __device__ inline int seg_of(const LIST& a, uint32_t block) {
    int k = 0;
    for (int j = 1; j < a.n; ++j) k += block >= a.first[j] ? 1 : 0;
    return k;
}
void launch_raygen(const Launch& l, const Queues& q, const ReqDesc* table, const WaveSeg* segs, int n);
// The rays of one launch are on one tree: r's (uni's; requests that share a wave are of one scene).
// cam (one request, no table): the queue is the request's camera rays, generated by the
// closest-hit and shading kernels themselves (no raygen launch, no path state read)
void launch_trace(const Launch& l, const Queues& q, int cur, const ReqDesc& r, int64_t n_upper, bool cam = false);
void launch_shade(const Launch& l, const Queues& q, int cur, int depth, const ReqDesc& uni, const ReqDesc* table,
                  int64_t n_upper, bool cam = false);
// depth: the bounce the shadow rays leave from (for the path records)
void launch_shadow(const Launch& l, const Queues& q, int which, const ReqDesc& uni, const ReqDesc* table,
                   int64_t n_upper, int depth);
// the whole forward of a small wave: n rays of one request, its camera's (cam) or those in the
// path queue; or the camera rays of several requests' segments (no metallic and normal maps).
// small_wave: where that pays, and the spill region holds n threads (segments: a workgroup's
// threads more for each).
void launch_paths(const Launch& l, const Queues& q, const ReqDesc& r, uint32_t n, bool cam);
void launch_paths(const Launch& l, const Queues& q, const ReqDesc* table, const WaveSeg* segs, int n);
bool small_wave(const Queues& q, const ReqDesc& r, int64_t n);
void launch_finalize(const Launch& l, const Queues& q, const ReqDesc& r, uint32_t p0, uint32_t p1);
void launch_finalize(const Launch& l, const Queues& q, const ReqDesc* table, const WaveSeg* segs, int n);
// table[slot[k]] = *r[k], k < n: up to DESC_BATCH descriptors as the arguments of one launch
constexpr int DESC_BATCH = 4;
void launch_set_desc(const Launch& l, ReqDesc* table, const int* slot, const ReqDesc* const* r, int n);

// adjoint kernels
// floats of the scalar-partials buffer (ReqDesc::d_part) for waves of up to
// pixels_per_wave pixels and a projector of proj_pixels pixels
size_t partial_floats(int64_t pixels_per_wave, int64_t proj_pixels);
// pix_dE (optional): per-pixel cotangent of the clipped pixel mean (rgb, -), whole image;
// per_sample: for the re-tracing replay (the record replay and the camera-pose gradient
// take the samples' radiance from sample_L, or q.L if null, themselves)
void launch_adj_pixel(const Launch& l, const Queues& q, const AdjQueues& aq, const ReqDesc& r, uint32_t p0,
                      uint32_t p1, const float* sample_L, float4* pix_dE, bool per_sample);
// (several requests: their scalar cotangents go to d_acc by atomics, so d_part has to be null)
void launch_adj_pixel(const Launch& l, const Queues& q, const AdjQueues& aq, const ReqDesc* table, const WaveSeg* segs,
                      int n, bool per_sample);
void launch_adj_raygen(const Launch& l, const Queues& q, const AdjQueues& aq, const ReqDesc& r, int slot, uint32_t g0,
                       uint32_t n);
void launch_adj_shade(const Launch& l, const Queues& q, const AdjQueues& aq, int cur, int depth, const ReqDesc& uni,
                      const ReqDesc* table, int64_t n_upper);
void launch_adj_shadow(const Launch& l, const Queues& q, const AdjQueues& aq, int which, int nxt, const ReqDesc& uni,
                       const ReqDesc* table, int64_t n_upper);
// replay of one bounce from the path records (no tracing): shade, next-event gradients
// for the recorded visibilities, bounce; sample_L (one request): the samples' radiance,
// null: q.L holds it
void launch_adj_replay(const Launch& l, const Queues& q, const AdjQueues& aq, int cur, int depth, const ReqDesc& uni,
                       const ReqDesc* table, int64_t n_upper, const float* sample_L = nullptr);
// The whole replay of a small wave from its records (small_replay: where that pays, and the bins
// hold every depth's records).  VJP from records by depth and whole, us, 4 k and 131 k samples:
// corner of 50k triangles, depth 1 93 and 92, 98 and 96; depth 2 108 and 104, 116 and 112; depth 4
// 127 and 123, 141 and 130; quad and cube, depth 1 69 and 68, 77 and 77; depth 4 98 and 90, 111 and
// 96.  Beyond, forward and VJP: quad and cube, 256 x 256 x 16 390 and 473; corner, 256 x 256 x 4 375
// and 389.
constexpr int64_t SMALL_REPLAY = 1 << 17;
bool small_replay(const AdjQueues& aq, const ReqDesc& r, int64_t n);
// The same for up to JOINT_SEGS requests of the loop at once, each with bins of its own, and the
// flush of all their maps (5-channel maps): six launches for the list instead of six per
// request, which fill the chip together (a request of 2^17 paths alone: replay 27 us on 512
// workgroups, flush 32; a step of 8 of them 1360 -> 1176 us).  Per launch, workgroups first[k] on belong to request k;
// na[k] of them to its texture map (accumulation: the number that takes its units in turn).
constexpr int JOINT_SEGS = 8;
struct JointList {
    int32_t n;
    int32_t slot[JOINT_SEGS];
    uint32_t paths[JOINT_SEGS], first[JOINT_SEGS], na[JOINT_SEGS];
    MapBins tb[JOINT_SEGS], eb[JOINT_SEGS];
    float *d_tex[JOINT_SEGS], *d_ep[JOINT_SEGS];
};
void launch_replay_joint(const Launch& l, const Queues& q, float4* delta, const ReqDesc* table, JointList& f);
void launch_replay_paths(const Launch& l, const Queues& q, const AdjQueues& aq, const ReqDesc& r, uint32_t n,
                         const float* sample_L = nullptr);
// adds the binned records of tb / eb into r.d_tex / r.dEp and empties the bins
void launch_map_flush(const Launch& l, const AdjQueues& aq, const ReqDesc& r);
// tile side and bin count for a W x H map (false: too many tiles, bin nothing)
bool map_tiling(int W, int H, int& T, int& nbx, int& nby);
// PRF backward, map de-interleave and scalar gradients; acc: 20 floats (see adjoint.hip)
// camera-pose gradient of a wave's camera samples (after launch_adj_pixel, with path
// records): per-workgroup partials into r.d_cam_part (cam_partial_floats of the wave's
// samples), summed in a fixed order into r.d_acc[20..32)
size_t cam_partial_floats(int64_t samples_per_wave);
void launch_cam_grad(const Launch& l, const Queues& q, const AdjQueues& aq, const ReqDesc& r, uint32_t p0, uint32_t p1,
                     const float* sample_L);
// dst[k] += the sum of nb partials part[b * stride + k], k < nv, in a fixed order
void launch_sum_partials(const Launch& l, const float* part, int nb, int stride, int nv, float* dst);
void launch_adj_finish(const Launch& l, const ReqDesc& r, float* d_proj, float* d_albedo, float* d_rough,
                       float* d_spec, float* d_scalars, float* acc, float* d_metal = nullptr,
                       float* d_nmap = nullptr);
// the same for several requests of the loop (5-channel maps, d_part null)
struct FinishSeg {
    int32_t slot;
    int64_t ep_pixels, map_texels;
    float *d_proj, *d_albedo, *d_rough, *d_spec, *d_scalars;
};
void launch_adj_finish(const Launch& l, const ReqDesc* table, const FinishSeg* segs, int n);
void launch_zero(const Launch& l, float* p, int64_t n);
// Float buffers cleared together by one launch on l's stream: add() collects them (a
// full list is cleared at once and started again), launch() clears what is held.
constexpr int ZERO_LIST_MAX = 8;
struct ZeroArgs {
    float* p[ZERO_LIST_MAX];
    int64_t n[ZERO_LIST_MAX];
};
struct ZeroList {
    explicit ZeroList(const Launch& l) : l(l) {}
    void add(float* ptr, int64_t count);
    void launch();
    Launch l;
    ZeroArgs a{};
    int k = 0;
};

// debug
void launch_debug_intersect(const Launch& l, const float4* nodes4, const float4* nodes, const float4* tris,
                            const int* leaf_of_prim, int nt, float tmin, const float* rays, int64_t n, int mode,
                            int32_t* prim, float* t, float* b1, float* b2);
void launch_debug_brdf(const Launch& l, int kind, const double* in, int64_t n, double* out);
// guide features through the pixel centres (out: Wc x Hc x 8 floats, 16-byte aligned)
void launch_gbuffer(const Launch& l, const ReqDesc& r, const float* albedo, float* out);
void launch_debug_philox(const Launch& l, uint64_t seed, const uint32_t* ctr, int64_t n, uint32_t* out);

}  // namespace dpcs
