// bvh_sah.hip -- device construction of the binary BVH by binned surface-area heuristic,
// top down.
//
// A task is a range [a, b) of the leaf order holding >= 2 triangles, with the box of
// their centroids.  Its triangles are binned by centroid into SAH_BINS bins along every
// axis with a non-zero centroid extent, and the split minimising
// area(left) x count(left) + area(right) x count(right) is taken (ties to the lower axis
// and bin).  A task whose centroids coincide is split at the middle of its range.  The
// range is then partitioned stably (left side first, order kept), and the task's node is
// written with both child boxes; children of >= 2 triangles become tasks, single triangles
// are leaves (leaf l is triangle order[l]).
//
// Nodes are numbered in preorder: the subtree over n triangles takes n - 1 numbers, so the
// children of node i with nl triangles on the left are i + 1 and i + nl, known without any
// count over the level, and the tree does not depend on scheduling.
//
// Three sizes of task, by what bounds them:
//   large   more than SAH_CHUNK triangles: breadth first, cut into chunks of SAH_CHUNK, one
//           workgroup each, whose bins are merged with global atomics (launches and the
//           atomics of neighbouring triangles that share a bin bound these levels);
//   medium  one workgroup splits it in LDS, in the same rounds;
//   small   at most SAH_SMALL triangles: one wave builds the whole subtree, a triangle per
//           lane, every node of a level at once (k_sah_small).  Split one workgroup per
//           node like the medium ones, these levels -- most of the nodes -- were nearly all
//           of the build: 200k triangles 13.8 ms, now 2.0 (10k: 2.7, now 1.0; 500k: 31, now 3.2).
// Boxes are accumulated as order-preserving integer images of the floats (exact min / max).
#include <algorithm>
#include <cfloat>
#include <climits>
#include <cstring>

#include "kernels.hpp"
#include "prefix.hpp"

namespace dpcs {

namespace {

constexpr int SAH_BINS = 32;
constexpr int SAH_CHUNK = 1024;
constexpr int SAH_SMALL = 64;   // one triangle per lane of a wave
constexpr int TB = SCAN_TB;     // threads of the chunk kernels
constexpr int PER = SAH_CHUNK / TB;
constexpr int BIN_INTS = 7;   // count, lo.xyz, hi.xyz
constexpr int LARGE_BIN_INTS = 3 * SAH_BINS * BIN_INTS;
constexpr int MAX_LEVELS = 64;

struct SahTask {
    int a, b, node;
    int c0;       // first chunk of the task in this level's chunk list
    int cb[6];    // centroid box (lo.xyz, hi.xyz), order-preserving integers
    int large;    // index among this level's large tasks, or -1
    int pad;
};
struct SahSmall {
    int a, b, node, buf;   // buf: which of the two order buffers holds the range
};
struct SahRes {        // split of a large task
    int axis, split;   // axis -1: coincident centroids, split at the middle of the range
    int nleft;
    int box[2][12];    // per child: box lo.xyz hi.xyz, centroid box lo.xyz hi.xyz (integers)
    int pad;
};
// counters of one level's lists
struct SahCount {
    int tasks, chunks, large, pad;
};
// what the splitting kernels append children to
struct SahNext {
    SahTask* tasks;
    int2* chunks;       // (task, first index) of every chunk
    int* large_task;    // task of every large index
    SahCount* count;
    SahSmall* small;
    int* small_count;
    int tcap, ccap, lcap, scap;
    int buf;            // order buffer this level's partitions are written to
    int* bad;
};

__device__ __forceinline__ int fenc(float f) {
    const int b = __float_as_int(f);
    return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float fdec(int i) { return __int_as_float(i ^ ((i >> 31) & 0x7fffffff)); }

__device__ __forceinline__ void box_init(int* b, int n6) {
    for (int k = 0; k < n6; ++k) {
        b[6 * k + 0] = b[6 * k + 1] = b[6 * k + 2] = fenc(FLT_MAX);
        b[6 * k + 3] = b[6 * k + 4] = b[6 * k + 5] = fenc(-FLT_MAX);
    }
}

__device__ __forceinline__ double box_area(const float* lo, const float* hi) {
    const double dx = fmax(0.0, (double)hi[0] - lo[0]), dy = fmax(0.0, (double)hi[1] - lo[1]),
                 dz = fmax(0.0, (double)hi[2] - lo[2]);
    return dx * dy + dy * dz + dz * dx;
}
__device__ __forceinline__ double enc_area(const int* b) {
    const float lo[3] = {fdec(b[0]), fdec(b[1]), fdec(b[2])}, hi[3] = {fdec(b[3]), fdec(b[4]), fdec(b[5])};
    return box_area(lo, hi);
}

// the bin of a centroid coordinate: floor((c - lo) * SAH_BINS / extent), clamped
__device__ __forceinline__ int sah_bin(float c, float lo, double sc) {
    return max(0, min(SAH_BINS - 1, (int)(((double)c - (double)lo) * sc)));
}

struct Tri {
    float lo[3], hi[3], c[3];
};
__device__ __forceinline__ Tri load_tri(const float4* __restrict__ tb, uint32_t p) {
    const float4 a = tb[3 * (size_t)p], b = tb[3 * (size_t)p + 1], c = tb[3 * (size_t)p + 2];
    return Tri{{a.x, a.y, a.z}, {b.x, b.y, b.z}, {c.x, c.y, c.z}};
}

// left side of the task's split?
__device__ __forceinline__ bool goes_left(const SahTask& t, int axis, int split, const Tri& x, int i) {
    if (axis < 0) return i < t.a + (t.b - t.a) / 2;
    const float lo = fdec(t.cb[axis]), hi = fdec(t.cb[3 + axis]);
    const double sc = SAH_BINS / ((double)hi - lo);
    return sah_bin(x.c[axis], lo, sc) < split;
}

// (cost, axis, split) of the better split: lower cost, then lower axis, then lower bin;
// cost < 0: no split
struct SahBest {
    double cost;
    int key;   // axis * SAH_BINS + split
};
__device__ __forceinline__ SahBest better(SahBest a, SahBest b) {
    const bool tb = b.cost >= 0.0 && (a.cost < 0.0 || b.cost < a.cost || (b.cost == a.cost && b.key < a.key));
    return tb ? b : a;
}

// best split of binned counts / boxes (bins[axis][bin][7]): one candidate (axis, first bin
// of the right side) per thread of the workgroup's first 96, then a reduction; every thread
// must call, all receive the result (key -1: none).  A side without triangles or an axis
// without centroid extent is no split.
__device__ __forceinline__ int sah_best(const int* bins, const int* cb, SahBest* red) {
    SahBest me{-1.0, -1};
    const int q = threadIdx.x;
    if (q < 3 * SAH_BINS) {
        const int ax = q / SAH_BINS, s = q % SAH_BINS;
        if (s > 0 && (double)fdec(cb[3 + ax]) - fdec(cb[ax]) > 0.0) {
            const int* B = bins + ax * SAH_BINS * BIN_INTS;
            int acc[2][6], n[2] = {0, 0};
            box_init(acc[0], 1);
            box_init(acc[1], 1);
            auto take = [&](int side, const int* b) {
                n[side] += b[0];
                for (int k = 0; k < 3; ++k) {
                    acc[side][k] = min(acc[side][k], b[1 + k]);
                    acc[side][3 + k] = max(acc[side][3 + k], b[4 + k]);
                }
            };
            for (int k = 0; k < s; ++k) take(0, B + k * BIN_INTS);
            for (int k = s; k < SAH_BINS; ++k) take(1, B + k * BIN_INTS);
            if (n[0] > 0 && n[1] > 0) me = SahBest{enc_area(acc[0]) * n[0] + enc_area(acc[1]) * n[1], q};
        }
    }
    if (q < 128) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            SahBest x;
            x.cost = __shfl_xor(me.cost, o);
            x.key = __shfl_xor(me.key, o);
            me = better(me, x);
        }
        if ((q & 63) == 0) red[q >> 6] = me;
    }
    __syncthreads();
    me = better(red[0], red[1]);
    __syncthreads();   // (red may be reused)
    return me.key;
}

// one thread: the child range [a, b) as a task of the next level (or of the small list);
// cb: its centroid box
__device__ __forceinline__ void push_task(const SahNext& nx, int a, int b, int node, const int* cb) {
    const int n = b - a;
    if (n <= SAH_SMALL) {
        const int s = atomicAdd(nx.small_count, 1);
        if (s >= nx.scap) atomicExch(nx.bad, 1);
        else nx.small[s] = SahSmall{a, b, node, nx.buf};
        return;
    }
    const int nc = (n + SAH_CHUNK - 1) / SAH_CHUNK;
    const int t = atomicAdd(&nx.count->tasks, 1), c0 = atomicAdd(&nx.count->chunks, nc);
    const int li = nc > 1 ? atomicAdd(&nx.count->large, 1) : -1;
    if (t >= nx.tcap || c0 + nc > nx.ccap || li >= nx.lcap) {
        atomicExch(nx.bad, 1);
        return;
    }
    SahTask k;
    k.a = a;
    k.b = b;
    k.node = node;
    k.c0 = c0;
    for (int q = 0; q < 6; ++q) k.cb[q] = cb[q];
    k.large = li;
    k.pad = 0;
    nx.tasks[t] = k;
    if (li >= 0) nx.large_task[li] = t;
    for (int c = 0; c < nc; ++c) nx.chunks[c0 + c] = make_int2(t, a + c * SAH_CHUNK);
}

// where the tree goes
struct SahTree {
    float4* nodes;
    int* child;
    int* parent_int;
    int* parent_leaf;
    int nt;
};
// the record of node `node` over [a, b) split at a + nl, its children's boxes (lo, hi) given
__device__ __forceinline__ void write_node(const SahTree& T, int a, int b, int node, int nl, const float* b0,
                                           const float* b1) {
    const int mid = a + nl;
    const int r0 = nl == 1 ? ~a : node + 1, r1 = b - mid == 1 ? ~mid : node + nl;
    T.nodes[4 * (size_t)node] = make_float4(b0[0], b0[1], b0[2], b0[3]);
    T.nodes[4 * (size_t)node + 1] = make_float4(b0[4], b0[5], b1[0], b1[1]);
    T.nodes[4 * (size_t)node + 2] = make_float4(b1[2], b1[3], b1[4], b1[5]);
    T.nodes[4 * (size_t)node + 3] = make_float4(__int_as_float(r0), __int_as_float(r1), 0.f, 0.f);
    T.child[2 * (size_t)node] = r0;
    T.child[2 * (size_t)node + 1] = r1;
    if (r0 < 0) T.parent_leaf[a] = node;
    else T.parent_int[r0] = node;
    if (r1 < 0) T.parent_leaf[mid] = node;
    else T.parent_int[r1] = node;
}
// one thread: the node of task t and its children as tasks.  box[child]: the child's box,
// then its centroid box (integers)
__device__ __forceinline__ void emit(const SahTree& T, const SahNext& nx, const SahTask& t, int nl,
                                     const int (*box)[12]) {
    const int mid = t.a + nl;
    if (nl < 1 || mid >= t.b || t.node < 0 || t.node >= T.nt - 1) {   // never: both sides hold a triangle
        atomicExch(nx.bad, 1);
        return;
    }
    float b[2][6];
    for (int j = 0; j < 2; ++j)
        for (int q = 0; q < 6; ++q) b[j][q] = fdec(box[j][q]);
    write_node(T, t.a, t.b, t.node, nl, b[0], b[1]);
    // (a single triangle goes to the small list too: its leaf order entry is written there)
    push_task(nx, t.a, mid, t.node + 1, box[0] + 6);
    push_task(nx, mid, t.b, t.node + nl, box[1] + 6);
}

// child boxes of a chunk: every thread's own in registers, one set of LDS atomics per wave
__device__ __forceinline__ void child_boxes(int (*mine)[12], int (*cbox)[12]) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 12; ++q) {
            int v = mine[j][q];
            const bool lo = (q % 6) < 3;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const int x = __shfl_xor(v, o);
                v = lo ? min(v, x) : max(v, x);
            }
            if ((threadIdx.x & 63) == 0) {
                if (lo) atomicMin(&cbox[j][q], v);
                else atomicMax(&cbox[j][q], v);
            }
        }
}
__device__ __forceinline__ void take_box(int (*mine)[12], bool left, const Tri& x) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (left == (j == 0))
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                mine[j][k] = min(mine[j][k], fenc(x.lo[k]));
                mine[j][3 + k] = max(mine[j][3 + k], fenc(x.hi[k]));
                mine[j][6 + k] = min(mine[j][6 + k], fenc(x.c[k]));
                mine[j][9 + k] = max(mine[j][9 + k], fenc(x.c[k]));
            }
}

}  // namespace

// per triangle: box and centroid (3 float4), the identity order
__global__ void __launch_bounds__(TB) k_sah_init(const float* __restrict__ V, const int* __restrict__ F, int nt,
                                                 float4* __restrict__ tb, uint32_t* __restrict__ ord,
                                                 int* __restrict__ large_bins, int nbins) {
    const int p = blockIdx.x * TB + threadIdx.x;
    for (int q = p; q < nbins; q += gridDim.x * TB) {   // every large task's bins start empty
        large_bins[q * BIN_INTS] = 0;
        box_init(large_bins + q * BIN_INTS + 1, 1);
    }
    if (p >= nt) return;
    const int a = F[3 * p], b = F[3 * p + 1], c = F[3 * p + 2];
    float lo[3], hi[3], ce[3];
    for (int k = 0; k < 3; ++k) {
        const float x = V[3 * a + k], y = V[3 * b + k], z = V[3 * c + k];
        lo[k] = fminf(x, fminf(y, z));
        hi[k] = fmaxf(x, fmaxf(y, z));
        ce[k] = (x + y + z) * (1.0f / 3.0f);   // the centroid as the Morton codes take it
    }
    tb[3 * (size_t)p] = make_float4(lo[0], lo[1], lo[2], 0.f);
    tb[3 * (size_t)p + 1] = make_float4(hi[0], hi[1], hi[2], 0.f);
    tb[3 * (size_t)p + 2] = make_float4(ce[0], ce[1], ce[2], 0.f);
    ord[p] = (uint32_t)p;
}

// the root task; its centroid box comes from the host, which reads every vertex anyway
__global__ void k_sah_root(SahNext nx, int nt, float lx, float ly, float lz, float hx, float hy, float hz) {
    const int cb[6] = {fenc(lx), fenc(ly), fenc(lz), fenc(hx), fenc(hy), fenc(hz)};
    push_task(nx, 0, nt, 0, cb);
}

// Binning of one chunk; a medium task (one chunk) is also split, partitioned and emitted
// here.  Each thread takes consecutive triangles (the partition keeps their order) and
// merges a run that shares a bin before its LDS atomics: neighbours on the mesh mostly do.
__global__ void __launch_bounds__(TB) k_sah_bin(const float4* __restrict__ tb, const uint32_t* __restrict__ ord,
                                                uint32_t* __restrict__ ord_out, const SahTask* __restrict__ tasks,
                                                const int2* __restrict__ chunks, int* __restrict__ large_bins,
                                                SahTree T, SahNext nx) {
    __shared__ int bins[3 * SAH_BINS * BIN_INTS];
    __shared__ int cbox[2][12];
    __shared__ uint32_t part[SAH_CHUNK];
    __shared__ uint64_t ws[TB / 64];
    __shared__ SahBest red[2];
    const int2 ch = chunks[blockIdx.x];
    const SahTask t = tasks[ch.x];
    const int s = ch.y, e = min(s + SAH_CHUNK, t.b);
    for (int q = threadIdx.x; q < 3 * SAH_BINS; q += TB) {
        bins[q * BIN_INTS] = 0;
        box_init(bins + q * BIN_INTS + 1, 1);
    }
    if (threadIdx.x == 0) box_init(&cbox[0][0], 4);
    float lo[3];
    double sc[3];
    for (int ax = 0; ax < 3; ++ax) {
        lo[ax] = fdec(t.cb[ax]);
        const double ext = (double)fdec(t.cb[3 + ax]) - lo[ax];
        sc[ax] = ext > 0.0 ? SAH_BINS / ext : 0.0;
    }
    __syncthreads();
    const int per = (e - s + TB - 1) / TB, i0 = s + per * threadIdx.x;   // per <= PER triangles per thread
    uint32_t p[PER];
    Tri x[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        p[k] = k < per && i0 + k < e ? ord[i0 + k] : UINT32_MAX;
        if (p[k] != UINT32_MAX) x[k] = load_tri(tb, p[k]);
    }
    for (int ax = 0; ax < 3; ++ax) {
        if (!(sc[ax] > 0.0)) continue;
        int bin = -1, run[BIN_INTS];
        auto flush = [&]() {
            if (bin < 0) return;
            int* q = bins + (ax * SAH_BINS + bin) * BIN_INTS;
            atomicAdd(q, run[0]);
            for (int j = 0; j < 3; ++j) {
                atomicMin(q + 1 + j, run[1 + j]);
                atomicMax(q + 4 + j, run[4 + j]);
            }
        };
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (p[k] == UINT32_MAX) continue;
            const int b = sah_bin(x[k].c[ax], lo[ax], sc[ax]);
            if (b != bin) {
                flush();
                bin = b;
                run[0] = 0;
                box_init(run + 1, 1);
            }
            ++run[0];
            for (int j = 0; j < 3; ++j) {
                run[1 + j] = min(run[1 + j], fenc(x[k].lo[j]));
                run[4 + j] = max(run[4 + j], fenc(x[k].hi[j]));
            }
        }
        flush();
    }
    __syncthreads();
    if (t.large >= 0) {   // merge into the task's bins
        int* B = large_bins + (size_t)t.large * LARGE_BIN_INTS;
        for (int q = threadIdx.x; q < 3 * SAH_BINS; q += TB) {
            const int* b = bins + q * BIN_INTS;
            if (b[0] == 0) continue;
            atomicAdd(B + q * BIN_INTS, b[0]);
            for (int j = 0; j < 3; ++j) {
                atomicMin(B + q * BIN_INTS + 1 + j, b[1 + j]);
                atomicMax(B + q * BIN_INTS + 4 + j, b[4 + j]);
            }
        }
        return;
    }
    const int key = sah_best(bins, t.cb, red);
    const int axis = key < 0 ? -1 : key / SAH_BINS, split = key < 0 ? 0 : key % SAH_BINS;
    int nl = 0, mine[2][12];
    box_init(&mine[0][0], 4);
    bool left[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        left[k] = false;
        if (p[k] == UINT32_MAX) continue;
        left[k] = goes_left(t, axis, split, x[k], i0 + k);
        nl += left[k];
        take_box(mine, left[k], x[k]);
    }
    child_boxes(mine, cbox);
    uint64_t tot;
    int li = (int)block_exclusive((uint64_t)nl, ws, &tot);   // (its barriers also cover cbox)
    const int nleft = (int)tot;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (p[k] == UINT32_MAX) continue;
        const int rel = i0 + k - s;
        const int pos = left[k] ? li++ : nleft + (rel - li);
        part[pos] = p[k];
    }
    __syncthreads();
    for (int i = s + threadIdx.x; i < e; i += TB) ord_out[i] = part[i - s];
    if (threadIdx.x == 0) emit(T, nx, t, nleft, cbox);
}

// the split of every large task from its merged bins, which are left empty for the next
// level's tasks
__global__ void __launch_bounds__(TB) k_sah_split(const SahTask* __restrict__ tasks, const int* __restrict__ large_task,
                                                  int* __restrict__ large_bins, SahRes* __restrict__ res) {
    __shared__ int bins[3 * SAH_BINS * BIN_INTS];
    __shared__ SahBest red[2];
    const SahTask t = tasks[large_task[blockIdx.x]];
    int* B = large_bins + (size_t)blockIdx.x * LARGE_BIN_INTS;
    for (int k = threadIdx.x; k < LARGE_BIN_INTS; k += TB) {
        bins[k] = B[k];
        const int f = k % BIN_INTS;
        B[k] = f == 0 ? 0 : (f < 4 ? fenc(FLT_MAX) : fenc(-FLT_MAX));
    }
    __syncthreads();
    const int key = sah_best(bins, t.cb, red);
    if (threadIdx.x == 0) {
        SahRes& r = res[blockIdx.x];
        r.axis = key < 0 ? -1 : key / SAH_BINS;
        r.split = key < 0 ? 0 : key % SAH_BINS;
        int nl = 0;
        if (key < 0) nl = (t.b - t.a) / 2;
        else
            for (int k = 0; k < r.split; ++k) nl += bins[(r.axis * SAH_BINS + k) * BIN_INTS];
        r.nleft = nl;
        box_init(&r.box[0][0], 4);
    }
}

// large tasks: left count of every chunk, and the children's boxes
__global__ void __launch_bounds__(TB) k_sah_part_count(const float4* __restrict__ tb, const uint32_t* __restrict__ ord,
                                                       const SahTask* __restrict__ tasks, const int2* __restrict__ chunks,
                                                       int* __restrict__ chunk_left, SahRes* __restrict__ res) {
    __shared__ int cbox[2][12];
    __shared__ int nl;
    const int c = blockIdx.x;
    const int2 ch = chunks[c];
    const SahTask t = tasks[ch.x];
    if (t.large < 0) return;
    SahRes& o = res[t.large];
    const int axis = o.axis, split = o.split;
    if (threadIdx.x == 0) {
        box_init(&cbox[0][0], 4);
        nl = 0;
    }
    __syncthreads();
    const int s = ch.y, e = min(s + SAH_CHUNK, t.b);
    int my = 0, mine[2][12];
    box_init(&mine[0][0], 4);
    for (int i = s + threadIdx.x; i < e; i += TB) {
        const Tri x = load_tri(tb, ord[i]);
        const bool l = goes_left(t, axis, split, x, i);
        my += l;
        take_box(mine, l, x);
    }
    child_boxes(mine, cbox);
    for (int w = 32; w > 0; w >>= 1) my += __shfl_xor(my, w);
    if ((threadIdx.x & 63) == 0) atomicAdd(&nl, my);
    __syncthreads();
    if (threadIdx.x < 24) {
        const int k = threadIdx.x / 12, j = threadIdx.x % 12;
        if ((j % 6) < 3) atomicMin(&o.box[k][j], cbox[k][j]);
        else atomicMax(&o.box[k][j], cbox[k][j]);
    }
    if (threadIdx.x == 0) chunk_left[c] = nl;
}

// large tasks: stable partition into the other order buffer; a task's first chunk emits it
__global__ void __launch_bounds__(TB) k_sah_part_scatter(const float4* __restrict__ tb, const uint32_t* __restrict__ ord,
                                                         uint32_t* __restrict__ ord_out,
                                                         const SahTask* __restrict__ tasks, const int2* __restrict__ chunks,
                                                         const int* __restrict__ chunk_left,
                                                         const SahRes* __restrict__ res, SahTree T, SahNext nx) {
    __shared__ uint64_t ws[TB / 64];
    const int c = blockIdx.x;
    const int2 ch = chunks[c];
    const SahTask t = tasks[ch.x];
    if (t.large < 0) return;
    const SahRes& r = res[t.large];
    const int axis = r.axis, split = r.split, nleft = r.nleft;
    int before = 0;   // left triangles of the task's earlier chunks
    for (int q = t.c0 + (int)threadIdx.x; q < c; q += TB) before += chunk_left[q];
    uint64_t tot;
    (void)block_exclusive((uint64_t)before, ws, &tot);
    before = (int)tot;
    const int s = ch.y, e = min(s + SAH_CHUNK, t.b);
    uint32_t p[PER];
    bool left[PER];
    int nl = 0;
    for (int k = 0; k < PER; ++k) {
        const int i = s + PER * threadIdx.x + k;
        left[k] = false;
        p[k] = 0;
        if (i >= e) continue;
        p[k] = ord[i];
        left[k] = goes_left(t, axis, split, load_tri(tb, p[k]), i);
        nl += left[k];
    }
    int li = before + (int)block_exclusive((uint64_t)nl, ws, &tot);
    for (int k = 0; k < PER; ++k) {
        const int i = s + PER * threadIdx.x + k;
        if (i >= e) continue;
        const int rel = i - t.a;   // index within the task
        const int pos = left[k] ? t.a + li++ : t.a + nleft + (rel - li);
        if (pos >= t.a && pos < t.b) ord_out[pos] = p[k];
    }
    if (c == t.c0 && threadIdx.x == 0) emit(T, nx, t, nleft, r.box);
}

// One wave (workgroup of 64) builds the subtree of a small task: lane = position in the
// range, every node of a level at once.  A lane's node is the segment [s0, s1) of lanes;
// each loop runs over the lane's own segment (its triangles in LDS), so a level costs its
// longest segment.  A lane proposes the split in front of its own bin on every axis -- the
// other bins split the segment no differently -- and the segment takes the best by the
// same order (cost, axis, bin).  The loops are bound by vector issue, about 90 instructions
// per step over the three axes.
__global__ void __launch_bounds__(SAH_SMALL) k_sah_small(const float4* __restrict__ tb, const uint32_t* __restrict__ ord0,
                                                         const uint32_t* __restrict__ ord1,
                                                         const SahSmall* __restrict__ small, uint32_t* __restrict__ order,
                                                         SahTree T, int* __restrict__ bad) {
    __shared__ float sx[9][SAH_SMALL];   // box lo, hi, centroid by position
    __shared__ uint32_t sid[SAH_SMALL], sbin[SAH_SMALL];
    __shared__ double scost[SAH_SMALL];
    __shared__ int skey[SAH_SMALL];
    const SahSmall t = small[blockIdx.x];
    const int n = t.b - t.a, pos = threadIdx.x;
    const bool live = pos < n;
    if (n < 1 || n > SAH_SMALL || t.a < 0 || t.b > T.nt || (n > 1 && (t.node < 0 || t.node + n - 1 > T.nt - 1))) {
        if (pos == 0) atomicExch(bad, 1);   // never
        return;
    }
    if (live) {
        const uint32_t p = (t.buf ? ord1 : ord0)[t.a + pos];
        const Tri x = load_tri(tb, p);
        for (int k = 0; k < 3; ++k) {
            sx[k][pos] = x.lo[k];
            sx[3 + k][pos] = x.hi[k];
            sx[6 + k][pos] = x.c[k];
        }
        sid[pos] = p;
    }
    int s0 = live ? 0 : pos, s1 = live ? n : pos + 1, node = t.node;
    while (__syncthreads_or(s1 - s0 > 1)) {
        const bool on = s1 - s0 > 1;
        // bins of the lane's triangle in its segment's centroid box
        float clo[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, chi[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
        if (on)
            for (int j = s0; j < s1; ++j)
                for (int k = 0; k < 3; ++k) {
                    clo[k] = fminf(clo[k], sx[6 + k][j]);
                    chi[k] = fmaxf(chi[k], sx[6 + k][j]);
                }
        int bin[3] = {0, 0, 0};
        if (on)
            for (int k = 0; k < 3; ++k) {
                const double ext = (double)chi[k] - clo[k];
                if (ext > 0.0) bin[k] = sah_bin(sx[6 + k][pos], clo[k], SAH_BINS / ext);
            }
        sbin[pos] = (uint32_t)bin[0] | (uint32_t)bin[1] << 8 | (uint32_t)bin[2] << 16;
        __syncthreads();
        SahBest me{-1.0, -1};
        if (on)
            for (int ax = 0; ax < 3; ++ax) {
                if (!((double)chi[ax] - clo[ax] > 0.0)) continue;
                float l0[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, l1[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
                float r0[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, r1[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
                int nl = 0;
                for (int j = s0; j < s1; ++j) {
                    const bool l = (int)((sbin[j] >> (8 * ax)) & 255u) < bin[ax];
                    nl += l;
                    for (int k = 0; k < 3; ++k) {
                        const float a = sx[k][j], b = sx[3 + k][j];
                        l0[k] = fminf(l0[k], l ? a : FLT_MAX);
                        l1[k] = fmaxf(l1[k], l ? b : -FLT_MAX);
                        r0[k] = fminf(r0[k], l ? FLT_MAX : a);
                        r1[k] = fmaxf(r1[k], l ? -FLT_MAX : b);
                    }
                }
                const int nr = s1 - s0 - nl;
                if (nl > 0 && nr > 0)
                    me = better(me, SahBest{box_area(l0, l1) * nl + box_area(r0, r1) * nr, ax * SAH_BINS + bin[ax]});
            }
        scost[pos] = me.cost;
        skey[pos] = me.key;
        __syncthreads();
        // the segment's split, its sides and this lane's place in them
        float b0[6], b1[6];
        int nl = 0, rank = 0;
        bool left = false;
        if (on) {
            me = SahBest{-1.0, -1};
            for (int j = s0; j < s1; ++j) me = better(me, SahBest{scost[j], skey[j]});
            const int ax = me.key < 0 ? 0 : me.key / SAH_BINS, sp = me.key % SAH_BINS, half = s0 + (s1 - s0) / 2;
            for (int k = 0; k < 3; ++k) {
                b0[k] = b1[k] = FLT_MAX;
                b0[3 + k] = b1[3 + k] = -FLT_MAX;
            }
            for (int j = s0; j < s1; ++j) {
                const bool l = me.key < 0 ? j < half : (int)((sbin[j] >> (8 * ax)) & 255u) < sp;
                if (j == pos) {
                    left = l;
                    rank = nl;   // left triangles before this one
                }
                nl += l;
                for (int k = 0; k < 3; ++k) {
                    const float a = sx[k][j], b = sx[3 + k][j];
                    b0[k] = fminf(b0[k], l ? a : FLT_MAX);
                    b0[3 + k] = fmaxf(b0[3 + k], l ? b : -FLT_MAX);
                    b1[k] = fminf(b1[k], l ? FLT_MAX : a);
                    b1[3 + k] = fmaxf(b1[3 + k], l ? -FLT_MAX : b);
                }
            }
            if (pos == s0) write_node(T, t.a + s0, t.a + s1, node, nl, b0, b1);
        }
        // move the triangles to their new positions
        float v[9];
        for (int k = 0; k < 9; ++k) v[k] = sx[k][pos];
        const uint32_t id = sid[pos];
        const int to = !on ? pos : (left ? s0 + rank : s0 + nl + (pos - s0 - rank));
        __syncthreads();
        for (int k = 0; k < 9; ++k) sx[k][to] = v[k];
        sid[to] = id;
        if (on) {   // the lane's segment by its position
            const int mid = s0 + nl;
            if (pos < mid) {
                node = node + 1;
                s1 = mid;
            } else {
                node = node + nl;
                s0 = mid;
            }
        }
        __syncthreads();
    }
    if (live) order[t.a + pos] = sid[pos];
}

static inline unsigned grid_of(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }
static inline size_t r256(size_t b) { return (b + 255) & ~size_t(255); }

namespace {
struct SahLayout {
    size_t tb, ord, order, tasks, res, chunks, chunk_left, large_task, large_bins, small, words, total;
    int tcap, ccap, lcap, scap;
    explicit SahLayout(int nt) {
        const size_t n = (size_t)nt;
        // tasks of one level are disjoint ranges of more than SAH_SMALL triangles, small
        // tasks disjoint ranges of at least one
        tcap = nt / (SAH_SMALL + 1) + 1;
        ccap = tcap + nt / SAH_CHUNK + 1;
        lcap = nt / (SAH_CHUNK + 1) + 1;
        scap = nt;
        size_t o = 0;
        auto put = [&](size_t b) {
            const size_t at = o;
            o += r256(b);
            return at;
        };
        tb = put(48 * n);
        ord = put(2 * r256(4 * n));
        order = put(4 * n);
        tasks = put(2 * sizeof(SahTask) * (size_t)tcap);
        res = put(sizeof(SahRes) * (size_t)lcap);
        chunks = put(2 * 8 * (size_t)ccap);
        chunk_left = put(4 * (size_t)ccap);
        large_task = put(2 * 4 * (size_t)lcap);
        large_bins = put(4 * (size_t)LARGE_BIN_INTS * lcap);
        small = put(sizeof(SahSmall) * (size_t)scap);
        words = put(sizeof(SahCount) * (MAX_LEVELS + 2) + 16);
        total = o;
    }
};
}  // namespace

size_t sah_scratch_bytes(int nt) { return SahLayout(nt).total; }

hipError_t build_sah(hipStream_t st, const BvhInputs& in, void* scratch, float4* nodes, const uint32_t** order_out) {
    const int nt = in.nt;
    if (nt < 2) return hipErrorInvalidValue;
    const SahLayout L(nt);
    char* base = (char*)scratch;
    float4* tb = (float4*)(base + L.tb);
    uint32_t* ord[2] = {(uint32_t*)(base + L.ord), (uint32_t*)(base + L.ord + r256(4 * (size_t)nt))};
    uint32_t* order = (uint32_t*)(base + L.order);
    SahTask* tasks[2] = {(SahTask*)(base + L.tasks), (SahTask*)(base + L.tasks) + L.tcap};
    SahRes* res = (SahRes*)(base + L.res);
    int2* chunks[2] = {(int2*)(base + L.chunks), (int2*)(base + L.chunks) + L.ccap};
    int* chunk_left = (int*)(base + L.chunk_left);
    int* large_task[2] = {(int*)(base + L.large_task), (int*)(base + L.large_task) + L.lcap};
    int* large_bins = (int*)(base + L.large_bins);
    SahSmall* small = (SahSmall*)(base + L.small);
    // counters: [0] small tasks, [1] bad flag, then the lists of every level
    int* words = (int*)(base + L.words);
    SahCount* counts = (SahCount*)(words + 4);
    const SahTree T{nodes, in.child, in.parent_int, in.parent_leaf, nt};
    auto next = [&](int level, int buf) {   // the lists of `level` (tasks alternate, counters do not)
        return SahNext{tasks[level & 1], chunks[level & 1], large_task[level & 1], counts + level, small, words,
                       L.tcap, L.ccap, L.lcap, L.scap, buf, words + 1};
    };
    *order_out = order;
    hipError_t e = hipMemsetAsync(words, 0, 16 + sizeof(SahCount) * (MAX_LEVELS + 2), st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sah_init, dim3(grid_of(nt, TB)), dim3(TB), 0, st, in.V, in.F, nt, tb, ord[0], large_bins,
                       3 * SAH_BINS * L.lcap);
    hipLaunchKernelGGL(k_sah_root, dim3(1), dim3(1), 0, st, next(0, 0), nt, in.clo[0], in.clo[1], in.clo[2], in.chi[0],
                       in.chi[1], in.chi[2]);
    // the first level's counts are known; later ones are read back, with the bad flag
    SahCount c{nt > SAH_SMALL ? 1 : 0, nt > SAH_SMALL ? (nt + SAH_CHUNK - 1) / SAH_CHUNK : 0, nt > SAH_CHUNK ? 1 : 0, 0};
    int cur = 0, nsmall = nt <= SAH_SMALL ? 1 : 0;
    for (int level = 0; c.tasks > 0; ++level) {
        // binary depth is capped at 64 levels for the traversal's stack; a deeper SAH tree is
        // refused rather than built
        if (level >= MAX_LEVELS) return hipErrorNotSupported;
        const int w = level & 1;
        const SahNext nx = next(level + 1, cur ^ 1);
        const dim3 g((unsigned)c.chunks), b(TB);
        hipLaunchKernelGGL(k_sah_bin, g, b, 0, st, tb, ord[cur], ord[cur ^ 1], tasks[w], chunks[w], large_bins, T, nx);
        if (c.large > 0) {
            hipLaunchKernelGGL(k_sah_split, dim3((unsigned)c.large), b, 0, st, tasks[w], large_task[w], large_bins, res);
            hipLaunchKernelGGL(k_sah_part_count, g, b, 0, st, tb, ord[cur], tasks[w], chunks[w], chunk_left, res);
            hipLaunchKernelGGL(k_sah_part_scatter, g, b, 0, st, tb, ord[cur], ord[cur ^ 1], tasks[w], chunks[w],
                               chunk_left, res, T, nx);
        }
        int hw[4 + 4 * (MAX_LEVELS + 2)];
        e = hipMemcpyAsync(hw, words, 16 + sizeof(SahCount) * (level + 2), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        nsmall = hw[0];
        std::memcpy(&c, hw + 4 + 4 * (level + 1), sizeof c);
        if (hw[1] != 0 || c.tasks > L.tcap || c.chunks > L.ccap || c.large > L.lcap || nsmall > L.scap)
            return hipErrorUnknown;
        cur ^= 1;
    }
    if (nsmall > 0)
        hipLaunchKernelGGL(k_sah_small, dim3((unsigned)nsmall), dim3(SAH_SMALL), 0, st, tb, ord[0], ord[1], small, order, T,
                           words + 1);
    e = hipGetLastError();
    return e;
}

}  // namespace dpcs
