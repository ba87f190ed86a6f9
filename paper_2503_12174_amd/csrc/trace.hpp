// trace.hpp -- ray queries on the device BVH.
//
// BVH2 node (64 B, 4 x float4): both children's boxes inline so one node fetch
// tests two boxes.
//   n0 = (lo0.x, lo0.y, lo0.z, hi0.x)  n1 = (hi0.y, hi0.z, lo1.x, lo1.y)
//   n2 = (lo1.z, hi1.x, hi1.y, hi1.z)  n3 = (child0, child1, -, -) as int bits
// BVH4 node (128 B, one cache line, 8 x float4): the four children's boxes as
// structure of arrays, lo.x[4], lo.y[4], lo.z[4], hi.x[4], hi.y[4], hi.z[4], then the
// four child references, the binary node it stands for (refits) and 12 unused bytes.
// child >= 0: internal node index; child < 0: leaf ~child (one triangle, leaf order).
// An unused slot of a BVH4 node holds an inverted box far from the scene, which the
// 4-wide box test never enters, and the dummy leaf nt (one record past the mesh's
// triangles, NaN vertices), which no ray hits, so the loop needs no test for them.
// Triangle record (64 B, half a cache line): v0 (w = original triangle index bits), v1 (w = u0),
// v2 (w = v0 of the texture coordinates), then (u1, v1, u2, v2): a triangle test and a
// vertex's shading each touch one aligned 64-byte block.  With 48-byte vertex records and
// 32-byte coordinate records apart a vertex's shading touched 2.4 lines: 256 x 256 x 64 of the
// 50k-triangle corner 1596 us, 1587 with this record; a step of its fit 2348 us, 2313.
//
// Closest hit: smallest t in (tmin, tmax); equal t -> smaller original triangle
// index, so the result equals a brute-force scan in the same arithmetic.  Box tests
// are widened by a few ulps so no triangle a brute-force scan would accept is culled.
#pragma once

#include "common.hpp"

namespace dpcs {

// watertight ray / triangle test (Woop, Benthin, Wald, JCGT 2013)
struct WtRay {
    V3 o;
    int kz;              // axis of the largest direction component; the others follow in cyclic order
    float Sx, Sy, Sz;
};
// a's components along the axes kz + 1, kz + 2 and kz (cyclic)
__device__ __forceinline__ V3 turned(V3 a, int kz) {
    return v3(kz == 0 ? a.y : (kz == 1 ? a.z : a.x), kz == 0 ? a.z : (kz == 1 ? a.x : a.y),
              kz == 0 ? a.x : (kz == 1 ? a.y : a.z));
}

__device__ __forceinline__ WtRay wt_setup(V3 o, V3 d) {
    WtRay r;
    r.o = o;
    const float ax = fabsf(d.x), ay = fabsf(d.y), az = fabsf(d.z);
    r.kz = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
    // (the method swaps the first two axes where the third component is negative, to keep
    // the winding; here the edge functions, the determinant and T all change sign with it,
    // exactly, and neither t nor the barycentrics do)
    const V3 q = turned(d, r.kz);
    // the shear need not be correctly rounded, only the same for every triangle a ray
    // meets (watertightness), so the hardware reciprocal (within 1 ulp) stands in for the
    // multi-instruction IEEE division; |dz| >= 1/sqrt(3) for a unit direction
    r.Sz = __builtin_amdgcn_rcpf(q.z);
    r.Sx = q.x * r.Sz;
    r.Sy = q.y * r.Sz;
    return r;
}

// returns false on a miss; on a hit t and the barycentrics (b1 of v1, b2 of v2)
__device__ __forceinline__ bool wt_intersect(const WtRay& r, V3 v0, V3 v1, V3 v2, float& t, float& b1, float& b2) {
    const V3 A = turned(v0 - r.o, r.kz), B = turned(v1 - r.o, r.kz), C = turned(v2 - r.o, r.kz);
    const float Akz = A.z, Bkz = B.z, Ckz = C.z;
    const float Ax = A.x - r.Sx * Akz, Ay = A.y - r.Sy * Akz;
    const float Bx = B.x - r.Sx * Bkz, By = B.y - r.Sy * Bkz;
    const float Cx = C.x - r.Sx * Ckz, Cy = C.y - r.Sy * Ckz;
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if (U == 0.0f || V == 0.0f || W == 0.0f) {  // edge case: decide in double
        U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
        V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
        W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
    }
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    const float det = U + V + W;
    if (det == 0.0f) return false;
    const float T = U * (r.Sz * Akz) + V * (r.Sz * Bkz) + W * (r.Sz * Ckz);
    const float inv = 1.0f / det;
    t = T * inv;
    b1 = V * inv;
    b2 = W * inv;
    return true;
}

// The traversal loops decide hits with this cheaper form of the same test: no
// barycentrics, and t = (Sz T') * rcp(det) with T' = U Akz + V Bkz + W Ckz (the hardware
// reciprocal, not the correctly rounded quotient).  Every query -- BVH or brute force --
// decides with it and then recomputes the reported t and barycentrics of its winner with
// wt_intersect, so all of them agree bit for bit.
__device__ __forceinline__ bool wt_hit(const WtRay& r, V3 v0, V3 v1, V3 v2, float& t) {
    const V3 A = turned(v0 - r.o, r.kz), B = turned(v1 - r.o, r.kz), C = turned(v2 - r.o, r.kz);
    const float Akz = A.z, Bkz = B.z, Ckz = C.z;
    const float Ax = A.x - r.Sx * Akz, Ay = A.y - r.Sy * Akz;
    const float Bx = B.x - r.Sx * Bkz, By = B.y - r.Sy * Bkz;
    const float Cx = C.x - r.Sx * Ckz, Cy = C.y - r.Sy * Ckz;
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if (U == 0.0f || V == 0.0f || W == 0.0f) {  // edge case: decide in double
        U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
        V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
        W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
    }
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    const float det = U + V + W;
    if (det == 0.0f) return false;
    const float T = U * Akz + V * Bkz + W * Ckz;
    t = (T * r.Sz) * __builtin_amdgcn_rcpf(det);
    return true;
}

struct Hit {
    float t;
    int leaf;   // leaf-order triangle index, -1 on a miss
    int prim;   // original triangle index
    float b1, b2;
};

struct BoxRay {
    V3 o, inv;
};
// (hardware reciprocals, within 1 ulp: the 4e-6 widening of every slab covers it)
__device__ __forceinline__ BoxRay box_setup(V3 o, V3 d) {
    return BoxRay{o, v3(__builtin_amdgcn_rcpf(d.x), __builtin_amdgcn_rcpf(d.y), __builtin_amdgcn_rcpf(d.z))};
}

// conservative entry distance of the ray into [lo, hi]; returns +inf when missed
__device__ __forceinline__ float box_enter(const BoxRay& r, float lx, float ly, float lz, float hx, float hy, float hz,
                                           float tmin, float tmax) {
    const float tx0 = (lx - r.o.x) * r.inv.x, tx1 = (hx - r.o.x) * r.inv.x;
    const float ty0 = (ly - r.o.y) * r.inv.y, ty1 = (hy - r.o.y) * r.inv.y;
    const float tz0 = (lz - r.o.z) * r.inv.z, tz1 = (hz - r.o.z) * r.inv.z;
    float tn = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fminf(tz0, tz1));
    float tf = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fmaxf(tz0, tz1));
    // widen by 4e-6 relative (a few ulps of every operation above)
    tn = tn - fabsf(tn) * 4e-6f;
    tf = tf + fabsf(tf) * 4e-6f;
    tn = fmaxf(tn, tmin);
    tf = fminf(tf, tmax);
    return tn <= tf ? tn : __builtin_inff();
}

__device__ __forceinline__ void load_tri(const float4* __restrict__ tris, int leaf, V3& v0, V3& v1, V3& v2, int& prim) {
    const float4* t = tris + 4 * (size_t)(uint32_t)leaf;
    const float4 a = t[0], b = t[1], c = t[2];
    v0 = xyz(a);
    v1 = xyz(b);
    v2 = xyz(c);
    prim = __float_as_int(a.w);
}
// the same with the corners' texture coordinates: ua = (u0 v0 u1 v1), ub = (u2 v2)
__device__ __forceinline__ void load_tri_uv(const float4* __restrict__ tris, int leaf, V3& v0, V3& v1, V3& v2, int& prim,
                                            float4& ua, float2& ub) {
    const float4* t = tris + 4 * (size_t)(uint32_t)leaf;
    const float4 a = t[0], b = t[1], c = t[2], d = t[3];
    v0 = xyz(a);
    v1 = xyz(b);
    v2 = xyz(c);
    prim = __float_as_int(a.w);
    ua = make_float4(b.w, c.w, d.x, d.y);
    ub = make_float2(d.z, d.w);
}

// Traversal stack of internal node indices: the first SHORT entries live in LDS, entry
// k of lane `lane` at stack[k * TBK + lane] (consecutive lanes on consecutive banks),
// plus one more LDS entry per lane (k = SHORT) that the 4-wide push writes candidates
// it does not keep to;
// deeper entries -- rare with near-child-first order -- go to the workgroup's region of
// global memory with the same interleaving, spill[(k - SHORT) * TBK + lane].  Both
// bases are uniform, so a lane holds only its index.  The host only launches on trees
// whose stack bound is <= 64, so at most 64 entries are ever live.
//
// Node and triangle visit counters for the profiler's counting pass; the timed
// kernels use Visits<false>, which keeps no registers.
template <bool ON>
struct Visits {
    uint32_t nodes = 0, tris = 0;
    __device__ __forceinline__ void node() { ++nodes; }
    __device__ __forceinline__ void tri() { ++tris; }
};
template <>
struct Visits<false> {
    static constexpr uint32_t nodes = 0, tris = 0;
    __device__ __forceinline__ void node() {}
    __device__ __forceinline__ void tri() {}
};

template <bool ANY, int SHORT, int TBK, class VIS>
__device__ __forceinline__ bool traverse(const float4* __restrict__ nodes, const float4* __restrict__ tris, V3 o, V3 d,
                                         float tmin, float tmax, int skip, Hit& h, int* stack, int* spill, int lane,
                                         VIS& vis) {
    const BoxRay br = box_setup(o, d);
    const WtRay wr = wt_setup(o, d);
    float best_t = tmax;
    int best_prim = 0x7fffffff, best_leaf = -1;
    int sp = 0;
    int node = 0;
    while (node >= 0) {   // the only exit (see traverse4)
        vis.node();
        const float4 n0 = nodes[4 * node], n1 = nodes[4 * node + 1], n2 = nodes[4 * node + 2];
        const int4 n3 = *reinterpret_cast<const int4*>(&nodes[4 * node + 3]);
        float t0 = box_enter(br, n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, tmin, best_t);
        float t1 = box_enter(br, n1.z, n1.w, n2.x, n2.y, n2.z, n2.w, tmin, best_t);
        const int c0 = n3.x, c1 = n3.y;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int c = k == 0 ? c0 : c1;
            const float tc = k == 0 ? t0 : t1;
            if (c < 0 && tc < __builtin_inff()) {
                const int leaf = ~c;
                V3 v0, v1, v2;
                int prim;
                vis.tri();
                load_tri(tris, leaf, v0, v1, v2, prim);
                float t;
                const bool hit = wt_hit(wr, v0, v1, v2, t);   // the skip test after it (one load)
                if (hit & (prim != skip) & (t > tmin) &&
                    (t < best_t || (t == best_t && best_leaf >= 0 && prim < best_prim))) {
                    best_t = t;
                    best_prim = prim;
                    best_leaf = leaf;
                }
            }
        }
        // a missed box reports +inf, which must not pass while best_t is still +inf
        const bool h0 = c0 >= 0 && t0 < __builtin_inff() && t0 <= best_t;
        const bool h1 = c1 >= 0 && t1 < __builtin_inff() && t1 <= best_t;
        if (ANY && best_leaf >= 0) {   // any hit ends the query
            node = -1;
        } else if (h0 && h1) {
            const bool first0 = t0 <= t1;
            const int far = first0 ? c1 : c0;
            if (sp < SHORT) stack[sp * TBK + lane] = far;
            else if constexpr (SHORT < MAX_STACK) {
                if (sp < MAX_STACK) spill[(sp - SHORT) * TBK + lane] = far;
            }
            sp = sp < MAX_STACK ? sp + 1 : sp;   // depth <= 64 is checked on the host
            node = first0 ? c0 : c1;
        } else if (h0) {
            node = c0;
        } else if (h1) {
            node = c1;
        } else if (sp > 0) {
            --sp;
            node = stack[min(sp, SHORT - 1) * TBK + lane];
            if constexpr (SHORT < MAX_STACK)
                if (sp >= SHORT) node = spill[(sp - SHORT) * TBK + lane];
        } else {
            node = -1;
        }
    }
    float bb1 = 0.f, bb2 = 0.f;
    if (best_leaf >= 0) {   // reported t and barycentrics: the exact test on the winner
        V3 v0, v1, v2;
        int prim;
        load_tri(tris, best_leaf, v0, v1, v2, prim);
        wt_intersect(wr, v0, v1, v2, best_t, bb1, bb2);
    }
    h.t = best_t;
    h.leaf = best_leaf;
    h.prim = best_leaf >= 0 ? best_prim : -1;
    h.b1 = bb1;
    h.b2 = bb2;
    return best_leaf >= 0;
}

__device__ __forceinline__ void sort2(uint32_t& a, uint32_t& b) {
    const uint32_t lo = min(a, b);
    b = max(a, b);
    a = lo;
}

// Ray constants of the 4-wide box tests.  Per axis, the sign of the direction says
// which of a child's two planes the ray meets first, so a node load fetches the near
// and the far coordinates directly (byte offsets below) and each slab takes one FMA,
// plane * (1 / d) + off, with no min/max per axis.  off is -o / d rounded outward:
// down by at least the rounding error of o / d for near planes, up for far planes.
// With that, a slab value can only err by the relative rounding of 1 / d and of the
// FMA, which the relative widening covers; it needs no absolute term that would grow for
// near-axis-parallel rays.  The widening, t x (1 -+ 4e-6), is in the constants, so a box
// test takes no product for it (the closest-hit loop is bound by vector issue: 256 x 256 x
// 64 of the 50k-triangle corner 1583 us with the two products, 1580 without, and 1587 before
// the triangle test lost its swap of two axes; with an environment map 2200, 2193, 2180).
// An axis along which the ray does not move (less than 2^-80 of its largest component, so for
// directions of any length, or 0) takes the reciprocal of that least movement -- infinite for
// directions shorter than 2^-46, whose slab values on the axis come out NaN or infinite and let
// every box pass.  Every offset is widened by 2^-40 in space besides, so such a slab lets pass
// exactly the boxes that hold the ray's coordinate, faces included.  (With 1 / 0 a unit
// direction's slab values came out NaN too: a bounce straight along the normal of an
// axis-aligned face, one sample in 2^24, walked a whole wall of the corner, 12 ms for one
// ray.)  The widening multiplies rather than adding a multiple of |t|, so infinite slab
// values stay infinite instead of turning NaN, and an inverted box (lo = +1e30, hi = -1e30:
// every near plane ahead of every far plane) is always missed.
struct Box4Ray {
    float ix, iy, iz;             // 1 / d, less the widening (near planes)
    float jx, jy, jz;             // 1 / d and the widening (far planes)
    float anx, any, anz;          // near-plane offsets
    float afx, afy, afz;          // far-plane offsets
    uint32_t onx, ony, onz;       // byte offset of the near coordinate float4 in a node
};
// the far coordinate float4 of each axis sits at the near one's offset XOR these
// (x: 0 <-> 48, y: 16 <-> 64, z: 32 <-> 80)
constexpr uint32_t FAR_X = 48u, FAR_Y = 80u, FAR_Z = 112u;

__device__ __forceinline__ Box4Ray box4_setup(V3 o, V3 d) {
    Box4Ray r;
    // hardware reciprocals (within 1 ulp) of components kept away from 0
    const float least = fmaxf(fmaxf(fabsf(d.x), fabsf(d.y)), fabsf(d.z)) * 0x1p-80f;
    r.ix = __builtin_amdgcn_rcpf(copysignf(fmaxf(fabsf(d.x), least), d.x));
    r.iy = __builtin_amdgcn_rcpf(copysignf(fmaxf(fabsf(d.y), least), d.y));
    r.iz = __builtin_amdgcn_rcpf(copysignf(fmaxf(fabsf(d.z), least), d.z));
    // |fl(o rcp(d)) - o rcp(d)| <= 2^-24 |o rcp(d)|, and as much again for each of the sum,
    // its product with 1 -+ 4e-6 and that of rcp(d) below: 2^-21 is twice what they take;
    // 2^-40 / |d|: the faces of an axis along which the ray does not move
    const float px = o.x * r.ix, py = o.y * r.iy, pz = o.z * r.iz;
    const float ex = fmaf(fabsf(r.ix), 0x1p-40f, fabsf(px) * 0x1p-21f);
    const float ey = fmaf(fabsf(r.iy), 0x1p-40f, fabsf(py) * 0x1p-21f);
    const float ez = fmaf(fabsf(r.iz), 0x1p-40f, fabsf(pz) * 0x1p-21f);
    constexpr float WN = 1.0f - 4e-6f, WF = 1.0f + 4e-6f;
    r.jx = r.ix * WF, r.jy = r.iy * WF, r.jz = r.iz * WF;
    r.ix *= WN, r.iy *= WN, r.iz *= WN;
    r.anx = (-px - ex) * WN;
    r.any = (-py - ey) * WN;
    r.anz = (-pz - ez) * WN;
    r.afx = (-px + ex) * WF;
    r.afy = (-py + ey) * WF;
    r.afz = (-pz + ez) * WF;
    // node float4s: 0 lo.x, 1 lo.y, 2 lo.z, 3 hi.x, 4 hi.y, 5 hi.z
    const bool sx = __builtin_signbit(r.ix), sy = __builtin_signbit(r.iy), sz = __builtin_signbit(r.iz);
    r.onx = sx ? 48u : 0u;
    r.ony = sy ? 64u : 16u;
    r.onz = sz ? 80u : 32u;
    return r;
}

// Whether the ray meets a child box of a node (near / far planes as loaded) before tmax,
// and the entry distance tn.  (A negative entry or exit is scaled the wrong way, which the
// clamp to tmin > 0 makes irrelevant.)
__device__ __forceinline__ bool box4_hit(const Box4Ray& r, float nx, float ny, float nz, float fx, float fy, float fz,
                                         float tmin, float tmax, float& tn) {
    tn = fmaxf(fmaxf(fmaf(nx, r.ix, r.anx), fmaf(ny, r.iy, r.any)), fmaf(nz, r.iz, r.anz));
    tn = fmaxf(tn, tmin);
    const float tf = fminf(fminf(fmaf(fx, r.jx, r.afx), fmaf(fy, r.jy, r.afy)), fmaf(fz, r.jz, r.afz));
    return tn <= fminf(tf, tmax);
}

// The top of the 4-wide tree in LDS: the collapse numbers nodes breadth first, so nodes
// [0, n) are its top levels; a workgroup copies them once and every ray that passes them
// reads LDS instead of L2.  bytes = 128 n (0: nothing staged).  (The scene only keeps a
// 4-wide tree whose worst-case stack fits MAX_STACK.)
struct TopNodes {
    const float4* lds;
    uint32_t bytes;
};


// all threads of the workgroup call it (it ends with a barrier); n <= TOP_NODES
template <int TBK>
__device__ __forceinline__ TopNodes stage_top(float4* lds, const float4* __restrict__ nodes4, int n) {
    for (int k = threadIdx.x; k < 8 * n; k += TBK) lds[k] = nodes4[k];
    __syncthreads();
    return TopNodes{lds, 128u * (uint32_t)n};
}

// One 4-wide query's state: the ray constants, the best hit so far, the stack depth, the
// next node (-1: the walk has ended) and a leaf ~pend whose triangle is still to be tested (0: none).
struct Trav4 {
    Box4Ray br;
    WtRay wr;
    float tmin, best_t;
    int skip, best_leaf, sp, node, pend;
};

__device__ __forceinline__ void trav4_start(Trav4& s, V3 o, V3 d, float tmin, float tmax, int skip) {
    s.br = box4_setup(o, d);
    s.wr = wt_setup(o, d);
    s.tmin = tmin;
    s.best_t = tmax;
    s.skip = skip;
    s.best_leaf = -1;
    s.sp = 0;
    s.node = 0;
    s.pend = 0;
}

// this lane's bit of a lane mask
__device__ __forceinline__ bool lane_of(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// the triangle of leaf ~s.pend
template <bool ANY, class VIS>
__device__ __forceinline__ void trav4_leaf(Trav4& s, const float4* __restrict__ tris, VIS& vis) {
    V3 v0, v1, v2;
    int prim;
    vis.tri();
    load_tri(tris, ~s.pend, v0, v1, v2, prim);
    float t;
    // the triangle left is rejected after the test, not before it: checked first, the
    // prim id was loaded alone and the vertices only after the compare (two dependent
    // round trips to memory per test)
    const bool hit = wt_hit(s.wr, v0, v1, v2, t);
    if (!hit | !(t > s.tmin) | (prim == s.skip)) return;
    bool take = t < s.best_t;
    if constexpr (!ANY) {
        // equal t: the smaller original index wins (the current best's index is read
        // back from its record, so no register holds it)
        if (!take && t == s.best_t && s.best_leaf >= 0) take = prim < __float_as_int(tris[4 * (size_t)(uint32_t)s.best_leaf].w);
    }
    if (take) {
        s.best_t = t;
        s.best_leaf = ~s.pend;
    }
}

// One node of the query (s.node >= 0): its four box tests, the leaf children hit tested
// or held back, the internal children still in range visited nearest first (the others
// pushed, farthest first); s.node becomes the next node, or -1 when the walk ends.
template <bool ANY, int SHORT, int TBK, class VIS>
__device__ __forceinline__ void trav4_visit(Trav4& s, const float4* __restrict__ nodes, const float4* __restrict__ tris,
                                            int* stack, int* spill, int lane, VIS& vis, TopNodes top) {
    vis.node();
    // 32-bit byte offsets from the tree's base (the build keeps 128 x nodes < 2^32), so
    // each load is base + one 32-bit register
    const uint32_t nb = (uint32_t)s.node * 128u;
    const uint32_t ax = nb | s.br.onx, ay = nb | s.br.ony, az = nb | s.br.onz;
    float4 nx, ny, nz, fx, fy, fz;
    int4 cr;
    // the empty asm ends the LDS branch differently from the global one: otherwise the
    // compiler sinks the two sets of loads into one generic (flat) load of a selected
    // address, which is slower for the global case
    if (nb < top.bytes) {   // staged top levels: same byte offsets from the LDS copy
        const char* lb = reinterpret_cast<const char*>(top.lds);
        nx = *reinterpret_cast<const float4*>(lb + ax);
        ny = *reinterpret_cast<const float4*>(lb + ay);
        nz = *reinterpret_cast<const float4*>(lb + az);
        fx = *reinterpret_cast<const float4*>(lb + (ax ^ FAR_X));
        fy = *reinterpret_cast<const float4*>(lb + (ay ^ FAR_Y));
        fz = *reinterpret_cast<const float4*>(lb + (az ^ FAR_Z));
        cr = *reinterpret_cast<const int4*>(lb + (nb + 96u));
        asm volatile("");
    } else {
        const char* base = reinterpret_cast<const char*>(nodes);
        nx = *reinterpret_cast<const float4*>(base + ax);
        ny = *reinterpret_cast<const float4*>(base + ay);
        nz = *reinterpret_cast<const float4*>(base + az);
        fx = *reinterpret_cast<const float4*>(base + (ax ^ FAR_X));
        fy = *reinterpret_cast<const float4*>(base + (ay ^ FAR_Y));
        fz = *reinterpret_cast<const float4*>(base + (az ^ FAR_Z));
        cr = *reinterpret_cast<const int4*>(base + (nb + 96u));
    }
    // The outcomes as lane masks: the choice of leaves and children is scalar work beside the
    // vector unit, which bounds the loop.  With it, the packed sort keys and one branch for
    // spilled stack entries, the launch of first bounces (256 x 256 x 64, 50k triangles) issues
    // 196 M vector instructions instead of 244 M, and the three bounces take 767 us instead of
    // 812; the loads of whole nodes by 64 lanes apart keep the address unit 75 % busy beside it.
    float tn[4];
    uint64_t h0 = __ballot(box4_hit(s.br, nx.x, ny.x, nz.x, fx.x, fy.x, fz.x, s.tmin, s.best_t, tn[0]));
    uint64_t h1 = __ballot(box4_hit(s.br, nx.y, ny.y, nz.y, fx.y, fy.y, fz.y, s.tmin, s.best_t, tn[1]));
    uint64_t h2 = __ballot(box4_hit(s.br, nx.z, ny.z, nz.z, fx.z, fy.z, fz.z, s.tmin, s.best_t, tn[2]));
    uint64_t h3 = __ballot(box4_hit(s.br, nx.w, ny.w, nz.w, fx.w, fy.w, fz.w, s.tmin, s.best_t, tn[3]));
    // Leaf children whose box is hit.  A lane holds one of them back (pend); all lanes that
    // hold one test it together once a lane has found a second.  Tested as they came, the
    // loop ran 0.82 triangle tests per node with 9 of 64 lanes in each (incoherent rays);
    // held back, the closest hits of 256 x 256 x 64 in the 50k-triangle corner beyond the camera's
    // take 797 us instead of 839, at a bound on the distance that is a step late.  (Two held
    // per lane: 908; a list per lane in LDS and leaves on the stack were slower still.)
    const uint64_t f0 = __ballot(cr.x < 0), f1 = __ballot(cr.y < 0), f2 = __ballot(cr.z < 0), f3 = __ballot(cr.w < 0);
    uint64_t l0 = h0 & f0, l1 = h1 & f1, l2 = h2 & f2, l3 = h3 & f3;
    h0 &= ~f0, h1 &= ~f1, h2 &= ~f2, h3 &= ~f3;
    if ((l0 | l1 | l2 | l3) != 0ull) {
        // the first leaf of the list, removed from it in the lanes `on`
        auto next = [&](uint64_t on) {
            const int leaf = lane_of(l0) ? cr.x : (lane_of(l1) ? cr.y : (lane_of(l2) ? cr.z : cr.w));
            l3 &= ~(on & ~(l0 | l1 | l2));
            l2 &= ~(on & ~(l0 | l1));
            l1 &= ~(on & ~l0);
            l0 &= ~on;
            return leaf;
        };
        const uint64_t free = __ballot(s.pend >= 0) & (l0 | l1 | l2 | l3);
        const int leaf = next(free);
        s.pend = lane_of(free) ? leaf : s.pend;
        if ((l0 | l1 | l2 | l3) != 0ull) {
#pragma clang loop unroll(disable)
            do {
                if (s.pend < 0) trav4_leaf<ANY>(s, tris, vis);
                const uint64_t more = l0 | l1 | l2 | l3;
                const int nl = next(~0ull);
                s.pend = lane_of(more) ? nl : 0;
            } while ((l0 | l1 | l2 | l3) != 0ull);
            h0 &= __ballot(tn[0] <= s.best_t), h1 &= __ballot(tn[1] <= s.best_t);
            h2 &= __ballot(tn[2] <= s.best_t), h3 &= __ballot(tn[3] <= s.best_t);
        }
    }
    // internal children still in range: the slot number in the two lowest bits of the entry
    // distance (positive, so ordered as an integer), sorted by minima and maxima; a node's
    // internal children are its first slots, numbered one after the other, so the slot
    // gives the child.  For any hit no order is worth its instructions: the slots' own (with an
    // environment map, 640 x 360 x 16 of the 50k-triangle corner, 2158 us sorted, 2099 not; the same
    // choice from the lane masks alone 2110).  For the closest hit it is: only the nearest put
    // first, 256 x 256 x 64 took 1586 us instead of 1573.
    uint32_t k0 = lane_of(h0) ? (__float_as_uint(tn[0]) & ~3u) : ~0u, k1 = lane_of(h1) ? (__float_as_uint(tn[1]) & ~3u) | 1u : ~0u;
    uint32_t k2 = lane_of(h2) ? (__float_as_uint(tn[2]) & ~3u) | 2u : ~0u, k3 = lane_of(h3) ? (__float_as_uint(tn[3]) & ~3u) | 3u : ~0u;
    if constexpr (ANY) {
        const uint32_t f = k0 != ~0u ? k0 : (k1 != ~0u ? k1 : (k2 != ~0u ? k2 : k3));
        if (k0 == ~0u) {   // the first child in range moves to the front, out of its slot
            if (k1 != ~0u) k1 = ~0u;
            else if (k2 != ~0u) k2 = ~0u;
            else k3 = ~0u;
        }
        k0 = f;
    } else {
        sort2(k0, k1);
        sort2(k2, k3);
        sort2(k0, k2);
        sort2(k1, k3);
        sort2(k1, k2);
    }
    if (ANY && s.best_leaf >= 0) {   // any hit ends the query
        s.node = -1;
    } else if (k0 != ~0u) {
        s.node = cr.x + (int)(k0 & 3u);
        // the others pushed, farthest first: each is written to LDS, at its place, or at the
        // lane's extra entry SHORT once the LDS part is full (a write that is not kept is
        // overwritten or never read); one branch for the rare ones that belong in global memory
        const bool p3 = k3 != ~0u, p2 = k2 != ~0u, p1 = k1 != ~0u;
        const int r3 = cr.x + (int)(k3 & 3u), r2 = cr.x + (int)(k2 & 3u), r1 = cr.x + (int)(k1 & 3u);
        const int a3 = s.sp, a2 = a3 + (p3 ? 1 : 0), a1 = a2 + (p2 ? 1 : 0), sp = a1 + (p1 ? 1 : 0);
        stack[min(a3, SHORT) * TBK + lane] = r3;
        stack[min(a2, SHORT) * TBK + lane] = r2;
        stack[min(a1, SHORT) * TBK + lane] = r1;
        if constexpr (SHORT < MAX_STACK)
            if (sp > SHORT) {
                if (p3 && a3 >= SHORT && a3 < MAX_STACK) spill[(a3 - SHORT) * TBK + lane] = r3;
                if (p2 && a2 >= SHORT && a2 < MAX_STACK) spill[(a2 - SHORT) * TBK + lane] = r2;
                if (p1 && a1 >= SHORT && a1 < MAX_STACK) spill[(a1 - SHORT) * TBK + lane] = r1;
            }
        s.sp = min(sp, MAX_STACK);
    } else if (s.sp > 0) {
        --s.sp;
        // an LDS read always (clamped index) and a global read only for spilled entries:
        // two plain loads rather than one generic (flat) load
        int nn = stack[min(s.sp, SHORT - 1) * TBK + lane];
        if constexpr (SHORT < MAX_STACK)
            if (s.sp >= SHORT)   // (a relaxed atomic load: the compiler cannot fold it with the
                                 // LDS read into one generic load of a selected address,
                                 // which would wait on every memory counter each pop)
                nn = __hip_atomic_load(&spill[(s.sp - SHORT) * TBK + lane], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WAVEFRONT);
        s.node = nn;
    } else {
        s.node = -1;
    }
}

template <bool ANY, int SHORT, int TBK, class VIS>
__device__ __forceinline__ bool traverse4(const float4* __restrict__ nodes, const float4* __restrict__ tris, V3 o,
                                          V3 d, float tmin, float tmax, int skip, Hit& h, int* stack, int* spill,
                                          int lane, VIS& vis, TopNodes top) {
    Trav4 s;
    trav4_start(s, o, d, tmin, tmax, skip);
    // the only exit is the loop test (node < 0 once the stack is empty or an any-hit
    // query has its hit): with no break inside, the compiler keeps the pop an ordinary
    // branch of the one loop, instead of a nested loop whose lanes wait until every
    // lane of the wave needs a pop
    while (s.node >= 0) trav4_visit<ANY, SHORT, TBK>(s, nodes, tris, stack, spill, lane, vis, top);
    if (s.pend < 0 && !(ANY && s.best_leaf >= 0)) trav4_leaf<ANY>(s, tris, vis);
    // the barycentrics of the hit: the same test on its triangle again (same arithmetic,
    // same bits), which keeps them out of the loop's registers
    float bb1 = 0.f, bb2 = 0.f;
    int best_prim = -1;
    if (s.best_leaf >= 0) {
        V3 v0, v1, v2;
        load_tri(tris, s.best_leaf, v0, v1, v2, best_prim);
        wt_intersect(s.wr, v0, v1, v2, s.best_t, bb1, bb2);
    }
    h.t = s.best_t;
    h.leaf = s.best_leaf;
    h.prim = best_prim;
    h.b1 = bb1;
    h.b2 = bb2;
    return s.best_leaf >= 0;
}

// closest or any hit on the request's BVH (4-wide when built)
template <bool ANY, int SHORT, int TBK, class VIS>
__device__ __forceinline__ bool trace_ray(const float4* __restrict__ nodes4, const float4* __restrict__ nodes,
                                          const float4* __restrict__ tris, V3 o, V3 d, float tmin, float tmax,
                                          int skip, Hit& h, int* stack, int* spill, int lane, VIS& vis,
                                          TopNodes top = TopNodes{nullptr, 0u}) {
    if (nodes4)
        return traverse4<ANY, SHORT, TBK>(nodes4, tris, o, d, tmin, tmax, skip, h, stack, spill, lane, vis, top);
    return traverse<ANY, SHORT, TBK>(nodes, tris, o, d, tmin, tmax, skip, h, stack, spill, lane, vis);
}

// reference: every triangle in original order, same arithmetic and tie rule
template <bool ANY>
__device__ __forceinline__ bool brute_force(const float4* __restrict__ tris, const int* __restrict__ leaf_of_prim,
                                            int ntri, V3 o, V3 d, float tmin, float tmax, int skip, Hit& h) {
    const WtRay wr = wt_setup(o, d);
    float best_t = tmax;
    int best = -1, best_leaf = -1;
    for (int p = 0; p < ntri; ++p) {
        if (p == skip) continue;
        const int leaf = leaf_of_prim[p];
        V3 v0, v1, v2;
        int prim;
        load_tri(tris, leaf, v0, v1, v2, prim);
        float t;
        // triangles are visited in increasing original index, so on equal t the first wins
        if (wt_hit(wr, v0, v1, v2, t) && t > tmin && t < best_t) {
            best_t = t;
            best = prim;
            best_leaf = leaf;
            if (ANY) break;
        }
    }
    float bb1 = 0.f, bb2 = 0.f;
    if (best_leaf >= 0) {
        V3 v0, v1, v2;
        int prim;
        load_tri(tris, best_leaf, v0, v1, v2, prim);
        wt_intersect(wr, v0, v1, v2, best_t, bb1, bb2);
    }
    h.t = best_t;
    h.leaf = best_leaf;
    h.prim = best;
    h.b1 = bb1;
    h.b2 = bb2;
    return best >= 0;
}

}  // namespace dpcs
