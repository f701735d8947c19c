// Ray launch + stackless BVH traversal + watertight ray-triangle test +
// specular multi-bounce, one lane per ray and 8x8 ray tiles per wavefront (small
// grids: 16 lanes per ray, 2x2 tiles).
#include <type_traits>

#include "sbr_internal.h"
#include "sbr_device.h"

namespace sbr {

namespace {

struct TraceArgs {
    const int32_t *header;   // BVH header: [0] faces, [1] seal
    const BvhNode *nodes;
    const LeafTri *tris;
    int32_t n_nodes;
    int32_t n_tris;
    GridDev g;
    double o[3];
    double rot[9];
    int32_t *tri;
    float *t;
    float *u;
    float *v;
    uint8_t *flags;
    unsigned long long *counters;
};

__device__ __forceinline__ float sel3(float3 p, int k) { return k == 0 ? p.x : (k == 1 ? p.y : p.z); }

struct Shear {
    int kx, ky, kz;
    float sx, sy, sz;
};

// Watertight ray/triangle intersection (Woop, Benthin, Wald, JCGT 2013),
// two-sided, inclusive edges.  Returns t and the barycentric weights.
__device__ __forceinline__ bool wt_hit(const Shear &sh, float3 o, float3 a, float3 b, float3 c,
                                       float &t, float &b0, float &b1, float &b2) {
    float3 A = make_float3(a.x - o.x, a.y - o.y, a.z - o.z);
    float3 B = make_float3(b.x - o.x, b.y - o.y, b.z - o.z);
    float3 C = make_float3(c.x - o.x, c.y - o.y, c.z - o.z);
    float Az = sel3(A, sh.kz), Bz = sel3(B, sh.kz), Cz = sel3(C, sh.kz);
    float Ax = fmaf(-sh.sx, Az, sel3(A, sh.kx));
    float Ay = fmaf(-sh.sy, Az, sel3(A, sh.ky));
    float Bx = fmaf(-sh.sx, Bz, sel3(B, sh.kx));
    float By = fmaf(-sh.sy, Bz, sel3(B, sh.ky));
    float Cx = fmaf(-sh.sx, Cz, sel3(C, sh.kx));
    float Cy = fmaf(-sh.sy, Cz, sel3(C, sh.ky));
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    float det = U + V + W;
    if (det == 0.0f) return false;
    float T = U * (sh.sz * Az) + V * (sh.sz * Bz) + W * (sh.sz * Cz);
    float inv = 1.0f / det;
    t = T * inv;
    b0 = U * inv;
    b1 = V * inv;
    b2 = W * inv;
    return true;
}

__device__ __forceinline__ Shear make_shear(float3 d) {
    Shear sh;
    float ax = fabsf(d.x), ay = fabsf(d.y), az = fabsf(d.z);
    sh.kz = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
    sh.kx = sh.kz == 2 ? 0 : sh.kz + 1;
    sh.ky = sh.kx == 2 ? 0 : sh.kx + 1;
    float dz = sel3(d, sh.kz);
    if (dz < 0.0f) {
        int tmp = sh.kx;
        sh.kx = sh.ky;
        sh.ky = tmp;
    }
    sh.sx = sel3(d, sh.kx) / dz;
    sh.sy = sel3(d, sh.ky) / dz;
    sh.sz = 1.0f / dz;
    return sh;
}

// ---- the stackless walk ------------------------------------------------------
// A node is 16 bytes (half of what its box takes in floats): it comes as 16-bit
// steps from the mesh's origin, so per query the ray's slab constants are scaled
// once, t = q (step / d) + (origin - o) / d, and a test is 6 conversions, 6 fused
// multiply-adds and the minima and maxima, about 30 instructions.  What bounds a
// large grid are these and the triangle tests of the few lanes at a leaf; a
// small one the latency of the loads.  The next node is loaded as soon as it is
// known, before a leaf's test, and the triangle in one piece: 20480 faces at
// 512^2 rays and 3 bounces 230 -> 199 us, 200k at 1024^2 with occlusion 346 -> 281
// us, 51200 at 2048^2 and 4 bounces 904 -> 868 us.
struct Slab {
    float3 m, b;   // step / d, (origin - o) / d
};
// zero direction components are replaced by tiny values
__device__ __forceinline__ Slab make_slab(float3 o, float3 d, float3 org, float3 step) {
    float3 id;
    id.x = 1.0f / (fabsf(d.x) > 1e-30f ? d.x : copysignf(1e-30f, d.x));
    id.y = 1.0f / (fabsf(d.y) > 1e-30f ? d.y : copysignf(1e-30f, d.y));
    id.z = 1.0f / (fabsf(d.z) > 1e-30f ? d.z : copysignf(1e-30f, d.z));
    Slab s;
    s.m = make_float3(step.x * id.x, step.y * id.y, step.z * id.z);
    s.b = make_float3((org.x - o.x) * id.x, (org.y - o.y) * id.y, (org.z - o.z) * id.z);
    return s;
}
__device__ __forceinline__ bool box_hit(const BvhNode &nd, const Slab &s, float tlim) {
    const float tx0 = fmaf((float)(nd.x & 0xffffu), s.m.x, s.b.x), tx1 = fmaf((float)(nd.x >> 16), s.m.x, s.b.x);
    const float ty0 = fmaf((float)(nd.y & 0xffffu), s.m.y, s.b.y), ty1 = fmaf((float)(nd.y >> 16), s.m.y, s.b.y);
    const float tz0 = fmaf((float)(nd.z & 0xffffu), s.m.z, s.b.z), tz1 = fmaf((float)(nd.z >> 16), s.m.z, s.b.z);
    const float tn = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fmaxf(fminf(tz0, tz1), 0.0f));
    float tf = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fmaxf(tz0, tz1));
    tf *= 1.0000005f;
    return tn <= tf && tn <= tlim;
}

// ---- several lanes per ray ----------------------------------------------------
// A grid of a few thousand rays is bound by the latency of the walk's steps (one
// wavefront per SIMD or fewer, about 1000 clocks per node with a leaf's test
// among the 64 lanes).  There L = 16 lanes take a ray: each walks a subtree, a
// hit of one culls for all, and the hits are merged at the end, with the results
// of the single walk.  The extra nodes (each lane's own way down, less culling)
// make it slower once the chip is full: 14 faces at 64^2 rays 32.8 -> 18.3 us,
// at 192^2 26.8 -> 22.0; 20000 faces at 64^2 84 -> 64 us, 128^2 80 -> 64, 160^2 79
// -> 68, 192^2 81 -> 83, 256^2 78 -> 143; 1000 faces at 128^2 38.6 -> 38.5, 192^2
// 41 -> 50.  The line is at 128^2.  (4 lanes: 28, 77 and 80 us at the first,
// third and fourth of these.)
constexpr long long kSplitRays = 128 * 128;
constexpr int kSplitLanes = 16;

// x of a lane of the other half of the 2 M lanes around, for M = 1, 2, 4, 8 in
// turn: lanes of a half hold equal values by then, so that mirrors will do.
template <int M>
__device__ __forceinline__ int other_half(int x) {
    constexpr int ctrl = M == 1 ? 0xb1     // quad_perm 1,0,3,2
                         : M == 2 ? 0x4e   // quad_perm 2,3,0,1
                         : M == 4 ? 0x141  // row_half_mirror
                                  : 0x140; // row_mirror
    return __builtin_amdgcn_update_dpp(x, x, ctrl, 0xf, 0xf, false);
}
template <int M>
__device__ __forceinline__ float other_half(float x) {
    return __int_as_float(other_half<M>(__float_as_int(x)));
}
// f<M>() for M = 1, 2, .. below L
template <int L, int M = 1, class F>
__device__ __forceinline__ void over_lanes(F &&f) {
    if constexpr (M < L) {
        f(std::integral_constant<int, M>{});
        over_lanes<L, 2 * M>(f);
    }
}

// The part of the depth-first node order that lane `sub` of L walks: the
// subtrees L leaves of the top log2 L levels hold.  A leaf met on the way down
// goes to the lowest of its lanes.
template <int L>
__device__ __forceinline__ void lane_range(const BvhNode *nodes, int n_nodes, int sub, int &first, int &last) {
    first = 0;
    last = n_nodes;
#pragma unroll
    for (int m = L / 2; m >= 1; m >>= 1) {
        if (first >= last) break;
        const uint32_t link = nodes[first].link;
        if (link & kLeafBit) {
            if (sub & (2 * m - 1)) last = first;
            break;
        }
        const int left = first + 1;   // an inner node's children follow it
        if (left >= last) break;
        const uint32_t ll = nodes[left].link;
        const int right = min((ll & kLeafBit) ? left + 1 : max((int)ll, left + 1), last);
        if (sub & m) first = right;
        else first = left, last = right;
    }
}

// Any hit of a triangle other than `self` at t in (tmin, tmax) along the unit
// direction s from x: the occlusion test of a return segment.  Same stackless
// walk as the closest-hit query, leaving at the first accepted hit of the ray's
// lanes.
template <int L>
__device__ bool any_hit(const TraceArgs &a, int first, int last, float3 x, float3 s, float tmin, float tmax, int self) {
    const Shear sh = make_shear(s);
    const float *h = reinterpret_cast<const float *>(a.header);
    const Slab sl = make_slab(x, s, make_float3(h[4], h[5], h[6]), make_float3(h[8], h[9], h[10]));
    int i = first;
    bool hit = false;
    BvhNode next = {};
    if (i < last) next = a.nodes[i];
    auto visit = [&]() {
        const BvhNode nd = next;
        const bool leaf = (nd.link & kLeafBit) != 0u;
        const bool in = box_hit(nd, sl, tmax);
        i = in || leaf ? i + 1 : max((int)nd.link, i + 1);
        if (i < last) next = a.nodes[i];
        const uint32_t slot = nd.link & ~kLeafBit;
        if (in && leaf && slot < (uint32_t)a.n_tris) {
            const LeafTri lt = a.tris[slot];
            float th, c0, c1, c2;
            const bool on = wt_hit(sh, x, make_float3(lt.a.x, lt.a.y, lt.a.z), make_float3(lt.b.x, lt.b.y, lt.b.z),
                                   make_float3(lt.c.x, lt.c.y, lt.c.z), th, c0, c1, c2);
            if (on && __float_as_int(lt.a.w) != self && th > tmin && th < tmax) hit = true;
        }
    };
    if (L == 1) {
        while (i < last && !hit) visit();
        return hit;
    }
    bool any = false;   // of the ray's lanes
    while (__ballot(i < last && !any)) {
        if (i < last && !any) visit();
        if (__ballot(hit && !any)) {
            int v = hit ? 1 : 0;
            over_lanes<L>([&](auto m) { v |= other_half<decltype(m)::value>(v); });
            any = v != 0;
        }
    }
    return any;
}

template <bool COUNT, bool SHADOW, int L>
__global__ __launch_bounds__(256) void k_trace(TraceArgs a) {
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    constexpr int W = L == 1 ? 8 : 2;   // W x W rays per wavefront
    static_assert(W * W * L == 64, "lanes per ray");
    const int tile = gid >> 6, sub = gid & (L - 1), l = (gid & 63) / L;
    const int tiles_x = (a.g.nx + W - 1) / W;
    const int ix = (tile % tiles_x) * W + l % W;
    const int iy = (tile / tiles_x) * W + l / W;
    const bool active = ix < a.g.nx && iy < a.g.ny;
    // a buffer that no BUILD for this face count has sealed is never walked:
    // every ray misses
    const int n_nodes = (a.n_nodes > 0 && a.header[1] == kBvhMagic && a.header[0] == a.n_tris) ? a.n_nodes : 0;
    const float *hd = reinterpret_cast<const float *>(a.header);
    float3 org = make_float3(0.f, 0.f, 0.f), step = org;   // frame of the nodes' boxes
    if (n_nodes > 0) {
        org = make_float3(hd[4], hd[5], hd[6]);
        step = make_float3(hd[8], hd[9], hd[10]);
    }
    int first, last;
    lane_range<L>(a.nodes, n_nodes, sub, first, last);
    const bool lead = sub == 0;
    unsigned long long n_q = 0, n_node = 0, n_tri = 0;
    if (active) {
        const size_t R = (size_t)a.g.nx * a.g.ny;
        const size_t r = (size_t)iy * a.g.nx + ix;
        // ray of the grid, formed in double and rounded once
        double dr[3], dw_unused;
        grid_dir_local(a.g, ix, iy, dr, &dw_unused);
        float3 d, o;
        d.x = (float)(a.rot[0] * dr[0] + a.rot[1] * dr[1] + a.rot[2] * dr[2]);
        d.y = (float)(a.rot[3] * dr[0] + a.rot[4] * dr[1] + a.rot[5] * dr[2]);
        d.z = (float)(a.rot[6] * dr[0] + a.rot[7] * dr[1] + a.rot[8] * dr[2]);
        o = make_float3((float)a.o[0], (float)a.o[1], (float)a.o[2]);
        const float3 o0 = o;   // array centre: where every return ends
        const float tmin = (float)a.g.t_min;
        int prev = -1;
        float Lprev = 0.0f;
        uint8_t anc = 0;
        bool alive = true;
        for (int k = 0; k < a.g.K; k++) {
            const size_t slot = (size_t)k * R + r;
            if (!alive) {
                if (lead) {
                    a.tri[slot] = -1;
                    a.t[slot] = 0.0f;
                    a.u[slot] = 0.0f;
                    a.v[slot] = 0.0f;
                    a.flags[slot] = 0;
                }
                continue;
            }
            n_q += lead;
            // per-ray shear constants of the watertight test
            const Shear sh = make_shear(d);
            const Slab sl = make_slab(o, d, org, step);
            int best = -1, bslot = -1;
            float t1 = INFINITY, t2 = INFINITY, bb0 = 0.f, bb1 = 0.f, bb2 = 0.f;
            float tlim = INFINITY;   // box cull limit: best t plus the tie margin
            int i = first;
            BvhNode next = {};
            if (i < last) next = a.nodes[i];
            auto visit = [&]() -> bool {   // whether a closer hit was found
                const BvhNode nd = next;
                if (COUNT) n_node++;
                const bool leaf = (nd.link & kLeafBit) != 0u;
                const bool in = box_hit(nd, sl, tlim);
                // left child, or the escape; escape links always point forward,
                // and the guard keeps the walk finite even for a corrupted buffer
                i = in || leaf ? i + 1 : max((int)nd.link, i + 1);
                if (i < last) next = a.nodes[i];   // in flight during the leaf's test
                const uint32_t slot = nd.link & ~kLeafBit;
                if (!in || !leaf || slot >= (uint32_t)a.n_tris) return false;
                const LeafTri lt = a.tris[slot];
                const int fid = __float_as_int(lt.a.w);
                if (COUNT) n_tri++;
                float th, c0, c1, c2;
                const bool on = wt_hit(sh, o, make_float3(lt.a.x, lt.a.y, lt.a.z), make_float3(lt.b.x, lt.b.y, lt.b.z),
                                       make_float3(lt.c.x, lt.c.y, lt.c.z), th, c0, c1, c2);
                // fid: a face of this mesh, and not the one the ray starts on
                if (on && th > tmin && fid != prev && (unsigned)fid < (unsigned)a.n_tris) {
                    if (th < t1 || (th == t1 && fid < best)) {
                        t2 = t1;
                        t1 = th;
                        best = fid;
                        bslot = (int)slot;
                        bb0 = c0;
                        bb1 = c1;
                        bb2 = c2;
                        return true;
                    }
                    if (th < t2) t2 = th;
                }
                return false;
            };
            if (L == 1) {
                while (i < last)
                    if (visit()) tlim = t1 + 1e-6f * fmaxf(1.0f, Lprev + t1);
            } else {
                // lanes that are done stay, so that a hit of one culls for all
                while (__ballot(i < last)) {
                    bool closer = false;
                    if (i < last) closer = visit();
                    if (__ballot(closer)) {
                        float t = t1;
                        over_lanes<L>([&](auto m) { t = fminf(t, other_half<decltype(m)::value>(t)); });
                        tlim = t + 1e-6f * fmaxf(1.0f, Lprev + t);
                    }
                }
                // the ray's closest hit (of equal ones the lowest face), and
                // the second closest, of all its lanes
                over_lanes<L>([&](auto m) {
                    constexpr int M = decltype(m)::value;
                    const float s1 = other_half<M>(t1), s2 = other_half<M>(t2), c0 = other_half<M>(bb0),
                                c1 = other_half<M>(bb1), c2 = other_half<M>(bb2);
                    const int sb = other_half<M>(best), ss = other_half<M>(bslot);
                    t2 = fminf(fmaxf(t1, s1), fminf(t2, s2));
                    if (s1 < t1 || (s1 == t1 && sb >= 0 && (best < 0 || sb < best))) {
                        t1 = s1;
                        best = sb;
                        bslot = ss;
                        bb0 = c0;
                        bb1 = c1;
                        bb2 = c2;
                    }
                });
            }
            if (best < 0) {
                alive = false;
                if (lead) {
                    a.tri[slot] = -1;
                    a.t[slot] = 0.0f;
                    a.u[slot] = 0.0f;
                    a.v[slot] = 0.0f;
                    a.flags[slot] = 0;
                }
                continue;
            }
            const LeafTri lt = a.tris[bslot];
            float3 v0 = make_float3(lt.a.x, lt.a.y, lt.a.z);
            float3 v1 = make_float3(lt.b.x, lt.b.y, lt.b.z);
            float3 v2 = make_float3(lt.c.x, lt.c.y, lt.c.z);
            float3 e1 = make_float3(v1.x - v0.x, v1.y - v0.y, v1.z - v0.z);
            float3 e2 = make_float3(v2.x - v0.x, v2.y - v0.y, v2.z - v0.z);
            float3 N = make_float3(e1.y * e2.z - e1.z * e2.y, e1.z * e2.x - e1.x * e2.z,
                                   e1.x * e2.y - e1.y * e2.x);
            float nl = sqrtf(N.x * N.x + N.y * N.y + N.z * N.z);
            float3 nh = make_float3(N.x / nl, N.y / nl, N.z / nl);
            float dn = d.x * nh.x + d.y * nh.y + d.z * nh.z;
            float Lk = Lprev + t1;
            float delta = 1e-6f * fmaxf(1.0f, Lk);
            // distance to the line of the edge opposite vertex i: b_i |N| / |e_i|
            float3 e0 = make_float3(v2.x - v1.x, v2.y - v1.y, v2.z - v1.z);
            float l0 = sqrtf(e0.x * e0.x + e0.y * e0.y + e0.z * e0.z);
            float l1 = sqrtf(e2.x * e2.x + e2.y * e2.y + e2.z * e2.z);
            float l2 = sqrtf(e1.x * e1.x + e1.y * e1.y + e1.z * e1.z);
            float de = fminf(fabsf(bb0) * nl / l0, fminf(fabsf(bb1) * nl / l1, fabsf(bb2) * nl / l2));
            uint8_t fl = anc ? SBR_HIT_PARENT : 0;
            if (de < delta) fl |= SBR_HIT_EDGE;
            if (t2 - t1 < delta) fl |= SBR_HIT_TIE;
            if (fabsf(dn) < 1e-6f) fl |= SBR_HIT_GRAZE;
            if (t1 < 2.0f * tmin) fl |= SBR_HIT_TMIN;
            anc |= fl;
            // the hit point (barycentric, lies on the face): the return's start
            // and the next bounce's origin
            o = make_float3(bb0 * v0.x + bb1 * v1.x + bb2 * v2.x, bb0 * v0.y + bb1 * v1.y + bb2 * v2.y,
                            bb0 * v0.z + bb1 * v1.z + bb2 * v2.z);
            if (SHADOW && k > 0) {
                const float3 q = make_float3(o0.x - o.x, o0.y - o.y, o0.z - o.z);
                const float D = sqrtf(q.x * q.x + q.y * q.y + q.z * q.z);
                const float3 sd = make_float3(q.x / D, q.y / D, q.z / D);
                if (any_hit<L>(a, first, last, o, sd, tmin, D - tmin, best)) fl |= SBR_HIT_OCCLUDED;
            }
            if (lead) {
                a.tri[slot] = best;
                a.t[slot] = t1;
                a.u[slot] = bb1;
                a.v[slot] = bb2;
                a.flags[slot] = fl;
            }
            d = make_float3(d.x - 2.0f * dn * nh.x, d.y - 2.0f * dn * nh.y, d.z - 2.0f * dn * nh.z);
            float dl = 1.0f / sqrtf(d.x * d.x + d.y * d.y + d.z * d.z);
            d = make_float3(d.x * dl, d.y * dl, d.z * dl);
            prev = best;
            Lprev = Lk;
        }
    }
    if (a.counters) {
        // wavefront sums, one atomic per wave and counter
        for (int off = 32; off >= 1; off >>= 1) {
            n_q += __shfl_xor(n_q, off);
            n_node += __shfl_xor(n_node, off);
            n_tri += __shfl_xor(n_tri, off);
        }
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(&a.counters[0], n_q);
            if (COUNT) {
                atomicAdd(&a.counters[1], n_node);
                atomicAdd(&a.counters[2], n_tri);
            }
        }
    }
}

}  // namespace

template <int L>
static void launch_walk(const TraceArgs &a, bool shadow, hipStream_t st) {
    constexpr int W = L == 1 ? 8 : 2;
    const long long tiles = (long long)((a.g.nx + W - 1) / W) * ((a.g.ny + W - 1) / W);
    const dim3 blocks((unsigned)((tiles + 3) / 4));
    if (a.counters && shadow) hipLaunchKernelGGL((k_trace<true, true, L>), blocks, dim3(256), 0, st, a);
    else if (a.counters) hipLaunchKernelGGL((k_trace<true, false, L>), blocks, dim3(256), 0, st, a);
    else if (shadow) hipLaunchKernelGGL((k_trace<false, true, L>), blocks, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_trace<false, false, L>), blocks, dim3(256), 0, st, a);
}

int trace_launch(const sbr_mesh *m, const void *bvh, const RadarDev &rd, const GridDev &gd,
                 const sbr_hits *h, uint64_t *counters, hipStream_t st) {
    BvhView bv = bvh_view(const_cast<void *>(bvh), m->nf, nullptr);
    TraceArgs a;
    a.header = bv.header;
    a.nodes = bv.nodes;
    a.tris = bv.tris;
    a.n_nodes = m->nf > 0 ? bv.n_nodes : 0;
    a.n_tris = m->nf;
    a.g = gd;
    for (int i = 0; i < 3; i++) a.o[i] = rd.o[i];
    for (int i = 0; i < 9; i++) a.rot[i] = rd.rot[i];
    a.tri = h->tri;
    a.t = h->t;
    a.u = h->u;
    a.v = h->v;
    a.flags = h->flags;
    a.counters = reinterpret_cast<unsigned long long *>(counters);
    const bool shadow = (gd.options & SBR_RAYS_SHADOW) != 0;
    ProfScope ps(kProfTrace, st);
    if ((long long)gd.nx * gd.ny <= kSplitRays) launch_walk<kSplitLanes>(a, shadow, st);
    else launch_walk<1>(a, shadow, st);
    SBR_LAUNCHED();
    return SBR_OK;
}

}  // namespace sbr
