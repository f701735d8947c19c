// Linear BVH over the triangle mesh: Morton codes, LSD radix sort, binary radix
// tree (Karras, HPG 2012), depth-first layout with escape links for stackless
// traversal, boxes by range unions over the sorted leaves.  Refit reuses the tree.
#include "sbr_internal.h"

namespace sbr {

namespace {

constexpr int kThreads = 256;
constexpr int kSortThreads = 1024;     // keys per step of a sort block
constexpr int kSortBlocks = 1024;      // at most so many sort blocks: larger meshes take more steps

__device__ __forceinline__ uint32_t f2ord(float f) {
    uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float ord2f(uint32_t u) {
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

__device__ __forceinline__ float3 load_vert(const float *v, int i) {
    return make_float3(v[3 * i], v[3 * i + 1], v[3 * i + 2]);
}

// Whether a refit may follow the buffer: sealed by a BUILD for n faces.
__device__ __forceinline__ bool sealed(const BvhView &bv) {
    return bv.header[1] == kBvhMagic && bv.header[0] == bv.n;
}

struct Tri {
    float3 a, b, c;
};
__device__ __forceinline__ Tri load_tri(const float *verts, const int32_t *faces, int f) {
    return {load_vert(verts, faces[3 * f]), load_vert(verts, faces[3 * f + 1]), load_vert(verts, faces[3 * f + 2])};
}
__device__ __forceinline__ float3 centroid(const Tri &t) {
    return make_float3((t.a.x + t.b.x + t.c.x) * (1.0f / 3.0f), (t.a.y + t.b.y + t.c.y) * (1.0f / 3.0f),
                       (t.a.z + t.b.z + t.c.z) * (1.0f / 3.0f));
}
__device__ __forceinline__ float min3(float a, float b, float c) { return fminf(a, fminf(b, c)); }
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(a, fmaxf(b, c)); }

// Bounds as ordered integers: [0..2] minima and [3..5] maxima of the
// centroids, [6..8] and [9..11] of the vertices.
constexpr int kBoundsWords = 12;
__device__ __forceinline__ bool is_min(int q) { return q % 6 < 3; }
__device__ __forceinline__ uint32_t bound_of(int q, uint32_t a, uint32_t b) { return is_min(q) ? min(a, b) : max(a, b); }

// Partial bounds of the block's share of the faces (bv.part[block]); in a build
// also clears the sort's later histograms, in a refit leaves a buffer alone
// that no build for this face count has sealed.
__global__ __launch_bounds__(kThreads) void k_bounds(const float *verts, const int32_t *faces, int nf, BvhView bv,
                                                     int build, uint32_t *hist, int nhist) {
    __shared__ uint32_t red[kThreads / 64][kBoundsWords];
    if (!build && !sealed(bv)) return;
    const int t0 = blockIdx.x * kThreads + threadIdx.x, stride = gridDim.x * kThreads;
    for (int i = t0; i < nhist; i += stride) hist[i] = 0u;
    uint32_t v[kBoundsWords];
#pragma unroll
    for (int q = 0; q < kBoundsWords; q++) v[q] = is_min(q) ? 0xffffffffu : 0u;
    for (int f = t0; f < nf; f += stride) {
        const Tri t = load_tri(verts, faces, f);
        const float3 c = centroid(t);
        const float x[kBoundsWords] = {c.x, c.y, c.z, c.x, c.y, c.z,
                                       min3(t.a.x, t.b.x, t.c.x), min3(t.a.y, t.b.y, t.c.y), min3(t.a.z, t.b.z, t.c.z),
                                       max3(t.a.x, t.b.x, t.c.x), max3(t.a.y, t.b.y, t.c.y), max3(t.a.z, t.b.z, t.c.z)};
#pragma unroll
        for (int q = 0; q < kBoundsWords; q++) v[q] = bound_of(q, v[q], f2ord(x[q]));
    }
#pragma unroll
    for (int q = 0; q < kBoundsWords; q++) {
        for (int off = 32; off >= 1; off >>= 1) v[q] = bound_of(q, v[q], (uint32_t)__shfl_xor((int)v[q], off));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < kBoundsWords) {
        uint32_t m = red[0][threadIdx.x];
        for (int w = 1; w < kThreads / 64; w++) m = bound_of(threadIdx.x, m, red[w][threadIdx.x]);
        bv.part[kBoundsWords * blockIdx.x + threadIdx.x] = m;
    }
}

// Six bounds (words first .. first + 5 of the partials) of all blocks, by the
// first kBoundsBlocks threads of a block; every thread calls it.
__device__ __forceinline__ void all_bounds(const uint32_t *part, int nparts, int first, uint32_t (&sh)[4][6],
                                           float (&lo)[3], float (&hi)[3]) {
    const int t = threadIdx.x;
    if (t < kBoundsBlocks) {
#pragma unroll
        for (int q = 0; q < 6; q++) {
            uint32_t v = t < nparts ? part[kBoundsWords * t + first + q] : is_min(q) ? 0xffffffffu : 0u;
            for (int off = 32; off >= 1; off >>= 1) v = bound_of(q, v, (uint32_t)__shfl_xor((int)v, off));
            if ((t & 63) == 0) sh[t >> 6][q] = v;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; q++) {
        lo[q] = ord2f(min(min(sh[0][q], sh[1][q]), min(sh[2][q], sh[3][q])));
        hi[q] = ord2f(max(max(sh[0][3 + q], sh[1][3 + q]), max(sh[2][3 + q], sh[3][3 + q])));
    }
}

__device__ __forceinline__ uint32_t expand_bits10(uint32_t v) {
    v = (v * 0x00010001u) & 0xFF0000FFu;
    v = (v * 0x00000101u) & 0x0F00F00Fu;
    v = (v * 0x00000011u) & 0xC30C30C3u;
    v = (v * 0x00000005u) & 0x49249249u;
    return v;
}

// Morton codes of the block's tile of faces, and the tile's histogram of their
// lowest digit (the first sort pass).
__global__ __launch_bounds__(kSortThreads) void k_morton(const float *verts, const int32_t *faces, int nf,
                                                         const uint32_t *part, int nparts, uint32_t *keys,
                                                         uint32_t *hist, int steps) {
    __shared__ uint32_t red[kBoundsBlocks / 64][6];
    __shared__ uint32_t h[256];
    const int t = threadIdx.x;
    if (t < 256) h[t] = 0u;
    float lo[3], ext[3];
    all_bounds(part, nparts, 0, red, lo, ext);
    for (int q = 0; q < 3; q++) ext[q] -= lo[q];
    for (int s = 0; s < steps; s++) {
        const int f = (blockIdx.x * steps + s) * kSortThreads + t;
        if (f >= nf) break;
        const float3 cc = centroid(load_tri(verts, faces, f));
        const float c[3] = {cc.x, cc.y, cc.z};
        uint32_t q[3];
        for (int i = 0; i < 3; i++) {
            float x = ext[i] > 0.0f ? (c[i] - lo[i]) / ext[i] : 0.5f;
            x = fminf(fmaxf(x * 1024.0f, 0.0f), 1023.0f);
            q[i] = (uint32_t)x;
        }
        const uint32_t key = (expand_bits10(q[0]) << 2) | (expand_bits10(q[1]) << 1) | expand_bits10(q[2]);
        keys[f] = key;
        atomicAdd(&h[key & 255u], 1u);
    }
    __syncthreads();
    if (t < 256) hist[blockIdx.x * 256 + t] = h[t];
}

// One stable pass of the LSD radix sort (8-bit digit).  Each block sums the
// digit counts of all tiles itself (at most 1024 rows of 256, four threads a
// digit) instead of waiting for a scan launch, ranks its tile's keys by wave
// ballots, scatters them, and counts the next digit of each key in the tile it
// goes to (hist_next, cleared beforehand; NULL in the last pass), so a pass is
// one launch: the sort took 12 launches, a third of them a one-block scan of
// 35 us at 200k triangles.  vin = NULL: the identity.
__global__ __launch_bounds__(kSortThreads) void k_sort_pass(const uint32_t *kin, const int32_t *vin, uint32_t *kout,
                                                            int32_t *vout, int n, int shift, const uint32_t *hist,
                                                            uint32_t *hist_next, int steps) {
    constexpr int W = kSortThreads / 64;
    __shared__ uint32_t tot[4][256], bef[4][256], base_d[256], wsum[4];
    __shared__ uint32_t wcnt[W][256];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63, d = t & 255, g = t >> 8;
    const int blk = blockIdx.x, nblk = gridDim.x;
    {
        uint32_t a = 0, b = 0;
#pragma unroll 4
        for (int i = g; i < nblk; i += 4) {
            const uint32_t x = hist[i * 256 + d];
            a += x;
            b += i < blk ? x : 0u;
        }
        tot[g][d] = a;
        bef[g][d] = b;
    }
    __syncthreads();
    uint32_t mine = 0, incl = 0, before = 0;
    if (t < 256) {   // exclusive scan of the digit totals
        mine = tot[0][t] + tot[1][t] + tot[2][t] + tot[3][t];
        before = bef[0][t] + bef[1][t] + bef[2][t] + bef[3][t];
        incl = mine;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)incl, off);
            if (lane >= off) incl += y;
        }
        if (lane == 63) wsum[w] = incl;
    }
    __syncthreads();
    if (t < 256) {
        uint32_t add = 0;
        for (int i = 0; i < w; i++) add += wsum[i];
        base_d[t] = add + incl - mine + before;
    }
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int tile = steps * kSortThreads;
    for (int s = 0; s < steps; s++) {
        for (int i = t; i < W * 256; i += kSortThreads) (&wcnt[0][0])[i] = 0u;
        __syncthreads();
        const int i = blk * tile + s * kSortThreads + t;
        const bool valid = i < n;
        const uint32_t key = valid ? kin[i] : 0u;
        const int32_t val = valid ? (vin ? vin[i] : i) : 0;
        const uint32_t dg = (key >> shift) & 255u;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < 8; b++) {
            const bool bit = (dg >> b) & 1u;
            const uint64_t m = __ballot(valid && bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t rank = __popcll(peers & lt);
        if (valid && rank == 0) wcnt[w][dg] = __popcll(peers);
        __syncthreads();
        uint32_t run = 0;
        if (t < 256) {
            for (int j = 0; j < W; j++) {
                const uint32_t c = wcnt[j][t];
                wcnt[j][t] = run;
                run += c;
            }
        }
        __syncthreads();
        if (valid) {
            const uint32_t pos = base_d[dg] + wcnt[w][dg] + rank;
            kout[pos] = key;
            vout[pos] = val;
            if (hist_next) atomicAdd(&hist_next[(pos / (uint32_t)tile) * 256u + ((key >> (shift + 8)) & 255u)], 1u);
        }
        __syncthreads();
        if (t < 256) base_d[t] += run;
    }
}

// ---- binary radix tree ----------------------------------------------------
__device__ __forceinline__ int prefix_len(const uint32_t *k, int n, int i, int j) {
    if (j < 0 || j >= n) return -1;
    uint32_t a = k[i], b = k[j];
    if (a == b) return 32 + __clz((uint32_t)(i ^ j));
    return __clz(a ^ b);
}

// tree indices: internal nodes 0..n-2, leaf slot i = n-1+i
__global__ void k_karras(const uint32_t *keys, int n, int32_t *parent, int2 *child, int32_t *other) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    int d = prefix_len(keys, n, i, i + 1) > prefix_len(keys, n, i, i - 1) ? 1 : -1;
    int dmin = prefix_len(keys, n, i, i - d);
    int lmax = 2;
    while (prefix_len(keys, n, i, i + lmax * d) > dmin) lmax <<= 1;
    int l = 0;
    for (int t = lmax >> 1; t >= 1; t >>= 1)
        if (prefix_len(keys, n, i, i + (l + t) * d) > dmin) l += t;
    int j = i + l * d;
    int dnode = prefix_len(keys, n, i, j);
    int s = 0;
    for (int div = 2;; div <<= 1) {
        int t = (l + div - 1) / div;
        if (prefix_len(keys, n, i, i + (s + t) * d) > dnode) s += t;
        if (t <= 1) break;
    }
    int g = i + s * d + min(d, 0);
    int lo = min(i, j), hi = max(i, j);
    int left = (lo == g) ? (n - 1 + g) : g;
    int right = (hi == g + 1) ? (n - 1 + g + 1) : g + 1;
    child[i] = make_int2(left, right);
    other[i] = j;
    parent[left] = i;
    parent[right] = i;
    if (i == 0) parent[0] = -1;
}

// depth-first index = 2 * (first leaf) + (left turns on the root path);
// escape = index + subtree size (2 * leaves - 1)
__global__ void k_dfs(int n, const int32_t *parent, const int2 *child, BvhView bv) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= 2 * n - 1) return;
    int first, nleaf;
    if (x >= n - 1) {
        first = x - (n - 1);
        nleaf = 1;
    } else {
        const int j = bv.other[x];
        first = min(x, j);
        nleaf = max(x, j) - first + 1;
    }
    int lefts = 0;
    if (n > 1)
        for (int c = x, p = parent[c]; p >= 0; c = p, p = parent[c]) lefts += child[p].x == c;
    const int di = 2 * first + lefts;
    bv.dfs_of[x] = di;
    bv.nodes[di].link = x >= n - 1 ? kLeafBit | (uint32_t)first : (uint32_t)(di + 2 * nleaf - 1);
}

__device__ __forceinline__ Box empty_box() {
    return {{INFINITY, INFINITY, INFINITY}, {-INFINITY, -INFINITY, -INFINITY}};
}
__device__ __forceinline__ Box unite(const Box &a, const Box &b) {
    Box r;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        r.lo[k] = fminf(a.lo[k], b.lo[k]);
        r.hi[k] = fmaxf(a.hi[k], b.hi[k]);
    }
    return r;
}

// The frame of the nodes' 16-bit boxes: steps of 1/65533 of the vertices'
// bounds per axis, one step of room on either side.
struct Frame {
    float org[3], step[3];
};
__device__ __forceinline__ Frame make_frame(const float (&lo)[3], const float (&hi)[3]) {
    Frame f;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        // flat meshes: steps that still move the coordinates
        const float m = fmaxf(fabsf(lo[k]), fabsf(hi[k]));
        const float ext = fmaxf(hi[k] - lo[k], m * 1e-3f + 1e-20f);
        f.step[k] = ext / 65531.0f;
        f.org[k] = lo[k] - 2.0f * f.step[k];
    }
    return f;
}
// lo rounded down and hi up, each by a full step more than needed: the
// traversal's decoding origin + q step rounds twice where a stored float did not.
__device__ __forceinline__ uint32_t quantize(float lo, float hi, float org, float step) {
    const float a = floorf((lo - org) / step) - 1.0f, b = ceilf((hi - org) / step) + 1.0f;
    const uint32_t qa = (uint32_t)fminf(fmaxf(a, 0.0f), 65535.0f), qb = (uint32_t)fminf(fmaxf(b, 0.0f), 65535.0f);
    return qa | (qb << 16);
}
__device__ __forceinline__ void put_box(BvhNode *nd, const Box &b, const Frame &f) {
    nd->x = quantize(b.lo[0], b.hi[0], f.org[0], f.step[0]);
    nd->y = quantize(b.lo[1], b.hi[1], f.org[1], f.step[1]);
    nd->z = quantize(b.lo[2], b.hi[2], f.org[2], f.step[2]);
}

// Leaf triangles and boxes of the block's kBoxBlock leaf slots, and the boxes of
// the internal nodes whose leaves all lie among them.  The leaves of a node
// are a run of slots, so its box is a range union: two overlapping
// power-of-two runs of a sparse table in LDS.  Also the unions from the block's
// first slot to each slot and from each slot to its last, for the nodes that
// span blocks (k_boxes_across).  The boxes used to be formed bottom-up, the
// second of two siblings to arrive going on to the parent: a chain of
// device-scope atomics and loads per level (0.27 ms at 51k triangles, 1.06 ms
// at 200k); unions are exact, so the boxes are the same.
// `build`: seals the buffer.  A refit follows the stored order, ranges and
// places only in a sealed buffer; otherwise it only sets the header's word 2.
__global__ __launch_bounds__(kBoxBlock) void k_boxes(const float *verts, const int32_t *faces, BvhView bv,
                                                     int nparts, int build) {
    constexpr int LV = 8;
    __shared__ float T[LV][6][kBoxBlock];
    __shared__ uint32_t red[kBoundsBlocks / 64][6];
    const int n = bv.n, tid = threadIdx.x, i = blockIdx.x * kBoxBlock + tid;
    if (!build && !sealed(bv)) {
        if (i == 0) bv.header[2] = 1;
        return;
    }
    float blo[3], bhi[3];
    all_bounds(bv.part, nparts, 6, red, blo, bhi);
    const Frame fr = make_frame(blo, bhi);
    Box b = empty_box();
    if (i < n) {
        const int f = bv.order[i];
        const Tri t = load_tri(verts, faces, f);
        LeafTri lt;
        lt.a = make_float4(t.a.x, t.a.y, t.a.z, __int_as_float(f));
        lt.b = make_float4(t.b.x, t.b.y, t.b.z, 0.0f);
        lt.c = make_float4(t.c.x, t.c.y, t.c.z, 0.0f);
        bv.tris[i] = lt;
        b = {{min3(t.a.x, t.b.x, t.c.x), min3(t.a.y, t.b.y, t.c.y), min3(t.a.z, t.b.z, t.c.z)},
             {max3(t.a.x, t.b.x, t.c.x), max3(t.a.y, t.b.y, t.c.y), max3(t.a.z, t.b.z, t.c.z)}};
        // pad by a few ulps so rounding in the slab test never culls a true hit
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const float m = fmaxf(fabsf(b.lo[k]), fabsf(b.hi[k]));
            const float pad = m * 2.4e-7f + 1e-30f;
            b.lo[k] -= pad;
            b.hi[k] += pad;
        }
        put_box(bv.nodes + bv.dfs_of[n - 1 + i], b, fr);
    }
    auto put = [&](int l) {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            T[l][k][tid] = b.lo[k];
            T[l][3 + k][tid] = b.hi[k];
        }
    };
    auto get = [&](int l, int at) {
        return Box{{T[l][0][at], T[l][1][at], T[l][2][at]}, {T[l][3][at], T[l][4][at], T[l][5][at]}};
    };
    put(0);
    __syncthreads();
    for (int l = 1; l < LV; l++) {   // T[l][s]: slots s .. s + 2^l - 1 (past the block's end: to it)
        const int at = tid + (1 << (l - 1));
        if (at < kBoxBlock) b = unite(b, get(l - 1, at));
        put(l);
        __syncthreads();
    }
    auto range = [&](int lo, int hi) {
        const int l = min(LV - 1, 31 - __clz(hi - lo + 1));
        return unite(get(l, lo), get(l, hi + 1 - (1 << l)));
    };
    const int first = blockIdx.x * kBoxBlock, last = min(n, first + kBoxBlock) - 1;
    if (i < n) {
        bv.prefix[i] = range(0, tid);
        bv.suffix[i] = range(tid, last - first);
    }
    if (i < n - 1) {
        const int j = bv.other[i], lo = min(i, j), hi = max(i, j);
        if (lo >= first && hi <= last) put_box(bv.nodes + bv.dfs_of[i], range(lo - first, hi - first), fr);
    }
    if (i == 0) {
        float *h = reinterpret_cast<float *>(bv.header);
        for (int k = 0; k < 3; k++) {
            h[4 + k] = fr.org[k];
            h[8 + k] = fr.step[k];
        }
        if (build) {
            bv.header[0] = n;
            bv.header[1] = kBvhMagic;
            bv.header[2] = 0;
        }
    }
}

// Boxes of the internal nodes that span blocks of leaf slots: the end of the
// first block, the start of the last, and the whole blocks between (all 64
// lanes of the wavefront together where there are many).
__global__ __launch_bounds__(kThreads) void k_boxes_across(BvhView bv, int build) {
    if (!build && !sealed(bv)) return;
    const int n = bv.n, i = blockIdx.x * kThreads + threadIdx.x, lane = threadIdx.x & 63;
    Box b = empty_box();
    int b0 = 0, b1 = 0;
    bool mine = false;
    if (i < n - 1) {
        const int j = bv.other[i], lo = min(i, j), hi = max(i, j);
        if (lo / kBoxBlock != hi / kBoxBlock) {
            mine = true;
            b = unite(bv.suffix[lo], bv.prefix[hi]);
            b0 = lo / kBoxBlock + 1;
            b1 = hi / kBoxBlock;
        }
    }
    if (b1 - b0 <= 8)
        for (int q = b0; q < b1; q++) b = unite(b, bv.suffix[q * kBoxBlock]);
    uint64_t pending = __ballot(b1 - b0 > 8);
    while (pending) {
        const int src = __ffsll((unsigned long long)pending) - 1;
        pending &= pending - 1;
        const int q0 = __shfl(b0, src), q1 = __shfl(b1, src);
        Box m = empty_box();
        for (int q = q0 + lane; q < q1; q += 64) m = unite(m, bv.suffix[q * kBoxBlock]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                m.lo[k] = fminf(m.lo[k], __shfl_xor(m.lo[k], off));
                m.hi[k] = fmaxf(m.hi[k], __shfl_xor(m.hi[k], off));
            }
        if (lane == src) b = unite(b, m);
    }
    if (mine) {
        const float *h = reinterpret_cast<const float *>(bv.header);
        const Frame fr = {{h[4], h[5], h[6]}, {h[8], h[9], h[10]}};
        put_box(bv.nodes + bv.dfs_of[i], b, fr);
    }
}

}  // namespace

BvhView bvh_view(void *buf, int32_t nf, size_t *bytes_out) {
    Carver cv(buf);
    BvhView v;
    v.n = nf;
    v.n_nodes = 2 * nf - 1;
    v.header = cv.take<int32_t>(16);
    v.nodes = cv.take<BvhNode>(v.n_nodes);
    v.tris = cv.take<LeafTri>(nf);
    v.order = cv.take<int32_t>(nf);
    v.other = cv.take<int32_t>(nf > 1 ? nf - 1 : 1);
    v.dfs_of = cv.take<int32_t>(v.n_nodes);
    v.part = cv.take<uint32_t>(12 * kBoundsBlocks);
    v.prefix = cv.take<Box>(nf);
    v.suffix = cv.take<Box>(nf);
    if (bytes_out) *bytes_out = align_up(cv.off, 256);
    return v;
}

struct BuildScratch {
    uint32_t *keys[2];
    int32_t *vals[2];
    uint32_t *hist;       // [4 passes][nblk][256]
    int2 *child;
    int32_t *parent;      // [2n - 1], -1: the root
    int nblk, steps;      // sort blocks, steps of kSortThreads keys each takes
};

static BuildScratch carve_build(void *buf, int32_t nf, size_t *bytes) {
    Carver cv(buf);
    BuildScratch s;
    const int tiles = (nf + kSortThreads - 1) / kSortThreads;
    s.steps = (tiles + kSortBlocks - 1) / kSortBlocks;
    s.nblk = (tiles + s.steps - 1) / s.steps;
    s.keys[0] = cv.take<uint32_t>(nf);
    s.keys[1] = cv.take<uint32_t>(nf);
    s.vals[0] = cv.take<int32_t>(nf);
    s.vals[1] = cv.take<int32_t>(nf);
    s.hist = cv.take<uint32_t>((size_t)4 * 256 * s.nblk);
    s.child = cv.take<int2>(nf > 1 ? nf - 1 : 1);
    s.parent = cv.take<int32_t>((size_t)2 * nf - 1);
    if (bytes) *bytes = align_up(cv.off, 256);
    return s;
}

size_t build_scratch_bytes(int32_t nf) {
    size_t b = 0;
    carve_build(nullptr, nf, &b);
    return b;
}

static inline int nblocks(long long n, int t) { return (int)((n + t - 1) / t); }

int bvh_build(const sbr_mesh *m, void *bvh, size_t bvh_bytes, int32_t mode, void *scratch,
              size_t scratch_bytes, hipStream_t st) {
    const int nf = m->nf;
    size_t need = 0;
    BvhView bv = bvh_view(bvh, nf, &need);
    if (bvh_bytes < need) {
        set_error("BVH buffer too small: %zu bytes given, %zu needed", bvh_bytes, need);
        return SBR_E_SCRATCH;
    }
    const int nparts = std::min(kBoundsBlocks, nblocks(nf, kThreads));
    if (mode == 0) {
        size_t sneed = 0;
        BuildScratch s = carve_build(scratch, nf, &sneed);
        if (!scratch || scratch_bytes < sneed) {
            set_error("BVH build scratch too small: %zu bytes given, %zu needed", scratch_bytes, sneed);
            return SBR_E_SCRATCH;
        }
        const int nh = 256 * s.nblk;
        hipLaunchKernelGGL(k_bounds, dim3(nparts), dim3(kThreads), 0, st, m->verts, m->faces, nf, bv, 1,
                           s.hist + nh, 3 * nh);
        hipLaunchKernelGGL(k_morton, dim3(s.nblk), dim3(kSortThreads), 0, st, m->verts, m->faces, nf, bv.part, nparts,
                           s.keys[0], s.hist, s.steps);
        for (int pass = 0; pass < 4; pass++) {
            const int cur = pass & 1;
            hipLaunchKernelGGL(k_sort_pass, dim3(s.nblk), dim3(kSortThreads), 0, st, s.keys[cur],
                               pass == 0 ? (const int32_t *)nullptr : s.vals[cur], s.keys[1 - cur],
                               pass == 3 ? bv.order : s.vals[1 - cur], nf, 8 * pass, s.hist + (size_t)pass * nh,
                               pass == 3 ? (uint32_t *)nullptr : s.hist + (size_t)(pass + 1) * nh, s.steps);
        }
        SBR_LAUNCHED();
        if (nf > 1)
            hipLaunchKernelGGL(k_karras, dim3(nblocks(nf - 1, kThreads)), dim3(kThreads), 0, st, s.keys[0], nf,
                               s.parent, s.child, bv.other);
        hipLaunchKernelGGL(k_dfs, dim3(nblocks(2 * nf - 1, kThreads)), dim3(kThreads), 0, st, nf, s.parent, s.child,
                           bv);
        SBR_LAUNCHED();
    } else {
        hipLaunchKernelGGL(k_bounds, dim3(nparts), dim3(kThreads), 0, st, m->verts, m->faces, nf, bv, 0,
                           (uint32_t *)nullptr, 0);
    }
    hipLaunchKernelGGL(k_boxes, dim3(nblocks(nf, kBoxBlock)), dim3(kBoxBlock), 0, st, m->verts, m->faces, bv,
                       nparts, mode == 0 ? 1 : 0);
    if (nf > kBoxBlock)
        hipLaunchKernelGGL(k_boxes_across, dim3(nblocks(nf - 1, kThreads)), dim3(kThreads), 0, st, bv,
                           mode == 0 ? 1 : 0);
    SBR_LAUNCHED();
    return SBR_OK;
}

}  // namespace sbr
