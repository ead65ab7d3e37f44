// Direction-binned primitive lists of an image tile (gfx950, device side).
//
// The candidate rays of one tile start close together and differ in
// direction.  A workgroup therefore culls the scene once per tile: the
// sphere of directions is cut into kBins cells of the octahedral map, and a
// bit mask per cell says which primitives a ray from the tile's origin box
// into that cell can reach.  A ray then tests only its cell's primitives,
// nearest first, instead of walking a grid.
//
// The masks are a superset of what any such ray can hit (every bound below is
// widened by far more than the FP32 rounding of the tests), and the closest
// hit is the smallest (t, id) pair over the primitives, so the result is that
// of the brute-force loop and of the grid walk, bit for bit.
//
// 12 x 12 cells: with 256 primitives a ray's list has some 9 of them and it
// tests 5 (the grid walk: 10, and 4 steps); 8 x 8 cells make that 14 and 7,
// 16 x 16 cells 7 and 5 for nearly twice the build, which costs 31,000 of a
// 16x16-pixel tile's 476,000 cycles.  The build is a chain of latencies
// rather than of work: taking four cells at a time halved it (60,000).
#pragma once

#include "gi_device.hpp"

namespace gi {

constexpr int kBinSide = 12;
constexpr int kBins = kBinSide * kBinSide;
constexpr uint32_t kListMaxPrims = 1024u;
constexpr int kListBuckets = 32;     // distance classes the primitives are ordered by
constexpr float kListFar = 1e18f;     // largest distance: the squares behind it stay finite

// 32-slot words of the lists: spheres fill the first ones, boxes the rest
// (so two of them may be partly filled); even, since a wave writes two
__host__ __device__ constexpr uint32_t list_words(uint32_t n_prims) { return ((n_prims + 31u) / 32u + 2u) & ~1u; }

// LDS bytes of the lists of a scene of n_prims primitives of any mix of
// types: 24 B of geometry per slot, a mask word per word and cell, each
// word's nearest distance, the slots' primitive ids
__host__ __device__ constexpr uint32_t list_bytes(uint32_t n_prims)
{
    const uint32_t w = list_words(n_prims);
    return (w * 32u * 24u + kBins * w * 4u + w * 4u + w * 32u * 2u + 15u) & ~15u;
}
// words of LDS the build needs besides (free again once it has returned)
constexpr uint32_t kListScratch = 6u * kBins + 2u * kListBuckets + 2u;

struct TileLists {
    float2 *geo;            // slot s: sphere (c.x, c.y) (c.z, r) or box (lo.x, lo.y) (lo.z, hi.x) (hi.y, hi.z) at 3 s
    uint32_t *mask;         // mask[cell * words + w]
    float *near;            // least distance from the origin box to a primitive of word w or a later one of its type
    uint16_t *ids;
    uint32_t words, sw, nw; // stride of the masks; sphere words; words in use
    __device__ __forceinline__ TileLists(void *lds, uint32_t n_prims)
    {
        words = list_words(n_prims);
        geo = reinterpret_cast<float2 *>(lds);
        mask = reinterpret_cast<uint32_t *>(geo + 3u * 32u * words);
        near = reinterpret_cast<float *>(mask + kBins * words);
        ids = reinterpret_cast<uint16_t *>(near + words);
        sw = nw = 0u;
    }
};

// Sort cell of a unit direction: 4 times its list cell plus the quarter of it
// the direction lies in; list cells in snake order (consecutive ones are
// neighbours)
__device__ __forceinline__ uint32_t sort_bin_of(V3 d)
{
    float u, w;
    oct_encode_signed(d, u, w);
    constexpr float h = (float)kBinSide;
    const int x = min(max((int)fmaf(u, h, h), 0), 2 * kBinSide - 1), y = min(max((int)fmaf(w, h, h), 0), 2 * kBinSide - 1);
    const int cx = x >> 1, cy = y >> 1;
    return (uint32_t)(4 * (cy * kBinSide + ((cy & 1) ? kBinSide - 1 - cx : cx)) + 2 * (y & 1) + ((x ^ y) & 1));
}

struct Box3 {
    V3 c, h;                // centre and half extents
};

// What the lists take for granted of a pixel's rays: that they start at a
// point, and that their directions are of unit length to within 1e-3 (a frame
// about a normal with |n|^2 within 2e-4 of 1 keeps them to 2e-4, a lobe's half
// vector to 8e-4), so that a ray parameter is a distance at least to the 1e-3
// that the lists' distances are lowered by.  A pixel without either shows in
// the normals' box, by a normal of kNoUnit or kNoPlace along x.  For directions
// of other lengths no word lies beyond a hit (what the cells leave out still
// lies off the ray); for an origin that is no point, or beyond kOrgFar, every
// cell lists every primitive.  Such a pixel's rays find what the brute-force
// loop finds.  (One component says it all: with three the glossy FP32 form
// spills 17 more scalars, 1920x1080 5.41 ms against 5.31.)
//
// kOrgFar: up to here an empty slot's bounds stay finite beside its radius of
// -inf (the tangent plane's normal below 2e22 before it cancels, times the
// box), so that it is never listed: its geometry and id are not set.
constexpr float kNoUnit = 1e6f, kNoPlace = 1e12f, kOrgFar = 1e12f;
__device__ __forceinline__ bool is_place(V3 o) { return fabsf(o.x) + fabsf(o.y) + fabsf(o.z) < kOrgFar; }
__device__ __forceinline__ V3 list_origin(V3 o) { return is_place(o) ? o : v3(0.0f, 0.0f, 0.0f); }
__device__ __forceinline__ V3 list_axis(V3 o, V3 n)
{
    V3 a = fabsf(dot(n, n) - 1.0f) <= 2e-4f ? n : v3(kNoUnit, 0.0f, 0.0f);
    a.x = is_place(o) ? a.x : kNoPlace;
    return a;
}

__device__ __forceinline__ V3 vabs(V3 a) { return v3(fabsf(a.x), fabsf(a.y), fabsf(a.z)); }

// Bounding cone (axis, cos) of direction cell b.  A cell is one planar patch
// of the octahedron or two that meet in its diagonal (kBinSide is even), so
// its farthest points from the axis are its corners.
__device__ __forceinline__ float4 bin_cone(int b)
{
    const int y = b / kBinSide, xs = b % kBinSide, x = (y & 1) ? kBinSide - 1 - xs : xs;
    constexpr float s = 1.0f / (float)kBinSide;
    V3 c[4], a = v3(0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c[k] = oct_decode((float)(x + (k & 1)) * s, (float)(y + (k >> 1)) * s);
        a = a + c[k];
    }
    a = frsq(dot(a, a)) * a;
    float ct = 1.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) ct = fminf(ct, dot(a, c[k]));
    return make_float4(a.x, a.y, a.z, ct - 1e-3f);
}

// Builds the lists for rays that start in box `org`, tight for directions d
// with n.d >= 0 for some n in box `nrm` (unit normals).  Every thread of the
// workgroup of NT threads calls it; it starts and ends with a barrier.
//  - Primitives are ordered by kListBuckets distance classes, per type, so
//    that a ray can stop at the first word that lies beyond its hit.
//  - A primitive is kept for a cell unless a plane through the cone's apex
//    separates it, the origin box added to its extent, from the cone: the
//    tangent plane of the cone toward the primitive's centre, or the plane
//    behind the apex.  Where a bound is no number (an infinite slab has no
//    centre) it stays; sizes count by their absolute values, as in the tests.
template <int NT>
__device__ __forceinline__ void build_lists(const gi_scene &sc, TileLists &L, Box3 org, Box3 nrm, uint32_t *scratch)
{
    constexpr uint32_t kPer = kListMaxPrims / NT, kWaves = NT / 64;
    const uint32_t t = threadIdx.x, n = sc.n_prims;
    const float top = nrm.c.x + nrm.h.x;                   // the longest list_axis along x
    const float lower = top < 2.0f ? 0.999f : 0.0f;
    // the cells in use: cone axis and cos, then sin and the cell
    float4 *cone = reinterpret_cast<float4 *>(scratch);
    float2 *cell = reinterpret_cast<float2 *>(scratch + 4 * kBins);
    uint32_t *hist = scratch + 6 * kBins, *dmax = hist + 2 * kListBuckets;
    __syncthreads();
    if (t < 2u * kListBuckets + 2u) hist[t] = 0u;
    if (t < L.words) L.near[t] = kInf;
    __syncthreads();
    if (t < (uint32_t)kBins) {
        const float4 c = bin_cone((int)t);
        const V3 a = v3(c.x, c.y, c.z);
        const float st = fsqrt(fmaxf(0.0f, fmaf(-c.w, c.w, 1.0f)));
        // no ray into a cell below every surface: largest n.d over the box and the cone
        if (top < 0.5f * kNoPlace && (top >= 2.0f || dot(nrm.c, a) + dot(nrm.h, vabs(a)) >= -st - 1e-2f)) {
            const uint32_t u = atomicAdd(&dmax[1], 1u);
            cone[u] = c;
            cell[u] = make_float2(st, __uint_as_float(t));
        }
    }
    const float4 *src = reinterpret_cast<const float4 *>(sc.prims);
    float4 ga[kPer], gb[kPer];
    float dist[kPer];
    uint32_t cls[kPer], rank[kPer];
    float far = 0.0f;
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t i = t + k * NT;
        if (i >= n) continue;
        const float4 a = src[4u * i], b = src[4u * i + 1u];
        geo_records(a, b, ga[k], gb[k]);
        cls[k] = __float_as_uint(a.w) == 0u ? 0u : 1u;
        const V3 v = vabs(xyz(a) - org.c), e = cls[k] ? vabs(xyz(b)) : v3(0.0f, 0.0f, 0.0f);
        const V3 q = v3(fmaxf(v.x - org.h.x - e.x, 0.0f), fmaxf(v.y - org.h.y - e.y, 0.0f),
                        fmaxf(v.z - org.h.z - e.z, 0.0f));
        const float d = fsqrt(dot(q, q)) - (cls[k] ? 0.0f : fabsf(b.x));
        const float slop = 1e-4f * (fabsf(a.x) + fabsf(a.y) + fabsf(a.z) + fabsf(org.c.x) + fabsf(org.c.y) + fabsf(org.c.z));
        dist[k] = fminf(fmaxf(0.0f, fmaf(d, lower, -slop)), kListFar);
        far = fmaxf(far, dist[k]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) far = fmaxf(far, __shfl_xor(far, o, 64));
    if ((t & 63u) == 0u) atomicMax(dmax, __float_as_uint(far));
    __syncthreads();
    const float scale = (float)kListBuckets * rcp(fmaxf(__uint_as_float(*dmax), 1e-30f));
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        if (t + k * NT >= n) continue;
        cls[k] = cls[k] * kListBuckets + min((uint32_t)(dist[k] * scale), (uint32_t)kListBuckets - 1u);
        rank[k] = atomicAdd(&hist[cls[k]], 1u);
    }
    __syncthreads();
    if (t < 64u) {
        // first slot of every class: spheres from 0, boxes from the word after them
        const uint32_t c = hist[t];
        uint32_t s = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = __shfl_up(s, o, 64);
            if ((int)t >= o) s += v;
        }
        const uint32_t ns = __shfl(s, kListBuckets - 1, 64);
        s -= c;
        if (t >= (uint32_t)kListBuckets) s = s - ns + ((ns + 31u) & ~31u);
        hist[t] = s;
        if (t == 0u) *dmax = ns;
    }
    __syncthreads();
    const uint32_t ns = __builtin_amdgcn_readfirstlane(*dmax);
    L.sw = (ns + 31u) >> 5;
    L.nw = L.sw + ((n - ns + 31u) >> 5);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63u;
    // every cell starts with every primitive: what a ray into a cell not in
    // use meets
    if (lane < L.nw) {
        const uint32_t first = lane < L.sw ? 32u * lane : 32u * (lane - L.sw), left = (lane < L.sw ? ns : n - ns) - first;
        const uint32_t all = left >= 32u ? ~0u : (1u << left) - 1u;
        for (uint32_t b = wave; b < (uint32_t)kBins; b += kWaves) L.mask[b * L.words + lane] = all;
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t i = t + k * NT;
        if (i >= n) continue;
        const uint32_t s = hist[cls[k]] + rank[k];
        const bool box = cls[k] >= (uint32_t)kListBuckets;
        L.geo[3u * s] = make_float2(ga[k].x, ga[k].y);
        L.geo[3u * s + 1u] = make_float2(ga[k].z, gb[k].x);
        if (box) L.geo[3u * s + 2u] = make_float2(gb[k].y, gb[k].z);
        L.ids[s] = (uint16_t)i;
        atomicMin(reinterpret_cast<uint32_t *>(L.near) + (s >> 5), __float_as_uint(dist[k]));
    }
    __syncthreads();
    // nearest distance of a word and the later ones of its type (at most 64 words)
    if (t < 64u) {
        const uint32_t end = t < L.sw ? L.sw : L.nw;
        float near = t < L.nw ? L.near[t] : kInf;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const float v = __shfl_down(near, o, 64);
            if (t + (uint32_t)o < end) near = fminf(near, v);
        }
        if (t < L.nw) L.near[t] = near;
    }
    // masks: a wave takes 64 slots and a share of the cells in use, one slot
    // per lane; kIlp cells at a time, since each test is a chain of some 25
    // dependent instructions
    constexpr uint32_t kIlp = 4u;
    const uint32_t used = __builtin_amdgcn_readfirstlane(dmax[1]);
    const uint32_t chunks = (L.nw + 1u) >> 1, parts = max(1u, kWaves / max(chunks, 1u));
    const uint32_t part = wave % parts;
    for (uint32_t c = wave / parts; c < chunks; c += kWaves / parts) {
        const uint32_t s = 64u * c + lane;
        const bool box = s >= 32u * L.sw;
        const bool valid = box ? s - 32u * L.sw < n - ns : s < ns;
        V3 v = v3(0.0f, 0.0f, 0.0f), h = v;
        float rad = 0.0f;
        if (valid) {
            const float2 p = L.geo[3u * s], q = L.geo[3u * s + 1u];
            if (box) {
                const float2 r = L.geo[3u * s + 2u];
                v = v3(0.5f * (p.x + q.y), 0.5f * (p.y + r.x), 0.5f * (q.x + r.y));
                h = v3(0.5f * (q.y - p.x), 0.5f * (r.x - p.y), 0.5f * (r.y - q.x));
            } else {
                v = v3(p.x, p.y, q.x);
                rad = q.y;
            }
        }
        const float slop = 1e-4f * (fabsf(v.x) + fabsf(v.y) + fabsf(v.z) + fabsf(org.c.x) + fabsf(org.c.y) + fabsf(org.c.z));
        v = v - org.c;
        h = 1.001f * (vabs(h) + org.h);
        rad = valid ? 1.001f * fabsf(rad) + slop : -kInf;  // an empty slot is behind every cone (see kOrgFar)
        const float vv = dot(v, v);
        for (uint32_t u0 = part * kIlp; u0 < used; u0 += parts * kIlp) {
            float4 cn[kIlp];
            float2 cs[kIlp];
            float side[kIlp], back[kIlp];
#pragma unroll
            for (uint32_t k = 0; k < kIlp; ++k) {
                cn[k] = cone[min(u0 + k, used - 1u)];
                cs[k] = cell[min(u0 + k, used - 1u)];
            }
#pragma unroll
            for (uint32_t k = 0; k < kIlp; ++k) {
                const float ct = cn[k].w, st = cs[k].x;
                const V3 a = v3(cn[k].x, cn[k].y, cn[k].z);
                const float z = dot(v, a), w2 = fmaxf(fmaf(-z, z, vv), 1e-20f), iw = frsq(w2);
                // tangent plane: normal m = ct (v - z a)/|v - z a| - st a
                const float kk = ct * iw, ka = fmaf(kk, z, st);
                const V3 m = v3(fabsf(fmaf(kk, v.x, -ka * a.x)), fabsf(fmaf(kk, v.y, -ka * a.y)),
                                fabsf(fmaf(kk, v.z, -ka * a.z)));
                side[k] = rad + dot(m, h) - (kk * w2 - st * z);
                back[k] = z + rad + dot(vabs(a), h);
            }
            uint64_t keep = 0u;
            uint32_t c_k = 0u;
#pragma unroll
            for (uint32_t k = 0; k < kIlp; ++k) {
                const uint64_t b = __builtin_amdgcn_ballot_w64(!(fminf(side[k], back[k]) < 0.0f));
                if (lane == k) {
                    keep = b;
                    c_k = __float_as_uint(cs[k].y);
                }
            }
            if (lane < kIlp) *reinterpret_cast<uint64_t *>(L.mask + c_k * L.words + 2u * c) = keep;
        }
    }
    __syncthreads();
}

// Closest hit of a ray of the tile (origin and cell b as the lists were built
// for) as cast<false> finds it; slot: the primitive's in the lists, or ~0
__device__ __forceinline__ bool cast_lists(const gi_scene &sc, const TileLists &L, uint32_t b, V3 o, V3 d, Hit &h,
                                           uint32_t &slot)
{
    h.t = kInf;
    h.prim = GI_MISS;
    h.axis = -1;
    const V3 inv = v3(rcp(d.x), rcp(d.y), rcp(d.z));
    if (sc.has_room) {
        int axis;
        uint32_t wall;
        const float tw = isect_room(sc, o, d, axis, wall);
        if (tw < h.t) { h.t = tw; h.prim = wall; h.axis = axis; }
    }
    const uint32_t *mask = L.mask + b * L.words;
    slot = ~0u;
    const auto take = [&](float t, uint32_t s) {
        if (t <= h.t && t < kInf) {
            const uint32_t i = L.ids[s];
            if (t < h.t || i < h.prim) {
                h.t = t;
                h.prim = i;
                slot = s;
            }
        }
    };
    for (uint32_t w = 0; w < L.sw; ++w) {
        if (L.near[w] > h.t) break;
        uint32_t m = mask[w];
        while (m != 0u) {
            const uint32_t s = 32u * w + (uint32_t)__builtin_ctz(m);
            m &= m - 1u;
            const float2 p = L.geo[3u * s], q = L.geo[3u * s + 1u];
            take(isect_sphere(o, d, v3(p.x, p.y, q.x), q.y), s);
        }
    }
    for (uint32_t w = L.sw; w < L.nw; ++w) {
        if (L.near[w] > h.t) break;
        uint32_t m = mask[w];
        while (m != 0u) {
            const uint32_t s = 32u * w + (uint32_t)__builtin_ctz(m);
            m &= m - 1u;
            const float2 p = L.geo[3u * s], q = L.geo[3u * s + 1u], r = L.geo[3u * s + 2u];
            take(isect_box(o, inv, v3(p.x, p.y, q.x), v3(q.y, r.x, r.y)), s);
        }
    }
    return h.prim != GI_MISS;
}

// facing normal of a hit of cast_lists, as hit_normal forms it; a wall's
// (slot ~0) has its axis in `axis`
__device__ __forceinline__ V3 list_normal(const TileLists &L, V3 o, V3 d, float t, uint32_t slot, int axis)
{
    if (slot < 32u * L.sw) {
        const float2 p = L.geo[3u * slot], q = L.geo[3u * slot + 1u];
        const V3 x = madd(o, t, d);
        const float ir = rcp(q.y);
        const V3 n = ir * (x - v3(p.x, p.y, q.x));
        return dot(n, d) > 0.0f ? -n : n;
    }
    if (slot != ~0u) {
        const V3 inv = v3(rcp(d.x), rcp(d.y), rcp(d.z));
        const float2 p = L.geo[3u * slot], q = L.geo[3u * slot + 1u], r = L.geo[3u * slot + 2u];
        axis = box_axis(o, inv, v3(p.x, p.y, q.x), v3(q.y, r.x, r.y));
    }
    const float s = comp(d, axis) > 0.0f ? -1.0f : 1.0f;
    return v3(axis == 0 ? s : 0.0f, axis == 1 ? s : 0.0f, axis == 2 ? s : 0.0f);
}

}  // namespace gi
