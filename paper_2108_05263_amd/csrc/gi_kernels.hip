// HIP kernels and C-ABI launchers of the DDGI-resampling path (gfx950).
//
// Per-pixel kernels use 256-thread workgroups over 16x16 pixel tiles, each
// wave64 covering an 8x8 sub-tile, so SoA float4 plane accesses of a wave
// fill whole 128-byte lines and neighbouring pixels share cache lines of the
// grid, probes and reservoirs.  One kernel per C-ABI entry point; all state
// lives in caller-owned buffers.
#include <hip/hip_runtime.h>

#include <cmath>
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "gi.h"
#include "gi_device.hpp"
#include "gi_lists.hpp"
#include "gi_mlp.hpp"

using namespace gi;

namespace {

constexpr int kTile = 16;
constexpr int kBlock = 256;
constexpr uint32_t kSelBytes = 64u;   // k_initial's per-thread slot: selected candidate (3 float4), residual

// Workgroups are dealt round-robin to the chip's 8 XCDs, each with its own L2
constexpr uint32_t kXcds = 8;

// The pixel of a lane of the passes of one thread per pixel: SW x 16 tiles in
// image order.  (48x16 tiles in stripes left XCDs without work where tile
// columns are few: 40x2000, 1024 primitives, shade 102 us, in image order 45;
// 1283x721 177 and 162; 3840x2160 1.28 and 1.25 ms.)
template <uint32_t SW = (uint32_t)kTile>
__device__ __forceinline__ bool tile_pixel(uint32_t W, uint32_t H, uint32_t &px, uint32_t &py)
{
    const uint32_t w = threadIdx.x >> 6, l = threadIdx.x & 63u;
    px = blockIdx.x * SW + (w % (SW / 8u)) * 8u + (l & 7u);
    py = blockIdx.y * kTile + (w / (SW / 8u)) * 8u + (l >> 3);
    return px < W && py < H;
}

dim3 tile_grid(uint32_t W, uint32_t H, uint32_t SW = (uint32_t)kTile)
{
    return dim3((W + SW - 1) / SW, (H + kTile - 1) / kTile);
}

// The spatial pass gathers from neighbours within its radius: its
// workgroups are given tiles in XCD stripes, so that a pixel's neighbours
// are mostly read through one XCD's L2.  Workgroup L runs on XCD L % 8 and
// takes tile L / 8 (row-major) of stripe L % 8, a band of ceil(tx / 8) tile
// columns (tiles of SW x 16 pixels, one of t's lanes each).
template <uint32_t SW>
__device__ __forceinline__ bool tile_pixel_striped(uint32_t W, uint32_t H, uint32_t &px, uint32_t &py, uint32_t t)
{
    const uint32_t w = t >> 6, l = t & 63u;
    const uint32_t tiles_x = (W + SW - 1) / SW;
    const uint32_t sw = (tiles_x + kXcds - 1) / kXcds;
    const uint32_t xcd = blockIdx.x % kXcds, m = blockIdx.x / kXcds;
    const uint32_t tx = xcd * sw + m % sw, ty = m / sw;
    px = tx * SW + (w % (SW / 8u)) * 8u + (l & 7u);
    py = ty * kTile + (w / (SW / 8u)) * 8u + (l >> 3);
    return tx < tiles_x && px < W && py < H;
}

dim3 striped_grid(uint32_t W, uint32_t H, uint32_t SW)
{
    const uint32_t tx = (W + SW - 1) / SW, ty = (H + kTile - 1) / kTile;
    const uint32_t sw = (tx + kXcds - 1) / kXcds;
    return dim3(kXcds * sw * ty);
}

struct GB {
    V3 pos;
    float depth;
    V3 n;
    uint32_t prim;
    V3 alb;
    float ks, rough;     // glossy layer (glossy loads only; else 0 and 1)
    V3 wo;               // unit direction toward the camera (glossy loads only)
};

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

// GLOSSY: also the glossy layer (k_s in albedo.w, roughness in emit.w) and
// the direction toward the camera position the buffer was traced from
template <bool GLOSSY = false>
__device__ __forceinline__ GB load_gb(const gi_gbuffer &g, uint32_t p)
{
    float4 a = reinterpret_cast<const float4 *>(g.pos_depth)[p];
    GB r;
    float ks = 0.0f;
    if (g.format == GI_GB_F16) {
        const half4_t b = reinterpret_cast<const half4_t *>(g.nrm_prim)[p];
        const half4_t c = reinterpret_cast<const half4_t *>(g.albedo)[p];
        const uint32_t prim16 = __builtin_bit_cast(uint16_t, b[3]);
        // a half-precision normal is renormalised: the sampling basis and the
        // cosines assume unit length
        V3 n = v3((float)b[0], (float)b[1], (float)b[2]);
        const float nn = dot(n, n);
        if (nn > 0.0f) n = frsq(nn) * n;
        r = GB{xyz(a), a.w, n, prim16 == 0xFFFFu ? GI_MISS : prim16, v3((float)c[0], (float)c[1], (float)c[2]),
               0.0f, 1.0f, v3(0.0f, 0.0f, 1.0f)};
        ks = (float)c[3];
    } else {
        float4 b = reinterpret_cast<const float4 *>(g.nrm_prim)[p];
        float4 c = reinterpret_cast<const float4 *>(g.albedo)[p];
        r = GB{xyz(a), a.w, xyz(b), __float_as_uint(b.w), xyz(c), 0.0f, 1.0f, v3(0.0f, 0.0f, 1.0f)};
        ks = c.w;
    }
    if constexpr (GLOSSY) {
        r.ks = ks;
        r.rough = reinterpret_cast<const float4 *>(g.emit)[p].w;
        V3 v = ld3(g.eye) - r.pos;
        r.wo = frsq(dot(v, v)) * v;
    }
    return r;
}

// normal + primitive and albedo (+ glossy weight k_s) records of the G-buffer's format
__device__ __forceinline__ void store_gb_na(const gi_gbuffer &g, uint32_t p, V3 n, uint32_t prim, V3 alb, float ks)
{
    if (g.format == GI_GB_F16) {
        const uint16_t prim16 = prim == GI_MISS ? (uint16_t)0xFFFFu : (uint16_t)prim;
        half4_t b = {(_Float16)n.x, (_Float16)n.y, (_Float16)n.z, __builtin_bit_cast(_Float16, prim16)};
        half4_t c = {(_Float16)alb.x, (_Float16)alb.y, (_Float16)alb.z, (_Float16)ks};
        reinterpret_cast<half4_t *>(g.nrm_prim)[p] = b;
        reinterpret_cast<half4_t *>(g.albedo)[p] = c;
        return;
    }
    reinterpret_cast<float4 *>(g.nrm_prim)[p] = make_float4(n.x, n.y, n.z, __uint_as_float(prim));
    reinterpret_cast<float4 *>(g.albedo)[p] = make_float4(alb.x, alb.y, alb.z, ks);
}

// a pixel is shaded when its surface reflects: diffuse albedo (or a glossy layer)
template <bool GLOSSY = false>
__device__ __forceinline__ bool active(const GB &g)
{
    return g.prim != GI_MISS && (!is_zero(g.alb) || (GLOSSY && g.ks > 0.0f));
}

__device__ __forceinline__ bool similar(const GB &g, const GB &q, const gi_params &pp)
{
    if (q.prim == GI_MISS) return false;
    if (dot(g.n, q.n) < pp.cos_n) return false;
    if (fabsf(g.depth - q.depth) > pp.depth_rel * g.depth) return false;
    return true;
}

// p_hat with the full BSDF of a glossy pixel: f(x, wo, wi) L min(G, G_max)
// (sky samples: f L cos)
__device__ __forceinline__ float target_glossy(const GB &g, V3 y, V3 ny, V3 L, float g_max)
{
    if (is_zero(ny)) {
        const float cx = dot(g.n, y);
        if (cx <= 0.0f) return 0.0f;
        return lum(bsdf(g.alb, g.ks, g.rough, g.n, g.wo, y) * L) * cx;
    }
    V3 v = y - g.pos;
    float d2 = dot(v, v);
    V3 w = frsq(d2) * v;
    float cx = dot(g.n, w), cy = -dot(ny, w);
    if (cx <= 0.0f || cy <= 0.0f) return 0.0f;
    return lum(bsdf(g.alb, g.ks, g.rough, g.n, g.wo, w) * L) * fminf(cx * cy * rcp(d2), g_max);
}

template <bool GLOSSY = false>
__device__ __forceinline__ float res_target(const GB &g, const Res &r, float g_max)
{
    if constexpr (GLOSSY) return target_glossy(g, r.y, r.n, r.L, g_max);
    return target(g.pos, g.n, g.alb, r.y, r.n, r.L, g_max);
}

// area density of emitter sampling at a point of primitive prim: 1/(n 4 pi r^2)
// on a listed emitter, else 0
__device__ __forceinline__ float light_pdf(const gi_scene &sc, uint32_t prim)
{
    for (uint32_t e = 0; e < sc.n_emitters; ++e)
        if (sc.emitters[e] == prim) {
            const float rad = reinterpret_cast<const float4 *>(sc.prims)[4 * prim + 1].x;
            return rcp((float)sc.n_emitters * 4.0f * kPi * rad * rad);
        }
    return 0.0f;
}

// --------------------------------------------------------------------------
// primary vertices
// --------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_gbuffer(gi_scene sc, gi_camera cam, gi_gbuffer gb)
{
    uint32_t px, py;
    if (!tile_pixel(cam.width, cam.height, px, py)) return;
    uint32_t p = py * cam.width + px;
    float aspect = (float)cam.width / (float)cam.height;
    float sx = (2.0f * ((float)px + 0.5f) / (float)cam.width - 1.0f) * cam.tan_half_fovy * aspect;
    float sy = (1.0f - 2.0f * ((float)py + 0.5f) / (float)cam.height) * cam.tan_half_fovy;
    V3 d = ld3(cam.fwd) + sx * ld3(cam.right) + sy * ld3(cam.up);
    d = rsqrtf(dot(d, d)) * d;
    V3 o = ld3(cam.eye);
    Hit h;
    const GeoGlobal acc(sc);
    float4 *pd = reinterpret_cast<float4 *>(gb.pos_depth);
    float4 *em = reinterpret_cast<float4 *>(gb.emit);
    const V3 zero = v3(0.0f, 0.0f, 0.0f);
    if (!cast<false>(sc, acc, o, d, kInf, h)) {
        pd[p] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        store_gb_na(gb, p, zero, GI_MISS, zero, 0.0f);
        em[p] = make_float4(sc.sky[0], sc.sky[1], sc.sky[2], 1.0f);
        return;
    }
    V3 x = madd(o, h.t, d);
    V3 n = hit_normal(sc, acc, o, d, h);
    V3 alb, emit;
    float ks = 0.0f, rough = 1.0f;
    if (sc.options & GI_OPT_GLOSSY) material_g(sc, h.prim, alb, emit, ks, rough);
    else material(sc, h.prim, alb, emit);
    pd[p] = make_float4(x.x, x.y, x.z, h.t * dot(d, ld3(cam.fwd)));
    store_gb_na(gb, p, n, h.prim, alb, ks);
    em[p] = make_float4(emit.x, emit.y, emit.z, rough);
}

// --------------------------------------------------------------------------
// probe update: one workgroup per probe
// --------------------------------------------------------------------------
constexpr int kProbeBlock = 256;
constexpr uint32_t kFilterRays = 8;    // rays that the filters read ahead

// Interior texel (row-major index into the N x N interior) that padded texel
// (x, y) shows: the interior itself, or for a gutter texel the interior texel
// mirrored along the tile edge (applied first across rows, then across
// columns, which maps a corner to the diagonally opposite interior corner).
__device__ __forceinline__ int gutter_source(int x, int y, int N)
{
    int sx = x, sy = y;
    if (sy == 0 || sy == N + 1) { sx = N + 1 - sx; sy = sy == 0 ? 1 : N; }
    if (sx == 0 || sx == N + 1) { sy = N + 1 - sy; sx = sx == 0 ? 1 : N; }
    return (sy - 1) * N + (sx - 1);
}

// GLOSSY: a hit on a glossy surface adds the glossy part of L_DDGI+ toward the
// probe (Eq. 6, one lobe sample, counter (probe, frame, 15, ray))
// F16: the volume's texel format is binary16 (else FP32)
//
// Bound by vector issue: 256 depth texels x R rays of ten instructions, two of
// them transcendental, then the traversal and the queries at the hits.  The
// rays are read from LDS by all lanes alike, so a loop that waits for each ray
// and branches on its side of the texel is two LDS latencies per ray: rays are
// read eight ahead and those behind the texel enter with weight zero, which
// leaves every sum as it is while all distances and radiances are finite.
// (With 16 ahead the registers cost more occupancy than the reads gain.)  The
// LDS block is sized for the rays asked for.  256 rays, before -> after:
// 32x8x32 probes, 256 primitives 848 -> 390 us, glossy 915 -> 450; 64x16x64
// probes, 1024 primitives 6.37 -> 4.10 ms; 4x4x4 probes, 64 rays 27 -> 20 us.
// Wavefronts per SIMD: with the scene in global memory seven (4.10 ms; five
// 4.36, unbounded 4.77), staged or glossy five (390 us, 450; seven 416, 574).
template <bool LDS, bool GLOSSY, bool F16>
__global__ void __launch_bounds__(kProbeBlock, LDS || GLOSSY ? 5 : 7)
    k_probe_update(gi_scene sc, gi_probes in, gi_probes out, gi_probe_params pp, uint64_t seed, uint32_t frame,
                   uint32_t scene_bytes)
{
    using Acc = typename std::conditional<LDS, GeoLds, GeoGlobal>::type;
    using F = ProbeFmt<F16>;
    if (LDS) stage_scene(sc);
    const Acc acc(sc);
    float4 *const s_ray = reinterpret_cast<float4 *>(reinterpret_cast<char *>(gi_lds) + scene_bytes);   // direction, distance
    float4 *const s_L = s_ray + pp.rays;
    __shared__ float s_irr[8 * 8][3];
    __shared__ float s_dep[16 * 16][2];
    const uint32_t pi = blockIdx.x;
    const uint32_t ix = pi % in.dims[0], iy = (pi / in.dims[0]) % in.dims[1], iz = pi / (in.dims[0] * in.dims[1]);
    const V3 P = v3(in.lo[0] + ((float)ix + 0.5f) * in.spacing[0], in.lo[1] + ((float)iy + 0.5f) * in.spacing[1],
                    in.lo[2] + ((float)iz + 0.5f) * in.spacing[2]);
    const uint32_t R = pp.rays;
    bool odd = false;                     // a squared distance or radiance that is no finite number
    for (uint32_t r = threadIdx.x; r < R; r += kProbeBlock) {
        uint4 rn = philox<true>(seed, pi, frame, kPassProbe, r);
        V3 w = sphere_dir(u01(rn.x), u01(rn.y));
        Hit h;
        V3 L;
        float dist;
        if (cast<false>(sc, acc, P, w, kInf, h)) {
            V3 hp = madd(P, h.t, w);
            V3 n = hit_normal(sc, acc, P, w, h);
            V3 alb, emit;
            float ks = 0.0f, ra = 1.0f;
            if (GLOSSY) material_g(sc, h.prim, alb, emit, ks, ra);
            else material(sc, h.prim, alb, emit);
            if (pp.distance_slider > 0.0f && !is_zero(emit)) {
                // distance heuristic: emission scaled by (t / (t + s d_b))^2, d_b the
                // probe's backward mean depth clipped to its cell
                const float2 m = fetch_dep<F16>(reinterpret_cast<const char *>(in.dep) + (size_t)pi * F::kDepProbe, -w);
                float clip = kInf;
                if (w.x != 0.0f) clip = fminf(clip, 0.5f * in.spacing[0] / fabsf(w.x));
                if (w.y != 0.0f) clip = fminf(clip, 0.5f * in.spacing[1] / fabsf(w.y));
                if (w.z != 0.0f) clip = fminf(clip, 0.5f * in.spacing[2] / fabsf(w.z));
                const float db = fminf(fmaxf(m.x, 0.0f), clip);
                const float ratio = h.t / (h.t + pp.distance_slider * db);
                emit = (ratio * ratio) * emit;
            }
            L = emit;
            if (!is_zero(alb)) {
                V3 q = probe_query_fmt<1, F16>(in, view_bias(hp, P, in.bias_dist), n);
                L = v3(fmaf(alb.x, q.x, emit.x), fmaf(alb.y, q.y, emit.y), fmaf(alb.z, q.z, emit.z));
            }
            if (GLOSSY && ks > 0.0f) {
                const uint4 rg = philox<true>(seed, pi, frame, kPassGlossyProbe, r);
                L = L + glossy_term<kTexOf<F16>>(in, view_bias(hp, P, in.bias_dist), n, -w, ks, ra, u01(rg.x), u01(rg.y));
            }
            dist = fminf(h.t, in.d_max);
        } else {
            L = ld3(sc.sky);
            dist = in.d_max;
        }
        s_ray[r] = make_float4(w.x, w.y, w.z, dist);
        s_L[r] = make_float4(L.x, L.y, L.z, 0.0f);
        odd = odd || !(fmaf(dist, dist, fabsf(L.x)) + fabsf(L.y) + fabsf(L.z) < kInf);
    }
    odd = __syncthreads_or(odd) != 0;
    // old interior texel (i, j) = first texel of quad record (i+1, j+1)
    // irradiance records are quad-major: record q of probe pi is record q * nP + pi
    const size_t nP = (size_t)in.dims[0] * in.dims[1] * in.dims[2];
    const char *iold = reinterpret_cast<const char *>(in.irr) + F::kIrrRec * (size_t)pi;
    const char *dold = reinterpret_cast<const char *>(in.dep) + F::kDepProbe * (size_t)pi;
    const float hy = pp.hysteresis;
    {   // depth texel t (16x16)
        uint32_t t = threadIdx.x;
        uint32_t tx = t & 15u, ty = t >> 4;
        V3 nt = oct_decode(((float)tx + 0.5f) / 16.0f, ((float)ty + 0.5f) / 16.0f);
        float m1 = 0.0f, m2 = 0.0f, den = 0.0f;
        // kAll: rays behind the texel enter with weight zero; kTiny: weights
        // below 2^-126 are kept
        const auto add = [&](const float4 ry, auto kAll, auto kTiny) {
            float c = nt.x * ry.x + nt.y * ry.y + nt.z * ry.z;
            if (kAll || c > 0.0f) {
                if (kAll) c = fmaxf(c, 0.0f);
                const float l = __log2f(c), e = pp.sharpness * l, d = ry.w;
                float w;
                if (kTiny) {
                    // 2^e, a denormal one by way of e + 64 (rounded once)
                    const bool low = e < -126.0f;
                    w = __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(fmaf(pp.sharpness, l, low ? 64.0f : 0.0f)), low ? -64 : 0);
                } else {
                    w = __builtin_amdgcn_exp2f(e);
                }
                m1 = fmaf(w, d, m1);
                m2 = fmaf(w, d * d, m2);
                den += w;
            }
        };
        uint32_t r = 0;
        if (!odd) {
            // Once the sums exceed 2^-80 a weight below 2^-126 times d^2 < 2^20
            // is less than half a unit in their last place, so that they do not
            // change whether it is flushed to zero or not: one instruction
            // instead of six for the power.
            bool tiny = true;
#pragma unroll 1
            for (; r + kFilterRays <= R; r += kFilterRays) {
                if (tiny) {
#pragma unroll
                    for (uint32_t u = 0; u < kFilterRays; ++u) add(s_ray[r + u], std::true_type{}, std::true_type{});
                    tiny = !(in.d_max < 1024.0f && __all(fminf(fminf(m1, m2), den) > 0x1p-80f));
                } else {
#pragma unroll
                    for (uint32_t u = 0; u < kFilterRays; ++u) add(s_ray[r + u], std::true_type{}, std::false_type{});
                }
            }
        }
        for (; r < R; ++r) add(s_ray[r], std::false_type{}, std::true_type{});
        // the stored old texel (first of quad (tx+1, ty+1)) as (mean, mean square);
        // the blend is kept as the format stores it (binary16: mean and variance)
        float2 ot[4];
        dep_texels<F16>(dold + F::kDepRec * (uint32_t)((ty + 1) * 17 + tx + 1), ot);
        const float2 old = ot[0];
        float n1 = den > 0.0f ? m1 / den : old.x;
        float n2 = den > 0.0f ? m2 / den : old.y;
        const float b1 = hy * old.x + (1.0f - hy) * n1, b2 = hy * old.y + (1.0f - hy) * n2;
        s_dep[t][0] = b1;
        s_dep[t][1] = F16 ? fmaf(-b1, b1, b2) : b2;
    }
    if (threadIdx.x < 64) {   // irradiance texel t (8x8)
        uint32_t t = threadIdx.x;
        uint32_t tx = t & 7u, ty = t >> 3;
        V3 nt = oct_decode(((float)tx + 0.5f) / 8.0f, ((float)ty + 0.5f) / 8.0f);
        V3 num = v3(0.0f, 0.0f, 0.0f);
        float den = 0.0f;
        const auto add = [&](const float4 ry, const float4 L, auto all) {
            float c = nt.x * ry.x + nt.y * ry.y + nt.z * ry.z;
            if (all || c > 0.0f) {
                if (all) c = fmaxf(c, 0.0f);
                num = v3(fmaf(c, L.x, num.x), fmaf(c, L.y, num.y), fmaf(c, L.z, num.z));
                den += c;
            }
        };
        uint32_t r = 0;
        if (!odd)
            for (; r + kFilterRays <= R; r += kFilterRays)
#pragma unroll
                for (uint32_t u = 0; u < kFilterRays; ++u) add(s_ray[r + u], s_L[r + u], std::true_type{});
        for (; r < R; ++r) add(s_ray[r], s_L[r], std::false_type{});
        const char *orec = iold + F::kIrrRec * nP * (size_t)((ty + 1) * 9 + tx + 1);
        const float4 old = F16 ? half4_to_float4(*reinterpret_cast<const uint2 *>(orec))
                               : *reinterpret_cast<const float4 *>(orec);
        float id = 1.0f / den;
        V3 nv = den > 0.0f ? id * num : xyz(old);
        s_irr[t][0] = hy * old.x + (1.0f - hy) * nv.x;
        s_irr[t][1] = hy * old.y + (1.0f - hy) * nv.y;
        s_irr[t][2] = hy * old.z + (1.0f - hy) * nv.z;
    }
    __syncthreads();
    // write quad records: each corner is an interior texel or the interior
    // texel its gutter position mirrors
    char *iout = reinterpret_cast<char *>(out.irr) + F::kIrrRec * (size_t)pi;
    char *dout = reinterpret_cast<char *>(out.dep) + F::kDepProbe * (size_t)pi;
    for (uint32_t q = threadIdx.x; q < (uint32_t)kDepQuads; q += kProbeBlock) {
        int cx = (int)(q % 17u), cy = (int)(q / 17u);
        int s0 = gutter_source(cx, cy, kDepN), s1 = gutter_source(cx + 1, cy, kDepN);
        int s2 = gutter_source(cx, cy + 1, kDepN), s3 = gutter_source(cx + 1, cy + 1, kDepN);
        if constexpr (F16) {
            *reinterpret_cast<uint4 *>(dout + F::kDepRec * q) =
                make_uint4(pack_half2(s_dep[s0][0], s_dep[s0][1]), pack_half2(s_dep[s1][0], s_dep[s1][1]),
                           pack_half2(s_dep[s2][0], s_dep[s2][1]), pack_half2(s_dep[s3][0], s_dep[s3][1]));
        } else {
            float4 *rec = reinterpret_cast<float4 *>(dout + F::kDepRec * q);
            rec[0] = make_float4(s_dep[s0][0], s_dep[s0][1], s_dep[s1][0], s_dep[s1][1]);
            rec[1] = make_float4(s_dep[s2][0], s_dep[s2][1], s_dep[s3][0], s_dep[s3][1]);
        }
    }
    for (uint32_t q = threadIdx.x; q < (uint32_t)kIrrQuads; q += kProbeBlock) {
        int cx = (int)(q % 9u), cy = (int)(q / 9u);
        int s0 = gutter_source(cx, cy, kIrrN), s1 = gutter_source(cx + 1, cy, kIrrN);
        int s2 = gutter_source(cx, cy + 1, kIrrN), s3 = gutter_source(cx + 1, cy + 1, kIrrN);
        char *rb = iout + F::kIrrRec * nP * q;
        if constexpr (F16) {
            // binary16 (nearest even), in the order of the FP32 corners
            uint2 *rec = reinterpret_cast<uint2 *>(rb);
            rec[0] = make_uint2(pack_half2(s_irr[s0][0], s_irr[s0][1]), pack_half2(s_irr[s0][2], s_irr[s1][0]));
            rec[1] = make_uint2(pack_half2(s_irr[s1][1], s_irr[s1][2]), pack_half2(s_irr[s2][0], s_irr[s2][1]));
            rec[2] = make_uint2(pack_half2(s_irr[s2][2], s_irr[s3][0]), pack_half2(s_irr[s3][1], s_irr[s3][2]));
        } else {
            float4 *rec = reinterpret_cast<float4 *>(rb);
            rec[0] = make_float4(s_irr[s0][0], s_irr[s0][1], s_irr[s0][2], s_irr[s1][0]);
            rec[1] = make_float4(s_irr[s1][1], s_irr[s1][2], s_irr[s2][0], s_irr[s2][1]);
            rec[2] = make_float4(s_irr[s2][2], s_irr[s3][0], s_irr[s3][1], s_irr[s3][2]);
        }
    }
}

// Q at a caller's points: probe_query's blend and sums, bit for bit on finite
// input, without the shortcuts that its callers' points allow.  The quotient
// is a division, so that points beyond every bound land in the outermost
// cell, and layers of weight zero are read, so that a texel that is no finite
// number shows.  One corner pair per iteration, with both probes' records
// loaded together, is also the faster form for points that are not sorted:
// 4,000,000 random ones, 65,536 binary16 probes 0.99 ms, probe_query 1.14
// (FP32 1.19 and 1.17).
struct PointAxis {
    float d0, d1, fr;
    uint32_t base, step;
};

__device__ __forceinline__ PointAxis point_axis(float pv, float lo, float sp, int na, uint32_t stride)
{
    PointAxis q;
    float g = (pv - lo) / sp - 0.5f;
    g = fminf(fmaxf(g, 0.0f), (float)(na - 1));
    const int b = min(max((int)floorf(g), 0), max(na - 2, 0));
    q.fr = na >= 2 ? g - (float)b : 0.0f;
    const int i1 = min(b + 1, na - 1);
    q.d0 = lo + ((float)b + 0.5f) * sp - pv;
    q.d1 = lo + ((float)i1 + 0.5f) * sp - pv;
    q.base = (uint32_t)b * stride;
    q.step = (uint32_t)(i1 - b) * stride;
    return q;
}

template <bool kF16>
__device__ __forceinline__ V3 point_query(const gi_probes &pr, V3 p, V3 n)
{
    using F = ProbeFmt<kF16>;
    const int nx = (int)pr.dims[0], ny = (int)pr.dims[1], nz = (int)pr.dims[2];
    const PointAxis ax = point_axis(p.x, pr.lo[0], pr.spacing[0], nx, 1u);
    const PointAxis ay = point_axis(p.y, pr.lo[1], pr.spacing[1], ny, (uint32_t)nx);
    const PointAxis az = point_axis(p.z, pr.lo[2], pr.spacing[2], nz, (uint32_t)(nx * ny));
    const uint32_t base = ax.base + ay.base + az.base;
    const Bilin bn = bilin(n, kIrrN);
    const uint32_t np = (uint32_t)(nx * ny * nz);
    const uint32_t irr_q = F::kIrrRec * (uint32_t)bn.q * np;   // slice of record q
    const __amdgpu_buffer_rsrc_t dep_r = tex_rsrc(pr.dep, np * F::kDepProbe);
    const __amdgpu_buffer_rsrc_t irr_r = tex_rsrc(pr.irr, np * (uint32_t)kIrrQuads * F::kIrrRec);
    const float w00 = (1.0f - bn.ax) * (1.0f - bn.ay), w10 = bn.ax * (1.0f - bn.ay);
    const float w01 = (1.0f - bn.ax) * bn.ay, w11 = bn.ax * bn.ay;
    float sx = 0.0f, sy = 0.0f, sz = 0.0f, wsum = 0.0f;
#pragma unroll 1
    for (int c = 0; c < 4; ++c) {
        const bool oy = (c & 1) != 0, oz = (c & 2) != 0;
        const float dy = oy ? ay.d1 : ay.d0, dz = oz ? az.d1 : az.d0;
        const float ty = oy ? ay.fr : 1.0f - ay.fr, tz = oz ? az.fr : 1.0f - az.fr;
        const uint32_t pyz = base + (oy ? ay.step : 0u) + (oz ? az.step : 0u);
#pragma unroll
        for (int ox = 0; ox < 2; ++ox) {
            const V3 tp = v3(ox ? ax.d1 : ax.d0, dy, dz);
            const float tx = ox ? ax.fr : 1.0f - ax.fr;
            const uint32_t pi = pyz + (ox ? ax.step : 0u);
            const float r2 = dot(tp, tp);
            const bool at_probe = !(r2 > 0.0f);
            const float ir = frsq(r2);
            const float r = r2 * ir;
            const float hh = 0.5f * (1.0f + dot(n, tp) * ir);
            // depth moments toward p (a probe sitting exactly at p reads any texel, unused)
            const V3 dv = at_probe ? v3(0.0f, 0.0f, 1.0f) : -tp;
            const Bilin bd = bilin(dv, kDepN);
            float2 d[4];
            dep_record<kF16>(dep_r, __umul24(pi, F::kDepProbe) + F::kDepRec * (uint32_t)bd.q, d);
            float4 e0, e1, e2;
            irr_record<kF16>(irr_r, irr_q + __umul24(pi, F::kIrrRec), e0, e1, e2);
            const float v00 = (1.0f - bd.ax) * (1.0f - bd.ay), v10 = bd.ax * (1.0f - bd.ay);
            const float v01 = (1.0f - bd.ax) * bd.ay, v11 = bd.ax * bd.ay;
            const float mu = v00 * d[0].x + v10 * d[1].x + v01 * d[2].x + v11 * d[3].x;
            const float mu2 = v00 * d[0].y + v10 * d[1].y + v01 * d[2].y + v11 * d[3].y;
            const float var = fmaxf(fmaf(-mu, mu, mu2), pr.var_floor);
            const float dd = r - mu;
            const float cheb = var * rcp(fmaf(dd, dd, var));
            const float vis = (!at_probe && r > mu) ? cheb * cheb * cheb : 1.0f;
            const float back = at_probe ? 0.45f : hh * hh + 0.2f;
            const float wgt = tx * ty * tz * fmaxf(back * vis, 1e-6f);
            sx = fmaf(wgt, w00 * e0.x + w10 * e0.w + w01 * e1.z + w11 * e2.y, sx);
            sy = fmaf(wgt, w00 * e0.y + w10 * e1.x + w01 * e1.w + w11 * e2.z, sy);
            sz = fmaf(wgt, w00 * e0.z + w10 * e1.y + w01 * e2.x + w11 * e2.w, sz);
            wsum += wgt;
        }
    }
    const float iw = rcp(wsum);
    return v3(iw * sx, iw * sy, iw * sz);
}

__global__ void k_probe_query(gi_probes pr, uint32_t n, const float *p, const float *nrm, float *out)
{
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const V3 a = ld3(p + 3 * i), b = ld3(nrm + 3 * i);
    const V3 q = pr.texel == GI_TEXEL_F16 ? point_query<true>(pr, a, b) : point_query<false>(pr, a, b);
    out[3 * i] = q.x;
    out[3 * i + 1] = q.y;
    out[3 * i + 2] = q.z;
}

// --------------------------------------------------------------------------
// initial resampling
// --------------------------------------------------------------------------
// Candidate planes of the learned-cache form of the initial pass: candidate
// i of pixel p at i*W*H + p; pos = (y or the miss direction, prim bits),
// nrm = (n_y, 0), q = cache value at (y, n_y).
struct CandWs {
    float4 *pos;
    float4 *nrm;
    float4 *q;
    uint32_t gate;   // kRunAlways, or run only when the cache is (kRunIfCache) / is not (kRunIfProbe) selected
};

// Gates of the learned cache's kernels in AUTO mode: the device decides per
// frame, so both forms are launched and the one not selected returns at once
// (a uniform exit before any barrier).
enum : uint32_t { kRunAlways = 0u, kRunIfCache = 1u, kRunIfProbe = 2u };

__device__ __forceinline__ bool gated_off(const CandWs &ws, const gi_mlp &mlp)
{
    return ws.gate != kRunAlways && (ws.gate == kRunIfCache) != mlp_selected(mlp);
}

// Traces the M candidates of every pixel into the candidate planes (the
// directions and hits k_initial computes itself in the probe form).
template <bool LDS>
__global__ void __launch_bounds__(kBlock)
    k_cand(gi_scene sc, gi_gbuffer gb, gi_params pp, CandWs ws, uint64_t seed, uint32_t frame, gi_mlp mlp)
{
    using Acc = typename std::conditional<LDS, GeoLds, GeoGlobal>::type;
    if (gated_off(ws, mlp)) return;
    uint32_t px, py;
    const bool inside = tile_pixel(gb.width, gb.height, px, py);
    if (LDS) stage_scene(sc);
    if (!inside) return;
    const Acc acc(sc);
    const uint32_t p = py * gb.width + px;
    const size_t npx = (size_t)gb.width * gb.height;
    const GB g = load_gb(gb, p);
    const float miss = __uint_as_float(GI_MISS);
    if (!active(g)) {
        for (uint32_t i = 0; i < pp.M; ++i) {
            ws.pos[i * npx + p] = make_float4(0.0f, 0.0f, 0.0f, miss);
            ws.nrm[i * npx + p] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        return;
    }
    const V3 o = madd(g.pos, sc.eps, g.n);
    for (uint32_t i = 0; i < pp.M; ++i) {
        uint4 rn = philox(seed, p, frame, kPassInitial, i);
        V3 w = cosine_dir(g.n, u01(rn.x), u01(rn.y));
        Hit h;
        float4 a, b = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (cast<false>(sc, acc, o, w, kInf, h)) {
            V3 y = madd(o, h.t, w), ny = hit_normal(sc, acc, o, w, h);
            a = make_float4(y.x, y.y, y.z, __uint_as_float(h.prim));
            b = make_float4(ny.x, ny.y, ny.z, 0.0f);
        } else {
            a = make_float4(w.x, w.y, w.z, miss);
        }
        ws.pos[i * npx + p] = a;
        ws.nrm[i * npx + p] = b;
    }
}

// Initial resampling.  WS = false: traces its candidates and queries the
// probes.  WS = true: takes the candidates from the planes k_cand wrote and,
// when the cache is selected, their cache values; otherwise the probe query
// of the same candidates, through the same arithmetic as WS = false.
// LIGHT: emitter candidates present (M_light > 0); without them the loop
// compiles to the plain cosine-candidate form.
// GLOSSY: the whole BSDF at x (Sec. 3.3): candidate directions from the
// mixture of the cosine and glossy lobes (lobe chosen by the candidate's
// fourth uniform), L_DDGI+ at the candidates with its glossy part (one lobe
// sample, counter (pixel, frame, 14, i)), weights p_hat over the mixture's
// density in area measure, residual f L (G - G_max) / p_A.
template <bool LDS, bool WS, bool LIGHT, bool GLOSSY, int TEX>
__global__ void __launch_bounds__(kBlock, 4)
    k_initial(gi_scene sc, gi_gbuffer gb, gi_probes pr, gi_params pp, gi_reservoirs out, float4 *resid,
              uint64_t seed, uint32_t frame, CandWs ws, gi_mlp mlp)
{
    using Acc = typename std::conditional<LDS, GeoLdsT<true>, GeoGlobal>::type;
    if (gated_off(ws, mlp)) return;
    uint32_t px, py;
    const bool inside = tile_pixel(gb.width, gb.height, px, py);
    if (LDS) stage_scene<true>(sc);
    if (!inside) return;
    const Acc acc(sc);
    const uint32_t p = py * gb.width + px;
    const GB g = load_gb<GLOSSY>(gb, p);
    if (!active<GLOSSY>(g)) {
        store_res(out, p, empty_res(0));
        resid[p] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        return;
    }
    const V3 o = madd(g.pos, sc.eps, g.n);
    const V3 rho_pi = kInvPi * g.alb;
    const float pg_x = GLOSSY ? p_gloss(g.alb, g.ks) : 0.0f;
    const bool use_cache = WS && mlp_selected(mlp);
    const size_t npx = (size_t)gb.width * gb.height;
    const uint32_t Mt = LIGHT ? pp.M + pp.M_light : pp.M;
    // balance heuristic: weights divide by the mixture density (M p_A + M_light p_light) / Mt
    const float mixb = (float)pp.M / (float)Mt, mixl = (float)pp.M_light / (float)Mt;
    Res r = empty_res(Mt);
    float wsum = 0.0f, p_sel = 0.0f;
    bool have = false;
    // The selected candidate so far, (y, tag), (n_y, prim), (L, -), and
    // candidate 0's residual wait in this thread's LDS slot past the staged
    // scene: kept in registers across the probe query they would push the
    // loop's invariants into scratch.
    float4 *const sel = reinterpret_cast<float4 *>(reinterpret_cast<char *>(gi_lds) + (LDS ? lds_scene_bytes(sc) : 0u)) +
                        4u * threadIdx.x;
    sel[3] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    // subsampling: a pixel off the pattern draws no candidates, only the residual's
    const bool draws = pp.subsample <= 1u || ((uint64_t)px + py + frame) % pp.subsample == 0u;
    for (uint32_t i = 0; i < (draws ? Mt : 1u); ++i) {
        uint4 rn = philox(seed, p, frame, kPassInitial, i);
        float u2 = u01(rn.z);
        V3 w, y, ny = v3(0.0f, 0.0f, 0.0f), L = v3(0.0f, 0.0f, 0.0f);
        float phat = 0.0f, wi = 0.0f;
        uint32_t prim = GI_MISS;
        bool hit;
        if (LIGHT && i >= pp.M) {
            // emitter candidate: a point uniform in the area of a uniformly chosen emitter
            u2 = u01(rn.w);
            hit = sc.n_emitters > 0u;
            if (hit) {
                const uint32_t e = min((uint32_t)(u01(rn.x) * (float)sc.n_emitters), sc.n_emitters - 1u);
                prim = sc.emitters[e];
                const float4 c = reinterpret_cast<const float4 *>(sc.prims)[4 * prim];
                const float rad = reinterpret_cast<const float4 *>(sc.prims)[4 * prim + 1].x;
                const V3 d = sphere_dir(u01(rn.y), u01(rn.z));
                y = madd(xyz(c), rad, d);
                ny = d;
            }
        } else if constexpr (WS) {
            const float4 a = ws.pos[i * npx + p];
            w = xyz(a);
            hit = __float_as_uint(a.w) != GI_MISS;
            if (hit) {
                y = w;
                ny = xyz(ws.nrm[i * npx + p]);
                prim = __float_as_uint(a.w);
            }
        } else {
            bool dir_ok = true;
            if (GLOSSY && pg_x > 0.0f && u01(rn.w) < pg_x) dir_ok = ggx_sample(g.n, g.wo, g.rough, u01(rn.x), u01(rn.y), w);
            else w = cosine_dir(g.n, u01(rn.x), u01(rn.y));
            Hit h;
            hit = dir_ok && cast<false>(sc, acc, o, w, kInf, h);
            if (hit) {
                y = madd(o, h.t, w);
                ny = hit_normal(sc, acc, o, w, h);
                prim = h.prim;
            }
            if (GLOSSY && !dir_ok) w = v3(0.0f, 0.0f, 0.0f);   // no candidate: neither surface nor sky
        }
        if (hit) {
            V3 v = y - g.pos;
            float d2 = dot(v, v);
            V3 wv = frsq(d2) * v;
            float cx = dot(g.n, wv), cy = -dot(ny, wv);
            if (cx > 0.0f && cy > 0.0f) {
                if constexpr (GLOSSY) {
                    const uint4 rg = philox(seed, p, frame, kPassGlossyCand, i);
                    L = radiance_toward_g<TEX>(sc, pr, prim, y, ny, g.pos, u01(rg.x), u01(rg.y));
                    const V3 f = bsdf(g.alb, g.ks, g.rough, g.n, g.wo, wv) * L;
                    const float G = cx * cy * rcp(d2);
                    const float pA = mix_pdf(g.alb, g.ks, g.rough, g.n, g.wo, wv) * cy * rcp(d2);
                    phat = lum(f) * fminf(G, pp.g_max);
                    if (!LIGHT)
                        wi = pA > 0.0f ? phat * rcp(pA) : 0.0f;
                    else
                        wi = phat * rcp(mixb * pA + mixl * light_pdf(sc, prim));
                    if (i == 0 && G > pp.g_max && pA > 0.0f) { const V3 q = ((G - pp.g_max) * rcp(pA)) * f; sel[3] = make_float4(q.x, q.y, q.z, 0.0f); }
                } else {
                    // (binary16 records: the query unrolled over two corner pairs is the
                    // faster form here; FP32 records: one pair, which needs no spills)
                    L = (use_cache && i < pp.M) ? radiance_cached(sc, prim, ws.q[i * npx + p])
                                                : radiance_toward<TEX == kTexF16 ? 2 : 1, TEX>(sc, pr, prim, y, ny, g.pos);
                    float G = cx * cy * rcp(d2);
                    float fl = lum(rho_pi * L);
                    float iG = rcp(G);
                    phat = fl * fminf(G, pp.g_max);
                    if (!LIGHT)
                        wi = kPi * phat * iG;   // p_hat / p_A with p_A = G / pi
                    else
                        wi = phat * rcp(mixb * kInvPi * G + mixl * light_pdf(sc, prim));
                    if (i == 0 && G > pp.g_max) { const V3 q = (1.0f - pp.g_max * iG) * (g.alb * L); sel[3] = make_float4(q.x, q.y, q.z, 0.0f); }
                }
            }
        } else if ((!LIGHT || i < pp.M) && (!GLOSSY || !is_zero(w))) {
            y = w;
            L = ld3(sc.sky);
            float cx = dot(g.n, w);
            if (cx > 0.0f) {
                if constexpr (GLOSSY) {
                    phat = lum(bsdf(g.alb, g.ks, g.rough, g.n, g.wo, w) * L) * cx;
                    const float pd = mix_pdf(g.alb, g.ks, g.rough, g.n, g.wo, w);
                    wi = pd > 0.0f ? phat * rcp(pd) : 0.0f;
                } else {
                    phat = lum(rho_pi * L) * cx;
                    wi = kPi * phat * rcp(cx);
                }
                if (LIGHT) wi *= rcp(mixb);
            }
        }
        if (!draws) break;
        wsum += wi;
        if (u2 * wsum < wi) {
            have = true;
            p_sel = phat;
            sel[0] = make_float4(y.x, y.y, y.z, __uint_as_float(((p & 0x7FFFFFu) << 9) | ((i & 31u) << 4) | (frame & 15u)));
            sel[1] = make_float4(ny.x, ny.y, ny.z, __uint_as_float(prim));
            sel[2] = make_float4(L.x, L.y, L.z, 0.0f);
        }
    }
    if (have) {
        const float4 a = sel[0], b = sel[1], c = sel[2];
        r.y = xyz(a);
        r.tag = __float_as_uint(a.w);
        r.n = xyz(b);
        r.prim = __float_as_uint(b.w);
        r.L = xyz(c);
    }
    r.wsum = wsum;
    if (!draws) r = empty_res(0);
    r.W = (have && p_sel > 0.0f) ? wsum * rcp((float)Mt * p_sel) : 0.0f;
    store_res(out, p, r);
    resid[p] = sel[3];
}

// --------------------------------------------------------------------------
// initial resampling by tiles
// --------------------------------------------------------------------------
// The probe form without emitter candidates, one workgroup per image tile.
// The candidate rays of all the tile's pixels are sorted by direction before
// they are traced and shaded: a wave's 64 rays then run through the same
// primitive lists (gi_lists.hpp) and land on the same surfaces, so its lanes
// stay together in the walk and its probe gathers share cache lines.  The
// RIS weights go back through LDS, where each pixel's owner streams them in
// candidate order; a second pass evaluates the selected candidates again and
// writes the reservoirs.  Every candidate goes through the arithmetic of
// k_initial and the weights are summed in its order, so the results are those
// of k_initial bit for bit.
// Bound by vector-ALU issue (0.87 of the peak at 1920x1080, M = 32) and as
// much by the L1's return path (0.85: the five 16-byte loads of a probe take
// about 35 cycles each, one per distinct line of four lanes).  Some of the
// issue is register traffic: the thread's own pixel lives across the trace, so
// 23 VGPRs (96 B a lane) and 75 scalars spill, 60 and 114 in the glossy forms,
// and a 1920x1080 launch writes 643 MB for 141 MB of output.  Against the
// pixel form, M = 32: 250x141 0.734 -> 0.218 ms, 1920x1080 5.77 -> 3.08 ms,
// with glossy layers 8.86 -> 5.20 ms, 3840x2160 with 1024 primitives 46.5 ->
// 21.3 ms.  512 threads and up to 80 KB let two workgroups share a CU, one
// tracing while the other sorts (one workgroup of 1024 threads: 4.7 ms against
// 3.9 at 1920x1080, when that was chosen).
constexpr int kTileBlock = 512;
constexpr uint32_t kTileLds = 80u * 1024u;                // LDS of a workgroup: two share a CU
constexpr uint32_t kSortBins = 4u * kBins;

// LDS after the lists: a word per ray (its sort key, then its weight), the
// ray order, the pixels' weight sums, the cells' counts; with kPx the pixels'
// position, normal and albedo
__host__ __device__ constexpr uint32_t tile_bytes(uint32_t rays, uint32_t pixels, bool px)
{
    return rays * 6u + pixels * (px ? 40u : 4u) + (kSortBins + 8u) * 4u;
}

// minimum over a wave by DPP moves: quads, rows of 16, then row totals
// broadcast into the next row and half (the wave's minimum ends in lane 63)
template <int kCtrl>
__device__ __forceinline__ float dpp_min(float v)
{
    const int i = __builtin_bit_cast(int, v);
    return fminf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, kCtrl, 0xF, 0xF, false)));
}
__device__ __forceinline__ float wave_min(float v)
{
    v = dpp_min<0xB1>(v);      // quad_perm [1, 0, 3, 2]
    v = dpp_min<0x4E>(v);      // quad_perm [2, 3, 0, 1]
    v = dpp_min<0x141>(v);     // row_half_mirror
    v = dpp_min<0x140>(v);     // row_mirror
    v = dpp_min<0x142>(v);     // row_bcast:15
    v = dpp_min<0x143>(v);     // row_bcast:31
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// boxes around every thread's p and q (threads with `on` only; the boxes'
// half extents are not >= 0 if there is none); red: 12 floats per wave.  Ends
// with a barrier.
template <int NT>
__device__ __forceinline__ void block_boxes(V3 p, V3 q, bool on, float4 *red, Box3 &bp, Box3 &bq)
{
    const float a[12] = {p.x, p.y, p.z, -p.x, -p.y, -p.z, q.x, q.y, q.z, -q.x, -q.y, -q.z};
    float m[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) m[i] = wave_min(on ? a[i] : kInf);
    if ((threadIdx.x & 63u) == 0u)
#pragma unroll
        for (int i = 0; i < 3; ++i) red[3u * (threadIdx.x >> 6) + i] = make_float4(m[4 * i], m[4 * i + 1], m[4 * i + 2], m[4 * i + 3]);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NT / 64; ++w)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const float4 v = red[3 * w + i];
            m[4 * i] = fminf(m[4 * i], v.x);
            m[4 * i + 1] = fminf(m[4 * i + 1], v.y);
            m[4 * i + 2] = fminf(m[4 * i + 2], v.z);
            m[4 * i + 3] = fminf(m[4 * i + 3], v.w);
        }
    __syncthreads();
    const auto box = [&](const float *v) {
        return Box3{v3(0.5f * (v[0] - v[3]), 0.5f * (v[1] - v[4]), 0.5f * (v[2] - v[5])),
                    v3(-0.5f * (v[0] + v[3]), -0.5f * (v[1] + v[4]), -0.5f * (v[2] + v[5]))};
    };
    bp = box(m);
    bq = box(m + 6);
}

// counts -> first positions of kCells cells, the total behind them (one wave)
template <uint32_t kCells>
__device__ __forceinline__ void bin_starts(uint32_t *hist)
{
    constexpr uint32_t kPer = (kCells + 63u) / 64u;
    const uint32_t l = threadIdx.x & 63u;
    uint32_t c[kPer], s = 0u;
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        c[q] = kPer * l + q < kCells ? hist[kPer * l + q] : 0u;
        s += c[q];
    }
    uint32_t a = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(a, o, 64);
        if ((int)l >= o) a += v;
    }
    if (l == 63u) hist[kCells] = a;
    a -= s;
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        if (kPer * l + q < kCells) hist[kPer * l + q] = a;
        a += c[q];
    }
}

// pixel k of a tile of 2^lw x 2^lh pixels: 8x8 sub-tiles in row-major order
// (tiles below 8 pixels wide are one sub-tile)
__device__ __forceinline__ void tile_pixel_of(uint32_t k, uint32_t lw, uint32_t lh, uint32_t &px, uint32_t &py)
{
    const uint32_t l = k & 63u, s = k >> 6, sw = lw > 3u ? lw - 3u : 0u, rw = min(lw, 3u);
    px = (blockIdx.x << lw) + ((s & ((1u << sw) - 1u)) << 3) + (l & ((1u << rw) - 1u));
    py = (blockIdx.y << lh) + ((s >> sw) << 3) + (l >> rw);
}

// Tiles of 2^lw x 2^lh pixels (at most NT, and at most 2^16 candidates).
template <bool GLOSSY, int TEX, int NT, bool PX>
__global__ void __launch_bounds__(NT, 4)
    k_initial_tile(gi_scene sc, gi_gbuffer gb, gi_probes pr, gi_params pp, gi_reservoirs out, float4 *resid,
                   uint64_t seed, uint32_t frame, uint32_t lw, uint32_t lh, uint32_t C, CandWs ws, gi_mlp mlp)
{
    if (gated_off(ws, mlp)) return;
    const uint32_t t = threadIdx.x, TP = 1u << (lw + lh), M = pp.M;
    TileLists lists(gi_lds, sc.n_prims);
    uint32_t *const word = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(gi_lds) + list_bytes(sc.n_prims));
    float *const sum = reinterpret_cast<float *>(word + (C << (lw + lh)));
    uint32_t *const hist = reinterpret_cast<uint32_t *>(sum + TP);
    float *const pxd = reinterpret_cast<float *>(hist + kSortBins + 8u);
    uint16_t *const order = reinterpret_cast<uint16_t *>(pxd + (PX ? 9u * TP : 0u));

    const auto pixel_of = [&](uint32_t k, uint32_t &px, uint32_t &py) { tile_pixel_of(k, lw, lh, px, py); };
    // this thread's pixel: it generates rays of it, and owns it if t < TP
    const uint32_t k_own = t & (TP - 1u);
    uint32_t px, py;
    pixel_of(k_own, px, py);
    const uint32_t p_own = py * gb.width + px;
    GB own{};
    bool on = false;
    V3 org = v3(0.0f, 0.0f, 0.0f);
    if (px < gb.width && py < gb.height) {
        own = load_gb<GLOSSY>(gb, p_own);
        on = active<GLOSSY>(own);
        org = madd(own.pos, sc.eps, own.n);
        if (!on && t < TP) {
            store_res(out, p_own, empty_res(0));
            resid[p_own] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    }
    {
        Box3 ob, nb;
        // (at.x < kInf always holds.  The Lambertian forms spill 27 fewer scalars
        // when the boxes have a mask of their own beside `on`, which lives on:
        // 3840x2160, 1024 primitives: 21.4 ms, with `on` 21.9; the glossy ones
        // more: 1920x1080 5.29 ms with `on`, 5.35 without)
        const V3 at = list_origin(org);
        block_boxes<NT>(at, list_axis(org, own.n), GLOSSY ? on : on && at.x < kInf, reinterpret_cast<float4 *>(word), ob, nb);
        if (__syncthreads_or(on) == 0) return;             // no pixel of the tile is active
        build_lists<NT>(sc, lists, ob, nb, word);          // in the rays' space
    }
    if (PX && t < TP) {
        const float v[9] = {own.pos.x, own.pos.y, own.pos.z, own.n.x, own.n.y, own.n.z, own.alb.x, own.alb.y, own.alb.z};
#pragma unroll
        for (uint32_t c = 0; c < 9u; ++c) pxd[c * TP + t] = v[c];
    }

    const bool draws = pp.subsample <= 1u || ((uint64_t)px + py + frame) % pp.subsample == 0u;
    const uint32_t mine = on ? (draws ? M : 1u) : 0u;      // candidates of this thread's pixel
    const float pg = GLOSSY ? p_gloss(own.alb, own.ks) : 0.0f;
    uint32_t chosen = ~0u;
    float wsum = 0.0f;
    // rounds of C candidates per pixel, then one of the selected candidates
#pragma unroll 1
    for (uint32_t base = 0;; base += C) {
        const bool last = base >= M;
        for (uint32_t b = t; b < kSortBins; b += NT) hist[b] = 0u;
        __syncthreads();
        // keys: the ray's cell in its list's cell, and its rank there
        const uint32_t n_gen = last ? TP : min(C, M - base) << (lw + lh);
        for (uint32_t e = t; e < n_gen; e += NT) {
            const uint32_t i = last ? chosen : base + (e >> (lw + lh));
            if (last ? i == ~0u : i >= mine) {
                word[e] = ~0u;
                continue;
            }
            const uint4 rn = philox<true>(seed, p_own, frame, kPassInitial, i);
            V3 w;
            bool ok = true;
            if (GLOSSY && pg > 0.0f && u01(rn.w) < pg) ok = ggx_sample(own.n, own.wo, own.rough, u01(rn.x), u01(rn.y), w);
            else w = cosine_dir(own.n, u01(rn.x), u01(rn.y));
            const uint32_t b = ok ? sort_bin_of(w) : 0u;
            word[e] = b | (atomicAdd(&hist[b], 1u) << 16);
        }
        __syncthreads();
        if (t < 64u) bin_starts<kSortBins>(hist);
        __syncthreads();
        for (uint32_t e = t; e < n_gen; e += NT) {
            const uint32_t v = word[e];
            if (v != ~0u) order[hist[v & 0xFFFFu] + (v >> 16)] = (uint16_t)(last ? (chosen << (lw + lh)) | e : e);
        }
        __syncthreads();
        const uint32_t total = hist[kSortBins];
        for (uint32_t at = t; at < total; at += NT) {
            const uint32_t r = order[at], k = r & (TP - 1u), i = (r >> (lw + lh)) + (last ? 0u : base);
            const uint32_t b = (word[last ? k : r] & 0xFFFFu) >> 2;
            uint32_t qx, qy;
            pixel_of(k, qx, qy);
            const uint32_t p = qy * gb.width + qx;
            GB g;
            if constexpr (PX) {
                g.pos = v3(pxd[k], pxd[TP + k], pxd[2u * TP + k]);
                g.n = v3(pxd[3u * TP + k], pxd[4u * TP + k], pxd[5u * TP + k]);
                g.alb = v3(pxd[6u * TP + k], pxd[7u * TP + k], pxd[8u * TP + k]);
            } else {
                g = load_gb<GLOSSY>(gb, p);
            }
            const V3 o = madd(g.pos, sc.eps, g.n);
            const uint4 rn = philox<true>(seed, p, frame, kPassInitial, i);
            V3 w, y = v3(0.0f, 0.0f, 0.0f), ny = y, L = y, res0 = y;
            float phat = 0.0f, wi = 0.0f;
            uint32_t prim = GI_MISS;
            bool dir_ok = true, lobe = false;
            if constexpr (GLOSSY) {
                const float pgx = p_gloss(g.alb, g.ks);
                lobe = pgx > 0.0f && u01(rn.w) < pgx;
                if (lobe) dir_ok = ggx_sample(g.n, g.wo, g.rough, u01(rn.x), u01(rn.y), w);
            }
            if (!lobe) w = cosine_dir(g.n, u01(rn.x), u01(rn.y));
            Hit h;
            uint32_t slot;
            const bool hit = dir_ok && cast_lists(sc, lists, b, o, w, h, slot);
            if (hit) {
                ny = list_normal(lists, o, w, h.t, slot, h.axis);
                y = madd(o, h.t, w);
                prim = h.prim;
                const V3 v = y - g.pos;
                const float d2 = dot(v, v);
                const V3 wv = frsq(d2) * v;
                const float cx = dot(g.n, wv), cy = -dot(ny, wv);
                if (cx > 0.0f && cy > 0.0f) {
                    if constexpr (GLOSSY) {
                        const uint4 rg = philox<true>(seed, p, frame, kPassGlossyCand, i);
                        L = radiance_toward_g<TEX>(sc, pr, prim, y, ny, g.pos, u01(rg.x), u01(rg.y));
                        const V3 f = bsdf(g.alb, g.ks, g.rough, g.n, g.wo, wv) * L;
                        const float G = cx * cy * rcp(d2);
                        const float pA = mix_pdf(g.alb, g.ks, g.rough, g.n, g.wo, wv) * cy * rcp(d2);
                        phat = lum(f) * fminf(G, pp.g_max);
                        wi = pA > 0.0f ? phat * rcp(pA) : 0.0f;
                        if (i == 0 && G > pp.g_max && pA > 0.0f) res0 = ((G - pp.g_max) * rcp(pA)) * f;
                    } else {
                        L = radiance_toward<TEX == kTexF16 ? 2 : 1, TEX>(sc, pr, prim, y, ny, g.pos);
                        const float G = cx * cy * rcp(d2);
                        const float fl = lum((kInvPi * g.alb) * L);
                        const float iG = rcp(G);
                        phat = fl * fminf(G, pp.g_max);
                        wi = kPi * phat * iG;   // p_hat / p_A with p_A = G / pi
                        if (i == 0 && G > pp.g_max) res0 = (1.0f - pp.g_max * iG) * (g.alb * L);
                    }
                }
            } else if (!GLOSSY || dir_ok) {
                y = w;
                L = ld3(sc.sky);
                const float cx = dot(g.n, w);
                if (cx > 0.0f) {
                    if constexpr (GLOSSY) {
                        phat = lum(bsdf(g.alb, g.ks, g.rough, g.n, g.wo, w) * L) * cx;
                        const float pd = mix_pdf(g.alb, g.ks, g.rough, g.n, g.wo, w);
                        wi = pd > 0.0f ? phat * rcp(pd) : 0.0f;
                    } else {
                        phat = lum((kInvPi * g.alb) * L) * cx;
                        wi = kPi * phat * rcp(cx);
                    }
                }
            }
            if (!last) {
                word[r] = __float_as_uint(wi);
                if (i == 0u) resid[p] = make_float4(res0.x, res0.y, res0.z, 0.0f);
            } else {
                Res s{y, 0.0f, ny, sum[k], L, M, ((p & 0x7FFFFFu) << 9) | (i << 4) | (frame & 15u), prim};
                s.W = phat > 0.0f ? s.wsum * rcp((float)M * phat) : 0.0f;
                store_res(out, p, s);
            }
        }
        if (last) break;
        __syncthreads();
        // the owners stream their candidates in order
        if (t < TP && on) {
            const uint32_t end = min(base + C, draws ? M : 0u);
#pragma unroll 4
            for (uint32_t i = base; i < end; ++i) {
                const float wi = __uint_as_float(word[((i - base) << (lw + lh)) + t]);
                wsum += wi;
                if (u01(philox<true>(seed, p_own, frame, kPassInitial, i).z) * wsum < wi) chosen = i;
            }
            sum[t] = wsum;
            if (base + C >= M && chosen == ~0u) {
                Res r = empty_res(draws ? M : 0u);
                r.wsum = wsum;
                store_res(out, p_own, r);
            }
        }
    }
}

// The candidate trace of the learned-cache form by tiles: k_cand's planes, bit
// for bit, from the sorted rays and primitive lists of k_initial_tile.  A
// thread keeps the directions of its RPT rays per round; through LDS go the
// directions in sorted order, which their hits overwrite, and each ray's place.
// Only the hits come back, so that a wave writes whole lines of the planes.
// Bound by vector issue and the L1's return path, as k_initial_tile is, and by
// the planes' 32 B a candidate: 1920x1080, M = 32, 256 primitives, the trace
// alone 3.1 -> 2.0 ms (2.1 GB of planes: 1.1 TB/s).
constexpr uint32_t cand_bytes(uint32_t rays, uint32_t pixels) { return rays * 14u + pixels * 12u + (kBins + 8u) * 4u; }

template <int RPT>
__global__ void __launch_bounds__(kTileBlock, 4)
    k_cand_tile(gi_scene sc, gi_gbuffer gb, gi_params pp, CandWs ws, uint64_t seed, uint32_t frame, uint32_t lw,
                uint32_t lh, gi_mlp mlp)
{
    if (gated_off(ws, mlp)) return;
    constexpr uint32_t kRays = (uint32_t)kTileBlock * RPT;
    const uint32_t t = threadIdx.x, TP = 1u << (lw + lh), M = pp.M, C = kRays >> (lw + lh);
    TileLists lists(gi_lds, sc.n_prims);
    float *const ray = reinterpret_cast<float *>(reinterpret_cast<char *>(gi_lds) + list_bytes(sc.n_prims));
    uint32_t *const hist = reinterpret_cast<uint32_t *>(ray + 3u * kRays);
    float *const orgs = reinterpret_cast<float *>(hist + kBins + 8u);
    uint16_t *const owner = reinterpret_cast<uint16_t *>(orgs + 3u * TP);     // pixel (low) of the sorted rays

    const uint32_t k = t & (TP - 1u);
    uint32_t px, py;
    tile_pixel_of(k, lw, lh, px, py);
    const bool inside = px < gb.width && py < gb.height;
    const uint32_t p = py * gb.width + px;
    const size_t npx = (size_t)gb.width * gb.height;
    V3 org = v3(0.0f, 0.0f, 0.0f), nrm = org;
    bool on = false;
    if (inside) {
        const GB g = load_gb(gb, p);
        on = active(g);
        org = madd(g.pos, sc.eps, g.n);
        nrm = g.n;
    }
    {
        Box3 ob, nb;
        block_boxes<kTileBlock>(list_origin(org), list_axis(org, nrm), on, reinterpret_cast<float4 *>(ray), ob, nb);
        if (__syncthreads_or(on) != 0) build_lists<kTileBlock>(sc, lists, ob, nb, reinterpret_cast<uint32_t *>(ray));
    }
    if (t < TP) {
        orgs[t] = org.x;
        orgs[TP + t] = org.y;
        orgs[2u * TP + t] = org.z;
    }
    const float miss = __uint_as_float(GI_MISS);
#pragma unroll 1
    for (uint32_t base = 0; base < M; base += C) {
        for (uint32_t b = t; b < (uint32_t)kBins; b += kTileBlock) hist[b] = 0u;
        __syncthreads();
        V3 w[RPT];
        uint32_t at[RPT];
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const uint32_t i = base + (((uint32_t)j * kTileBlock + t) >> (lw + lh));
            at[j] = ~0u;
            if (!on || i >= M) continue;
            const uint4 rn = philox<true>(seed, p, frame, kPassInitial, i);
            w[j] = cosine_dir(nrm, u01(rn.x), u01(rn.y));
            const uint32_t b = sort_bin_of(w[j]) >> 2;
            at[j] = b | (atomicAdd(&hist[b], 1u) << 16);
        }
        __syncthreads();
        if (t < 64u) bin_starts<kBins>(hist);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            if (at[j] == ~0u) continue;
            const uint32_t b = at[j] & 0xFFFFu, a = hist[b] + (at[j] >> 16);
            at[j] = a;
            ray[a] = w[j].x;
            ray[kRays + a] = w[j].y;
            ray[2u * kRays + a] = w[j].z;
            owner[a] = (uint16_t)k;
        }
        __syncthreads();
        for (uint32_t a = t; a < hist[kBins]; a += kTileBlock) {
            const V3 d = v3(ray[a], ray[kRays + a], ray[2u * kRays + a]);
            const uint32_t q = owner[a];
            Hit h;
            uint32_t slot;
            cast_lists(sc, lists, sort_bin_of(d) >> 2, v3(orgs[q], orgs[TP + q], orgs[2u * TP + q]), d, h, slot);
            ray[a] = h.t;
            // slot, or 2^16 + a wall's index, or ~0 for a miss
            reinterpret_cast<uint32_t *>(ray)[kRays + a] = slot != ~0u ? slot : (h.prim == GI_MISS ? ~0u : 0x10000u + (h.prim - sc.n_prims));
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const uint32_t i = base + (((uint32_t)j * kTileBlock + t) >> (lw + lh));
            if (!inside || i >= M) continue;
            float4 a = make_float4(0.0f, 0.0f, 0.0f, miss), b = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (at[j] != ~0u) {
                const float ht = ray[at[j]];
                uint32_t slot = reinterpret_cast<uint32_t *>(ray)[kRays + at[j]];
                if (slot == ~0u) {
                    a = make_float4(w[j].x, w[j].y, w[j].z, miss);
                } else {
                    const V3 y = madd(org, ht, w[j]);
                    uint32_t prim;
                    int axis = 0;
                    if (slot >= 0x10000u) {
                        prim = sc.n_prims + (slot - 0x10000u);
                        axis = (int)((slot - 0x10000u) >> 1);
                        slot = ~0u;
                    } else {
                        prim = lists.ids[slot];
                    }
                    const V3 ny = list_normal(lists, org, w[j], ht, slot, axis);
                    a = make_float4(y.x, y.y, y.z, __uint_as_float(prim));
                    b = make_float4(ny.x, ny.y, ny.z, 0.0f);
                }
            }
            ws.pos[i * npx + p] = a;
            ws.nrm[i * npx + p] = b;
        }
        __syncthreads();
    }
}

// --------------------------------------------------------------------------
// reservoir merging (temporal and spatial reuse)
// --------------------------------------------------------------------------
struct Merge {
    float wsum;
    uint32_t Msum;
    bool have;
    Res sel;
};

template <bool GLOSSY = false>
__device__ __forceinline__ void merge_in(Merge &m, const GB &g, const Res &q, uint32_t Mq, float u, float g_max)
{
    float w = 0.0f;
    if (q.W > 0.0f && Mq > 0u) w = res_target<GLOSSY>(g, q, g_max) * q.W * (float)Mq;
    m.wsum += w;
    m.Msum += Mq;
    if (u * m.wsum < w) {
        m.have = true;
        m.sel = q;
    }
}


// Normalise the merged reservoir.  Domain slot j holds M_j (0 = slot unused:
// a neighbour that was rejected or never drawn) and is loaded by dom(j);
// slot 0 is the pixel itself.  Slots are static so that the unrolled loop
// keeps everything in registers.
template <bool GLOSSY, int ND, class DomFn, class G>
__device__ __forceinline__ Res finish(const gi_scene &sc, const G &acc, const Merge &m, const GB &g,
                                      const uint32_t (&Mdom)[ND], DomFn dom, const gi_params &pp)
{
    if (!m.have) {
        Res e = empty_res(m.Msum);
        e.wsum = m.wsum;
        return e;
    }
    Res r = m.sel;
    float ph = res_target<GLOSSY>(g, r, pp.g_max);
    float Z;
    bool keep = true;
    if (pp.unbiased) {
        // W is zero unless x sees y and p_hat(y) > 0; the domains' rays only
        // decide Z, so they are cast only then (the result is the same)
        bool sky = is_zero(r.n);
        bool vis_x = ph > 0.0f && visible(sc, acc, g.pos, g.n, r.y, r.n, sky);
        keep = vis_x;
        uint32_t z = vis_x ? Mdom[0] : 0u;     // the target at x supports y (it was chosen)
        if (vis_x) {
#pragma unroll
            for (int j = 1; j < ND; ++j) {
                if (Mdom[j] == 0u) continue;
                GB q = dom(j);
                if (res_target<GLOSSY>(q, r, pp.g_max) <= 0.0f) continue;
                if (visible(sc, acc, q.pos, q.n, r.y, r.n, sky)) z += Mdom[j];
            }
        }
        Z = (float)z;
    } else {
        Z = (float)m.Msum;
    }
    r.wsum = m.wsum;
    r.M = m.Msum;
    r.W = (keep && Z > 0.0f && ph > 0.0f) ? m.wsum * rcp(Z * ph) : 0.0f;
    return r;
}

__device__ __forceinline__ int reproject(const gi_camera &c, V3 x)
{
    V3 v = x - ld3(c.eye);
    float z = dot(v, ld3(c.fwd));
    if (z <= 0.0f) return -1;
    float aspect = (float)c.width / (float)c.height;
    float sx = dot(v, ld3(c.right)) / (z * c.tan_half_fovy * aspect);
    float sy = dot(v, ld3(c.up)) / (z * c.tan_half_fovy);
    float fx = floorf((sx + 1.0f) * 0.5f * (float)c.width);
    float fy = floorf((1.0f - sy) * 0.5f * (float)c.height);
    if (!(fx >= 0.0f && fy >= 0.0f && fx < (float)c.width && fy < (float)c.height)) return -1;
    return (int)fy * (int)c.width + (int)fx;
}

// 8 waves per SIMD: the latency-bound gathers and walks gain more from
// occupancy than they lose to a few spilled values
template <bool LDS, bool GLOSSY, uint32_t SW>
__global__ void __launch_bounds__(SW * kTile, SW == 16u ? 8 : 6)
    k_temporal(gi_scene sc, gi_gbuffer gb, gi_gbuffer gbp, gi_camera cam_prev, gi_reservoirs cur,
               gi_reservoirs hist, gi_params pp, uint32_t m_hist_cap, gi_reservoirs out, uint64_t seed,
               uint32_t frame)
{
    using Acc = typename std::conditional<SW != (uint32_t)kTile, GeoSmall, typename std::conditional<LDS, GeoLds, GeoGlobal>::type>::type;
    uint32_t px, py;
    const bool inside = tile_pixel<SW>(gb.width, gb.height, px, py);
    if constexpr (SW != (uint32_t)kTile) {
        stage_small(sc);
        __syncthreads();
    } else if (LDS) {
        stage_scene(sc);
    }
    if (!inside) return;
    const Acc acc(sc);
    const uint32_t p = py * gb.width + px;
    const GB g = load_gb<GLOSSY>(gb, p);
    const Res rc = load_res(cur, p);
    if (!active<GLOSSY>(g)) {
        store_res(out, p, rc);
        return;
    }
    Merge m{0.0f, 0u, false, rc};
    uint32_t Mdom[2] = {rc.M, 0u};
    uint32_t qprev = 0u;
    merge_in<GLOSSY>(m, g, rc, rc.M, 0.0f, pp.g_max);
    int q = reproject(cam_prev, g.pos);
    if (q >= 0) {
        GB gq = load_gb<GLOSSY>(gbp, (uint32_t)q);
        if (similar(g, gq, pp)) {
            Res rh = load_res(hist, (uint32_t)q);
            const uint32_t Mh = min(rh.M, m_hist_cap);
            uint4 rn = philox(seed, p, frame, kPassTemporal, 0u);
            merge_in<GLOSSY>(m, g, rh, Mh, u01(rn.x), pp.g_max);
            Mdom[1] = Mh;
            qprev = (uint32_t)q;
        }
    }
    store_res(out, p, finish<GLOSSY>(sc, acc, m, g, Mdom, [&](int) { return load_gb<GLOSSY>(gbp, qprev); }, pp));
}

// The temporal pass of an image of few pixels: an 8x8 tile's two rays per
// pixel go to a wave each instead of one after the other, and the tiles to four
// times as many CUs.  Bound by the latency of one walk; k_temporal -> this:
// 64x64, 8 primitives 28 -> 17 us, 256 53 -> 29, 1024 93 -> 48; 320x200 27 ->
// 17, 56 -> 32, 94 -> 50.  (The second ray is cast whether or not x sees the
// sample; W is zero if it does not.)
template <bool LDS>
__global__ void __launch_bounds__(128)
    k_temporal_small(gi_scene sc, gi_gbuffer gb, gi_gbuffer gbp, gi_camera cam_prev, gi_reservoirs cur,
                     gi_reservoirs hist, gi_params pp, uint32_t m_hist_cap, gi_reservoirs out, uint64_t seed,
                     uint32_t frame)
{
    using Acc = typename std::conditional<LDS, GeoLds, GeoGlobal>::type;
    __shared__ uint32_t prev[64], seen[64];      // the pixel whose ray the second wave casts (~0: none), its answer
    const uint32_t t = threadIdx.x & 63u, tx = (gb.width + 7u) / 8u;
    const bool first = threadIdx.x < 64u;
    const uint32_t px = (blockIdx.x % tx) * 8u + (t & 7u), py = (blockIdx.x / tx) * 8u + (t >> 3);
    const bool inside = px < gb.width && py < gb.height;
    const uint32_t p = py * gb.width + px;
    if (LDS) stage_scene(sc);
    const Acc acc(sc);
    bool have = false, ray = false;
    float wsum = 0.0f, ph = 0.0f;
    uint32_t M0 = 0u, M1 = 0u, Msum = 0u, q1 = ~0u;
    const auto merge = [&] {
        const GB g = load_gb<false>(gb, p);
        const Res rc = load_res(cur, p);
        if (!active<false>(g)) {
            store_res(out, p, rc);
            return;
        }
        Merge m{0.0f, 0u, false, rc};
        M0 = rc.M;
        uint32_t qprev = 0u;
        merge_in<false>(m, g, rc, rc.M, 0.0f, pp.g_max);
        const int q = reproject(cam_prev, g.pos);
        if (q >= 0) {
            const GB gq = load_gb<false>(gbp, (uint32_t)q);
            if (similar(g, gq, pp)) {
                const Res rh = load_res(hist, (uint32_t)q);
                M1 = min(rh.M, m_hist_cap);
                const uint4 rn = philox<true>(seed, p, frame, kPassTemporal, 0u);
                merge_in<false>(m, g, rh, M1, u01(rn.x), pp.g_max);
                qprev = (uint32_t)q;
            }
        }
        have = m.have;
        wsum = m.wsum;
        Msum = m.Msum;
        Res r = m.sel;
        if (!have) r = empty_res(Msum);
        r.wsum = wsum;
        r.M = Msum;
        if (have) {
            ph = res_target<false>(g, r, pp.g_max);
            r.W = 0.0f;
            ray = pp.unbiased && ph > 0.0f;
            if (ray && M1 != 0u && !(res_target<false>(load_gb<false>(gbp, qprev), r, pp.g_max) <= 0.0f)) q1 = qprev;
        }
        store_res(out, p, r);
    };
    if (first) {
        if (inside) merge();
        prev[t] = q1;
    }
    __syncthreads();
    // the sample as its pixel has written it (the barrier orders this
    // workgroup's writes before its reads)
    const uint32_t q = first ? p : prev[t];
    bool vis = false;
    if (first ? ray : q != ~0u) {
        const GB d = load_gb<false>(first ? gb : gbp, q);
        const V3 y = xyz(reinterpret_cast<const float4 *>(out.y_W)[p]), n = xyz(reinterpret_cast<const float4 *>(out.n_wsum)[p]);
        vis = visible(sc, acc, d.pos, d.n, y, n, is_zero(n));
    }
    if (!first) seen[t] = vis ? 1u : 0u;
    __syncthreads();
    if (!first || !have) return;
    float W = 0.0f;
    if (pp.unbiased) {
        const uint32_t z = M0 + (seen[t] ? M1 : 0u);
        if (vis && z > 0u) W = wsum * rcp((float)z * ph);
    } else if (Msum > 0u && ph > 0.0f) {
        W = wsum * rcp((float)Msum * ph);
    }
    out.y_W[4u * (size_t)p + 3u] = W;
}

// The visibility rays of a workgroup's pixels: up to KM + 1 of each, sorted
// by direction cell, so that all lanes of a wave walk and walk together.
template <int KM, int NT>
struct RayPool {
    uint32_t q[KM][NT];                  // the domains' pixels
    uint32_t seen[NT];                   // bit j: domain j sees the pixel's sample
    uint32_t hist[kBins + 8];
    uint16_t order[(KM + 1) * NT];
};

// The pixel of slot k of a tile: 8x8 pixels for 256 threads (SW = 8, tiles in
// image order), else SW x 16 in stripes.
template <uint32_t SW>
__device__ __forceinline__ bool spatial_pixel(uint32_t W, uint32_t H, uint32_t &px, uint32_t &py, uint32_t k)
{
    if constexpr (SW == 8u) {
        const uint32_t tx = (W + 7u) / 8u;
        px = (blockIdx.x % tx) * 8u + (k & 7u);
        py = (blockIdx.x / tx) * 8u + (k >> 3);
        return px < W && py < H;
    } else {
        return tile_pixel_striped<SW>(W, H, px, py, k);
    }
}

// Neighbour slots are static (KM of them, KM >= k): a slot that draws no
// pixel (off-screen, the pixel itself, j >= k) points at the pixel itself,
// so every neighbour load is in bounds and unconditional, and the loads of
// all slots can be in flight together instead of one neighbour after the
// other.
// The visibility rays of all pixels go into one pool, sorted by direction
// (about 5 per pixel at k = 5): cast pixel by pixel they kept 24 of a wave's
// 64 lanes busy, pooled 42.  The pass took 0.74 of the vector-issue peak
// before the pool and takes 0.61 with it: as much as by issue it is bound by
// the gathers of the pooled rays, which read their pixel's sample and their
// domain's vertex again (104 M L2 requests, 78 M before).  0.776 -> 0.617 ms
// at 1920x1080, 6.46 -> 3.03 ms at 3840x2160 with 1024 primitives (k = 5).
// The rays that only decide Z are cast whether or not x sees the sample; W is
// zero if it does not.  Waves per SIMD: 5 (74 VGPRs at k <= 5; k <= 8 takes
// 96 and spills 3), 4 with glossy layers, 6 for the 768-thread tiles (k <= 8
// there spills 17, with glossy layers 46).
template <bool LDS, bool GLOSSY, int KM, uint32_t SW>
__global__ void __launch_bounds__(SW == 8u ? 256u : SW * kTile, SW == 48u ? 6 : GLOSSY ? 4 : 5)
    k_spatial(gi_scene sc, gi_gbuffer gb, gi_reservoirs in, gi_params pp, uint32_t pass, gi_reservoirs out,
              uint64_t seed, uint32_t frame)
{
    constexpr int NT = SW == 8u ? 256 : (int)SW * kTile, NP = SW == 8u ? 64 : NT;
    using Acc = typename std::conditional<LDS, GeoSmall, GeoGlobal>::type;
    uint32_t px, py;
    const bool inside = (NP == NT || threadIdx.x < (uint32_t)NP) && spatial_pixel<SW>(gb.width, gb.height, px, py, threadIdx.x);
    if (LDS) stage_small(sc);
    const Acc acc(sc);
    const uint32_t W = gb.width, H = gb.height, t = threadIdx.x;
    const uint32_t p = py * W + px;
    char *const lds = reinterpret_cast<char *>(gi_lds) + (LDS ? lds_small_bytes(sc) : 0u);
    RayPool<KM, NP> &pool = *reinterpret_cast<RayPool<KM, NP> *>(lds);
    if (t < kBins) pool.hist[t] = 0u;
    if (NP == NT || t < (uint32_t)NP) pool.seen[t] = 0u;

    float ph = 0.0f, wsum = 0.0f;
    uint32_t Msum = 0u;
    bool have = false;
    uint32_t key[KM + 1], Mdom[KM + 1];
#pragma unroll
    for (int j = 0; j <= KM; ++j) {
        key[j] = ~0u;
        Mdom[j] = 0u;
    }
    __syncthreads();
    const auto merge = [&] {
        const GB g = load_gb<GLOSSY>(gb, p);
        const Res rc = load_res(in, p);
        if (!active<GLOSSY>(g)) {
            store_res(out, p, rc);
            return;
        }
        // neighbour pixels: uniform in the disk (counter (pixel, frame, 2+pass, j))
        uint32_t qidx[KM + 1];
        bool drawn[KM];
        float uq[KM];
        qidx[0] = p;
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            qidx[j + 1] = p;
            drawn[j] = false;
            uq[j] = 0.0f;
            if ((uint32_t)j >= pp.k) continue;
            const uint4 rn = philox<true>(seed, p, frame, kPassSpatial0 + pass, (uint32_t)j);
            const float rad = pp.radius * fsqrt(u01(rn.x));
            const float s_ = sin_rev(u01(rn.y)), c_ = cos_rev(u01(rn.y));
            const int qx = (int)px + (int)floorf(rad * c_ + 0.5f);
            const int qy = (int)py + (int)floorf(rad * s_ + 0.5f);
            uq[j] = u01(rn.z);
            if (qx < 0 || qy < 0 || qx >= (int)W || qy >= (int)H) continue;
            if (qx == (int)px && qy == (int)py) continue;
            drawn[j] = true;
            qidx[j + 1] = (uint32_t)qy * W + (uint32_t)qx;
        }
        // geometric validation of every drawn neighbour (its normal and depth)
        bool use[KM];
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            const uint32_t q = qidx[j + 1];
            const float4 a = reinterpret_cast<const float4 *>(gb.pos_depth)[q];
            GB gq;
            gq.depth = a.w;
            if (gb.format == GI_GB_F16) {
                const GB full = load_gb<false>(gb, q);
                gq.n = full.n;
                gq.prim = full.prim;
            } else {
                const float4 b = reinterpret_cast<const float4 *>(gb.nrm_prim)[q];
                gq.n = xyz(b);
                gq.prim = __float_as_uint(b.w);
            }
            use[j] = drawn[j] && similar(g, gq, pp);
        }
        // merge the pixel's own reservoir, then the neighbours in order
        Merge m{0.0f, 0u, false, rc};
        Mdom[0] = rc.M;
        merge_in<GLOSSY>(m, g, rc, rc.M, 0.0f, pp.g_max);
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            const Res rq = load_res(in, qidx[j + 1]);
            Mdom[j + 1] = use[j] ? rq.M : 0u;
            if (use[j]) merge_in<GLOSSY>(m, g, rq, rq.M, uq[j], pp.g_max);
        }
        wsum = m.wsum;
        Msum = m.Msum;
        have = m.have;
        if (!have) {
            Res e = empty_res(Msum);
            e.wsum = wsum;
            store_res(out, p, e);
        } else {
            const Res &r = m.sel;
            ph = res_target<GLOSSY>(g, r, pp.g_max);
            reinterpret_cast<float4 *>(out.y_W)[p] = make_float4(r.y.x, r.y.y, r.y.z, 0.0f);
            reinterpret_cast<float4 *>(out.n_wsum)[p] = make_float4(r.n.x, r.n.y, r.n.z, wsum);
            reinterpret_cast<float4 *>(out.L_M)[p] = make_float4(r.L.x, r.L.y, r.L.z, __uint_as_float(Msum));
            reinterpret_cast<uint2 *>(out.tag_prim)[p] = make_uint2(r.tag, r.prim);
            // the visibility rays: x's own, then those of the domains whose target supports y
            if (pp.unbiased && ph > 0.0f) {
#pragma unroll
                for (int j = 0; j <= KM; ++j) {
                    if (j > 0 && Mdom[j] == 0u) continue;
                    const GB q = j == 0 ? g : load_gb<GLOSSY>(gb, qidx[j]);
                    if (j > 0 && res_target<GLOSSY>(q, r, pp.g_max) <= 0.0f) continue;
                    if (j > 0) pool.q[j - 1][t] = qidx[j];
                    const uint32_t b = sort_bin_of(is_zero(r.n) ? r.y : r.y - q.pos) >> 2;
                    key[j] = b | (atomicAdd(&pool.hist[b], 1u) << 16);
                }
            }
        }
    };
    if (inside) merge();
    __syncthreads();
    if (t < 64u) bin_starts<kBins>(pool.hist);
    __syncthreads();
#pragma unroll
    for (int j = 0; j <= KM; ++j)
        if (key[j] != ~0u) pool.order[pool.hist[key[j] & 0xFFFFu] + (key[j] >> 16)] = (uint16_t)((j << 12) | t);
    __syncthreads();
    for (uint32_t at = t; at < pool.hist[kBins]; at += NT) {
        const uint32_t e = pool.order[at], k = e & 0xFFFu, j = e >> 12;
        uint32_t kx, ky;
        spatial_pixel<SW>(W, H, kx, ky, k);
        const uint32_t pk = ky * W + kx, q = j == 0u ? pk : pool.q[j - 1u][k];
        const GB d = load_gb<false>(gb, q);
        // the sample as its pixel has written it (the barriers order this
        // workgroup's writes before its reads)
        const V3 y = xyz(reinterpret_cast<const float4 *>(out.y_W)[pk]), n = xyz(reinterpret_cast<const float4 *>(out.n_wsum)[pk]);
        if (visible(sc, acc, d.pos, d.n, y, n, is_zero(n))) atomicOr(&pool.seen[k], 1u << j);
    }
    __syncthreads();
    if (!have) return;
    // W is zero unless x sees y and p_hat(y) > 0
    float Wt = 0.0f;
    if (pp.unbiased) {
        const uint32_t seen = pool.seen[t];
        uint32_t z = Mdom[0];                 // the target at x supports y (it was chosen)
#pragma unroll
        for (int j = 1; j <= KM; ++j) z += (seen >> j) & 1u ? Mdom[j] : 0u;
        if ((seen & 1u) && z > 0u) Wt = wsum * rcp((float)z * ph);
    } else if (Msum > 0u && ph > 0.0f) {
        Wt = wsum * rcp((float)Msum * ph);
    }
    out.y_W[4u * (size_t)p + 3u] = Wt;
}

// --------------------------------------------------------------------------
// shading
// --------------------------------------------------------------------------
// Specular recursion for shading (Sec. 3.3, Eq. 7-8) from the selected
// sample v (primitive prim, normal nv) toward prev: at each vertex the
// emission and the diffuse probe term rho Q(v_b, n_v), then one direction
// from the glossy lobe (counter (pixel, frame, 16, depth)) weighted
// k_s f_g cos / pdf.  While the footprint a = foot^2 stays within a_0 c and
// below the depth limit the direction is traced (the sky if it leaves) and
// the walk continues at the hit, adding sqrt(|z - v|^2 / (pdf cos_z)) to
// foot; otherwise the probes estimate the glossy integral (Q(v_b, wi)/2).
// The loop form carries the product of the weights so far (grey).
template <int TEX, class G>
__device__ V3 shade_glossy(const gi_scene &sc, const G &acc, const gi_probes &pr, const gi_params &pp, uint64_t seed,
                           uint32_t pixel, uint32_t frame, uint32_t prim, V3 v, V3 nv, V3 prev, float foot, float a0c)
{
    V3 L = v3(0.0f, 0.0f, 0.0f);
    float thr = 1.0f;
    for (uint32_t depth = 1; depth <= GI_MAX_GLOSSY_DEPTH; ++depth) {
        V3 alb, emit;
        float ks, a;
        material_g(sc, prim, alb, emit, ks, a);
        L = L + thr * emit;
        const V3 pb = view_bias(v, prev, pr.bias_dist);
        if (!is_zero(alb)) L = L + thr * (alb * probe_query<1, TEX>(pr, pb, nv));
        if (!(ks > 0.0f)) break;
        V3 wo = prev - v;
        wo = frsq(dot(wo, wo)) * wo;
        const uint4 rn = philox(seed, pixel, frame, kPassGlossyShade, depth);
        V3 wi;
        if (!ggx_sample(nv, wo, a, u01(rn.x), u01(rn.y), wi)) break;
        const float pdf = ggx_pdf(nv, wo, wi, a);
        if (!(pdf > 0.0f)) break;
        const float wgt = ks * ggx_eval(nv, wo, wi, a) * dot(nv, wi) * rcp(pdf);
        if (foot * foot > a0c || depth >= pp.glossy_depth) {
            L = L + (thr * 0.5f * wgt) * probe_query<1, TEX>(pr, pb, wi);
            break;
        }
        const V3 o = madd(v, sc.eps, nv);
        Hit h;
        if (!cast<false>(sc, acc, o, wi, kInf, h)) {
            L = L + (thr * wgt) * ld3(sc.sky);
            break;
        }
        const V3 z = madd(o, h.t, wi);
        const V3 nz = hit_normal(sc, acc, o, wi, h);
        const V3 dz = z - v;
        const float cz = -dot(nz, wi);
        foot += cz > 0.0f ? fsqrt(dot(dz, dz) * rcp(pdf * cz)) : kInf;
        thr *= wgt;
        prev = v;
        v = z;
        nv = nz;
        prim = h.prim;
    }
    return L;
}

// WS = true: the fresh query is the cache value q[p] evaluated at the
// reservoir's sample when the cache is selected (probe query otherwise).
// GLOSSY: f(x) replaces rho_x/pi and the fresh radiance follows the specular
// recursion, started with the footprint of the segment x -> y (density of
// the BSDF mixture at x) and a_0 c = c |x_0 - x|^2 / (4 pi cos) from the camera.
// The Lambertian kernel is held to 5 waves per SIMD (no spills).
template <bool LDS, bool WS, bool GLOSSY, int TEX, uint32_t SW>
__global__ void __launch_bounds__(SW * kTile, GLOSSY ? 1 : SW == 16u ? 5 : 6)
    k_shade(gi_scene sc, gi_gbuffer gb, gi_probes pr, gi_reservoirs res, const float4 *resid, gi_params pp,
            float4 *img, const float4 *q, gi_mlp mlp, uint64_t seed, uint32_t frame)
{
    using Acc = typename std::conditional<SW != (uint32_t)kTile, GeoSmall, typename std::conditional<LDS, GeoLds, GeoGlobal>::type>::type;
    uint32_t px, py;
    const bool inside = tile_pixel<SW>(gb.width, gb.height, px, py);
    if constexpr (SW != (uint32_t)kTile) {
        stage_small(sc);
        __syncthreads();
    } else if (LDS) {
        stage_scene(sc);
    }
    if (!inside) return;
    const Acc acc(sc);
    const uint32_t p = py * gb.width + px;
    const GB g = load_gb<GLOSSY>(gb, p);
    float4 e = reinterpret_cast<const float4 *>(gb.emit)[p];
    V3 o = xyz(e);
    if (g.prim != GI_MISS) {
        o = o + xyz(resid[p]);
        Res r = load_res(res, p);
        if (r.W > 0.0f) {
            V3 L, wd = r.y;
            float geo = 0.0f;
            bool ok = false;
            if (is_zero(r.n)) {
                geo = dot(g.n, r.y);
                if (geo > 0.0f && visible(sc, acc, g.pos, g.n, r.y, r.n, true)) {
                    L = ld3(sc.sky);
                    ok = true;
                }
            } else {
                V3 v = r.y - g.pos;
                float d2 = dot(v, v);
                V3 w = frsq(d2) * v;
                wd = w;
                float cx = dot(g.n, w), cy = -dot(r.n, w);
                if (cx > 0.0f && cy > 0.0f) {
                    geo = fminf(cx * cy * rcp(d2), pp.g_max);
                    if (visible(sc, acc, g.pos, g.n, r.y, r.n, false)) {
                        if constexpr (GLOSSY) {
                            const V3 vc = ld3(gb.eye) - g.pos;
                            const float c1 = dot(g.n, g.wo);
                            const float a0c = c1 > 0.0f ? pp.foot_c * dot(vc, vc) * rcp(4.0f * kPi * c1) : kInf;
                            const float p1 = mix_pdf(g.alb, g.ks, g.rough, g.n, g.wo, w);
                            const float foot = p1 > 0.0f ? fsqrt(d2 * rcp(p1 * cy)) : kInf;
                            L = shade_glossy<TEX>(sc, acc, pr, pp, seed, p, frame, r.prim, r.y, r.n, g.pos, foot, a0c);
                        } else {
                            L = (WS && mlp_selected(mlp)) ? radiance_cached(sc, r.prim, q[p])
                                                           : radiance_toward<1, TEX>(sc, pr, r.prim, r.y, r.n, g.pos);
                        }
                        ok = true;
                    }
                }
            }
            if (ok) {
                if constexpr (GLOSSY)
                    o = o + (geo * r.W) * (bsdf(g.alb, g.ks, g.rough, g.n, g.wo, wd) * L);
                else
                    o = o + (kInvPi * geo * r.W) * (g.alb * L);
            }
        }
    }
    img[p] = make_float4(o.x, o.y, o.z, 1.0f);
}

// --------------------------------------------------------------------------
// training samples of the learned cache
// --------------------------------------------------------------------------
// Sample j: pixel p = floor(u0 W H), candidate i = floor(u1 M) of the
// initial pass (its own counter), label gathered along (u2, u3) about n_y.
template <bool LDS>
__global__ void __launch_bounds__(kBlock)
    k_mlp_batch(gi_scene sc, gi_gbuffer gb, gi_probes pr, uint32_t M, uint32_t n, uint64_t seed, uint32_t frame,
                float4 *pos, float4 *nrm, float4 *tgt, float4 *qp)
{
    using Acc = typename std::conditional<LDS, GeoLds, GeoGlobal>::type;
    const uint32_t j = blockIdx.x * kBlock + threadIdx.x;
    if (LDS) stage_scene(sc);
    if (j >= n) return;
    const Acc acc(sc);
    const uint4 rn = philox(seed, j, frame, kPassTrainBatch, 0u);
    // floor(u W H) and floor(u M) exactly: u = (x >> 8) 2^-24
    const uint64_t npx = (uint64_t)gb.width * gb.height;
    const uint32_t p = (uint32_t)(((uint64_t)(rn.x >> 8) * npx) >> 24);
    const uint32_t i = (uint32_t)(((uint64_t)(rn.y >> 8) * M) >> 24);
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    pos[j] = zero;
    nrm[j] = zero;
    tgt[j] = zero;
    qp[j] = zero;
    const GB g = load_gb(gb, p);
    if (!active(g)) return;
    // the candidate, as the initial pass traces it
    const uint4 rc = philox(seed, p, frame, kPassInitial, i);
    const V3 w = cosine_dir(g.n, u01(rc.x), u01(rc.y));
    const V3 o = madd(g.pos, sc.eps, g.n);
    Hit hy;
    if (!cast<false>(sc, acc, o, w, kInf, hy)) return;
    const V3 y = madd(o, hy.t, w), ny = hit_normal(sc, acc, o, w, hy);
    V3 alb, emit;
    material(sc, hy.prim, alb, emit);
    if (is_zero(alb)) return;
    // its label
    const V3 wl = cosine_dir(ny, u01(rn.z), u01(rn.w));
    const V3 ol = madd(y, sc.eps, ny);
    Hit h;
    V3 L;
    if (cast<false>(sc, acc, ol, wl, kInf, h)) {
        const V3 z = madd(ol, h.t, wl);
        L = radiance_toward(sc, pr, h.prim, z, hit_normal(sc, acc, ol, wl, h), y);
    } else {
        L = ld3(sc.sky);
    }
    const V3 q = probe_query(pr, view_bias(y, g.pos, pr.bias_dist), ny);
    pos[j] = make_float4(y.x, y.y, y.z, 0.0f);
    nrm[j] = make_float4(ny.x, ny.y, ny.z, 0.0f);
    tgt[j] = make_float4(L.x, L.y, L.z, 1.0f);
    qp[j] = make_float4(q.x, q.y, q.z, 0.0f);
}

// --------------------------------------------------------------------------
// reference path tracer (converged images for the error statements)
// --------------------------------------------------------------------------
// GLOSSY: at every vertex the BSDF mixture of the initial pass (glossy lobe
// with probability k_s / (k_s + lum rho), chosen by u3), throughput times
// f cos / pdf, roulette after that product
template <bool LDS, bool GLOSSY>
__global__ void __launch_bounds__(kBlock)
    k_path_trace(gi_scene sc, gi_gbuffer gb, uint32_t spp, uint32_t s0, uint64_t seed, float4 *out)
{
    using Acc = typename std::conditional<LDS, GeoLds, GeoGlobal>::type;
    uint32_t px, py;
    const bool inside = tile_pixel(gb.width, gb.height, px, py);
    if (LDS) stage_scene(sc);
    if (!inside) return;
    const Acc acc(sc);
    const uint32_t p = py * gb.width + px;
    const GB g = load_gb<GLOSSY>(gb, p);
    const V3 e0 = xyz(reinterpret_cast<const float4 *>(gb.emit)[p]);
    V3 sum = v3(0.0f, 0.0f, 0.0f);
    for (uint32_t s = 0; s < spp; ++s) {
        V3 x = g.pos, n = g.n, rho = g.alb, L = e0, thr = v3(1.0f, 1.0f, 1.0f);
        if constexpr (GLOSSY) {
            if (g.prim == GI_MISS) {
                sum = sum + L;
                continue;
            }
            float ks = g.ks, ra = g.rough;
            V3 wo = g.wo;
            for (uint32_t b = 1; b <= 32; ++b) {
                if (is_zero(rho) && !(ks > 0.0f)) break;
                const uint4 rn = philox(seed, p, s0 + s, kPassReference, b);
                const float pg = p_gloss(rho, ks);
                V3 w;
                if (pg > 0.0f && u01(rn.w) < pg) {
                    if (!ggx_sample(n, wo, ra, u01(rn.x), u01(rn.y), w)) break;
                } else {
                    w = cosine_dir(n, u01(rn.x), u01(rn.y));
                }
                const float pd = mix_pdf(rho, ks, ra, n, wo, w);
                if (!(pd > 0.0f)) break;
                thr = thr * ((dot(n, w) * rcp(pd)) * bsdf(rho, ks, ra, n, wo, w));
                if (b >= 4) {
                    const float P = fminf(1.0f, fmaxf(thr.x, fmaxf(thr.y, thr.z)));
                    if (!(u01(rn.z) < P)) break;
                    thr = v3(thr.x / P, thr.y / P, thr.z / P);
                }
                const V3 o = madd(x, sc.eps, n);
                Hit h;
                if (!cast<false>(sc, acc, o, w, kInf, h)) {
                    L = L + thr * ld3(sc.sky);
                    break;
                }
                x = madd(o, h.t, w);
                n = hit_normal(sc, acc, o, w, h);
                wo = -w;
                V3 emit;
                material_g(sc, h.prim, rho, emit, ks, ra);
                L = L + thr * emit;
            }
            sum = sum + L;
            continue;
        }
        for (uint32_t b = 1; b <= 32; ++b) {
            if (is_zero(rho)) break;
            const uint4 rn = philox(seed, p, s0 + s, kPassReference, b);
            thr = thr * rho;
            if (b >= 4) {
                const float P = fminf(1.0f, fmaxf(thr.x, fmaxf(thr.y, thr.z)));
                if (!(u01(rn.z) < P)) break;
                thr = v3(thr.x / P, thr.y / P, thr.z / P);
            }
            const V3 w = cosine_dir(n, u01(rn.x), u01(rn.y));
            const V3 o = madd(x, sc.eps, n);
            Hit h;
            if (!cast<false>(sc, acc, o, w, kInf, h)) {
                L = L + thr * ld3(sc.sky);
                break;
            }
            x = madd(o, h.t, w);
            n = hit_normal(sc, acc, o, w, h);
            V3 emit;
            material(sc, h.prim, rho, emit);
            L = L + thr * emit;
        }
        sum = sum + L;
    }
    const float inv = 1.0f / (float)spp;
    out[p] = make_float4(sum.x * inv, sum.y * inv, sum.z * inv, 1.0f);
}

// --------------------------------------------------------------------------
// test hooks
// --------------------------------------------------------------------------
__global__ void k_philox(uint64_t seed, uint32_t n, const uint4 *ctr, uint4 *out)
{
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint4 c = ctr[i];
    out[i] = philox(seed, c.x, c.y, c.z, c.w);
}

__global__ void k_trace(gi_scene sc, uint32_t n, const float *org, const float *dir, float4 *out, uint32_t *prim)
{
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    V3 o = ld3(org + 3 * i), d = ld3(dir + 3 * i);
    Hit h;
    const GeoGlobal acc(sc);
    if (cast<false>(sc, acc, o, d, kInf, h)) {
        V3 nn = hit_normal(sc, acc, o, d, h);
        out[i] = make_float4(h.t, nn.x, nn.y, nn.z);
        prim[i] = h.prim;
    } else {
        out[i] = make_float4(kInf, 0.0f, 0.0f, 0.0f);
        prim[i] = GI_MISS;
    }
}

// --------------------------------------------------------------------------
// host-side validation
// --------------------------------------------------------------------------
gi_status launched()
{
    return hipGetLastError() == hipSuccess ? GI_OK : GI_ERR_LAUNCH;
}

gi_status check_scene(const gi_scene *sc)
{
    if (!sc) return GI_ERR_NULL;
    if (sc->n_prims > 0 && !sc->prims) return GI_ERR_NULL;
    if (sc->n_emitters > GI_MAX_EMITTERS) return GI_ERR_SHAPE;
    for (uint32_t e = 0; e < sc->n_emitters; ++e)
        if (sc->emitters[e] >= sc->n_prims) return GI_ERR_PARAM;
    if (!(sc->eps >= 0.0f)) return GI_ERR_PARAM;
    if (sc->cell_start) {
        if (!sc->cell_items && sc->n_items) return GI_ERR_NULL;
        if (sc->grid_res[0] == 0 || sc->grid_res[1] == 0 || sc->grid_res[2] == 0) return GI_ERR_SHAPE;
        if ((uint64_t)sc->grid_res[0] * sc->grid_res[1] * sc->grid_res[2] > (1u << 26)) return GI_ERR_SHAPE;
        for (int a = 0; a < 3; ++a)
            if (!(sc->grid_hi[a] > sc->grid_lo[a])) return GI_ERR_PARAM;
    }
    return GI_OK;
}

gi_status check_gb(const gi_gbuffer *g, uint32_t W, uint32_t H)
{
    if (!g || !g->pos_depth || !g->nrm_prim || !g->albedo || !g->emit) return GI_ERR_NULL;
    if (g->format > GI_GB_F16) return GI_ERR_PARAM;
    if (g->width != W || g->height != H) return GI_ERR_SHAPE;
    return GI_OK;
}

gi_status check_res(const gi_reservoirs *r, uint32_t W, uint32_t H)
{
    if (!r || !r->y_W || !r->n_wsum || !r->L_M || !r->tag_prim) return GI_ERR_NULL;
    if (r->width != W || r->height != H) return GI_ERR_SHAPE;
    return GI_OK;
}

bool res_alias(const gi_reservoirs *a, const gi_reservoirs *b)
{
    const void *pa[4] = {a->y_W, a->n_wsum, a->L_M, a->tag_prim};
    const void *pb[4] = {b->y_W, b->n_wsum, b->L_M, b->tag_prim};
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j)
            if (pa[i] == pb[j]) return true;
    return false;
}

gi_status check_probes(const gi_probes *p)
{
    if (!p || !p->irr || !p->dep) return GI_ERR_NULL;
    if (p->irr_res != 8 || p->dep_res != 16) return GI_ERR_SHAPE;
    if (p->dims[0] == 0 || p->dims[1] == 0 || p->dims[2] == 0) return GI_ERR_SHAPE;
    // the depth texture (the larger) must stay below 4 GiB: kernels use 32-bit byte offsets
    if ((uint64_t)p->dims[0] * p->dims[1] * p->dims[2] > kMaxProbes) return GI_ERR_SHAPE;
    for (int a = 0; a < 3; ++a)
        if (!(p->spacing[a] > 0.0f)) return GI_ERR_PARAM;
    if (p->texel != GI_TEXEL_F32 && p->texel != GI_TEXEL_F16) return GI_ERR_PARAM;
    return GI_OK;
}

gi_status check_params(const gi_params *pp)
{
    if (!pp) return GI_ERR_NULL;
    if (pp->M < 1 || pp->M > GI_MAX_M || pp->k > GI_MAX_K) return GI_ERR_PARAM;
    if (pp->M_light > GI_MAX_M - pp->M) return GI_ERR_PARAM;
    if (pp->subsample < 1) return GI_ERR_PARAM;
    if (!(pp->radius >= 0.0f) || !(pp->g_max > 0.0f) || !(pp->m_cap >= 0.0f) || !(pp->depth_rel >= 0.0f))
        return GI_ERR_PARAM;
    return GI_OK;
}

hipStream_t S(void *s) { return reinterpret_cast<hipStream_t>(s); }

// Dynamic LDS a tracing kernel needs to stage the scene, or 0 to read it from
// global memory (no grid, staging switched off, or over budget: 40 KB keeps
// four 256-thread workgroups per CU; a kernel with static LDS stays within
// 64 KB in total).
constexpr uint32_t kLdsScene = 40u * 1024u;
constexpr uint32_t kLdsTotal = 64u * 1024u;
uint32_t scene_lds(const gi_scene *sc, uint32_t static_lds = 0)
{
    if (!sc->cell_start || sc->n_items == 0 || (sc->options & GI_OPT_NO_LDS)) return 0;
    uint32_t b = lds_scene_bytes(*sc);
    if (static_lds == 0) return b <= kLdsScene ? b : 0u;
    return b + static_lds <= kLdsTotal ? b : 0u;
}

#define GI_LAUNCH_LDS(kernel, grid, block, lds, stream, ...)                                   \
    do {                                                                                      \
        if (lds) kernel<true><<<(grid), (block), (lds), (stream)>>>(__VA_ARGS__);             \
        else kernel<false><<<(grid), (block), 0, (stream)>>>(__VA_ARGS__);                   \
    } while (0)
// k_initial with the scene staging (lds bytes, 0: none), emitter candidates,
// the glossy BSDF and the probes' texel format chosen at run time (the
// learned cache, WS, serves Lambertian scenes only and reads the texel format
// at run time: its probe queries are the emitter candidates' alone)
template <bool WS, bool LIGHT, int TEX, class... A>
void launch_initial_t(bool glossy, uint32_t lds, dim3 grid, hipStream_t st, A... a)
{
    // past the staged scene: every thread's selected-candidate slot
    const uint32_t extra = kBlock * kSelBytes;
    if (!WS && glossy) {
        if (lds) k_initial<true, WS, LIGHT, !WS, TEX><<<grid, kBlock, lds + extra, st>>>(a...);
        else k_initial<false, WS, LIGHT, !WS, TEX><<<grid, kBlock, extra, st>>>(a...);
    } else {
        if (lds) k_initial<true, WS, LIGHT, false, TEX><<<grid, kBlock, lds + extra, st>>>(a...);
        else k_initial<false, WS, LIGHT, false, TEX><<<grid, kBlock, extra, st>>>(a...);
    }
}
template <bool WS, bool LIGHT, class... A>
void launch_initial_l(bool glossy, bool f16, uint32_t lds, dim3 grid, hipStream_t st, A... a)
{
    if constexpr (WS) {
        launch_initial_t<WS, LIGHT, kTexAny>(glossy, lds, grid, st, a...);
    } else {
        if (f16) launch_initial_t<WS, LIGHT, kTexF16>(glossy, lds, grid, st, a...);
        else launch_initial_t<WS, LIGHT, kTexF32>(glossy, lds, grid, st, a...);
    }
}

// scene bytes to stage for k_initial: the scene and the selected-candidate
// slots together within kLdsScene, so that 4 workgroups share a CU
uint32_t initial_scene_lds(const gi_scene *sc)
{
    const uint32_t b = scene_lds(sc);
    return b && b + kBlock * kSelBytes <= kLdsScene ? b : 0u;
}

template <bool WS, class... A>
void launch_initial(bool light, bool glossy, bool f16, uint32_t lds, dim3 grid, hipStream_t st, A... a)
{
    if (light) launch_initial_l<WS, true>(glossy, f16, lds, grid, st, a...);
    else launch_initial_l<WS, false>(glossy, f16, lds, grid, st, a...);
}

// Where k_initial_tile takes the probe form.  It needs no emitter candidates
// and primitives that fit its lists.  A tile costs about 50 us before its
// first ray (two share a CU) and then 1.4 us per 64 rays, the pixel form 23 us
// per candidate while the chip is not full and 0.086 us per 1000 candidates
// once it is (256 primitives).  So the tile form pays where a pixel takes many
// candidates: at M = 32 from 64x36 pixels (3.0x) to 3840x2160 (2.1x).  With
// fewer it still pays for large images, where tiles hold many rays (M = 8:
// 1.13x at 1280x720, 1.19x at 1920x1080), and for small ones, where the pixel
// form leaves most of the chip idle (M = 8: 1.2-1.6x up to 320x180), unless
// the primitives outnumber a small tile's rays; in between it does not
// (640x360: M = 8 0.75x, M = 13 0.91x), nor below M = 8.  The line for large
// images holds for other numbers of primitives too: 8 primitives, 1283x721, M
// = 8 453 -> 302 us; 1024, 1283x721, M = 8 1.58 -> 1.29 ms, M = 13 2.55 ->
// 1.92; 1920x1080, M = 8 3.26 -> 2.16 ms, M = 13 5.24 -> 3.12, M = 23 9.20 ->
// 4.93.
bool tile_form(const gi_scene *sc, const gi_params *pp, uint32_t W, uint32_t H)
{
    if (pp->M_light > 0u || sc->n_prims > kListMaxPrims || (sc->options & GI_OPT_NO_LDS) || pp->M < 8u) return false;
    const uint64_t px = (uint64_t)W * H;
    return pp->M >= 24u || px >= 900000u || (px <= 96000u && 256u * pp->M >= 3u * sc->n_prims);
}

// An image of so few pixels leaves most of the chip idle to the forms of one
// thread per pixel.
constexpr uint64_t kSmallImage = 65536u;

// Where the learned-cache form traces its candidates by tiles.  The walks it
// replaces cost less than the probe form's pixels, so fewer frames gain: up to
// 512 primitives from M = 8 on (256 primitives, 1920x1080: M = 32 5.69 -> 4.46
// ms, M = 13 2.33 -> 1.97, M = 8 1.47 -> 1.26, whole pass; 64x36, M = 32: 765
// -> 234 us; M = 4 0.81 -> 0.84).  Longer lists leave room for half the rays
// per round.  Small images, which the pixel form does not spread over the
// chip, gain all the same (1024 primitives: 238x121, M = 13: 556 -> 337 us;
// 320x200, M = 8: 362 -> 300; 64x36, M = 8: 321 -> 215), larger ones only from
// M = 24 on (1283x721, 1024 primitives: M = 24 2.97 -> 2.97 ms, M = 32 3.94 ->
// 3.55), and the largest later the more primitives there are (1920x1080 and
// 2560x1440: 600 primitives, M = 24 6.24 -> 5.89 and 10.81 -> 10.98 ms, M = 26
// 11.71 -> 11.60; 1024, M = 24 6.04 -> 6.24 and 10.6 -> 11.5, M = 30 7.60 ->
// 7.14 and 13.31 -> 13.25).
bool cand_tiles(const gi_scene *sc, const gi_params &pp, uint32_t W, uint32_t H)
{
    const uint32_t n = sc->n_prims;
    if (n > kListMaxPrims || (sc->options & GI_OPT_NO_LDS) != 0u) return false;
    const uint64_t px = (uint64_t)W * H;
    if (n <= 512u || px <= kSmallImage) return pp.M >= 8u;
    return pp.M >= 24u + (px > 1500000u ? 6u * (n - 512u) / 512u : 0u);
}

bool glossy_scene(const gi_scene *sc) { return (sc->options & GI_OPT_GLOSSY) != 0u; }

void launch_initial_tile(const gi_scene *sc, const gi_gbuffer &gb, const gi_probes &pr, const gi_params &pp,
                         const gi_reservoirs &out, float4 *resid, uint64_t seed, uint32_t frame, const CandWs &ws,
                         const gi_mlp &mlp, hipStream_t st)
{
    const uint32_t W = gb.width, H = gb.height;
    const bool f16 = pr.texel == GI_TEXEL_F16, glossy = glossy_scene(sc);
    // the pixels' records stay in LDS where the lists leave room for them
    const bool px = !glossy && sc->n_prims <= 512u;
    // The largest tile that still leaves some 1500 of them (three rounds of
    // two workgroups per CU), down to 8x8 pixels and, for images that would
    // not reach every CU with those, 4x4: large tiles sort more rays together
    // and cull the scene less often, but their primitive lists are longer.
    // 1920x1080, M = 32, when this was chosen: 16x16 3.62 ms, 32x16 3.95, 16x8
    // 4.35, 8x8 5.80; 3840x2160: 32x16 23.4 ms, 16x16 24.5, 16x8 29.0.
    const auto tiles = [&](uint32_t a, uint32_t b) {
        return (uint64_t)((W + (1u << a) - 1u) >> a) * ((H + (1u << b) - 1u) >> b);
    };
    uint32_t lw = pp.M <= 16u || tiles(5u, 4u) >= 8192u ? 5u : 4u, lh = 4u;
    while (lw + lh > 6u && tiles(lw, lh) < 1500u) {
        if (lw > lh) --lw;
        else --lh;
    }
    if (tiles(3u, 3u) < 256u) lw = lh = 2u;
    const dim3 grid((W + (1u << lw) - 1u) >> lw, (H + (1u << lh) - 1u) >> lh);
    // candidates per round: all that leave room for two workgroups on a CU
    const uint32_t list = list_bytes(sc->n_prims), TP = 1u << (lw + lh);
    uint32_t C = pp.M;
    while (C > 1u && list + tile_bytes(C * TP, TP, px) > kTileLds) C = (C + 1u) / 2u;
    const uint32_t lds = list + std::max(tile_bytes(C * TP, TP, px), 4u * kListScratch);
#define GI_IT(G, T, X)                                                                                       \
    k_initial_tile<G, T, kTileBlock, X><<<grid, kTileBlock, lds, st>>>(*sc, gb, pr, pp, out, resid, seed, frame, lw, lh, C, ws, mlp)
    if (glossy) { if (f16) GI_IT(true, kTexF16, false); else GI_IT(true, kTexF32, false); }
    else if (px) { if (f16) GI_IT(false, kTexF16, true); else GI_IT(false, kTexF32, true); }
    else { if (f16) GI_IT(false, kTexF16, false); else GI_IT(false, kTexF32, false); }
#undef GI_IT
}

void launch_cand(const gi_scene *sc, const gi_gbuffer &gb, const gi_params &pp, const CandWs &ws, uint64_t seed,
                 uint32_t frame, const gi_mlp &mlp, hipStream_t st)
{
    const uint32_t W = gb.width, H = gb.height, lds = scene_lds(sc);
    if (!cand_tiles(sc, pp, W, H)) {
        GI_LAUNCH_LDS(k_cand, tile_grid(W, H), kBlock, lds, st, *sc, gb, pp, ws, seed, frame, mlp);
        return;
    }
    // Some 4000 rays per tile, which two rounds trace; less, but not below
    // 1000 (500 where a round holds half as many), where the image would not
    // make 2048 tiles.  1920x1080: M = 32
    // 16x8 4.46 ms (16x16 4.42, 32x16 4.64, 8x8 4.79), M = 13 16x16 1.97
    // (16x8 2.13), M = 8 32x16 1.26 (16x16 1.29, 16x8 1.56); 320x180, M = 32:
    // 8x8 299 us, 16x8 419, 16x16 679.
    uint32_t lw = pp.M >= 12u ? 4u : 5u, lh = pp.M >= 24u ? 3u : 4u;
    const uint32_t least = sc->n_prims > 512u ? 512u : 1024u;
    while (lw + lh > 6u && (pp.M << (lw + lh - 1u)) >= least &&
           (uint64_t)((W + (1u << lw) - 1u) >> lw) * ((H + (1u << lh) - 1u) >> lh) < 2048u) {
        if (lw > lh) --lw;
        else --lh;
    }
    const dim3 grid((W + (1u << lw) - 1u) >> lw, (H + (1u << lh) - 1u) >> lh);
    const uint32_t list = list_bytes(sc->n_prims), TP = 1u << (lw + lh);
    const uint32_t big = list + std::max(cand_bytes(4u * kTileBlock, TP), 4u * kListScratch);
    if (big <= kTileLds)
        k_cand_tile<4><<<grid, kTileBlock, big, st>>>(*sc, gb, pp, ws, seed, frame, lw, lh, mlp);
    else
        k_cand_tile<2><<<grid, kTileBlock, list + std::max(cand_bytes(2u * kTileBlock, TP), 4u * kListScratch), st>>>(
            *sc, gb, pp, ws, seed, frame, lw, lh, mlp);
}

// the probe form of the initial pass
void launch_initial_probe(const gi_scene *sc, const gi_gbuffer &gb, const gi_probes &pr, const gi_params &pp,
                          const gi_reservoirs &out, float4 *resid, uint64_t seed, uint32_t frame, const CandWs &ws,
                          const gi_mlp &mlp, hipStream_t st)
{
    if (tile_form(sc, &pp, gb.width, gb.height))
        launch_initial_tile(sc, gb, pr, pp, out, resid, seed, frame, ws, mlp, st);
    else
        launch_initial<false>(pp.M_light > 0, glossy_scene(sc), pr.texel == GI_TEXEL_F16, initial_scene_lds(sc),
                              tile_grid(gb.width, gb.height), st, *sc, gb, pr, pp, out, resid, seed, frame, ws, mlp);
}

#define GI_LAUNCH_LDS2(kernel, T2, grid, block, lds, stream, ...)                             \
    do {                                                                                      \
        if (lds) kernel<true, T2><<<(grid), (block), (lds), (stream)>>>(__VA_ARGS__);         \
        else kernel<false, T2><<<(grid), (block), 0, (stream)>>>(__VA_ARGS__);               \
    } while (0)

// How the passes of one thread per pixel (temporal, shade) hold the scene: in
// LDS for each 16x16 tile where four of them fit a CU; a larger one, in its
// small form, shared by the 768 threads of a 48x16 tile, two of which fill a
// CU; else in global memory.  1024 primitives, global memory -> wide tiles:
// 3840x2160 shade 1.95 -> 1.25 ms, temporal 1.71 -> 1.55; 640x360 89 -> 62 us,
// 119 -> 102; 40x2000 61 -> 45 us, 80 -> 65.  (The small form in 16x16 tiles,
// 1920x1080, 256 primitives: shade 232 us against 224, temporal 247 against
// 240.)  Glossy layers keep to the first and the last: their walks hold too
// many registers for 768 threads.
struct SceneTiles {
    uint32_t lds;
    bool wide;
    explicit SceneTiles(const gi_scene *sc) : lds(scene_lds(sc)), wide(false)
    {
        if (lds || !sc->cell_start || sc->n_items == 0 || (sc->options & (GI_OPT_NO_LDS | GI_OPT_GLOSSY))) return;
        const uint32_t b = lds_small_bytes(*sc);
        if (b == 0u || b > kTileLds) return;
        lds = b;
        wide = true;
    }
};

template <int KM, uint32_t SW, class... A>
void launch_spatial_t(const gi_scene *sc, uint32_t lds, uint32_t W, uint32_t H, hipStream_t st, A... a)
{
    constexpr uint32_t nt = SW == 8u ? 256u : SW * kTile, np = SW == 8u ? 64u : nt;
    const uint32_t bytes = lds + (uint32_t)sizeof(RayPool<KM, (int)np>);
    const dim3 grid = SW == 8u ? dim3(((W + 7u) / 8u) * ((H + 7u) / 8u)) : striped_grid(W, H, SW);
    if (glossy_scene(sc)) {
        if (lds) k_spatial<true, true, KM, SW><<<grid, nt, bytes, st>>>(a...);
        else if constexpr (SW != 48u) k_spatial<false, true, KM, SW><<<grid, nt, bytes, st>>>(a...);
    } else {
        if (lds) k_spatial<true, false, KM, SW><<<grid, nt, bytes, st>>>(a...);
        else if constexpr (SW != 48u) k_spatial<false, false, KM, SW><<<grid, nt, bytes, st>>>(a...);
    }
}

// The scene in LDS where that leaves four workgroups of 256 threads on a CU
// (1920x1080, 256 primitives, when this was chosen: 0.59 ms, from global
// memory 0.88); a larger one is shared by the 768 threads of a 48x16 tile, two
// of which fill a CU (3840x2160, 1024 primitives: 2.87 ms, from global memory
// 3.76, shared by 256 threads 5.18, by 512 3.85).
//
// An image of few pixels leaves most of the chip idle, and six rays in a row
// per thread are its time: tiles of 8x8 pixels share their rays between 256
// threads (two rounds of the pool instead of six).  64x64, 16x16 -> 8x8 tiles:
// 8 primitives 41 -> 20 us, 256: 50 -> 36, 1024 (from global memory): 49 -> 46;
// 320x180: 41 -> 22, 57 -> 43, 74 -> 64; from 480x270 on the waves without
// pixels cost as much as they gain (44 -> 46, 91 -> 77, 97 -> 85; 640x360: 56
// -> 60, 114 -> 108, 133 -> 130).
template <int KM, class... A>
void launch_spatial(const gi_scene *sc, uint32_t W, uint32_t H, hipStream_t st, A... a)
{
    const uint32_t lds = sc->cell_start && sc->n_items && !(sc->options & GI_OPT_NO_LDS) ? lds_small_bytes(*sc) : 0u;
    if ((uint64_t)W * H <= kSmallImage) launch_spatial_t<KM, 8u>(sc, lds + sizeof(RayPool<KM, 64>) <= kLdsScene ? lds : 0u, W, H, st, a...);
    else if (lds && lds + sizeof(RayPool<KM, 256>) <= kLdsScene) launch_spatial_t<KM, 16u>(sc, lds, W, H, st, a...);
    else if (lds && lds + sizeof(RayPool<KM, 768>) <= kTileLds) launch_spatial_t<KM, 48u>(sc, lds, W, H, st, a...);
    else launch_spatial_t<KM, 16u>(sc, 0u, W, H, st, a...);
}

#define GI_LAUNCH_LDS_G(kernel, glossy, grid, block, lds, stream, ...)                          \
    do {                                                                                      \
        if (glossy) GI_LAUNCH_LDS2(kernel, true, grid, block, lds, stream, __VA_ARGS__);       \
        else GI_LAUNCH_LDS2(kernel, false, grid, block, lds, stream, __VA_ARGS__);            \
    } while (0)

}  // namespace

// ==========================================================================
// C ABI
// ==========================================================================
extern "C" {

const char *gi_status_string(gi_status s)
{
    switch (s) {
    case GI_OK: return "ok";
    case GI_ERR_NULL: return "null pointer";
    case GI_ERR_SHAPE: return "shape mismatch or size limit";
    case GI_ERR_PARAM: return "parameter out of range";
    case GI_ERR_ALIAS: return "output aliases an input";
    case GI_ERR_LAUNCH: return "kernel launch failed";
    case GI_ERR_DEVICE: return "no usable HIP device";
    }
    return "unknown status";
}

int gi_device(void)
{
    int d = -1;
    if (hipGetDevice(&d) != hipSuccess) return -1;
    return d;
}

gi_status gi_trace_gbuffer(const gi_scene *scene, const gi_camera *cam, gi_gbuffer *out, void *stream)
{
    gi_status s;
    if (!cam || !out) return GI_ERR_NULL;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if ((s = check_gb(out, cam->width, cam->height)) != GI_OK) return s;
    if (out->format == GI_GB_F16 && scene->n_prims + 6u >= 0xFFFFu) return GI_ERR_SHAPE;
    if (cam->width == 0 || cam->height == 0) return GI_OK;
    k_gbuffer<<<tile_grid(cam->width, cam->height), kBlock, 0, S(stream)>>>(*scene, *cam, *out);
    return launched();
}

gi_status gi_probe_update(const gi_scene *scene, const gi_probes *in, gi_probes *out, const gi_probe_params *pp,
                          uint64_t seed, uint32_t frame, void *stream)
{
    gi_status s;
    if (!pp || !out) return GI_ERR_NULL;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if ((s = check_probes(in)) != GI_OK) return s;
    if ((s = check_probes(out)) != GI_OK) return s;
    for (int a = 0; a < 3; ++a)
        if (in->dims[a] != out->dims[a]) return GI_ERR_SHAPE;
    if (in->texel != out->texel) return GI_ERR_PARAM;
    const void *ii = in->irr, *id = in->dep, *oi = out->irr, *od = out->dep;
    if (ii == oi || id == od || ii == od || id == oi) return GI_ERR_ALIAS;
    if (pp->rays < 1 || pp->rays > GI_MAX_PROBE_RAYS) return GI_ERR_PARAM;
    if (!(pp->hysteresis >= 0.0f && pp->hysteresis <= 1.0f) || !(pp->sharpness > 0.0f)) return GI_ERR_PARAM;
    if (!(pp->distance_slider >= 0.0f)) return GI_ERR_PARAM;
    uint32_t P = in->dims[0] * in->dims[1] * in->dims[2];
    uint32_t lds = scene_lds(scene, 32u * pp->rays + (uint32_t)sizeof(float) * (64u * 3u + 256u * 2u));
    const bool glossy = glossy_scene(scene), f16 = in->texel == GI_TEXEL_F16;
    const dim3 grid(P);
#define GI_PU(L, G, H) k_probe_update<L, G, H><<<grid, kProbeBlock, lds + 32u * pp->rays, S(stream)>>>(*scene, *in, *out, *pp, seed, frame, lds)
    if (lds) {
        if (glossy) { if (f16) GI_PU(true, true, true); else GI_PU(true, true, false); }
        else { if (f16) GI_PU(true, false, true); else GI_PU(true, false, false); }
    } else {
        if (glossy) { if (f16) GI_PU(false, true, true); else GI_PU(false, true, false); }
        else { if (f16) GI_PU(false, false, true); else GI_PU(false, false, false); }
    }
#undef GI_PU
    return launched();
}

gi_status gi_probe_query(const gi_probes *probes, uint32_t n, const float *p, const float *nrm, float *out,
                         void *stream)
{
    gi_status s;
    if ((s = check_probes(probes)) != GI_OK) return s;
    if (n == 0) return GI_OK;
    if (!p || !nrm || !out) return GI_ERR_NULL;
    k_probe_query<<<(n + 255) / 256, 256, 0, S(stream)>>>(*probes, n, p, nrm, out);
    return launched();
}

gi_status gi_resample_initial(const gi_scene *scene, const gi_gbuffer *gb, const gi_probes *probes,
                              const gi_params *params, gi_reservoirs *out, float *resid, uint64_t seed,
                              uint32_t frame, void *stream)
{
    gi_status s;
    if (!gb || !out || !resid) return GI_ERR_NULL;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if ((s = check_gb(gb, gb->width, gb->height)) != GI_OK) return s;
    if ((s = check_probes(probes)) != GI_OK) return s;
    if ((s = check_params(params)) != GI_OK) return s;
    if ((s = check_res(out, gb->width, gb->height)) != GI_OK) return s;
    if ((uint64_t)gb->width * gb->height > (1u << 23)) return GI_ERR_SHAPE;   // 23-bit tag origin
    if (gb->width == 0 || gb->height == 0) return GI_OK;
    launch_initial_probe(scene, *gb, *probes, *params, *out, reinterpret_cast<float4 *>(resid), seed, frame, CandWs{},
                         gi_mlp{}, S(stream));
    return launched();
}

gi_status gi_resample_temporal(const gi_scene *scene, const gi_gbuffer *gb, const gi_gbuffer *gb_prev,
                               const gi_camera *prev_cam, const gi_reservoirs *cur_in,
                               const gi_reservoirs *history, const gi_params *params, gi_reservoirs *out,
                               uint64_t seed, uint32_t frame, void *stream)
{
    gi_status s;
    if (!gb || !gb_prev || !prev_cam || !cur_in || !history || !out) return GI_ERR_NULL;
    uint32_t W = gb->width, H = gb->height;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if ((s = check_gb(gb, W, H)) != GI_OK) return s;
    if ((s = check_gb(gb_prev, W, H)) != GI_OK) return s;
    if (prev_cam->width != W || prev_cam->height != H) return GI_ERR_SHAPE;
    if ((s = check_params(params)) != GI_OK) return s;
    if ((s = check_res(cur_in, W, H)) != GI_OK) return s;
    if ((s = check_res(history, W, H)) != GI_OK) return s;
    if ((s = check_res(out, W, H)) != GI_OK) return s;
    if (res_alias(out, cur_in) || res_alias(out, history)) return GI_ERR_ALIAS;
    if (W == 0 || H == 0) return GI_OK;
    // the history's M is capped at a multiple of the candidates a drawing pixel
    // takes per frame, so pixels that drew none this frame (candidate
    // subsampling, Sec. 6) still take over their history
    const double capd = floor((double)params->m_cap * (double)(params->M + params->M_light));
    const uint32_t m_hist_cap = capd >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)capd;
    // few pixels, where the spatial pass takes small tiles too (Lambertian
    // scenes: the glossy target has no form of its own there)
    if ((uint64_t)W * H <= kSmallImage && !glossy_scene(scene)) {
        const uint32_t lds = scene_lds(scene);
        GI_LAUNCH_LDS(k_temporal_small, dim3(((W + 7u) / 8u) * ((H + 7u) / 8u)), 128, lds, S(stream), *scene, *gb, *gb_prev,
                      *prev_cam, *cur_in, *history, *params, m_hist_cap, *out, seed, frame);
        return launched();
    }
    const SceneTiles st(scene);
#define GI_TP(L, G, SW)                                                                                        \
    k_temporal<L, G, SW><<<tile_grid(W, H, SW), SW * kTile, st.lds, S(stream)>>>(*scene, *gb, *gb_prev, *prev_cam, *cur_in, \
                                                                                    *history, *params, m_hist_cap, *out, seed, frame)
    if (glossy_scene(scene)) {
        if (st.lds) GI_TP(true, true, 16u); else GI_TP(false, true, 16u);
    } else {
        if (st.wide) GI_TP(true, false, 48u); else if (st.lds) GI_TP(true, false, 16u); else GI_TP(false, false, 16u);
    }
#undef GI_TP
    return launched();
}

gi_status gi_resample_spatial(const gi_scene *scene, const gi_gbuffer *gb, const gi_reservoirs *in,
                              const gi_params *params, uint32_t pass, gi_reservoirs *out, uint64_t seed,
                              uint32_t frame, void *stream)
{
    gi_status s;
    if (!gb || !in || !out) return GI_ERR_NULL;
    uint32_t W = gb->width, H = gb->height;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if ((s = check_gb(gb, W, H)) != GI_OK) return s;
    if ((s = check_params(params)) != GI_OK) return s;
    if ((s = check_res(in, W, H)) != GI_OK) return s;
    if ((s = check_res(out, W, H)) != GI_OK) return s;
    if (res_alias(out, in)) return GI_ERR_ALIAS;
    if (pass > 5) return GI_ERR_PARAM;
    if (W == 0 || H == 0) return GI_OK;
    // neighbour slots: 5 (the workloads' k) or GI_MAX_K
    if (params->k <= 5u)
        launch_spatial<5>(scene, W, H, S(stream), *scene, *gb, *in, *params, pass, *out, seed, frame);
    else
        launch_spatial<(int)GI_MAX_K>(scene, W, H, S(stream), *scene, *gb, *in, *params, pass, *out, seed,
                                      frame);
    return launched();
}

gi_status gi_shade(const gi_scene *scene, const gi_gbuffer *gb, const gi_probes *probes, const gi_reservoirs *res,
                   const float *resid, const gi_params *params, float *out_rgba, uint64_t seed, uint32_t frame,
                   void *stream)
{
    gi_status s;
    if (!gb || !res || !resid || !out_rgba) return GI_ERR_NULL;
    uint32_t W = gb->width, H = gb->height;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if ((s = check_gb(gb, W, H)) != GI_OK) return s;
    if ((s = check_probes(probes)) != GI_OK) return s;
    if ((s = check_params(params)) != GI_OK) return s;
    if ((s = check_res(res, W, H)) != GI_OK) return s;
    const bool glossy = glossy_scene(scene);
    if (glossy && (!(params->foot_c >= 0.0f) || params->glossy_depth < 1u || params->glossy_depth > GI_MAX_GLOSSY_DEPTH))
        return GI_ERR_PARAM;
    if (W == 0 || H == 0) return GI_OK;
    const SceneTiles st(scene);
    const float4 *rs = reinterpret_cast<const float4 *>(resid);
    float4 *img = reinterpret_cast<float4 *>(out_rgba);
    const bool f16 = probes->texel == GI_TEXEL_F16;
#define GI_SH(L, G, T, SW)                                                                                     \
    k_shade<L, false, G, T, SW><<<tile_grid(W, H, SW), SW * kTile, st.lds, S(stream)>>>(                    \
        *scene, *gb, *probes, *res, rs, *params, img, nullptr, gi_mlp{}, seed, frame)
    if (glossy) {
        if (st.lds) { if (f16) GI_SH(true, true, kTexF16, 16u); else GI_SH(true, true, kTexF32, 16u); }
        else { if (f16) GI_SH(false, true, kTexF16, 16u); else GI_SH(false, true, kTexF32, 16u); }
    } else if (st.wide) {
        if (f16) GI_SH(true, false, kTexF16, 48u); else GI_SH(true, false, kTexF32, 48u);
    } else {
        if (st.lds) { if (f16) GI_SH(true, false, kTexF16, 16u); else GI_SH(true, false, kTexF32, 16u); }
        else { if (f16) GI_SH(false, false, kTexF16, 16u); else GI_SH(false, false, kTexF32, 16u); }
    }
#undef GI_SH
    return launched();
}

gi_status gi_mlp_make_batch(const gi_scene *scene, const gi_gbuffer *gb, const gi_probes *probes, uint32_t M,
                            uint32_t n, uint64_t seed, uint32_t frame, float *pos4, float *nrm4, float *target4,
                            float *qprobe4, void *stream)
{
    gi_status s;
    if (!gb) return GI_ERR_NULL;
    uint32_t W = gb->width, H = gb->height;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if (glossy_scene(scene)) return GI_ERR_PARAM;   // the learned cache serves Lambertian scenes
    if ((s = check_gb(gb, W, H)) != GI_OK) return s;
    if ((s = check_probes(probes)) != GI_OK) return s;
    if (M < 1 || M > GI_MAX_M) return GI_ERR_PARAM;
    if (n > GI_MLP_MAX_BATCH) return GI_ERR_SHAPE;
    if (n == 0) return GI_OK;
    if (!pos4 || !nrm4 || !target4 || !qprobe4) return GI_ERR_NULL;
    if (W == 0 || H == 0) return GI_ERR_SHAPE;
    GI_LAUNCH_LDS(k_mlp_batch, (n + kBlock - 1) / kBlock, kBlock, scene_lds(scene), S(stream), *scene, *gb, *probes,
                  M, n, seed, frame, reinterpret_cast<float4 *>(pos4), reinterpret_cast<float4 *>(nrm4),
                  reinterpret_cast<float4 *>(target4), reinterpret_cast<float4 *>(qprobe4));
    return launched();
}

uint64_t gi_initial_mlp_workspace_bytes(uint32_t width, uint32_t height, uint32_t M)
{
    return 48ull * width * height * M;
}

gi_status gi_resample_initial_mlp(const gi_scene *scene, const gi_gbuffer *gb, const gi_probes *probes,
                                  const gi_mlp *mlp, const gi_params *params, gi_reservoirs *out, float *resid,
                                  void *workspace, uint64_t workspace_bytes, uint64_t seed, uint32_t frame,
                                  void *stream)
{
    gi_status s;
    if (!gb || !out || !resid || !workspace) return GI_ERR_NULL;
    uint32_t W = gb->width, H = gb->height;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if (glossy_scene(scene)) return GI_ERR_PARAM;   // the learned cache serves Lambertian scenes
    if ((s = check_gb(gb, W, H)) != GI_OK) return s;
    if ((s = check_probes(probes)) != GI_OK) return s;
    if ((s = check_mlp(mlp)) != GI_OK) return s;
    if ((s = check_params(params)) != GI_OK) return s;
    if ((s = check_res(out, W, H)) != GI_OK) return s;
    if ((uint64_t)W * H > (1u << 23)) return GI_ERR_SHAPE;   // 23-bit tag origin
    const uint64_t ncand = (uint64_t)W * H * params->M;
    if (ncand >= (1ull << 31)) return GI_ERR_SHAPE;
    if (workspace_bytes < gi_initial_mlp_workspace_bytes(W, H, params->M)) return GI_ERR_SHAPE;
    if (W == 0 || H == 0) return GI_OK;
    float4 *base = reinterpret_cast<float4 *>(workspace);
    // NEVER: the probe form alone.  ALWAYS: the cache form (candidates traced
    // into the workspace, the cache evaluated on all of them, resampling with
    // the cached values).  AUTO: both, each gated on the device's usability
    // word, so that a frame the cache is not used in costs the probe form
    // (bit-identical to gi_resample_initial) and not the cache form's trace.
    if (mlp->mode != GI_MLP_NEVER) {
        const uint32_t gate = mlp->mode == GI_MLP_AUTO ? kRunIfCache : kRunAlways;
        CandWs ws{base, base + ncand, base + 2 * ncand, gate};
        launch_cand(scene, *gb, *params, ws, seed, frame, *mlp, S(stream));
        if ((s = launched()) != GI_OK) return s;
        if ((s = mlp_infer_launch(*mlp, (uint32_t)ncand, ws.pos, ws.nrm, ws.q, true, S(stream))) != GI_OK) return s;
        launch_initial<true>(params->M_light > 0, false, probes->texel == GI_TEXEL_F16, 0u, tile_grid(W, H), S(stream), *scene, *gb, *probes,
                             *params, *out, reinterpret_cast<float4 *>(resid), seed, frame, ws, *mlp);
        if ((s = launched()) != GI_OK) return s;
    }
    if (mlp->mode != GI_MLP_ALWAYS) {
        const uint32_t gate = mlp->mode == GI_MLP_AUTO ? kRunIfProbe : kRunAlways;
        launch_initial_probe(scene, *gb, *probes, *params, *out, reinterpret_cast<float4 *>(resid), seed, frame,
                             CandWs{nullptr, nullptr, nullptr, gate}, *mlp, S(stream));
    }
    return launched();
}

uint64_t gi_shade_mlp_workspace_bytes(uint32_t width, uint32_t height) { return 16ull * width * height; }

gi_status gi_shade_mlp(const gi_scene *scene, const gi_gbuffer *gb, const gi_probes *probes, const gi_mlp *mlp,
                       const gi_reservoirs *res, const float *resid, const gi_params *params, float *out_rgba,
                       void *workspace, uint64_t workspace_bytes, void *stream)
{
    gi_status s;
    if (!gb || !res || !resid || !out_rgba || !workspace) return GI_ERR_NULL;
    uint32_t W = gb->width, H = gb->height;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if (glossy_scene(scene)) return GI_ERR_PARAM;   // the learned cache serves Lambertian scenes
    if ((s = check_gb(gb, W, H)) != GI_OK) return s;
    if ((s = check_probes(probes)) != GI_OK) return s;
    if ((s = check_mlp(mlp)) != GI_OK) return s;
    if ((s = check_params(params)) != GI_OK) return s;
    if ((s = check_res(res, W, H)) != GI_OK) return s;
    if (workspace_bytes < gi_shade_mlp_workspace_bytes(W, H)) return GI_ERR_SHAPE;
    if (W == 0 || H == 0) return GI_OK;
    float4 *q = reinterpret_cast<float4 *>(workspace);
    if ((s = mlp_infer_launch(*mlp, W * H, reinterpret_cast<const float4 *>(res->y_W),
                              reinterpret_cast<const float4 *>(res->n_wsum), q, true, S(stream))) != GI_OK)
        return s;
    {
        const SceneTiles st(scene);
        const float4 *rs = reinterpret_cast<const float4 *>(resid);
        float4 *img = reinterpret_cast<float4 *>(out_rgba);
#define GI_SH(L, SW)                                                                                   \
    k_shade<L, true, false, kTexAny, SW><<<tile_grid(W, H, SW), SW * kTile, st.lds, S(stream)>>>(      \
        *scene, *gb, *probes, *res, rs, *params, img, q, *mlp, 0ull, 0u)
        if (st.wide) GI_SH(true, 48u);
        else if (st.lds) GI_SH(true, 16u);
        else GI_SH(false, 16u);
#undef GI_SH
    }
    return launched();
}

gi_status gi_path_trace(const gi_scene *scene, const gi_gbuffer *gb, uint32_t spp, uint32_t sample0, uint64_t seed,
                        float *out_rgba, void *stream)
{
    gi_status s;
    if (!gb || !out_rgba) return GI_ERR_NULL;
    uint32_t W = gb->width, H = gb->height;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if ((s = check_gb(gb, W, H)) != GI_OK) return s;
    if (spp < 1 || spp > 65536) return GI_ERR_PARAM;
    if (W == 0 || H == 0) return GI_OK;
    GI_LAUNCH_LDS_G(k_path_trace, glossy_scene(scene), tile_grid(W, H), kBlock, scene_lds(scene), S(stream), *scene,
                    *gb, spp, sample0, seed,
                  reinterpret_cast<float4 *>(out_rgba));
    return launched();
}

gi_status gi_philox(uint64_t seed, uint32_t n, const uint32_t *ctr, uint32_t *out, void *stream)
{
    if (n == 0) return GI_OK;
    if (!ctr || !out) return GI_ERR_NULL;
    k_philox<<<(n + 255) / 256, 256, 0, S(stream)>>>(seed, n, reinterpret_cast<const uint4 *>(ctr),
                                                    reinterpret_cast<uint4 *>(out));
    return launched();
}

gi_status gi_trace_rays(const gi_scene *scene, uint32_t n, const float *org, const float *dir, float *out,
                        uint32_t *prim, void *stream)
{
    gi_status s;
    if ((s = check_scene(scene)) != GI_OK) return s;
    if (n == 0) return GI_OK;
    if (!org || !dir || !out || !prim) return GI_ERR_NULL;
    k_trace<<<(n + 255) / 256, 256, 0, S(stream)>>>(*scene, n, org, dir, reinterpret_cast<float4 *>(out), prim);
    return launched();
}

}  // extern "C"
